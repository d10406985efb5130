// Distance stage for query batches: d(q, k) = ||q||^2 - 2 q.k + ||k||^2, the
// squared L2 distance whose negative is the paper's similarity (Section 2.2),
// with the q.k term on the gfx950 matrix cores.
//
// When many queries share one key set (speculative verification scores every
// draft position of a sequence against that sequence's store), the dot
// products form a dense [queries x d] . [d x keys] contraction: every key
// element is used by up to 128 queries, so streaming the keys from HBM once
// needs up to 128 flop per byte -- beyond the vector ALUs, within the
// matrix cores.  A workgroup takes passes of PK keys of one set against up to
// 128 of the set's queries (MQ blocks of 16), walking d in steps of SPAN
// elements.
//
// Bound: HBM.  Each step's keys and queries go straight from HBM (L2 for the
// queries) to LDS -- 16 bytes a lane, whole 128- or 256-byte pieces of a row,
// no registers in between -- into a ring of NB span buffers, NB - 1 steps
// ahead, and one barrier a step orders the buffers.  With the spans staged
// through registers (two LDS buffers, two to four register sets) a 35-query
// workgroup ran one wave per SIMD, 98 KiB of LDS and 1.9 us a step; 48 to 72 KiB and
// 60 to 130 registers let two or three workgroups of up to 64 queries share a
// CU.  Measured, before and after, bf16 keys of d = 4096: 8 x 65,536 keys, 16 / 32
// / 64 queries 792 / 915 / 1,080 us and 746 / 804 / 905 us (5.75 / 5.35 / 4.75
// TB/s); 128 queries on 4 x 65,536 keys of d = 2048: 304 and 295 us.  What is left
// is the access pattern: 128 bytes of each row at a time stream below the
// whole-row kernels' 7 TB/s.
//
// The LDS copy is swizzled -- chunk c (16 bytes) of row n sits at slot n * CH +
// (c ^ (n % CH)), CH the chunks of a row's span -- so that the fragment reads
// (lane l reads row l % 16, chunk 4 * step + l / 16) touch every bank once; the
// loads' lanes pick their chunks accordingly.  In MFMA step c lane l holds key
// (or query) row l % 16 and elements 32c + 8 (l / 16) .. +8 of the span -- the
// same elements for both operands, so the contraction is exact up to fp32
// rounding -- for v_mfma_f32_16x16x32 (bf16 or f16, fp32 accumulate).  The
// steps run in the same k order whatever the variant, so the sums are the
// same.  Rows past the data read the tile's last row, and steps past the tile's
// end read on in its last pass's rows.
#include "knnlm_internal.h"
#include "mfma_device.h"
#include "tile_rows.h"

namespace knnlm {

namespace {

constexpr int kTileQuantum = 128;  // tile rows: a multiple of the largest pass, or 64 or 32

// Where the epilogue stores the (discarded) distances of rows past the tile or
// query slots past the group: one word per device, written, never read.
__device__ float g_mfma_sink;

constexpr int kSpan = kMfmaSpan;    // d is a multiple of this

// MQ: 16-query blocks per workgroup; WK x WQ waves: WK groups split the
// pass's PK / 16 key blocks, WQ groups split the query blocks (MQ / WQ each);
// NB: span buffers (NB - 1 spans in flight); NORMS: ||k||^2 comes precomputed;
// PK keys per pass and SPAN elements of d per pipeline step.
//
// FM (the fused select of query batches on long rows): 0 every tile, the
// distances written; 1 only the sample pieces (the first sample_rows rows of
// every sample_every-th tile), the distances written; 2 every row outside the
// sample pieces, and instead of the distances each query's candidates -- keys
// whose distance bits are below the query's threshold -- are staged in LDS
// and appended to the query's list once the tile is done (the list's count is
// true even past its capacity; a full LDS stage sets the fallback word).
template <knn_dtype DT, int MQ, int WK, int WQ, int NB, bool NORMS, int PK, int SPAN, int FM = 0>
__global__ __launch_bounds__(WK * WQ * kWave, 2) void k_dist_mfma(DistArgs a, int64_t n_tiles, int64_t groups) {
    constexpr int QW = WQ;
    constexpr int kChunks = SPAN * 2 / 16;          // 16-byte chunks per row and step
    constexpr int KSTEPS = SPAN / 32;               // MFMA steps per span
    constexpr int KBW = PK / 16 / WK;                    // key blocks per wave
    constexpr int NW = WK * WQ;
    constexpr int kThreads = NW * kWave;
    constexpr int QB = MQ * 16;
    constexpr int MQW = MQ / QW;                         // query blocks per wave
    constexpr int kRowsPerLoad = kWave / kChunks;        // rows a wave's load covers
    constexpr int KLD = (PK / kRowsPerLoad + NW - 1) / NW;   // key loads per wave and step
    constexpr int QLD = (QB / kRowsPerLoad + NW - 1) / NW;   // query loads per wave and step
    static_assert(MQ % QW == 0 && (PK / 16) % WK == 0, "whole blocks per wave");
    static_assert(SPAN % 32 == 0 && kSpan % SPAN == 0 && kChunks <= 16, "whole MFMA steps, spans dividing d");
    // native 4 x u32 vectors throughout, so that every 16-byte LDS access is
    // one ds_read_b128 (a struct is split by the compiler)
    __shared__ __align__(16) u32x4_t klds[NB][PK * kChunks];
    __shared__ __align__(16) u32x4_t qlds[NB][QB * kChunks];
    __shared__ uint32_t smin[QB], smax[QB];
    constexpr int kStage = FM == 2 ? 1024 : 1;  // candidates staged per tile (about 120 at 128 x 4096 keys)
    __shared__ uint64_t stage_key[kStage];
    __shared__ uint8_t stage_q[kStage];
    __shared__ uint32_t stage_n;
    static_assert(FM != 2 || QB <= 256, "a staged query fits a byte");

    if constexpr (FM == 0) {
        if (a.gate != nullptr && *a.gate != a.gate_run) return;
    }
    // Consecutive workgroups land on different XCDs (round robin over 8).  The
    // query groups of one key tile are numbered 8 apart, so they run on one XCD
    // at about the same time and all but the first read the tile from its L2.
    const int64_t L = blockIdx.x;
    const int64_t grp = (L >> 3) % groups;
    const int64_t tl = ((L >> 3) / groups) * 8 + (L & 7);
    if (tl >= n_tiles) return;
    const int64_t tiles = a.tiles_per_set;
    const int64_t se = FM == 0 ? 1 : a.sample_every;
    const int64_t per_set = FM == 1 ? (tiles + se - 1) / se : tiles;  // tiles (sample pieces) per set
    const int64_t s = tl / per_set;
    const int64_t tile = FM == 1 ? (tl - s * per_set) * se : tl - s * per_set;
    const int64_t k0 = a.key_offsets[s];
    int64_t N = a.key_offsets[s + 1] - k0;
    if (N > a.ld) N = a.ld;
    const int64_t qb = a.query_offsets[s] + grp * QB;
    const int64_t qe = a.query_offsets[s + 1];
    // this workgroup's rows [r0, r1): the tile, its sample piece (FM 1), or the
    // tile past its piece (FM 2).  None past the set's end, and none where the
    // piece is the whole tile: the loads below need a row to read.
    const RowRange rows = mfma_rows(FM, tile, a.rows_per_tile, a.sample_rows, se, N);
    const int64_t r0 = rows.first, r1 = rows.end;
    if (qb >= qe || r0 >= r1) return;  // uniform over the block
    const int nq = static_cast<int>(qe - qb < QB ? qe - qb : QB);

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wid = __builtin_amdgcn_readfirstlane(tid / kWave);
    const int wave = wid / QW;        // this wave's group of key blocks
    const int jq = (wid % QW) * MQW;  // its first query block
    const int g = lane >> 4, lr = lane & 15;
    const int64_t row_bytes = a.d * 2;
    const int64_t nspan = a.d / SPAN;
    const int64_t npass = (r1 - r0 + PK - 1) / PK;
    const int64_t T = npass * nspan;  // pipeline steps of this tile
    const char *qbase = static_cast<const char *>(a.queries) + qb * row_bytes;
    const char *kset = static_cast<const char *>(a.keys) + k0 * row_bytes;

    for (int q = tid; q < QB; q += kThreads) {
        smin[q] = 0xffffffffu;
        smax[q] = 0u;
    }
    if (FM == 2 && tid == 0) stage_n = 0u;
    // FM 2: the thresholds of this lane's query rows (jq + j) * 16 + lr (0 past the group: nothing passes)
    uint32_t thr_l[MQW];
#pragma unroll
    for (int j = 0; j < MQW; ++j) {
        const int q = (jq + j) * 16 + lr;
        thr_l[j] = (FM == 2 && q < nq) ? a.cand_thr[qb + q] : 0u;
    }

    // Loads: a wave's load fills 64 consecutive slots (kRowsPerLoad rows) of a
    // buffer, each lane with the chunk that the swizzle puts into its slot.
    // Loads past the pass's (query block's) rows repeat its last.
    // Addresses: a uniform base per step plus a 32-bit offset per load (a tile
    // is at most 4096 rows of at most 128 KiB).
    const int lrow = lane / kChunks;
    auto lcol = [&](int row) __attribute__((always_inline)) {
        return static_cast<uint32_t>((lane ^ row) & (kChunks - 1)) * 16u;
    };
    const uint32_t nrows = static_cast<uint32_t>(r1 - r0);
    const uint32_t rb = static_cast<uint32_t>(row_bytes);
    const uint32_t ns = static_cast<uint32_t>(nspan);  // steps fit 32 bits: at most 128 passes of 1024 spans
    const uint32_t kat = lds_offset(&klds[0][0]), qat = lds_offset(&qlds[0][0]);
    uint32_t qoff[QLD], qslot[QLD], koff[KLD], kslot[KLD];
#pragma unroll
    for (int i = 0; i < QLD; ++i) {
        const int k = min(wid * QLD + i, QB / kRowsPerLoad - 1);
        const int row = k * kRowsPerLoad + lrow;
        qoff[i] = static_cast<uint32_t>(row < nq ? row : 0) * rb + lcol(row);
        qslot[i] = qat + static_cast<uint32_t>(k) * 1024u;
    }
#pragma unroll
    for (int i = 0; i < KLD; ++i) kslot[i] = kat + static_cast<uint32_t>(min(wid * KLD + i, PK / kRowsPerLoad - 1)) * 1024u;
    // the rows of pass p (those past the end read the tile's last row)
    auto set_pass = [&](uint32_t p) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < KLD; ++i) {
            const int k = min(wid * KLD + i, PK / kRowsPerLoad - 1);
            const int row = k * kRowsPerLoad + lrow;
            koff[i] = mfma_load_row(p * PK + static_cast<uint32_t>(row), nrows) * rb + lcol(row);
        }
    };
    const char *kspan = kset + r0 * row_bytes, *qspan = qbase;  // the next step to load: its span of the rows
    uint32_t lsp = 0u, lpass = 0u;
    set_pass(0u);
    auto load = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < KLD; ++i) load_to_lds_16_nt(kspan, koff[i], kslot[i] + static_cast<uint32_t>(buf * PK * kChunks * 16));
#pragma unroll
        for (int i = 0; i < QLD; ++i) load_to_lds_16(qspan, qoff[i], qslot[i] + static_cast<uint32_t>(buf * QB * kChunks * 16));
        kspan += 2 * SPAN;
        qspan += 2 * SPAN;
        if (++lsp == ns) {  // the next pass (past the last one: its rows again)
            lsp = 0u;
            kspan -= row_bytes;
            qspan -= row_bytes;
            set_pass(++lpass);
        }
    };

    f32x4_t acc[MQW][KBW];
    float kkp[KBW], qqp[MQW];
#pragma unroll
    for (int j = 0; j < MQW; ++j) qqp[j] = 0.0f;  // ||q||^2 partials: the first pass adds them up, later passes reuse them
    auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < MQW; ++j)
#pragma unroll
            for (int kb = 0; kb < KBW; ++kb) acc[j][kb] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int kb = 0; kb < KBW; ++kb) kkp[kb] = 0.0f;
    };
    clear();

    // The matrix cores over one span in LDS buffer buf (with qn_pass, also
    // the query norms).
    auto compute = [&](int buf, bool qn_pass) __attribute__((always_inline)) {
#pragma unroll
        for (int c = 0; c < KSTEPS; ++c) {
            const int ch = (4 * c + g) ^ (lr & (kChunks - 1));
            u32x4_t bk[KBW], af[MQW];
#pragma unroll
            for (int kb = 0; kb < KBW; ++kb) bk[kb] = klds[buf][((wave * KBW + kb) * 16 + lr) * kChunks + ch];
#pragma unroll
            for (int j = 0; j < MQW; ++j) af[j] = qlds[buf][((jq + j) * 16 + lr) * kChunks + ch];
#pragma unroll
            for (int j = 0; j < MQW; ++j)
#pragma unroll
                for (int kb = 0; kb < KBW; ++kb) acc[j][kb] = mfma16<DT>(af[j], bk[kb], acc[j][kb]);
            if constexpr (!NORMS) {
#pragma unroll
                for (int kb = 0; kb < KBW; ++kb) kkp[kb] = dot_vec<DT>(bk[kb], kkp[kb]);
            }
            if (qn_pass) {
#pragma unroll
                for (int j = 0; j < MQW; ++j) qqp[j] = dot_vec<DT>(af[j], qqp[j]);
            }
        }
    };

    // Distances of pass p: lane (g, lr) holds dot(query (jq + j)*16 + 4g + i,
    // key c0 + (wave*KBW + kb)*16 + lr) in acc[j][kb][i].
    auto epilogue = [&](int64_t p) __attribute__((always_inline)) {
        const int64_t c0 = r0 + p * PK;
        float kk[KBW];
        bool mk[KBW];  // masked key rows (Section 3.4): distance +infinity, no part in the extrema
#pragma unroll
        for (int kb = 0; kb < KBW; ++kb) {
            const int64_t row = c0 + (wave * KBW + kb) * 16 + lr;
            kk[kb] = NORMS ? (row < r1 ? a.key_sqnorms[k0 + row] : 0.0f) : group4_sum(kkp[kb]);
            mk[kb] = a.key_mask != nullptr && row < r1 && key_masked(a.key_mask, k0 + row);
        }
        if constexpr (FM == 2) {
            // candidates: distance bits below the query's threshold, appended to
            // the LDS stage a wave at a time (one LDS atomic per wave that has any)
#pragma unroll
            for (int j = 0; j < MQW; ++j) {
                const float qsum = group4_sum(qqp[j]);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int q = (jq + j) * 16 + g * 4 + i;
                    const float qn = __shfl(qsum, g * 4 + i);
                    const uint32_t th = __shfl(thr_l[j], g * 4 + i);
#pragma unroll
                    for (int kb = 0; kb < KBW; ++kb) {
                        const int64_t row = c0 + (wave * KBW + kb) * 16 + lr;
                        const float dist = mk[kb] ? __uint_as_float(kMaskedBits)
                                                  : clamp_nonneg(fmaf(-2.0f, acc[j][kb][i], qn + kk[kb]));
                        const bool c = q < nq && row < r1 && __float_as_uint(dist) < th;
                        const uint64_t bal = __ballot(c);
                        if (bal != 0ull) {
                            const int first = __ffsll(static_cast<unsigned long long>(bal)) - 1;
                            uint32_t base = 0u;
                            if (lane == first) base = atomicAdd(&stage_n, static_cast<uint32_t>(__popcll(bal)));
                            base = readlane_u32(base, first);
                            if (c) {
                                const uint32_t p = base + static_cast<uint32_t>(
                                                              __popcll(bal & ((1ull << lane) - 1ull)));
                                if (p < static_cast<uint32_t>(kStage)) {
                                    stage_key[p] = (static_cast<uint64_t>(__float_as_uint(dist)) << 32) |
                                                   static_cast<uint32_t>(row);
                                    stage_q[p] = static_cast<uint8_t>(q);
                                }
                            }
                        }
                    }
                }
            }
            clear();
            return;
        }
        // the pass's extrema of each query fold into the tile's (LDS atomics) here,
        // so that no per-lane extrema stay live through the main loop
#pragma unroll
        for (int j = 0; j < MQW; ++j) {
            const float qsum = group4_sum(qqp[j]);  // ||q||^2 of query (jq + j)*16 + lr
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int q = (jq + j) * 16 + g * 4 + i;
                const float qn = __shfl(qsum, g * 4 + i);
                float tmn = __builtin_huge_valf(), tmx = 0.0f;
#pragma unroll
                for (int kb = 0; kb < KBW; ++kb) {
                    const int64_t row = c0 + (wave * KBW + kb) * 16 + lr;
                    const float dist = mk[kb] ? __uint_as_float(kMaskedBits)
                                              : clamp_nonneg(fmaf(-2.0f, acc[j][kb][i], qn + kk[kb]));
                    const bool ok = q < nq && row < r1;
                    // no branch around the store (nor any other memory operation in the loop)
                    *(ok ? a.dist + (qb + q) * a.ld + row : &g_mfma_sink) = dist;
                    tmn = ok && !mk[kb] ? fminf(tmn, dist) : tmn;
                    tmx = ok && !mk[kb] ? fmaxf(tmx, dist) : tmx;
                }
                tmn = row16_min(tmn);
                tmx = row16_max(tmx);
                if (lr == 0 && q < nq) {
                    atomicMin(&smin[q], __float_as_uint(tmn));
                    atomicMax(&smax[q], __float_as_uint(tmx));
                }
            }
        }
        clear();
    };

    // Step t: once span t is in LDS for every wave (a wave waits for its own
    // loads of it -- those of the NB - 2 newer steps may still be in flight --
    // and the barrier for the others'), span t + NB - 1 starts loading into the
    // buffer that step t - 1 has been read from, and the matrix cores take
    // span t.  Every step issues the same loads (steps past the tile's last
    // one load too), so the count in the wait is exact; other memory operations
    // only make it wait longer.  The step count is padded to a multiple of NB
    // with steps whose products are never stored.
#pragma unroll
    for (int k = 0; k < NB - 1; ++k) load(k);
    uint32_t sp = 0u, pass = 0u;
    for (int64_t t = 0; t < T; t += NB) {
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            // (and every LDS access of the steps before is done)
            __builtin_amdgcn_s_waitcnt(vmcnt_encoding<(NB - 2) * (KLD + QLD)>() & ~kLgkmcntAny);
            // a bare barrier: a fenced one would wait for every load in flight
            asm volatile("" ::: "memory");
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
            load((k + NB - 1) % NB);
            compute(k, pass == 0u);
            if (++sp == ns) {  // (padding steps may end a pass past the last)
                sp = 0u;
                if (pass < static_cast<uint32_t>(npass)) epilogue(pass);
                ++pass;
            }
        }
    }
    __builtin_amdgcn_s_waitcnt(kVmcntZero);  // no load may land in LDS after the workgroup's end

    if constexpr (FM == 2) {
        // the staged candidates to their queries' lists (no loads are in flight any more)
        __syncthreads();
        const uint32_t n = stage_n;
        if (n > static_cast<uint32_t>(kStage) && tid == 0) *a.fallback = 1u;
        const uint32_t m = n < static_cast<uint32_t>(kStage) ? n : static_cast<uint32_t>(kStage);
        for (uint32_t e = tid; e < m; e += kThreads) {
            const int64_t qq = qb + stage_q[e];
            const uint32_t pos = atomicAdd(a.cand_count + qq, 1u);
            if (pos < static_cast<uint32_t>(kFusedCap)) a.cand_list[qq * kFusedCap + pos] = stage_key[e];
        }
        return;
    }
    // the tile's extrema of each query (folded in by every pass's epilogue)
    if (a.tile_min != nullptr) {
        __syncthreads();
        for (int q = tid; q < nq; q += kThreads) {
            a.tile_min[(qb + q) * tiles + tile] = __uint_as_float(smin[q]);
            a.tile_max[(qb + q) * tiles + tile] = __uint_as_float(smax[q]);
        }
    }
}

// The variants: waves, keys per pass, elements per step and span buffers for
// each group size, for tiles of 32, of 64 and of more rows (one pass a tile for
// the small ones; then more of d per step, since a step's latency and not its
// bytes is what takes the time).  Measured on bf16 keys of d = 4096, 8 x 65,536
// keys: 16 queries 746 us (64-key passes of 128 elements 765 us), 32 queries
// 804 us (64 keys, 4 buffers: 815 us), 64 queries 905 us (64 keys, 4 buffers: 955 us).
// 128-query groups on tiles of whole 256-row passes take those: a pass stages
// the 128 query rows anew, so half as many passes load a quarter less.  256- and
// 128-key passes (four buffers), f16: 8.4 M keys of d = 1024, fused, 3.81 and 4.19
// ms (2 x 4 wave groups, which read more of LDS, 4.01 ms); 2 x 262,144 keys of d =
// 4096 0.99 and 1.06 ms; 100 queries on each of 50 sets of 20,000 keys of d = 128,
// whose passes have two steps, 199 and 203 us.
template <knn_dtype DT, int MQ, int WK, int WQ, int NB, bool NORMS, int PK, int SPAN, int FM = 0>
hipError_t launch_one(const DistArgs &a, int64_t n_tiles, int64_t groups, dim3 grid, hipStream_t st) {
    hipLaunchKernelGGL((k_dist_mfma<DT, MQ, WK, WQ, NB, NORMS, PK, SPAN, FM>), grid, dim3(WK * WQ * kWave), 0, st, a,
                       n_tiles, groups);
    return hipGetLastError();
}

template <knn_dtype DT, bool NORMS>
hipError_t launch_mq(int mq, const DistArgs &a, int64_t n_tiles, int64_t groups, dim3 grid, hipStream_t st,
                     int fm) {
    if (fm != 0) {  // the fused select: 128-query workgroups only
        if (mq != 8) return hipErrorInvalidValue;
        if (fm == 1) return launch_one<DT, 8, 4, 2, 3, NORMS, 256, 64, 1>(a, n_tiles, groups, grid, st);
        return launch_one<DT, 8, 4, 2, 3, NORMS, 256, 64, 2>(a, n_tiles, groups, grid, st);
    }
    const int tile = a.rows_per_tile;
    switch (mq) {
    case 1:
        if (tile == 32) return launch_one<DT, 1, 2, 1, 4, NORMS, 32, 128>(a, n_tiles, groups, grid, st);
        if (tile == 64) return launch_one<DT, 1, 4, 1, 3, NORMS, 64, 128>(a, n_tiles, groups, grid, st);
        return launch_one<DT, 1, 4, 1, 4, NORMS, 128, 64>(a, n_tiles, groups, grid, st);
    case 2:
        if (tile == 32) return launch_one<DT, 2, 2, 2, 4, NORMS, 32, 128>(a, n_tiles, groups, grid, st);
        if (tile == 64) return launch_one<DT, 2, 4, 1, 3, NORMS, 64, 128>(a, n_tiles, groups, grid, st);
        return launch_one<DT, 2, 4, 1, 3, NORMS, 128, 64>(a, n_tiles, groups, grid, st);
    case 4:
        if (tile == 32) return launch_one<DT, 4, 2, 2, 4, NORMS, 32, 128>(a, n_tiles, groups, grid, st);
        if (tile == 64) return launch_one<DT, 4, 2, 2, 3, NORMS, 64, 128>(a, n_tiles, groups, grid, st);
        return launch_one<DT, 4, 2, 2, 3, NORMS, 128, 64>(a, n_tiles, groups, grid, st);
    case 8:
        if (tile == 32) return launch_one<DT, 8, 2, 4, 3, NORMS, 32, 128>(a, n_tiles, groups, grid, st);
        if (tile == 64) return launch_one<DT, 8, 2, 4, 4, NORMS, 64, 64>(a, n_tiles, groups, grid, st);
        if (tile % 256 == 0) return launch_one<DT, 8, 4, 2, 3, NORMS, 256, 64>(a, n_tiles, groups, grid, st);
        return launch_one<DT, 8, 2, 4, 4, NORMS, 128, 64>(a, n_tiles, groups, grid, st);
    default: return hipErrorInvalidValue;
    }
}

template <knn_dtype DT>
hipError_t launch_dt(int mq, const DistArgs &a, int64_t n_tiles, int64_t groups, dim3 grid, hipStream_t st, int fm) {
    return a.key_sqnorms != nullptr ? launch_mq<DT, true>(mq, a, n_tiles, groups, grid, st, fm)
                                    : launch_mq<DT, false>(mq, a, n_tiles, groups, grid, st, fm);
}

}  // namespace

// Key rows per workgroup: at least 256, and enough that a tile runs at least
// 64 pipeline steps of 128 keys x 128 elements, at most 4096 rows; always a
// multiple of 256.
int mfma_tile_rows(int64_t d) {
    const int64_t nspan = d / kSpan > 0 ? d / kSpan : 1;
    int64_t rows = (64 + nspan - 1) / nspan * 128;
    rows = (rows + 255) / 256 * 256;
    if (rows > 4096) rows = 4096;
    return static_cast<int>(rows);
}

// Finer tiles where those of `rows` would leave CUs idle.  Two or three
// workgroups share a CU, so tiles are halved (down to one 128-key pass) while
// they are fewer than four for each CU, or three for 128-query groups, which have
// a CU to themselves (two / three / four for each CU: 25 sets of 20,000 keys of d =
// 1024 and 100 queries 272 / 271 / 289 us, 8 sets of 70,000 keys and 128 queries 378
// / 335 / 336 us).  Where 64-row or 32-row tiles still fit one a CU (two a CU for
// up to 32 queries at 64 rows: there the queries' share of the loads is small),
// each workgroup's few keys are all in flight at once.
// Measured at d = 4096, 128 / 64 / 32 rows a tile: 7,000 keys, 30 queries 33 / 22
// / 17 us (256 rows 72 us); 2 x 7,000 keys, 16 queries 30 / 25 / 28 us; 4 x 7,000
// keys, 32 queries 53 / 49 / 61 us, 64 queries 56 / 63 / 84 us; 8 sets of 4,000 to
// 8,000 keys, 16 to 35 queries 82 / 114 / 137 us (256 rows 102 us).
int mfma_fine_rows(int rows, int64_t S, int64_t max_keys, int64_t max_queries) {
    constexpr int64_t kCus = 256;
    const int64_t groups = (max_queries + 127) / 128;
    auto blocks = [&](int64_t n) { return S * ((max_keys + n - 1) / n) * groups; };
    if (S >= 4 * kCus) return rows;
    int64_t n = rows;
    while (n > 128 && blocks(n) < (max_queries > 64 ? 3 : 4) * kCus) n = (n / 2 + 127) / 128 * 128;
    if (n > 128) return static_cast<int>(n);
    if (blocks(32) <= kCus) return 32;
    if (blocks(64) <= (max_queries <= 32 ? 2 * kCus : kCus)) return 64;
    return 128;
}

hipError_t launch_distances_mfma(int mq, knn_dtype dtype, const DistArgs &args, int64_t S, int64_t groups,
                                 hipStream_t stream, int fm) {
    if (groups < 1 || args.d % kSpan != 0 ||
        (args.rows_per_tile % kTileQuantum != 0 && args.rows_per_tile != 64 && args.rows_per_tile != 32))
        return hipErrorInvalidConfiguration;
    if (fm != 0 && (args.sample_every < 1 || args.sample_rows < kTileQuantum || args.sample_rows % kTileQuantum != 0 ||
                    args.sample_rows > args.rows_per_tile))
        return hipErrorInvalidConfiguration;
    if (fm == 2 && (args.cand_thr == nullptr || args.cand_count == nullptr || args.cand_list == nullptr ||
                    args.fallback == nullptr))
        return hipErrorInvalidValue;
    const int64_t per_set = fm == 1 ? (args.tiles_per_set + args.sample_every - 1) / args.sample_every
                                    : args.tiles_per_set;
    const int64_t n_tiles = S * per_set;
    const int64_t nblocks = (n_tiles + 7) / 8 * 8 * groups;
    if (nblocks > 0x7fffffffLL) return hipErrorInvalidConfiguration;
    const dim3 grid(static_cast<unsigned>(nblocks));
    switch (dtype) {
    case KNN_BF16: return launch_dt<KNN_BF16>(mq, args, n_tiles, groups, grid, stream, fm);
    case KNN_F16: return launch_dt<KNN_F16>(mq, args, n_tiles, groups, grid, stream, fm);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace knnlm
