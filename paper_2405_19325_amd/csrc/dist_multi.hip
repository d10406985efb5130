// Distance stage for a few queries per key set on the vector ALUs: the same
// d(q, k) = ||q||^2 - 2 q.k + ||k||^2 (paper Section 2.2) as the streaming
// kernel, bit for bit, with each key row read from HBM once for up to 16
// queries.  It serves the sets that the matrix cores do not: short proposed
// spans (under 16 rows), fp32 elements, d that is no multiple of 128.
//
// Bound: HBM up to 8 queries; at 16 the dot2 rate (17 products of a row at 4
// cycles a wave instruction are 600 cycles of a CU, its share of HBM 730).  The
// streaming kernel holds its queries in registers, which have room for two at
// d = 4096 and for one at d = 8192, so that it read the keys of an 8-query set
// 4 to 8 times.  Here the queries sit in LDS, and a wave takes four key rows at
// a time, so that every 16 bytes of query read from LDS meet 64 bytes of keys:
//   * a step is four rows by 128 chunks of 16 bytes (two a lane); its keys load
//     two steps ahead into a ring of register sets, every load unconditional
//     (rows past the end read the last row, chunks past the row its first).
//     Two sets and not four: the ring is unrolled, and the code of four is read
//     from L2 too slowly at the start (4 x 1,024 keys of d = 1024: 16 against
//     12.5 us);
//   * one workgroup of 8 waves per CU (the queries take up to 128 KiB of LDS),
//     as many workgroups as CUs; each takes an equal, contiguous share of the
//     tiles of all sets, found from the offsets on the device, so that ragged
//     sets leave no CU idle;
//   * the 64-lane sums of 4 rows x NQ queries are reduced together: each
//     exchange step halves the values a lane holds (three instructions for two
//     values) and ends with one value per lane, where a sum of its own for each
//     would take about 15 instructions.  The additions pair the same lanes in
//     the same order as wave_allsum, so every sum has its bits.
// Measured, the streaming kernel and this one (bf16, the distance stage): 4 sets
// of 6,000 to 8,000 keys, 5 to 8 queries, d = 8192: 408 and 86 us (5.3 TB/s); 4 x
// 65,536 keys, 15 queries, d = 4096: 2,498 and 426 us (5.0 TB/s); 4 x 65,536 keys,
// 8 queries, d = 1024: 148 and 97 us; 2 x 145,792 keys, 6 and 13 queries (two
// groups), d = 8192: 6,211 and 1,200 us.
#include "knnlm_internal.h"
#include "mfma_device.h"

namespace knnlm {

namespace {

// Where the distances of rows past the end and of query slots past the group go.
__device__ float g_multi_sink;
constexpr int kMultiWaves = 8;
constexpr int kMultiThreads = kMultiWaves * kWave;
constexpr int kRows = 4;            // key rows per wave and step
constexpr int kCols = 2;            // 16-byte chunks per lane, row and step
constexpr int kPartChunks = kCols * kWave;
constexpr int kSegTiles = 32;       // tiles whose extrema a workgroup keeps in LDS at a time

// The value of lane l ^ 2^BIT.
template <int BIT>
__device__ __forceinline__ float lane_xor(float v) {
    static_assert(BIT >= 0 && BIT < 4, "within a row of 16 lanes");
    if constexpr (BIT == 0) return dpp_f32<0xB1>(v);                        // quad_perm [1,0,3,2]
    else if constexpr (BIT == 1) return dpp_f32<0x4E>(v);                   // quad_perm [2,3,0,1]
    else if constexpr (BIT == 2) return dpp_f32<0x141>(dpp_f32<0x1B>(v));   // l ^ 3, then l ^ 7
    else return dpp_f32<0x140>(dpp_f32<0x141>(v));                          // l ^ 7, then l ^ 15
}

// Lanes with bit BIT clear: x(l) + x(l ^ 2^BIT); the others: the same of y.
template <int BIT>
__device__ __forceinline__ float sum_pair(float x, float y, int lane) {
    if constexpr (BIT < 4) {
        const bool up = (lane >> BIT) & 1;
        const float keep = up ? y : x, send = up ? x : y;
        return keep + lane_xor<BIT>(send);
    } else {
        // rows (halves) of 16 (32) lanes: the odd ones of x change places with the even ones of y
        const uint32_t a = __float_as_uint(x), b = __float_as_uint(y);
        if constexpr (BIT == 4) {
            const auto s = __builtin_amdgcn_permlane16_swap(a, b, false, false);
            return __uint_as_float(s[0]) + __uint_as_float(s[1]);
        } else {
            const auto s = __builtin_amdgcn_permlane32_swap(a, b, false, false);
            return __uint_as_float(s[0]) + __uint_as_float(s[1]);
        }
    }
}

// x(l) + x(l ^ 2^BIT) in every lane.
template <int BIT>
__device__ __forceinline__ float sum_same(float x) {
    if constexpr (BIT < 4) return x + lane_xor<BIT>(x);
    else return sum_pair<BIT>(x, x, 0);
}

// Sums over the 64 lanes of N = 2^k values: lane l gets that of value l % N
// (of those that differ from bit FIRST on: value (l >> FIRST) % N).  The tree
// is wave_allsum's.
template <int N, int FIRST, int BIT = 0>
__device__ __forceinline__ float sum_lanes(float (&v)[N], int lane) {
    if constexpr (BIT == 6) {
        static_assert(N == 1, "at most as many values as lanes");
        return v[0];
    } else if constexpr (N == 1 || BIT < FIRST) {
#pragma unroll
        for (int i = 0; i < N; ++i) v[i] = sum_same<BIT>(v[i]);
        return sum_lanes<N, FIRST, BIT + 1>(v, lane);
    } else {
        float h[N / 2];
#pragma unroll
        for (int i = 0; i < N / 2; ++i) h[i] = sum_pair<BIT>(v[2 * i], v[2 * i + 1], lane);
        return sum_lanes<N / 2, FIRST, BIT + 1>(h, lane);
    }
}

constexpr int log2_of(int x) { return x <= 1 ? 0 : 1 + log2_of(x / 2); }

// Set s as one lane holds it: its first key, first query row of the group, and
// query rows from there on (at most 64 of them matter), its tiles (0: no such
// set, no key, no query of the group) and keys.
struct LaneSet {
    int64_t k0, qb;
    uint32_t nq, tiles, keys;
};

__device__ __forceinline__ LaneSet lane_set(const DistArgs &a, int64_t S, int64_t s, int64_t first_q) {
    const bool in = s < S;
    const int64_t i = in ? s : S - 1;
    const int64_t k0 = a.key_offsets[i], k1 = a.key_offsets[i + 1];
    const int64_t q0 = a.query_offsets[i], q1 = a.query_offsets[i + 1];
    int64_t N = k1 - k0;
    if (N > a.ld) N = a.ld;
    const int64_t nq = q1 - q0 - first_q;
    LaneSet x;
    x.k0 = k0;
    x.qb = q0 + first_q;
    const bool some = in && N > 0 && nq > 0;
    x.nq = some ? static_cast<uint32_t>(nq < kWave ? nq : kWave) : 0u;
    x.keys = some ? static_cast<uint32_t>(N) : 0u;
    x.tiles = some ? (static_cast<uint32_t>(N) + static_cast<uint32_t>(a.rows_per_tile) - 1u) / static_cast<uint32_t>(a.rows_per_tile) : 0u;
    return x;
}

__device__ __forceinline__ int64_t readlane_i64(int64_t v, int lane) {
    const uint32_t lo = readlane_u32(static_cast<uint32_t>(v), lane);
    const uint32_t hi = readlane_u32(static_cast<uint32_t>(static_cast<uint64_t>(v) >> 32), lane);
    return static_cast<int64_t>((static_cast<uint64_t>(hi) << 32) | lo);
}

template <knn_dtype DT, int NQ, int NS, bool MASK>
__global__ __launch_bounds__(kMultiThreads, 2) void k_dist_multi(DistArgs a, int64_t S, int ranges, int groups) {
    constexpr int EB = Elem<DT>::BYTES;
    constexpr int NV = NQ * kRows;  // values reduced together; lane l ends with value l % NV
    constexpr int QB = log2_of(NQ);
    static_assert(NV <= kWave, "one value per lane");
    extern __shared__ __align__(16) u32x4_t qlds[];  // [part][kCols][NQ][lane]
    __shared__ float sqq[NQ];
    __shared__ uint32_t gmin[kSegTiles * NV];  // [tile][row % 4][query]: the select's group minima
    __shared__ uint32_t tmax[kSegTiles * NQ];

    const int tid = threadIdx.x;
    const int lane = tid & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(tid / kWave);
    if (a.zero_words != nullptr && blockIdx.x == 0)
        for (int64_t i = tid; i < a.n_zero_words; i += kMultiThreads) a.zero_words[i] = 0u;

    // The query groups of one share are numbered 8 apart, so they run on one
    // XCD at about the same time and all but the first read its keys from L2.
    const int L = blockIdx.x;
    const int grp = (L >> 3) % groups;
    const int range = ((L >> 3) / groups) * 8 + (L & 7);
    if (range >= ranges) return;
    const int64_t first_q = static_cast<int64_t>(grp) * NQ;

    // The share: of the tiles of all the sets that own queries of this group, in
    // order, the range-th of `ranges` equal parts.  The sets are looked at 64 at
    // a time, one a lane (every wave does the same).
    LaneSet ls = lane_set(a, S, lane, first_q);
    uint32_t incl = wave_incl_scan_u32(ls.tiles, lane);
    int64_t total = readlane_u32(incl, kWave - 1);
    for (int64_t s0 = kWave; s0 < S; s0 += kWave) {
        const LaneSet x = lane_set(a, S, s0 + lane, first_q);
        total += readlane_u32(wave_incl_scan_u32(x.tiles, lane), kWave - 1);
    }
    // Few sets: each gets workgroups of its own in proportion to its tiles (one
    // that crosses from one set to the next stages the queries twice, 8 us).
    uint32_t t0 = 0u, tiles = static_cast<uint32_t>(total), nth = static_cast<uint32_t>(range);
    uint32_t nwg = static_cast<uint32_t>(ranges);
    const uint32_t sets = static_cast<uint32_t>(__popcll(__ballot(ls.tiles != 0u)));
    if (S <= kWave && sets * 8u <= nwg) {
        const float per = static_cast<float>(nwg - sets) / static_cast<float>(tiles);
        const uint32_t mine = ls.tiles != 0u ? 1u + static_cast<uint32_t>(static_cast<float>(ls.tiles) * per) : 0u;
        const uint32_t upto = wave_incl_scan_u32(mine, lane);
        const uint64_t past = __ballot(upto > nth);
        if (past == 0ull) return;  // (rounded down: a few workgroups are left over)
        const int k = __ffsll(static_cast<unsigned long long>(past)) - 1;
        nwg = readlane_u32(mine, k);
        nth -= readlane_u32(upto, k) - nwg;
        tiles = readlane_u32(ls.tiles, k);
        t0 = readlane_u32(incl, k) - tiles;
    }
    // the nth of nwg equal parts of tiles [t0, t0 + tiles), the first of them one tile longer (total < 2^31)
    const uint32_t each = tiles / nwg, more = tiles - each * nwg;
    int64_t at = static_cast<int64_t>(t0 + each * nth + (nth < more ? nth : more));  // the next tile to do
    const int64_t end = at + each + (nth < more ? 1 : 0);

    const int64_t row_bytes = a.d * EB;
    const int nchunks = static_cast<int>(row_bytes / 16);
    const int nparts = (nchunks + kPartChunks - 1) / kPartChunks;
    const bool tail = nchunks % kPartChunks != 0;
    const bool have_norms = a.key_sqnorms != nullptr;
    const bool extrema = a.tile_min != nullptr || a.group_min != nullptr;
    const u32x4_t zero = {0u, 0u, 0u, 0u};
    const int lq = lane & (NQ - 1), lr = (lane >> QB) & (kRows - 1);  // this lane's query and row of a step

    int64_t s0 = 0, before = 0;  // the sets held by the lanes start at s0; tiles before them
    int64_t staged = -1;         // the set whose queries are in LDS
    while (at < end) {
        // the set holding tile `at` (at < total: there is one)
        for (;;) {
            const uint32_t sum = readlane_u32(incl, kWave - 1);
            if (at < before + sum) break;
            before += sum;
            s0 += kWave;
            ls = lane_set(a, S, s0 + lane, first_q);
            incl = wave_incl_scan_u32(ls.tiles, lane);
        }
        const uint32_t want = static_cast<uint32_t>(at - before);
        const int sl = __ffsll(static_cast<unsigned long long>(__ballot(incl > want))) - 1;
        const int64_t s = s0 + sl;
        const uint32_t n_tiles = readlane_u32(ls.tiles, sl);
        const uint32_t t_first = want - (readlane_u32(incl, sl) - n_tiles);
        uint32_t nt = n_tiles - t_first;  // tiles of this segment: of this set, this share and the LDS table
        if (static_cast<int64_t>(nt) > end - at) nt = static_cast<uint32_t>(end - at);
        if (nt > static_cast<uint32_t>(kSegTiles)) nt = kSegTiles;
        at += nt;

        const int64_t k0 = readlane_i64(ls.k0, sl);
        const int64_t N = readlane_u32(ls.keys, sl);
        const int64_t qb = readlane_i64(ls.qb, sl);
        const int nq = min(static_cast<int>(readlane_u32(ls.nq, sl)), NQ);
        const int64_t r0 = static_cast<int64_t>(t_first) * a.rows_per_tile;  // first row, of the set
        const int64_t rend = r0 + static_cast<int64_t>(nt) * a.rows_per_tile;
        const uint32_t nrows = static_cast<uint32_t>((rend < N ? rend : N) - r0);
        const char *kseg = static_cast<const char *>(a.keys) + (k0 + r0) * row_bytes;
        const char *qrow0 = static_cast<const char *>(a.queries) + qb * row_bytes;
        const float *knorm = have_norms ? a.key_sqnorms + k0 + r0 : a.dist;  // a.dist: a valid word, never used

        u32x4_t kv[NS][kRows][kCols];
        float kn[NS];     // ||k||^2 of this lane's row of the set
        uint32_t mw[NS];  // and its mask word
        uint32_t lrow = static_cast<uint32_t>(wave) * kRows;  // first row and part of the next step to load
        int lpart = 0;
        auto load = [&](int set) __attribute__((always_inline)) {
            uint32_t off[kCols];
#pragma unroll
            for (int c = 0; c < kCols; ++c) {
                const int ch = lpart * kPartChunks + c * kWave + lane;
                off[c] = 16u * static_cast<uint32_t>(ch < nchunks ? ch : 0);
            }
#pragma unroll
            for (int r = 0; r < kRows; ++r) {
                const uint32_t row = min(lrow + static_cast<uint32_t>(r), nrows - 1u);
                const char *krow = kseg + static_cast<int64_t>(row) * row_bytes;
#pragma unroll
                for (int c = 0; c < kCols; ++c)
                    kv[set][r][c] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(krow + off[c]));
            }
            const uint32_t mine = lrow + static_cast<uint32_t>(lr);
            const uint32_t rr = mine < nrows ? mine : 0u;
            kn[set] = knorm[have_norms ? rr : 0u];
            if constexpr (MASK) mw[set] = a.key_mask[(k0 + r0 + rr) >> 5];
            if (++lpart == nparts) {
                lpart = 0;
                lrow += kMultiWaves * kRows;
            }
        };
        // The first keys, and the set's queries straight into LDS (a KiB per
        // wave and load; slots past the group repeat its last query).
        __syncthreads();  // the previous segment's reads of LDS are done
#pragma unroll
        for (int i = 0; i < NS; ++i) load(i);
        const uint32_t qlds_at = static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) u32x4_t *)qlds));
        const int qloads = nparts * (kCols * NQ);  // KiB i: part, column, query
        if (staged != s) {
            for (int i = wave; i < qloads; i += kMultiWaves) {
                const int ch = (i >> QB) * kWave + lane, j = i & (NQ - 1);
                load_to_lds_16(qrow0 + (j < nq ? j : nq - 1) * row_bytes + 16 * (ch < nchunks ? ch : 0), qlds_at + i * 1024u);
            }
        }
        for (int i = tid; i < kSegTiles * NV; i += kMultiThreads) gmin[i] = kMaskedBits;
        for (int i = tid; i < kSegTiles * NQ; i += kMultiThreads) tmax[i] = 0u;
        __builtin_amdgcn_s_waitcnt(kVmcntZero);  // the direct loads are known to no register dependence
        __syncthreads();
        if (tail && staged != s) {  // zeros past the row
            for (int i = (nparts - 1) * (kCols * NQ) + wave; i < qloads; i += kMultiWaves)
                if ((i >> QB) * kWave + lane >= nchunks) qlds[i * kWave + lane] = zero;
            __syncthreads();
        }
        if (staged != s) {
            for (int j = wave; j < NQ; j += kMultiWaves) {  // ||q||^2
                float acc = 0.0f;
                for (int p = 0; p < nparts; ++p)
#pragma unroll
                    for (int c = 0; c < kCols; ++c) {
                        const u32x4_t v = qlds[((p * kCols + c) * NQ + j) * kWave + lane];
                        const uint4 q4 = make_uint4(v.x, v.y, v.z, v.w);
                        acc = dot_chunk<DT>(q4, q4, acc);
                    }
                acc = wave_allsum(acc);
                if (lane == 0) sqq[j] = acc;
            }
            staged = s;
        }
        __syncthreads();
        const float qq = sqq[lq];
        float *dq = a.dist + (qb + (lq < nq ? lq : 0)) * a.ld + r0;
        const bool mine_q = lq < nq && lane < NV;

        float acc[NV], acc_k[kRows];  // value of query j and row r at j + NQ * r
#pragma unroll
        for (int i = 0; i < NV; ++i) acc[i] = 0.0f;
#pragma unroll
        for (int r = 0; r < kRows; ++r) acc_k[r] = 0.0f;
        uint32_t row = static_cast<uint32_t>(wave) * kRows;  // first row and part of the step at hand
        int part = 0;
        uint32_t tile = 0, tile_end = static_cast<uint32_t>(a.rows_per_tile);
        // kAhead query chunks are read from LDS ahead of the one at hand (the
        // scheduler's own order read each just before its use, and waited)
        constexpr int kAhead = 3;
        auto consume = [&](int set) __attribute__((always_inline)) {
            if (tail && part == nparts - 1) {
                // chunks past the row hold its first: zeroed here, where the data is used
#pragma unroll
                for (int c = 0; c < kCols; ++c) {
                    const bool has = part * kPartChunks + c * kWave + lane < nchunks;
#pragma unroll
                    for (int r = 0; r < kRows; ++r) kv[set][r][c] = has ? kv[set][r][c] : zero;
                }
            }
            const u32x4_t *qp = qlds + part * (kCols * NQ * kWave) + lane;
            u32x4_t q[kAhead + 1];
#pragma unroll
            for (int i = 0; i < kAhead; ++i) q[i] = qp[i * kWave];
#pragma unroll
            for (int c = 0; c < kCols; ++c) {
                uint4 k4[kRows];
#pragma unroll
                for (int r = 0; r < kRows; ++r) {
                    const u32x4_t k = kv[set][r][c];
                    k4[r] = make_uint4(k.x, k.y, k.z, k.w);
                    acc_k[r] = dot_chunk<DT>(k4[r], k4[r], acc_k[r]);
                }
#pragma unroll
                for (int j = 0; j < NQ; ++j) {
                    const int i = c * NQ + j;
                    if (i + kAhead < kCols * NQ) q[(i + kAhead) % (kAhead + 1)] = qp[(i + kAhead) * kWave];
                    const u32x4_t x = q[i % (kAhead + 1)];
                    const uint4 q4 = make_uint4(x.x, x.y, x.z, x.w);
#pragma unroll
                    for (int r = 0; r < kRows; ++r) acc[j + NQ * r] = dot_chunk<DT>(q4, k4[r], acc[j + NQ * r]);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        // the rows are done: their distances, one a lane
        auto finish = [&](int set) __attribute__((always_inline)) {
            const float kk_sum = sum_lanes<kRows, QB>(acc_k, lane);
            const float dot = sum_lanes<NV, 0>(acc, lane);
            const float kk = have_norms ? kn[set] : kk_sum;
            const uint32_t mine = row + static_cast<uint32_t>(lr);
            const bool in = mine_q && mine < nrows;
            float dist = clamp_nonneg(fmaf(-2.0f, dot, qq + kk));
            bool counted = in;
            if constexpr (MASK) {
                const bool masked = ((mw[set] >> ((k0 + r0 + mine) & 31)) & 1u) != 0u;
                dist = masked ? __uint_as_float(kMaskedBits) : dist;
                counted = counted && !masked;
            }
            *(in ? dq + mine : &g_multi_sink) = dist;
            if (extrema) {
                while (row >= tile_end && tile + 1 < nt) {
                    ++tile;
                    tile_end += static_cast<uint32_t>(a.rows_per_tile);
                }
                if (counted) {
                    atomicMin(&gmin[tile * NV + lane], __float_as_uint(dist));
                    atomicMax(&tmax[tile * NQ + lq], __float_as_uint(dist));
                }
            }
#pragma unroll
            for (int i = 0; i < NV; ++i) acc[i] = 0.0f;
#pragma unroll
            for (int r = 0; r < kRows; ++r) acc_k[r] = 0.0f;
        };
        while (row < nrows) {
#pragma unroll
            for (int i = 0; i < NS; ++i) {
                // the scheduler may not mix the steps' work: that would wait for every load in flight
                __builtin_amdgcn_sched_barrier(0);
                consume(i);
                if (++part == nparts) {
                    finish(i);
                    part = 0;
                    row += kMultiWaves * kRows;
                }
                load(i);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        if (extrema) {
            __syncthreads();
            const int64_t tile0 = t_first;
            for (int i = tid; i < static_cast<int>(nt) * nq; i += kMultiThreads) {
                const int t = i / nq, j = i - t * nq;
                float4 g;
                g.x = __uint_as_float(gmin[t * NV + j]);
                g.y = __uint_as_float(gmin[t * NV + NQ + j]);
                g.z = __uint_as_float(gmin[t * NV + 2 * NQ + j]);
                g.w = __uint_as_float(gmin[t * NV + 3 * NQ + j]);
                if (a.tile_min != nullptr) {
                    a.tile_min[(qb + j) * a.tiles_per_set + tile0 + t] = fminf(fminf(g.x, g.y), fminf(g.z, g.w));
                    a.tile_max[(qb + j) * a.tiles_per_set + tile0 + t] = __uint_as_float(tmax[t * NQ + j]);
                }
                if (a.group_min != nullptr)
                    *reinterpret_cast<float4 *>(a.group_min + (qb + j) * a.groups_per_set + 4 * (tile0 + t)) = g;
            }
        }
    }
}

template <knn_dtype DT, int NQ, int NS>
hipError_t launch_nq(const DistArgs &a, int64_t S, int ranges, int groups, dim3 grid, size_t lds, hipStream_t st) {
    if (a.key_mask != nullptr)
        hipLaunchKernelGGL((k_dist_multi<DT, NQ, NS, true>), grid, dim3(kMultiThreads), lds, st, a, S, ranges, groups);
    else
        hipLaunchKernelGGL((k_dist_multi<DT, NQ, NS, false>), grid, dim3(kMultiThreads), lds, st, a, S, ranges, groups);
    return hipGetLastError();
}

template <knn_dtype DT>
hipError_t launch_dt(int nq, const DistArgs &a, int64_t S, int ranges, int groups, dim3 grid, size_t lds,
                     hipStream_t st) {
    switch (nq) {
    case 2: return launch_nq<DT, 2, 2>(a, S, ranges, groups, grid, lds, st);
    case 4: return launch_nq<DT, 4, 2>(a, S, ranges, groups, grid, lds, st);
    case 8: return launch_nq<DT, 8, 2>(a, S, ranges, groups, grid, lds, st);
    case 16: return launch_nq<DT, 16, 2>(a, S, ranges, groups, grid, lds, st);
    default: return hipErrorInvalidValue;
    }
}

size_t query_lds(int64_t row_bytes, int nq) {
    const int64_t parts = (row_bytes / 16 + kPartChunks - 1) / kPartChunks;
    return static_cast<size_t>(parts * kPartChunks * 16 * nq);
}

}  // namespace

int multi_queries(int64_t d, knn_dtype dtype, int64_t max_queries) {
    int nq = 2;
    while (nq < 16 && nq < max_queries) nq <<= 1;
    while (nq > 2 && query_lds(d * elem_bytes(dtype), nq) > kMultiQueryLds) nq >>= 1;
    return nq;
}

// Shares of the key rows: as many as leave at most a workgroup per CU over all
// query groups (the registers leave room for one), in whole rows of 8, one an
// XCD, each of which takes its workgroups apart from the others' -- but at
// least one row.  With 88 shares of 3 groups an XCD had 33 workgroups for 32 CUs,
// the last in a second pass: 4 x 7,000 keys of d = 256, 40 fp32 queries 73 us, 45 us with 80.
int64_t multi_ranges(int64_t groups) {
    const int64_t ranges = kMultiBlocks / (8 * groups) * 8;
    return ranges < 8 ? 8 : ranges;
}

// Each set past the shares costs every workgroup its place in the walk over
// the sets (2 us for 64 of them) and one workgroup a barrier and the staging of
// its queries: 25 to 35 ns a set and query group over the chip, where the streaming kernel finds its
// set by one division.  That has to be a part of what the streaming kernel takes for the set,
// about 0.3 ns and 0.1 ns a KiB for each row it reads.  Streaming kernel and this one, 4,096 sets:
// 16 keys of d = 256, 8 queries, 38 and 137 us, 128 keys 216 and 241 us, 256 keys
// 419 and 378 us; d = 1024, 12 queries (two passes), 16 keys 97 and 173 us, 64 keys 294 and
// 237 us; d = 1000, 40 queries (5 passes, three groups here), 16 keys 248 and 504 us, 128 keys 1,413 and 1,046 us.
bool multi_pays(int64_t S, int64_t rows, int64_t row_bytes, int64_t groups) {
    return S <= multi_ranges(groups) || rows >= (600 * 1024 * groups + 3 * 1024 + row_bytes - 1) / (3 * 1024 + row_bytes);
}

hipError_t launch_distances_multi(const DistPlan &plan, knn_dtype dtype, const DistArgs &args, int64_t S,
                                  hipStream_t stream) {
    const int64_t tiles = S * plan.tiles_per_set;
    if (tiles > 0x7fffffffLL || plan.groups < 1 || plan.groups > 65535 || args.rows_per_tile % kRows != 0)
        return hipErrorInvalidConfiguration;
    const int64_t ranges = multi_ranges(plan.groups);
    const int64_t nblocks = ranges * plan.groups;
    const size_t lds = query_lds(args.d * elem_bytes(dtype), plan.nq);
    const dim3 grid(static_cast<unsigned>(nblocks));
    const int r = static_cast<int>(ranges), g = static_cast<int>(plan.groups);
    switch (dtype) {
    case KNN_F32: return launch_dt<KNN_F32>(plan.nq, args, S, r, g, grid, lds, stream);
    case KNN_BF16: return launch_dt<KNN_BF16>(plan.nq, args, S, r, g, grid, lds, stream);
    case KNN_F16: return launch_dt<KNN_F16>(plan.nq, args, S, r, g, grid, lds, stream);
    }
    return hipErrorInvalidValue;
}

}  // namespace knnlm
