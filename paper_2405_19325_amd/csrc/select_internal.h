// Internal interfaces of the select, mixture and verification stages.
#pragma once

#include "knnlm_internal.h"

namespace knnlm {

// How a batch's rows are selected (chosen with the workspace layout).
enum SelectPath {
    kRowSelect,       // one workgroup a row: in registers (short rows, r <= 1024) or streamed
    kSplitSelect,     // short rows in parts, or from group minima
    kWideSelect,      // rows in parts, threshold from the tile minima
    kSampledSelect,   // rows in parts, threshold from 4096 sampled keys
    kSampled4Select   // the same from 16384
};

enum MixMode { kNoMix = 0, kMixFixed = 1, kMixRrc = 2, kMixNest = 3 };

struct SelectArgs {
    SelectPath path;
    int parts;                   // parts per row (split, wide and sampled paths)
    const float *dist;           // [B, ld]
    const float *tile_min;       // [B, tiles_per_set] or null
    const float *tile_max;
    const int64_t *key_offsets;
    const int64_t *query_offsets;
    int64_t S;
    int64_t ld;
    int64_t tiles_per_set;
    int rows_per_tile;
    int r;
    int32_t *ids;                // [B, r]
    float *dists;                // [B, r]
    uint64_t *cand;              // split select: [B, parts, kSplitKeys] candidate keys, or null
    uint32_t *part_count;        // split select: [B, parts] candidates per part
    uint32_t *part_min;          // split select: [B, parts] smallest candidate distance bits per part
    uint32_t *part_thr;          // split select: [B] threshold on the distance bits
    // Split select from group minima: the smallest unmasked distance of every
    // group of group_rows keys of a row ([B, groups_per_set], written by the
    // distance stage; group 4 t + w: rows 4 group_rows t + w + 4 e, e <
    // group_rows), or null.
    const float *group_min;
    int64_t groups_per_set;
    int group_rows;
    // Gate: unless null, a wide-select launch does nothing when *gate != gate_run.
    const uint32_t *gate;
    uint32_t gate_run;
};

// The fused select of query batches on long rows (the 128-query matrix-core
// distance kernel): a threshold per query from sampled keys, candidates
// listed by the distance kernel itself, so that the distance matrix is
// written only when the sample misjudges a query (the fallback word).
struct FusedArgs {
    int sample_rows;     // the first sample_rows rows of every sample_every-th tile are the sample
    int sample_every;
    uint32_t *thr;       // [B] threshold on the distance bits
    uint32_t *count;     // [B] candidates listed (true even past kFusedCap)
    uint64_t *list;      // [B, kFusedCap] (distance bits << 32 | local key index)
    uint32_t *fallback;  // 0: the lists hold every query's pi; 1: the distance matrix is written and selected
};

struct MixArgs {
    const int32_t *ids;          // [B, r]
    const float *dists;          // [B, r]
    const int32_t *values;
    const int64_t *key_offsets;
    const int64_t *query_offsets;
    const float *p_lm;           // [B, V]
    float *p_m;                  // [B, V]
    int64_t S;
    int64_t V;
    int r;
    float mu;
    float lambda;                // weight of p_LM (rrc == 0)
    int rrc;                     // 1: a weight per query from relative retrieval confidence
    float alpha, tau;            // its parameters (rrc == 1; tau > 0)
    float *lambda_out;           // [B] the weight each query used, or null (rrc == 1)
    // Decoding outputs of a NEST step (rrc == 1; all null, or next_token,
    // p_max, span_key and use_span given):
    const int32_t *draft;        // [B] the draft token each row checks, or null
    float *p_draft;              // [B] p_M(draft[b]) (0 for a token outside [0, V)); with draft
    float *p_max;                // [B] max_w p_M(w)
    int32_t *next_token;         // [B] the lowest w with p_M(w) = p_max
    int32_t *span_key;           // [B] the nearest neighbour in pi whose value is next_token, or -1
    int32_t *use_span;           // [B] 1 if lambda_t <= delta and span_key >= 0
    float delta;
    // Split select whose finish writes each row in slices (NEST outputs):
    // [B] each, the row's largest entry key and its workgroup count, cleared
    // by the parts kernel or (no parts kernel) by the distance stage; or null.
    uint64_t *best;
    uint32_t *ticket;
};

hipError_t launch_spec_verify(const float *p_max, const float *p_draft, const int32_t *next_token,
                              const int64_t *draft_offsets, int64_t n_drafts, float gamma, const float *uniforms,
                              int32_t *n_accept, int32_t *out_token, hipStream_t stream);

int select_capacity(int r);
// Whether the select of one workgroup a row holds the row in registers.
bool select_in_registers(int64_t ld, int r);
// What a select of one mode (V: 0 without a mixture) launches: the layout's
// path, or one workgroup a row in registers where that is the faster.
struct SelectRoute {
    enum Kind { kGroups, kParts, kWide, kSampled, kSampled4, kRegisters, kStreamed } kind;
    int64_t slices;  // of a row in the split finish (0: whole rows)
};
SelectRoute select_route(const SelectArgs &a, int64_t B, MixMode mode, int64_t V, bool nest_words);
constexpr int64_t kChipCus = 256;
constexpr int64_t kRegisterKeys = 32768;
constexpr int64_t kLargeVocab = 16384;
// Split select: rows of at most kSplitMaxN keys are cut into parts of
// kSplitKeys keys, one workgroup each, when r <= kSplitMaxR and there are at
// most max_blocks parts over all queries (two passes of the chip.  184 rows of
// up to 8,000 keys, a NEST step: 30 us, 48 us with a workgroup a row in registers; 64 rows
// of up to 65,536 keys, fixed lambda: 40 and 51 us).  Returns the parts per query, or 0
// when a query's row is selected by a single workgroup.
constexpr int kSplitKeys = 4096;
constexpr int kSplitCap = 4096;
constexpr int64_t kSplitMaxN = 65536;
constexpr int kSplitMaxR = 1024;
constexpr int64_t kSplitMaxBlocks = 1024;
constexpr int64_t kSplitFewBlocks = 256;  // of a workspace that the lists of more would not fit
int select_split_parts(int64_t B, int64_t ld, int r, int64_t max_blocks);
// Split select from group minima (no parts kernel): the rows per key group
// (4 or 8) when a batch of split rows is served by the streaming distance
// kernels with rows_per_tile = 4 * group rows and every row holds at least 2 r
// groups (`many`) or, by the shortest row, 5/4 r; else 0.  The finish reads
// each row's group minima, takes as threshold the end of the histogram bin
// holding the r-th smallest (so at least r keys lie below it), and gathers the
// keys of the groups below it: of random keys 1.07 r at 8 r groups, 1.27 r at 2 r,
// 1.66 r at 5/4 r (groups of 4).  7,437 keys of d = 4096, r = 1024: a NEST step
// and its verification 32.8 us with the parts kernel's sample, 31.2 us so.
constexpr int kGroupMaxPerRow = 4 * kSelectThreads * 4;  // 16384: four 16-byte loads per thread
int select_group_rows(int64_t ld, int64_t min_keys, int r, int rows_per_tile, bool streaming, bool &many);
// Wide select: rows longer than kSplitMaxN keys are cut into parts (their
// candidate lists use the split layout, [B, parts, kSplitKeys]) when r <= 2048
// and the row has at least 2 r distance tiles; returns the parts per query
// (at most 64), or 0.
constexpr int64_t kWideBlocks = 2048;  // workgroups the wide select aims at
// and the sampled one: one pass of the chip, since each part samples the row
// anew (128 rows of 262,144 keys: 55 us; 1024 workgroups 70 us, 2048 88 us)
constexpr int64_t kSampledBlocks = 512;
int select_wide_parts(int64_t B, int64_t ld, int r, int64_t tiles_per_set);
// Sampled select: any rows with r <= 2048 where the keys below a sampled
// threshold fit the lists (4 standard deviations above their mean); sets the
// path.  The streamed select of one workgroup a row, which it replaces, passes
// over the row three times or more: 128 rows of 262,144 keys 141 us, 96 us so;
// 463 rows of 185,000 to 245,000 keys 335 and 215 us; 278 rows of 8,500 keys,
// r = 2048, 128 and 59 us.  Rows that fit the registers are read once there:
// up to 32768 keys the sampled select is ahead or level (2,000 rows of 12,000 keys,
// r = 1024, V = 8000: 0.77 of the time; of 32,000 keys 0.88), longer ones are not sampled
// (200 rows of 48,000 keys, V = 32000: 43 us, 33 us in registers; 600 rows 1.0 of the time).
// Its lists (32 KiB each) stay under 128 MiB, or under the distances: 100,000
// rows of 1,000 keys would need 3 GiB of them beside 0.8 GiB of the rest.
constexpr int64_t kSampledMaxLists = 4096;
int select_sampled_parts(int64_t B, int64_t ld, int r, SelectPath &path);
hipError_t launch_select(const SelectArgs &args, int64_t B, hipStream_t stream);
hipError_t launch_select_mix(const SelectArgs &args, const MixArgs &mix, int64_t B, hipStream_t stream);
hipError_t launch_mix(const MixArgs &args, int64_t B, hipStream_t stream);
// Fused select, after the sample pieces' distances (launch_distances_mfma fm 1):
// each query's threshold and the sample's candidates; clears the fallback word.
hipError_t launch_fused_threshold(const SelectArgs &args, const FusedArgs &f, int64_t B, hipStream_t stream);
// After the filter launch (fm 2): the fallback word is set if any query's
// candidate count lies outside [min(r, N), kFusedCap].
hipError_t launch_fused_check(const SelectArgs &args, const FusedArgs &f, int64_t B, hipStream_t stream);
// Select (and mixture) after the fused distance stage: from the lists when the
// fallback word is 0, else by the wide select over the distance matrix.
hipError_t launch_select_fused(const SelectArgs &args, const MixArgs *mix, const FusedArgs &f, int64_t B,
                               hipStream_t stream);
// Stores v into *word (a one-thread kernel, so that graph capture records no memset).
hipError_t launch_set_word(uint32_t *word, uint32_t v, hipStream_t stream);

}  // namespace knnlm
