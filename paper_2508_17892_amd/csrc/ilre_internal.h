// Internal declarations shared by the translation units of libilre (not part of the C ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "ilre.h"

namespace ilre {

constexpr int kHeadDim = ILRE_HEAD_DIM;
constexpr int kNumCU = 256;  // MI355X: 256 compute units in 8 XCDs
constexpr int kNumXCD = 8;

// Asynchronous 16-byte-per-lane copy from a buffer resource straight into LDS: lane l of the
// wavefront lands at lds_addr + 16*l; bytes past the resource's num_records read as zero.  Tracked
// by vmcnt.  Issued as inline assembly so that the compiler's conservative alias handling does not
// put a full vmcnt wait in front of every later LDS read.  (s_nop: a copy to LDS has to be one wait state behind a scalar write
// of M0, which the assembler does not insert by itself.)
typedef __attribute__((ext_vector_type(4))) int i32x4;
__device__ __forceinline__ void lds_dma16(i32x4 rsrc, unsigned lds_addr, int voffset)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(lds_addr), "v"(voffset), "s"(rsrc)
                 : "memory", "m0");
}
// The same from an address a lane.
__device__ __forceinline__ void lds_dma16(uint64_t src, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(src) : "memory", "m0");
}

// ---------------------------------------------------------------- scoring (Eq. 4 / Eq. 5)

// How one scoring pass is cut into workgroups.  A workgroup owns (kv head g, query block qb,
// token split s): `waves` wavefronts of 32*nb query rows each, streaming its token tiles.
struct ScorePlan {
    int dtype;            // ilre_dtype
    int waves;            // wavefronts per workgroup (4 or 8)
    int nb;               // 32-row query blocks per wavefront
    int rows_per_group;   // G * Lq query rows served by one kv head
    int rows_per_wg;      // waves * nb * 32
    bool mixed;           // two query blocks a kv head, the second with one 32-row block a wavefront
    int nqb;              // query blocks per kv group
    int tile_tokens;      // tokens per LDS tile
    int64_t ntiles;       // ceil(L / tile_tokens)
    int nsplit;           // token splits per (g, qb)
    int64_t tiles_per_split;
    int nunits;           // Hkv * nqb  (partial score vectors of pass 2)
    int grid;             // workgroups launched (a few may be idle padding for the XCD mapping)
    bool merge_in_cols;   // whole path: pass 2 merges the partial row statistics (no launch in between)
    bool balanced;        // pass 2's token ranges are sized by the XCDs' speed in pass 1
    uint64_t table_tag;   // header of a range table made for this plan
    size_t lds_bytes_stats, lds_bytes_cols;
};

// Words a launch sets to zero on the side, for a kernel behind it.
struct ClearWords {
    uint32_t *at;  // 16-byte aligned (n = 0: nothing to clear)
    uint32_t n;    // a multiple of 4
};

struct ScoreArgs {
    const void *q;
    const void *k;
    int64_t L;
    int Lq, Hq, Hkv, G;
    int64_t q_stride_head, q_stride_token, k_stride_head, k_stride_token;  // in elements
    float c;  // scale * log2(e): logits leave the MFMA in raw units and are exponentiated base 2
    int rows_per_group, rows_per_wg, nqb, nsplit;
    int64_t ntiles, tiles_per_split;
    // pass 1 (row statistics): per-split partial maxima (base-2 units) and sums
    float *part_m, *part_z;  // [nsplit][Hq*Lq]
    int force_online;        // 1: follow the running maximum throughout (the always-safe form)
    uint32_t *wg_time;       // [grid] how long each workgroup of pass 1 ran, 10 ns ticks (null: not recorded)
    int32_t *split_table;    // [2 + nsplit + 1] pass 2's token ranges: written behind pass 1, read by pass 2 (null: even ranges)
    uint64_t table_tag;
    // pass 2 (column scores)
    const float *row_max, *row_sumexp;  // [Hq*Lq]
    bool merge;                         // whole path: no row statistics, pass 2 merges the partials itself
    ClearWords clear;                   // what pass 2 sets to zero on the side
    float *partial;                     // [nunits][L]
    float *dump;                        // 16 floats nobody reads: target of stores that have nothing to store
};

// `roomy`: query blocks may be of unequal size, which can take one partial score vector more a kv head, and workgroups may be
// more (in several rounds, and with few tiles of fp32 states), which takes more partial row statistics.
ScorePlan make_score_plan(int dtype, int64_t L, int Lq, int Hq, int Hkv, bool roomy);

// With a.merge the partials are all that is left behind.
hipError_t launch_row_stats(const ScorePlan &p, const ScoreArgs &a, float *row_max, float *row_sumexp, hipStream_t s);
// reduce = false leaves the per-unit partial score vectors in a.partial for launch_reduce_units (or for the
// selection's first pass, which can do the reduction on its way).
hipError_t launch_col_scores(const ScorePlan &p, const ScoreArgs &a, int score_mode, float *out_scores,
                             hipStream_t s, bool reduce = true);
hipError_t launch_reduce_units(const float *partial, int nunits, int64_t L, int rmax, float *out_scores, hipStream_t s);

// ---------------------------------------------------------------- selection (Algorithm 1)

constexpr int kSelFine = 256;       // elements a wavefront pools at a time ("fine chunk")
constexpr int kAvgBins = 256;       // printed form: histogram bins per combination
constexpr int kSeedBins = 2048;     // window-max form: histogram bins
constexpr int kSelSmall = 2048;     // seeds beyond the wanted ones that are not worth sorting out
constexpr int kCandCap = 10240;     // candidate capacity in tokens (>= ILRE_MAX_BUDGET + kSelSmall)

// Two forms of Algorithm 1 share the selection kernels.  A "combination" j ranks the elements of a
// source array (value descending, element ascending) and offers the tokens of its best elements:
//   kSelWindowMax  stride-1 max pooling: source = the scores, element = token, value = maximum over a
//                  window of radius r_j clipped to the context; candidates are never exhausted.
//   kSelMaxAvg     the algorithm as printed: source = the cells of a strided max pooling (size = stride
//                  = m), value = stride-1 average over n cells (zeros outside), element p stands for
//                  tokens p*m .. p*m+m-1, and only the best K_m = B/m + 1 cells are candidates.
enum SelMode { kSelWindowMax = 0, kSelMaxAvg = 1 };

struct SelectJob {
    int mode;                    // SelMode
    int64_t L;                   // tokens the pooling sees (the context without its sink part)
    int sink;                    // leading tokens that are always allocated (indices are offset by it)
    int budget;
    int n_max, n_avg;            // kSelWindowMax: n_max window sizes, n_avg = 1
    const int32_t *max_kernels;  // host: window sizes w_j, or max-pooling sizes m_i
    const int32_t *avg_kernels;  // host: average-pooling sizes n_j (kSelMaxAvg only)
    int combos() const { return n_max * n_avg; }
};

// Histogram bins of the window-max form: monotone in the key (ordered_bits of a score), fine where the cut is expected,
// coarse on either side.  Bin 0 is what lies below the first range and is not counted.
constexpr int kBinRanges = 5;
struct KeyBins {
    uint32_t start[kBinRanges];  // keys where the ranges start (a range may be empty)
    uint32_t shift[kBinRanges];  // keys a bin spans, as a shift
    uint32_t pad[2];
};

// Device state of one seed search (window-max form); all zero when its first pass starts.
struct SeedState {
    KeyBins bins;         // left by seed_init where the scores' scale is not known to the host
    uint64_t lists_n;     // keys above the cut bin, collected in `cand` (low half), keys in it, collected in `tie` (high half)
    uint32_t cut;         // bin that holds the K-th largest key
    uint32_t refined;     // not 0: the seeds are the first `refined` of `cand`, else both lists
    uint32_t active_n;    // pre-pass: fine chunks left
    uint32_t done[2];     // workgroups finished: counting, collecting
    uint32_t pad[45];
    uint32_t hist[kSeedBins];
};
static_assert(sizeof(SeedState) % 16 == 0 && sizeof(KeyBins) % 16 == 0 && offsetof(SeedState, hist) % 16 == 0, "cleared in 16-byte words");

struct SelectLayout {
    size_t state;     // kSelWindowMax: SeedState [2]  (the seeds, the pruning pre-pass)
    size_t hist;      // kSelMaxAvg: uint32 [n][kAvgBins]
    size_t ctrl;      // kSelMaxAvg: SelCtrl [n]
    size_t done;      // kSelMaxAvg: uint32 [n]: workgroups finished per max kernel and group of average kernels
    size_t cmax;      // kSelWindowMax: float [ceil(L / kSelFine)]: fine-chunk maxima (pruning pre-pass)
    size_t active;    // kSelWindowMax: uint32 [ceil(L / kSelFine)]: fine chunks left after pruning
    size_t cells;     // float: the max-pooled cell arrays, one per max kernel (kSelMaxAvg)
    size_t picked;    // uint32 [ILRE_MAX_BUDGET] the allocated tokens in the order they were taken, then their count
    size_t seed;      // kSelWindowMax, by rank: uint32 token[kCandCap], uint32 distances to the outranking neighbours[kCandCap]
    size_t cand;      // uint64 [n][kCandCap], one list per combination (kSelWindowMax: one, the seeds)
    size_t tie;       // uint64: per combination two ping-pong lists of boundary elements, each as long as its source
    size_t total;
};

// Printed form: one combination's state.
struct SelCtrl {
    uint32_t want;        // K_j: ranked elements that are candidates
    uint32_t tie_n;       // elements collected
    uint32_t len;         // elements in the source array
    float edge;           // window sums below it are not counted: the bins start here
    uint32_t span[2];     // keys (of float bits) from there on that the first range of bins covers, the first two cover
    uint32_t shifts;      // keys a bin of the three ranges spans, as shifts, a byte each
    uint32_t cut;         // 1 + the lowest bin of which elements are collected (0: all elements)
    uint64_t tie_off;     // lists of elements: uint64 words from the base of the tie region
};

// Workspace carving for a job (only mode, L, counts and the max kernels are read).
SelectLayout make_select_layout(const SelectJob &job);

// Scores that still lie as per-unit partial vectors (the whole path): the selection reduces them into
// `scores` (all L positions, sink part included) itself, in its first pass where it can.
struct FusedScores {
    const float *partial;  // [nunits][L]
    int nunits;
    int rmax;              // 0 sum, 1 max over the units
    float *scores;         // L floats
    int64_t L;
    float mean;            // the scores' scale (window-max form): their mean (sum over the rows) or a lower bound of it (max)
};

// The words of a workspace's selection region (at `base`) that have to be zero before a window-max selection with
// FusedScores starts.
ClearWords select_clear_words(const SelectJob &job, const SelectLayout &lay, void *base);

// `scores` points at the body (the first token after the sink part).
hipError_t launch_select(const float *scores, const SelectJob &job, int32_t *out_idx, int32_t *out_count,
                         void *workspace, const SelectLayout &lay, hipStream_t s, const FusedScores *fused = nullptr);

hipError_t launch_gather_ids(const int32_t *ids, int64_t L, const int32_t *idx, int n, int32_t *out, hipStream_t s);

// ---------------------------------------------------------------- DCA re-RoPE of the key cache

struct RopeArgs {
    const unsigned char *in;
    unsigned char *out;
    int64_t L;
    int Hkv;
    int64_t stride_head, stride_token;  // in elements, the same for in and out
    int chunk, first_extra, nchunks;
    double inv_freq[ILRE_HEAD_DIM / 2];
};

hipError_t launch_rerope(const RopeArgs &a, int dtype, int pairing, hipStream_t s);

// ---------------------------------------------------------------- measurement aid: MFMA ceiling probes

int probe_variants();
const char *probe_describe(int variant);
hipError_t launch_probe(int variant, int iters, const void *operands, float *out, unsigned long long *clocks, double *flops,
                        hipStream_t s);

}  // namespace ilre
