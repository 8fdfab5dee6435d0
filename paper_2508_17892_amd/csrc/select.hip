// Context allocation (paper Section 3.2, Algorithm 1) for gfx950, in two forms: one stride-1 max
// pooling per kernel size (the "window-max" form), and the algorithm as printed (strided max pooling,
// then stride-1 average pooling, one combination per pair of kernel sizes, the best K_m cells only).
//
// Algorithm 1 pools the scores per combination, takes a ranked candidate list per combination and
// walks it, skipping tokens an earlier combination already allocated, until the combination's share
// is filled.  What a combination's candidates are does not depend on the combinations before it (in
// the window-max form its share can be met from its top K_j = B_j + (shares before it) ranked tokens,
// whatever the earlier ones took; in the printed form K_m is given), so the candidate sets are built
// for all combinations at once:
//
//   pool_cells   (cells of other than 1, 2, 3, 4 and 8 tokens, or long windows) the strided max pooling, one cell array per
//                max kernel
//   sel_init     clears histograms and counters, and per combination places the histogram's bins by a sample of its averages
//   pool_averages<0>   the strided max pooling, if not there yet, and per combination a histogram of the averages;
//                the last workgroup of a max kernel finds its combinations' cuts, the bin that holds the K_j-th best
//   pool_averages<1>   the averages at or above the cut, into the combination's list
//   refine       per combination: the list ranked, the first K_j elements kept; a list too long to sort (many equal
//                averages) is radix-selected down first, 8 bits a pass, survivors compacted
//   rank_short   few windows: a workgroup a combination does all of that in one launch; or one for each part of its cells, and
//                refine_parts ranks what they leave
//   allocate_walk   one workgroup walks the combinations in order over their ranked cells: the allocated set is
//                a bitmap in LDS, tokens that it holds are skipped, the first B_j others are taken; the ascending
//                output is then read off the bitmap.  allocate_relay: the same, the wavefronts taking turns, for many
//                combinations with small shares
//   emit_sorted  contexts whose bitmap does not fit the LDS: the allocated set in ascending order (each token
//                counts the tokens below it)
//
// The window-max form does not pool while it scans.  With B' = min(B, L), only the B' best raw scores by
// (score descending, token ascending), the "seeds", can decide anything: the K_j-th largest pooled value
// of any kernel size is at least the B'-th largest raw score (pooling only raises values and K_j <= B'),
// so every candidate token has a seed inside its window, and a seed that B' others outrank owns no token
// of any candidate prefix.  Hence:
//
//   seed_init    (ilre_select alone) clears the state and places the histogram's bins by a sample of the scores; in the
//                whole path the second scoring pass clears it on the side and the bins follow the scores' mean
//   count_scores a 2048-bin histogram of the scores' order-preserving keys, in LDS, added to the global one; the last
//                workgroup to finish finds the bin that holds the B'-th largest (reduce_count: the same on the scores'
//                way from per-unit partial vectors)
//   collect      keys above the cut bin go to the seed list, keys in it to a boundary list (a few hundred on real
//                scores; everything on all-equal scores).  Boundary keys are seeds too (extra seeds rank last and are
//                harmless) unless that makes over kSelSmall too many: the last workgroup to finish then radix-selects
//                them down first
//   seed_rank    per seed: its rank among the seeds (counting: a wavefront's lanes share out the staged keys
//                and compare them with its four seeds) and the nearest seed that outranks it on either side
//                (a scan of the raw scores around it, 16 lanes a seed: whatever outranks a seed is a seed)
//   allocate_walk   for kernel size j seed u owns the tokens whose window holds u and no seed that outranks u, an
//                interval [max(u-r, a+r+1), min(u+r, b-r-1)]; their pooled value is u's score.  Seeds in rank
//                order, each interval ascending, is the kernel size's ranked token list: the walk takes the
//                intervals as they are, no list is written
//   select_brief short contexts: one workgroup does all of that in one launch
//
// Long contexts in the window-max form (L >= 4M and >= 1024 tokens per budgeted token) start with a
// pruning pre-pass: the maximum of every fine chunk (one streaming read of the scores), the bin that
// holds the budget-th largest of those maxima (the same histogram, run on the maxima), and the list of
// fine chunks that can still hold a seed; counting and collecting then visit only that list.
//
// Ranking is (pooled value descending, token index ascending): the 64-bit key is the ordered value
// bits above the complemented element index, so all keys are distinct and every step is
// order-independent; the integer atomics only reserve list slots and build histograms, and the result
// is deterministic.  An element of m tokens ranks its tokens in ascending order, which is the order
// the same key gives them once the element index is replaced by the token index.
#include "ilre_internal.h"
#include "seed_interval.h"

#include <float.h>
#include <string.h>

#include <algorithm>
#include <type_traits>

namespace ilre {
namespace {

constexpr int kThreads = 1024;                    // sel_init, seed_init, refine: one large workgroup
constexpr int kPoolThreads = 256;                 // passes over the scores: four wavefronts
constexpr int kPoolWaves = kPoolThreads / 64;
constexpr int kPerThread = kSelFine / 64;         // 4 tokens per lane
constexpr uint32_t kEmpty = 0xFFFFFFFFu;
constexpr uint32_t kSortSmall = 4096;             // printed form: lists up to this long are sorted whole,
constexpr uint32_t kSortLarge = 10240;            // and up to this long where more than kSortSmall elements are wanted

// Per-combination description, host -> sel_init (by value).
struct SelParams {
    const float *src;                             // the body, or the cells
    uint64_t off[ILRE_MAX_POOL_KERNELS];
    uint32_t want[ILRE_MAX_POOL_KERNELS], len[ILRE_MAX_POOL_KERNELS];
    uint64_t tie_off[ILRE_MAX_POOL_KERNELS];
    uint32_t m[ILRE_MAX_POOL_KERNELS], avg[ILRE_MAX_POOL_KERNELS];
    uint32_t ranks[ILRE_MAX_POOL_KERNELS];        // in the sample: lo, mid, hi and 0, a byte each
};

// Order-preserving map of a finite float onto uint32 (larger float -> larger key; the two zeros share one).
__device__ __forceinline__ uint32_t ordered_bits(float x)
{
    const uint32_t b = __float_as_uint(x + 0.0f);  // -0 ranks with +0
    return b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u);
}

__device__ __forceinline__ uint64_t make_key(float pooled, uint32_t token)
{
    return ((uint64_t)ordered_bits(pooled) << 32) | (uint64_t)(0xFFFFFFFFu - token);
}

__device__ __forceinline__ float float_of_key(uint32_t key) { return __uint_as_float(key ^ (key >> 31 ? 0x80000000u : 0xFFFFFFFFu)); }

__device__ __forceinline__ uint32_t key_token(uint64_t key) { return 0xFFFFFFFFu - (uint32_t)key; }

__device__ __forceinline__ uint32_t load_u32(const uint32_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ uint64_t load_u64(const uint64_t *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

__device__ __forceinline__ void store_u64(uint64_t *p, uint64_t x)
{
    __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Wavefront scans and reductions with DPP row shifts and row broadcasts: six plain vector instructions,
// where a shuffle-based version pays six trips through the LDS crossbar.
#define ILRE_DPP(old, x, ctrl, rows) __builtin_amdgcn_update_dpp((int)(old), (int)(x), ctrl, rows, 0xF, false)
__device__ __forceinline__ uint32_t wave_scan_add(uint32_t x)  // inclusive prefix sum over the 64 lanes
{
    x += (uint32_t)ILRE_DPP(0, x, 0x111, 0xF);  // row_shr:1
    x += (uint32_t)ILRE_DPP(0, x, 0x112, 0xF);  // row_shr:2
    x += (uint32_t)ILRE_DPP(0, x, 0x114, 0xF);  // row_shr:4
    x += (uint32_t)ILRE_DPP(0, x, 0x118, 0xF);  // row_shr:8
    x += (uint32_t)ILRE_DPP(0, x, 0x142, 0xA);  // row_bcast:15 into rows 1 and 3
    x += (uint32_t)ILRE_DPP(0, x, 0x143, 0xC);  // row_bcast:31 into rows 2 and 3
    return x;
}
__device__ __forceinline__ uint32_t wave_scan_max(uint32_t x)  // inclusive running maximum over the 64 lanes
{
    x = max(x, (uint32_t)ILRE_DPP(0, x, 0x111, 0xF));
    x = max(x, (uint32_t)ILRE_DPP(0, x, 0x112, 0xF));
    x = max(x, (uint32_t)ILRE_DPP(0, x, 0x114, 0xF));
    x = max(x, (uint32_t)ILRE_DPP(0, x, 0x118, 0xF));
    x = max(x, (uint32_t)ILRE_DPP(0, x, 0x142, 0xA));
    x = max(x, (uint32_t)ILRE_DPP(0, x, 0x143, 0xC));
    return x;
}
__device__ __forceinline__ uint32_t wave_total(uint32_t scanned)  // lane 63 of an inclusive scan, in every lane
{
    return (uint32_t)__builtin_amdgcn_readlane((int)scanned, 63);
}
// Copy n items from global memory into LDS with the whole block, eight loads in flight per thread.
template <typename T, int THREADS>
__device__ __forceinline__ void stage_to_lds(T *dst, const T *src, uint32_t n)
{
    constexpr int kBatch = 8;
    for (uint32_t i0 = threadIdx.x; i0 < n; i0 += THREADS * kBatch) {
        T x[kBatch];
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const uint32_t i = i0 + b * THREADS;
            x[b] = src[i < n ? i : n - 1];
        }
#pragma unroll
        for (int b = 0; b < kBatch; ++b) {
            const uint32_t i = i0 + b * THREADS;
            if (i < n) dst[i] = x[b];
        }
    }
}

// Inclusive prefix sum over the THREADS threads of the block; wsum is THREADS / 64 words of LDS
// scratch.  Every thread also receives the block total.  Contains two barriers.
template <int THREADS>
__device__ __forceinline__ uint32_t block_scan_inclusive(uint32_t x, uint32_t *wsum, uint32_t &total)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    x = wave_scan_add(x);
    __syncthreads();  // protect wsum against a previous use
    if (lane == 63) wsum[wave] = x;
    __syncthreads();
    uint32_t before = 0, all = 0;
#pragma unroll
    for (int w = 0; w < THREADS / 64; ++w) {
        const uint32_t s = wsum[w];
        if (w < wave) before += s;
        all += s;
    }
    total = all;
    return x + before;
}

// Samples of n elements: one at a hashed place in each of kBaseSamples equal parts, because scores have a structure
// (the first token of every chunk, the sink at the very front) that a regular grid can fall in with.
constexpr int kBaseSamples = 256;
__device__ __forceinline__ int64_t sample_at(uint32_t t, int64_t n)
{
    const int64_t begin = (int64_t)t * n / kBaseSamples, end = (int64_t)(t + 1) * n / kBaseSamples;
    uint32_t h = (t + 1) * 0x9E3779B1u;
    h = (h ^ (h >> 15)) * 0x85EBCA77u;
    h = (h ^ (h >> 13)) * 0xC2B2AE3Du;
    h ^= h >> 16;
    return begin + (int64_t)(((uint64_t)h * (uint64_t)(end - begin)) >> 32);
}

// The sample's keys of N <= 4 ranks (0: the largest; a byte of `ranks` each) into `bound`: a wavefront each finds one bit by
// bit, with the whole sample in its registers.  (Comparing each sample with all others took the workgroup 3 us.)
template <int N>
__device__ __forceinline__ void sampled_bounds(const uint32_t (&key)[kBaseSamples], uint32_t ranks, uint32_t (&bound)[N])
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    __syncthreads();
    if (wave < N) {
        constexpr int kOwn = kBaseSamples / 64;
        uint32_t k[kOwn], at = 0;
#pragma unroll
        for (int i = 0; i < kOwn; ++i) k[i] = key[64 * i + lane];
        const int want = (int)(ranks >> (8 * wave) & 255u) + 1;
        for (uint32_t bit = 0x80000000u; bit; bit >>= 1) {
            int n = 0;
#pragma unroll
            for (int i = 0; i < kOwn; ++i) n += __popcll(__ballot(k[i] >= (at | bit)));
            at |= n >= want ? bit : 0u;
        }
        if (lane == 0) bound[wave] = at;
    }
    __syncthreads();
}

// The ranks of `samples` elements out of `len` that enclose the `want`-th largest element with four standard deviations of
// a sample's count; the upper one has two samples above it, which may be far above everything else.
struct SampleRanks {
    uint32_t lo, hi;
};
SampleRanks sample_ranks(double want_lo, double want_hi, double len)
{
    const double lo = kBaseSamples * want_lo / len, hi = kBaseSamples * want_hi / len;
    const double last = kBaseSamples - 1.0;
    return {(uint32_t)std::min(lo + 4 * sqrt(lo) + 4, last), (uint32_t)std::min(std::max(hi - 4 * sqrt(hi) - 4, 2.0), last)};
}

// Clears the counters and places each combination's bins by a sample of its own window sums: a quarter of them between its
// keys of the ranks lo and mid, a quarter of mid (where the cut is expected) and hi, an eighth of hi and 0, and the rest
// beyond, three times as far again (of many elements the few best lie far above the best sample).  At most a few hundredths of
// the elements more than are wanted reach the lowest bin, whatever the scores look like, and few are in one.
// (Bins of a fixed width, 64 a binade, upward from the scores' median: 1M scores that differ by a thousandth 1170 us,
// their logarithms 831, raised at every 1024th token 847, where others take 100.  More bins than these do not pay: every
// workgroup adds its counts to the global ones, a request per cache line; with 1024 bins counting took 50 us on 1M tokens.)
__global__ __launch_bounds__(kThreads) void sel_init(const SelParams prm, uint32_t *hist, SelCtrl *ctrl, uint32_t *done)
{
    __shared__ __align__(16) uint32_t key[kBaseSamples];
    __shared__ uint32_t bound[4];
    const int j = blockIdx.x;
    static_assert(kThreads == 4 * kBaseSamples, "four threads a sample");
    static_assert(kAvgBins <= kThreads, "a word a thread");
    if (threadIdx.x < (unsigned)kAvgBins) hist[(size_t)j * kAvgBins + threadIdx.x] = 0;
    const uint32_t len = prm.len[j];
    SelCtrl c{};
    if (len) {  // uniform
        // a window's cells are tokens side by side: four threads share a window, or sixteen a long one, a quarter as many
        // of them (all samples of 1024 cells: 35 us of loads for one compute unit), each four times in the sample
        const int n = (int)prm.avg[j], lanes = n > 64 ? 16 : 4, part = threadIdx.x & (lanes - 1);
        const int64_t m = prm.m[j], first = sample_at((threadIdx.x - part) >> 2, len) - (n - 1) / 2;
        auto sum_of = [&](auto size_tag, auto batch_tag) {
            constexpr int M = decltype(size_tag)::value;  // 0: any
            constexpr int kBatch = decltype(batch_tag)::value;
            float sum = 0.0f;
            for (int c0 = part; c0 < n; c0 += lanes * kBatch) {
                float v[kBatch];
#pragma unroll
                for (int b = 0; b < kBatch; ++b) {
                    const int64_t at = first + c0 + lanes * b;
                    const bool in = c0 + lanes * b < n && at >= 0 && at < (int64_t)len;
                    const float *src = prm.src + prm.off[j] + (in ? at : 0) * (M ? M : m);
                    float x = src[0];
                    if (M != 0) {
#pragma unroll
                        for (int u = 1; u < M; ++u) x = fmaxf(x, src[u]);
                    } else {
                        for (int u = 1; u < (int)m; ++u) x = fmaxf(x, src[u]);
                    }
                    v[b] = in ? x : 0.0f;
                }
#pragma unroll
                for (int b = 0; b < kBatch; ++b) sum += v[b];
            }
            return sum;
        };
        using std::integral_constant;
        float sum;
        if (m == 1 && lanes == 16)
            sum = sum_of(integral_constant<int, 1>{}, integral_constant<int, 16>{});
        else if (m == 1)
            sum = sum_of(integral_constant<int, 1>{}, integral_constant<int, 4>{});
        else if (m == 2)
            sum = sum_of(integral_constant<int, 2>{}, integral_constant<int, 4>{});
        else if (m == 4)
            sum = sum_of(integral_constant<int, 4>{}, integral_constant<int, 4>{});
        else if (m == 8)
            sum = sum_of(integral_constant<int, 8>{}, integral_constant<int, 4>{});
        else
            sum = sum_of(integral_constant<int, 0>{}, integral_constant<int, 4>{});
        sum += __shfl_xor(sum, 1);
        sum += __shfl_xor(sum, 2);
        if (lanes == 16) {
            sum += __shfl_xor(sum, 4);
            sum += __shfl_xor(sum, 8);
        }
        if ((threadIdx.x & 3) == 0) key[threadIdx.x >> 2] = ordered_bits(sum);
        sampled_bounds(key, prm.ranks[j], bound);
        static_assert(kAvgBins == 4 << 6, "a quarter of the bins, an eighth");
        auto shift_for = [](uint32_t keys, int bits) { return keys >> bits ? (uint32_t)(32 - bits - __clz((int)keys)) : 0u; };
        c.span[0] = bound[1] - bound[0];
        c.span[1] = bound[2] - bound[0];
        c.shifts = shift_for(bound[1] - bound[0], 6) | shift_for(bound[2] - bound[1], 6) << 8;
        c.shifts |= (bound[3] > bound[2] ? shift_for(bound[3] - bound[2], 5) : 21u) << 16;  // four a binade where the sample says nothing
        c.edge = float_of_key(bound[0]);
    }
    if (threadIdx.x == 0) {
        c.want = prm.want[j];
        c.len = len;
        c.tie_off = prm.tie_off[j];
        ctrl[j] = c;
        done[j] = 0;
    }
}

// A histogram's bins for scores whose scale is known to the host, as an attention's is.  In the sum form their mean is
// exact, and 256 bins a binade lie from half the mean to four times it, where many scores of a flat distribution lie side
// by side; the 3 % around the mean, where all scores of an attention lie that hardly tells its keys apart, have 16 bins
// for each of those (one bin held most of 128K such scores: 482 us where other scores take 290).  Down to 2^-17 of the
// mean, where scores lie if a sink has most of the mass, there are 16 bins a binade, up to 2^18 of it 32; by Markov's
// inequality one score in 2^18 is above, and what is below is not counted.  In the max form `mean` is only a lower bound of
// the mean (a flat attention's is not far above it): the cut then lies in the range above more often.
KeyBins bins_of_mean(float mean)
{
    uint32_t bits;
    memcpy(&bits, &mean, sizeof bits);
    const uint32_t key = bits | 0x80000000u;  // ordered_bits of a positive float
    KeyBins b{};
    b.start[0] = key - (17u << 23), b.shift[0] = 19;
    b.start[1] = key - (1u << 23), b.shift[1] = 15;
    b.start[2] = key - (1u << 17), b.shift[2] = 9;
    b.start[3] = key + (1u << 17), b.shift[3] = 15;
    b.start[4] = key + (2u << 23), b.shift[4] = 18;
    return b;
}

__device__ __forceinline__ uint32_t bin_of(const KeyBins &b, uint32_t key)
{
    uint32_t bin = 1;
#pragma unroll
    for (int i = 0; i < kBinRanges; ++i) {
        const uint32_t at = i + 1 < kBinRanges ? min(max(key, b.start[i]), b.start[i + 1]) : max(key, b.start[i]);
        bin += (at - b.start[i]) >> b.shift[i];
    }
    return key < b.start[0] ? 0u : min(bin, (uint32_t)kSeedBins - 1u);
}

// Clears the states of a seed search on scores of unknown scale and places the bins by a sample of what is counted first:
// the scores, or the maxima of fine chunks.  A quarter of the bins lies between the sample's two keys, a quarter from there to
// 16 times as far as the sample's largest: of many scores the few best lie well above that one.  The others cover all keys
// below (four binades each) and above.  Whatever the sample is, the result is the same.  (With the upper quarter ending as
// far above the upper key as the lower one is below it, the cut of the best 64 of 3M tokens had 2000 others in its bin.)
struct SeedInit {
    const float *vals;
    int64_t n;
    SampleRanks ranks;
};
__global__ __launch_bounds__(kThreads) void seed_init(const SeedInit p, SeedState *st)
{
    __shared__ __align__(16) uint32_t key[kBaseSamples];
    __shared__ uint32_t bound[3];
    constexpr int kWords = sizeof(SeedState) / 16, kKept = sizeof(KeyBins) / 16;  // (the bins are written below)
    for (int i = threadIdx.x; i < 2 * kWords; i += kThreads)
        if (i % kWords >= kKept) ((uint4 *)st)[i] = make_uint4(0, 0, 0, 0);
    if (threadIdx.x < kBaseSamples) key[threadIdx.x] = ordered_bits(p.vals[sample_at(threadIdx.x, p.n)]);
    sampled_bounds(key, p.ranks.lo | p.ranks.hi << 8, bound);  // and rank 0
    if (threadIdx.x == 0) {
        // sizes of bins for which a number of keys takes fewer than 2^bits of them
        auto shift_for = [](uint32_t keys, int bits) { return keys >> bits ? (uint32_t)(32 - bits - __clz((int)keys)) : 0u; };
        const uint32_t low = bound[0], mid = bound[1], top = bound[2];
        const uint32_t tail = top > mid ? shift_for(top - mid, 5) : 17u;  // 64 bins a binade where the sample says nothing
        const uint32_t end = mid + min(512u << tail, 0xFFFFFFFEu - mid);
        uint32_t far = 0;
        constexpr uint32_t kFar = kSeedBins - 1 - 128 - 512 - 512 - 4;  // (a range may end inside a bin)
        while ((0xFFFFFFFFu - end) >> far >= kFar) ++far;
        const KeyBins b{{0, low, mid, end, end}, {25, shift_for(mid - low, 9), tail, 0, far}, {}};
        st[0].bins = st[1].bins = b;
    }
}

// The fine chunks (kSelFine elements) a pooling pass visits: all of the source array, or a list built
// by the pruning pre-pass.
struct Entries {
    const uint32_t *list;    // null: entry i is fine chunk i
    const uint32_t *list_n;  // device count of list entries
};
__device__ __forceinline__ uint32_t entry_count(const Entries &e, uint32_t len)
{
    return e.list ? load_u32(e.list_n) : (len + kSelFine - 1) / kSelFine;
}
__device__ __forceinline__ uint32_t entry_chunk(const Entries &e, uint32_t i) { return e.list ? e.list[i] : i; }

// A wavefront's LDS operations complete in order; waiting for them (and telling the compiler that
// memory changed) is all the synchronisation a wavefront-private buffer needs.
__device__ __forceinline__ void lds_wave_sync() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// BATCH fine chunks (entries e0 .. e0 + BATCH - 1 of the visit list) are fetched at once; fcs[u] < 0 marks a
// missing entry.
constexpr int kRawBatch = 4;
template <int BATCH>
__device__ __forceinline__ void raw_fetch(const float *src, int64_t len, const Entries &ent, uint32_t e0, uint32_t nent,
                                          int64_t (&fcs)[BATCH], float (&vals)[BATCH][kPerThread])
{
    const int lane = threadIdx.x & 63;
#pragma unroll
    for (int u = 0; u < BATCH; ++u) fcs[u] = e0 + u < nent ? (int64_t)entry_chunk(ent, e0 + u) : -1;
#pragma unroll
    for (int u = 0; u < BATCH; ++u)
#pragma unroll
        for (int k = 0; k < kPerThread; ++k) {
            const int64_t e = (fcs[u] < 0 ? 0 : fcs[u]) * kSelFine + lane + k * 64;
            vals[u][k] = src[e < len ? e : len - 1];  // lanes past the end are ignored by the callers
        }
}

// Append the selected items of a wavefront to a list: one slot reservation per wavefront.
template <typename T>
__device__ __forceinline__ void wave_append(bool pred, T item, T *list, uint32_t *counter)
{
    const uint64_t mask = __ballot(pred);
    if (mask == 0) return;
    const int lane = threadIdx.x & 63;
    const int leader = __ffsll((unsigned long long)mask) - 1;
    uint32_t base = 0;
    if (lane == leader) base = atomicAdd(counter, (uint32_t)__popcll(mask));
    base = (uint32_t)__builtin_amdgcn_readlane((int)base, leader);
    if (pred) list[base + __popcll(mask & ((1ull << lane) - 1ull))] = item;
}

// The same for N items a lane (item g of every lane forms group g) and two lists at once: one slot reservation
// per list for the whole lot, both in flight together.  A reservation is a returning atomic on one address, a
// round trip to the memory side; one per group would chain N of them.
template <int N>
__device__ __forceinline__ void wave_append2(const bool (&pa)[N], const bool (&pb)[N], const uint64_t (&item)[N], uint64_t *la,
                                             uint32_t *ca, uint64_t *lb, uint32_t *cb)
{
    const int lane = threadIdx.x & 63;
    uint32_t na = 0, nb = 0;
#pragma unroll
    for (int g = 0; g < N; ++g) {
        na += (uint32_t)__popcll(__ballot(pa[g]));
        nb += (uint32_t)__popcll(__ballot(pb[g]));
    }
    if (na + nb == 0) return;  // uniform
    uint32_t base_a = 0, base_b = 0;
    if (lane == 0) {
        base_a = atomicAdd(ca, na);
        base_b = atomicAdd(cb, nb);
    }
    base_a = (uint32_t)__builtin_amdgcn_readfirstlane((int)base_a);
    base_b = (uint32_t)__builtin_amdgcn_readfirstlane((int)base_b);
    const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
    for (int g = 0; g < N; ++g) {
        const uint64_t ma = __ballot(pa[g]), mb = __ballot(pb[g]);
        if (pa[g]) store_u64(&la[base_a + (uint32_t)__popcll(ma & below)], item[g]);
        if (pb[g]) store_u64(&lb[base_b + (uint32_t)__popcll(mb & below)], item[g]);
        base_a += (uint32_t)__popcll(ma);
        base_b += (uint32_t)__popcll(mb);
    }
}

// Completion counting.  A workgroup's additions to the histograms are device-scope atomics, performed at the memory side,
// common to all eight L2s.  Each thread waits until its own have been performed (vmcnt counts them), then one thread
// counts the workgroup in with another: whoever reads the final count reads, with atomic loads issued after it, bins that
// hold every addition.  A device-scope release fence in their place would also write this L2's unrelated dirty lines back,
// tens of microseconds per workgroup; the acquire side, one workgroup per counter, is cheap and is there.
__device__ __forceinline__ bool count_in(uint32_t *counter, uint32_t workgroups, uint32_t *is_last)
{
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0)
        *is_last = __hip_atomic_fetch_add(counter, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == workgroups - 1;
    __syncthreads();
    if (!*is_last) return false;
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
    return true;
}

// The workgroup's LDS histogram goes to the global one; the last workgroup to count in finds the cut: the bin b with
// count(bins > b) < want <= count(bins >= b), bin 0 (everything not counted) if fewer than `want` were.
__device__ __forceinline__ void count_finish(uint32_t *lh, SeedState *st, uint32_t want)
{
    __shared__ uint32_t is_last, wsum[kPoolWaves];
    __syncthreads();
    constexpr int kPer = kSeedBins / kPoolThreads;
    // neighbouring lanes, neighbouring bins: an atomic request is a cache line
    uint32_t c[kPer];
#pragma unroll
    for (int k = 0; k < kPer; ++k) c[k] = lh[k * kPoolThreads + threadIdx.x];
#pragma unroll
    for (int k = 0; k < kPer; ++k)
        if (c[k]) atomicAdd(&st->hist[k * kPoolThreads + threadIdx.x], c[k]);
    if (!count_in(&st->done[0], gridDim.x, &is_last)) return;
    // thread t: bins top - kPer + 1 .. top
    const int top = kSeedBins - 1 - (int)threadIdx.x * kPer;
    const uint64_t *h2 = (const uint64_t *)&st->hist[top - kPer + 1];
    uint64_t two[kPer / 2];
#pragma unroll
    for (int k = 0; k < kPer / 2; ++k) two[k] = load_u64(&h2[k]);
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < kPer / 2; ++k) sum += (uint32_t)two[k] + (uint32_t)(two[k] >> 32);
    uint32_t total;
    uint32_t above = block_scan_inclusive<kPoolThreads>(sum, wsum, total) - sum;
    if (total < want) {
        if (threadIdx.x == 0) st->cut = 0;
    } else if (above < want && want <= above + sum) {  // one thread
#pragma unroll
        for (int k = kPer - 1; k >= 0; --k) {
            const uint32_t n = (uint32_t)(two[k / 2] >> (k & 1 ? 32 : 0));
            if (above < want && want <= above + n) st->cut = (uint32_t)(top - kPer + 1 + k);
            above += n;
        }
    }
}

__device__ __forceinline__ void count_clear(uint32_t *lh)
{
    for (int i = threadIdx.x * 4; i < kSeedBins; i += kPoolThreads * 4) *(uint4 *)&lh[i] = make_uint4(0, 0, 0, 0);
    __syncthreads();
}
__device__ __forceinline__ void count_one(uint32_t *lh, const KeyBins &bins, float x, bool valid)
{
    const uint32_t bin = bin_of(bins, ordered_bits(x));
    if (valid && bin) atomicAdd(&lh[bin], 1u);
}

// Histogram of the visited scores (or chunk maxima), bins from the state.  A wavefront fetches kRawBatch fine chunks
// before it counts any, so that their loads are in flight together.
__global__ __launch_bounds__(kPoolThreads) void count_scores(const float *vals, int64_t len, uint32_t want, SeedState *st, const Entries ent)
{
    __shared__ __align__(16) uint32_t lh[kSeedBins];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const KeyBins bins = st->bins;
    count_clear(lh);
    const uint32_t nent = entry_count(ent, (uint32_t)len);
    for (uint32_t e0 = (blockIdx.x * kPoolWaves + wave) * kRawBatch; e0 < nent; e0 += gridDim.x * kPoolWaves * kRawBatch) {
        float v[kRawBatch][kPerThread];
        int64_t fcs[kRawBatch];
        raw_fetch(vals, len, ent, e0, nent, fcs, v);
#pragma unroll
        for (int u = 0; u < kRawBatch; ++u) {
            if (fcs[u] < 0) break;  // uniform
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) count_one(lh, bins, v[u][k], fcs[u] * kSelFine + lane + k * 64 < len);
        }
    }
    count_finish(lh, st, want);
}

// The whole path's first selection pass, fused with the last scoring step: score[t] = sum (or max) over the
// (kv head, query block) units of their partial column results, written out for every token, and the
// histogram of the body's scores (tokens sink .. L-1), in one pass over the partial vectors.  The sum runs in unit
// order, as in the stand-alone reduction.  Bound: the partial vectors are 64 MiB at 1M tokens, this pass is their one
// reader; on short contexts the chain clear - load - count - add - find.  PER tokens a lane: one, so that the loads are
// spread over the chip; four from 32K tokens on, because every workgroup adds its counts to the global ones and it is the
// number of those additions that counts (128K tokens: 512 workgroups, and bins four times finer, 42 us).  Measured
// (kernel trace), before (two histogram passes of 11 key bits, two chunks of 256 tokens a wavefront, a kernel to clear)
// -> after: 32K tokens 4.7 + 10.5 + 6.9 -> 7.3 us, 128K 4.7 + 11.3 + 7.4 -> 8.7 us.
template <int RMAX, int PER>
__global__ __launch_bounds__(kPoolThreads) void reduce_count(const float *partial, int nunits, int64_t L, int sink, float *score,
                                                             const KeyBins bins, uint32_t want, SeedState *st)
{
    __shared__ __align__(16) uint32_t lh[kSeedBins];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    count_clear(lh);
    constexpr int kUnits = PER == 1 ? 16 : 8;  // units whose loads are in flight together
    constexpr int kTokens = 64 * PER;          // of a wavefront at a time
    for (int64_t t0 = (int64_t)(blockIdx.x * kPoolWaves + wave) * kTokens; t0 < L; t0 += (int64_t)gridDim.x * kPoolWaves * kTokens) {
        float v[PER];
        int64_t tok[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) tok[k] = t0 + lane + k * 64 < L ? t0 + lane + k * 64 : L - 1;
        for (int u0 = 0; u0 < nunits; u0 += kUnits) {
            float x[kUnits][PER];
#pragma unroll
            for (int uu = 0; uu < kUnits; ++uu) {
                const int64_t u = u0 + uu < nunits ? u0 + uu : nunits - 1;
#pragma unroll
                for (int k = 0; k < PER; ++k) x[uu][k] = partial[u * L + tok[k]];
            }
#pragma unroll
            for (int uu = 0; uu < kUnits; ++uu) {
                if (u0 + uu >= nunits) break;  // uniform
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    if (u0 + uu == 0)
                        v[k] = x[uu][k];
                    else
                        v[k] = RMAX ? fmaxf(v[k], x[uu][k]) : v[k] + x[uu][k];
                }
            }
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const int64_t t = t0 + lane + k * 64;
            if (t < L) score[t] = v[k];
            count_one(lh, bins, v[k], t >= sink && t < L);
        }
    }
    count_finish(lh, st, want);
}

// Pruning pre-pass for long contexts, step 1: cm[c] = max of the scores of fine chunk c.  Pure
// streaming; a wavefront reads four chunks (4 KiB) per iteration.
__device__ __forceinline__ float wave_max(float x)
{
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, true)));   // quad 1,0,3,2
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, true)));   // quad 2,3,0,1
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x141, 0xF, 0xF, true)));  // row_half_mirror
    x = fmaxf(x, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x140, 0xF, 0xF, true)));  // row_mirror
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), 48));
    return fmaxf(fmaxf(r0, r1), fmaxf(r2, r3));
}

__global__ __launch_bounds__(kPoolThreads) void chunk_max(const float *scores, int64_t L, uint32_t nfine, float *cm)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t stride = gridDim.x * kPoolWaves * 4;
    const bool aligned = ((size_t)scores & 15) == 0;  // a sink part may shift the body off the 16-byte grid
    for (uint32_t c0 = (blockIdx.x * kPoolWaves + wave) * 4; c0 < nfine; c0 += stride) {
        float4 v[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int64_t tok = (int64_t)(c0 + u) * kSelFine + lane * 4;
            if (aligned && tok + 3 < L) {
                v[u] = *(const float4 *)(scores + tok);
            } else {
                v[u].x = tok + 0 < L ? scores[tok + 0] : -INFINITY;
                v[u].y = tok + 1 < L ? scores[tok + 1] : -INFINITY;
                v[u].z = tok + 2 < L ? scores[tok + 2] : -INFINITY;
                v[u].w = tok + 3 < L ? scores[tok + 3] : -INFINITY;
            }
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float m = wave_max(fmaxf(fmaxf(v[u].x, v[u].y), fmaxf(v[u].z, v[u].w)));
            if (lane == 0 && c0 + u < nfine) cm[c0 + u] = m;
        }
    }
}

// Pruning pre-pass, step 3 (step 2 is the histogram run on cm for the `budget`-th largest chunk maximum): at least
// `budget` scores, one a chunk, are in that maximum's bin or above it, so no seed is in a bin below; a fine chunk can
// only hold a seed if its maximum reaches the bin.
// One slot reservation per workgroup (same-address atomics serialise at about 13 ns each, and a few thousand
// scattered hits would otherwise mean a few thousand of them): a thread looks at kMarkPerThread consecutive chunks.
constexpr int kMarkPerThread = 16;
__global__ __launch_bounds__(kPoolThreads) void mark_active(const float *cm, uint32_t nfine, SeedState *pre, uint32_t *list)
{
    __shared__ uint32_t wsum[kPoolWaves];
    __shared__ uint32_t base_slot;
    const uint32_t c0 = (blockIdx.x * kPoolThreads + threadIdx.x) * kMarkPerThread;
    const KeyBins bins = pre->bins;
    const uint32_t cut = pre->cut;
    uint32_t hits = 0;  // bit i: chunk c0 + i is active
#pragma unroll
    for (int i = 0; i < kMarkPerThread; ++i)
        if (c0 + i < nfine && bin_of(bins, ordered_bits(cm[c0 + i])) >= cut) hits |= 1u << i;
    uint32_t total;
    const uint32_t mine = (uint32_t)__popc(hits);
    uint32_t at = block_scan_inclusive<kPoolThreads>(mine, wsum, total) - mine;
    if (total == 0) return;  // uniform
    if (threadIdx.x == 0) base_slot = atomicAdd(&pre->active_n, total);
    __syncthreads();
    at += base_slot;
#pragma unroll
    for (int i = 0; i < kMarkPerThread; ++i)
        if ((hits >> i) & 1u) list[at++] = c0 + i;
}

// ---------------------------------------------------------------- printed form: averages, thresholds, candidates

// x / n, correctly rounded, n a small integer and y = 1 / n rounded: a quotient refined with its exact remainder
// twice.  (After one step it is within an ulp, and a quotient within an ulp refined with the rounded reciprocal is
// the rounded quotient: Markstein, IBM J. R&D 34 (1990).)  The remainder must not underflow.
__device__ __forceinline__ float divide_small(float x, float n, float y)
{
    float q = x * y;
    q = fmaf(fmaf(-n, q, x), y, q);
    q = fmaf(fmaf(-n, q, x), y, q);
    const float ax = fabsf(x);
    if (ax < 0x1p-90f || ax > 0x1p100f) q = __fdiv_rn(x, n);
    return q;
}

constexpr int kAvgThreads = 512;
constexpr int kAvgWaves = kAvgThreads / 64;
constexpr int kAvgNarrow = 2, kAvgWide = 4;       // windows a lane sums
constexpr int kAvgGroup = 16;                     // average kernels a workgroup handles
// Collected elements a wavefront holds before it writes them.  64 KiB for a workgroup: with twice as much, and one workgroup a
// compute unit, the wavefront that meets a span of high scores writes once instead of four times, but 16M tokens take 275
// us to collect instead of 188.
constexpr int kAvgQueue = 1024;
constexpr uint16_t kNoAvg = 0xFFFF;
// LDS of pool_averages: counts or collected elements, then a buffer of cells per wavefront (readable kAvgAhead past the last)
constexpr int kAvgAhead = 8;
constexpr size_t avg_shared(int pass, int rows)
{
    return pass == 0 ? ((size_t)rows * kAvgBins + 64) * sizeof(uint32_t)
                     : (size_t)kAvgWaves * kAvgQueue * sizeof(uint64_t);
}
constexpr size_t avg_lds(int pass, int per, bool small, int rows, int n_top)
{
    return avg_shared(pass, rows) + (size_t)kAvgWaves * (size_t)(64 * per + (small ? kAvgGroup : n_top) + kAvgAhead) * sizeof(float);
}

struct AvgParams {
    int n_avg, groups, rows;                              // average kernels, groups of kAvgGroup of them, kernels in the first group
    bool pooled;                                          // the cells are there already (pool_cells)
    uint32_t m[ILRE_MAX_POOL_KERNELS], len[ILRE_MAX_POOL_KERNELS];  // per max kernel: size, cells
    uint64_t off[ILRE_MAX_POOL_KERNELS];                  // its cells
    uint16_t avg[ILRE_MAX_POOL_KERNELS], at[ILRE_MAX_POOL_KERNELS];  // average kernels ascending, and their number in the order given
    uint16_t at_of_size[kAvgGroup];                       // SMALL: number of the average kernel of size 1, 2, .. (kNoAvg: none)
    uint32_t wg_end[ILRE_MAX_POOL_KERNELS];               // per max kernel: its workgroups end before that one (0xFFFFFFFF: not used)
};

// The strided max pooling on its own, where cells are large or windows reach over so many of them that each would be pooled
// several times: 1, 4, 16 or 64 neighbouring lanes read a cell's tokens side by side, kCellBatch cells of each in flight.
// grid = (workgroups, max kernels).
constexpr int kCellBatch = 4;
__host__ __device__ constexpr uint32_t cell_lanes(uint32_t m) { return m < 4 ? 1u : m < 16 ? 4u : m < 64 ? 16u : 64u; }
__global__ __launch_bounds__(kPoolThreads) void pool_cells(const float *body, const AvgParams ap, float *cells)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t m = ap.m[blockIdx.y], len = ap.len[blockIdx.y];
    float *out = cells + ap.off[blockIdx.y];
    const uint32_t lanes = cell_lanes(m), side = 64u / lanes, sub = lane & (lanes - 1);
    const uint32_t step = side * kCellBatch;
    for (uint64_t p0 = (uint64_t)(blockIdx.x * kPoolWaves + wave) * step; p0 < len; p0 += (uint64_t)gridDim.x * kPoolWaves * step) {
        float v[kCellBatch];
        const float *src[kCellBatch];
        uint32_t p[kCellBatch];
#pragma unroll
        for (int b = 0; b < kCellBatch; ++b) {
            p[b] = (uint32_t)p0 + b * side + lane / lanes;
            src[b] = body + (size_t)min(p[b], len - 1) * m;
            v[b] = src[b][0];
        }
        for (uint32_t u = sub; u < m; u += lanes)
#pragma unroll
            for (int b = 0; b < kCellBatch; ++b) v[b] = fmaxf(v[b], src[b][u]);
        for (uint32_t o = 1; o < lanes; o <<= 1)
#pragma unroll
            for (int b = 0; b < kCellBatch; ++b) v[b] = fmaxf(v[b], __shfl_xor(v[b], (int)o));
#pragma unroll
        for (int b = 0; b < kCellBatch; ++b)
            if (sub == 0 && p[b] < len) out[p[b]] = v[b];
    }
}

// The cut of a combination: 1 + the highest bin b with at least `need` elements in the bins from b up (0: fewer than that
// were counted, everything is wanted).  By one wavefront: lane l sums 16 bins in descending order of bins, a scan over the
// lanes finds the lane whose segment holds the crossing.
__device__ __forceinline__ uint32_t find_cut(const uint32_t *h, uint32_t need)
{
    const int lane = threadIdx.x & 63;
    constexpr int BPL = kAvgBins / 64;
    const uint64_t *h2 = (const uint64_t *)(h + kAvgBins - (lane + 1) * BPL);  // this lane's bins, lowest first
    uint64_t two[BPL / 2];
#pragma unroll
    for (int k = 0; k < BPL / 2; ++k) two[k] = load_u64(&h2[k]);
    uint32_t sum = 0;
#pragma unroll
    for (int k = 0; k < BPL / 2; ++k) sum += (uint32_t)two[k] + (uint32_t)(two[k] >> 32);
    const uint32_t incl = wave_scan_add(sum);
    // in the lane with the crossing: how many of its bins, from the top, are needed
    uint32_t above = incl - sum, bins = 0;
#pragma unroll
    for (int k = BPL / 2 - 1; k >= 0; --k) {
        bins += above < need ? 1u : 0u;
        above += (uint32_t)(two[k] >> 32);
        bins += above < need ? 1u : 0u;
        above += (uint32_t)two[k];
    }
    const uint64_t hit = __ballot(incl - sum < need && need <= incl);
    if (hit == 0) return 0;  // uniform
    const int seg = __ffsll((unsigned long long)hit) - 1;
    return (uint32_t)(kAvgBins - seg * BPL) - (uint32_t)__builtin_amdgcn_readlane((int)bins, seg) + 1u;
}

// Both passes over the averages of Algorithm 1.  PASS 0: the strided max pooling (each cell computed where its windows
// are, and written out), and per combination a histogram, whose cut the last workgroup finds.  PASS 1: the elements
// at or above the cut, into the combination's list.  grid = (workgroups of all max kernels, groups).
//
// A window's sum for average kernel n is its sum for n - 1 plus one cell if both windows start at the same cell, which is
// also the order the definition sums in: a lane takes windows by their first cell and gets all average kernels' sums from
// n_max additions.  Counting and comparing go by the sum; the average itself (the quotient ranks, two sums may share
// one) is computed for what is collected only, a full wavefront at a time.  For that the cut is lowered by 2^-21 of its
// value (and by two of the smallest floats a cell): whatever lies below has a smaller quotient than everything at or above
// the cut.
//
// Bins follow the bits of the sum upward from ctrl.edge, the last one open above; they are placed by a sample (sel_init), so
// that the bin of the K_j-th best holds few others and one pass of counting does (two passes of 11 key bits from the
// sign down took twice as long).  With PER = kAvgWide only the largest of a lane's four sums, 64 windows apart, is counted:
// the K_j-th best of those is at most the K_j-th best of all, the few elements more that reach it are sorted out later,
// and a quarter of the additions to LDS, of which 16 lanes' worth takes about as long as all the rest of the loop, are
// left.  It needs K_j to be well below a quarter of the cells.
//
// SMALL: average kernels of sizes 1 .. 16, each once (the paper's set): straight-line code without branches.
// Bound: instructions and LDS round trips of few workgroups on short contexts, additions to the global counts on long ones.
// Measured (kernel trace), 48 combinations, budget 4096, before -> after (before: every combination pooled its own
// windows, two histogram passes): counting 29.6 + 26 -> 10.1 us on 128K tokens, 40.6 + 34.0 -> 15.9 us on 1M; collecting
// 8.1 -> 10.5 us and 23.6 -> 21.1 us; the separate max pooling, 4.7 and 10.1 us, is gone.  (1M since workgroups follow the cells, and
// collecting passes over what cannot reach the cut: 18.2 and 14.1.)
template <int PASS, int PER, bool SMALL>
__global__ __launch_bounds__(kAvgThreads) void pool_averages(const float *body, float *cells, const AvgParams ap, SelCtrl *ctrl,
                                                             uint32_t *hist, uint32_t *done, uint64_t *lists)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t c_comb[kAvgGroup], c_count[kAvgGroup], c_base[kAvgGroup];
    __shared__ uint64_t c_list[kAvgGroup];
    __shared__ float c_rcp[kAvgGroup];
    __shared__ uint32_t is_last;
    constexpr int CHUNK = 64 * PER;            // windows a wavefront sums at a time
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    // the workgroup's max kernel (the first ends are at fixed places of the arguments, loaded together)
    constexpr int kEnds = 8;
    int i = 0;
#pragma unroll
    for (int k = 0; k < kEnds; ++k) i += blockIdx.x >= ap.wg_end[k] ? 1 : 0;
    while (i >= kEnds && blockIdx.x >= ap.wg_end[i]) ++i;  // (the last end is the grid's)
    const uint32_t wg0 = i ? ap.wg_end[i - 1] : 0u, wg = blockIdx.x - wg0, nwg = ap.wg_end[i] - wg0;
    const int g0 = blockIdx.y * kAvgGroup;
    const int ng = min(kAvgGroup, ap.n_avg - g0), rows = SMALL ? kAvgGroup : ng;
    const uint32_t m = ap.m[i], len = ap.len[i];
    const int n_top = ap.avg[g0 + ng - 1], ahead = (n_top - 1) / 2;  // the first windows start before the first cell
    const uint32_t pitch = CHUNK + (SMALL ? kAvgGroup : n_top) - 1;
    uint32_t *lh = (uint32_t *)smem;      // PASS 0: [kAvgGroup][kAvgBins], then a word per lane
    uint64_t *queue = (uint64_t *)smem + wave * kAvgQueue;  // PASS 1: sum above average kernel, chunk and window
    float *buf = (float *)(smem + avg_shared(PASS, SMALL ? kAvgGroup : ap.rows)) + (size_t)wave * (pitch + kAvgAhead);
    float *out = cells + ap.off[i];
    const uint32_t chunks = len ? (uint32_t)(((uint64_t)len + ahead + CHUNK - 1) / CHUNK) : 0u;

    // a chunk's cells from clamped addresses (so that loads need no branch), zero outside the array
    auto stage = [&](auto size_tag, int64_t cell) {
        constexpr int M = decltype(size_tag)::value;  // 0: any
        const uint32_t at = cell < 0 ? 0u : (cell < (int64_t)len ? (uint32_t)cell : len - 1);
        float v;
        if (PASS == 1 || (M == 1 && ap.pooled)) {
            v = out[at];
        } else if (M != 0) {
            const float *src = body + (size_t)at * M;
            v = src[0];
#pragma unroll
            for (int u = 1; u < M; ++u) v = fmaxf(v, src[u]);
        } else {
            const float *src = body + (size_t)at * m;
            v = src[0];
            for (uint32_t u = 1; u < m; ++u) v = fmaxf(v, src[u]);
        }
        return cell < 0 || cell >= (int64_t)len ? 0.0f : v;
    };
    auto fetch = [&](uint32_t c, float(&v)[PER + 1]) {
        const int64_t first = (int64_t)c * CHUNK - ahead;
        auto all = [&](auto size_tag) {
#pragma unroll
            for (int k = 0; k <= PER; ++k) v[k] = stage(size_tag, first + lane + 64 * k);
        };
        if (PASS == 1 || ap.pooled || m == 1)
            all(std::integral_constant<int, 1>{});
        else if (m == 2)
            all(std::integral_constant<int, 2>{});
        else if (m == 4)
            all(std::integral_constant<int, 4>{});
        else if (m == 8)
            all(std::integral_constant<int, 8>{});
        else
            all(std::integral_constant<int, 0>{});
    };
    float cell[PER + 1];
    if (wg * kAvgWaves < chunks) fetch(wg * kAvgWaves + wave, cell);

    // average kernel q's numbers are lane q's, in every wavefront (SMALL: the one of size n has number n - 1)
    uint32_t l_size, l_want, l_span0, l_span1, l_shift;
    uint32_t l_len;  // SMALL: elements of that size: none of a size that was not asked for (an edge alone would let sums of +inf pass)
    float l_edge;    // the sum from which on elements matter to this pass
    {
        uint32_t q, at;
        if (SMALL) {
            q = min(lane, kAvgGroup - 1);
            at = ap.at_of_size[q];
            l_size = q + 1;
        } else {
            q = min(lane, ng - 1);
            at = ap.at[g0 + q];
            l_size = ap.avg[g0 + q];
        }
        const bool used = !SMALL || at != kNoAvg;
        const uint32_t j = (uint32_t)(i * ap.n_avg) + (used ? at : 0u), cut = ctrl[j].cut;
        l_want = ctrl[j].want;
        l_span0 = ctrl[j].span[0];
        l_span1 = ctrl[j].span[1];
        l_shift = ctrl[j].shifts;
        l_edge = ctrl[j].edge;
        if (PASS == 1) {
            const uint32_t s0 = l_shift & 31u, s1 = l_shift >> 8 & 31u, s2 = l_shift >> 16, n0 = l_span0 >> s0, n1 = n0 + ((l_span1 - l_span0) >> s1);
            const uint32_t bin = cut - 1, at = bin <= n0 ? bin << s0 : bin <= n1 ? l_span0 + ((bin - n0) << s1) : l_span1 + ((bin - n1) << s2);
            // (a bin that holds something starts at a float's key, +inf at most)
            const float low = fminf(float_of_key(ordered_bits(l_edge) + at), FLT_MAX);
            l_edge = cut ? low - (fabsf(low) * 0x1p-21f + (float)l_size * 0x1p-148f) : -INFINITY;
        }
        if (!used) l_edge = INFINITY;
        l_len = used ? len : 0u;
        if ((int)threadIdx.x < rows) {
            c_comb[threadIdx.x] = used ? j : 0xFFFFFFFFu;
            c_count[threadIdx.x] = 0;
            c_rcp[threadIdx.x] = __fdiv_rn(1.0f, (float)l_size);
            c_list[threadIdx.x] = ctrl[j].tie_off;
        }
    }
    auto of = [](uint32_t x, int q) { return (uint32_t)__builtin_amdgcn_readlane((int)x, q); };
    // bin of a sum that is not below the edge (differences of float bits in signed order, modulo 2^32)
    auto bin_from = [](float x, float edge, uint32_t span0, uint32_t span1, uint32_t shifts) {
        auto bits = [](float f) { return __float_as_uint(f) ^ ((uint32_t)(__float_as_int(f) >> 31) >> 1); };
        const uint32_t d = bits(x) - bits(edge);
        const uint32_t d0 = min(d, span0), d1 = min(max(d, span0), span1) - span0, d2 = max(d, span1) - span1;
        return min((d0 >> (shifts & 31u)) + (d1 >> (shifts >> 8 & 31u)) + (d2 >> (shifts >> 16)), (uint32_t)kAvgBins - 1u);
    };
    auto of_f = [](float x, int q) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), q)); };
    if (PASS == 0)
        for (int x = threadIdx.x * 4; x < rows * kAvgBins; x += kAvgThreads * 4) *(uint4 *)&lh[x] = make_uint4(0, 0, 0, 0);
    __syncthreads();

    // PASS 1: a wavefront's elements wait in its queue until the workgroup is done: one reservation per workgroup and list
    // then, and no barrier before (one per chunk: 45 - 77 us of a call for the best 64 of 3M tokens, 3.7 ms at 64 max
    // kernels on 16M).  A queue that fills up is written by its wavefront alone.  The word beside a sum names the average
    // kernel, the element's place among the queue's of that kernel, and its chunk and window.
    constexpr uint32_t kWindowBits = 7, kRoundBits = 10, kPlaceBits = 11, kPlaceAt = kWindowBits + kRoundBits, kKernelAt = kPlaceAt + kPlaceBits;
    static_assert(kAvgNarrow * 64 == 1 << kWindowBits && kKernelAt + 4 == 32 && kAvgGroup == 16 && kAvgQueue <= 1 << kPlaceBits, "32 bits");
    uint32_t queued = 0, l_mine = 0;  // uniform; lane q: queued elements of average kernel q
    uint32_t round = 0, first_round = 0;  // chunks done; when the queue was empty
    auto write_queue = [&](uint32_t l_to) {  // l_to: lane q's place in average kernel q's list
        for (uint32_t x = lane; x < ((queued + 63u) & ~63u); x += 64) {
            const bool valid = x < queued;
            const uint64_t e = queue[valid ? x : 0];
            const uint32_t name = (uint32_t)e, q = name >> kKernelAt;
            const uint32_t to = (uint32_t)__shfl((int)l_to, (int)q) + (name >> kPlaceAt & ((1u << kPlaceBits) - 1u));
            const uint32_t size = SMALL ? q + 1 : (uint32_t)__shfl((int)l_size, (int)q);
            const uint32_t chunk = wg * kAvgWaves + wave + (first_round + (name >> kWindowBits & ((1u << kRoundBits) - 1u))) * (nwg * kAvgWaves);
            const uint32_t el = chunk * (uint32_t)CHUNK - (uint32_t)ahead + (name & ((1u << kWindowBits) - 1u)) + (size - 1) / 2;
            const float avg = divide_small(__uint_as_float((uint32_t)(e >> 32)), (float)size, c_rcp[q]);
            if (valid) lists[c_list[q] + to] = make_key(avg, el);
        }
        queued = 0;
        l_mine = 0;
        first_round = round;
    };
    auto spill = [&](uint32_t room) {  // for so many more
        if (queued + room <= (uint32_t)kAvgQueue && round - first_round < 1u << kRoundBits) return;
        uint32_t l_to = 0;
        if (l_mine) l_to = atomicAdd(&ctrl[c_comb[lane]].tie_n, l_mine);
        write_queue(l_to);
    };
    auto enqueue = [&](float x, bool hit, int q, int k, uint32_t place) {  // place: of the queue's next element, less its index
        const uint64_t mask = __ballot(hit);
        const uint32_t at = queued + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
        const uint32_t where = (uint32_t)q << kKernelAt | (round - first_round) << kWindowBits | (uint32_t)(lane + 64 * k);
        if (hit) queue[at] = (uint64_t)__float_as_uint(x) << 32 | (where + ((at + place) << kPlaceAt));
        queued += (uint32_t)__popcll(mask);
    };
    for (uint32_t c0 = wg * kAvgWaves; c0 < chunks; c0 += nwg * kAvgWaves, ++round) {
        const uint32_t c = c0 + wave;  // a chunk past the last one has no elements
        const int64_t first = (int64_t)c * CHUNK - ahead;  // first cell of the chunk's first window
        lds_wave_sync();  // the previous chunk's reads of the buffer are done
#pragma unroll
        for (int k = 0; k <= PER; ++k) {
            const uint32_t x = lane + 64 * k;
            if (x < pitch) buf[x] = cell[k];
            if (PASS == 0 && !ap.pooled && g0 == 0 && k < PER && first + x >= 0 && first + x < (int64_t)len) out[first + x] = cell[k];
        }
        if (!SMALL) {
            constexpr int kBatch = 8;
            for (uint32_t x0 = lane + 64 * (PER + 1); x0 < pitch + lane; x0 += 64 * kBatch) {  // uniform
                float more[kBatch];
#pragma unroll
                for (int b = 0; b < kBatch; ++b) {
                    const int64_t at = first + x0 + 64 * b;
                    more[b] = ap.pooled ? stage(std::integral_constant<int, 1>{}, at) : stage(std::integral_constant<int, 0>{}, at);
                }
#pragma unroll
                for (int b = 0; b < kBatch; ++b)
                    if (x0 + 64 * b < pitch) buf[x0 + 64 * b] = more[b];
            }
        }
        lds_wave_sync();
        if (c0 + nwg * kAvgWaves < chunks) fetch(c + nwg * kAvgWaves, cell);  // in flight while this chunk is summed

        float sum[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) sum[k] = 0.0f;
        const uint32_t el0 = (uint32_t)first + lane;  // modulo 2^32: an element before the array is one far behind it
        if (SMALL) {
            auto size = [&](int u, const float(&x)[PER]) {
                const float edge = of_f(l_edge, u);
                if (PASS == 1) {  // most chunks hold nothing that reaches the cut
                    bool any = false;
#pragma unroll
                    for (int k = 0; k < PER; ++k) {
                        sum[k] = sum[k] + x[k];
                        any = any | !(sum[k] < edge);
                    }
                    if (__ballot(any) == 0) return;  // uniform
                }
                const uint32_t before = queued, els = of(l_len, u), span0 = of(l_span0, u), span1 = of(l_span1, u), shifts = of(l_shift, u);
                float best = -INFINITY;
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    if (PASS == 0) sum[k] = sum[k] + x[k];
                    const bool in = el0 + 64u * k + u / 2 < els;
                    // (what is not counted goes to a word of the lane's own)
                    auto count = [&](float x, bool hit) {
                        const uint32_t bin = bin_from(x, edge, span0, span1, shifts);
                        atomicAdd(&lh[hit ? u * kAvgBins + bin : (uint32_t)(kAvgGroup * kAvgBins + lane)], 1u);
                    };
                    if (PASS == 0 && PER == kAvgWide) {
                        best = fmaxf(best, in ? sum[k] : -INFINITY);
                        if (k == PER - 1) count(best, best >= edge);
                    } else if (PASS == 0) {
                        count(sum[k], in & !(sum[k] < edge));
                    } else {
                        enqueue(sum[k], in & !(sum[k] < edge), u, k, of(l_mine, u) - before);
                    }
                }
                if (PASS == 1) l_mine += lane == u ? queued - before : 0u;
            };
            // (up to the next multiple of four of the largest size that was asked for)
            if (PASS == 0) {
#pragma unroll
                for (int u = 0; u < kAvgGroup; ++u) {
                    if (u % 4 == 0 && u >= n_top) break;
                    float x[PER];
#pragma unroll
                    for (int k = 0; k < PER; ++k) x[k] = buf[lane + 64 * k + u];
                    size(u, x);
                }
            } else {
                float x[4][PER], next[4][PER];
                auto read = [&](int u0, float(&v)[4][PER]) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int k = 0; k < PER; ++k) v[i][k] = buf[lane + 64 * k + u0 + i];
                };
                read(0, x);
#pragma unroll 1
                for (int u0 = 0; u0 < n_top; u0 += 4) {
                    spill(4 * CHUNK);
                    read(u0 + 4, next);
#pragma unroll
                    for (int i = 0; i < 4; ++i) size(u0 + i, x[i]);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int k = 0; k < PER; ++k) x[i][k] = next[i][k];
                }
            }
            continue;
        }

        // any sizes: a rolled loop, kAvgAhead cells a window read ahead of their additions (one by one with two in flight, a
        // window of 1024 cells took 3 - 5 times as long as the whole selection otherwise does)
        for (int q = 0, from = 0; q < ng;) {
            const int to = (int)of(l_size, q);
            if (to - from <= 2) {  // sizes side by side
                for (; from < to; ++from)
#pragma unroll
                    for (int k = 0; k < PER; ++k) sum[k] = sum[k] + buf[lane + 64 * k + from];
            }
            for (int u = from; u < to; u += kAvgAhead) {
                float x[PER][kAvgAhead];
#pragma unroll
                for (int i = 0; i < kAvgAhead; ++i)
#pragma unroll
                    for (int k = 0; k < PER; ++k) x[k][i] = buf[lane + 64 * k + u + i];
                if (u + kAvgAhead <= to) {
#pragma unroll
                    for (int i = 0; i < kAvgAhead; ++i)
#pragma unroll
                        for (int k = 0; k < PER; ++k) sum[k] = sum[k] + x[k][i];
                } else {
#pragma unroll
                    for (int i = 0; i < kAvgAhead; ++i)
#pragma unroll
                        for (int k = 0; k < PER; ++k) sum[k] = u + i < to ? sum[k] + x[k][i] : sum[k];
                }
            }
            from = to;
            for (; q < ng && (int)of(l_size, q) == to; ++q) {  // average kernel q's sums are complete
                if (PASS == 1) spill(CHUNK);
                const float edge = of_f(l_edge, q);
                const uint32_t before = queued;
                if (PASS == 1) {
                    bool any = false;
#pragma unroll
                    for (int k = 0; k < PER; ++k) any = any | !(sum[k] < edge);
                    if (__ballot(any) == 0) continue;  // uniform
                }
#pragma unroll
                for (int k = 0; k < PER; ++k) {
                    const bool hit = !(sum[k] < edge) && el0 + 64u * k + (uint32_t)(to - 1) / 2 < len;
                    if (PASS == 1)
                        enqueue(sum[k], hit, q, k, of(l_mine, q) - before);
                    else if (hit)
                        atomicAdd(&lh[q * kAvgBins + bin_from(sum[k], edge, of(l_span0, q), of(l_span1, q), of(l_shift, q))], 1u);
                }
                if (PASS == 1) l_mine += lane == q ? queued - before : 0u;
            }
        }
    }
    __syncthreads();
    if (PASS == 0) {
        // neighbouring lanes, neighbouring bins: an atomic request is a cache line, and all workgroups want the same few (four
        // bins a lane, 1M tokens, one combination: 46 us for this pass)
        constexpr int kBatch = 8;
        for (int x0 = threadIdx.x; x0 < rows * kAvgBins; x0 += kAvgThreads * kBatch) {
            uint32_t v[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int x = x0 + b * kAvgThreads;
                v[b] = x < rows * kAvgBins ? lh[x] : 0u;
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const int x = x0 + b * kAvgThreads;
                if (v[b]) atomicAdd(&hist[(size_t)c_comb[x / kAvgBins] * kAvgBins + x % kAvgBins], v[b]);
            }
        }
        if (count_in(&done[i * ap.groups + blockIdx.y], nwg, &is_last)) {
            for (int q = wave; q < rows; q += kAvgWaves) {
                if (c_comb[q] == 0xFFFFFFFFu) continue;
                const uint32_t cut = find_cut(hist + (size_t)c_comb[q] * kAvgBins, of(l_want, q));
                if (lane == 0) ctrl[c_comb[q]].cut = cut;
            }
        }
    } else {
        uint32_t l_off = 0;
        if (l_mine) l_off = atomicAdd(&c_count[lane], l_mine);
        __syncthreads();
        if ((int)threadIdx.x < rows && c_count[threadIdx.x]) c_base[threadIdx.x] = atomicAdd(&ctrl[c_comb[threadIdx.x]].tie_n, c_count[threadIdx.x]);
        __syncthreads();
        write_queue((lane < rows ? c_base[lane] : 0u) + l_off);
    }
}

// Of the `need` largest of A's nA distinct keys those that a radix selection finds on its way are appended to
// cand[candn ..]; the rest is among the remaining list, which shrinks by 8 key bits a pass, from A into B and back.
// Stops when what there is fits `keep`, or is exactly what is needed.  By one workgroup.  Keys that share all of a
// digit (equal values do in all of theirs) cost one pass, which also says where they differ first; lanes that share
// one count with a single addition.
template <int THREADS>
__device__ void peel(uint64_t *&A, uint64_t *&B, uint32_t &nA, uint32_t &need, uint64_t *cand, uint32_t &candn, uint32_t keep)
{
    __shared__ uint32_t h[256];
    __shared__ uint32_t cnt[2];
    __shared__ uint32_t pick[3];  // digit, count above it, count in it
    __shared__ unsigned long long differ;  // bits in which keys differ
    constexpr int kFew = 256;
    __shared__ __align__(16) uint64_t few[kFew];
    constexpr int kBatch = 8;  // keys a thread has in flight
    const int lane = threadIdx.x & 63;
    int shift = 56;
    while (nA + candn > keep && need < nA) {
        if (nA <= (uint32_t)kFew) {  // uniform: each counts those ahead of it
            if (threadIdx.x < (uint32_t)kFew) few[threadIdx.x] = threadIdx.x < nA ? load_u64(&A[threadIdx.x]) : 0ull;
            __syncthreads();
            if (threadIdx.x < nA) {
                const uint64_t mine = few[threadIdx.x];
                uint32_t rank = 0;
#pragma unroll 8
                for (uint32_t i = 0; i < (uint32_t)kFew; ++i) rank += few[i] > mine ? 1u : 0u;
                if (rank < need) store_u64(&cand[candn + rank], mine);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            candn += need;
            need = nA = 0;
            break;
        }
        __syncthreads();
        if (threadIdx.x < 256) h[threadIdx.x] = 0;
        if (threadIdx.x < 2) cnt[threadIdx.x] = 0;
        if (threadIdx.x == 0) differ = 0;
        __syncthreads();
        const uint64_t any = load_u64(&A[0]);
        uint64_t bits = 0;
        for (uint32_t first = 0; first < nA; first += THREADS * kBatch) {  // uniform
            uint64_t key[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) key[b] = load_u64(&A[min(first + b * THREADS + threadIdx.x, nA - 1)]);
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const uint32_t i = first + b * THREADS + threadIdx.x, d = (uint32_t)(key[b] >> shift) & 255u;
                const uint64_t there = __ballot(i < nA);
                bits |= key[b] ^ any;
                if (__ballot(d == (uint32_t)__builtin_amdgcn_readfirstlane((int)d)) == ~0ull) {
                    if (lane == 0 && there) atomicAdd(&h[d], (uint32_t)__popcll(there));
                } else if (i < nA) {
                    atomicAdd(&h[d], 1u);
                }
            }
        }
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) bits |= (uint64_t)__shfl_xor((unsigned long long)bits, o);
        if (lane == 0) atomicOr(&differ, (unsigned long long)bits);
        __syncthreads();
        if (threadIdx.x < 64) {
            // lane l owns digits 255-4l .. 252-4l (descending); find the digit holding the need-th key
            uint32_t own[4], sum = 0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                own[k] = h[255 - (lane * 4 + k)];
                sum += own[k];
            }
            const uint32_t incl = wave_scan_add(sum);
            uint32_t above = incl - sum;
            if (above < need && need <= incl) {
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    if (above < need && need <= above + own[k]) {
                        pick[0] = 255 - (lane * 4 + k);
                        pick[1] = above;
                        pick[2] = own[k];
                    }
                    above += own[k];
                }
            }
        }
        __syncthreads();
        const uint32_t digit = pick[0], above = pick[1], inside = pick[2];
        if (inside == nA) {  // all share the digit, and those above it
            if (differ == 0) break;  // (never: keys are distinct)
            shift = max(63 - __clzll((long long)differ) - 7, 0);
            continue;
        }
        for (uint32_t first = 0; first < nA; first += THREADS * kBatch) {  // uniform
            uint64_t key[kBatch];
            bool more[kBatch], same[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) key[b] = load_u64(&A[min(first + b * THREADS + threadIdx.x, nA - 1)]);
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const bool valid = first + b * THREADS + threadIdx.x < nA;
                const uint32_t d = (uint32_t)(key[b] >> shift) & 255u;
                more[b] = valid && d > digit;
                same[b] = valid && d == digit;
            }
            wave_append2<kBatch>(more, same, key, cand + candn, &cnt[0], B, &cnt[1]);
        }
        // The survivors go through global memory to the next pass of this same workgroup: wait until
        // the stores have reached the L2 and read them back past the L1 (load_u64).  A fence would do
        // too, at the price of an L2 write-back per pass.
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        candn += above;
        need -= above;
        nA = inside;
        shift = max(shift - 8, 0);
        uint64_t *t = A;
        A = B;
        B = t;
    }
}

// Window-max form: keys above the cut bin are seeds, keys in it go to the boundary list.  A workgroup reserves its slots
// in both lists with one atomic on the two counters (they are one word for it): a returning atomic on an address that
// everybody wants takes its turn at about 13 ns (128K tokens: one per wavefront and list 21 us, this 6.2 us).  Both lists are
// written with device-scope stores, so that the last workgroup (on whichever XCD) may read the boundary list if it is
// one of the long ones (a kernel of its own for that took 2 - 4.7 us to find nothing to do).  All keys equal, that workgroup
// is most of the whole call: 32K tokens 86 us with four wavefronts, 128K 135 us with eight (203 with four), 1M 833 us (1483).
template <int BATCH, int THREADS>
__global__ __launch_bounds__(THREADS) void collect(const float *vals, int64_t len, uint32_t want, const KeyBins known, bool sampled,
                                                   SeedState *st, uint64_t *cand, uint64_t *tie, const Entries ent)
{
    constexpr int WAVES = THREADS / 64;
    __shared__ uint32_t is_last;
    __shared__ uint64_t wave_n[WAVES], base;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const KeyBins bins = sampled ? st->bins : known;
    const uint32_t cut = st->cut;
    const uint32_t nent = entry_count(ent, (uint32_t)len);
    for (uint32_t e0 = blockIdx.x * WAVES * BATCH; e0 < nent; e0 += gridDim.x * WAVES * BATCH) {  // uniform
        float v[BATCH][kPerThread];
        int64_t fcs[BATCH];
        raw_fetch(vals, len, ent, e0 + wave * BATCH, nent, fcs, v);
        bool above[BATCH * kPerThread], same[BATCH * kPerThread];
        uint32_t na = 0, ns = 0;
#pragma unroll
        for (int u = 0; u < BATCH; ++u)
#pragma unroll
            for (int k = 0; k < kPerThread; ++k) {
                const int g = u * kPerThread + k;
                const bool valid = fcs[u] >= 0 && fcs[u] * kSelFine + lane + k * 64 < len;
                const uint32_t bin = bin_of(bins, ordered_bits(v[u][k]));
                above[g] = valid && bin > cut;
                same[g] = valid && bin == cut;
                na += (uint32_t)__popcll(__ballot(above[g]));
                ns += (uint32_t)__popcll(__ballot(same[g]));
            }
        const uint64_t mine = (uint64_t)ns << 32 | na;
        if (lane == 0) wave_n[wave] = mine;
        __syncthreads();
        uint64_t before = 0, all = 0;
#pragma unroll
        for (int w = 0; w < WAVES; ++w) {
            before += w < wave ? wave_n[w] : 0;
            all += wave_n[w];
        }
        if (threadIdx.x == 0 && all) base = atomicAdd((unsigned long long *)&st->lists_n, all);
        __syncthreads();
        if (mine) {  // uniform in the wavefront
            const uint64_t at = base + before;
            uint32_t at_a = (uint32_t)at, at_s = (uint32_t)(at >> 32);
            const uint64_t below = (1ull << lane) - 1ull;
#pragma unroll
            for (int g = 0; g < BATCH * kPerThread; ++g) {
                const uint64_t ma = __ballot(above[g]), ms = __ballot(same[g]);
                if ((ma | ms) == 0) continue;  // uniform
                const uint64_t key = make_key(v[g / kPerThread][g % kPerThread], (uint32_t)(fcs[g / kPerThread] * kSelFine + lane + g % kPerThread * 64));
                if (above[g]) store_u64(&cand[at_a + (uint32_t)__popcll(ma & below)], key);
                if (same[g]) store_u64(&tie[at_s + (uint32_t)__popcll(ms & below)], key);
                at_a += (uint32_t)__popcll(ma);
                at_s += (uint32_t)__popcll(ms);
            }
        }
    }
    if (!count_in(&st->done[1], gridDim.x, &is_last)) return;
    const uint64_t lists_n = load_u64(&st->lists_n);
    uint32_t candn = (uint32_t)lists_n, nA = (uint32_t)(lists_n >> 32), need = want - candn;
    if (candn + nA <= want + (uint32_t)kSelSmall) return;  // uniform
    uint64_t *A = tie, *B = tie + len;
    peel<THREADS>(A, B, nA, need, cand, candn, want + (uint32_t)kSelSmall);
    for (uint32_t i = threadIdx.x; i < nA; i += THREADS) cand[candn + i] = load_u64(&A[i]);
    if (threadIdx.x == 0) st->refined = candn + nA;
}

// Elements in rank order by a counting sort of one workgroup: kRankBins bins over the range of the values' key bits,
// descending, a scan of the counts places every bin, and inside a bin an element counts the ones that rank ahead of it.
// Where a bin is crowded (a few values far above the others stretch the range) every bin is split in proportion to what it holds,
// and the elements are counted once more.  Thread t holds PER keys, of which the ones in `have` exist (`all` in all; `top` and
// `low` enclose their value bits); the elements of the first `want` go out in order.  False where one of the bins they are in
// still holds more than kRankDeep (equal values): the keys then lie in srt[0 .. all) in some order, for the network.
// (A list of 4096 elements all in bins of 128: the whole call 50 us, of 256: 67, of 512: 100; by the network 68.)
constexpr int kRankBins = 2048;
// Counting once more takes 1.5 us (27 combinations, 20000 tokens, budget 4096, bins split that hold more than 48 33.6 us, 160 32.2,
// 255 32.2; 4 combinations, 40000 tokens, budget 4096 31.3, 31.5, 36.2).
constexpr uint32_t kRankCrowd = 160, kRankDeep = 256;
struct RankShared {
    uint32_t bin_n[2 * kRankBins];
    uint32_t split[kRankBins];  // first of a bin's parts, and their number's logarithm in 5 bits
    uint32_t wmax[kThreads / 64], wmin[kThreads / 64], wsum[kThreads / 64];
    uint32_t cut, above, within;  // last bin that is wanted, elements ahead of it and in it
};

// the range's top 11 bits number the bins
__device__ __forceinline__ uint32_t rank_shift(uint32_t top, uint32_t low)
{
    static_assert(kRankBins == 1 << 11, "11 bits");
    const uint32_t bits = 32 - __clz((int)(top - low));
    return bits > 11 ? bits - 11 : 0;
}

// the largest and the smallest of all threads' value bits; bin_n is zero behind it
__device__ __forceinline__ void rank_range(RankShared &sh, uint32_t &top, uint32_t &low)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    static_assert(kRankBins == 2 * kThreads, "two bins a thread");
    *(uint2 *)&sh.bin_n[2 * threadIdx.x] = make_uint2(0, 0);
    const uint32_t t = wave_scan_max(top), l = wave_scan_max(~low);
    if (lane == 63) sh.wmax[wave] = t, sh.wmin[wave] = l;
    __syncthreads();
    uint32_t not_low = 0;
#pragma unroll
    for (int w = 0; w < kThreads / 64; ++w) top = max(top, sh.wmax[w]), not_low = max(not_low, sh.wmin[w]);
    low = ~not_low;
}

// The bin that holds the `want`-th of the elements counted in bin_n, in descending order.
__device__ __forceinline__ void rank_cut(RankShared &sh, uint32_t want)
{
    __syncthreads();
    const uint2 n2 = *(const uint2 *)&sh.bin_n[2 * threadIdx.x];
    uint32_t all;
    const uint32_t upto = block_scan_inclusive<kThreads>(n2.x + n2.y, sh.wsum, all), before = upto - n2.x - n2.y;
    if (before < want && want <= upto) {  // one thread
        const bool second = before + n2.x < want;
        sh.cut = 2 * threadIdx.x + (second ? 1u : 0u);
        sh.above = second ? before + n2.x : before;
        sh.within = second ? n2.y : n2.x;
    }
    __syncthreads();
}

// Of the keys in `have` the `want` best, and no more than `slack` others: 11 bits a pass of what the keys at the cut differ in, first
// of their values, then of their elements.
template <int PER, typename KEY>
__device__ __forceinline__ uint32_t narrow(RankShared &sh, const KEY &key, uint32_t have, uint32_t want, uint32_t slack)
{
    uint32_t taken = 0;
    bool by_value = true;
    while (true) {
        auto word = [&](int k) { return by_value ? (uint32_t)(key(k) >> 32) : (uint32_t)key(k); };
        uint32_t top = 0, low = 0xFFFFFFFFu;
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (have >> k & 1u) top = max(top, word(k)), low = min(low, word(k));
        rank_range(sh, top, low);
        if (by_value && top == low) {  // uniform: equal values
            by_value = false;
            __syncthreads();
            continue;
        }
        const uint32_t shift = rank_shift(top, low);
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (have >> k & 1u) atomicAdd(&sh.bin_n[(top - word(k)) >> shift], 1u);
        rank_cut(sh, want);
        const uint32_t cut = sh.cut;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t bin = (top - word(k)) >> shift;
            if ((have >> k & 1u) && bin < cut) taken |= 1u << k;
            if (bin != cut) have &= ~(1u << k);
        }
        want -= sh.above;
        if (sh.within - want <= slack) return taken | have;
    }
}

template <int PER>
__device__ bool rank_keys(RankShared &sh, uint64_t *srt, const uint64_t (&key)[PER], uint32_t have, uint32_t top, uint32_t low, uint32_t want,
                          uint32_t *ranked, uint32_t &all)
{
    const uint32_t shift = rank_shift(top, low);
    uint32_t bin[PER], place[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        bin[k] = (top - (uint32_t)(key[k] >> 32)) >> shift;
        if (have >> k & 1u) place[k] = atomicAdd(&sh.bin_n[bin[k]], 1u);
    }
    __syncthreads();
    // a bin's word: how many elements rank ahead of it, and its own number
    static_assert(PER * kThreads < 1 << 15, "15 bits a count");
    const uint2 n2 = *(const uint2 *)&sh.bin_n[2 * threadIdx.x];
    const uint32_t before = block_scan_inclusive<kThreads>(n2.x + n2.y, sh.wsum, all) - n2.x - n2.y;
    *(uint2 *)&sh.bin_n[2 * threadIdx.x] = make_uint2(before << 15 | n2.x, (before + n2.x) << 15 | n2.y);
    const bool crowd = __syncthreads_or((n2.x > kRankCrowd && before < want) || (n2.y > kRankCrowd && before + n2.x < want));
    const bool split = crowd && shift;
    auto part_of = [&](uint64_t x) {
        const uint32_t d = top - (uint32_t)(x >> 32), w = sh.split[d >> shift], e = w & 31u;
        return (w >> 5) + ((d & ((1u << shift) - 1u)) >> (shift - e));
    };
    bool deep = false;
    if (__builtin_expect(split, 0)) {  // uniform
        // 2^e parts, about as many as a bin's elements are of the whole list's 2048ths
        auto parts = [&](uint32_t n) { return n ? min(31u - (uint32_t)__clz((int)max(n * (uint32_t)kRankBins / all, 1u)), shift) : 0u; };
        const uint32_t e0 = parts(n2.x), e1 = parts(n2.y), p0 = n2.x ? 1u << e0 : 0u, p1 = n2.y ? 1u << e1 : 0u;
        uint32_t total;
        const uint32_t first = block_scan_inclusive<kThreads>(p0 + p1, sh.wsum, total) - p0 - p1;  // (at most 2 kRankBins in all)
        *(uint2 *)&sh.split[2 * threadIdx.x] = make_uint2(first << 5 | e0, (first + p0) << 5 | e1);
        *(uint4 *)&sh.bin_n[4 * threadIdx.x] = make_uint4(0, 0, 0, 0);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            if (have >> k & 1u) {  // (the other keys may lie outside the bins)
                bin[k] = part_of(key[k]);
                place[k] = atomicAdd(&sh.bin_n[bin[k]], 1u);
            }
        }
        __syncthreads();
        const uint4 n4 = *(const uint4 *)&sh.bin_n[4 * threadIdx.x];
        const uint32_t sum = n4.x + n4.y + n4.z + n4.w, b0 = block_scan_inclusive<kThreads>(sum, sh.wsum, all) - sum;
        const uint32_t b1 = b0 + n4.x, b2 = b1 + n4.y, b3 = b2 + n4.z;
        *(uint4 *)&sh.bin_n[4 * threadIdx.x] = make_uint4(b0 << 15 | n4.x, b1 << 15 | n4.y, b2 << 15 | n4.z, b3 << 15 | n4.w);
        deep = __syncthreads_or((n4.x > kRankDeep && b0 < want) || (n4.y > kRankDeep && b1 < want) || (n4.z > kRankDeep && b2 < want) ||
                                (n4.w > kRankDeep && b3 < want));
    } else if (crowd) {
        deep = __syncthreads_or((n2.x > kRankDeep && before < want) || (n2.y > kRankDeep && before + n2.x < want));
    }
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (have >> k & 1u) srt[(sh.bin_n[bin[k]] >> 15) + place[k]] = key[k];
    __syncthreads();
    if (deep) return false;
    // neighbouring threads, neighbouring places: a deep bin is the work of the few wavefronts that hold it, from one address
    for (uint32_t x = threadIdx.x; x < all; x += kThreads) {
        const uint64_t mine = srt[x];
        const uint32_t at = sh.bin_n[split ? part_of(mine) : (top - (uint32_t)(mine >> 32)) >> shift], first = at >> 15, n = at & 32767u;
        if (first >= want) break;  // (so are those behind it)
        uint32_t rank = first;
#pragma unroll 8
        for (uint32_t i = 0; i < n; ++i) rank += srt[first + i] > mine ? 1u : 0u;
        if (rank < want) ranked[rank] = key_token(mine);
    }
    return true;
}

// Bitonic sort of the keys in srt[0 .. total) (descending; padding keys of 0 sink to the end), one barrier per stage; the
// elements of the first `want` go out in order.
__device__ void rank_network(uint64_t *srt, uint32_t total, uint32_t want, uint32_t *ranked)
{
    uint32_t padded = 2;
    while (padded < total) padded *= 2;
    for (uint32_t i = total + threadIdx.x; i < padded; i += kThreads) srt[i] = 0ull;
    __syncthreads();
    for (uint32_t k = 2; k <= padded; k <<= 1) {
        for (uint32_t d = k >> 1; d > 0; d >>= 1) {
            for (uint32_t i = threadIdx.x; i < padded / 2; i += kThreads) {
                const uint32_t lo = ((i & ~(d - 1)) << 1) | (i & (d - 1)), hi = lo + d;
                const uint64_t a = srt[lo], b = srt[hi];
                const bool descending = (lo & k) == 0;
                if ((a < b) == descending) {
                    srt[lo] = b;
                    srt[hi] = a;
                }
            }
            __syncthreads();
        }
    }
    for (uint32_t r = threadIdx.x; r < want; r += kThreads) ranked[r] = key_token(srt[r]);
}

// Printed form: the list of a combination in rank order, cut to the K_j best elements.  A list too long to sort (many
// equal averages) is radix-selected down first.  The rest goes by the counting sort: bound by the latency
// of its few rounds through LDS on one workgroup a combination, where the network takes a round and a barrier for each of
// 55 - 78 stages.  Measured (kernel trace): 9001 tokens 8.7 -> 4.8 us, 128K 15.6 -> 5.8 us, 1M
// 14.4 -> 4.8 us; values in two clusters (spans just as many as are wanted, and the background's top) 47 -> 19 us; the best
// 8192 of 3M 118 us by radix selection and network.  Where a bin is deep (equal averages in number) the network, for up to
// sort_n elements, is the faster one still.
__global__ __launch_bounds__(kThreads) void refine(const SelCtrl *ctrl, uint64_t *cand, uint64_t *tie, uint32_t sort_n)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ __align__(16) RankShared sh;
    uint64_t *srt = (uint64_t *)smem;
    const int j = blockIdx.x;
    uint64_t *cand_j = cand + (size_t)j * kCandCap;
    uint64_t *A = tie + ctrl[j].tie_off;
    uint64_t *B = A + ctrl[j].len;
    const uint32_t want = ctrl[j].want;
    uint32_t nA = ctrl[j].tie_n, need = want, candn = 0;
    const bool large = sort_n > kSortSmall;  // uniform: there is room for kSortLarge keys
    peel<kThreads>(A, B, nA, need, cand_j, candn, large ? kSortLarge : kSortSmall);
    uint32_t total = candn + nA;
    auto element = [&](uint32_t i) { return i < candn ? load_u64(&cand_j[i]) : load_u64(&A[i - candn]); };
    // the walk wants the elements in rank order; the list (uint32) takes over the storage of the keys
    uint32_t *ranked = (uint32_t *)cand_j;
    auto by_counting = [&](auto per_tag) {
        constexpr int PER = decltype(per_tag)::value;
        uint64_t key[PER];
        uint32_t top = 0, low = 0xFFFFFFFFu, have = 0;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            const uint32_t i = threadIdx.x + k * kThreads;
            key[k] = element(i < total ? i : total - 1);
            have |= i < total ? 1u << k : 0u;
            top = max(top, (uint32_t)(key[k] >> 32));
            low = min(low, (uint32_t)(key[k] >> 32));
        }
        rank_range(sh, top, low);
        uint32_t all;
        return rank_keys(sh, srt, key, have, top, low, want, ranked, all);
    };
    if (total == 0) return;  // uniform
    if (total <= kSortSmall ? by_counting(std::integral_constant<int, (int)kSortSmall / kThreads>{})
                            : by_counting(std::integral_constant<int, (int)kSortLarge / kThreads>{}))
        return;
    if (total > sort_n) peel<kThreads>(A, B, nA, need, cand_j, candn, sort_n);
    total = candn + nA;
    for (uint32_t i = threadIdx.x; i < total; i += kThreads) srt[i] = element(i);
    rank_network(srt, total, want, ranked);
}

// The same where several workgroups have collected a combination's elements, each the best of its part of the cells: part c's
// lie in the list from c * size on.
constexpr int kShortParts = 64;  // most parts
static_assert(kShortParts <= kAvgBins, "their counts lie where the histograms do otherwise");
__global__ __launch_bounds__(kThreads) void refine_parts(const SelParams prm, uint32_t size, const uint32_t *part_n, uint64_t *cand, const uint64_t *tie)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ __align__(16) RankShared sh;
    __shared__ uint32_t part_at[kShortParts + 1];
    uint64_t *srt = (uint64_t *)smem;
    const int j = blockIdx.x;
    const uint32_t want = prm.want[j], len = prm.len[j], parts = (len + size - 1) / size;
    if (want == 0) return;  // uniform
    if (threadIdx.x < 64) {
        static_assert(kShortParts == 64, "a lane a part");
        part_at[threadIdx.x + 1] = wave_scan_add(threadIdx.x < parts ? part_n[j * kShortParts + threadIdx.x] : 0u);
        if (threadIdx.x == 0) part_at[0] = 0;
    }
    __syncthreads();
    const uint64_t *list = tie + prm.tie_off[j];
    uint64_t *cand_j = cand + (size_t)j * kCandCap;
    uint32_t *ranked = (uint32_t *)cand_j;
    const uint32_t total = part_at[kShortParts];  // kSortLarge at most
    uint32_t half = 1;  // of a power of two of parts
    while (2 * half < parts) half *= 2;
    auto by_counting = [&](auto per_tag) {
        constexpr int PER = decltype(per_tag)::value;
        uint64_t key[PER];
        uint32_t c[PER], top = 0, low = 0xFFFFFFFFu, have = 0, all;
#pragma unroll
        for (int k = 0; k < PER; ++k) {
            c[k] = 0;
            have |= threadIdx.x + k * kThreads < total ? 1u << k : 0u;
        }
        for (uint32_t step = half; step; step >>= 1) {  // the parts they are in
#pragma unroll
            for (int k = 0; k < PER; ++k) c[k] += part_at[c[k] + step] <= min(threadIdx.x + k * kThreads, total - 1) ? step : 0u;
        }
#pragma unroll
        for (int k = 0; k < PER; ++k) key[k] = list[min(threadIdx.x + k * kThreads, total - 1) - part_at[c[k]] + c[k] * size];
#pragma unroll
        for (int k = 0; k < PER; ++k) top = max(top, (uint32_t)(key[k] >> 32)), low = min(low, (uint32_t)(key[k] >> 32));
        rank_range(sh, top, low);
        if (rank_keys(sh, srt, key, have, top, low, want, ranked, all)) return;
        // many equal averages
        const uint32_t subset = narrow<PER>(sh, [&](int k) { return key[k]; }, have, want, 0);
        rank_range(sh, top, low);
        if (!rank_keys(sh, srt, key, subset, top, low, want, ranked, all)) rank_network(srt, all, want, ranked);
    };
    if (total <= kSortSmall)
        by_counting(std::integral_constant<int, (int)kSortSmall / kThreads>{});
    else
        by_counting(std::integral_constant<int, (int)kSortLarge / kThreads>{});
}

// Printed form, few windows: the cut of a combination is not looked for by all workgroups over all windows but by one, or by one
// for each part of the cells.  It pools the cells into LDS, sums the windows (four neighbouring ones a thread, from
// 16-byte reads; in the order of the definition), finds the cut with a histogram over the range of the sums' keys, and ranks what
// reaches it; a part's elements are left for refine_parts.  Equal sums are narrowed down by their places before that.  Where few are wanted only the largest of a thread's four neighbours is
// counted: the K_j-th best of those is at most the K_j-th best of all.
// Bound: latency (one round of loads, a dozen barriers); a workgroup a combination and 4096 windows share nothing, so that the
// number of windows decides, see the launch.  Against sel_init, both passes over the averages and refine (kernel trace, 48
// combinations, budget 4096 resp. 1000): 9001 tokens 6.9 + 10.1 + 8.8 + 4.5 -> 10.4 us, 128K 6.7 + 11.6 + 10.7 + 4.7 -> 16.8 + 8.5.
constexpr uint32_t kShortCells = 16384;  // most cells a combination may have, ..
constexpr int kShortMax = 8, kShortAvg = 64;  // .. tokens a cell, and cells a window
constexpr size_t short_lds(uint32_t len, int n_top, bool ranks)
{
    size_t keys = ranks ? 2 : 0;
    while (ranks && keys < len) keys *= 2;
    const size_t cells = (size_t)((len + 3) & ~3u) + (size_t)n_top + 8;
    return std::max(keys * sizeof(uint64_t), cells * sizeof(float));
}
template <int QUADS, bool PARTS>
__global__ __launch_bounds__(kThreads, PARTS ? 8 : 4) void rank_short(const SelParams prm, uint32_t slack, uint64_t *cand, uint64_t *tie, uint32_t *part_n)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ __align__(16) RankShared sh;
    constexpr int PER = 4 * QUADS;
    const int j = blockIdx.y, tid = threadIdx.x;
    const uint32_t cells = prm.len[j], m = prm.m[j], n = prm.avg[j], first = blockIdx.x * (PER * kThreads);
    if (first >= cells || prm.want[j] == 0) return;  // uniform
    const uint32_t len = min(cells - first, (uint32_t)(PER * kThreads)), want = min(prm.want[j], len);
    float *buf = (float *)smem;
    const uint32_t lead = (n - 1) / 2, padded = ((len + 3) & ~3u) + n + 8;  // cell p lies at p - first + lead, zeros around all
    auto pool = [&](auto size_tag) {
        constexpr int M = decltype(size_tag)::value;  // 0: any
        constexpr int kBatch = 4;
        for (uint32_t i0 = tid; i0 < padded; i0 += kThreads * kBatch) {
            float v[kBatch];
#pragma unroll
            for (int b = 0; b < kBatch; ++b) {
                const uint32_t p = first + i0 + b * kThreads - lead;  // (modulo 2^32)
                const float *src = prm.src + (size_t)min(p, cells - 1) * (M ? (uint32_t)M : m);
                v[b] = src[0];
                if (M != 0) {
#pragma unroll
                    for (int u = 1; u < M; ++u) v[b] = fmaxf(v[b], src[u]);
                } else {
                    for (uint32_t u = 1; u < m; ++u) v[b] = fmaxf(v[b], src[u]);
                }
                if (p >= cells) v[b] = 0.0f;
            }
#pragma unroll
            for (int b = 0; b < kBatch; ++b)
                if (i0 + b * kThreads < padded) buf[i0 + b * kThreads] = v[b];
        }
    };
    using std::integral_constant;
    if (m == 1)
        pool(integral_constant<int, 1>{});
    else if (m == 2)
        pool(integral_constant<int, 2>{});
    else if (m == 4)
        pool(integral_constant<int, 4>{});
    else if (m == 8)
        pool(integral_constant<int, 8>{});
    else
        pool(integral_constant<int, 0>{});
    __syncthreads();
    const float size = (float)n, rcp = __fdiv_rn(1.0f, size);
    uint32_t value[PER];  // ordered
    uint32_t have = 0, best[QUADS];
    auto key = [&](int k) { return (uint64_t)value[k] << 32 | (0xFFFFFFFFu - (first + 4 * (tid + k / 4 * kThreads) + k % 4)); };  // as make_key
#pragma unroll
    for (int q = 0; q < QUADS; ++q) {
        const uint32_t el = 4 * (tid + q * kThreads);
        float sum[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (el < len) {
            for (uint32_t u = 0; u < n + 3; u += 4) {  // window i of the four holds cells i .. i + n - 1 from here
                const float4 x4 = *(const float4 *)&buf[el + u];
                const float x[4] = {x4.x, x4.y, x4.z, x4.w};
                if (u >= 4 && u + 3 < n) {  // uniform
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int i = 0; i < 4; ++i) sum[i] += x[r];
                } else {
#pragma unroll
                    for (int r = 0; r < 4; ++r)
#pragma unroll
                        for (int i = 0; i < 4; ++i)
                            if (u + r >= (uint32_t)i && u + r - i < n) sum[i] += x[r];  // uniform
                }
            }
        }
        best[q] = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            value[4 * q + i] = ordered_bits(divide_small(sum[i], size, rcp));
            if (el + i < len) {
                have |= 1u << (4 * q + i);
                best[q] = max(best[q], value[4 * q + i]);
            }
        }
    }
    uint32_t subset = have;
    bool many = true;
    if (2 * want <= (len + 3) / 4) {  // uniform: down to the bin that holds the K_j-th of the best of each four
        uint32_t top = 0, low = 0xFFFFFFFFu;
#pragma unroll
        for (int q = 0; q < QUADS; ++q)
            if (have >> (4 * q) & 1u) top = max(top, best[q]), low = min(low, best[q]);
        rank_range(sh, top, low);
        const uint32_t shift = rank_shift(top, low);
#pragma unroll
        for (int q = 0; q < QUADS; ++q)
            if (have >> (4 * q) & 1u) atomicAdd(&sh.bin_n[(top - best[q]) >> shift], 1u);
        rank_cut(sh, want);
        const uint32_t cut = sh.cut;
        many = PARTS || sh.above + sh.within > want + slack;
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if ((top - value[k]) >> shift > cut) subset &= ~(1u << k);
    }
    if (many) subset = narrow<PER>(sh, key, subset, want, slack);
    if (!PARTS) {
        uint32_t top = 0, low = 0xFFFFFFFFu, total;
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if (subset >> k & 1u) top = max(top, value[k]), low = min(low, value[k]);
        rank_range(sh, top, low);
        uint64_t *srt = (uint64_t *)smem, keys[PER];
#pragma unroll
        for (int k = 0; k < PER; ++k) keys[k] = key(k);
        uint32_t *ranked = (uint32_t *)(cand + (size_t)j * kCandCap);
        if (!rank_keys(sh, srt, keys, subset, top, low, want, ranked, total)) rank_network(srt, total, want, ranked);
        return;
    }
    uint32_t total;
    const uint32_t mine = (uint32_t)__popc(subset);
    uint64_t *at = tie + prm.tie_off[j] + first + (block_scan_inclusive<kThreads>(mine, sh.wsum, total) - mine);
#pragma unroll
    for (int k = 0; k < PER; ++k)
        if (subset >> k & 1u) *at++ = key(k);
    if (tid == 0) part_n[j * kShortParts + blockIdx.x] = total;
}

// Last step of the allocation: the sink indices, then the nsel allocated tokens in ascending order, then -1
// up to sink + n_out.  The walk leaves the tokens in the order it took them; here every token counts the
// tokens below it, which is its place in the output whatever order they arrived in and however they
// cluster.  The list is staged in LDS; a wavefront owns kEmitPerWave tokens and its lanes read disjoint
// quarters of the list (every LDS word is fetched once per wavefront) and compare them with all of the
// wavefront's tokens.
constexpr int kEmitThreads = 512;
constexpr int kEmitPerWave = 4;
constexpr int kEmitPerBlock = kEmitThreads / 64 * kEmitPerWave;  // 32 tokens a workgroup
__global__ __launch_bounds__(kEmitThreads) void emit_sorted(const uint32_t *picked, const uint32_t *picked_n, int n_out, int sink,
                                                            int32_t *out_idx, int32_t *out_count)
{
    __shared__ __align__(16) uint32_t all[ILRE_MAX_BUDGET];
    static_assert(ILRE_MAX_BUDGET % 256 == 0, "the staged list is padded to whole rounds of 64 lanes x 4 tokens");
    const uint32_t nsel = *picked_n;
    const uint32_t gtid = blockIdx.x * kEmitThreads + threadIdx.x, gsize = gridDim.x * kEmitThreads;
    for (uint32_t i = gtid; i < (uint32_t)sink; i += gsize) out_idx[i] = (int32_t)i;
    for (uint32_t i = nsel + gtid; i < (uint32_t)n_out; i += gsize) out_idx[sink + i] = -1;
    if (gtid == 0 && out_count) *out_count = sink + (int32_t)nsel;
    if (blockIdx.x * kEmitPerBlock >= nsel) return;  // uniform
    stage_to_lds<uint32_t, kEmitThreads>(all, picked, nsel);
    const uint32_t padded = (nsel + 255u) & ~255u;  // the padding holds tokens no token is below
    if (threadIdx.x < 256 && nsel + threadIdx.x < padded) all[nsel + threadIdx.x] = 0xFFFFFFFFu;
    __syncthreads();
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const uint32_t i0 = blockIdx.x * kEmitPerBlock + wave * kEmitPerWave;
    if (i0 >= nsel) return;  // whole wavefronts leave together, no barrier follows
    uint32_t t[kEmitPerWave], below[kEmitPerWave];
#pragma unroll
    for (int q = 0; q < kEmitPerWave; ++q) {
        t[q] = (uint32_t)__builtin_amdgcn_readfirstlane((int)all[i0 + q < nsel ? i0 + q : nsel - 1]);
        below[q] = 0;
    }
#pragma unroll 2
    for (uint32_t v = 4u * lane; v < padded; v += 256) {
        const uint4 x = *(const uint4 *)&all[v];
#pragma unroll
        for (int q = 0; q < kEmitPerWave; ++q)
            below[q] += (x.x < t[q] ? 1u : 0u) + (x.y < t[q] ? 1u : 0u) + (x.z < t[q] ? 1u : 0u) + (x.w < t[q] ? 1u : 0u);
    }
#pragma unroll
    for (int q = 0; q < kEmitPerWave; ++q) {
        const uint32_t place = wave_total(wave_scan_add(below[q]));
        if (lane == q && i0 + q < nsel) out_idx[sink + place] = (int32_t)(t[q] + (uint32_t)sink);
    }
}

// The allocated set I of Algorithm 1 as a bitmap over the body's tokens, 32 tokens a word.  Up to kBitmapTokens
// tokens the whole bitmap lies in LDS (128 KiB at 1M tokens); beyond that LDS holds an open-addressing table of
// the words that have a bit set: at most ILRE_MAX_BUDGET of them, half of its slots.
constexpr int kBitmapChunk = 256;                      // words a wavefront turns into output at a time
constexpr int kBitmapChunks = 136;                     // 136 KiB of the compute unit's 160
constexpr int kBitmapTokens = kBitmapChunks * kBitmapChunk * 32;
constexpr int kWordSlots = 16384;
static_assert(kWordSlots >= 2 * ILRE_MAX_BUDGET, "the word table stays half empty");

template <bool HASHED>
struct TokenSet {
    uint32_t *key, *mask;  // HASHED: word index and bits per slot; otherwise mask[word]
    static __device__ __forceinline__ uint32_t slot_of(uint32_t word) { return (word * 0x9E3779B1u) >> 18; }
    __device__ __forceinline__ uint32_t get(uint32_t word) const
    {
        if (!HASHED) return mask[word];
        uint32_t s = slot_of(word);
        while (true) {
            const uint32_t k = key[s];
            if (k == word) return mask[s];
            if (k == kEmpty) return 0u;
            s = (s + 1) & (kWordSlots - 1);
        }
    }
    __device__ __forceinline__ void set(uint32_t word, uint32_t bits) const
    {
        if (!HASHED) {
            atomicOr(&mask[word], bits);
            return;
        }
        uint32_t s = slot_of(word);
        while (true) {
            const uint32_t old = atomicCAS(&key[s], kEmpty, word);
            if (old == kEmpty || old == word) break;
            s = (s + 1) & (kWordSlots - 1);
        }
        atomicOr(&mask[s], bits);
    }
};

// bits of word w that lie in the token interval [first, last]
__device__ __forceinline__ uint32_t interval_bits(uint32_t w, uint32_t first, uint32_t last)
{
    uint32_t m = 0xFFFFFFFFu;
    if (w == first >> 5) m &= 0xFFFFFFFFu << (first & 31);
    if (w == last >> 5) m &= 0xFFFFFFFFu >> (31 - (last & 31));
    return m;
}

// LDS writes of this wavefront done, then the workgroup barrier; global loads in flight stay in flight.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Algorithm 1's walk.  Combination j offers its tokens as ranked intervals that do not overlap -- in the window-max
// form the tokens each seed owns, seeds in rank order; in the printed form the tokens of each cell, cells in rank
// order -- and takes the first B_j of them, in that order and ascending inside an interval, that the set does not
// hold yet.  A thread looks at kWalkPer neighbouring intervals: the free tokens in one are a population count of one
// or two words of the set, a scan over the workgroup gives every interval the number of free tokens ranked ahead of
// it, and those up to the share's end are marked, a word at a time.
//
// Bound: the chain of dependent LDS round trips and instructions per combination (gather, scan, exchange, marks) on
// one compute unit, about 1300 cycles.  Hence the gathers of a thread's intervals are in flight together, no atomic
// returns a value, a combination's numbers come from a register lane, its list is in LDS before it is needed, and
// there is one scan and two barriers per 1024 intervals.  Two wavefronts a SIMD: with one (four intervals a thread)
// nothing hides the LDS latency, with four (one interval a thread) the scan is repeated by as many.
// Measured (kernel trace): four kernel sizes at budget 4096 on 32K tokens 11.4 us and five on 1M 20.2 us, where the predecessor took 15.0 and
// 19.5 us and two more kernels of 5.7 - 9.5 us each (one to write every kernel size's ranked tokens out, one to put the
// result in order); it walked single tokens through a hash set, a wavefront's round trip per token and probe.
constexpr int kWalkThreads = 512;
constexpr int kWalkWaves = kWalkThreads / 64;
constexpr int kWalkPer = 2;                                                   // intervals a thread looks at in one pass
constexpr int kWalkSpan = kWalkThreads * kWalkPer;                            // intervals per pass
constexpr int kWalkPasses = kCandCap / kWalkSpan;                             // passes a list may need
constexpr int kWalkAhead = 4;                                                 // cells: passes fetched ahead
static_assert(kCandCap % kWalkSpan == 0, "whole passes");
static_assert(ILRE_MAX_POOL_KERNELS <= 64, "a lane holds a combination's numbers");
constexpr int kRingBytes = kWalkAhead * kWalkSpan * (int)sizeof(uint32_t);    // also holds a 16-bit word number per place in the output
static_assert(kRingBytes >= ILRE_MAX_BUDGET * (int)sizeof(uint16_t) && (kWalkAhead & (kWalkAhead - 1)) == 0, "the ring's memory is used again");
static_assert(kBitmapTokens / 32 < 65536 && ILRE_MAX_BUDGET < 65536, "16-bit word numbers and places");

__device__ __forceinline__ uint32_t seed_count(const SeedState &s) { return s.refined ? s.refined : (uint32_t)s.lists_n + (uint32_t)(s.lists_n >> 32); }

// What the intervals of a list are.
enum WalkItems {
    kWalkSeeds,      // tokens owned by a seed: found from its position, its outranking neighbours and the window radius
    kWalkWordCells,  // cells of 1, 2, 4 .. 32 tokens: inside one word of the set
    kWalkCells       // cells of any size
};

struct WalkArgs {
    int n, n_out, sink;
    uint32_t len;                             // tokens of the body
    uint32_t share[ILRE_MAX_POOL_KERNELS];    // B_j
    uint32_t reach[ILRE_MAX_POOL_KERNELS];    // window radius, or tokens per cell
    uint32_t cells[ILRE_MAX_POOL_KERNELS];    // cells: length of the list (>= 1)
    const SeedState *seeds;                   // seeds: their number
    const uint32_t *pos, *dom;                // seeds, by rank: token, and the distances to its outranking neighbours
    const uint64_t *cand;                     // cells: per combination the ranked cells, uint32
    uint32_t *picked, *picked_n;              // HASHED: the allocated tokens in the order they are taken
    int32_t *out_idx, *out_count;
};

// the lowest `n` set bits of x
__device__ __forceinline__ uint32_t lowest_bits(uint32_t x, uint32_t n)
{
    uint32_t keep = 0;
    for (; n; --n) {
        keep |= x & (0u - x);
        x &= x - 1;
    }
    return keep;
}

// position of set bit number k (counted from 0) of x
__device__ __forceinline__ uint32_t nth_set_bit(uint32_t x, uint32_t k)
{
    uint32_t at = 0;
#pragma unroll
    for (int half = 16; half > 0; half >>= 1) {
        const uint32_t c = __popc(x & ((1u << half) - 1u));
        const bool up = k >= c;
        k -= up ? c : 0u;
        x >>= up ? half : 0;
        at += up ? half : 0;
    }
    return at;
}

// The allocated set in ascending order, read off its bitmap by the walk's workgroup.  slot_word: per place in the output the
// word (number + 1) whose first token goes there, or 0.
template <int THREADS>
__device__ __forceinline__ void emit_bitmap(const WalkArgs &a, const uint32_t *mask, uint16_t *slot_word, uint32_t *chunk_n, uint32_t nsel)
{
    constexpr int WAVES = THREADS / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t chunks = (a.len + 32 * kBitmapChunk - 1) / (32 * kBitmapChunk);
    // The tokens per chunk (a lane counts four neighbouring words) and
    // their running sum place every word's first token; the place notes the word.  Then one lane a place: the nearest
    // noted place at or before its own is at most 31 back and names the word, the distance the bit in it.
    // All of it is latency: kEmitBatch chunks (groups of 64 places) of a wavefront advance together.
    constexpr int kEmitBatch = 4;
    // Sixteen wavefronts take no more at a time than they have: chunks that are not there make their scans all the same, with four wavefronts a
    // SIMD in each other's way (48 combinations, budget 1000, the whole walk with eight wavefronts, sixteen in batches of four, so:
    // 116363 scores 19.7, 20.1, 19.1 us, 200000 19.8, 20.3, 19.6, 300000, still four, 21.2, 20.6, 20.6).
    auto by_batches = [&](auto loop) {
        if (WAVES == kWalkWaves || chunks > 2 * WAVES)  // uniform
            loop(std::integral_constant<int, kEmitBatch>{});
        else if (chunks > WAVES)
            loop(std::integral_constant<int, 2>{});
        else
            loop(std::integral_constant<int, 1>{});
    };
    __syncthreads();  // every wavefront is done with the set, and with what slot_word held
    for (uint32_t i = tid * 8; i < (uint32_t)a.n_out; i += THREADS * 8) *(uint4 *)&slot_word[i] = make_uint4(0, 0, 0, 0);
    auto words4 = [&](uint32_t c) {  // the lane's four words of a chunk, none past the last chunk
        return c < chunks ? *(const uint4 *)&mask[c * kBitmapChunk + 4 * lane] : make_uint4(0, 0, 0, 0);
    };
    auto count = [&](auto batch) {
        constexpr int BATCH = decltype(batch)::value;
        for (uint32_t c0 = wave; c0 < chunks; c0 += WAVES * BATCH) {
            uint32_t sum[BATCH];
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const uint4 x = words4(c0 + b * WAVES);
                sum[b] = __popc(x.x) + __popc(x.y) + __popc(x.z) + __popc(x.w);
            }
#pragma unroll
            for (int b = 0; b < BATCH; ++b) sum[b] = wave_scan_add(sum[b]);
#pragma unroll
            for (int b = 0; b < BATCH; ++b)
                if (lane == 63 && c0 + b * WAVES < chunks) chunk_n[c0 + b * WAVES] = sum[b];
        }
    };
    by_batches(count);
    __syncthreads();
    // every wavefront sums the chunks before each of its own by itself (lane l holds chunks l, l + 64, l + 128)
    uint32_t cn[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) cn[i] = (uint32_t)(lane + 64 * i) < chunks ? chunk_n[lane + 64 * i] : 0u;
    static_assert(kBitmapChunks <= 3 * 64, "three chunks a lane");
    auto note_places = [&](auto batch) {
        constexpr int BATCH = decltype(batch)::value;
        for (uint32_t c0 = wave; c0 < chunks; c0 += WAVES * BATCH) {
            uint4 x[BATCH];
            uint32_t n3[BATCH], at[BATCH];
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const uint32_t c = c0 + b * WAVES;
                x[b] = words4(c);
                n3[b] = __popc(x[b].x) + __popc(x[b].y) + __popc(x[b].z) + __popc(x[b].w);
                at[b] = ((uint32_t)lane < c ? cn[0] : 0u) + ((uint32_t)lane + 64 < c ? cn[1] : 0u) + ((uint32_t)lane + 128 < c ? cn[2] : 0u);
            }
#pragma unroll
            for (int b = 0; b < BATCH; ++b) at[b] = wave_total(wave_scan_add(at[b])) + wave_scan_add(n3[b]) - n3[b];
#pragma unroll
            for (int b = 0; b < BATCH; ++b) {
                const uint32_t w = (c0 + b * WAVES) * kBitmapChunk + 4 * lane;
                if (x[b].x) slot_word[at[b]] = (uint16_t)(w + 1);
                at[b] += __popc(x[b].x);
                if (x[b].y) slot_word[at[b]] = (uint16_t)(w + 2);
                at[b] += __popc(x[b].y);
                if (x[b].z) slot_word[at[b]] = (uint16_t)(w + 3);
                at[b] += __popc(x[b].z);
                if (x[b].w) slot_word[at[b]] = (uint16_t)(w + 4);
            }
        }
    };
    by_batches(note_places);
    __syncthreads();
    int32_t *out = a.out_idx + a.sink;
    // a wavefront's places lie side by side: the last note of one group of 64 serves the next
    const uint32_t span = (nsel + THREADS - 1) / THREADS * 64, s_begin = wave * span, s_end = min(s_begin + span, nsel);
    auto note_of = [&](uint32_t s) {  // place and word in one number, larger for a later place
        const uint32_t x = s < nsel ? slot_word[s] : 0u;
        return x ? (s & 0xFFFFu) << 16 | x : 0u;
    };
    uint32_t carry = 0;
    if (s_begin >= 64 && s_begin < nsel) carry = wave_total(wave_scan_max(note_of(s_begin - 64 + lane)));
    for (uint32_t s0 = s_begin; s0 < s_end; s0 += 64 * kEmitBatch) {
        uint32_t note[kEmitBatch], bits[kEmitBatch];
#pragma unroll
        for (int b = 0; b < kEmitBatch; ++b) note[b] = note_of(s0 + 64 * b + lane);
#pragma unroll
        for (int b = 0; b < kEmitBatch; ++b) note[b] = wave_scan_max(note[b]);
#pragma unroll
        for (int b = 0; b < kEmitBatch; ++b) {
            note[b] = max(note[b], carry);
            carry = wave_total(note[b]);
            bits[b] = mask[(note[b] & 0xFFFFu) - 1u];  // (place 0 is noted: there is always one)
        }
#pragma unroll
        for (int b = 0; b < kEmitBatch; ++b) {
            const uint32_t s = s0 + 64 * b + lane;
            if (s < s_end) out[s] = (int32_t)(((note[b] & 0xFFFFu) - 1u) * 32 + nth_set_bit(bits[b], s - (note[b] >> 16)) + (uint32_t)a.sink);
        }
    }
    for (uint32_t i = tid; i < (uint32_t)a.sink; i += THREADS) a.out_idx[i] = (int32_t)i;
    for (uint32_t i = nsel + tid; i < (uint32_t)a.n_out; i += THREADS) out[i] = -1;
    if (tid == 0 && a.out_count) *a.out_count = a.sink + (int32_t)nsel;
}

// `load` gives a thread its seeds of a pass; there are `nseeds`, in PASSES passes at most.
template <int ITEMS, bool HASHED, int PASSES, typename LOAD>
__device__ __forceinline__ void walk_items(const WalkArgs &a, unsigned char *smem, uint32_t nseeds, const LOAD &load)
{
    __shared__ uint32_t wsum[2][kWalkWaves], wlen[kWalkWaves];
    __shared__ uint32_t chunk_n[kBitmapChunks];
    constexpr bool SEEDS = ITEMS == kWalkSeeds;
    const TokenSet<HASHED> set{(uint32_t *)smem, (uint32_t *)smem + (HASHED ? kWordSlots : 0)};
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t chunks = (a.len + 32 * kBitmapChunk - 1) / (32 * kBitmapChunk);

    // combination j's numbers are lane j's: a readlane away, where memory would be a round trip per combination
    uint32_t l_share = a.share[lane], l_reach = a.reach[lane], l_cells = SEEDS ? 0u : a.cells[lane];
    asm volatile("" : "+v"(l_share), "+v"(l_reach), "+v"(l_cells));  // wait for them here, not behind every fetch of the loop
    auto of = [](uint32_t x, int j) { return (uint32_t)__builtin_amdgcn_readlane((int)x, j); };

    // The seeds serve every kernel size: a thread keeps the ones it looks at in registers.
    uint32_t seed[SEEDS ? PASSES : 1][kWalkPer], dom[SEEDS ? PASSES : 1][kWalkPer];
    if (SEEDS) {
#pragma unroll
        for (int p = 0; p < PASSES; ++p) {
            uint2 x, d;
            load(p * kWalkThreads + tid, x, d);
            seed[p][0] = x.x, seed[p][1] = x.y;
            dom[p][0] = d.x, dom[p][1] = d.y;
        }
        // (What lies behind the last one is told apart where it is used.  Here it would be a wait for all passes' loads, where the first kernel
        // size seldom looks beyond the first pass: recall of 32768 tokens 73.2 -> 72.5 us, of 100003, 28/4 heads 70.6 -> 69.8.)
    }
    const uint32_t clear = HASHED ? kWordSlots : chunks * kBitmapChunk;
    uint32_t *ring = set.mask + clear;  // cells: kWalkAhead passes of kWalkSpan cells
    // Cells come in a list per combination, written by other compute units a kernel ago: fetching one takes longer than
    // walking one, so kWalkAhead passes are under way, copied straight into LDS.  A wavefront fetches what its own
    // lanes look at, so its own wait is all the synchronisation there is.  (fj, fbase) is the next pass to fetch; past
    // the last one the last list is fetched again.
    const unsigned ring_lds = (unsigned)(size_t)(__attribute__((address_space(3))) uint32_t *)ring;
    int fj = 0;
    uint32_t fbase = 0;
    auto fetch = [&](int slot) {
        const unsigned long long list = (unsigned long long)((const uint32_t *)(a.cand + (size_t)fj * kCandCap) + fbase + wave * 64 * kWalkPer);
        i32x4 rsrc;
        rsrc[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)list);
        rsrc[1] = __builtin_amdgcn_readfirstlane((int)((unsigned)(list >> 32) & 0xFFFFu));
        rsrc[2] = 64 * kWalkPer * (int)sizeof(uint32_t);
        rsrc[3] = 0x00020000;
        if (lane < 64 * kWalkPer / 4)
            lds_dma16(rsrc, __builtin_amdgcn_readfirstlane(ring_lds + (unsigned)((slot * kWalkSpan + wave * 64 * kWalkPer) * sizeof(uint32_t))), lane * 16);
        fbase += kWalkSpan;
        if (fbase >= of(l_cells, fj)) {
            fbase = 0;
            if (fj + 1 < a.n) ++fj;
        }
    };
    // the oldest pass under way has arrived (HASHED: so have the notes, which are stores of the same counter)
    auto arrived = [&](int slot, uint32_t(&x)[kWalkPer]) {
        if (HASHED)
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        else
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kWalkAhead - 1) : "memory");
        const uint2 v = *(const uint2 *)&ring[slot * kWalkSpan + tid * kWalkPer];
        x[0] = v.x;
        x[1] = v.y;
    };
    if (!SEEDS && a.n > 0) {
#pragma unroll
        for (int d = 0; d < kWalkAhead; ++d) fetch(d);
    }

    for (uint32_t i = tid * 4; i < clear; i += kWalkThreads * 4) {
        if (HASHED) *(uint4 *)&set.key[i] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
        *(uint4 *)&set.mask[i] = make_uint4(0, 0, 0, 0);
    }
    lds_barrier();

    uint32_t nsel = 0, taken = 0, share = 0, reach = 0;
    bool wide = false;  // an interval may touch more than two words
    bool huge = false;  // HASHED: .. more than sixteen
    int gen = 0;
    auto start = [&](int j) {
        share = min(of(l_share, j), (uint32_t)a.n_out - nsel);
        reach = of(l_reach, j);
        wide = ITEMS != kWalkWordCells && (SEEDS ? 2 * reach + 1 : reach) > 33;
        huge = HASHED && wide && (SEEDS ? 2 * reach + 1 : reach) > 512;
        taken = 0;
    };
    // one pass: this thread's two neighbouring intervals, of which the ones from `cn` on (cells) do not exist
    auto pass = [&](uint32_t base, uint32_t cn, const uint32_t(&it)[kWalkPer], const uint32_t(&dm)[kWalkPer]) __attribute__((always_inline)) {
        uint32_t first[kWalkPer], last[kWalkPer], mask0[kWalkPer], mask1[kWalkPer], free0[kWalkPer], free1[kWalkPer], nfree[kWalkPer];
#pragma unroll
        for (int i = 0; i < kWalkPer; ++i) {
            bool some;
            if (SEEDS) {
                const SeedInterval own = seed_interval(base + tid * kWalkPer + i < nseeds, it[i], dm[i], reach, a.len);
                some = own.some;
                first[i] = own.first;
                last[i] = own.last;
            } else {
                some = base + tid * kWalkPer + i < cn;
                first[i] = some ? it[i] * reach : 0u;
                last[i] = first[i] + reach - 1;
            }
            if (ITEMS == kWalkWordCells) {
                mask0[i] = (0xFFFFFFFFu >> (32 - reach)) << (first[i] & 31);
            } else {
                mask0[i] = interval_bits(first[i] >> 5, first[i], last[i]);
                mask1[i] = some && last[i] >> 5 > first[i] >> 5 ? interval_bits((first[i] >> 5) + 1, first[i], last[i]) : 0u;
            }
            mask0[i] = some ? mask0[i] : 0u;
        }
        if (HASHED && wide) {  // uniform
            // Of intervals this long few fill a share, and each costs a probe per word: those behind as many tokens as the share
            // and the tokens allocated so far are together cannot matter.
            const uint32_t len0 = mask0[0] ? last[0] - first[0] + 1 : 0u, len1 = mask0[1] ? last[1] - first[1] + 1 : 0u;
            const uint32_t upto = wave_scan_add(len0 + len1);
            if (lane == 63) wlen[wave] = upto;
            lds_barrier();
            uint32_t ahead = upto - len0 - len1;
#pragma unroll
            for (int w = 0; w < kWalkWaves; ++w) ahead += w < wave ? wlen[w] : 0u;
            if (ahead >= share + nsel) mask0[0] = mask1[0] = 0u;
            if (ahead + len0 >= share + nsel) mask0[1] = mask1[1] = 0u;
        }
#pragma unroll
        for (int i = 0; i < kWalkPer; ++i) {
            free0[i] = set.get(first[i] >> 5);
            if (ITEMS != kWalkWordCells) free1[i] = set.get(min((first[i] >> 5) + 1, last[i] >> 5));
        }
#pragma unroll
        for (int i = 0; i < kWalkPer; ++i) {
            free0[i] = ~free0[i] & mask0[i];
            nfree[i] = __popc(free0[i]);
            if (ITEMS != kWalkWordCells) {
                free1[i] = ~free1[i] & mask1[i];
                nfree[i] += __popc(free1[i]);
            }
        }
        // Words beyond the second.  A lane goes through its interval's, but in the table, where each is a probe, a mark and up to 32
        // notes, the wavefront takes huge intervals one at a time, a word a lane (at most 2047 tokens: 63 words).  One window of
        // 2047 on 3M tokens, the whole call: 300 us a lane alone, 108 so; 64 windows of up to 127: 325 and 1000 us.
        auto long_ones = [&](int i, bool some, auto each) {
            for (uint64_t todo = __ballot(some && last[i] >> 5 > (first[i] >> 5) + 1); todo; todo &= todo - 1) {
                const int of_lane = __ffsll((unsigned long long)todo) - 1;
                const uint32_t f = of(first[i], of_lane), l = of(last[i], of_lane), w = (f >> 5) + 2 + lane;
                each(of_lane, w, w <= l >> 5 ? ~set.get(w) & interval_bits(w, f, l) : 0u);
            }
        };
        static_assert(ILRE_MAX_POOL_KERNEL <= 2047 && ILRE_MAX_MAX_KERNEL <= 2047, "an interval's words beyond the second are no more than lanes");
        if (wide) {  // uniform
#pragma unroll
            for (int i = 0; i < kWalkPer; ++i) {
                if (huge)
                    long_ones(i, mask0[i] != 0, [&](int of_lane, uint32_t, uint32_t bits) {
                        const uint32_t n = wave_total(wave_scan_add((uint32_t)__popc(bits)));
                        nfree[i] += lane == of_lane ? n : 0u;
                    });
                else if (mask0[i])
                    for (uint32_t w = (first[i] >> 5) + 2; w <= last[i] >> 5; ++w) nfree[i] += __popc(~set.get(w) & interval_bits(w, first[i], last[i]));
            }
        }
        const uint32_t mine = nfree[0] + nfree[1];
        static_assert(kWalkPer == 2, "two intervals a thread");
        const uint32_t upto = wave_scan_add(mine);
        if (lane == 63) wsum[gen][wave] = upto;
        lds_barrier();
        // the wavefronts' totals, one a lane, summed along the row of eight
        static_assert(kWalkWaves == 8, "three steps sum eight wavefronts' totals");
        uint32_t ws = wsum[gen][lane & (kWalkWaves - 1)];
        ws += (uint32_t)ILRE_DPP(0, ws, 0x111, 0xF);
        ws += (uint32_t)ILRE_DPP(0, ws, 0x112, 0xF);
        ws += (uint32_t)ILRE_DPP(0, ws, 0x114, 0xF);
        const uint32_t total = of(ws, kWalkWaves - 1);
        uint32_t before = upto - mine + (wave ? of(ws, wave - 1) : 0u);
        gen ^= 1;
        const uint32_t room = share - taken;
        auto note = [&](uint32_t w, uint32_t bits, uint32_t &at) {  // only where the output cannot be read off the set
            for (; bits; bits &= bits - 1) a.picked[at++] = w * 32 + (uint32_t)__ffs((int)bits) - 1;
        };
#pragma unroll
        for (int i = 0; i < kWalkPer; ++i) {
            const uint32_t w0 = first[i] >> 5;
            uint32_t quota = room > before ? room - before : 0u, at = nsel + taken + before;
            if (quota < nfree[i]) {  // the share ends in (or before) this interval: the lowest tokens of it are taken
                const uint32_t c0 = __popc(free0[i]);
                if (quota < c0) free0[i] = lowest_bits(free0[i], quota);
                if (ITEMS != kWalkWordCells) free1[i] = quota > c0 ? lowest_bits(free1[i], min(quota - c0, (uint32_t)__popc(free1[i]))) : 0u;
            }
            if (free0[i]) set.set(w0, free0[i]);
            if (HASHED) note(w0, free0[i], at);
            if (ITEMS != kWalkWordCells) {
                if (free1[i]) set.set(w0 + 1, free1[i]);
                if (HASHED) note(w0 + 1, free1[i], at);
                if (wide) {  // uniform
                    uint32_t more = mask0[i] ? min(quota, nfree[i]) - __popc(free0[i]) - __popc(free1[i]) : 0u;
                    if (huge)
                        long_ones(i, more != 0, [&](int of_lane, uint32_t w, uint32_t bits) {
                            const uint32_t n = __popc(bits), ahead = wave_scan_add(n) - n, want = of(more, of_lane);
                            const uint32_t take = want > ahead ? min(n, want - ahead) : 0u;
                            if (take < n) bits = lowest_bits(bits, take);
                            if (bits) set.set(w, bits);
                            uint32_t place = of(at, of_lane) + ahead;
                            note(w, bits, place);
                        });
                    else
                        for (uint32_t w = w0 + 2; more; ++w) {
                            uint32_t bits = ~set.get(w) & interval_bits(w, first[i], last[i]);
                            if ((uint32_t)__popc(bits) > more) bits = lowest_bits(bits, more);
                            more -= __popc(bits);
                            if (bits) set.set(w, bits);
                            if (HASHED) note(w, bits, at);
                        }
                }
            }
            before += nfree[i];
        }
        taken += min(total, room);
    };
    if (SEEDS) {
        for (int j = 0; j < a.n; ++j) {
            start(j);
#pragma unroll
            for (int p = 0; p < PASSES; ++p)
                if (taken < share && (uint32_t)(p * kWalkSpan) < nseeds) pass(p * kWalkSpan, 0, seed[p], dom[p]);
            nsel += taken;
            lds_barrier();  // the set is complete before the next kernel size counts in it
        }
    } else {
        uint32_t base = 0, it[kWalkPer];
        int j = 0, slot = 0;
        if (a.n > 0) {
            start(0);
            arrived(0, it);
        }
        while (j < a.n) {
            const uint32_t cn = of(l_cells, j);
            if (taken < share) pass(base, cn, it, dom[0]);
            fetch(slot);
            slot = (slot + 1) & (kWalkAhead - 1);
            arrived(slot, it);
            base += kWalkSpan;
            if (base >= cn) {  // the list is done
                nsel += taken;
                lds_barrier();
                base = 0;
                if (++j < a.n) start(j);
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // nothing writes into the ring any more
    }
    if (HASHED) {
        if (tid == 0) *a.picked_n = nsel;
        return;
    }

    emit_bitmap<kWalkThreads>(a, set.mask, (uint16_t *)ring, chunk_n, nsel);
}

template <int ITEMS, bool HASHED>
__global__ __launch_bounds__(kWalkThreads) void allocate_walk(const WalkArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    walk_items<ITEMS, HASHED, kWalkPasses>(a, smem, ITEMS == kWalkSeeds ? seed_count(*a.seeds) : 0u, [&](int r2, uint2 &x, uint2 &d) {
        x = ((const uint2 *)a.pos)[r2];
        d = ((const uint2 *)a.dom)[r2];
    });
}

// The same walk where many combinations share the budget: the wavefronts take turns, a combination each, and nothing but the
// turn itself is serial.  Until it has the turn a wavefront sorts out its list on its own: cells whose tokens are all
// allocated already stay so, whatever the others do meanwhile, and are dropped, first from the whole list (while the seven before
// it have their turns), again from the front of what is left when its turn is near.  With the turn it looks at the first
// cells left once more: one gather, one scan and the marks for the usual share, without a barrier.  What was dropped before only
// saves time, the turn decides on what the set holds then.
// Bound: the chain of a turn, about 650 cycles, half of them LDS round trips (see the turn, fetch the words, mark, pass it on),
// where a pass of the workgroup over the whole list took 1300.  Measured (kernel trace), 48 combinations: 9001 tokens, budget
// 1000 33.9 -> 19.7 us; 1M, budget 4096 40.8 -> 26.5 us.
constexpr int kRelayCombos = 4;                                 // from that many combinations on, and where ..
constexpr uint32_t kRelayShare = 96, kRelayShareTable = 48;      // .. no share is more cells (with the word table)
constexpr int kRelayRaw = 16;                                   // cells of a list a lane fetches ahead
constexpr int kRelayKept = kRingBytes / 4 / kWalkWaves;         // cells a wavefront keeps
// Eight wavefronts take turns, sixteen clear the set and read it off at the end (1M scores, 48 combinations 26.5 -> 24.4 us, 9001 19.4 -> 18.7).
constexpr int kRelayThreads = 1024;
constexpr uint32_t kRelayChunk = 64 * kWalkPer;                 // cells it looks at at a time with the turn
template <bool HASHED>
__global__ __launch_bounds__(kRelayThreads) void allocate_relay(const WalkArgs a)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t chunk_n[kBitmapChunks];
    __shared__ uint32_t turn;  // whose turn it is, and the number of tokens allocated, above 8 bits
    const TokenSet<HASHED> set{(uint32_t *)smem, (uint32_t *)smem + (HASHED ? kWordSlots : 0)};
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t chunks = (a.len + 32 * kBitmapChunk - 1) / (32 * kBitmapChunk);
    const uint32_t clear = HASHED ? kWordSlots : chunks * kBitmapChunk;
    uint32_t *ring = set.mask + clear, *kept = ring + wave * kRelayKept;

    uint32_t l_share = a.share[lane], l_reach = a.reach[lane], l_cells = a.cells[lane];
    asm volatile("" : "+v"(l_share), "+v"(l_reach), "+v"(l_cells));
    auto of = [](uint32_t x, int j) { return (uint32_t)__builtin_amdgcn_readlane((int)x, j); };
    auto list_of = [&](int j) { return (const uint32_t *)(a.cand + (size_t)j * kCandCap); };
    uint32_t raw[kRelayRaw];
    auto fetch = [&](int j) {
        const uint32_t cn = of(l_cells, j);
#pragma unroll
        for (int k = 0; k < kRelayRaw; ++k)
            if (64u * k < cn) raw[k] = list_of(j)[min(64u * k + lane, cn - 1)];  // uniform
    };
    if (wave < kWalkWaves && wave < a.n) fetch(wave);
    for (uint32_t i = tid * 4; i < clear; i += kRelayThreads * 4) {
        if (HASHED) *(uint4 *)&set.key[i] = make_uint4(kEmpty, kEmpty, kEmpty, kEmpty);
        *(uint4 *)&set.mask[i] = make_uint4(0, 0, 0, 0);
    }
    if (tid == 0) turn = 0;
    __syncthreads();
    auto whose = [&]() { return __hip_atomic_load(&turn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP); };

    for (int j = wave < kWalkWaves ? wave : a.n; j < a.n; j += kWalkWaves) {
        const uint32_t cn = of(l_cells, j), reach = of(l_reach, j), ones = 0xFFFFFFFFu >> (32 - reach);
        const uint32_t *list = list_of(j);
        auto word_of = [&](uint32_t c) { return c * reach >> 5; };
        auto bits_of = [&](uint32_t c) { return ones << (c * reach & 31); };
        auto keep = [&](uint32_t c, bool some, uint32_t &n) {  // the next of the cells kept
            const uint64_t mask = __ballot(some);
            const uint32_t at = n + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
            if (some) kept[at] = c;
            n += (uint32_t)__popcll(mask);
        };
        // the list's cells that still have something free
        uint32_t n = 0, seen = 0;  // kept; cells of the list looked at
        {
            uint32_t word[kRelayRaw];
#pragma unroll
            for (int k = 0; k < kRelayRaw; ++k)
                if (64u * k < cn) word[k] = set.get(word_of(raw[k]));  // uniform
#pragma unroll
            for (int k = 0; k < kRelayRaw; ++k) {
                if (64u * k < cn && n + 64 <= (uint32_t)kRelayKept) {  // uniform
                    keep(raw[k], (64u * k + lane < cn) & ((~word[k] & bits_of(raw[k])) != 0), n);
                    seen = min(64u * (k + 1), cn);
                }
            }
        }
        if (j + kWalkWaves < a.n) fetch(j + kWalkWaves);
        // close to its turn: once more, as many as it looks at at a time
        while ((int)(whose() & 255u) < j - 2) __builtin_amdgcn_s_sleep(1);
        uint32_t front = 0, rest = 0;
        for (; rest < n && front < kRelayChunk; rest += 64) {
            const uint32_t c = kept[min(rest + lane, n - 1)];
            keep(c, (rest + lane < n) & ((~set.get(word_of(c)) & bits_of(c)) != 0), front);
        }
        // Two neighbouring cells a lane: their words of the set, the bits of their tokens, and what is free.
        uint32_t word[kWalkPer], bits[kWalkPer], free[kWalkPer];
        static_assert(kWalkPer == 2, "two cells a lane");
        auto look = [&](uint2 c, uint32_t left) __attribute__((always_inline)) {
            word[0] = word_of(c.x), word[1] = word_of(c.y);
            bits[0] = lane * 2 < left ? bits_of(c.x) : 0u, bits[1] = lane * 2 + 1 < left ? bits_of(c.y) : 0u;
            word[0] = bits[0] ? word[0] : 0u, word[1] = bits[1] ? word[1] : 0u;
            asm volatile("" : "+v"(word[0]), "+v"(word[1]), "+v"(bits[0]), "+v"(bits[1]));  // (now, not when they are used)
        };
        uint32_t nsel = 0, taken = 0, share = 0;
        auto take = [&]() __attribute__((always_inline)) {
            free[0] = ~free[0] & bits[0], free[1] = ~free[1] & bits[1];
            const uint32_t n0 = __popc(free[0]), n1 = __popc(free[1]);
            const uint32_t upto = wave_scan_add(n0 + n1), total = wave_total(upto), room = share - taken;
            if (HASHED || total > room) {  // uniform: the share ends here
                const uint32_t before = upto - n0 - n1;
                const uint32_t q0 = room > before ? room - before : 0u, q1 = room > before + n0 ? room - before - n0 : 0u;
                free[0] = q0 ? free[0] : 0u, free[1] = q1 ? free[1] : 0u;
                // in the cell where it ends the lowest tokens are taken: lane i counts the free ones below token i
                const bool here0 = (q0 != 0) & (q0 < n0), here1 = (q1 != 0) & (q1 < n1);
                const uint64_t ends = __ballot(here0 | here1);
                if (ends) {  // uniform
                    const int l = __ffsll((unsigned long long)ends) - 1;
                    const uint32_t x = of(here0 ? free[0] : free[1], l), q = of(here0 ? q0 : q1, l);
                    const uint32_t some = (uint32_t)__ballot((x >> (lane & 31) & 1u) & (__builtin_amdgcn_mbcnt_lo(x, 0u) < q ? 1u : 0u));
                    free[0] = here0 ? some : free[0];
                    free[1] = here1 ? some : free[1];
                }
                if (HASHED) {
                    uint32_t place = nsel + taken + before;
#pragma unroll
                    for (int i = 0; i < kWalkPer; ++i)
                        for (uint32_t x = free[i]; x; x &= x - 1) a.picked[place++] = word[i] * 32 + (uint32_t)__ffs((int)x) - 1;
                }
            }
            if (free[0]) set.set(word[0], free[0]);
            if (free[1]) set.set(word[1], free[1]);
            taken += min(total, room);
        };
        look(*(const uint2 *)&kept[2 * lane], front);
        __builtin_amdgcn_s_setprio(3);
        // (a wavefront's LDS operations are performed in order: the words are read after the turn is, and the turn is
        // passed on after the marks)
        uint32_t now;
        do {
            now = whose();
            asm volatile("" ::: "memory");
            free[0] = set.get(word[0]), free[1] = set.get(word[1]);
            asm volatile("" : "+v"(free[0]), "+v"(free[1]));
            now = (uint32_t)__builtin_amdgcn_readfirstlane((int)now);
        } while ((int)(now & 255u) != j);
        nsel = now >> 8;
        share = min(of(l_share, j), (uint32_t)a.n_out - nsel);
        take();
        if (taken < share) {
            // the cells behind them, and those of the list that were not looked at
            uint32_t at = kRelayChunk, end = front;
            if (at >= front) at = rest, end = n;
            while (taken < share && at < n) {
                look(make_uint2(kept[min(at + 2 * lane, end - 1)], kept[min(at + 2 * lane + 1, end - 1)]), end - at);
                free[0] = set.get(word[0]), free[1] = set.get(word[1]);
                take();
                at += kRelayChunk;
                if (at >= end && end == front) at = rest, end = n;
            }
            for (; taken < share && seen < cn; seen += kRelayChunk) {
                look(make_uint2(list[min(seen + 2 * lane, cn - 1)], list[min(seen + 2 * lane + 1, cn - 1)]), cn - seen);
                free[0] = set.get(word[0]), free[1] = set.get(word[1]);
                take();
            }
        }
        nsel += taken;
        asm volatile("" ::: "memory");
        if (lane == 0) __hip_atomic_store(&turn, (nsel << 8) | (uint32_t)(j + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_s_setprio(0);
    }
    __syncthreads();
    const uint32_t nsel = turn >> 8;
    if (HASHED) {
        if (tid == 0) *a.picked_n = nsel;
        return;
    }
    emit_bitmap<kRelayThreads>(a, set.mask, (uint16_t *)ring, chunk_n, nsel);
}


// ---------------------------------------------------------------- window-max form: seeds

// Per seed (one of the ns best raw scores, keys distinct): its rank = the number of seeds with a larger key, and
// the distances to the nearest token on either side, within `reach` tokens, whose key is larger (such a token is
// itself a seed, the seeds being the best keys; kNoDom if there is none).  Written in rank order, the two distances
// as the halves of a word.  A wavefront owns four seeds.  For the count its
// lanes read disjoint parts of the staged key list (every LDS word is fetched once per wavefront) and
// compare them with all four keys; for the scan 16 lanes share a seed and split its neighbourhood.
constexpr int kSeedRankThreads = 512;  // 32 seeds a workgroup
constexpr uint32_t kNoDom = 0x7FFF;    // farther than two radii: binds no kernel size
static_assert(kNoDom > ILRE_MAX_POOL_KERNEL, "reach is twice the largest radius");
__global__ __launch_bounds__(kSeedRankThreads) void seed_rank(const float *scores, int64_t L, const SeedState *st, const uint64_t *cand,
                                                              const uint64_t *tie, int reach, uint32_t *by_rank, uint32_t *dom)
{
    extern __shared__ __align__(16) unsigned char smem[];
    uint64_t *all = (uint64_t *)smem;  // every seed's key, staged once per workgroup (kCandCap at most)
    const uint32_t ns = seed_count(*st), nc = st->refined ? ns : (uint32_t)st->lists_n;
    if (blockIdx.x * (kSeedRankThreads / 16) >= ns) return;  // uniform
    // (the seeds were written by earlier kernels: plain loads, all in flight together)
    stage_to_lds<uint64_t, kSeedRankThreads>(all, cand, nc);
    if (nc < ns) stage_to_lds<uint64_t, kSeedRankThreads>(all + nc, tie, ns - nc);
    const uint32_t padded = (ns + 127u) & ~127u;  // whole rounds of 64 lanes x 2 keys; the padding outranks nothing
    if (threadIdx.x < 128 && ns + threadIdx.x < padded) all[ns + threadIdx.x] = 0ull;
    __syncthreads();
    const int lane = threadIdx.x & 63;
    const uint32_t u0 = blockIdx.x * (kSeedRankThreads / 16) + (threadIdx.x >> 6) * 4;  // the wavefront's first seed
    if (u0 >= ns) return;  // whole wavefronts leave together, no barrier follows
    uint64_t wkey[4];
    uint32_t wcnt[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const uint64_t k = all[u0 + q < ns ? u0 + q : ns - 1];
        wkey[q] = ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)(k >> 32)) << 32) |
                  (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(uint32_t)k);
        wcnt[q] = 0;
    }
#pragma unroll 2
    for (uint32_t v = 2u * lane; v < padded; v += 128) {
        const uint4 x = *(const uint4 *)&all[v];
        const uint64_t k0 = ((uint64_t)x.y << 32) | x.x, k1 = ((uint64_t)x.w << 32) | x.z;
#pragma unroll
        for (int q = 0; q < 4; ++q) wcnt[q] += (k0 > wkey[q] ? 1u : 0u) + (k1 > wkey[q] ? 1u : 0u);
    }
    uint32_t wtot[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) wtot[q] = wave_total(wave_scan_add(wcnt[q]));
    const int grp = lane >> 4;
    const uint32_t u = u0 + grp;
    const int sub = lane & 15;
    if (u >= ns) return;  // whole 16-lane groups leave together
    const uint64_t key = grp == 0 ? wkey[0] : (grp == 1 ? wkey[1] : (grp == 2 ? wkey[2] : wkey[3]));
    const uint32_t cnt = grp == 0 ? wtot[0] : (grp == 1 ? wtot[1] : (grp == 2 ? wtot[2] : wtot[3]));
    const int64_t pos = (int64_t)key_token(key);
    // nearest outranking token: distance d = 1 .. reach, 16 distances a round, both sides at once
    uint32_t left = kNoDom, right = kNoDom;
    for (int d0 = 1; d0 <= reach; d0 += 16) {
        const int d = d0 + sub;
        const int64_t pl = pos - d, pr = pos + d;
        const bool hit_l = d <= reach && pl >= 0 && make_key(scores[pl < 0 ? 0 : pl], (uint32_t)(pl < 0 ? 0 : pl)) > key;
        const bool hit_r = d <= reach && pr < L && make_key(scores[pr < L ? pr : L - 1], (uint32_t)(pr < L ? pr : L - 1)) > key;
        // lowest lane of this 16-lane group with a hit = smallest distance
        const uint64_t bl = __ballot(left == kNoDom && hit_l), br = __ballot(right == kNoDom && hit_r);
        const int shift = (threadIdx.x & 63) & ~15;
        const uint32_t ml = (uint32_t)(bl >> shift) & 0xFFFFu, mr = (uint32_t)(br >> shift) & 0xFFFFu;
        if (left == kNoDom && ml) left = (uint32_t)(d0 + __ffs((int)ml) - 1);
        if (right == kNoDom && mr) right = (uint32_t)(d0 + __ffs((int)mr) - 1);
        if (left != kNoDom && right != kNoDom) break;  // uniform within the group; ballots are wave-wide but only read per group
    }
    if (sub == 15) {
        by_rank[cnt] = (uint32_t)pos;
        dom[cnt] = left | (right << 16);
    }
}

// Window-max form, short contexts: the whole selection in one launch of one workgroup, with the last scoring step where it is
// fused (as in reduce_count).  The scores' keys stay in registers and in LDS: the seeds are cut and ranked there, a
// thread a seed looks for its outranking neighbours, eight wavefronts walk.
// Bound: latency (loads, a few dozen barriers), where the launches it replaces each start with memory round trips of their own.
// Measured (whole calls, budget a quarter of the tokens at most): selection alone 4096 tokens, budget 256 28.3 -> 15 us, 16384, 256
// 28.3 -> 21, 16384, 2048 29.6 -> 28.2; in a recall 1000 tokens 29.6 -> 23.9 us, 4096 41.8 -> 32.7, 8192, budget 2000 46.7 -> 44.5, and
// 16384 50.4 -> 57.8, which is why a recall's limit is lower.  One compute unit adds up 8 vectors of 4096 partial scores in the time of a
// launch (more are added up before it: 8 of 8192 45.9 -> 44.5 us).
constexpr int kBriefTokens = 16384, kBriefFused = 8192, kBriefSeeds = 2048, kBriefReach = 64;
constexpr int64_t kBriefPartial = 32768;  // partial scores that the one workgroup adds up itself
constexpr int kBriefSpare = 1024;  // seeds' keys beyond the wanted ones that may be sorted with them
constexpr size_t brief_lds(int64_t len)
{
    const size_t bitmap = ((size_t)len + 32 * kBitmapChunk - 1) / (32 * kBitmapChunk) * kBitmapChunk * 4;
    return bitmap + kRingBytes + 2 * kBriefSeeds * 4 + 2 * kBriefSeeds * 8 + (size_t)len * 4;
}
template <int PER>
__global__ __launch_bounds__(kThreads) void select_brief(const float *partial, int nunits, int rmax, float *score, const float *body, int sink, uint32_t want,
                                                         int reach, const WalkArgs w)
{
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ __align__(16) RankShared sh;
    static_assert(kBriefSeeds + kBriefSpare <= 2 * kBriefSeeds, "the keys fit");
    const int tid = threadIdx.x;
    const uint32_t len = w.len, bitmap = (len + 32 * kBitmapChunk - 1) / (32 * kBitmapChunk) * kBitmapChunk;
    uint32_t *ranked = (uint32_t *)smem + bitmap + kRingBytes / 4, *dom = ranked + kBriefSeeds;
    uint64_t *srt = (uint64_t *)(dom + kBriefSeeds);
    uint32_t *bits = (uint32_t *)(srt + 2 * kBriefSeeds);  // every token's ordered score
    uint32_t value[PER], have = 0;
    float v[PER];
    if (partial) {  // uniform
        const uint32_t L = len + (uint32_t)sink;
        constexpr int kUnits = 64 / PER < 16 ? 64 / PER : 16;  // units whose loads are in flight together
        for (int u0 = 0; u0 < nunits; u0 += kUnits) {
            float x[kUnits][PER];
#pragma unroll
            for (int uu = 0; uu < kUnits; ++uu)
#pragma unroll
                for (int k = 0; k < PER; ++k)
                    x[uu][k] = partial[(size_t)(u0 + uu < nunits ? u0 + uu : nunits - 1) * L + min((uint32_t)(tid + k * kThreads), L - 1)];
#pragma unroll
            for (int uu = 0; uu < kUnits; ++uu) {
                if (u0 + uu >= nunits) break;  // uniform
#pragma unroll
                for (int k = 0; k < PER; ++k) v[k] = u0 + uu == 0 ? x[uu][k] : (rmax ? fmaxf(v[k], x[uu][k]) : v[k] + x[uu][k]);
            }
        }
#pragma unroll
        for (int k = 0; k < PER; ++k)
            if ((uint32_t)(tid + k * kThreads) < L) score[tid + k * kThreads] = v[k];
    } else {
#pragma unroll
        for (int k = 0; k < PER; ++k) v[k] = body[min((uint32_t)(tid + k * kThreads), len - 1)];
    }
    const int first = tid - (partial ? sink : 0);  // token of the body
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        const int t = first + k * kThreads;
        value[k] = ordered_bits(v[k]);
        if (t >= 0 && t < (int)len) {
            bits[t] = value[k];
            have |= 1u << k;
        }
    }
    auto key = [&](int k) { return (uint64_t)value[k] << 32 | (0xFFFFFFFFu - (uint32_t)(first + k * kThreads)); };  // as make_key
    const uint32_t subset = narrow<PER>(sh, key, have, want, kBriefSpare);
    uint32_t top = 0, low = 0xFFFFFFFFu, total;
    uint64_t keys[PER];
#pragma unroll
    for (int k = 0; k < PER; ++k) {
        keys[k] = key(k);
        if (subset >> k & 1u) top = max(top, value[k]), low = min(low, value[k]);
    }
    rank_range(sh, top, low);
    if (!rank_keys(sh, srt, keys, subset, top, low, want, ranked, total)) rank_network(srt, total, want, ranked);
    __syncthreads();
    // The distances to the nearest tokens that outrank a seed.  Those are seeds too: a thread goes through the seeds on either side,
    // near ones first, by a bitmap of them (of the seed's own score only those before it outrank it).
    uint32_t *seeds = (uint32_t *)smem;
    for (uint32_t i = tid; i < bitmap; i += kThreads) seeds[i] = 0;
    __syncthreads();
    for (uint32_t r = tid; r < want; r += kThreads) atomicOr(&seeds[ranked[r] >> 5], 1u << (ranked[r] & 31));
    __syncthreads();
    for (uint32_t r = tid; r < want; r += kThreads) {
        const uint32_t at = ranked[r], mine = bits[at], o = at & 31;
        const int w = (int)(at >> 5);
        auto word = [&](int i) { return (uint64_t)(i >= 0 && i < (int)bitmap ? seeds[max(min(i, (int)bitmap - 1), 0)] : 0u); };
        const uint64_t here = word(w);
        static_assert(kBriefReach <= 64, "a bit a token");
        // bit 63: the token before, bit 0: the one behind
        uint64_t l = (word(w - 1) << 32 | word(w - 2)) >> o | (o ? here << (64 - o) : 0ull);
        uint64_t e = (word(w + 1) << 32 | here) >> (o + 1) | word(w + 2) << (63 - o);
        l = reach ? l & ~0ull << (64 - reach) : 0ull;
        e = reach ? e & ~0ull >> (64 - reach) : 0ull;
        uint32_t left = kNoDom, right = kNoDom;
        while (l | e) {
            const uint32_t dl = l ? (uint32_t)__clzll((long long)l) + 1 : 0u, de = e ? (uint32_t)__ffsll((unsigned long long)e) : 0u;
            const uint32_t vl = bits[at - dl], ve = bits[at + de];
            if (dl) {
                const bool found = vl >= mine;
                left = found ? dl : left;
                l = found ? 0ull : l & ~(1ull << (64 - dl));
            }
            if (de) {
                const bool found = ve > mine;
                right = found ? de : right;
                e = found ? 0ull : e & (e - 1);
            }
        }
        dom[r] = left | right << 16;
    }
    __syncthreads();
    if (tid >= kWalkThreads) return;  // whole wavefronts; barriers count those that are left
    walk_items<kWalkSeeds, false, kBriefSeeds / kWalkSpan>(w, smem, want, [&](int r2, uint2 &x, uint2 &d) {
        x = ((const uint2 *)ranked)[r2];
        d = ((const uint2 *)dom)[r2];
    });
}

// Last line of Algorithm 1: the input IDs of the allocated tokens, C[I].  Unused index slots (-1) give -1.
__global__ __launch_bounds__(kPoolThreads) void gather_ids_kernel(const int32_t *ids, int64_t L, const int32_t *idx, int n,
                                                                  int32_t *out)
{
    const int i = blockIdx.x * kPoolThreads + threadIdx.x;
    if (i >= n) return;
    const int32_t t = idx[i];
    out[i] = (t >= 0 && t < L) ? ids[t] : -1;
}

}  // namespace

hipError_t launch_gather_ids(const int32_t *ids, int64_t L, const int32_t *idx, int n, int32_t *out, hipStream_t s)
{
    hipLaunchKernelGGL(gather_ids_kernel, dim3((n + kPoolThreads - 1) / kPoolThreads), dim3(kPoolThreads), 0, s, ids, L, idx, n, out);
    return hipGetLastError();
}

// Elements of combination j's source array and the tokens one element stands for.
static void combo_shape(const SelectJob &job, int j, int64_t &len, int &cell)
{
    if (job.mode == kSelMaxAvg) {
        cell = job.max_kernels[j / job.n_avg];
        len = job.L / cell;
    } else {
        cell = 1;
        len = job.L;
    }
}

SelectLayout make_select_layout(const SelectJob &job)
{
    auto up = [](size_t x) { return (x + 255) & ~(size_t)255; };
    SelectLayout lay{};
    const int n = job.combos() > 0 ? job.combos() : 1;
    const bool window = job.mode == kSelWindowMax;
    const int nh = window ? 1 : n;
    const size_t nfine = window ? (size_t)((job.L + kSelFine - 1) / kSelFine) : 0;
    size_t off = 0;
    lay.state = off;
    off = up(off + (window ? 2 * sizeof(SeedState) : 0));
    lay.hist = off;
    off = up(off + (window ? 0 : (size_t)n * kAvgBins * sizeof(uint32_t)));
    lay.ctrl = off;
    off = up(off + (window ? 0 : (size_t)n * sizeof(SelCtrl)));
    lay.done = off;
    off = up(off + (window ? 0 : (size_t)n * sizeof(uint32_t)));
    lay.cmax = off;
    off = up(off + nfine * sizeof(float));
    lay.active = off;
    off = up(off + nfine * sizeof(uint32_t));
    lay.cells = off;
    size_t ncell = 0, ntie = 0;
    if (!window) {
        for (int i = 0; i < job.n_max; ++i) ncell += (size_t)(job.L / job.max_kernels[i]);
        ntie = 2 * ncell * (size_t)job.n_avg;
    } else {
        ntie = 2 * (size_t)job.L;
    }
    off = up(off + ncell * sizeof(float));
    lay.picked = off;
    off = up(off + ((size_t)ILRE_MAX_BUDGET + 64) * sizeof(uint32_t));
    lay.seed = off;
    off = up(off + (window ? 2 * (size_t)kCandCap * sizeof(uint32_t) : 0));
    lay.cand = off;
    off = up(off + (size_t)nh * kCandCap * sizeof(uint64_t));
    lay.tie = off;
    off = up(off + ntie * sizeof(uint64_t));
    lay.total = off;
    return lay;
}

namespace {

template <int PASS, int PER, bool SMALL>
hipError_t raise_avg_lds()
{
    return hipFuncSetAttribute((const void *)pool_averages<PASS, PER, SMALL>, hipFuncAttributeMaxDynamicSharedMemorySize,
                               (int)avg_lds(PASS, PER, SMALL, kAvgGroup, SMALL ? kAvgGroup : ILRE_MAX_AVG_KERNEL));
}

// One chunk of windows a wavefront where that is at most two workgroups a compute unit, more of them beyond: a
// workgroup carries the clearing and flushing of its 16 KiB of counts, and all want the same lines of the global ones.  Of chunks of
// kAvgWide up to two a wavefront with one workgroup a compute unit (whole selection, budget 4096, 1M scores, two workgroups -> one: 48
// combinations, three draws of a background with a few dozen spans far above it, whose places decide how many elements share a bin and a
// list, 89.4 -> 86.8, 69.9 -> 68.6 and 67.7 -> 67.8 us, uniform scores 69.2 -> 67.3; cells of 1, windows of 7, the same draws 74.0 -> 71.3, 64.7
// -> 61.8, 58.5 -> 57.6; 4M scores, up to seven chunks, 148.9 -> 154.5; chunks of kAvgNarrow, 20 combinations of 512K 68.1 -> 72.5).
// Max kernels get workgroups in proportion to their cells (as many each, cells of 2 had four times as much a workgroup as cells
// of 8: 48 combinations 4M scores 173.7 -> 160.3 us; max kernels 1, 2, 4, 8, 16 with four others 1M 142.5 -> 109.7; 64 max kernels 1M 355 -> 231).
template <int PASS, int PER, bool SMALL>
void launch_averages(const float *scores, float *cells, AvgParams &ap, int n_max, int n_top, SelCtrl *ctrl, uint32_t *hist, uint32_t *done,
                     uint64_t *lists, hipStream_t s)
{
    constexpr uint64_t per_wg = kAvgWaves * 64 * PER;
    uint64_t all = 0;
    for (int i = 0; i < n_max; ++i) all += ap.len[i];
    const int per_cu = PASS == 0 && PER == kAvgWide && all <= 2 * kNumCU * per_wg ? 1 : 2;
    const uint64_t most = std::max(per_cu * kNumCU / ap.groups, 16 * n_max);
    uint32_t wgs = 0;
    for (int i = 0; i < ILRE_MAX_POOL_KERNELS; ++i) {
        if (i < n_max) wgs += (uint32_t)std::max<uint64_t>(std::min((ap.len[i] + n_top + per_wg - 1) / per_wg, most * ap.len[i] / std::max<uint64_t>(all, 1)), 1);
        ap.wg_end[i] = i < n_max ? wgs : 0xFFFFFFFFu;
    }
    const size_t lds = avg_lds(PASS, PER, SMALL, SMALL ? kAvgGroup : ap.rows, n_top);
    hipLaunchKernelGGL((pool_averages<PASS, PER, SMALL>), dim3(wgs, ap.groups), dim3(kAvgThreads), lds, s, scores, cells, ap, ctrl, hist, done, lists);
}

// Dynamic LDS ceilings of the selection kernels: the same constants on every call, set once per process
// and device-independent.
hipError_t set_select_attributes()
{
    static hipError_t status = [] {
        constexpr int kWalkLds = kBitmapTokens / 8 + kRingBytes;
        static_assert(kWalkLds >= 2 * kWordSlots * (int)sizeof(uint32_t) + kRingBytes, "the word table fits where the bitmap does");
        constexpr int kSortLdsMax = 16384 * (int)sizeof(uint64_t);  // >= ILRE_MAX_BUDGET + 1 keys, padded to a power of two
        constexpr int kSeedRankLds = kCandCap * (int)sizeof(uint64_t);
        hipError_t e;
        for (const void *walk : {(const void *)allocate_walk<kWalkSeeds, false>, (const void *)allocate_walk<kWalkSeeds, true>,
                                 (const void *)allocate_walk<kWalkWordCells, false>, (const void *)allocate_walk<kWalkWordCells, true>,
                                 (const void *)allocate_walk<kWalkCells, false>, (const void *)allocate_walk<kWalkCells, true>,
                                 (const void *)allocate_relay<false>, (const void *)allocate_relay<true>})
            if ((e = hipFuncSetAttribute(walk, hipFuncAttributeMaxDynamicSharedMemorySize, kWalkLds)) != hipSuccess) return e;
        if ((e = raise_avg_lds<0, kAvgWide, true>()) != hipSuccess || (e = raise_avg_lds<0, kAvgNarrow, true>()) != hipSuccess ||
            (e = raise_avg_lds<0, kAvgNarrow, false>()) != hipSuccess || (e = raise_avg_lds<1, kAvgNarrow, true>()) != hipSuccess ||
            (e = raise_avg_lds<1, kAvgNarrow, false>()) != hipSuccess)
            return e;
        for (const void *rank : {(const void *)rank_short<1, false>, (const void *)rank_short<2, false>, (const void *)rank_short<4, false>,
                                 (const void *)rank_short<1, true>, (const void *)rank_short<2, true>})
            if ((e = hipFuncSetAttribute(rank, hipFuncAttributeMaxDynamicSharedMemorySize, (int)short_lds(kShortCells, kShortAvg, true))) != hipSuccess) return e;
        for (const void *brief : {(const void *)select_brief<4>, (const void *)select_brief<8>, (const void *)select_brief<16>})
            if ((e = hipFuncSetAttribute(brief, hipFuncAttributeMaxDynamicSharedMemorySize, (int)brief_lds(kBriefTokens))) != hipSuccess) return e;
        for (const void *rank : {(const void *)refine, (const void *)refine_parts})
            if ((e = hipFuncSetAttribute(rank, hipFuncAttributeMaxDynamicSharedMemorySize, kSortLdsMax)) != hipSuccess) return e;
        if ((e = hipFuncSetAttribute((const void *)seed_rank, hipFuncAttributeMaxDynamicSharedMemorySize, kSeedRankLds)) != hipSuccess) return e;
        return hipSuccess;
    }();
    return status;
}

uint32_t pool_blocks(uint32_t entries, uint32_t cap)
{
    const uint32_t want = (entries + kPoolWaves - 1) / kPoolWaves;
    return want < cap ? (want ? want : 1u) : cap;
}

// The walk and its ascending output: straight from the bitmap where it fits the LDS, else through the list of
// allocated tokens, which emit_sorted puts in order.
template <int ITEMS>
void launch_walk(WalkArgs &w, const SelectJob &job, int n_out, unsigned char *ws, const SelectLayout &lay, int32_t *out_idx,
                 int32_t *out_count, hipStream_t s)
{
    w.n_out = n_out;
    w.sink = job.sink;
    w.len = (uint32_t)job.L;
    w.picked = (uint32_t *)(ws + lay.picked);
    w.picked_n = w.picked + ILRE_MAX_BUDGET;
    w.out_idx = out_idx;
    w.out_count = out_count;
    // Taking turns pays while a turn is one look at kRelayChunk cells, of which those of the turns just before it are taken by
    // then, and there are other turns to prepare in.  Whole selection, workgroup -> turns: 48 combinations, shares of 85, 42 and
    // 21 cells 91.4 -> 81.0 us, 27 of 152, 76 and 38 59.2 -> 59.7; 32 of 128 and 64 94.3 -> 94.3 (with the word table 141.6 ->
    // 165.6); 4 of 125 30.1 -> 31.0, of 37 28.8 -> 28.8, of 19 and 10 31.6 -> 30.8; one of 16 26.3 -> 26.8.
    // With the word table, where looking through a list is a probe per cell: 20 of 51 91.0 -> 100.6, 48 of up to 42 141.5 -> 122.4.
    const bool bitmap = job.L <= kBitmapTokens;
    bool relay = ITEMS == kWalkWordCells && w.n >= kRelayCombos;
    for (int j = 0; j < w.n; ++j) relay = relay && w.share[j] <= (bitmap ? kRelayShare : kRelayShareTable) * w.reach[j];
    if (bitmap) {
        const size_t chunks = ((size_t)job.L + 32 * kBitmapChunk - 1) / (32 * kBitmapChunk);
        const size_t lds = chunks * kBitmapChunk * sizeof(uint32_t) + kRingBytes;
        hipLaunchKernelGGL((relay ? allocate_relay<false> : allocate_walk<ITEMS, false>), dim3(1), dim3(relay ? kRelayThreads : kWalkThreads), lds, s, w);
    } else {
        hipLaunchKernelGGL((relay ? allocate_relay<true> : allocate_walk<ITEMS, true>), dim3(1), dim3(relay ? kRelayThreads : kWalkThreads),
                           2 * (size_t)kWordSlots * sizeof(uint32_t) + kRingBytes, s, w);
        hipLaunchKernelGGL(emit_sorted, dim3((unsigned)((n_out + kEmitPerBlock - 1) / kEmitPerBlock) + 1u), dim3(kEmitThreads), 0, s,
                           w.picked, w.picked_n, n_out, job.sink, out_idx, out_count);
    }
}

// Whether a window-max selection starts with the pruning pre-pass.
bool prunes(int64_t L, int n_out)
{
    const int64_t nfine = (L + kSelFine - 1) / kSelFine;
    return nfine >= 4 * (int64_t)n_out && nfine >= 16384;
}

// Whether one launch does a whole window-max selection, of scores that are there or still lie in partial vectors.
bool in_brief(const SelectJob &job, bool fused)
{
    bool yes = job.L > 0 && job.L + job.sink <= (fused ? kBriefFused : kBriefTokens) && std::min<int64_t>(job.budget, job.L) <= kBriefSeeds;
    for (int j = 0; j < job.n_max; ++j) yes = yes && job.max_kernels[j] - 1 <= kBriefReach;
    return yes;
}

// Window-max form: the seeds (best raw scores), their ranks and neighbours, the walk.
hipError_t launch_select_window(const float *scores, const SelectJob &job, int32_t *out_idx, int32_t *out_count,
                                unsigned char *ws, const SelectLayout &lay, hipStream_t s, const FusedScores *fused)
{
    const int64_t L = job.L;
    const int n = job.combos();
    const int n_out = (int)(job.budget < L ? job.budget : L);
    SeedState *st = (SeedState *)(ws + lay.state);  // [0] the seeds, [1] the pruning pre-pass
    uint64_t *cand = (uint64_t *)(ws + lay.cand);
    uint64_t *tie = (uint64_t *)(ws + lay.tie);
    uint32_t *by_rank = (uint32_t *)(ws + lay.seed), *dom = by_rank + kCandCap;
    const uint32_t want = (uint32_t)n_out;  // the best raw scores that are seeds

    // B_c: floor(B / n), the first B mod n kernel sizes one more
    WalkArgs walk{};
    walk.n = n;
    const int base = job.budget / n, rem = job.budget % n;
    int r_max = 0;
    for (int j = 0; j < n; ++j) {
        const int r = (job.max_kernels[j] - 1) / 2;
        walk.reach[j] = (uint32_t)r;
        walk.share[j] = (uint32_t)(base + (j < rem ? 1 : 0));
        if (r > r_max) r_max = r;
    }
    walk.seeds = st;
    walk.pos = by_rank;
    walk.dom = dom;

    if (in_brief(job, fused != nullptr)) {
        const int64_t tokens = L + job.sink;
        if (fused && fused->nunits * tokens > kBriefPartial) {
            const hipError_t e = launch_reduce_units(fused->partial, fused->nunits, fused->L, fused->rmax, fused->scores, s);
            if (e != hipSuccess) return e;
            fused = nullptr;
        }
        walk.n_out = n_out;
        walk.sink = job.sink;
        walk.len = (uint32_t)L;
        walk.out_idx = out_idx;
        walk.out_count = out_count;
        auto kernel = tokens <= 4 * kThreads ? select_brief<4> : tokens <= 8 * kThreads ? select_brief<8> : select_brief<16>;
        hipLaunchKernelGGL(kernel, dim3(1), dim3(kThreads), brief_lds(L), s, fused ? fused->partial : nullptr, fused ? fused->nunits : 0,
                           fused ? fused->rmax : 0, fused ? fused->scores : nullptr, scores, job.sink, want, 2 * r_max, walk);
        return hipGetLastError();
    }

    const uint32_t nfine = (uint32_t)((L + kSelFine - 1) / kSelFine);
    Entries ent{nullptr, nullptr};
    uint32_t entries = nfine;
    const bool pruned = prunes(L, n_out);
    if (fused && pruned) {  // the pre-pass wants the finished scores
        const hipError_t e = launch_reduce_units(fused->partial, fused->nunits, fused->L, fused->rmax, fused->scores, s);
        if (e != hipSuccess) return e;
        fused = nullptr;
    }
    auto start_search = [&](const float *vals, int64_t len) {
        const SeedInit init{vals, len, sample_ranks(want, want, (double)len)};
        hipLaunchKernelGGL(seed_init, dim3(1), dim3(kThreads), 0, s, init, st);
    };
    if (!fused && !pruned) start_search(scores, L);
    if (pruned) {
        // Long contexts: only fine chunks whose maximum reaches the n_out-th largest chunk maximum (up to its
        // bin) can hold one of the n_out best scores; visit only those.
        float *cm = (float *)(ws + lay.cmax);
        uint32_t *active = (uint32_t *)(ws + lay.active);
        const uint32_t nfine2 = (nfine + kSelFine - 1) / kSelFine;
        const Entries all{nullptr, nullptr};
        hipLaunchKernelGGL(chunk_max, dim3(2048), dim3(kPoolThreads), 0, s, scores, L, nfine, cm);
        start_search(cm, nfine);
        hipLaunchKernelGGL(count_scores, dim3(pool_blocks((nfine2 + kRawBatch - 1) / kRawBatch, 256u)), dim3(kPoolThreads), 0, s, cm, (int64_t)nfine,
                           want, st + 1, all);
        hipLaunchKernelGGL(mark_active, dim3((nfine + kPoolThreads * kMarkPerThread - 1) / (kPoolThreads * kMarkPerThread)), dim3(kPoolThreads), 0, s, cm,
                           nfine, st + 1, active);
        ent = Entries{active, &st[1].active_n};
        // with a list the entry count is only known on the device: size the grid for the worst case the
        // pruning rule is meant for (a few times the budget) and let the wavefronts loop
        entries = 4u * (uint32_t)n_out + 1024u;
    }
    KeyBins bins{};
    if (fused) {
        // the last step of the scoring (sum of the partial score vectors) and the histogram in one pass
        bins = bins_of_mean(fused->mean);
        const uint32_t groups = (uint32_t)((fused->L + 63) / 64);  // of 64 tokens
        const bool wide = groups > 128u * kPoolWaves;
        auto kernel = fused->rmax ? (wide ? reduce_count<1, 4> : reduce_count<1, 1>) : (wide ? reduce_count<0, 4> : reduce_count<0, 1>);
        hipLaunchKernelGGL(kernel, dim3(pool_blocks(wide ? (groups + 3) / 4 : groups, 512u)), dim3(kPoolThreads), 0, s, fused->partial, fused->nunits,
                           fused->L, job.sink, fused->scores, bins, want, st);
    } else {
        hipLaunchKernelGGL(count_scores, dim3(pool_blocks((entries + kRawBatch - 1) / kRawBatch, 256u)), dim3(kPoolThreads), 0, s, scores, L, want, st, ent);
    }
    // Workgroups of eight wavefronts, a fine chunk a wavefront while that is one workgroup a compute unit; of four up to 64K
    // tokens, where the smaller one is done sooner (1000 tokens 27.2 us against 27.7 for the whole call, 32K 35.1 against 35.6;
    // 128K 37.4 against 36.9, 1M 50.4 against 48.5).
    auto collect_with = [&](auto kernel, int threads, uint32_t per_wave) {
        const uint32_t per_wg = (uint32_t)threads / 64 * per_wave, want_wg = (entries + per_wg - 1) / per_wg;
        hipLaunchKernelGGL(kernel, dim3(std::min(want_wg, (uint32_t)kNumCU)), dim3(threads), 0, s, scores, L, want, bins, !fused, st, cand, tie, ent);
    };
    if (entries <= 256)
        collect_with(collect<1, 256>, 256, 1);
    else if (entries <= (uint32_t)kNumCU * 8)
        collect_with(collect<1, 512>, 512, 1);
    else
        collect_with(collect<kRawBatch, 512>, 512, kRawBatch);
    // at most n_out + kSelSmall <= kCandCap seeds
    const uint32_t max_seeds = (uint32_t)n_out + (uint32_t)kSelSmall;
    hipLaunchKernelGGL(seed_rank, dim3((max_seeds + kSeedRankThreads / 16 - 1) / (kSeedRankThreads / 16)), dim3(kSeedRankThreads),
                       (size_t)((max_seeds + 127u) & ~127u) * sizeof(uint64_t), s, scores, L, st, cand, tie, 2 * r_max, by_rank, dom);
    launch_walk<kWalkSeeds>(walk, job, n_out, ws, lay, out_idx, out_count, s);
    return hipGetLastError();
}

}  // namespace

ClearWords select_clear_words(const SelectJob &job, const SelectLayout &lay, void *base)
{
    const int n_out = (int)(job.budget < job.L ? job.budget : job.L);
    if (job.mode != kSelWindowMax || job.L == 0 || in_brief(job, true) || prunes(job.L, n_out)) return ClearWords{};
    return ClearWords{(uint32_t *)((unsigned char *)base + lay.state), (uint32_t)(sizeof(SeedState) / sizeof(uint32_t))};
}

hipError_t launch_select(const float *scores, const SelectJob &job, int32_t *out_idx, int32_t *out_count,
                         void *workspace, const SelectLayout &lay, hipStream_t s, const FusedScores *fused)
{
    const int64_t L = job.L;
    const int n = job.combos();
    const int budget = job.budget;
    const int n_out = (int)(budget < L ? budget : L);
    unsigned char *ws = (unsigned char *)workspace;
    uint32_t *hist = (uint32_t *)(ws + lay.hist);
    SelCtrl *ctrl = (SelCtrl *)(ws + lay.ctrl);
    uint32_t *done = (uint32_t *)(ws + lay.done);
    uint64_t *cand = (uint64_t *)(ws + lay.cand);
    uint64_t *tie = (uint64_t *)(ws + lay.tie);
    float *cells = (float *)(ws + lay.cells);
    WalkArgs walk{};
    walk.cand = cand;

    hipError_t e = set_select_attributes();
    if (e != hipSuccess) return e;
    if (fused && (job.mode != kSelWindowMax || L == 0)) {  // only the window-max form takes the scores unreduced
        if ((e = launch_reduce_units(fused->partial, fused->nunits, fused->L, fused->rmax, fused->scores, s)) != hipSuccess) return e;
        fused = nullptr;
    }
    if (L == 0) {  // nothing but the sink part
        launch_walk<kWalkCells>(walk, job, 0, ws, lay, out_idx, out_count, s);
        return hipGetLastError();
    }
    if (job.mode == kSelWindowMax) return launch_select_window(scores, job, out_idx, out_count, ws, lay, s, fused);

    // The algorithm as printed.  B_c: floor(B / n), the first B mod n combinations one more; K_m = B / m + 1 cells.
    SelParams prm{};
    AvgParams ap{};
    const int base = budget / n, rem = budget % n;
    int64_t before = 0, tie_off = 0, len_max = 0;
    uint64_t cell_off = 0;
    bool coarse = true;  // windows can be counted kAvgWide at a time
    int share_of[ILRE_MAX_POOL_KERNELS], cell_of[ILRE_MAX_POOL_KERNELS];
    for (int j = 0; j < n; ++j) {
        const int share = base + (j < rem ? 1 : 0);
        int64_t len;
        int cell;
        combo_shape(job, j, len, cell);
        share_of[j] = share;
        cell_of[j] = cell;
        prm.len[j] = (uint32_t)len;
        prm.m[j] = (uint32_t)cell;
        prm.avg[j] = (uint32_t)job.avg_kernels[j % job.n_avg];
        prm.tie_off[j] = (uint64_t)tie_off;
        tie_off += 2 * len;
        if (j % job.n_avg == 0) {
            const int i = j / job.n_avg;
            ap.m[i] = (uint32_t)cell;
            ap.len[i] = (uint32_t)len;
            ap.off[i] = cell_off;
            cell_off += (uint64_t)len;
        }
        // K_m = B / m + 1 cells are candidates; of those the walk can only reach the first
        // ceil((shares up to and including this one) / m): at most (shares before) tokens are taken
        // when it starts and it stops after B_c free ones.  Only that many are found and sorted.
        int64_t km = (int64_t)budget / cell + 1;
        const int64_t reach = (before + share + cell - 1) / cell;
        if (reach < km) km = reach;
        prm.want[j] = (uint32_t)(km < len ? km : len);
        before += share;
        if (len > len_max) len_max = len;
        coarse = coarse && 2 * kAvgWide * (int64_t)prm.want[j] <= len;
    }
    ap.n_avg = job.n_avg;
    ap.groups = (job.n_avg + kAvgGroup - 1) / kAvgGroup;
    ap.rows = std::min(job.n_avg, kAvgGroup);
    int order[ILRE_MAX_POOL_KERNELS];
    for (int k = 0; k < job.n_avg; ++k) order[k] = k;
    std::stable_sort(order, order + job.n_avg, [&](int x, int y) { return job.avg_kernels[x] < job.avg_kernels[y]; });
    for (int k = 0; k < job.n_avg; ++k) {
        ap.at[k] = (uint16_t)order[k];
        ap.avg[k] = (uint16_t)job.avg_kernels[order[k]];
    }
    const int n_top = ap.avg[job.n_avg - 1];
    bool small = n_top <= kAvgGroup;  // every size once, 16 at most
    for (int k = 0; k < kAvgGroup; ++k) ap.at_of_size[k] = kNoAvg;
    for (int k = 0; k < job.n_avg && small; ++k) {
        uint16_t &at = ap.at_of_size[ap.avg[k] - 1];
        small = at == kNoAvg;
        at = ap.at[k];
    }
    const bool wide = small && coarse;
    // Cells are pooled where their windows are summed while that is a straight line of loads (1, 2, 4 and 8 tokens) and few cells
    // are in two chunks, else by a kernel of their own.  One average kernel, 128K tokens, there and apart: cells of 8, windows
    // of 5 28.2 and 31.2 us, of 64 32.0 and 33.2, of 96 47.3 and 37.4; cells of 6 32.8 and 31.9, 52.6 and 33.6; cells of 16
    // 53.5 and 31.7, 115 and 32.4; cells of 3 30.2 and 31.5, with windows of 33 34.5 and 31.9.
    ap.pooled = n_top > 64;
    for (int i = 0; i < job.n_max; ++i) {
        const int m = job.max_kernels[i];
        ap.pooled = ap.pooled || !(m == 1 || m == 2 || m == 4 || m == 8 || (m == 3 && n_top <= 16));
    }
    prm.src = ap.pooled ? cells : scores;
    for (int j = 0; j < n; ++j) {
        if (ap.pooled) {
            prm.off[j] = ap.off[j / job.n_avg];
            prm.m[j] = 1;
        }
        // counted kAvgWide at a time, the K_j best ones may be as few as a quarter as many, next to each other
        const SampleRanks r = sample_ranks((wide ? kAvgWide : 1.0) * prm.want[j], prm.want[j], std::max(1.0, (double)prm.len[j]));
        const uint32_t hi = std::min(r.hi, r.lo);
        const double mid = 1.25 * kBaseSamples * prm.want[j] / std::max(1.0, (double)prm.len[j]) + 1;
        prm.ranks[j] = r.lo | std::min(std::max((uint32_t)mid, hi), r.lo) << 8 | hi << 16;
    }
    uint32_t sort_n = kSortSmall;  // elements are sorted in LDS, up to a power of two of them
    for (int j = 0; j < n; ++j)
        while (sort_n < prm.want[j]) sort_n *= 2;
    // Few windows: see rank_short.  A workgroup a combination up to kShortCells cells; beyond, one for 4096 of them (up to 2M windows in
    // all) or 8192 (4M), as long as what the parts may hand on, with some room, can be sorted at once.  Whole selection, by
    // all workgroups -> so: 48 combinations 20000 tokens (0.8M windows) 68.6 -> 38.8 us, 128K (1.8M) 55.4 -> 47.4, 256K (3.7M) 50.4 -> 46.7,
    // 512K (7.3M) 55.6 -> 64.2; 27 combinations 256K (2.1M) 41.7 -> 36.8; one, cells of 4 128K 27.8 -> 18.1, 1M 33.6 -> 26.7.  Parts of 16384
    // cells: 256K, budget 4096 55.2 -> 63.0 us, one combination of 32K cells 28.7 -> 29.9.
    int quads = 0;  // 4096 cells each
    bool parts = false;
    uint32_t most = 0;
    int64_t windows = 0;
    for (int j = 0; j < n; ++j) most = std::max(most, prm.want[j]), windows += prm.len[j];
    bool brief = n_top <= kShortAvg;
    for (int i = 0; i < job.n_max; ++i) brief = brief && job.max_kernels[i] <= kShortMax;
    auto shared_by = [&](int64_t len, int q) { return (len + q * 4 * kThreads - 1) / (q * 4 * kThreads); };
    if (brief && len_max <= (int64_t)kShortCells) {
        quads = len_max <= 4 * kThreads ? 1 : len_max <= 8 * kThreads ? 2 : 4;
    } else if (brief) {
        for (int q = 1; q <= 2 && !quads; q *= 2)
            if (windows <= (q << 21) && shared_by(len_max, q) <= kShortParts && shared_by(len_max, q) * (most + most / 8 + 32) <= (int64_t)kSortLarge)
                quads = q;
        parts = quads != 0;
    }
    if (quads) {
        for (int j = 0; j < n; ++j) prm.m[j] = (uint32_t)cell_of[j];
        prm.src = scores;
        if (!parts) {
            auto kernel = quads == 1 ? rank_short<1, false> : quads == 2 ? rank_short<2, false> : rank_short<4, false>;
            hipLaunchKernelGGL(kernel, dim3(1, n), dim3(kThreads), short_lds((uint32_t)len_max, n_top, true), s, prm, 1024u, cand, tie, hist);
        } else {
            const uint32_t size = (uint32_t)quads * 4 * kThreads;
            auto kernel = quads == 1 ? rank_short<1, true> : rank_short<2, true>;
            const uint32_t by = (uint32_t)shared_by(len_max, quads);
            hipLaunchKernelGGL(kernel, dim3(by, n), dim3(kThreads), short_lds(size, n_top, false), s, prm, kSortLarge / by - most, cand, tie, hist);
            hipLaunchKernelGGL(refine_parts, dim3(n), dim3(kThreads), (size_t)kSortLarge * sizeof(uint64_t), s, prm, size, hist, cand, tie);
        }
    } else {
        if (ap.pooled) {
            uint32_t wgs = 1;
            for (int i = 0; i < job.n_max; ++i) {
                const uint32_t per_wg = 64u / cell_lanes(ap.m[i]) * kCellBatch * kPoolWaves;
                wgs = std::max(wgs, std::min((ap.len[i] + per_wg - 1) / per_wg, 4u * kNumCU));
            }
            hipLaunchKernelGGL(pool_cells, dim3(wgs, job.n_max), dim3(kPoolThreads), 0, s, scores, ap, cells);
        }
        hipLaunchKernelGGL(sel_init, dim3(n), dim3(kThreads), 0, s, prm, hist, ctrl, done);
        if (wide)
            launch_averages<0, kAvgWide, true>(scores, cells, ap, job.n_max, n_top, ctrl, hist, done, tie, s);
        else if (small)
            launch_averages<0, kAvgNarrow, true>(scores, cells, ap, job.n_max, n_top, ctrl, hist, done, tie, s);
        else
            launch_averages<0, kAvgNarrow, false>(scores, cells, ap, job.n_max, n_top, ctrl, hist, done, tie, s);
        if (small)
            launch_averages<1, kAvgNarrow, true>(scores, cells, ap, job.n_max, n_top, ctrl, hist, done, tie, s);
        else
            launch_averages<1, kAvgNarrow, false>(scores, cells, ap, job.n_max, n_top, ctrl, hist, done, tie, s);
        const uint32_t sort_keys = sort_n > kSortSmall ? std::max(sort_n, kSortLarge) : sort_n;
        hipLaunchKernelGGL(refine, dim3(n), dim3(kThreads), (size_t)sort_keys * sizeof(uint64_t), s, ctrl, cand, tie, sort_n);
    }
    walk.n = n;
    bool word_cells = true;  // cells lie inside words of the set: sizes 1, 2, 4, 8, 16, 32
    for (int j = 0; j < n; ++j) {
        walk.share[j] = (uint32_t)share_of[j];
        walk.reach[j] = (uint32_t)cell_of[j];
        walk.cells[j] = prm.want[j];
        word_cells = word_cells && 32 % cell_of[j] == 0;
    }
    if (word_cells)
        launch_walk<kWalkWordCells>(walk, job, n_out, ws, lay, out_idx, out_count, s);
    else
        launch_walk<kWalkCells>(walk, job, n_out, ws, lay, out_idx, out_count, s);
    return hipGetLastError();
}

}  // namespace ilre
