// Scoring kernels of the token-recall path (paper Section 3.2, Eq. 4 and Eq. 5) for gfx950.
//
// Two passes over the key cache, both built on one MFMA skeleton (this is the one for bf16 states; the one for fp32 states,
// score_f32_kernel, splits them into bf16 parts):
//   pass 1 (MODE 0, row statistics)  S^T = K_tile . Q^T : tokens are the MFMA rows, query rows the
//           columns, so each lane owns one query row and sees 16 tokens of it per 32x32 block; the
//           running maximum and sum of exponentials of Eq. 4's softmax stay in that lane's registers.
//   pass 2 (MODE 1, column scores)   S = Q . K_tile^T : query rows are the MFMA rows, tokens the
//           columns, so each lane owns one token and the Eq. 5 reduction over heads and queries is
//           an in-lane sum (or max) over its 16 accumulator registers per block.
// In both passes a wavefront keeps the fragments of its 32*NB query rows in registers for the whole
// kernel.  K tiles are copied once per workgroup from HBM straight into LDS (buffer loads with the LDS
// flag, three buffers in flight, chunks XOR-swizzled so that the 16-byte fragment reads of 16
// consecutive rows fall in distinct banks) and shared by all query heads of the GQA group.  The loop is
// software pipelined: the MFMA chains of one 32-token block are interleaved, instruction by
// instruction, with the exponentials of the block before it and with the LDS reads of the block after
// it.  Logits leave the MFMA unscaled; scale*log2(e) is folded into the single fma that feeds
// v_exp_f32.  No atomics anywhere: every reduction has a fixed order.
#include "ilre_internal.h"

#include <math.h>

#include <algorithm>
#include <mutex>

#include <type_traits>

namespace ilre {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

namespace {

constexpr float kNegBig = -1.0e30f;
// a partial sum against a frozen reference beyond this is redone against the running maximum: far above anything
// a row with moderate logits reaches, far enough below the fp32 limit that merging 512 splits stays finite
constexpr float kFrozenSumLimit = 1.0e30f;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// bf16: one 16-byte chunk holds 8 elements; v_mfma_f32_32x32x16_bf16 contracts 16 per issue
// (lanes 0-31 supply k = 0..7, lanes 32-63 k = 8..15 of the same row).
struct Bf16 {
    static constexpr int kElemBytes = 2;
    static constexpr int kSteps = 8;
    static constexpr int kChunksPerRow = 16;
    // tokens per LDS tile: four 16-byte chunks staged per thread
    static constexpr int tile_tokens(int waves) { return 16 * waves; }
    static __device__ __forceinline__ void mma(f32x16 &acc, const uint4 &a, const uint4 &b)
    {
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                      acc, 0, 0, 0);
    }
};

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// Online update of one query row's running (max, sum of exponentials) with 16 new logits.
// Logits are raw dot products; c = scale*log2(e) turns them into base-2 exponents.
// A row's running sum is kept as four partial sums (accumulator registers v, v+4, v+8, v+12 feed
// partial v & 3), so that an element costs exactly one fma, one exp2 and one add; they are added up
// once, when the kernel ends.
template <bool MASKED>
__device__ __forceinline__ void row_update(const f32x16 &acc, float c, float &m, float (&z)[4], int64_t tok0, int64_t L)
{
    float s[16];
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        s[v] = acc[v];
        if (MASKED) {
            const int64_t tok = tok0 + 8 * (v >> 2) + (v & 3);
            if (tok >= L) s[v] = -INFINITY;
        }
    }
    float smax = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) smax = fmaxf(smax, s[v]);
    const float mnew = fmaxf(m, smax * c);
    const float rescale = fast_exp2(m - mnew);
    m = mnew;
    const float nm = -mnew;
#pragma unroll
    for (int k = 0; k < 4; ++k) z[k] *= rescale;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v & 3] += fast_exp2(fmaf(s[v], c, nm));
}

__device__ __forceinline__ float quad_swap1(float x)  // lanes 0<->1, 2<->3 of every quad
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0xB1, 0xF, 0xF, true));
}
__device__ __forceinline__ float quad_swap2(float x)  // lanes 0<->2, 1<->3 of every quad
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), 0x4E, 0xF, 0xF, true));
}

// The same sum against a frozen reference m: no maximum, no rescale.  Any finite m gives the same
// (m, z) pair up to rounding as long as 2^(x - m) stays in range; a row whose later logits exceed m by
// more than ~2^7 base-2 units overflows to inf, which the kernel detects and redoes with row_update.
__device__ __forceinline__ void row_accumulate(const f32x16 &acc, float c, float m, float (&z)[4])
{
    const float nm = -m;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v & 3] += fast_exp2(fmaf(acc[v], c, nm));
}

// A row's exponent offset in pass 2 from its statistics in the natural-log units of Eq. 4.
__device__ __forceinline__ float row_offset(float row_max, float row_sumexp) { return -fmaf(row_max, kLog2e, __log2f(row_sumexp)); }

// The same straight from the per-split partials m[s*pitch], z[s*pitch], added up in the order of combine_row_stats: the
// splits are dealt to kCombineLanes sums, which a tree of neighbours reduces.  SHARERS threads (1, or 2 neighbouring
// lanes) share a row, each with its kCombineLanes / SHARERS sums.  All loads are in flight together, next to those of
// the first K tiles.  It saves a launch of 3.8 - 5 us; on the other hand every workgroup of a kv head reads all of the
// head's partials.  Measured, merge kernel -> this, whole recall: 16 splits (1000 tokens) 33.1 -> 29.1 us, 32 splits
// (40000 tokens, 32/8 heads, 128 queries) 115.4 -> 113.9 us; 64 splits (20000 tokens fp32) 132.4 -> 134.2 us,
// 256 splits (100000 tokens, 8/2 heads, 64 queries) 72.2 -> 86.9 us.  Four splits a sum is where it stops to pay (64 splits, 32/8 heads: 64 queries,
// 32768 tokens 78.0 -> 76.2 us, 100003 147.7 -> 146.9; 32 queries, 128 rows a workgroup 62.5 -> 61.6; 28/4 heads, 64 queries, 512 rows 74.6 -> 73.2;
// 128 splits of 128 rows 73.5 -> 75.0 and, 20000 tokens, 54.0 -> 56.5), in blocks of 256 and 128 rows two (96 queries, 30000 tokens, 64 splits 90.0
// -> 90.7).
constexpr int kCombineLanes = 16;
constexpr int kMergeSplits = 2 * kCombineLanes;
// The loads are issued before those of Q and K, which arrive while the sums are made (K first: the wait for the partials was one for Q
// and two tiles as well, and the sums came after it).  Wavefronts without a row load none: 4000 tokens, 8/2 heads, 16 queries, 63 splits,
// 64 of 128 rows 6.6 -> 5.7 us, 2681, 11 queries 6.4 -> 5.8.
template <int SHARERS, int ROUNDS>
struct RowParts {
    static constexpr int OWN = kCombineLanes / SHARERS;
    float m[ROUNDS][OWN], z[ROUNDS][OWN];
    __device__ __forceinline__ void load(const float *pm, const float *pz, int nsplit, int64_t pitch, int part)
    {
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k)
#pragma unroll
            for (int i = 0; i < OWN; ++i) {
                const int s = k * kCombineLanes + part * OWN + i;
                const int64_t at = (int64_t)(s < nsplit ? s : nsplit - 1) * pitch;
                m[k][i] = pm[at];
                z[k][i] = pz[at];
            }
    }
    __device__ __forceinline__ float offset(int nsplit, int part) const
    {
        float mm = kNegBig, sum[OWN];
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k)
#pragma unroll
            for (int i = 0; i < OWN; ++i) mm = fmaxf(mm, m[k][i]);
        if (SHARERS == 2) mm = fmaxf(mm, quad_swap1(mm));
#pragma unroll
        for (int i = 0; i < OWN; ++i) sum[i] = 0.f;
#pragma unroll
        for (int k = 0; k < ROUNDS; ++k)
#pragma unroll
            for (int i = 0; i < OWN; ++i)
                if (k * kCombineLanes + part * OWN + i < nsplit) sum[i] = fmaf(z[k][i], fast_exp2(m[k][i] - mm), sum[i]);  // (as combine_row_stats, bit for bit)
#pragma unroll
        for (int o = 1; o < OWN; o <<= 1)
#pragma unroll
            for (int i = 0; i < OWN; i += 2 * o) sum[i] += sum[i + o];
        if (SHARERS == 2) sum[0] += quad_swap1(sum[0]);
        return row_offset(mm * kLn2, sum[0]);
    }
};

// One workgroup's share: NB 32-row blocks a wavefront of query block qb, tiles tile0 .. tile1 - 1 of kv head g.
// MODE 0: row statistics.  MODE 1: column scores (RMAX = 0 sum over rows, 1 max over rows; MANY: it may have to merge 2 kMergeSplits).
template <int NB, int WAVES, int MODE, int RMAX, bool MANY>
__device__ __forceinline__ void score_rows(const ScoreArgs &a, int g, int split, int qb, int64_t tile0, int64_t tile1, bool timed, unsigned long long t_begin)
{
    using T = Bf16;
    constexpr int ES = T::kElemBytes;
    constexpr int STEPS = T::kSteps;
    constexpr int TN = T::tile_tokens(WAVES);
    constexpr int CPR = T::kChunksPerRow;
    constexpr int ROWB = CPR * 16;
    constexpr int TILE_BYTES = TN * ROWB;
    constexpr int NLW = TN * CPR / 64 / WAVES;  // 1 KiB DMA issues per wavefront and tile
    constexpr int TBLOCKS = TN / 32;
    constexpr int UNITS = TBLOCKS;              // pipeline units per tile: one per 32-token block
    constexpr int NPART = WAVES * 2;            // partial column results per token (pass 2)
    // Row pitch of the partial-result buffers.  The flush reads them with four lanes per token, lane group g
    // taking partials g*NPART/4 ..: the four groups of a half-wave must start 8 banks apart (8 tokens each)
    // to cover the 32 LDS banks once.  The stores (32 consecutive tokens of one partial) never conflict.
    constexpr int RSTR = TN + (NPART == 16 ? 34 : 36);
    static_assert((NPART / 4 * RSTR) % 32 == 8 || (NPART / 4 * RSTR) % 32 == 24, "flush lane groups 8 banks apart");
    static_assert(TN * CPR % (64 * WAVES) == 0, "tile must divide over the wavefronts");
    static_assert(UNITS % 2 == 0, "units alternate between two accumulators");
    static_assert(TN == 16 * WAVES && NPART % 4 == 0, "column flush: 16 tokens per wavefront, 4 lanes per token");

    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int l32 = lane & 31;
    const int half = lane >> 5;
    const int rl0 = qb * a.rows_per_wg + wave * (NB * 32);
    // One block a wavefront: a wavefront without a single row copies its share of the tiles, but no query rows, and in pass 2 adds up its tokens; it
    // computes nothing.  Both passes, all wavefronts alike -> so (where rows it has no use for are copied all the same): 500000 tokens, 32/8 heads, 8
    // queries (32 of 128 rows) 165.5 + 235 -> 161.7 + 224 us (161.9 + 225), staged 167 + 235 -> 161.4 + 224.5; 9000 tokens, 8/2, staged
    // 5.4 + 5.8 -> 4.8 + 5.2 (5.2 + 5.6); 119 of 128 rows, none idle, 100003 tokens 20.1 + 21.7 -> 20.4 + 21.6.  With two
    // blocks the branch costs full workgroups more than it saves the others (32768 tokens, 64 queries 75.4 -> 76.5; 65536, 28/4, 64 103.8 -> 101.6).
    const bool idle = NB == 1 && __builtin_amdgcn_readfirstlane(rl0) >= a.rows_per_group;
    const int64_t nrows = (int64_t)a.Hq * a.Lq;

    // Pass 2: what the exponent offset of a row is made of, one row a thread (NB = 1: a pair of threads).
    constexpr int ROWS = WAVES * NB * 32, SHARERS = WAVES * 64 / ROWS;
    const int off_row = qb * a.rows_per_wg + tid / SHARERS;
    RowParts<SHARERS, 2> parts;
    RowParts<SHARERS, 4> more_parts;
    float stat_m, stat_z;
    const bool many = MANY && (NB == 2 || (a.merge && a.nsplit > kMergeSplits));  // (the kernel for NB = 2 is launched for nothing else)
    if (MODE == 1 && !idle) {  // (idle: the pairs' rows are the wavefront's)
        const int64_t r = (int64_t)g * a.rows_per_group + min(off_row, a.rows_per_group - 1);
        if (many) {
            more_parts.load(a.part_m + r, a.part_z + r, a.nsplit, nrows, tid % SHARERS);
        } else if (a.merge) {
            parts.load(a.part_m + r, a.part_z + r, a.nsplit, nrows, tid % SHARERS);
        } else {
            stat_m = a.row_max[r];
            stat_z = a.row_sumexp[r];
        }
    }

    // Query fragments, resident for the whole kernel: lane holds, for each of its NB blocks, row
    // l32 of the block, 16-byte chunk (2*step + half) of that row.  Rows past the group's last one are read as that one and become
    // zeros: pass 1 does not store their statistics, pass 2 gives them the offset -inf.
    // They come by way of LDS, where a wavefront's copy of 32 rows is twice its share of a tile, so that all of them fill two tile buffers (behind the
    // first two, laid out as a tile is), one block after the other.  Read straight into the registers a load takes 16 bytes from each of 64
    // cache lines, and the K tiles queue up behind 16 of them a wavefront: 131072 tokens, 512 rows a workgroup, the tiles were there 5.2 us
    // after the start of a first pass and 7.7 of a second, 3.0 and 5.3 now (1M 6.8 and 6.3, 5.0 and 4.8).  Passes before -> after, together with the
    // order of the partials, the flag of the redo below and sums as fma, which were not timed one by one: 32768 tokens, 32/8 heads, 64 queries 24.4 + 22.9
    // -> 22.5 + 21.8 us, 100003, 28/4, 17 21.3 -> 20.4 the first, 20000, 16/4, 40 13.1 + 11.9 -> 12.0 + 11.5, 1M no change.
    static_assert(WAVES * 32 * ROWB == 2 * TILE_BYTES, "the query rows end where `behind` begins");
    uint4 qf[NB][STEPS];
    const unsigned lds0 = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)smem;
    const unsigned qlds = lds0 + 2 * TILE_BYTES + wave * (32 * ROWB);
    const bool in_line = a.q_stride_head == (int64_t)a.Lq * a.q_stride_token;  // a head's rows follow the one's before
    auto issue_queries = [&](int b) {
        const int64_t row_bytes = a.q_stride_token * ES, head_bytes = a.q_stride_head * ES;
        constexpr int ISSUES = 32 * CPR / 64;  // four rows at a time
        auto issue = [&](int j, uint64_t row_at) {
            const int row = j * 4 + (lane >> 4);
            lds_dma16(row_at + (((lane & 15) ^ (row & 15)) * 16), __builtin_amdgcn_readfirstlane(qlds + j * 1024));
        };
        if (in_line) {  // uniform
            const uint64_t first = (uint64_t)a.q + (uint64_t)((int64_t)g * a.G * head_bytes);
#pragma unroll
            for (int j = 0; j < ISSUES; ++j)
                issue(j, first + (uint64_t)(min(rl0 + b * 32 + j * 4 + (lane >> 4), a.rows_per_group - 1) * row_bytes));
        } else {  // lane l32 works out where row l32 lies
            const int rl = min(rl0 + b * 32 + l32, a.rows_per_group - 1);
            const uint64_t own = (uint64_t)a.q + (uint64_t)((int64_t)(g * a.G + rl / a.Lq) * head_bytes + (int64_t)(rl % a.Lq) * row_bytes);
#pragma unroll
            for (int j = 0; j < ISSUES; ++j) {
                const int row = j * 4 + (lane >> 4);
                issue(j, (uint64_t)(uint32_t)__shfl((int)(uint32_t)(own >> 32), row) << 32 | (uint32_t)__shfl((int)(uint32_t)own, row));
            }
        }
    };
    auto read_queries = [&](int b) {
#pragma unroll
        for (int st = 0; st < STEPS; ++st)
            qf[b][st] = *(const uint4 *)(__attribute__((address_space(3))) unsigned char *)(size_t)(qlds + l32 * ROWB + (((2 * st + half) ^ (l32 & 15)) * 16));
        if (rl0 + b * 32 + 32 > a.rows_per_group) {  // uniform
            // (matrix instructions draw less power on zeros, and the clock follows: 60000 tokens, 64 of 128 rows 62.1 -> 60.7 us a recall)
#pragma unroll
            for (int st = 0; st < STEPS; ++st) qf[b][st] = rl0 + b * 32 + l32 < a.rows_per_group ? qf[b][st] : make_uint4(0, 0, 0, 0);
        }
    };

    // K tiles: three LDS buffers of TN rows, row r's 16-byte chunk c stored at chunk position
    // c ^ (r & 15), so that the fragment reads of 16 consecutive rows fall in distinct banks while a
    // wavefront's DMA still fills 1 KiB of consecutive LDS.
    const unsigned char *kbase = (const unsigned char *)a.k + (int64_t)g * a.k_stride_head * ES;
    const int64_t krow_bytes = a.k_stride_token * ES;
    int dma_voff[NLW];
#pragma unroll
    for (int j = 0; j < NLW; ++j) {
        const int pchunk = (wave * NLW + j) * 64 + lane;
        const int row = pchunk / CPR, cpos = pchunk % CPR;
        dma_voff[j] = (int)(row * krow_bytes) + (cpos ^ (row & 15)) * 16;
    }
    // Pass 2 walks its split backwards: pass 1 has just streamed the same split forwards, so what it read
    // last is what the memory-side cache still holds (an eighth of K at 1M tokens).  `tile` counts in
    // processing order everywhere; only the two places that turn it into tokens go through here.
    auto first_token = [&](int64_t tile) { return (MODE == 1 ? tile0 + tile1 - 1 - tile : tile) * TN; };
    auto issue_tile = [&](int64_t tile, int buf) {
        const int64_t tok0 = first_token(tile);
        const unsigned long long base = (unsigned long long)(kbase + tok0 * krow_bytes);
        long long avail = (a.L - tok0 - 1) * krow_bytes + ROWB;  // bytes up to the end of row L-1
        if (avail > 0xFFFFFFFFll) avail = 0xFFFFFFFFll;
        i32x4 rsrc;
        rsrc[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)base);
        rsrc[1] = __builtin_amdgcn_readfirstlane((int)((unsigned)(base >> 32) & 0xFFFFu));
        rsrc[2] = __builtin_amdgcn_readfirstlane((int)(unsigned)avail);
        rsrc[3] = 0x00020000;
#pragma unroll
        for (int j = 0; j < NLW; ++j)
            lds_dma16(rsrc, __builtin_amdgcn_readfirstlane(lds0 + buf * TILE_BYTES + (wave * NLW + j) * 1024), dma_voff[j]);
    };

    // per-lane LDS byte offset of fragment chunk (2*st + half) of row l32 within a 32-row block,
    // relative to the tile buffer being read; advanced from buffer to buffer in place
    unsigned frag_addr[STEPS];

    // the first two tiles go to buffers 0 and 1
    auto issue_first = [&]() {
        issue_tile(tile0, 0);
        if (tile0 + 1 < tile1) issue_tile(tile0 + 1, 1);
    };

    // pass-1 state: one (max, sum) per owned query row, in base-2 exponent units
    float m[NB], z[NB][4];
    // pass-2 state: per accumulator register the row's exponent offset -(max*log2e + log2 sum)
    float noff[MODE == 1 ? NB : 1][16];
    float *red = (float *)(smem + 3 * TILE_BYTES);  // [3][NPART][RSTR], pass 2 only
    const int unit = g * a.nqb + qb;

    uint32_t *behind = (uint32_t *)(smem + 4 * TILE_BYTES);  // behind the wavefronts' query rows
    if (!idle) issue_queries(0);
    issue_first();
    if (tile0 + 1 < tile1)  // (the tiles may stay on their way)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * NLW) : "memory");
    else
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(NLW) : "memory");
    read_queries(0);
    if (NB == 2) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        issue_queries(1);
    }

    if (MODE == 0) {
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            m[b] = kNegBig;
#pragma unroll
            for (int k = 0; k < 4; ++k) z[b][k] = 0.f;
        }
        if (tid == 0) *behind = 0;  // set where a split has to be walked again
    } else {
        // The exponent offsets of the workgroup's rows, handed out through LDS (a kernel that wrote them to a table before took
        // 4.7 us of a staged call: 50001 tokens 149.9 -> 146.9 us):
        // accumulator registers 4j .. 4j+3 of a lane are four consecutive rows.  Rows past the group's last one
        // (q = 0) get -inf: exp2(0*c - inf) = 0.
        float *offs = (float *)behind;
        float off = -INFINITY;
        if (!idle)
            off = many ? more_parts.offset(a.nsplit, tid % SHARERS) : a.merge ? parts.offset(a.nsplit, tid % SHARERS) : row_offset(stat_m, stat_z);
        if (tid % SHARERS == 0) offs[tid / SHARERS] = off_row < a.rows_per_group ? off : -INFINITY;
        __syncthreads();
#pragma unroll
        for (int b = 0; b < NB; ++b) {
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float4 x = *(const float4 *)&offs[wave * (NB * 32) + b * 32 + 8 * j + 4 * half];
                noff[b][4 * j + 0] = x.x;
                noff[b][4 * j + 1] = x.y;
                noff[b][4 * j + 2] = x.z;
                noff[b][4 * j + 3] = x.w;
            }
        }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (NB == 2) read_queries(NB - 1);
    // (the barrier in front of the first tile lies between these reads and what else goes there: the third tile, pass 2's partial results)

    // Pass 2: combine the NPART partial column results of a finished tile in a fixed order.  Wave w
    // takes tokens 16w..16w+15, four lanes per token, each lane NPART/4 partials, then the quad.
    // In the tile loop the LDS reads are issued inside the first unit and consumed in the last one, so
    // that their latency hides behind MFMAs.
    float fl[NPART / 4];
    auto flush_load = [&](int64_t tile) {
        const float *rb = red + (int)(tile - tile0) % 3 * NPART * RSTR;
        const int tl = wave * 16 + (lane >> 2), part0 = (lane & 3) * (NPART / 4);
#pragma unroll
        for (int k = 0; k < NPART / 4; ++k) fl[k] = rb[(part0 + k) * RSTR + tl];
    };
    // `live` false: nothing to flush yet.  Lanes with nothing to store write to a dump slot instead of
    // branching around the store, which would cut the tile body into separately scheduled pieces.
    auto flush_finish = [&](int64_t tile, bool live) {
        const int tl = wave * 16 + (lane >> 2);
        float acc = fl[0];
#pragma unroll
        for (int k = 1; k < NPART / 4; ++k) acc = RMAX ? fmaxf(acc, fl[k]) : acc + fl[k];
        const float x1 = quad_swap1(acc);
        acc = RMAX ? fmaxf(acc, x1) : acc + x1;
        const float x2 = quad_swap2(acc);
        acc = RMAX ? fast_exp2(fmaxf(acc, x2)) : acc + x2;
        const int64_t tok = first_token(tile) + tl;
        // after the quad reduction the four lanes of a token hold the same value and all store it
        float *dst = (live && tok < a.L) ? a.partial + ((int64_t)unit * a.L + tok) : a.dump + (lane & 15);
        *dst = acc;
    };
    auto flush_columns = [&](int64_t tile) {
        flush_load(tile);
        flush_finish(tile, true);
    };

    // The softmax arithmetic of one finished 32x32 block ("unit": token block tb, query block b).
    // It runs one unit behind the MFMAs, so that the matrix pipe works on unit u while the vector
    // pipe exponentiates unit u-1 from the other accumulator.
    float col = 0.f;  // pass 2: running column result of the token block over its NB query blocks
    // `rb` is the partial-result buffer (0..2) of the unit's tile, pass 2 only.
    auto finish_unit = [&](const f32x16 &acc, int b, int tb, int64_t tile, int rb, auto masked_tag, auto frozen_tag) {
        constexpr bool MASKED = decltype(masked_tag)::value;
        constexpr bool FROZEN = decltype(frozen_tag)::value;
        if (MODE == 0) {
            if (FROZEN)
                row_accumulate(acc, a.c, m[b], z[b]);
            else
                row_update<MASKED>(acc, a.c, m[b], z[b], tile * TN + tb * 32 + 4 * half, a.L);
        } else {
            // RMAX: the exponents' maximum, of which flush_finish takes the one exp2 a token (exp2 being monotonic).  Two fma and two maxima a
            // matrix instruction keep up with it, two exp2 more do not: 131072 tokens, 128 queries, 32/8 heads 144 -> 114 us this pass, 1M
            // tokens, 256 queries 1981 -> 1621.
            float e[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float x = fmaf(acc[v], a.c, noff[b][v]);
                e[v] = RMAX ? x : fast_exp2(x);
            }
            float p0 = e[0], p1 = e[1], p2 = e[2], p3 = e[3];
#pragma unroll
            for (int v = 4; v < 16; v += 4) {
                if (RMAX) {
                    p0 = fmaxf(p0, e[v]), p1 = fmaxf(p1, e[v + 1]), p2 = fmaxf(p2, e[v + 2]), p3 = fmaxf(p3, e[v + 3]);
                } else {
                    p0 += e[v], p1 += e[v + 1], p2 += e[v + 2], p3 += e[v + 3];
                }
            }
            const float part = RMAX ? fmaxf(fmaxf(p0, p1), fmaxf(p2, p3)) : (p0 + p1) + (p2 + p3);
            if (b == 0)
                col = part;
            else
                col = RMAX ? fmaxf(col, part) : col + part;
            // (the unit before a split's very first one stores zeros, max: -inf, into a buffer that is rewritten
            // before it is read: no condition here, the tile body stays free of branches)
            if (b == NB - 1) red[(rb * NPART + wave * 2 + half) * RSTR + tb * 32 + l32] = col;
        }
    };

    f32x16 acc[2][NB];
    uint4 kf[STEPS];
    auto start_split = [&]() {
#pragma unroll
        for (int st = 0; st < STEPS; ++st) frag_addr[st] = lds0 + l32 * ROWB + (((2 * st + half) ^ (l32 & 15)) * 16);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
        if (MODE == 1 && idle)  // what it has to add, once for all tiles
            for (int i = lane; i < 3 * 2 * TN; i += 64)
                red[(i / (2 * TN) * NPART + wave * 2 + i / TN % 2) * RSTR + i % TN] = RMAX ? -INFINITY : 0.f;

        // acc[u & 1] receives unit u (a 32-token block against the wave's NB query blocks); the unit
        // before the very first one is all -inf, which the softmax arithmetic turns into zeros (max over rows: leaves).
    #pragma unroll
        for (int b = 0; b < NB; ++b) {
    #pragma unroll
            for (int v = 0; v < 16; ++v) acc[1][b][v] = -INFINITY;
        }
    #pragma unroll
        for (int st = 0; st < STEPS; ++st)
            kf[st] = *(const uint4 *)(__attribute__((address_space(3))) unsigned char *)(size_t)frag_addr[st];
    };

    // One tile.  Its buffer and the next tile's are already published; the tile after that is
    // requested now and published by the barrier at the end.  Per 32-token block the NB independent
    // MFMA chains are interleaved step by step; as soon as a step's fragment has fed all chains it is
    // refilled from LDS for the next block (for the last block, from the next tile's buffer).
    // CUR_RAGGED is only ever true for the last tile of the context, and only in pass 1.
    auto do_tile = [&](int64_t tile, auto ragged_tag, auto frozen_tag) {
        constexpr bool CUR_RAGGED = decltype(ragged_tag)::value;
        constexpr bool FROZEN = decltype(frozen_tag)::value;  // pass 1: reference maxima no longer move
        const int it = (int)(tile - tile0);
        const int rb_cur = it % 3, rb_prev = (it + 2) % 3;
        if (tile + 2 < tile1) issue_tile(tile + 2, (it + 2) % 3);
        if (idle) {
            if (MODE == 1) {
                flush_load(it >= 2 ? tile - 2 : tile);
                flush_finish(tile - 2, it >= 2);
            }
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
            __syncthreads();
            return;
        }
        // byte distance from this tile's buffer to the next tile's
        const int to_next = (it % 3 == 2) ? -2 * TILE_BYTES : TILE_BYTES;

#pragma unroll
        for (int u = 0; u < UNITS; ++u) {
            if (u == UNITS - 1) {
#pragma unroll
                for (int st = 0; st < STEPS; ++st) frag_addr[st] += to_next;
            }
            const int next_block = (u == UNITS - 1) ? 0 : (u + 1) * 32 * ROWB;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[u & 1][b][v] = 0.f;
            }
#pragma unroll
            for (int st = 0; st < STEPS; ++st) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    if (MODE == 0)
                        T::mma(acc[u & 1][b], kf[st], qf[b][st]);
                    else
                        T::mma(acc[u & 1][b], qf[b][st], kf[st]);
                }
                kf[st] = *(const uint4 *)((__attribute__((address_space(3))) unsigned char *)(size_t)frag_addr[st] + next_block);
            }
            // column results of the tile before the previous one: LDS reads behind the first unit's
            // MFMAs (in straight-line code, so the fragment waits can leave them in flight), sums and
            // store in the tile's last unit
            if (MODE == 1 && u == 0) flush_load(it >= 2 ? tile - 2 : tile);
            if (MODE == 1 && u == UNITS - 1) flush_finish(tile - 2, it >= 2);
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (u == 0)
                    finish_unit(acc[1][b], b, UNITS - 1, tile - 1, rb_prev, std::false_type{}, frozen_tag);
                else
                    finish_unit(acc[(u - 1) & 1][b], b, u - 1, tile, rb_cur, std::bool_constant<CUR_RAGGED>{}, frozen_tag);
            }
            // ask the scheduler for: one MFMA (group), a slice of the vector work, and a fragment
            // read after every NB-th MFMA
#pragma unroll
            for (int st = 0; st < STEPS; ++st) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    if (b == NB - 1) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, (MODE == 0 && !FROZEN) ? 8 : RMAX ? 4 : 6, 0);
                }
            }
        }

        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();
    };

    // Only pass 1 has to mask the tokens past L (in pass 2 a lane is a token and is simply not
    // stored); the ragged tile, if any, is the last tile of the last split.
    const bool last_ragged = MODE == 0 && tile1 * TN > a.L;
    const int64_t tile_full_end = last_ragged ? tile1 - 1 : tile1;
    // One walk over the split.  Pass 1 follows the running maximum for the first two tiles, then freezes each
    // row's reference and only accumulates -- unless `online_all`, the always-safe form.
    auto run_split = [&](bool online_all) {
    start_split();
    int64_t online_end = tile_full_end;
    if (MODE == 0 && !online_all && tile0 + 2 < tile_full_end) online_end = tile0 + 2;
    int64_t tile = tile0;
    for (; tile < online_end; ++tile) do_tile(tile, std::false_type{}, std::false_type{});
    if (MODE == 0)
        for (; tile < tile_full_end; ++tile) do_tile(tile, std::false_type{}, std::true_type{});
    if (last_ragged) do_tile(tile1 - 1, std::true_type{}, std::false_type{});
    if (idle) return;
    // drain the pipeline: the last unit of the last tile
    const int rb_last = (int)((tile1 - 1 - tile0) % 3);
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (last_ragged)
            finish_unit(acc[(UNITS - 1) & 1][b], b, UNITS - 1, tile1 - 1, rb_last, std::true_type{}, std::false_type{});
        else
            finish_unit(acc[(UNITS - 1) & 1][b], b, UNITS - 1, tile1 - 1, rb_last, std::false_type{}, std::false_type{});
    }
    };
    run_split(MODE == 0 && a.force_online);
    if (MODE == 0 && !a.force_online) {
        // A row whose later logits lie far above its frozen reference sums to inf (or to something a merge over
        // the splits could push out of range): the workgroup then walks its split again, following the maximum.
        bool bad = false;
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int k = 0; k < 4; ++k) bad = bad || !(z[b][k] <= kFrozenSumLimit);
        if (bad) *behind = 1;
        __syncthreads();
        if (*behind) {  // uniform; the barrier also orders the last reads of the tile buffers before the new DMA
            issue_first();
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                m[b] = kNegBig;
#pragma unroll
                for (int k = 0; k < 4; ++k) z[b][k] = 0.f;
            }
            run_split(true);
        }
    }

    if (MODE == 1) {
        __syncthreads();
        if (tile1 - tile0 >= 2) flush_columns(tile1 - 2);
        flush_columns(tile1 - 1);
    } else {
        // The two half-waves saw disjoint tokens of the same query rows: merge, then one partial
        // (max, sum) per row and split.
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const float zb = (z[b][0] + z[b][1]) + (z[b][2] + z[b][3]);
            const float mo = __shfl_xor(m[b], 32);
            const float zo = __shfl_xor(zb, 32);
            const float mm = fmaxf(m[b], mo);
            const float zz = zb * fast_exp2(m[b] - mm) + zo * fast_exp2(mo - mm);
            const int rl = rl0 + b * 32 + l32;
            if (half == 0 && rl < a.rows_per_group) {
                const int64_t r = (int64_t)g * a.rows_per_group + rl;
                a.part_m[(int64_t)split * nrows + r] = mm;
                a.part_z[(int64_t)split * nrows + r] = zz;
            }
        }
        if (timed) {
            const unsigned long long dt = wall_clock64() - t_begin;  // 10 ns ticks
            a.wg_time[blockIdx.x] = dt < 0xFFFFFFFFull ? (uint32_t)(dt ? dt : 1) : 0xFFFFFFFFu;
        }
    }
}

// MIXED: two query blocks a kv head, of which the second is one 32-row block a wavefront.  Workgroups 32 slots apart share a compute
// unit, so that every other 32 slots have the two blocks the other way round: one of each kind a compute unit.
template <int NB, int WAVES, int MODE, int RMAX, bool MIXED, bool MANY = false>
__global__ __launch_bounds__(WAVES * 64, 2) void score_kernel(const ScoreArgs a)
{
    // blockIdx -> (kv head, token split, query block).  Workgroups are dealt round-robin to the 8
    // XCDs, so the query blocks that stream the same K range are given ids with equal id % 8 and
    // consecutive id / 8: they run on one XCD at about the same time and share its L2.
    const int xcd = blockIdx.x % kNumXCD;
    const int slot = blockIdx.x / kNumXCD;
    const int qb = MIXED ? (slot ^ slot >> 5) & 1 : slot % a.nqb;
    const int64_t pair = (int64_t)(slot / a.nqb) * kNumXCD + xcd;
    // Pass 1 notes how long each workgroup ran (0: it had nothing to do); the merge kernel behind it turns the
    // times into pass 2's token ranges.
    const bool timed = MODE == 0 && a.wg_time != nullptr && threadIdx.x == 0;
    const unsigned long long t_begin = timed ? wall_clock64() : 0ull;
    if (timed) a.wg_time[blockIdx.x] = 0u;
    // what the selection counts in is cleared on the side (a launch of its own took 4.7 us)
    if (MODE == 1 && blockIdx.x == 0)
        for (uint32_t i = threadIdx.x * 4; i < a.clear.n; i += WAVES * 64 * 4) *(uint4 *)&a.clear.at[i] = make_uint4(0, 0, 0, 0);
    if (pair >= (int64_t)a.Hkv * a.nsplit) return;
    const int g = (int)(pair / a.nsplit);
    const int split = (int)(pair % a.nsplit);
    int64_t tile_lo = (int64_t)split * a.tiles_per_split;
    int64_t tile_hi = (tile_lo + a.tiles_per_split < a.ntiles) ? tile_lo + a.tiles_per_split : a.ntiles;
    if (MODE == 1 && a.split_table != nullptr) {
        // Pass 2's column results do not depend on how the tokens are cut into ranges, so the ranges may follow the
        // speed of the XCD they run on (the table's header says which launch shape it was made for; the table is
        // only used if it is a cut of the context, whatever the workspace holds).
        const int32_t *tb = a.split_table;
        if ((uint32_t)tb[0] == (uint32_t)a.table_tag && (uint32_t)tb[1] == (uint32_t)(a.table_tag >> 32)) {
            // every wavefront checks the whole table (a few loads a lane): edges from 0 to ntiles that never
            // step back cut the context into ranges that cover every tile once, whatever else they are
            bool bad = false;
            for (int i = threadIdx.x & 63; i <= a.nsplit; i += 64) {
                const int64_t e0 = tb[2 + i], e1 = i < a.nsplit ? (int64_t)tb[3 + i] : a.ntiles;
                bad = bad || e0 < 0 || e0 > e1 || e1 > a.ntiles || (i == 0 && e0 != 0) || (i == a.nsplit && e0 != a.ntiles);
            }
            if (!__any(bad)) {
                tile_lo = tb[2 + split];
                tile_hi = tb[3 + split];
            }
        }
    }
    if (tile_lo >= tile_hi) return;
    if (MIXED && qb == 1)
        score_rows<1, WAVES, MODE, RMAX, false>(a, g, split, qb, tile_lo, tile_hi, timed, t_begin);
    else
        score_rows<NB, WAVES, MODE, RMAX, MANY>(a, g, split, qb, tile_lo, tile_hi, timed, t_begin);
}

// ---------------------------------------------------------------- fp32 states
//
// The fp32 matrix instructions run at a sixteenth of the bf16 rate.  An fp32 number is the sum of three bf16 numbers, exactly
// (24 bits of significand: x = h + m + l, each the rest rounded to nearest, so that m is 2^-8 of x at most and l 2^-17), and a
// product of two such sums is the nine products of their parts, each exact in fp32.  Six of them are taken, added up in fp32: what
// is left out (m l, l m and l l) is 2^-24 of a product at most, as much as the rounding of one addition, and 2^-27.5 rms (h cut off
// instead of rounded: m reaches 2^-7, l 2^-16, and what is left out 2^-22).  The large products (h h) have an accumulator of their
// own and the others two, so that a logit sees 8 roundings at its own size, where the fp32 instructions took 64.  (Splitting into
// parts: Dekker, Numerische Mathematik 18 (1971); several low-precision products for one of high precision: Henry, Tang and
// Heinecke, ARITH 2019.)
//
// A workgroup owns 128 query rows of a kv head, 32 a wavefront, whose parts stay in registers, and streams 32 tokens of K at a
// time: a thread fetches 64 bytes a tile ahead, splits them and writes the three parts to LDS, chunks swizzled as above.  Two
// workgroups a compute unit work in each other's shadow; the split is done once for four wavefronts.
// Bound: 48 matrix instructions of 32 cycles for 32 x 32 logits (the fp32 instructions: 4096 cycles), 1.2 PFLOP/s of them on 32768 tokens
// and 8192 rows, what the matrix pipe reaches beside such vector work.  Measured, whole recall, fp32 instructions -> so: 4096
// tokens, 32/8 heads, 32 queries 61.0 -> 38.6 us; 32768 tokens, 256 queries 1102 -> 717 us; 20000, 28/4, 64 209 -> 140.  Errors against 64 bits, logarithms of
// the rows' sums: 4.1e-7 -> 3.0e-7 rms, 1.5e-6 -> 1.1e-6 largest; scores 2.4e-6 -> 1.1e-6 largest; single logits of normally distributed
// states with 1, 2, 4, 16 and 128 channels at work 3.6e-8, 3.4e-8, 3.1e-8, 2.9e-8, 2.8e-8 -> 3.6e-8, 3.1e-8, 2.5e-8, 1.6e-8, 1.0e-8 rms of
// the sum of their products' magnitudes, 1.6, 2.2, 2.9, 3.8, 3.9 -> 2.0, 2.2, 2.3, 2.7, 1.5 times 2^-24 largest.  (The softmax arithmetic a tile
// behind the matrix instructions, as in score_kernel: 3 % faster on 32768 tokens, 3 % slower on 4096.)
constexpr int kF32Waves = 4, kF32Tokens = 32;
constexpr int kF32Plane = kF32Tokens * 256, kF32Buffer = 3 * kF32Plane;  // bytes
constexpr int kF32Parts = 2 * kF32Waves, kF32Pitch = kF32Tokens + 4;    // pass 2's partial column results, floats
constexpr size_t kF32Lds = std::max<size_t>(2 * kF32Buffer + 2 * kF32Parts * kF32Pitch * sizeof(float), kF32Waves * 32 * 512);  // two tiles; Q first
static_assert(2 * kF32Parts * kF32Pitch >= kF32Waves * 32, "holds the rows' offsets first");

// m and l lie in the range of x as well (without a scale a number below 2^-110 lost the bits below 2^-134, which a large partner
// brings back: 1e-38 times 3.4e38 was 1e-3 off); 2^8 would take the largest floats' m to infinity.
constexpr float kPartScale = 128.0f;
struct Parts {
    uint4 h, m, l;  // x = h + m / kPartScale + l / kPartScale^2
};
constexpr float kLargestBf16 = 0x1.fep127f;
__device__ __forceinline__ Parts split3(const float4 &a, const float4 &b)
{
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
    const float x[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    auto round2 = [](float x0, float x1) { return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x0, x1}, bf16x2)); };
    auto near = [](float x) { return __builtin_amdgcn_fmed3f(x, -kLargestBf16, kLargestBf16); };  // (no finite number rounds to infinity)
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float x0 = x[2 * i], x1 = x[2 * i + 1];
        h[i] = round2(near(x0), near(x1));
        const float r0 = x0 - __uint_as_float(h[i] << 16), r1 = x1 - __uint_as_float(h[i] & 0xFFFF0000u);
        const float s0 = r0 * kPartScale, s1 = r1 * kPartScale;
        m[i] = round2(s0, s1);
        l[i] = round2((s0 - __uint_as_float(m[i] << 16)) * kPartScale, (s1 - __uint_as_float(m[i] & 0xFFFF0000u)) * kPartScale);
    }
    return {make_uint4(h[0], h[1], h[2], h[3]), make_uint4(m[0], m[1], m[2], m[3]), make_uint4(l[0], l[1], l[2], l[3])};
}

// BY_LDS: the query rows come by way of LDS.  Read straight into the registers, a load takes 32 bytes from each of 64 rows, and the loads of four
// wavefronts queue up; those of one or two are there before a copy that is read again behind the whole workgroup's barrier.  Measured,
// straight -> by LDS, the two passes: 128 rows a kv head, 4096 tokens, 32/8 heads 13.4 + 13.3 -> 12.8 + 12.5 us; 9220 tokens, 96 rows 22.4 + 21.6
// -> 21.9 + 21.7, 72 21.8 + 21.0 -> 21.6 + 21.0, 64 21.1 + 20.3 -> 21.0 + 20.9, 32 19.7 + 19.8 -> 20.5 + 20.6; 40 rows, 30000 tokens, 16/4 26.7 + 25.8
// -> 27.2 + 26.7.
constexpr int kF32StraightRows = 64;
template <int MODE, int RMAX, bool BY_LDS>
__global__ __launch_bounds__(kF32Waves * 64, 2) void score_f32_kernel(const ScoreArgs a)
{
    using T = Bf16;
    constexpr int THREADS = kF32Waves * 64, ROWS = kF32Waves * 32, STEPS = 8;
    constexpr int CHUNKS = kF32Tokens * 16 / THREADS;  // of 8 elements a thread fetches of a tile
    extern __shared__ __align__(16) unsigned char smem[];
    // workgroups that stream the same K range run on one XCD (see score_kernel)
    const int xcd = blockIdx.x % kNumXCD, slot = blockIdx.x / kNumXCD, qb = slot % a.nqb;
    const int64_t pair = (int64_t)(slot / a.nqb) * kNumXCD + xcd;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, l32 = lane & 31, half = lane >> 5;
    if (MODE == 1 && blockIdx.x == 0)
        for (uint32_t i = tid * 4; i < a.clear.n; i += THREADS * 4) *(uint4 *)&a.clear.at[i] = make_uint4(0, 0, 0, 0);
    if (pair >= (int64_t)a.Hkv * a.nsplit) return;
    const int g = (int)(pair / a.nsplit), split = (int)(pair % a.nsplit);
    const int64_t tile0 = (int64_t)split * a.tiles_per_split;
    const int64_t tile1 = tile0 + a.tiles_per_split < a.ntiles ? tile0 + a.tiles_per_split : a.ntiles;
    if (tile0 >= tile1) return;
    const int64_t nrows = (int64_t)a.Hq * a.Lq;
    const int rl = qb * ROWS + wave * 32 + l32;  // the lane's query row in the group
    float *red = (float *)(smem + 2 * kF32Buffer);  // [2][kF32Parts][kF32Pitch], pass 2 only

    const unsigned char *kbase = (const unsigned char *)a.k + (int64_t)g * a.k_stride_head * 4;
    auto first_token = [&](int64_t tile) { return (MODE == 1 ? tile0 + tile1 - 1 - tile : tile) * kF32Tokens; };
    float4 raw[CHUNKS][2];
    auto fetch = [&](int64_t tile) {
#pragma unroll
        for (int j = 0; j < CHUNKS; ++j) {
            const int id = j * THREADS + tid;
            const int64_t tok = first_token(tile) + (id >> 4);
            const unsigned char *src = kbase + (tok < a.L ? tok : a.L - 1) * (a.k_stride_token * 4) + (id & 15) * 32;
            raw[j][0] = *(const float4 *)src;
            raw[j][1] = *(const float4 *)(src + 16);
        }
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int j = 0; j < CHUNKS; ++j) {
            const int id = j * THREADS + tid, row = id >> 4;
            unsigned char *dst = smem + buf * kF32Buffer + row * 256 + ((id & 15) ^ (row & 15)) * 16;
            const Parts x = split3(raw[j][0], raw[j][1]);
            *(uint4 *)dst = x.h;
            *(uint4 *)(dst + kF32Plane) = x.m;
            *(uint4 *)(dst + 2 * kF32Plane) = x.l;
        }
    };
    // pass 2: see score_rows
    constexpr int SHARERS = THREADS / ROWS;
    const int off_row = qb * ROWS + tid / SHARERS;
    RowParts<SHARERS, 2> parts;
    float stat_m, stat_z;
    if (MODE == 1) {
        const int64_t r = (int64_t)g * a.rows_per_group + min(off_row, a.rows_per_group - 1);
        if (a.merge) {
            parts.load(a.part_m + r, a.part_z + r, a.nsplit, nrows, tid % SHARERS);
        } else {
            stat_m = a.row_max[r];
            stat_z = a.row_sumexp[r];
        }
    }
    fetch(tile0);

    Parts qf[STEPS];
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    if constexpr (BY_LDS) {
        // As in score_rows: 16-byte chunks, chunk c of row r at c ^ r, rows past the group's last one read as that one.  A wavefront without a row
        // copies none, it would only stand in the others' way.
        const int rl0 = qb * ROWS + wave * 32;
        const unsigned qlds = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char *)smem + wave * (32 * 512);
        auto copy = [&](auto row_at) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {  // two rows at a time
                const int row = j * 2 + half;
                lds_dma16(row_at(row) + ((l32 ^ row) * 16), __builtin_amdgcn_readfirstlane(qlds + j * 1024));
            }
        };
        if (__builtin_amdgcn_readfirstlane(rl0) < a.rows_per_group) {
            const int64_t row_bytes = a.q_stride_token * 4, head_bytes = a.q_stride_head * 4;
            if (a.q_stride_head == (int64_t)a.Lq * a.q_stride_token) {  // uniform: a head's rows follow the one's before
                const uint64_t first = (uint64_t)a.q + (uint64_t)((int64_t)g * a.G * head_bytes);
                copy([&](int row) { return first + (uint64_t)(min(rl0 + row, a.rows_per_group - 1) * row_bytes); });
            } else {  // lane l32 works out where row l32 lies
                const int at = min(rl, a.rows_per_group - 1);
                const uint64_t own = (uint64_t)a.q + (uint64_t)((int64_t)(g * a.G + at / a.Lq) * head_bytes + (int64_t)(at % a.Lq) * row_bytes);
                copy([&](int row) { return (uint64_t)(uint32_t)__shfl((int)(uint32_t)(own >> 32), row) << 32 | (uint32_t)__shfl((int)(uint32_t)own, row); });
            }
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const unsigned char *src = smem + wave * (32 * 512) + l32 * 512;
            const int c = 2 * (2 * st + half);
            const float4 x = *(const float4 *)(src + (c ^ l32) * 16), y = *(const float4 *)(src + ((c + 1) ^ l32) * 16);
            qf[st] = split3(rl < a.rows_per_group ? x : zero, rl < a.rows_per_group ? y : zero);
        }
        __syncthreads();  // the tiles go to the same place
    } else {
        const bool real = rl < a.rows_per_group;
        const int at = real ? rl : 0, h = g * a.G + at / a.Lq, i = at % a.Lq;
        const unsigned char *src = (const unsigned char *)a.q + ((int64_t)h * a.q_stride_head + (int64_t)i * a.q_stride_token) * 4;
        float4 x[STEPS][2];
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            x[st][0] = *(const float4 *)(src + (st * 2 + half) * 32);
            x[st][1] = *(const float4 *)(src + (st * 2 + half) * 32 + 16);
        }
#pragma unroll
        for (int st = 0; st < STEPS; ++st) qf[st] = split3(real ? x[st][0] : zero, real ? x[st][1] : zero);
    }

    float m = kNegBig, z[4] = {0.f, 0.f, 0.f, 0.f};  // pass 1
    float noff[MODE == 1 ? 16 : 1];                  // pass 2, see score_kernel
    if (MODE == 1) {
        const float off = a.merge ? parts.offset(a.nsplit, tid % SHARERS) : row_offset(stat_m, stat_z);
        if (tid % SHARERS == 0) red[tid / SHARERS] = off_row < a.rows_per_group ? off : -INFINITY;
    }
    stage(0);
    if (tile0 + 1 < tile1) fetch(tile0 + 1);
    __syncthreads();
    if (MODE == 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float4 x = *(const float4 *)&red[wave * 32 + 8 * j + 4 * half];
            noff[4 * j] = x.x, noff[4 * j + 1] = x.y, noff[4 * j + 2] = x.z, noff[4 * j + 3] = x.w;
        }
        __syncthreads();  // the buffers are written from here on
    }

    unsigned frag[STEPS];
#pragma unroll
    for (int st = 0; st < STEPS; ++st) frag[st] = (unsigned)(l32 * 256 + (((2 * st + half) ^ (l32 & 15)) * 16));
    const int unit = g * a.nqb + qb;
    for (int64_t tile = tile0; tile < tile1; ++tile) {
        const int buf = (int)(tile - tile0) & 1;
        if (tile + 1 < tile1) {
            stage(buf ^ 1);
            if (tile + 2 < tile1) fetch(tile + 2);
        }
        f32x16 big, s1, s2;  // of the logits, kPartScale and kPartScale^2 times them
#pragma unroll
        for (int v = 0; v < 16; ++v) big[v] = s1[v] = s2[v] = 0.f;
        const unsigned char *kb = smem + buf * kF32Buffer;
        auto mma = [](f32x16 &acc, const uint4 &k, const uint4 &q) {
            if (MODE == 0)
                T::mma(acc, k, q);
            else
                T::mma(acc, q, k);
        };
#pragma unroll
        for (int st = 0; st < STEPS; ++st) {
            const uint4 kh = *(const uint4 *)(kb + frag[st]), km = *(const uint4 *)(kb + frag[st] + kF32Plane),
                        kl = *(const uint4 *)(kb + frag[st] + 2 * kF32Plane);
            mma(s2, kh, qf[st].l);
            mma(s1, km, qf[st].h);
            mma(s2, kl, qf[st].h);
            mma(s1, kh, qf[st].m);
            mma(s2, km, qf[st].m);
            mma(big, kh, qf[st].h);
        }
        const int64_t tok0 = first_token(tile);
#pragma unroll
        for (int v = 0; v < 16; ++v) big[v] = fmaf(fmaf(s2[v], 1.0f / kPartScale, s1[v]), 1.0f / kPartScale, big[v]);
        if (MODE == 0) {
            if (tok0 + kF32Tokens > a.L)  // uniform
                row_update<true>(big, a.c, m, z, tok0 + 4 * half, a.L);
            else
                row_update<false>(big, a.c, m, z, tok0 + 4 * half, a.L);
        } else {
            float p[4];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float x = fmaf(big[v], a.c, noff[v]);
                const float e = RMAX ? x : fast_exp2(x);
                p[v & 3] = v < 4 ? e : RMAX ? fmaxf(p[v & 3], e) : p[v & 3] + e;
            }
            red[(buf * kF32Parts + wave * 2 + half) * kF32Pitch + l32] =
                RMAX ? fmaxf(fmaxf(p[0], p[1]), fmaxf(p[2], p[3])) : (p[0] + p[1]) + (p[2] + p[3]);
        }
        __syncthreads();
        // the wavefronts' results of the tile's tokens, in a fixed order, by one of them
        if (MODE == 1 && wave == (int)((tile - tile0) & 3) && half == 0) {
            float x[kF32Parts];
#pragma unroll
            for (int i = 0; i < kF32Parts; ++i) x[i] = red[(buf * kF32Parts + i) * kF32Pitch + l32];
#pragma unroll
            for (int o = 1; o < kF32Parts; o <<= 1)
#pragma unroll
                for (int i = 0; i < kF32Parts; i += 2 * o) x[i] = RMAX ? fmaxf(x[i], x[i + o]) : x[i] + x[i + o];
            if (tok0 + l32 < a.L) a.partial[(int64_t)unit * a.L + tok0 + l32] = RMAX ? fast_exp2(x[0]) : x[0];
        }
    }
    if (MODE == 0) {  // the half-waves saw disjoint tokens of the same rows
        const float zb = (z[0] + z[1]) + (z[2] + z[3]);
        const float mo = __shfl_xor(m, 32), zo = __shfl_xor(zb, 32), mm = fmaxf(m, mo);
        const float zz = zb * fast_exp2(m - mm) + zo * fast_exp2(mo - mm);
        if (half == 0 && rl < a.rows_per_group) {
            const int64_t r = (int64_t)g * a.rows_per_group + rl;
            a.part_m[(int64_t)split * nrows + r] = mm;
            a.part_z[(int64_t)split * nrows + r] = zz;
        }
    }
}

// Pass 2's token ranges from pass 1's workgroup times.  The 8 XCDs of the chip do not run at one speed (their
// workgroups finish up to 6 % apart, the same dies ahead in every launch), and a launch lasts as long as its
// slowest XCD.  Split s of every kv head runs on the same XCD when the splits per head are a multiple of 8, so
// the ranges are sized by the mean time the workgroups of split s took in pass 1: range s gets a share of the
// tiles proportional to 1 / time, within 15 % of an even share (a workgroup that walked its split twice, or a
// disturbed launch, must not skew the next one).  Only pass 2 is cut this way: its results do not depend on the
// cut, pass 1's rounding would.
constexpr int kMaxBalancedSplits = 512;
struct BalanceArgs {
    const uint32_t *wg_time;  // null: no table wanted
    int32_t *table;           // [2 + nsplit + 1]: tag (low, high), then the first tile of every range and ntiles
    uint64_t tag;
    int grid, nqb, nsplit, Hkv;
    int64_t ntiles;
};
__device__ void make_split_table(const BalanceArgs &b)
{
    __shared__ uint32_t sum[kMaxBalancedSplits], cnt[kMaxBalancedSplits];
    for (int s = threadIdx.x; s < b.nsplit; s += blockDim.x) sum[s] = cnt[s] = 0;
    __syncthreads();
    for (int w = threadIdx.x; w < b.grid; w += blockDim.x) {
        const uint32_t t = b.wg_time[w];
        const int64_t pair = (int64_t)((w / kNumXCD) / b.nqb) * kNumXCD + w % kNumXCD;
        if (t != 0 && pair < (int64_t)b.Hkv * b.nsplit) {
            atomicAdd(&sum[pair % b.nsplit], t >> 4);  // 160 ns units: the sum over all workgroups of a split fits
            atomicAdd(&cnt[pair % b.nsplit], 1u);
        }
    }
    __syncthreads();
    // One wavefront, eight splits a lane: mean time per split, weight = mean of those over the split's own,
    // running sum of the weights, edges.  (One thread doing this in a loop was a 20 us chain at 32 splits.)
    if (threadIdx.x >= 64) return;
    constexpr int kPer = kMaxBalancedSplits / 64;
    const int lane = threadIdx.x;
    float d[kPer], lsum = 0.f, lcnt = 0.f;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int sp = lane * kPer + k;
        d[k] = (sp < b.nsplit && cnt[sp] && sum[sp]) ? (float)sum[sp] / (float)cnt[sp] : 0.f;
        lsum += d[k];
        lcnt += d[k] > 0.f ? 1.f : 0.f;
    }
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        lsum += __shfl_xor(lsum, o);
        lcnt += __shfl_xor(lcnt, o);
    }
    const float mean = lcnt > 0.f ? lsum / lcnt : 1.f;
    float w[kPer], lw = 0.f;
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int sp = lane * kPer + k;
        float x = d[k] > 0.f ? mean / d[k] : 1.f;
        x = x < 0.85f ? 0.85f : (x > 1.15f ? 1.15f : x);
        w[k] = sp < b.nsplit ? x : 0.f;
        lw += w[k];
    }
    float incl = lw;  // inclusive running sum over the lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const float up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
    }
    const float weights = __shfl(incl, 63);
    float upto = incl - lw;
    if (lane == 0) {
        b.table[0] = (int32_t)(uint32_t)b.tag;
        b.table[1] = (int32_t)(uint32_t)(b.tag >> 32);
        b.table[2] = 0;
    }
#pragma unroll
    for (int k = 0; k < kPer; ++k) {
        const int sp = lane * kPer + k;
        upto += w[k];
        if (sp < b.nsplit) {
            int64_t edge = (int64_t)((double)b.ntiles * (double)(upto / weights) + 0.5);
            if (edge > b.ntiles || sp == b.nsplit - 1) edge = b.ntiles;
            b.table[3 + sp] = (int32_t)edge;  // non-decreasing: the running sum is, and so are the steps behind it
        }
    }
}

// Merge the per-split partial statistics of each row (fixed order) and convert to the natural-log units of
// Eq. 4: row_max = a reference <= max_t logit, row_sumexp = sum_t exp(logit - row_max).
// Sixteen lanes share a row and the splits among them, so that all of a row's partials are fetched in one
// round of loads (a thread a row would fetch them in a chain of memory latencies: this kernel sits between
// the two scoring passes and is all latency).
__global__ __launch_bounds__(256) void combine_row_stats(const float *part_m, const float *part_z, int nsplit, int64_t nrows,
                                                         float *row_max, float *row_sumexp, const BalanceArgs bal,
                                                         unsigned stat_blocks)
{
    constexpr int kBlock = 4;
    if (blockIdx.x >= stat_blocks) {  // one workgroup is there for the table alone
        make_split_table(bal);
        return;
    }
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int64_t r = gid / kCombineLanes;
    const int sub = (int)(gid % kCombineLanes);
    const int64_t rr = r < nrows ? r : nrows - 1;  // surplus groups redo the last row and store nothing
    float mm = kNegBig;
    for (int s0 = sub; s0 < nsplit; s0 += kCombineLanes * kBlock) {
        float m[kBlock];
#pragma unroll
        for (int i = 0; i < kBlock; ++i) {
            const int s = s0 + i * kCombineLanes;
            m[i] = part_m[(int64_t)(s < nsplit ? s : nsplit - 1) * nrows + rr];
        }
#pragma unroll
        for (int i = 0; i < kBlock; ++i) mm = fmaxf(mm, m[i]);
    }
#pragma unroll
    for (int o = 1; o < kCombineLanes; o <<= 1) mm = fmaxf(mm, __shfl_xor(mm, o));
    float zz = 0.f;
    for (int s0 = sub; s0 < nsplit; s0 += kCombineLanes * kBlock) {
        float m[kBlock], z[kBlock];
#pragma unroll
        for (int i = 0; i < kBlock; ++i) {
            const int s = s0 + i * kCombineLanes;
            const int64_t at = (int64_t)(s < nsplit ? s : nsplit - 1) * nrows + rr;
            m[i] = part_m[at];
            z[i] = part_z[at];
        }
#pragma unroll
        for (int i = 0; i < kBlock; ++i)
            if (s0 + i * kCombineLanes < nsplit) zz = fmaf(z[i], fast_exp2(m[i] - mm), zz);
    }
#pragma unroll
    for (int o = 1; o < kCombineLanes; o <<= 1) zz += __shfl_xor(zz, o);
    if (sub != 0 || r >= nrows) return;
    row_max[r] = mm * kLn2;
    row_sumexp[r] = zz;
}

// score[t] = sum (or max) over the (kv head, query block) units of their partial column results.
template <int RMAX>
__global__ void reduce_units(const float *partial, int nunits, int64_t L, float *score)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= L) return;
    // eight units at a time, their loads issued together; the sum runs in unit order
    constexpr int kBlock = 8;
    float acc = 0.f;
    for (int u0 = 0; u0 < nunits; u0 += kBlock) {
        float x[kBlock];
#pragma unroll
        for (int i = 0; i < kBlock; ++i) x[i] = partial[(int64_t)(u0 + i < nunits ? u0 + i : nunits - 1) * L + t];
#pragma unroll
        for (int i = 0; i < kBlock; ++i) {
            if (u0 + i >= nunits) break;
            if (u0 + i == 0)
                acc = x[i];
            else
                acc = RMAX ? fmaxf(acc, x[i]) : acc + x[i];
        }
    }
    score[t] = acc;
}

// of three tiles, of two tiles and 32 query rows a wavefront (as much as two tiles)
constexpr size_t tile_lds_bytes(int waves, int tiles) { return tiles * (size_t)Bf16::tile_tokens(waves) * (Bf16::kChunksPerRow * 16); }

// Behind the query rows, which start behind two tiles: pass 1's flag, or the offsets of pass 2's rows.
constexpr size_t stats_lds_bytes(int waves) { return tile_lds_bytes(waves, 4) + 16; }
constexpr size_t cols_lds_bytes(int waves, int rows)
{
    return std::max(tile_lds_bytes(waves, 4) + rows * sizeof(float),
                    tile_lds_bytes(waves, 3) + 3 * 2 * (size_t)waves * (Bf16::tile_tokens(waves) + 36) * sizeof(float));  // pitch <= tokens + 36
}

// The dynamic-LDS ceiling of a kernel is raised once per process (beyond the most any plan asks of it: 8 wavefronts' query rows
// behind two tiles, and their offsets), not on every launch.
constexpr int kMaxDynamicLds = 144 * 1024;  // leaves room for the few bytes of static LDS a kernel may hold
static_assert(std::max(stats_lds_bytes(8), cols_lds_bytes(8, 512)) <= kMaxDynamicLds && kF32Lds <= kMaxDynamicLds, "room for every plan");
hipError_t raise_lds_limit_once(const void *kernel)
{
    static std::mutex mutex;
    static const void *done[32];
    static int ndone = 0;
    std::lock_guard<std::mutex> lock(mutex);
    for (int i = 0; i < ndone; ++i)
        if (done[i] == kernel) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kMaxDynamicLds);
    if (e == hipSuccess && ndone < 32) done[ndone++] = kernel;
    return e;
}

template <typename K>
hipError_t launch_score(K kernel, int grid, int threads, size_t lds, const ScoreArgs &a, hipStream_t s)
{
    hipError_t e = raise_lds_limit_once((const void *)kernel);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), lds, s, a);
    return hipGetLastError();
}

}  // namespace

ScorePlan make_score_plan(int dtype, int64_t L, int Lq, int Hq, int Hkv, bool roomy)
{
    ScorePlan p{};
    p.dtype = dtype;
    const int G = Hq / Hkv;
    p.rows_per_group = G * Lq;
    if (dtype == ILRE_F32) {
        p.waves = 4;
        p.nb = 1;
    } else {
        // 8 waves (512 rows) unless 4 waves (256 rows) leave fewer padded rows.  Up to 128 rows take one 32-row block a
        // wavefront: half the matrix work of a mostly padded 256, and what is left is the K stream (100003 tokens, 4 kv
        // heads, 119 rows each: 31.0 -> 22.0 us a pass, 4.7 TB/s).  More rows do not: a K fragment then feeds one MFMA
        // instead of two, about 1.2 times as much per row (50001 tokens, 8 kv heads, 384 rows each: three blocks of
        // 128 rows 52.5 + 53.7 us and 16 more score vectors to add up, one padded block of 512 60.1 + 55.0 us).
        const int64_t pad8 = ((p.rows_per_group + 511) / 512) * 512;
        const int64_t pad4 = ((p.rows_per_group + 255) / 256) * 256;
        p.waves = pad4 < pad8 ? 4 : 8;
        p.nb = p.rows_per_group <= 128 ? 1 : 2;
        // 257 - 384 rows: a block of 256 and one of 128, which a quarter of 512 would be padding for (whole recall, 384 rows a kv head,
        // 9000 tokens 64.5 -> 60.3 us, 50001 130.2 -> 124.0, 400000 799 -> 755; 280 rows, 131072 tokens 251 -> 240).  513 - 640 rows as
        // two and one are no faster than three, the larger blocks decide: 600 rows, 131072 tokens 411 and 405 us, 800 of 4 heads 259 and 274.
        p.mixed = roomy && p.rows_per_group > 256 && p.rows_per_group <= 384;
        if (p.mixed) p.waves = 4;
    }
    p.tile_tokens = dtype == ILRE_F32 ? kF32Tokens : Bf16::tile_tokens(p.waves);
    p.rows_per_wg = p.waves * p.nb * 32;
    p.nqb = (p.rows_per_group + p.rows_per_wg - 1) / p.rows_per_wg;
    p.ntiles = (L + p.tile_tokens - 1) / p.tile_tokens;
    p.nunits = Hkv * p.nqb;
    // As many splits as there is room for at a time: one workgroup of 8 waves (two of 4 waves) a compute unit, and on each XCD no
    // more workgroups than that, because one too many runs behind all others, for as long as they do.  (Splits rounded up to
    // the next number, 131072 tokens: 28/4 heads, 630 rows a kv head, 516 workgroups 299 us a call, 504 232; 64/8, 1360 rows, 528 1282
    // us, 480 816; 28/4, 1050 rows, 500 workgroups, but 65 on some XCDs 468 us, 480, 60 an XCD, 381.)
    // Several rounds of workgroups where that takes a quarter off the tiles one place goes through, two a workgroup for its start
    // counted in: query blocks that are many against an XCD's places leave most of them empty otherwise, or have no round of their own.
    // (One round, then so, 131072 tokens: 16/2 heads, 2080 queries 10.81 -> 2.37 ms, 64/4, 1360 11.77 -> 5.69, 32/1, 540 12.17 -> 1.34, 40/5, 1280
    // 6.11 -> 3.90; fp32, 32768 tokens, 32/1, 260 6.85 -> 0.91.  Splits rounded up: 2.90, 6.14, 1.79, 4.73, 1.63.)
    const int room = kNumCU / kNumXCD * (p.waves == 8 ? 1 : 2);
    const int64_t step = dtype == ILRE_F32 ? 2 : 1;  // a split's tiles come in twos there
    auto cut = [&](int rounds) {
        int64_t nsplit = std::max<int64_t>((int64_t)kNumXCD * ((int64_t)rounds * room / p.nqb) / Hkv, 1);
        nsplit = std::min(nsplit, (p.ntiles + step - 1) / step);
        auto into = [&](int64_t n) {
            p.tiles_per_split = step * ((p.ntiles + step * n - 1) / (step * n));
            p.nsplit = (int)((p.ntiles + p.tiles_per_split - 1) / p.tiles_per_split);
            return ((int64_t)p.nunits * p.nsplit + kNumCU - 1) / kNumCU * p.tiles_per_split;  // tiles of the busiest compute unit
        };
        const int64_t busiest = into(nsplit);
        // fp32, few tiles: no more splits than pass 2 merges itself, unless a compute unit then has more to do (32 queries, 32/8 heads, 4096
        // tokens 41.3 -> 38.8 us, 6000 52.2 -> 47.4; 24/6 heads, 3000 41.6 -> 38.4, but 2100, 4 tiles instead of 2, 35.2 -> 38.1; 16 queries, 16/4
        // heads, 4096 34.0 -> 36.7).  Beyond 6 tiles a split it gains nothing: 24/6 heads, 6500 tokens 52.1 -> 53.6, 32/8, 8192 53.8 either way.
        if (dtype == ILRE_F32 && p.nsplit > kMergeSplits && p.ntiles <= 6 * kMergeSplits && into(kMergeSplits) > busiest && roomy) into(nsplit);
        const int64_t on_xcd = ((int64_t)Hkv * p.nsplit + kNumXCD - 1) / kNumXCD * p.nqb;
        return (on_xcd + room - 1) / room * (p.tiles_per_split + 2);
    };
    int rounds = 1;
    int64_t least = cut(1);
    for (int r = std::max(2, p.nqb / room); roomy && r <= 4 + p.nqb / room; ++r) {  // (fewer hold no split of every query block)
        const int64_t tiles = cut(r);
        if (4 * tiles < 3 * least) {
            rounds = r;
            least = tiles;
        }
    }
    cut(rounds);
    const int64_t pairs = (int64_t)Hkv * p.nsplit;
    p.grid = (int)(((pairs + kNumXCD - 1) / kNumXCD) * kNumXCD * p.nqb);
    // pass 2's ranges follow the XCDs' speed where a range is long enough for that to matter
    p.balanced = dtype != ILRE_F32 && p.tiles_per_split >= 64 && p.nsplit >= kNumXCD && p.nsplit <= kMaxBalancedSplits;
    p.merge_in_cols = !p.balanced && p.nsplit <= (dtype == ILRE_F32 || p.mixed ? 1 : 2) * kMergeSplits;
    uint64_t tag = 0x494c52652d584344ull;  // what a table has to have been made for
    for (uint64_t v : {(uint64_t)L, (uint64_t)p.ntiles, (uint64_t)p.nsplit, (uint64_t)p.nqb, (uint64_t)Hkv, (uint64_t)p.tile_tokens,
                       (uint64_t)p.grid})
        tag = (tag ^ v) * 0x9E3779B97F4A7C15ull + 0x7F4A7C15ull;
    p.table_tag = tag;
    p.lds_bytes_stats = p.lds_bytes_cols = kF32Lds;
    if (dtype == ILRE_F32) return p;
    p.lds_bytes_stats = stats_lds_bytes(p.waves);
    p.lds_bytes_cols = cols_lds_bytes(p.waves, p.rows_per_wg);
    return p;
}

hipError_t launch_row_stats(const ScorePlan &p, const ScoreArgs &a, float *row_max, float *row_sumexp, hipStream_t s)
{
    // One launch: a workgroup whose sums against frozen references leave the safe range walks its split a second
    // time in the always-safe form before it writes its partials.
    const size_t lds = p.lds_bytes_stats;
    const int64_t nrows = (int64_t)a.Hq * a.Lq;
    hipError_t e;
    if (p.dtype == ILRE_F32)
        e = p.rows_per_group > kF32StraightRows ? launch_score(score_f32_kernel<0, 0, true>, p.grid, kF32Waves * 64, lds, a, s)
                                                : launch_score(score_f32_kernel<0, 0, false>, p.grid, kF32Waves * 64, lds, a, s);
    else if (p.nb == 1)
        e = launch_score(score_kernel<1, 4, 0, 0, false>, p.grid, 256, lds, a, s);
    else if (p.mixed)
        e = launch_score(score_kernel<2, 4, 0, 0, true>, p.grid, 256, lds, a, s);
    else if (p.waves == 4)
        e = launch_score(score_kernel<2, 4, 0, 0, false>, p.grid, 256, lds, a, s);
    else
        e = launch_score(score_kernel<2, 8, 0, 0, false>, p.grid, 512, lds, a, s);
    if (e != hipSuccess) return e;
    if (a.merge) return hipSuccess;  // pass 2 takes the partials
    const bool balance = a.wg_time != nullptr && a.split_table != nullptr;
    const BalanceArgs bal{balance ? a.wg_time : nullptr, a.split_table, a.table_tag, p.grid, p.nqb, p.nsplit, a.Hkv, p.ntiles};
    const unsigned stat_blocks = (unsigned)((nrows * kCombineLanes + 255) / 256);
    hipLaunchKernelGGL(combine_row_stats, dim3(stat_blocks + (balance ? 1u : 0u)), dim3(256), 0, s, a.part_m, a.part_z, a.nsplit, nrows,
                       row_max, row_sumexp, bal, stat_blocks);
    return hipGetLastError();
}

hipError_t launch_reduce_units(const float *partial, int nunits, int64_t L, int rmax, float *out_scores, hipStream_t s)
{
    const unsigned blocks = (unsigned)((L + 255) / 256);
    if (rmax)
        hipLaunchKernelGGL(reduce_units<1>, dim3(blocks), dim3(256), 0, s, partial, nunits, L, out_scores);
    else
        hipLaunchKernelGGL(reduce_units<0>, dim3(blocks), dim3(256), 0, s, partial, nunits, L, out_scores);
    return hipGetLastError();
}

hipError_t launch_col_scores(const ScorePlan &p, const ScoreArgs &a, int score_mode, float *out_scores, hipStream_t s, bool reduce)
{
    hipError_t e;
    const size_t lds = p.lds_bytes_cols;
    const bool mx = score_mode == ILRE_SCORE_MAX;
    if (p.dtype == ILRE_F32 && p.rows_per_group > kF32StraightRows)
        e = mx ? launch_score(score_f32_kernel<1, 1, true>, p.grid, kF32Waves * 64, lds, a, s)
               : launch_score(score_f32_kernel<1, 0, true>, p.grid, kF32Waves * 64, lds, a, s);
    else if (p.dtype == ILRE_F32)
        e = mx ? launch_score(score_f32_kernel<1, 1, false>, p.grid, kF32Waves * 64, lds, a, s)
               : launch_score(score_f32_kernel<1, 0, false>, p.grid, kF32Waves * 64, lds, a, s);
    else if (p.nb == 1)
        e = mx ? launch_score(score_kernel<1, 4, 1, 1, false, true>, p.grid, 256, lds, a, s)
               : launch_score(score_kernel<1, 4, 1, 0, false, true>, p.grid, 256, lds, a, s);
    else if (p.mixed)
        e = mx ? launch_score(score_kernel<2, 4, 1, 1, true>, p.grid, 256, lds, a, s)
               : launch_score(score_kernel<2, 4, 1, 0, true>, p.grid, 256, lds, a, s);
    else if (p.waves == 4 && a.merge && a.nsplit > kMergeSplits)  // (of its own: with both in one kernel up to 32 splits took 0.4 % longer)
        e = mx ? launch_score(score_kernel<2, 4, 1, 1, false, true>, p.grid, 256, lds, a, s)
               : launch_score(score_kernel<2, 4, 1, 0, false, true>, p.grid, 256, lds, a, s);
    else if (p.waves == 4)
        e = mx ? launch_score(score_kernel<2, 4, 1, 1, false>, p.grid, 256, lds, a, s)
               : launch_score(score_kernel<2, 4, 1, 0, false>, p.grid, 256, lds, a, s);
    else if (a.merge && a.nsplit > kMergeSplits)
        e = mx ? launch_score(score_kernel<2, 8, 1, 1, false, true>, p.grid, 512, lds, a, s)
               : launch_score(score_kernel<2, 8, 1, 0, false, true>, p.grid, 512, lds, a, s);
    else
        e = mx ? launch_score(score_kernel<2, 8, 1, 1, false>, p.grid, 512, lds, a, s)
               : launch_score(score_kernel<2, 8, 1, 0, false>, p.grid, 512, lds, a, s);
    if (e != hipSuccess || !reduce) return e;
    return launch_reduce_units(a.partial, p.nunits, a.L, mx ? 1 : 0, out_scores, s);
}

}  // namespace ilre
