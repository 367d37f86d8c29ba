// Clustered-head attention over a block of prompt positions (the prefill that follows the membership decision;
// Section 3.5, attention definition of Section 2 with the causal mask of a decoder-only model).  Many query rows
// per key make this the one compute-bound step of the method, so it runs on the matrix cores: a flash-style
// kernel (scores, online softmax and output accumulation tile by tile, nothing T x T ever leaves the chip) in
// which the score tile of a cluster is computed ONCE from the representative's queries and keys and then applied
// to the values of up to kGroup member heads -- the saving the method is about.
//
// MFMA tiles (v_mfma_f32_32x32x16, wave64), lane l = (r = l % 32, hl = l / 32):
//   A[32][16]: lane holds A[r][8*hl .. 8*hl+7]     B[16][32]: lane holds B[8*hl .. 8*hl+7][r]
//   D[32][32]: lane holds D[(v/4)*8 + hl*4 + v%4][r] for v = 0..15
// Scores are computed transposed, S^T = K_tile Q^T (bf16 inputs): a lane then owns ONE query column and half of
// the keys of the tile, so row maxima and sums are in-lane plus one exchange with lane l^32, and the tile of
// probabilities is already in the A-operand layout of O += P V: a lane then has one column of 16 rows in an
// accumulator tile, and what is per row (the factors of a rescaling, one over the row sum) comes from the lanes
// that own the rows.  (As O^T += V^T P^T, the same registers in the other order, a lane had its own row's factors, but
// every 16-byte store of an output row touched 64 cache lines, and the output rows of a query tile cost as much as four
// tiles of keys.)  That second product runs in fp16 (P in [0,256] keeps 11 bits instead of bf16's 8).  Its B operand
// needs 8 keys of one value column per lane, which a
// row-major V cache cannot deliver, so a first kernel writes V^T once per call: fp16 (exact from bf16 inside
// the fp16 range, |v| <= 65504), in blocks of 64 keys x 128 columns, keys permuted inside every group of 16 into
// the order the probability registers have, zero beyond the last key.  The main kernel then stages K and V^T
// tiles in LDS with 16-byte direct loads and feeds every MFMA operand with one ds_read_b128.  Calls with few query tiles
// per head do without that kernel and its pass over all values: their workgroups take the rows of V themselves, and the
// conversion transposes on the way into LDS (prefill_direct_kernel).  (The LDS transpose reads of this chip could hand the
// operand over from a row-major bf16 tile, but only as bf16: the probabilities would then be rounded to 8 bits as well, up to
// 2^-9 of relative error per element, which is the whole error budget of the 16-bit contract.)
#include "chai_internal.h"

#include <hip/hip_ext.h>

#include <type_traits>
#include <utility>

namespace chai {

namespace {

constexpr int kGroup = 2;          // member heads that share one score tile
constexpr int kRec = 2 + kGroup;   // ints per work-list record: cluster and member count, members, representative
constexpr int kRecCount = 24;      // the member count stands above this bit of a record's first word
constexpr int kKTile = 64;         // keys per tile
constexpr int kXcds = 8;
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kRescaleSlack = 8.0f;      // log2 units a tile may exceed the running maximum before a rescale

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

union Frag16 {            // 16 bytes seen as a raw load, bf16 x 8 or fp16 x 8
    u32x4 raw;
    bf16x8 bf;
    f16x8 h;
};

// Both halves of a wave get x of lanes 0..31 and x of lanes 32..63 (lane l and lane l ^ 32 see the same pair, in
// the same order): one v_permlane32_swap instead of a round trip through the LDS crossbar.
__device__ __forceinline__ void both_halves(float x, float &lo, float &hi)
{
    const unsigned int bits = __float_as_uint(x);
    const auto sw = __builtin_amdgcn_permlane32_swap(bits, bits, false, false);
    lo = __uint_as_float(sw[0]);
    hi = __uint_as_float(sw[1]);
}

// Position of key jj (0..15) inside its group of 16 in V^T: lane half hl of MFMA step s multiplies its
// probability registers e = 0..7, which hold keys 16s + (e/4)*8 + hl*4 + e%4, with 8 consecutive halves.
__device__ __forceinline__ int key_slot16(int r16) { return 8 * ((r16 & 7) >> 2) + 4 * (r16 >> 3) + (r16 & 3); }

// Row of V^T that holds value column d: the columns 4 r + 0 .. 3 are row r of its four blocks of 32, so that a lane of the second
// product has four neighbouring columns of an output row in its four accumulator tiles, and a store writes whole rows.
__host__ __device__ constexpr int value_row(int d) { return (d & 3) * 32 + (d >> 2); }

// ---------------------------------------------------------------------------------------------------------
// Work list: the heads of every cluster, in ascending order, cut into groups of at most kGroup members.
// groups[b][g] = {cluster | n << kRecCount, head_0 .., representative}, kRec ints per record; clusters in ascending order.  One
// workgroup per batch row: the membership row is copied to LDS, thread j counts cluster j, thread h ranks head h among
// the heads of its cluster, and every head writes its own slot.  Heads that name no live cluster are left out.
// lds: (H + 2k) ints.
// ---------------------------------------------------------------------------------------------------------
__device__ __forceinline__ void plan_row(const int32_t *__restrict__ h2c, const int32_t *__restrict__ rep, int H, int k,
                                         int max_groups, int32_t *__restrict__ groups, int32_t *__restrict__ n_groups,
                                         int b, int32_t *lds)
{
    int32_t *member = lds, *count = lds + H, *base = count + k;
    const int tid = threadIdx.x, n_thr = blockDim.x;
    for (int h = tid; h < H; h += n_thr) {
        const int c = h2c[(size_t)b * H + h];
        member[h] = (c >= 0 && c < k && rep[(size_t)b * k + c] >= 0) ? c : -1;
    }
    __syncthreads();
    for (int j = tid; j < k; j += n_thr) {
        int n = 0;
        for (int h = 0; h < H; ++h) n += member[h] == j;
        count[j] = n;
    }
    __syncthreads();
    for (int j = tid; j < k; j += n_thr) {
        int first = 0;
        for (int i = 0; i < j; ++i) first += (count[i] + kGroup - 1) / kGroup;
        base[j] = first;
        if (j == k - 1) {
            const int ng = first + (count[j] + kGroup - 1) / kGroup;
            n_groups[b] = ng < max_groups ? ng : max_groups;
        }
    }
    __syncthreads();
    int32_t *g = groups + (size_t)b * max_groups * kRec;
    for (int h = tid; h < H; h += n_thr) {
        const int c = member[h];
        if (c < 0) continue;
        int rank = 0;
        for (int i = 0; i < h; ++i) rank += member[i] == c;
        const int gi = base[c] + rank / kGroup, slot = rank % kGroup;
        if (gi >= max_groups) continue;
        g[gi * kRec + 1 + slot] = h;
        if (slot == 0) {
            const int left = count[c] - rank;
            g[gi * kRec] = c | (left < kGroup ? left : kGroup) << kRecCount;
            g[gi * kRec + 1 + kGroup] = min(rep[(size_t)b * k + c], H - 1);
        }
    }
}

// ---------------------------------------------------------------------------------------------------------
// Pre-pass, one launch.  V^T in blocks of 64 keys: vt[b][h][t/64][value_row(d)][16*((t%64)/16) + key_slot16(t%16)] =
// fp16(V[b][h][t][d]) for t < n_keys, 0 up to Tp (a multiple of 64).  A block is 16 KB of consecutive memory with whole
// cache lines per value column, which is what the main kernels' direct loads to LDS ask for (rows of 64 bytes in blocks
// of 32 keys made each of those loads touch twice as many lines).  grid (n_lists + Tp/64 * H * B), 256 threads; a 64 x 128 tile
// goes through LDS.  The first n_lists workgroups make the work list, one per batch row (0 without maps; a launch of its
// own took 5 us for a few thousand instructions; as one workgroup more per head, all but B of them empty, 3 us on 520
// heads of one block).  Dynamic LDS: the tile, or what
// plan_row needs if that is more.
// ---------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prepass_kernel(const char *__restrict__ v, int H, int T_cap, int n_keys, int Tp,
                                                      _Float16 *__restrict__ vt, int n_lists, const int32_t *__restrict__ h2c,
                                                      const int32_t *__restrict__ rep, int k, int max_groups,
                                                      int32_t *__restrict__ groups, int32_t *__restrict__ n_groups,
                                                      int32_t *__restrict__ tickets, int ticket_stride)
{
    extern __shared__ __attribute__((aligned(16))) char pre_lds[];
    if (blockIdx.x == 0 && threadIdx.x < kXcds) tickets[(threadIdx.x >> 2) * ticket_stride + (threadIdx.x & 3)] = 0;
    _Float16 (*tile)[kKTile + 2] = reinterpret_cast<_Float16 (*)[kKTile + 2]>(pre_lds);
    const int tid = threadIdx.x;
    if ((int)blockIdx.x < n_lists) {
        plan_row(h2c, rep, H, k, max_groups, groups, n_groups, blockIdx.x, reinterpret_cast<int32_t *>(pre_lds));
        return;
    }
    const unsigned item = blockIdx.x - n_lists, n_blocks = (unsigned)Tp / kKTile, row = item / n_blocks;
    // (consecutive workgroups go to the 8 XCDs in turn: the blocks of a head begin one later every eight heads, or the last
    // blocks, which may hold a few keys only, would all meet on the same XCDs: 12 x 52 heads of 200 keys 20.4 -> 18.5 us)
    const int block = (int)((item - row * n_blocks + row / kXcds) % n_blocks), t0 = block * kKTile;
    const int h = (int)(row % (unsigned)H), b = (int)(row / (unsigned)H);
    const char *vhead = v + ((size_t)b * H + h) * (size_t)T_cap * (kHeadDim * 2);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int piece = tid + i * 256, jj = piece >> 4, c8 = piece & 15;       // key row, 8-column block
        Frag16 x;
        x.raw = u32x4{0u, 0u, 0u, 0u};
        if (t0 + jj < n_keys)
            x.raw = __builtin_nontemporal_load(reinterpret_cast<const u32x4 *>(vhead + (size_t)(t0 + jj) * (kHeadDim * 2) + c8 * 16));
        const int slot = 16 * (jj >> 4) + key_slot16(jj & 15);
#pragma unroll
        for (int e = 0; e < 8; ++e) tile[value_row(c8 * 8 + e)][slot] = (_Float16)(float)x.bf[e];
    }
    __syncthreads();
    _Float16 *dst = vt + (((size_t)b * H + h) * (Tp / kKTile) + block) * (size_t)(kHeadDim * kKTile);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int idx = tid + i * 256, c4 = idx & 15, dd = idx >> 4;                                       // 4 keys each
        const unsigned int lo = *reinterpret_cast<const unsigned int *>(&tile[dd][c4 * 4]);
        const unsigned int hi = *reinterpret_cast<const unsigned int *>(&tile[dd][c4 * 4 + 2]);
        *reinterpret_cast<uint2 *>(dst + (size_t)dd * kKTile + c4 * 4) = make_uint2(lo, hi);
    }
}

// ---------------------------------------------------------------------------------------------------------
// Main kernel.  Clustered: workgroups of NW = 4 waves, one per SIMD; a wave owns U (2 or 1) streams of 32 query rows and
// the accumulators of up to kGroup member heads for them (256 or 128 accumulation registers).  Dense attention (IDENT:
// every head its own cluster, the work list is not read) needs 64 of them, so that two waves fit a SIMD: NW = 8, U = 1.
//
// Per 32-key block i of its keys a wave has three independent pieces of work, from three successive blocks: the value
// products of block i-1, the softmax of block i, the score products of block i+1.  One straight stretch of code (`body`)
// interleaves them instruction by instruction: a SLOT is one 16-byte LDS fragment and the U MFMAs that multiply with
// it (both streams of a wave use every fragment, which halves the LDS reads per MFMA: 24 KB instead of 48 KB per 64 rows
// and block), value and score slots alternate so that no MFMA waits for the one before it, the maxima stand behind the
// first MFMAs and the exponentials behind the others (OpSchedule).  Fragments are requested kAhead slots ahead, also
// across the end of a block: the next block's keys and values are always in LDS already.  A lone wave is bound by its issue
// slots, so that every instruction counts: requests in pairs (one wait for two) and addresses that are moved on once per tile
// made narrow tiles 3 to 7 % faster (1 row x 32 heads, 24 positions behind 1792 keys 49.3 -> 46.6 us), wide ones 1 to 2 %.
//
// What bounds it, two members, U = 2 (cycles of one wave per 64-key tile; the MFMAs alone are 96 x 32 = 3072): 4500 to
// 4600 on a chip with free CUs -- the replayed body is 2 x 1940 (MFMA only 1536, + LDS reads 1570, + vector work 1700,
// all of it 1940: issue slots), the 12 direct loads to LDS about 25 each, the barrier 40 to 150 -- and about 5000 with every
// CU busy, at 1.8 to 1.9 GHz instead of 2.4: the chip lowers its clock on this data (these products alone reach 64 % of
// the nominal rate on N(0,1) operands), so that fewer cycles there buy less time than on small launches.  Each query
// tile adds its start (4600 cycles alone, 7000 on a full chip), the diagonal that the four waves finish one after the other, and
// the output rows (64 stores of two whole rows per wave; 8500 cycles as 256 of two cache lines each, some 16 000 as 16 bytes of 64
// lines).  The rows of a workgroup's first query tile are written while the second one's first tiles are on their way.
// Both together, and queries fetched as whole lines (dma_q): 16 rows x 2043 positions, 32 heads in 8 clusters 598 -> 569 us, 4 x 507,
// 72 in 16 51.9 -> 47.0, dense 8 x 2043, 32 heads 391 -> 372.
// Against the kernel before (eight waves, one stream of 32 rows each, two waves per SIMD), whole calls timed in turn: 16 rows
// x 2043 positions, 32 heads in 8 clusters 663 -> 616 us, dense 809 -> 780 us; 4 rows x 4000, 4 clusters 520 -> 467 us (with
// the balanced numbering below); 1 row x 2043 97 -> 63 us; 256 positions behind 1792 keys, 4 rows x 52 heads 128 -> 93 us.
//
// NW = 4 with U = 1 halves a workgroup's rows for launches that leave CUs without work (rules in launch_prefill): a wave's LDS
// reads per MFMA double, but twice as many CUs work, on half as long a chain.
//
// LDS: rings of three K and three V^T tiles (64 keys).  While tile t is computed, K(t+2) and V(t+1) are loaded with
// direct loads, requested in the first half of the tile; K runs ahead of V because the scores of a block are issued one
// block before its softmax, and V lags because its products come one block after.  ONE barrier per tile.
// Dense attention of thousands of heads over at most one tile of keys has rings of two (BUFS), 80 KB: it is all start and end,
// and two workgroups on a CU cover each other's (64 x 72 heads of 24 keys 55 us, 67 us with one, values converted on the way).
//
// A score block is shared by TWO members.  Wider schemes were built on the kernel before and were slower: four members
// through LDS (670-840 against 578 us per 8-cluster LLaMa-7B layer), three members in one wave (630 against 553 us).
// ---------------------------------------------------------------------------------------------------------
constexpr int kBufs = 3;
constexpr size_t kKBufBytes = (size_t)kKTile * kHeadDim * 2;        // 64 rows of 256 B (16 pieces), swizzled
constexpr size_t kVBufBytes = (size_t)kHeadDim * kKTile * 2;        // one member: 128 rows of 128 B (8 pieces), swizzled
// rows: query rows of a workgroup, which stand behind the first value tile at the start
__host__ __device__ constexpr size_t prefill_rings(bool ident, int bufs, int rows)
{
    const size_t v_tile = (ident ? 1 : kGroup) * kVBufBytes, rings = bufs * (kKBufBytes + v_tile);
    const size_t start = bufs * kKBufBytes + v_tile + (size_t)rows * (kHeadDim * 2);
    return rings > start ? rings : start;
}
constexpr size_t prefill_lds_bytes(bool ident, int bufs, int rows) { return prefill_rings(ident, bufs, rows) + (bufs == 2 ? 0 : 16); }

// ---------------------------------------------------------------------------------------------------------
// Which query tiles of which (batch row, group) a workgroup takes.  The hardware deals consecutive workgroup ids
// round-robin to the 8 XCDs, each with an L2 of its own; every XCD has a queue of tiles, from which its 32 workgroups, one per CU, draw
// one after the other (or which has a workgroup for every tile: launch_prefill).  The unit of the deal is a PAIR of query tiles of
// one group, the p-th largest and the p-th smallest: under the causal mask tile q walks q+1 key tiles' worth of work, so all
// pairs cost the same.  The pairs that EXIST (the groups of all rows, counted here from the plan) are dealt to the XCDs in equal
// contiguous ranges, so that the pairs of one group share its keys and values in one L2.  A queue has whole rounds of 32
// pairs first; the last 32 to 63 pairs stand in it as single tiles, the largest first, which fills the last round.  The pairs of the
// whole rounds stand there one by one while a group has fewer than 32 (fewer groups at a time: 834 MiB fetched for 16 rows x 2043
// positions, 32 heads in 8 clusters, 1013 with a workgroup for every pair).  Longer prompts have the larger tiles of 32 pairs, then the
// smaller ones, the last first: the CUs walk a group's keys side by side, which do not fit an L2 any more, and small tiles in
// between would begin them anew (4 x 32 763 positions, 32 heads in clusters of 20, 6, 4 and 2 21.9 -> 20.8 ms, one row 5.6 -> 5.1; 16 379
// 5.68 -> 5.35; with a workgroup for every pair 21.1, 5.2 and 5.48).
// ---------------------------------------------------------------------------------------------------------
constexpr int kXcdCus = 32;
constexpr int kSmallTiles = 450, kFewTiles = 1450;      // see launch_prefill
struct WorkQueue {
    unsigned n_pairs, lo, hi, mid, first, n_first, n_items;      // pairs lo .. mid-1, then mid .. hi-1, of n_first groups from `first`
    int upto;                                                // groups of the first rows up to this lane's
};
template <bool IDENT>
__device__ __forceinline__ WorkQueue make_queue(const int32_t *__restrict__ n_groups, int n_rows, int H, int n_qt)
{
    const int lane = threadIdx.x & 63;
    WorkQueue w;
    w.n_pairs = (unsigned)(n_qt + 1) / 2;
    unsigned total = 0;                                     // groups; total * n_pairs < 2^30 (launch_prefill)
    w.upto = 0;
    if (IDENT) total = (unsigned)n_rows * (unsigned)H;
    else {
        for (int r0 = 0; r0 < n_rows; r0 += 64) {
            int upto = r0 + lane < n_rows ? n_groups[r0 + lane] : 0;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int other = __shfl_up(upto, o);
                upto += lane >= o ? other : 0;
            }
            total += (unsigned)__builtin_amdgcn_readlane(upto, 63);
            if (r0 == 0) w.upto = upto;
        }
    }
    const unsigned xcd = blockIdx.x % kXcds, pairs = total * w.n_pairs;
    const unsigned each = pairs / kXcds, rest = pairs % kXcds;               // the first `rest` XCDs take one more
    w.lo = each * xcd + min(xcd, rest);
    w.hi = w.lo + each + (xcd < rest ? 1u : 0u);
    const unsigned rounds = (w.hi - w.lo) / kXcdCus;
    w.mid = w.lo + (rounds > 1 ? (rounds - 1) * kXcdCus : 0u);
    w.first = w.mid / w.n_pairs;
    w.n_first = w.mid < w.hi ? (w.hi - 1) / w.n_pairs - w.first + 1 : 0u;
    w.n_items = n_qt == 1 ? w.hi - w.lo : 2 * (w.mid - w.lo) + 2 * w.n_first * w.n_pairs;
    return w;
}
// Item i: group and query tile; false where there is none of that number.
__device__ __forceinline__ bool queue_item(const WorkQueue &w, int n_qt, unsigned i, unsigned &group, int &qt)
{
    if (n_qt == 1) {
        group = w.lo + i;
        qt = 0;
        return true;
    }
    if (i < 2 * (w.mid - w.lo)) {
        // `block` pairs' larger tiles, then their smaller ones, the last pair's first
        const unsigned block = w.n_pairs >= kXcdCus ? kXcdCus : 1, first = i / (2 * block) * block, r = i - 2 * first;
        const bool small = r >= block;
        const unsigned at = w.lo + first + (small ? 2 * block - 1 - r : r);
        group = at / w.n_pairs;
        const int pi = (int)(at - group * w.n_pairs);
        qt = small ? pi : n_qt - 1 - pi;
        return !small || n_qt - 1 - pi != pi;                // the middle tile of an odd count is alone
    }
    unsigned j = i - 2 * (w.mid - w.lo);
    const unsigned m = w.n_first * w.n_pairs;
    const bool large = j < m;
    if (!large) j -= m;
    const unsigned row = j / w.n_first;
    const int pi = (int)(large ? row : w.n_pairs - 1 - row);
    group = w.first + j - row * w.n_first;
    qt = large ? n_qt - 1 - pi : pi;
    const unsigned at = group * w.n_pairs + (unsigned)pi;
    return at >= w.mid && at < w.hi && (large || n_qt - 1 - pi != pi);
}
// Row and number in the row of a group.
template <bool IDENT>
__device__ __forceinline__ void find_row(const WorkQueue &w, const int32_t *__restrict__ n_groups, int n_rows, int H, unsigned group, int &b,
                                         int &gi)
{
    const int lane = threadIdx.x & 63;
    if (IDENT) {
        b = (int)(group / (unsigned)H);
        gi = (int)(group % (unsigned)H);
        return;
    }
    b = gi = 0;
    for (int r0 = 0; r0 < n_rows; r0 += 64) {
        int upto = w.upto;
        if (r0 != 0) {
            upto = r0 + lane < n_rows ? n_groups[r0 + lane] : 0;
#pragma unroll
            for (int o = 1; o < 64; o <<= 1) {
                const int other = __shfl_up(upto, o);
                upto += lane >= o ? other : 0;
            }
        }
        const unsigned all = (unsigned)__builtin_amdgcn_readlane(upto, 63);
        if (group < all) {
            const int row = __popcll(__ballot((unsigned)upto <= group));
            b = r0 + row;
            gi = (int)group - (row > 0 ? __builtin_amdgcn_readlane(upto, row - 1) : 0);
            return;
        }
        group -= all;
    }
}

// Accumulator tile T of the kernel below: registers a[16 T .. 16 T + 15] of the accumulation half, BY NAME.  The compiler
// never sees the accumulators as values (offered as operands it carried them through ordinary registers at every branch,
// 688 spills); matrix results of its own are kept in ordinary registers by the build's -amdgpu-mfma-vgpr-form, and the
// clobbers keep whatever else it may put into that half (copies of ordinary registers, in the kernel with two waves per
// SIMD) away from the named ones.  What the compiler would insert
// between dependent instructions stands here: two idle slots between an ordinary write and a matrix read
// (acc_written), twenty between a matrix write and an ordinary read (acc_settle).
template <int T>
struct AccTile;
#if defined(__HIP_DEVICE_COMPILE__)
#define CHAI_ACC_ZERO(r) asm volatile("v_accvgpr_write_b32 " r ", 0" ::: r)
#define CHAI_ACC_SCALE(i, r)                                                                                           \
    {                                                                                                                  \
        float t;                                                                                                       \
        asm volatile("v_accvgpr_read_b32 %0, " r "\n\tv_mul_f32 %0, %1, %0\n\tv_accvgpr_write_b32 " r ", %0"           \
                     : "=&v"(t)                                                                                        \
                     : "v"(by[i])                                                                                      \
                     : r);                                                                                             \
    }
#define CHAI_ACC_READ(i, r) asm volatile("v_accvgpr_read_b32 %0, " r : "=v"(x[i]))
#define CHAI_ACC_MFMA(range, ...)                                                                                      \
    asm volatile("v_mfma_f32_32x32x16_f16 " range ", %0, %1, " range ::"v"(p), "v"(v) : __VA_ARGS__)
#else
#define CHAI_ACC_ZERO(r) (void)0
#define CHAI_ACC_SCALE(i, r) (void)by
#define CHAI_ACC_READ(i, r) x[i] = 0.f
#define CHAI_ACC_MFMA(range, ...) (void)0
#endif
#define CHAI_ACC_TILE(T, range, r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15)                   \
    template <>                                                                                                        \
    struct AccTile<T> {                                                                                                \
        static __device__ __forceinline__ void mfma(const f16x8 &p, const f16x8 &v)                                    \
        {                                                                                                              \
            CHAI_ACC_MFMA(range, r0, r1, r2, r3, r4, r5, r6, r7, r8, r9, r10, r11, r12, r13, r14, r15);                 \
        }                                                                                                              \
        static __device__ __forceinline__ void zero()                                                                  \
        {                                                                                                              \
            CHAI_ACC_ZERO(r0); CHAI_ACC_ZERO(r1); CHAI_ACC_ZERO(r2); CHAI_ACC_ZERO(r3);                                 \
            CHAI_ACC_ZERO(r4); CHAI_ACC_ZERO(r5); CHAI_ACC_ZERO(r6); CHAI_ACC_ZERO(r7);                                 \
            CHAI_ACC_ZERO(r8); CHAI_ACC_ZERO(r9); CHAI_ACC_ZERO(r10); CHAI_ACC_ZERO(r11);                               \
            CHAI_ACC_ZERO(r12); CHAI_ACC_ZERO(r13); CHAI_ACC_ZERO(r14); CHAI_ACC_ZERO(r15);                             \
        }                                                                                                              \
        static __device__ __forceinline__ void scale(const float (&by)[4], std::integral_constant<int, 0>)              \
        {                                                                                                              \
            CHAI_ACC_SCALE(0, r0); CHAI_ACC_SCALE(1, r1); CHAI_ACC_SCALE(2, r2); CHAI_ACC_SCALE(3, r3);                 \
        }                                                                                                              \
        static __device__ __forceinline__ void scale(const float (&by)[4], std::integral_constant<int, 1>)              \
        {                                                                                                              \
            CHAI_ACC_SCALE(0, r4); CHAI_ACC_SCALE(1, r5); CHAI_ACC_SCALE(2, r6); CHAI_ACC_SCALE(3, r7);                 \
        }                                                                                                              \
        static __device__ __forceinline__ void scale(const float (&by)[4], std::integral_constant<int, 2>)              \
        {                                                                                                              \
            CHAI_ACC_SCALE(0, r8); CHAI_ACC_SCALE(1, r9); CHAI_ACC_SCALE(2, r10); CHAI_ACC_SCALE(3, r11);               \
        }                                                                                                              \
        static __device__ __forceinline__ void scale(const float (&by)[4], std::integral_constant<int, 3>)              \
        {                                                                                                              \
            CHAI_ACC_SCALE(0, r12); CHAI_ACC_SCALE(1, r13); CHAI_ACC_SCALE(2, r14); CHAI_ACC_SCALE(3, r15);             \
        }                                                                                                              \
        static __device__ __forceinline__ void read(float (&x)[4], std::integral_constant<int, 0>)                      \
        {                                                                                                              \
            CHAI_ACC_READ(0, r0); CHAI_ACC_READ(1, r1); CHAI_ACC_READ(2, r2); CHAI_ACC_READ(3, r3);                     \
        }                                                                                                              \
        static __device__ __forceinline__ void read(float (&x)[4], std::integral_constant<int, 1>)                      \
        {                                                                                                              \
            CHAI_ACC_READ(0, r4); CHAI_ACC_READ(1, r5); CHAI_ACC_READ(2, r6); CHAI_ACC_READ(3, r7);                     \
        }                                                                                                              \
        static __device__ __forceinline__ void read(float (&x)[4], std::integral_constant<int, 2>)                      \
        {                                                                                                              \
            CHAI_ACC_READ(0, r8); CHAI_ACC_READ(1, r9); CHAI_ACC_READ(2, r10); CHAI_ACC_READ(3, r11);                   \
        }                                                                                                              \
        static __device__ __forceinline__ void read(float (&x)[4], std::integral_constant<int, 3>)                      \
        {                                                                                                              \
            CHAI_ACC_READ(0, r12); CHAI_ACC_READ(1, r13); CHAI_ACC_READ(2, r14); CHAI_ACC_READ(3, r15);                 \
        }                                                                                                              \
    };
CHAI_ACC_TILE(0, "a[0:15]", "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15")
CHAI_ACC_TILE(1, "a[16:31]", "a16", "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31")
CHAI_ACC_TILE(2, "a[32:47]", "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46", "a47")
CHAI_ACC_TILE(3, "a[48:63]", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61", "a62", "a63")
CHAI_ACC_TILE(4, "a[64:79]", "a64", "a65", "a66", "a67", "a68", "a69", "a70", "a71", "a72", "a73", "a74", "a75", "a76", "a77", "a78", "a79")
CHAI_ACC_TILE(5, "a[80:95]", "a80", "a81", "a82", "a83", "a84", "a85", "a86", "a87", "a88", "a89", "a90", "a91", "a92", "a93", "a94", "a95")
CHAI_ACC_TILE(6, "a[96:111]", "a96", "a97", "a98", "a99", "a100", "a101", "a102", "a103", "a104", "a105", "a106", "a107", "a108", "a109", "a110", "a111")
CHAI_ACC_TILE(7, "a[112:127]", "a112", "a113", "a114", "a115", "a116", "a117", "a118", "a119", "a120", "a121", "a122", "a123", "a124", "a125", "a126", "a127")
CHAI_ACC_TILE(8, "a[128:143]", "a128", "a129", "a130", "a131", "a132", "a133", "a134", "a135", "a136", "a137", "a138", "a139", "a140", "a141", "a142", "a143")
CHAI_ACC_TILE(9, "a[144:159]", "a144", "a145", "a146", "a147", "a148", "a149", "a150", "a151", "a152", "a153", "a154", "a155", "a156", "a157", "a158", "a159")
CHAI_ACC_TILE(10, "a[160:175]", "a160", "a161", "a162", "a163", "a164", "a165", "a166", "a167", "a168", "a169", "a170", "a171", "a172", "a173", "a174", "a175")
CHAI_ACC_TILE(11, "a[176:191]", "a176", "a177", "a178", "a179", "a180", "a181", "a182", "a183", "a184", "a185", "a186", "a187", "a188", "a189", "a190", "a191")
CHAI_ACC_TILE(12, "a[192:207]", "a192", "a193", "a194", "a195", "a196", "a197", "a198", "a199", "a200", "a201", "a202", "a203", "a204", "a205", "a206", "a207")
CHAI_ACC_TILE(13, "a[208:223]", "a208", "a209", "a210", "a211", "a212", "a213", "a214", "a215", "a216", "a217", "a218", "a219", "a220", "a221", "a222", "a223")
CHAI_ACC_TILE(14, "a[224:239]", "a224", "a225", "a226", "a227", "a228", "a229", "a230", "a231", "a232", "a233", "a234", "a235", "a236", "a237", "a238", "a239")
CHAI_ACC_TILE(15, "a[240:255]", "a240", "a241", "a242", "a243", "a244", "a245", "a246", "a247", "a248", "a249", "a250", "a251", "a252", "a253", "a254", "a255")
#undef CHAI_ACC_TILE
#undef CHAI_ACC_ZERO
#undef CHAI_ACC_SCALE
#undef CHAI_ACC_READ
#undef CHAI_ACC_MFMA

// Nothing of the compiler's lives in a0 .. a63 across this point.  In the kernel with two waves per SIMD, which needs the
// rest of the accumulation half for copies of ordinary registers, one stands behind every matrix instruction: the products'
// own clobbers left it room to park a value in a0 between two products of another tile.
__device__ __forceinline__ void acc_hold()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" :::
                 "a0", "a1", "a2", "a3", "a4", "a5", "a6", "a7", "a8", "a9", "a10", "a11", "a12", "a13", "a14", "a15", "a16",
                 "a17", "a18", "a19", "a20", "a21", "a22", "a23", "a24", "a25", "a26", "a27", "a28", "a29", "a30", "a31",
                 "a32", "a33", "a34", "a35", "a36", "a37", "a38", "a39", "a40", "a41", "a42", "a43", "a44", "a45", "a46",
                 "a47", "a48", "a49", "a50", "a51", "a52", "a53", "a54", "a55", "a56", "a57", "a58", "a59", "a60", "a61",
                 "a62", "a63");
#endif
}

__device__ __forceinline__ void acc_written()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_nop 3");
#endif
}
__device__ __forceinline__ void acc_settle()
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("s_nop 15\n\ts_nop 3");
#endif
}

// Two probabilities to fp16, nearest even, HERE: the empty statement pins the place (the compiler would gather all
// conversions at the end of a block).  The conversion itself is left to the compiler, which knows how long an exponential
// takes to arrive.
__device__ __forceinline__ unsigned int pack_f16(float lo, float hi)
{
    typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
    union {
        f16x2 h;
        unsigned int u;
    } x;
    x.h[0] = (_Float16)lo;
    x.h[1] = (_Float16)hi;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x.u));
#endif
    return x.u;
}

// f(integral_constant 0), f(1), .. f(N - 1): loops whose index names registers
template <typename F, int... I>
__device__ __forceinline__ void unroll_seq(F &&f, std::integer_sequence<int, I...>)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void unroll(F &&f)
{
    unroll_seq(f, std::make_integer_sequence<int, N>{});
}

// Which of the 34 * 4 softmax operations of a block stand behind which of its MFMAs: by cost (quarter cycles: a vector
// instruction 18, an exponential 32), a step with an LDS request takes a quarter of what the step without takes.
template <int STEPS, int ELEMS, int EVEN, int ODD>
struct OpSchedule {
    int first[STEPS + 1];
    constexpr OpSchedule() : first{}
    {
        auto cost = [](int i) {
            const int g = i / 4, kind = i % 4;
            if (kind == 0) return g < ELEMS ? 18 : 0;
            if (kind == 1) return g >= 1 && g <= ELEMS ? 32 : 0;
            if (kind == 2) return g >= 2 ? 18 : 0;
            return g >= 2 && (g & 1) ? 18 : 0;
        };
        constexpr int kOps = (ELEMS + 2) * 4, kTotal = ELEMS * (18 + 32 + 18) + ELEMS / 2 * 18;
        int i = 0, spent = 0, share = 0;
        for (int n = 0; n < STEPS; ++n) {
            first[n] = i;
            share += n % 2 == 0 ? EVEN : ODD;
            while (i < kOps && (n == STEPS - 1 || (spent + cost(i) / 2) * (STEPS / 2) * (EVEN + ODD) <= kTotal * share))
                spent += cost(i++);
        }
        first[STEPS] = kOps;
    }
};

// x is what is loaded, here (what is worked out from it by both sides of a branch is not worked out before the branch, where it
// would wait for the load)
__device__ __forceinline__ void hold(u32x4 &x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(x));
#endif
}

// What is left to do for a query tile whose accumulators are complete
template <int U>
struct Finished {
    int n_mem;                                               // of how many members (0: none)
    int i0;                                                  // first query row of the wave
    size_t b;                                                // batch row, members
    int heads[kGroup];
    float inv[U];                                            // one over this lane's row sum
};

// One query tile (NW waves x 32 U rows; has_tile) of one group of NM members, and before it, once the tile's first requests are on
// their way, the output rows of the tile before, if that one was of NM members too (done).  heads, vsrc: the members' heads and
// V^T; brow: batch row.
// LDS: rings of BUFS tiles (2: one key tile only), a value tile with room for G members.
// DIRECT: vsrc are the members' rows of the value cache itself (see prefill_direct_kernel).
// draw: called once, two tiles of keys before the end
template <int NM, int U, int NW, int G, int BUFS, bool DIRECT, typename Draw>
__device__ __forceinline__ void prefill_tile(char *k_lds, char *v_lds, const char *ksrc, const char *const (&vsrc)[kGroup],
                                          const char *q, const int (&heads)[kGroup], size_t brow, int H, int Tq, int q_start,
                                          int qt, bool has_tile, int rhead, float scale2, float *__restrict__ out,
                                          Finished<U> &done, Draw draw)
{
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    int lane = tid & 63;
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(lane));                           // (what follows from it is worked out again for every query tile)
#endif
    const int r = lane & 31, hl = lane >> 5;
    const int n_keys = q_start + Tq;
    const int i0 = (qt * NW + w) * (32 * U);                // first query row of this wave
    const int wave_first = q_start + min(i0, Tq - 1);
    const int wave_last = q_start + min(i0 + 32 * U - 1, Tq - 1);
    const int wg_last = q_start + min((qt + 1) * (NW * 32 * U) - 1, Tq - 1);
    const int n_tiles = wg_last / kKTile + 1;
    const int n_hb = i0 < Tq ? wave_last / 32 + 1 : -1;      // 32-key blocks of this wave (-1: a padding wave)

    Frag16 qf[U][kHeadDim / 16];
    int q_abs[U];                                            // sequence position of this lane's row in every stream

    // Staging with direct loads to LDS: one instruction moves 64 pieces of 16 bytes into 1 KB of consecutive LDS (lane l's
    // piece lands at base + 16 l), no registers and no LDS write instructions.  The BUFFER form of the instruction is
    // used: with the global form in a loop the compiler gives up counting LDS reads and waits for all of them before
    // every MFMA.  Rows are unpadded, and bank conflicts of the fragment reads are avoided by a swizzle instead: piece c
    // of K row R sits in slot c ^ (R & 15) of the row, piece c of V^T row R in slot c ^ ((R >> 1) & 7); 16 consecutive rows
    // read at one piece index then touch 16 different 16-byte slots of the 256-byte bank window (measured: 16 cycles per
    // read with four waves reading, the same as for linear addresses).  A lane fetches whichever piece belongs in the
    // slot it fills.  Instruction i (of kDma) of wave w fills K rows 4(w + NW i) .. +3, or V^T rows 8(w + NW i) .. +7 of a
    // member.
    constexpr int kDma = 16 / NW;
    const int k_row = 4 * w + (lane >> 4);
    const int v_row = 8 * w + (lane >> 3);
#if defined(__HIP_DEVICE_COMPILE__)
    auto make_rsrc = [](const char *base, int bytes = 0x7fffffff) {
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), 0, bytes, 0x00020000);
    };
    auto load_to_lds = [](__amdgpu_buffer_rsrc_t rs, unsigned int off, char *dst) {
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)dst, 16, (int)off, 0, 0, 0);
    };
#else
    auto make_rsrc = [](const char *base, int = 0) { return base; };
    auto load_to_lds = [](const char *, unsigned int, char *) {};
#endif
    const auto k_rs = make_rsrc(ksrc);
    const int v_bytes = DIRECT ? n_keys * (kHeadDim * 2) : 0x7fffffff;       // rows past the last key read as zeros
    const auto v_rs0 = make_rsrc(vsrc[0], v_bytes);
    const auto v_rs1 = make_rsrc(vsrc[NM - 1], v_bytes);
    const int k_piece = ((lane & 15) ^ (k_row & 15)) << 4;   // rows 4 NW apart share the swizzle
    const int k_off = k_row * (kHeadDim * 2) + k_piece, k_last = (n_keys - 1) * (kHeadDim * 2) + k_piece;
    auto dma_k1 = [&](int kt, int buf, int i) {
        load_to_lds(k_rs, (unsigned int)min(k_off + (kt * kKTile + 4 * NW * i) * (kHeadDim * 2), k_last),
                    k_lds + buf * kKBufBytes + (w + NW * i) * 1024);
    };
    const int v_piece = (lane & 7) ^ ((v_row >> 1) & 7);     // rows 8 NW apart share the swizzle
    const unsigned int v_off = (unsigned int)(v_row * (kKTile * 2) + v_piece * 16);
    auto dma_v1 = [&](int kt, int buf, int g, int i) {
        load_to_lds(g == 0 ? v_rs0 : v_rs1, (unsigned int)kt * (unsigned int)kVBufBytes + v_off + i * 8 * NW * (kKTile * 2),
                    v_lds + (buf * G + g) * kVBufBytes + (w + NW * i) * 1024);
    };
    auto dma_k = [&](int kt, int buf) {
#pragma unroll
        for (int i = 0; i < kDma; ++i) dma_k1(kt, buf, i);
    };
    // The wave's query rows, as whole cache lines: as fragments from memory every line is asked for by four instructions, and the
    // rows of a workgroup are more than the first cache holds.  They stand where the value tiles after the first will.
    char *const q_lds = v_lds + G * kVBufBytes + w * (32 * U * kHeadDim * 2);
    auto dma_q = [&]() {
        const auto q_rs = make_rsrc(q + (brow * H + rhead) * (size_t)Tq * (kHeadDim * 2));
#pragma unroll
        for (int i = 0; i < 8 * U; ++i) {
            const int row = 4 * i + (lane >> 4);
            load_to_lds(q_rs, (unsigned int)(min(i0 + row, Tq - 1) * (kHeadDim * 2) + (((lane & 15) ^ (row & 15)) << 4)), q_lds + i * 1024);
        }
    };
    auto dma_v = [&](int kt, int buf) {
#pragma unroll
        for (int g = 0; g < NM; ++g)
#pragma unroll
            for (int i = 0; i < kDma; ++i) dma_v1(kt, buf, g, i);
    };
    // (No scalar offset: with one the compiler takes it that the data registers may be written again in the very next
    // instruction, and a 16-byte store then wrote what had come after it.)
    auto store_row = [&](char *base, int n_rows, int off, const float (&x)[4]) {
#if defined(__HIP_DEVICE_COMPILE__)
        const u32x4 bits = {__float_as_uint(x[0]), __float_as_uint(x[1]), __float_as_uint(x[2]), __float_as_uint(x[3])};
        __builtin_amdgcn_raw_buffer_store_b128(bits, make_rsrc(base, n_rows * (kHeadDim * 4)), off, 0, 0);
#endif
    };
    // every wave waits for its own requests (the compiler does not track loads that land in LDS), then a bare s_barrier:
    // __syncthreads() would add fences that the loads to LDS do not need
    auto tile_barrier = [&]() {
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#endif
    };
    auto landed = [&](auto n) {
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"(decltype(n)::value) : "memory");
#endif
    };
    // what this wave wrote to LDS is there, what it read has arrived, and all but the youngest N requests have landed
    auto written_barrier = [&](auto n) {
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(decltype(n)::value) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#endif
    };
    // fragments: this lane's row r of a 32-row block of K, fragment p = 8 * member + 4 * (16 keys) + 32-column block of V^T
    const int k_sw = r & 15, v_sw = (r >> 1) & 7;
    auto k_frag = [&](const char *kb, int ks) { return *reinterpret_cast<const u32x4 *>(kb + (((2 * ks + hl) ^ k_sw) << 4)); };
    auto v_frag = [&](const char *vb, int half, int p) {
        const int j = p & 7;
        return *reinterpret_cast<const u32x4 *>(vb + (p >> 3) * kVBufBytes + (j & 3) * 32 * (kKTile * 2) +
                                                (((4 * half + 2 * (j >> 2) + hl) ^ v_sw) << 4));
    };

    // DIRECT: this thread's piece of every value tile is 8 columns (8 co ..) of the 8 keys that an MFMA operand holds side by
    // side, piece v_p of a V^T row, of one member (NM = 2), or half of those keys (NM = 1).  Transposing is no work of its
    // own: a conversion packs the same column of two keys.  Row R of V^T is row R ^ (R >> 4 & 1) of the tile in LDS, and piece p
    // of row R sits in slot p ^ ((R >> 1) & 7): reads of 16 rows at one piece and writes of 16 threads' columns at one piece (every
    // other row of 32) both touch 16 different 16-byte bank groups.
    constexpr int kKeys = NM == 2 ? 8 : 4;
    const int co = lane & 15, v_rest = 4 * w + (lane >> 4);
    const int v_p = NM == 2 ? v_rest & 7 : v_rest >> 1, v_half = NM == 2 ? 0 : v_rest & 1;
    const unsigned int v_in = (unsigned int)((16 * (v_p >> 1) + 4 * (v_p & 1) + 8 * v_half) * (kHeadDim * 2) + co * 16);
    struct Raw {
        u32x4 key[kKeys];
    };
    auto fetch_key = [&](Raw &raw, int kt, auto ic) {
#if defined(__HIP_DEVICE_COMPILE__)
        constexpr int i = decltype(ic)::value;
        const unsigned int off = v_in + (unsigned int)kt * (kKTile * kHeadDim * 2) + ((i & 3) + 8 * (i >> 2)) * (kHeadDim * 2);
        raw.key[i] = __builtin_amdgcn_raw_buffer_load_b128(NM == 2 && w >= 2 ? v_rs1 : v_rs0, (int)off, 0, 0);
#else
        (void)v_in;
#endif
    };
    // column 2 m + h of the eight: unit u = 2 m + h of a tile
    unsigned int packed[kKeys / 2];
    auto convert = [&](const Raw &raw, auto uc) {
        constexpr int m = decltype(uc)::value >> 1, h = decltype(uc)::value & 1;
#pragma unroll
        for (int i = 0; i < kKeys; i += 2) {
            const unsigned int x0 = raw.key[i][m], x1 = raw.key[i + 1][m];
            packed[i / 2] = pack_f16(__uint_as_float(h == 0 ? x0 << 16 : x0 & 0xffff0000u),
                                     __uint_as_float(h == 0 ? x1 << 16 : x1 & 0xffff0000u));
        }
    };
    char *const v_out = v_lds + (NM == 2 ? (w >> 1) * kVBufBytes : 0) + co * 2 * (kKTile * 2) + ((v_p ^ (co & 7)) << 4) + v_half * 8;
    const int v_flip[2] = {(co >> 3) * (kKTile * 2), (1 - (co >> 3)) * (kKTile * 2)};
    auto store_unit = [&](int buf, auto uc) {
        constexpr int u = decltype(uc)::value;
        static_assert(value_row(8 * 3 + u) == 2 * 3 + (u & 3) * 32 + (u >> 2), "rows of this thread's columns");
        char *at = v_out + buf * (G * kVBufBytes) + (u & 3) * 32 * (kKTile * 2) + v_flip[u >> 2];
        if constexpr (NM == 2) *reinterpret_cast<u32x4 *>(at) = u32x4{packed[0], packed[1], packed[2], packed[3]};
        else *reinterpret_cast<uint2 *>(at) = make_uint2(packed[0], packed[1]);
    };
    // Tile kt's share of that work, in as many steps as its two blocks have hooks: convert tile kt + 1 out of `raw`, then
    // request tile kt + 3 into it (its neighbour holds kt + 2); the keys of tile kt + 2 in between.
    constexpr int kHooks = NM == 2 ? 12 : 8;
    auto value_work = [&](Raw &raw, int far, int buf, auto hc, auto keys) {
        constexpr int hk = decltype(hc)::value;
        if constexpr (hk < 8) {
            convert(raw, std::integral_constant<int, hk>{});
            store_unit(buf, std::integral_constant<int, hk>{});
        } else if constexpr (hk % 2 == 0 && hk < 8 + 2 * kKeys) fetch_key(raw, far, std::integral_constant<int, (hk - 8) / 2>{});
        if constexpr (hk % 2 == 1 && hk < 8) keys(hk / 2);
    };

    // accumulators: tile (stream * NM + member) * 4 + 32-column block; zeroed at the end of the first block
    constexpr int kTiles = 4 * U * NM;
    auto product = [&](auto t, const f16x8 &p, const f16x8 &v) {
        AccTile<t.value>::mfma(p, v);
        if constexpr (NW == 8) acc_hold();
    };
    // Registers 4 q .. 4 q + 3 of an accumulator tile are rows 8 q + 4 hl .. + 3: of a value per row, which the row's two lanes
    // hold, what these registers need.  (The lane is counted here: no register is kept for it through the loop.)
    auto half_of_lane = []() {
        int at = 0;
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=&v"(at));
#endif
        return at >> 5;
    };
    auto of_rows = [](float x, int half, auto quad, float (&y)[4]) {
#pragma unroll
        for (int e = 0; e < 4; ++e)
            y[e] = __int_as_float(__builtin_amdgcn_ds_bpermute(16 * half + 4 * (8 * decltype(quad)::value + e), __float_as_int(x)));
    };
    float m_run[U], l_run[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        m_run[u] = -INFINITY;
        l_run[u] = 0.f;
    }

    // the output rows of the pass before, while this one's first tiles are on their way
    auto write_rows = [&]() {
        if (done.i0 >= Tq) return;                           // a padding wave
        acc_settle();
        // Rows past the block's last lie beyond the end of the buffer that is written to.
        const int n_rows = min(Tq - done.i0, 32 * U);
        int at = hl * 4 * (kHeadDim * 4) + r * 16;
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+v"(at));                         // (not worked out, with all that is added to it, before the loop)
#endif
        char *row0[NM];
#pragma unroll
        for (int g = 0; g < NM; ++g) row0[g] = reinterpret_cast<char *>(out + ((DIRECT ? brow * H + heads[g] : done.b * H + done.heads[g]) * Tq + done.i0) * kHeadDim);
        auto eight_rows = [&](auto c) __attribute__((always_inline)) {
            constexpr int u = c.value / 4, rows = 32 * u + 8 * (c.value % 4);
            const std::integral_constant<int, c.value % 4> quad;
            float inv[4];
            of_rows(done.inv[u], hl, quad, inv);
            unroll<NM>([&](auto g) {
                float x[4][4];                               // [32-column block][row]
                unroll<4>([&](auto blk) { AccTile<(u * NM + g.value) * 4 + blk.value>::read(x[blk.value], quad); });
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float y[4] = {x[0][e] * inv[e], x[1][e] * inv[e], x[2][e] * inv[e], x[3][e] * inv[e]};
                    store_row(row0[g.value], n_rows, at + rows * (kHeadDim * 4) + e * (kHeadDim * 4), y);
                }
            });
        };
        if constexpr (DIRECT || BUFS == 2) {
            unroll<2>(eight_rows);
            if (n_rows > 16) {                               // (short blocks: half of the stores would be of rows that are not there)
                acc_settle();
                unroll<2>([&](auto c) __attribute__((always_inline)) { eight_rows(std::integral_constant<int, c.value + 2>{}); });
            }
        } else
            unroll<4 * U>(eight_rows);
    };

    struct Prob {
        Frag16 f[U][2];                                      // [stream][16 keys]
    };
    struct Score {
        f32x16 s[U];
    };

    // Products of the wave's last block, whose probabilities are pp: of all streams, or without the first one if that one's
    // rows end before the block (its probabilities there are zero, but the values may be infinite).
    const bool all_streams = U == 1 || (q_start + min(i0 + 31, Tq - 1)) / 32 >= n_hb - 1;
    auto pv_streams = [&](auto from, const Prob &pp, const char *vb, int vhalf) {
        acc_written();
        unroll<8 * NM>([&](auto pc) {
            constexpr int p = pc.value;
            Frag16 vf;
            vf.raw = v_frag(vb, vhalf, p);
            unroll<U>([&](auto uc) {
                constexpr int u = uc.value;
                if constexpr (u >= decltype(from)::value)
                    product(std::integral_constant<int, (u * NM + (p >> 3)) * 4 + (p & 3)>{}, pp.f[u][(p >> 2) & 1].h, vf.h);
            });
        });
    };
    auto pv_last = [&](const Prob &pp, const char *vb, int vhalf) {
        if (all_streams) pv_streams(std::integral_constant<int, 0>{}, pp, vb, vhalf);
        else pv_streams(std::integral_constant<int, U - 1>{}, pp, vb, vhalf);
    };

    // slots of a block: 8 NM value fragments and 8 key fragments, every third (NM = 2) or second one a key fragment
    constexpr int kSlots = 8 * NM + 8, kAhead = U == 1 && NW == 4 && BUFS > 2 ? 6 : 4, kHead = 5, kMaxSteps = 4 * U;
    struct Carry {
        Frag16 f[kAhead];
    };
    // LDS addresses of this lane's fragments, eight of the keys and four of the values, moved on by a tile where a fragment of an
    // even block is the last one to use them (added up for every fragment they were a tenth of all instructions).
    // Even blocks multiply the second half of the tile's keys and of the values before it, odd blocks the first halves of
    // the next tile's keys and of the tile's values.
    const char *k_at[8], *v_at[4];
    int k_step = 0, v_step = 0;                              // to the next tile, of the even block whose fragments are requested
    auto frag_of = [&](auto sl, auto even) {
        constexpr int s = sl.value;
        constexpr bool e = decltype(even)::value, qk = NM == 2 ? s % 3 == 2 : s % 2 == 1;
        if constexpr (qk) {
            constexpr int ks = NM == 2 ? s / 3 : s / 2;
            const u32x4 f = *reinterpret_cast<const u32x4 *>(k_at[ks] + (e ? 32 * (kHeadDim * 2) : 0));
            if constexpr (e) k_at[ks] += k_step;
            return f;
        } else {
            constexpr int p = NM == 2 ? s - s / 3 : s / 2, j = p & 7, piece = (e ? 4 : 0) + 2 * (j >> 2);
            const u32x4 f = *reinterpret_cast<const u32x4 *>(v_at[piece / 2] + (p >> 3) * kVBufBytes + (j & 3) * 32 * (kKTile * 2));
            if constexpr (e && p >= 8 * NM - 8 && (j & 3) == 3) {
                v_at[piece / 2] += v_step;
                v_at[piece / 2 - 2] += v_step;               // of the odd block
            }
            return f;
        }
    };
    // Block kbase .. kbase+31: softmax of its scores sc into pn; scores of the next block into sn; products of the block before
    // (probabilities pp).  carry: the first fragments, and then those of the next call; even: block 0 may be among them.
    // Fragments are requested in pairs, the one that is needed first last: one wait serves both.
    auto body = [&](Score &sc, Score &sn, const Prob &pp, Prob &pn, int kbase, Carry &carry, auto dma, auto even) {
        // causal mask: only blocks that reach past the wave's first query need it (a branch uniform per wave; out of line,
        // like the rescaling below: a taken branch costs a lone wave 40 cycles)
        if (__builtin_expect(kbase + 31 > wave_first, 0)) {
            asm volatile("" ::: "memory");
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int key = kbase + (e >> 2) * 8 + hl * 4 + (e & 3);
                    sc.s[u][e] = key <= q_abs[u] ? sc.s[u][e] : -INFINITY;
                }
        }
        Frag16 fr[kSlots + kAhead];
        unroll<kAhead>([&](auto i) { fr[i.value] = carry.f[i.value]; });
        auto fetch = [&](auto sl) {
            constexpr int s = sl.value;
            if constexpr (s < kSlots) fr[s].raw = frag_of(sl, even);
            else fr[s].raw = frag_of(std::integral_constant<int, s - kSlots>{}, std::integral_constant<bool, !decltype(even)::value>{});
        };
        // step j: MFMA of stream j % U of slot j / U
        auto step = [&](auto jc) {
            constexpr int s = jc.value / U, u = jc.value % U;
            if constexpr (s < kSlots) {
                constexpr bool qk = NM == 2 ? s % 3 == 2 : s % 2 == 1;
                if constexpr (u == 0) fetch(std::integral_constant<int, (s + kAhead) ^ 1>{});
                if constexpr (u == U - 1 && s % 2 == 0) dma(std::integral_constant<int, s / 2>{});
                if constexpr (qk) {
                    constexpr int ks = NM == 2 ? s / 3 : s / 2;
                    f32x16 c;
                    if constexpr (ks == 0) {
#pragma unroll
                        for (int e = 0; e < 16; ++e) c[e] = 0.f;
                    } else
                        c = sn.s[u];
                    sn.s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fr[s].bf, qf[u][ks].bf, c, 0, 0, 0);
                    if constexpr (NW == 8) acc_hold();
                } else {
                    constexpr int p = NM == 2 ? s - s / 3 : s / 2;
                    product(std::integral_constant<int, (u * NM + (p >> 3)) * 4 + (p & 3)>{}, pp.f[u][(p >> 2) & 1].h, fr[s].h);
                }
            }
        };
        acc_written();
        float ext[U];
        // maxima, two vector instructions behind every MFMA
        unroll<U * kHead>([&](auto jc) {
            constexpr int j = jc.value, u = j / 4, c = j % 4;
            step(jc);
            if constexpr (j < kMaxSteps) {
                if constexpr (c == 0) ext[u] = sc.s[u][0];
#pragma unroll
                for (int e = c == 0 ? 1 : c * 4; e < c * 4 + 4; ++e) ext[u] = fmaxf(ext[u], sc.s[u][e]);
                if constexpr (c == 3) ext[u] *= scale2;
                __builtin_amdgcn_sched_barrier(0);
            }
        });
        // Lazy reference: the running maximum (log2 units, of the raw scores times scale2; scale > 0 is required) only
        // moves when a block exceeds it by more than kRescaleSlack, so p < 2^slack and most blocks skip the rescaling.
        // A lane sees half of its row's keys; the halves are compared only when one of them is over.
        bool over = ext[0] > m_run[0] + kRescaleSlack;
        if constexpr (U == 2) over = over || ext[1] > m_run[1] + kRescaleSlack;
        const bool moved = __any(over);
        float alpha[U];
#pragma unroll
        for (int u = 0; u < U; ++u) alpha[u] = 1.f;
        if (__builtin_expect(moved, 0)) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                float lo, hi;
                both_halves(ext[u], lo, hi);
                const float mx = fmaxf(lo, hi);
                const bool need = mx > m_run[u] + kRescaleSlack;
                const float m_new = need ? mx : m_run[u];
                alpha[u] = need ? __builtin_amdgcn_exp2f(m_run[u] - m_new) : 1.0f;
                l_run[u] *= alpha[u];
                m_run[u] = m_new;
            }
        }
        __builtin_amdgcn_sched_barrier(0);
        // probabilities: element n's exponent, element n-1's exponential and element n-2's sum and conversion together, so
        // that no instruction waits for the one before it
        constexpr int kRest = U * (kSlots - kHead), kElems = 16 * U;
        float x[kElems], pe[kElems];
        // operation i: group i / 4 holds element g's exponent, g-1's exponential, g-2's sum, (odd g-2) the conversion
        auto op = [&](auto ic) {
            constexpr int g = ic.value / 4, kind = ic.value % 4;
            if constexpr (kind == 0 && g < kElems) x[g] = fmaf(sc.s[g >> 4][g & 15], scale2, -m_run[g >> 4]);
            if constexpr (kind == 1 && g >= 1 && g <= kElems) pe[g - 1] = __builtin_amdgcn_exp2f(x[g - 1]);
            if constexpr (kind == 2 && g >= 2) l_run[(g - 2) >> 4] += pe[g - 2];
            if constexpr (kind == 3 && g >= 2 && (g & 1)) {
                constexpr int e = g - 2;
                pn.f[e >> 4][(e >> 3) & 1].raw[(e & 7) >> 1] = pack_f16(pe[e - 1], pe[e]);
            }
        };
        constexpr OpSchedule<kRest, kElems, 1, U == 2 ? 3 : 1> sched{};
        unroll<kRest>([&](auto nc) {
            constexpr int n = nc.value;
            step(std::integral_constant<int, U * kHead + n>{});
            unroll<sched.first[n + 1] - sched.first[n]>(
                [&](auto q) { op(std::integral_constant<int, sched.first[n] + q.value>{}); });
            __builtin_amdgcn_sched_barrier(0);
        });
        unroll<kAhead>([&](auto i) { carry.f[i.value] = fr[kSlots + i.value]; });
        // The first block's products are of no block before it (what multiplied zero may be infinite): the accumulators
        // start from zero behind them.  There `moved` is set, or no score of the wave is a number.
        if (__builtin_expect(moved, 0)) {
            acc_settle();
            if (decltype(even)::value && kbase == 0) unroll<kTiles>([&](auto t) { AccTile<t.value>::zero(); });
            else {
                const int half = half_of_lane();
                unroll<4 * U>([&](auto c) {
                    __builtin_amdgcn_sched_barrier(0);
                    constexpr int u = c.value / 4;
                    const std::integral_constant<int, c.value % 4> quad;
                    float by[4];
                    of_rows(alpha[u], half, quad, by);
                    unroll<4 * NM>([&](auto t) { AccTile<u * 4 * NM + t.value>::scale(by, quad); });
                });
            }
        }
    };

    Raw raw_a, raw_b;                                        // DIRECT: tiles 0, 2, .. and 1, 3, ..
    if (has_tile) {
        dma_k(0, 0);
        if constexpr (!DIRECT) {
            dma_q();
            dma_v(0, 0);
            if (BUFS > 2 && n_tiles > 1) dma_k(1, 1);
        }
    }
    if (DIRECT ? !has_tile : done.n_mem == NM) write_rows();
    if (!has_tile) {
        done.n_mem = 0;
        return;
    }
    // query fragments (B operand of S^T = K Q^T): Q[row][16*ks + 8*hl .. +7]
#pragma unroll
    for (int u = 0; u < U; ++u) q_abs[u] = q_start + min(i0 + u * 32 + r, Tq - 1);
    auto read_q = [&]() {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int ks = 0; ks < kHeadDim / 16; ++ks) qf[u][ks].raw = k_frag(q_lds + (u * 32 + r) * (kHeadDim * 2), ks);
    };                                                       // (before the barrier: behind it the other waves' values come here)
    if constexpr (DIRECT) {
        auto first_values = [&]() {
            __builtin_amdgcn_sched_barrier(0);
            unroll<kKeys>([&](auto i) { hold(raw_a.key[i.value]); });
            unroll<8>([&](auto u) {
                convert(raw_a, u);
                store_unit(0, u);
            });
            __builtin_amdgcn_sched_barrier(0);
        };
        __builtin_amdgcn_sched_barrier(0);
        unroll<kKeys>([&](auto i) { fetch_key(raw_a, 0, i); });
        __builtin_amdgcn_sched_barrier(0);
        dma_q();                                             // (they and what follows land under the conversion of the values)
        if (n_tiles == 1) {                                  // no requests that nobody reads
            first_values();
            landed(std::integral_constant<int, 0>{});
        } else {
            dma_k(1, 1);
            unroll<kKeys>([&](auto i) { fetch_key(raw_b, 1, i); });
            first_values();
            unroll<kKeys>([&](auto i) { fetch_key(raw_a, min(2, n_tiles - 1), i); });
            __builtin_amdgcn_sched_barrier(0);
            landed(std::integral_constant<int, 2 * kKeys>{});                // behind the keys of tiles 0 and 1: the values of 1 and 2
        }
        read_q();
        written_barrier(std::integral_constant<int, 2 * kKeys>{});
    } else {
        landed(std::integral_constant<int, 0>{});
        read_q();
        written_barrier(std::integral_constant<int, 0>{});
    }
    Score sa, sb;
    Prob pa, pb;
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            pb.f[u][i].raw = u32x4{0u, 0u, 0u, 0u};
#if defined(__HIP_DEVICE_COMPILE__)
            // keeps the zeros in these registers: as a known constant they were written again right before a product,
            // closer than the matrix unit allows
            asm volatile("" : "+v"(pb.f[u][i].raw));
#endif
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) sa.s[u][e] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            Frag16 kf;
            kf.raw = k_frag(k_lds + r * (kHeadDim * 2), ks);
            sa.s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf.bf, qf[u][ks].bf, sa.s[u], 0, 0, 0);
        }
    }
    const char *kb_lane = k_lds + r * (kHeadDim * 2);
    const char *vb_lane = v_lds + (DIRECT ? r ^ (r >> 4) : r) * (kKTile * 2);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) k_at[ks] = kb_lane + (((2 * ks + hl) ^ k_sw) << 4);
#pragma unroll
    for (int c = 0; c < 4; ++c) v_at[c] = vb_lane + (((2 * c + hl) ^ v_sw) << 4);
    k_step = (int)kKBufBytes;                                // (v_step: even block 0 reads its own tile's values)
    Carry carry;
    unroll<kAhead>([&](auto i) { carry.f[i.value ^ 1].raw = frag_of(std::integral_constant<int, i.value ^ 1>{}, std::true_type{}); });
    // Tile kt: blocks 2 kt (keys already multiplied; scores of the tile's second half, values of the block before) and
    // 2 kt + 1.  The first block multiplies zero probabilities with the first tile's values, for accumulators that it then zeroes.
    int b3 = 0, b3p = 0;                                     // buffers of tile kt and of the values before it
    auto tile = [&](int kt, Raw &raw) __attribute__((always_inline)) {
        const int b3n = b3 == BUFS - 1 ? 0 : b3 + 1, b3nn = b3n == BUFS - 1 ? 0 : b3n + 1;
        const int kt2 = min(kt + 2, n_tiles - 1), kt1 = min(kt + 1, n_tiles - 1);      // past the end: requested, not read
        const int hb = 2 * kt;
        const char *vprev = vb_lane + b3p * (G * kVBufBytes), *vcur = vb_lane + b3 * (G * kVBufBytes);
        auto keys = [&](int i) { dma_k1(kt2, b3nn, i); };
        auto dma0 = [&](auto ic) {                           // the next tiles' kDma (NM + 1) requests, early in this one
            const int i = decltype(ic)::value;
            if constexpr (DIRECT) value_work(raw, min(kt + 3, n_tiles - 1), b3n, ic, keys);
            else if (BUFS == 2) return;                      // one tile: nothing comes after it
            else if (i < kDma) dma_v1(kt1, b3n, 0, i);
            else if (i < kDma * NM) dma_v1(kt1, b3n, 1, i - kDma);
            else if (i < kDma * (NM + 1)) dma_k1(kt2, b3nn, i - kDma * NM);
        };
        auto dma1 = [&](auto ic) {
            if constexpr (DIRECT)
                value_work(raw, min(kt + 3, n_tiles - 1), b3n, std::integral_constant<int, kHooks + decltype(ic)::value>{}, keys);
        };
        k_step = (b3n - b3) * (int)kKBufBytes;
        v_step = (b3 - b3p) * (int)(G * kVBufBytes);
        if (hb < n_hb) body(sa, sb, pb, pa, hb * 32, carry, dma0, std::true_type{});
        else {
            unroll<DIRECT ? kHooks : kDma * (NM + 1)>([&](auto i) { dma0(i); });
            if (hb == n_hb) pv_last(pb, vprev, 1);
        }
        k_step = (b3nn - b3n) * (int)kKBufBytes;             // the next tile's first fragments are requested here
        if (hb + 1 < n_hb) body(sb, sa, pa, pb, hb * 32 + 32, carry, dma1, std::false_type{});
        else {
            if constexpr (DIRECT) unroll<kHooks>([&](auto i) { dma1(i); });
            if (hb + 1 == n_hb) pv_last(pa, vcur, 0);
        }
        // (after the last tile nobody waits for the requests past the end: they fill buffers that are not read any more)
        if (kt + 1 < n_tiles) {
            if constexpr (DIRECT) written_barrier(std::integral_constant<int, kKeys>{});     // behind the keys of kt + 2: the values of kt + 3
            else tile_barrier();
        }
        b3p = b3;
        b3 = b3n;
    };
    if constexpr (DIRECT) {
        for (int kt = 0;;) {
            tile(kt, raw_b);
            if (++kt == n_tiles) break;
            tile(kt, raw_a);
            if (++kt == n_tiles) break;
        }
    } else
        for (int kt = 0; kt < n_tiles; ++kt) {
            if (__builtin_expect(kt == max(n_tiles - 2, 0), 0)) draw();
            tile(kt, raw_a);
        }
    if (n_hb == 2 * n_tiles) pv_last(pb, vb_lane + b3p * (G * kVBufBytes), 1);

    done.n_mem = NM;
    done.i0 = i0;
    done.b = brow;
#pragma unroll
    for (int g = 0; g < NM; ++g) done.heads[g] = heads[g];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        float lo, hi;
        both_halves(l_run[u], lo, hi);
        done.inv[u] = 1.0f / (lo + hi);
    }
#if defined(__HIP_DEVICE_COMPILE__)
    // the requests past the end have landed before LDS is given to another tile or workgroup
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
}

// One query tile of one group
struct Job {
    const char *ksrc, *vsrc[kGroup];                         // keys, the members' V^T
    int heads[kGroup], b, rhead, qt, n_mem;
};

// One workgroup per CU (two with rings of two) takes query tiles from its XCD's queue until that is empty.  tickets: how many tiles
// of the queue have been taken, per XCD, without the first one of every workgroup; zero at the start.
// The next tile is drawn during the last but one tile of keys of the one before, whose output rows are written when the next one's
// first requests are out.
template <int U, int NW, bool IDENT, int BUFS>
__global__ __launch_bounds__(NW * 64, NW / 4) void prefill_kernel(const char *__restrict__ q, const char *__restrict__ kc,
                                                                  const _Float16 *__restrict__ vt,
                                                                  const int32_t *__restrict__ groups,
                                                                  const int32_t *__restrict__ n_groups, int H, int k,
                                                                  int Tq, int q_start, int Tc_cap, int Tp, int n_qt,
                                                                  int n_slots, int n_rows, float scale,
                                                                  float *__restrict__ out, int32_t *__restrict__ tickets,
                                                                  int ticket_stride)
{
    extern __shared__ __attribute__((aligned(1024))) char lds_raw[];
    constexpr int G = IDENT ? 1 : kGroup;
    char *const k_lds = lds_raw, *const v_lds = lds_raw + BUFS * kKBufBytes;
    // the next item for all waves: behind the rings, or in the second key tile, which rings of two do not use
    unsigned *const drawn = reinterpret_cast<unsigned *>(lds_raw + (BUFS == 2 ? kKBufBytes : prefill_rings(IDENT, BUFS, NW * 32 * U)));
    const WorkQueue queue = make_queue<IDENT>(n_groups, n_rows, H, n_qt);
    const unsigned xcd = blockIdx.x % kXcds, n_wg = gridDim.x / kXcds;
    int32_t *const ticket = tickets + (xcd >> 2) * ticket_stride + (xcd & 3);
    const bool draws = threadIdx.x == 0;
    // the item after i of this workgroup's kind that exists, by the draws of thread 0
    auto settle = [&](unsigned i) {
        unsigned group;
        int qt;
        while (i < queue.n_items && !queue_item(queue, n_qt, i, group, qt)) i = n_wg + (unsigned)atomicAdd(ticket, 1);
        return i;
    };
    auto look_up = [&](unsigned i, Job &job) {
        unsigned group;
        int b, gi, cluster, rhead, heads[kGroup];
        queue_item(queue, n_qt, i, group, job.qt);
        find_row<IDENT>(queue, n_groups, n_rows, H, group, b, gi);
        b = __builtin_amdgcn_readfirstlane(b);
        gi = __builtin_amdgcn_readfirstlane(gi);
        job.qt = __builtin_amdgcn_readfirstlane(job.qt);
        if (IDENT) {
            cluster = rhead = heads[0] = heads[1] = gi;
            job.n_mem = 1;
        } else {
            const int32_t *gr = groups + ((size_t)b * n_slots + gi) * kRec;
            cluster = min(gr[0] & ((1 << kRecCount) - 1), k - 1);
            job.n_mem = min(max(gr[0] >> kRecCount, 1), kGroup);
#pragma unroll
            for (int g = 0; g < kGroup; ++g) heads[g] = min(max(gr[1 + min(g, job.n_mem - 1)], 0), H - 1);
            rhead = min(max(gr[1 + kGroup], 0), H - 1);
        }
        job.ksrc = kc + ((size_t)b * k + cluster) * (size_t)Tc_cap * (kHeadDim * 2);
        job.rhead = rhead;
        job.b = b;
#pragma unroll
        for (int g = 0; g < kGroup; ++g) {
            job.vsrc[g] = reinterpret_cast<const char *>(vt + ((size_t)b * H + heads[g]) * (size_t)kHeadDim * Tp);
            job.heads[g] = heads[g];
        }
    };
    auto barrier = [&]() {
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#endif
    };

    unsigned item = blockIdx.x / kXcds, group;
    int qt;
    const bool each = queue.n_items <= n_wg;                 // every item has a workgroup of its own: nothing is drawn
    if (item >= queue.n_items) return;
    if (!queue_item(queue, n_qt, item, group, qt)) {
        if (each) return;
        if (draws) *drawn = settle(item);
        barrier();
        item = (unsigned)__builtin_amdgcn_readfirstlane((int)*drawn);
        if (item >= queue.n_items) return;
    }
    Job job;
    look_up(item, job);
    Finished<U> done;
    done.n_mem = 0;
    int later = 0;
    auto draw = [&]() {
        if (BUFS > 2 && !each && draws) later = atomicAdd(ticket, 1);
    };
    for (bool more = true;;) {
        // rows of another number of members than the next tile's are written by themselves
        const bool tile = more && (done.n_mem == 0 || done.n_mem == job.n_mem);
        const int n_mem = tile ? job.n_mem : done.n_mem;
        if (!IDENT && n_mem == 2)
            prefill_tile<2, U, NW, G, BUFS, false>(k_lds, v_lds, job.ksrc, job.vsrc, q, job.heads, job.b, H, Tq, q_start, job.qt, tile,
                                                   job.rhead, scale * kLog2e, out, done, draw);
        else
            prefill_tile<1, U, NW, G, BUFS, false>(k_lds, v_lds, job.ksrc, job.vsrc, q, job.heads, job.b, H, Tq, q_start, job.qt, tile,
                                                   job.rhead, scale * kLog2e, out, done, draw);
        if (!tile) {
            if (!more) break;
            continue;
        }
        if (BUFS == 2 || each) {
            more = false;
            continue;
        }
        if (draws) *drawn = settle(n_wg + (unsigned)later);
        barrier();                                           // nobody reads this tile's keys and values any more
        item = (unsigned)__builtin_amdgcn_readfirstlane((int)*drawn);
        more = item < queue.n_items;
        if (more) look_up(item, job);
    }
}

// Cluster, members and representative of group gi of row b (the groups of plan_row, in the same order), found by every workgroup
// for itself; false: the row has fewer groups.  All the map entries are requested at once.  LDS: kPlanClusters ints.
constexpr int kPlanClusters = 64, kPlanHeads = 256;          // most of them
__device__ __forceinline__ bool find_group(const int32_t *__restrict__ h2c, const int32_t *__restrict__ rep, int b, int gi, int H,
                                           int k, int32_t *count, int &cluster, int &n_mem, int (&heads)[kGroup], int &rhead)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int32_t *row = h2c + (size_t)b * H;
    const int rep_j = lane < k ? rep[(size_t)b * k + lane] : -1, mine = tid < H ? row[tid] : -1;
    int label[kPlanHeads / 64];
#pragma unroll
    for (int i = 0; i < kPlanHeads / 64; ++i) label[i] = i * 64 + lane < H ? row[i * 64 + lane] : -1;
    if (tid < kPlanClusters) count[tid] = 0;
    __syncthreads();
    if (mine >= 0 && mine < k) atomicAdd(&count[mine], 1);
    __syncthreads();
    const int n = rep_j >= 0 ? count[lane] : 0;
    __syncthreads();                                         // the counts give way to tiles
    int upto = (n + kGroup - 1) / kGroup;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int other = __shfl_up(upto, o);
        upto += lane >= o ? other : 0;
    }
    if (gi >= __builtin_amdgcn_readlane(upto, 63)) return false;
    cluster = __popcll(__ballot(upto <= gi));
    const int first = kGroup * (gi - (cluster > 0 ? __builtin_amdgcn_readlane(upto, cluster - 1) : 0));
    n_mem = min(__builtin_amdgcn_readlane(n, cluster) - first, kGroup);
    rhead = min(__builtin_amdgcn_readlane(rep_j, cluster), H - 1);
    int seen = -first;
#pragma unroll
    for (int i = 0; i < kPlanHeads / 64; ++i) {
        const unsigned long long votes = __ballot(label[i] == cluster);
        const int rank = seen + __popcll(votes & ((1ull << lane) - 1ull));
#pragma unroll
        for (int g = 0; g < kGroup; ++g) {
            const unsigned long long it = __ballot(label[i] == cluster && rank == g);
            if (it != 0ull) heads[g] = i * 64 + __ffsll((long long)it) - 1;
        }
        seen += __popcll(votes);
    }
    if (n_mem < kGroup) heads[1] = heads[0];
    return true;
}

// ---------------------------------------------------------------------------------------------------------
// The kernel of 128-row tiles without the pre-pass: for calls with few query tiles per head (rule in prefill_is_direct), which
// spent up to half of their time on writing V^T for a few rows to read it (256 positions behind 1792 keys, 4 rows x 52 heads in
// 8 clusters: 37 of 93 us).  A value tile comes as rows through registers, requested two tiles ahead; while a block is
// multiplied, a thread turns 8 keys x 8 columns (NM = 2) into eight pieces of V^T and writes them to the tile after this one,
// spread over the slots of both blocks.  What it costs: 64 conversions' worth of instructions and 8 LDS writes per wave and tile
// (about 400 cycles), loads to registers instead of to LDS (about 380, 8 requests of 1 KB each); a tile of 64 keys and two
// members takes 3400 cycles, 2550 without all of it, of which the products are 1536: a lone wave's issue slots.  The call above
// 86 us with the pre-pass, 56 so; 507 positions behind 5 keys, 4 x 72 heads in 16 clusters 58 and 48 us; 24 behind 4000, 16 x 32 in 8 394
// and 191 us.  One tile of keys has a start of its own, which requests no second one, and a wave of at most 16 rows leaves out half
// of the stores: 37 x 12 positions, 128 heads in 8 clusters 62.3 -> 56.5 us.
//
// The groups of a row are found by every workgroup for itself (a launch for the work list would cost 5 us).  Workgroups are
// numbered group by group, all rows of one before the next, the longest query tiles first: the XCDs get equal shares without
// any of them knowing the other rows' groups.  (by_group: all query tiles of a group before the next group.  The groups that the
// rows do not have are all at the end then, and the others' tiles fill the CUs of all XCDs alike: 1 row x 64 heads in 2 clusters, 862
// positions behind 3018 keys, 33 groups of seven tiles, 144 -> 104 us when the tile took 3400 cycles; 100 now, 105 with the pre-pass.)
// ---------------------------------------------------------------------------------------------------------
template <bool IDENT>
__global__ __launch_bounds__(256, 1) void prefill_direct_kernel(const char *__restrict__ q, const char *__restrict__ kc,
                                                                const char *__restrict__ v, const int32_t *__restrict__ h2c,
                                                                const int32_t *__restrict__ rep, int H, int k, int Tq, int q_start,
                                                                int Tc_cap, int T_cap, int n_qt, int n_rows, int per_xcd, int by_group,
                                                                float scale, float *__restrict__ out)
{
    extern __shared__ __attribute__((aligned(1024))) char lds_raw[];
    const unsigned inner = by_group ? (unsigned)n_qt : kXcds * (unsigned)per_xcd, quot = blockIdx.x / inner, rest = blockIdx.x - quot * inner;
    const int qt = n_qt - 1 - (int)(by_group ? rest : quot);
    const unsigned at = by_group ? quot : rest;
    int gi = (int)(at / (unsigned)n_rows);
    const int b = (int)(at - (unsigned)gi * (unsigned)n_rows);
    int cluster = gi, n_mem = 1, rhead = gi, heads[kGroup] = {gi, gi};
    if (IDENT) {
        if (gi >= H) return;
    } else {
        if (!find_group(h2c, rep, b, gi, H, k, reinterpret_cast<int32_t *>(lds_raw), cluster, n_mem, heads, rhead)) return;
#pragma unroll
        for (int g = 0; g < kGroup; ++g) heads[g] = __builtin_amdgcn_readfirstlane(heads[g]);
    }
    const char *vsrc[kGroup];
#pragma unroll
    for (int g = 0; g < kGroup; ++g) vsrc[g] = v + ((size_t)b * H + heads[g]) * (size_t)T_cap * (kHeadDim * 2);
    const char *ksrc = kc + ((size_t)b * k + cluster) * (size_t)Tc_cap * (kHeadDim * 2);
    Finished<1> done;
    done.n_mem = 0;
    auto none = []() {};
    if (!IDENT && n_mem == 2)
        for (int pass = 0; pass < 2; ++pass)
            prefill_tile<2, 1, 4, kGroup, kBufs, true>(lds_raw, lds_raw + kBufs * kKBufBytes, ksrc, vsrc, q, heads, b, H, Tq, q_start, qt,
                                                       pass < 1, rhead, scale * kLog2e, out, done, none);
    else
        for (int pass = 0; pass < 2; ++pass)
            prefill_tile<1, 1, 4, IDENT ? 1 : kGroup, kBufs, true>(lds_raw, lds_raw + kBufs * kKBufBytes, ksrc, vsrc, q, heads, b, H, Tq,
                                                                   q_start, qt, pass < 1, rhead, scale * kLog2e, out, done, none);
}

size_t round256(size_t x) { return (x + 255) / 256 * 256; }

}  // namespace

int prefill_max_groups(int H, int k) { return (H + kGroup - 1) / kGroup + k; }

// work list + group counts + V^T
size_t prefill_workspace_bytes(int B, int H, int k, int n_keys)
{
    const size_t Tp = ((size_t)n_keys + kKTile - 1) / kKTile * kKTile;
    return round256((size_t)B * prefill_max_groups(H, k) * kRec * sizeof(int32_t)) +
           round256((size_t)B * sizeof(int32_t)) + round256((size_t)B * H * kHeadDim * Tp * sizeof(_Float16));
}

// The most groups of a row that there can be: a cluster has half a group more than half its heads at most.
static int direct_groups(int H, int k, bool identity)
{
    static_assert(kGroup == 2, "half a group");
    return identity || (H + k) / 2 > H ? H : (H + k) / 2;
}

// Which calls skip the pre-pass: those with few query tiles per head.  The pre-pass reads and writes all values once (two bytes each
// way at 6.5 TB/s, and 3 us); converting them in the 128-row tiles costs every tile of 64 keys 0.3 us per group of two members and
// 0.15 us per head alone, in each query tile again, where longer calls have 256-row tiles, which are a fifth faster per row.
// Whole calls, with pre-pass / direct in us:
// * one or two query tiles: 4 rows x 52 heads in 8 clusters, 24 behind 0 / 400 / 1792 / 4000 keys 12 / 7, 30 / 16, 71 / 45 and 148 /
//   90, 256 behind the same 23 / 14, 38 / 25, 86 / 56 and 168 / 115; 16 x 72 in 16, 128 behind 0 / 1792 43 / 32 and 396 / 189;
//   dense, 16 x 32 heads, 24 behind 0 / 1792 13 / 9 and 191 / 90, 200 behind 0 / 400 / 1792 40 / 37, 82 / 74 and 235 / 225.  Not
//   where a handful of heads makes the pre-pass cheap next to a long chain of tiles: 1 x 32 in 8, 24 behind 400 / 1792 / 4000
//   18 / 16, 48 / 44 and 87 / 89; dense, 1 x 8, 128 behind 1000 / 2500 / 4000 25 / 24, 48 / 49 and 72 / 74.  Nor for blocks
//   of at most one key tile on thousands of heads, which have two workgroups per CU (64 x 72, 24 keys 55 / 67, but 65 keys
//   153 / 114, and 32 x 52, 24 keys 30 / 28).
// * clustered, more: three 4 x 72 in 16, 384 behind 0 / 1792 41 / 31 and 153 / 129; four 4 x 72, 507 behind 0 / 1792 57 / 43 and
//   201 / 171, 16 x 72 in 16, 507 behind 0 / 400 178 / 174 and 299 / 312; five 16 x 32 in 8, 600 behind 0 / 800 108 / 98 and 243 /
//   227; six (three whole wide tiles) 4 x 52 in 8, 700 behind 0 / 800 65 / 53 and 122 / 114, 4 x 72 in 16, 700 behind 200 / 800 96 / 104
//   and 145 / 168.  Each key tile behind costs seven query tiles seven conversions: 12 x 52 in 4, 860 behind 0 / 200 200 / 186 and 257 /
//   251, but 3 x 72 in 8, 842 behind 1223 174 / 188, 9 x 52 in 8, 885 behind 555 259 / 300, 4 x 32 in 8, 872 behind 2090 161 / 188;
//   eight 4 x 52 in 8, 1000 behind 0 83 / 80, but 6 x 52 in 4, 926 behind 0 114 / 118.
// * dense, more: while the tiles are one round of the chip (1 x 32, 1000 behind 0 / 800 30 / 23 and 45 / 38); beyond, three 6 x 52,
//   300 behind 0 / 800 44 / 39 and 118 / 98, but just over one round 2 x 52, 384 behind 1792 / 4000 76 / 76 and 146 / 153, and on
//   many heads 12 x 72, 384 behind 400 230 / 252; four 6 x 52, 400 behind 0 / 200 / 800 59 / 56, 79 / 82 and 140 / 136, 8 x 72, 400
//   behind 0 94 / 100; five 4 x 52, 600 behind 0 / 200 63 / 57 and 78 / 82; six 2 x 52, 700 behind 0 38 / 35, 4 x 52, 733 behind 0
//   70 / 72, 6 x 52 102 / 111; seven 2 x 52, 869 behind 0 49 / 44, 2 x 96 81 / 87, 6 x 52 133 / 141; eight 4 x 52, 1000 behind 0
//   108 / 116.
// The lines were drawn with kernels of which the direct one was 4 to 10 % slower and the other, without a queue, up to 13 %.  Of 1171
// clustered and 631 dense calls drawn at random (8 to 128 heads, 1 to 24 rows, up to 1024 positions behind up to 6000 keys) 2.6 and 2.9 %
// are more than 3 % slower than the other way, mostly with five to seven query tiles and just beyond one round of the chip (17 x 709
// behind 87, 64 in 4 283 / 331, dense 1 x 987, 40 heads 30 / 23); against the pre-pass everywhere they take 1 / 1.43 and 1 / 1.35.
static bool prefill_is_direct(int B, int H, int k, int Tq, int q_start, bool identity)
{
    const long long heads = (long long)B * H, n_keys = (long long)q_start + Tq;
    const int n = (Tq + 127) / 128;
    if (identity) {
        if (n_keys <= kKTile && heads >= 2048) return false;
        if (n_keys * (2200 - 79 * heads) > 3800000) return false;
        if (n <= 2) return true;
        if (heads * n <= 256) return n <= 8;
        if (n == 3) return q_start <= 256 || (heads <= 600 && (heads * n > 512 || q_start <= 1024));
        return n <= 7 && q_start <= 128 && heads <= (n == 4 ? 400 : (n == 5 ? 320 : (n == 6 ? 128 : 180)));
    }
    if (H > kPlanHeads || k > kPlanClusters) return false;  // (more than a workgroup looks through for its group)
    if (n_keys * (4700 - 79 * heads) > 3300000) return false;
    if (n <= 3) return true;
    const long long most = (long long)direct_groups(H, k, false) * B, wide = (long long)(n / 2) * prefill_max_groups(H, k) * B;
    if (n == 4) return q_start <= 128 || wide <= 420 || (wide <= 1300 && q_start <= 512);
    if (n == 5) return q_start <= 512 || most <= 420;
    if (n == 6) return (q_start <= 128 && most <= 800) || most <= 110 || (most <= 180 && q_start <= 512);
    if (n == 7) return most * (q_start + 400) <= 195000;
    return n == 8 && most * (q_start + 100) <= 20000;
}

int launch_prefill(const void *q, const void *kc, const void *v, const int32_t *h2c, const int32_t *rep, int B, int H,
                   int k, int Tq, int q_start, int Tc_cap, int T_cap, float scale, float *out, void *workspace,
                   bool identity, const KernelEvents &ev, hipStream_t stream)
{
    const int n_keys = q_start + Tq;
    const int Tp = (n_keys + kKTile - 1) / kKTile * kKTile;
    const int max_groups = identity ? H : prefill_max_groups(H, k);
    char *ws = static_cast<char *>(workspace);
    int32_t *groups = reinterpret_cast<int32_t *>(ws);
    ws += round256((size_t)B * prefill_max_groups(H, k) * kRec * sizeof(int32_t));
    int32_t *n_groups = reinterpret_cast<int32_t *>(ws);
    ws += round256((size_t)B * sizeof(int32_t));
    _Float16 *vt = reinterpret_cast<_Float16 *>(ws);

    if (prefill_is_direct(B, H, k, Tq, q_start, identity)) {
        auto *kernel = identity ? prefill_direct_kernel<true> : prefill_direct_kernel<false>;
        const size_t lds_bytes = prefill_rings(identity, kBufs, 128);
        static DeviceFlags lds_allowed[2];
        const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), lds_bytes, lds_allowed[identity ? 1 : 0]);
        if (e != hipSuccess) return (int)e;
        const int n_qt = (Tq + 127) / 128;
        const long long groups = (long long)direct_groups(H, k, identity) * B, tiles = groups * n_qt;
        long long per_xcd = ((long long)max_groups * B + kXcds - 1) / kXcds;
        // One round of the chip, or nearly: no room for groups that cannot be, and where whole groups per XCD would still make two
        // rounds on some, group by group.  Not where a second round can be of short chains only, which the longest are better not.
        // (Beyond, the numbering with room was as fast on average, and up to 10 % either way.)
        if (per_xcd * n_qt > kXcdCus && tiles <= (kXcds + 1) * kXcdCus) per_xcd = (groups + kXcds - 1) / kXcds;
        const bool by_group = per_xcd * n_qt > kXcdCus && kXcdCus % n_qt != 0 &&
                              (identity ? tiles <= kXcds * kXcdCus
                                        : (q_start >= 256 ? tiles <= (kXcds + 1) * kXcdCus : (tiles <= kXcds * kXcdCus && n_qt < 7)));
        const long long n_wg = kXcds * per_xcd * n_qt;
        if (n_wg > 0xffffff) return (int)hipErrorInvalidConfiguration;
        return (int)launch_kernel(kernel, dim3((unsigned int)n_wg), dim3(256), lds_bytes, stream, ev,
                                  static_cast<const char *>(q), static_cast<const char *>(kc), static_cast<const char *>(v), h2c, rep,
                                  H, k, Tq, q_start, Tc_cap, T_cap, n_qt, B, (int)per_xcd, by_group, scale, out);
    }

    const size_t tile_lds = (size_t)kHeadDim * (kKTile + 2) * sizeof(_Float16), plan_lds = (size_t)(H + 2 * k) * sizeof(int32_t);
    // Eight tickets in ints of the workspace that nothing else uses: the work list of a dense call; the last records of the first two
    // rows' lists (a row has at most (H + k) / 2 groups, one less than its list has room for); behind the count of a single row.
    int32_t *const tickets = identity ? groups : (B == 1 ? n_groups + 4 : groups + (size_t)(max_groups - 1) * kRec);
    const int ticket_stride = identity || B == 1 ? 4 : max_groups * kRec;
    static_assert(kRec >= 4 && kXcds == 8, "four tickets to a record");
    const int n_lists = identity ? 0 : B;
    const long long n_pre = n_lists + (long long)(Tp / kKTile) * H * B;
    if (n_pre > 0xffffff) return (int)hipErrorInvalidConfiguration;       // 256 GB of values
    hipError_t e = launch_kernel(prepass_kernel, dim3((unsigned int)n_pre), dim3(256),
                                 identity || plan_lds < tile_lds ? tile_lds : plan_lds, stream, KernelEvents(),
                                 static_cast<const char *>(v), H, T_cap, n_keys, Tp, vt, n_lists, h2c, rep, k, max_groups, groups,
                                 n_groups, tickets, ticket_stride);
    if (e != hipSuccess) return (int)e;
    // Tiles of 256 or of 128 query rows: 128 where the wide tiles would leave CUs without work or end in a ragged last round,
    // and where a block has no more rows than that.  The lines lie at a number of 256-row tiles of the most groups the maps
    // can have; they were drawn when every workgroup took a pair of tiles.  Since workgroups draw tiles from a queue, which does away
    // with ragged rounds, they send many calls of five and six narrow tiles the wrong way.  Whole calls with 256 / 128 rows, in us:
    // five narrow tiles, 513 positions, 12 rows x 52 heads in 8 clusters 122 / 115, 16 x 52 in 4 155 / 146, 30 x 32 in 8 190 / 191, but 64 x
    // 32 in 8 380 / 394, behind 200 498 / 533, 16 x 72 in 16 behind 1000 550 / 589.  Three, where launch and block are short: 257
    // positions, 12 x 52 and 30 x 32 in 8 (816 and 1440 tiles) 74 / 62 and 107 / 90, behind 128 88 / 76 and 131 / 118, behind 200 99 /
    // 87 and 146 / 135, 16 x 72 in 16 (1664 tiles) 118 / 109 and with 300 positions 126 / 117, 64 x 32 (3072) 207 / 196.  Six against
    // three wide ones between 900 and 1450: 768 positions, 16 x 52 in 4 (1440) 203 / 224, 16 x 32 in 4 (960) 131 / 140, 8 x 52 (720)
    // 110 / 108, and 641 positions, 64 x 32 in 8 (4608) 444 / 523.  (Of three and five tiles what is
    // left here is past the lines of prefill_is_direct, or of more heads or clusters than it takes: 1 x 260 in 4, 300 positions.)
    // Dense: up to 128 wide tiles the narrow ones are one round too, above 256 the wide ones fill the chip better.
    // Between, two narrow tiles share a CU one after the other, the longest with the shortest: the second
    // round starts with the 256-th longest, 128 * 256 / heads keys below the longest.  With 7 us for a start and 20 against 30
    // ns per key of a narrow and a wide tile, two of those take less than one wide tile where
    // heads * (4 (q_start + Tq in whole tiles) - 3 keys + 700) <= 131072.  Wide / narrow: one query tile per head, 256 keys,
    // 160 / 192 / 256 heads 22.9 / 24.4, 23.9 / 25.7, 27.0 / 31.1 us, 256 behind 1000 keys 78 / 89; two tiles, 512 keys,
    // 72 / 96 / 128 heads 26.3 / 23.9, 27.8 / 27.5, 30.1 / 34.0; four, 1000 keys, 64 heads 40.3 / 41.2, behind 1000 73 / 77; eight, 2000,
    // 32 heads 62 / 56, behind 1000 91 / 91.  Blocks of up to 128 rows fill half a wide tile: 512 heads, 100 rows
    // 27.0 / 27.2, 24 rows 16.3 / 12.8.
    const long long tiles = (long long)((Tq + 255) / 256) * max_groups * B;
    const int n_narrow = (Tq + 127) / 128;
    bool small = Tq <= 128 || tiles <= (identity ? 128 : kSmallTiles);
    if (!identity)
        small = small || (n_narrow == 3 && q_start <= 128 && tiles <= kFewTiles) || n_narrow == 5 ||
                (n_narrow == 6 && tiles >= 2 * kSmallTiles && tiles <= kFewTiles);
    if (identity && tiles <= 256)
        small = small || (long long)B * H * (4LL * (q_start + (Tq + 127) / 128 * 128) - 3LL * n_keys + 700) <= 131072;
    const bool brief = identity && n_keys <= kKTile;        // (thousands of heads of one narrow query tile)
    auto *kernel = small ? (identity ? (brief ? prefill_kernel<1, 4, true, 2> : prefill_kernel<1, 4, true, kBufs>)
                                     : prefill_kernel<1, 4, false, kBufs>)
                         : (identity ? prefill_kernel<1, 8, true, kBufs> : prefill_kernel<2, 4, false, kBufs>);
    const int threads = identity && !small ? 512 : 256, tile_rows = small ? 128 : 256;
    const size_t lds_bytes = prefill_lds_bytes(identity, brief ? 2 : kBufs, tile_rows);
    static DeviceFlags lds_allowed[5];
    e = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), lds_bytes, lds_allowed[brief ? 4 : (small ? 2 : 0) + (identity ? 1 : 0)]);
    if (e != hipSuccess) return (int)e;
    const int n_qt = (Tq + tile_rows - 1) / tile_rows;
    // items are numbered in 32 bits (make_queue)
    if ((long long)max_groups * B * (n_qt + 1) > 0x1fffffff) return (int)hipErrorInvalidConfiguration;
    // One workgroup per CU, which draws tile after tile, from two rounds on; fewer tiles, and dense ones of at most two tiles of keys,
    // have a workgroup each (as many as an XCD's queue can have items: its tiles, and room for two groups' where the last pairs are
    // dealt as single tiles).  Drawing / a workgroup per tile or pair of tiles: 16 x 2043 positions, 32 heads in 8 clusters 556 / 569
    // us, 12 x 900 behind 200, 52 in 8 270 / 279, 2 x 2043, 72 in 16 166 / 169, dense 64 x 300 behind 300, 32 heads 403 / 444, 16 x 400
    // behind 200, 72 heads 247 / 261; but 1 x 2043, 32 in 8 (300 tiles) 53.9 / 51.9, dense 64 x 65, 72 heads
    // 117.6 / 115.7; level within 1 % for short prompts of many rows (64 x 300, 32 in 8 198.1 / 196.8; 64 x 600 428 / 426).
    const long long tiles_most = (long long)max_groups * B * n_qt, n_pairs = (n_qt + 1) / 2;
    const long long per_xcd = ((long long)max_groups * B * n_pairs + kXcds - 1) / kXcds;
    const bool drawn = tiles_most >= 2 * kXcds * kXcdCus && !(identity && n_keys <= 2 * kKTile);
    const long long n_wg = drawn ? kXcds * kXcdCus : kXcds * (n_qt == 1 ? per_xcd : 2 * per_xcd + 4 * n_pairs);
    if (n_wg > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    return (int)launch_kernel(kernel, dim3((unsigned int)n_wg), dim3(threads), lds_bytes, stream, ev,
                              static_cast<const char *>(q), static_cast<const char *>(kc), vt, groups, n_groups, H, k, Tq,
                              q_start, Tc_cap, Tp, n_qt, max_groups, B, scale, out, tickets, ticket_stride);
}

}  // namespace chai
