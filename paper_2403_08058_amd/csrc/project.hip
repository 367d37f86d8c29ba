// Query / key projections of the representative heads only (Fig. 3, Section 3.5: clustered attention needs the
// query and key vectors of one head per cluster, so the columns of W_Q and W_K that belong to the other heads are
// never multiplied; the new keys go straight into the pruned K cache).  A dense contraction with reuse on both
// operands, so it runs on the matrix cores.
//
//   for batch row b, slot j, r = rep_heads[b][j] >= 0, token i < Tn:
//       q_out[b][r][i][:]            = bf16( x[b][i][:] . w_q[r*128 .. r*128+127][:]^T )
//       k_compact[b][j][pos0 + i][:] = bf16( x[b][i][:] . w_k[r*128 .. r*128+127][:]^T )
//
// Three kernels, chosen in launch_project_qk by the number of tokens; this is the one for prompts.  One workgroup
// (8 waves) computes a 256-token x 256-column tile: the 128 query columns and the 128 key columns of one
// representative, which share the activation tile.  The product is formed transposed, C^T = W X^T, with
// v_mfma_f32_32x32x16_bf16: both operands are then read along the contraction axis (weights are stored one row
// per output feature), a lane owns one token and gets 4 consecutive output features per register quad, so rows
// are written in 8-byte pieces.  Operand tiles of 64 contraction steps go global -> registers -> LDS (double
// buffered, one barrier per step); fp32 accumulation, one rounding to bf16 at the end.
#include "chai_internal.h"

#include <hip/hip_ext.h>

namespace chai {

namespace {

constexpr int kJBlock = 512;                 // threads (8 waves: 4 along the tokens x 2 along the columns)
constexpr int kJTok = 256;                   // tokens per workgroup tile
constexpr int kJCol = 2 * kHeadDim;          // columns per workgroup tile: query + key columns of one head
constexpr int kJStep = 64;                   // contraction elements per LDS tile
constexpr int kJStride = kJStep + 8;         // halves per LDS row (144 B: rows land on different banks)
constexpr size_t kJTileBytes = (size_t)(kJTok + kJCol) * kJStride * 2;     // activations + weights, one stage
constexpr size_t kJLdsBytes = 2 * kJTileBytes;
constexpr int kJPieces = (kJTok + kJCol) * kJStep * 2 / 16 / kJBlock;      // 16-byte pieces per thread per stage (8)

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

union Frag {
    u32x4 raw;
    bf16x8 bf;
};

// 1-D grid of n_mt * k * B workgroups, renumbered so that each XCD owns a contiguous range of (batch row, token
// tile) pairs with all their cluster slots: the slots of a pair read the same activations and find them in L2.
__global__ __launch_bounds__(kJBlock) void project_kernel(const char *__restrict__ x, const char *__restrict__ w_q,
                                                          const char *__restrict__ w_k,
                                                          const int32_t *__restrict__ rep, int H, int k, int Tn, int D,
                                                          int n_mt, char *__restrict__ q_out,
                                                          char *__restrict__ k_compact, int pos0, int Tc_cap)
{
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int r = lane & 31, hl = lane >> 5;
    const int wm = w & 3, wn = w >> 2;               // wave's 64-token strip, and query (0) or key (1) half

    int j, mt, b;
    {
        const unsigned n = blockIdx.x, N = gridDim.x;
        const unsigned xcd = n & 7u, per = N >> 3, rem = N & 7u;
        const unsigned item = xcd * per + min(xcd, rem) + (n >> 3);
        j = (int)(item % (unsigned)k);
        const unsigned rest = item / (unsigned)k;
        mt = (int)(rest % (unsigned)n_mt);
        b = (int)(rest / (unsigned)n_mt);
    }
    const int head = rep[(size_t)b * k + j];
    if (head < 0) return;
    const int rh = min(head, H - 1);
    const int t0 = mt * kJTok;

    // staging: a thread's piece i (of 8) is 16 bytes of row (tid >> 3) + 64 i of the stage, rows 0..255 being the
    // activation tile and rows 256..511 the weight tile (query rows, then key rows).  Uniform base pointers plus
    // 32-bit per-lane offsets (one batch row of activations and one head's weights are far below 4 GiB).
    const unsigned int row_bytes = (unsigned int)D * 2u;
    const int srow = tid >> 3, c = tid & 7;
    const char *xb = x + (size_t)b * Tn * row_bytes;
    const char *wqb = w_q + (size_t)rh * kHeadDim * row_bytes;
    const char *wkb = w_k + (size_t)rh * kHeadDim * row_bytes;
    unsigned int xoff[4], woff[2];
#pragma unroll
    for (int i = 0; i < 4; ++i) xoff[i] = (unsigned int)min(t0 + srow + 64 * i, Tn - 1) * row_bytes + c * 16;
#pragma unroll
    for (int i = 0; i < 2; ++i) woff[i] = (unsigned int)(srow + 64 * i) * row_bytes + c * 16;
    const int dst0 = (srow * kJStride + c * 8) * 2;
    u32x4 regs[kJPieces];
    auto fetch = [&](int step) {
        const unsigned int so = (unsigned int)step * (kJStep * 2);
#pragma unroll
        for (int i = 0; i < 4; ++i) regs[i] = *reinterpret_cast<const u32x4 *>(xb + (xoff[i] + so));
#pragma unroll
        for (int i = 0; i < 2; ++i) regs[4 + i] = *reinterpret_cast<const u32x4 *>(wqb + (woff[i] + so));
#pragma unroll
        for (int i = 0; i < 2; ++i) regs[6 + i] = *reinterpret_cast<const u32x4 *>(wkb + (woff[i] + so));
    };
    auto stage = [&](int buf) {
#pragma unroll
        for (int i = 0; i < kJPieces; ++i)
            *reinterpret_cast<u32x4 *>(lds + buf * kJTileBytes + dst0 + i * 64 * kJStride * 2) = regs[i];
    };

    f32x16 acc[4][2];                                // [column block of 32][token block of 32]
#pragma unroll
    for (int nb = 0; nb < 4; ++nb)
#pragma unroll
        for (int tb = 0; tb < 2; ++tb)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[nb][tb][e] = 0.f;

    // fragment addresses inside a stage: weights (A operand) rows kJTok + wn*128 + nb*32 + r, activations
    // (B operand) rows wm*64 + tb*32 + r; 8 halves at 16*ks + 8*hl
    const int a_off = ((kJTok + wn * kHeadDim + r) * kJStride + hl * 8) * 2;
    const int b_off = ((wm * 64 + r) * kJStride + hl * 8) * 2;

    const int n_steps = D / kJStep;
    fetch(0);
    stage(0);
    if (n_steps > 1) fetch(1);
    __syncthreads();
    for (int s = 0; s < n_steps; ++s) {
        const int buf = s & 1;
        if (s + 1 < n_steps) stage(buf ^ 1);          // fetched one iteration ago
        if (s + 2 < n_steps) fetch(s + 2);
        const char *base = lds + buf * kJTileBytes;
        // scheduling hint: spread the LDS reads and the stage's global loads and LDS writes between the MFMAs of
        // the step instead of grouping them (measured: about 2 % faster)
        __builtin_amdgcn_iglp_opt(1);
#pragma unroll
        for (int ks = 0; ks < kJStep / 16; ++ks) {
            Frag af[4], bfr[2];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
                af[nb].raw = *reinterpret_cast<const u32x4 *>(base + a_off + (nb * 32 * kJStride + ks * 16) * 2);
#pragma unroll
            for (int tb = 0; tb < 2; ++tb)
                bfr[tb].raw = *reinterpret_cast<const u32x4 *>(base + b_off + (tb * 32 * kJStride + ks * 16) * 2);
#pragma unroll
            for (int nb = 0; nb < 4; ++nb)
#pragma unroll
                for (int tb = 0; tb < 2; ++tb)
                    acc[nb][tb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[nb].bf, bfr[tb].bf, acc[nb][tb], 0, 0, 0);
        }
        __syncthreads();
    }

    // D[(v/4)*8 + hl*4 + v%4][r]: this lane's token is t0 + wm*64 + tb*32 + r, its features nb*32 + (v/4)*8 + hl*4 ..+3
    char *orow_base = wn == 0 ? q_out + ((size_t)b * H + rh) * (size_t)Tn * (kHeadDim * 2)
                              : k_compact + (((size_t)b * k + j) * (size_t)Tc_cap + pos0) * (kHeadDim * 2);
#pragma unroll
    for (int tb = 0; tb < 2; ++tb) {
        const int t = t0 + wm * 64 + tb * 32 + r;
        if (t >= Tn) continue;
        char *orow = orow_base + (size_t)t * (kHeadDim * 2);
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)acc[nb][tb][v4 * 4 + e];
                *reinterpret_cast<bf16x4 *>(orow + (nb * 32 + v4 * 8 + hl * 4) * 2) = o;
            }
    }
}

// The (row, slot) pairs that `head` represents, as indexes into rep, ascending: all workgroups of a head agree which
// tokens belong to which chunk.  Returns their number; B*k <= kJrMaxSlots.  Every thread of the workgroup calls it.
constexpr int kJrMaxSlots = 1024;
template <int WAVES>
__device__ __forceinline__ int list_slots(const int32_t *__restrict__ rep, int n, int head, int H, int *slots, int *wave_slots)
{
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    int n_slots = 0;
    for (int i0 = 0; i0 < n; i0 += WAVES * 64) {
        const int i = i0 + tid, r = i < n ? rep[i] : -1;
        const bool mine = r >= 0 && min(r, H - 1) == head;
        const unsigned long long votes = __ballot(mine);
        if (lane == 0) wave_slots[w] = __popcll(votes);
        __syncthreads();
        int at = n_slots;
#pragma unroll
        for (int v = 0; v < WAVES; ++v) {
            at += v < w ? wave_slots[v] : 0;
            n_slots += wave_slots[v];
        }
        if (mine) slots[at + __popcll(votes & ((1ull << lane) - 1ull))] = i;
        __syncthreads();
    }
    return n_slots;
}

// ---------------------------------------------------------------------------------------------------------
// One token, or a few of one request: the call is bound by reading the representatives' weights once.  One workgroup
// per (head, 16 output features), the 16 rows of a 16 x 16 x 32 MFMA tile: it looks up which (row, slot) pairs the head
// represents -- none: done -- and gathers their tokens as the tile's columns.  The contraction is dealt to the 8 waves
// in blocks of 64 elements (the workgroup walks 1 KB of every weight row per round), operands go from memory straight
// into the MFMA registers -- a weight element is used by one workgroup only, LDS would be a detour --, kJrBlocks
// blocks ahead, and the waves' fp32 sums are added in wave order.  grid (H * 16).
// ---------------------------------------------------------------------------------------------------------
constexpr int kJrWaves = 8, kJrBlocks = 4;
constexpr int kJrTokens = 8;                 // tokens of all rows up to which this kernel is the faster one
constexpr int kJrParts = kJCol / 16;                 // workgroups per head

typedef float f32x4 __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(kJrWaves * 64) void project_rows_kernel(const char *__restrict__ x,
                                                                     const char *__restrict__ w_q,
                                                                     const char *__restrict__ w_k,
                                                                     const int32_t *__restrict__ rep, int B, int H, int k,
                                                                     int Tn, int D, char *__restrict__ q_out,
                                                                     char *__restrict__ k_compact, int pos0, int Tc_cap)
{
    __shared__ int slots[kJrMaxSlots];
    __shared__ int wave_slots[kJrWaves];
    __shared__ f32x4 red[kJrWaves][64];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int head = blockIdx.x / kJrParts, f0 = blockIdx.x % kJrParts * 16;     // features 0..127 query, 128..255 key

    const int n_items = list_slots<kJrWaves>(rep, B * k, head, H, slots, wave_slots) * Tn;   // tokens of this head
    const size_t row_bytes = (size_t)D * 2;
    const int col = lane & 15, g = lane >> 4;        // operand row (weights) or token (activations), 8-element group
    const char *wsrc = (f0 < kHeadDim ? w_q : w_k) + ((size_t)head * kHeadDim + (f0 & (kHeadDim - 1)) + col) * row_bytes + g * 16;
    const int n_blk = D / 64;

    for (int c0 = 0; c0 < n_items; c0 += 16) {
        const int item = c0 + col, it = min(item, n_items - 1);      // columns past the end repeat the last token, unused
        const int sl = slots[it / Tn], tok = it % Tn;
        const char *xsrc = x + ((size_t)(sl / k) * Tn + tok) * row_bytes + g * 16;
        f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};

        // blocks w, w + 8, ... of 64 elements; a wave's surplus requests re-read the last block and are not used
        struct Block {
            Frag a[2], b[2];
        };
        auto request = [&](Block &bl, int blk) {
            const size_t at = (size_t)min(blk, n_blk - 1) * 128;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                bl.a[i].raw = *reinterpret_cast<const u32x4 *>(wsrc + at + i * 64);
                bl.b[i].raw = *reinterpret_cast<const u32x4 *>(xsrc + at + i * 64);
            }
        };
        Block bl[kJrBlocks];
#pragma unroll
        for (int u = 0; u < kJrBlocks; ++u) request(bl[u], w + u * kJrWaves);
        for (int b0 = w; b0 < n_blk; b0 += kJrBlocks * kJrWaves) {
#pragma unroll
            for (int u = 0; u < kJrBlocks; ++u) {
                if (b0 + u * kJrWaves < n_blk) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
                        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bl[u].a[i].bf, bl[u].b[i].bf, acc, 0, 0, 0);
                }
                request(bl[u], b0 + (u + kJrBlocks) * kJrWaves);
            }
        }
        red[w][lane] = acc;
        __syncthreads();
        // lane l holds features f0 + 4*(l/16) .. +3 of token l%16
        if (w == 0 && item < n_items) {
            f32x4 sum = red[0][lane];
#pragma unroll
            for (int i = 1; i < kJrWaves; ++i) sum += red[i][lane];
            char *orow = f0 < kHeadDim ? q_out + ((((size_t)(sl / k) * H + head) * Tn) + tok) * (kHeadDim * 2)
                                       : k_compact + ((size_t)sl * Tc_cap + pos0 + tok) * (kHeadDim * 2);
            bf16x4 o;
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (__bf16)sum[e];
            *reinterpret_cast<bf16x4 *>(orow + ((f0 & (kHeadDim - 1)) + g * 4) * 2) = o;
        }
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------------------------------------
// More tokens than one MFMA tile per head, too few to fill the chip with 256-token tiles: 64 tokens x 128 columns (the
// query or the key columns of one head) per workgroup, or 64 columns while that still gives every workgroup a CU of its
// own.  Head-major like the kernel above: rows that share a representative share its weights, and short blocks of
// several rows fill one tile.
//
// Which tiles exist depends on the maps: every workgroup counts the heads' tokens itself (B*k map entries) and takes
// the tile that its number stands for.  The 1-D grid is an upper bound, renumbered so that each XCD owns a contiguous
// range of the tiles that EXIST: equal shares, and the tiles of one head, which read the same weights, on one L2
// (numbered head by head without that, B 1 x 1024 tokens took 70 us, tile by tile 40 us, this way 32 us; B 4, D 9216,
// 128 tokens 115, 189 and 73 us).
//
// A tile is a chain of D/64 dependent stages.  Two teams of four waves take half of the contraction each, with a ring
// of three stages per team filled by direct loads to LDS two stages ahead; the second team's sums are added to the
// first's at the end.  What bounds a tile is the rate at which one CU takes its operands in (64 tokens x 64 columns at
// D = 4096, 1 MB: 14 us), which is why narrow tiles on more CUs win while there are CUs left.
// ---------------------------------------------------------------------------------------------------------
constexpr int kJtWaves = 4, kJtTeams = 2, kJtTok = 64, kJtStages = 3;
constexpr int kJtBlock = kJtWaves * kJtTeams * 64;
constexpr int kJtNarrow = 256;               // tiles are 64 columns wide while that gives at most so many (one per CU)
constexpr int kJtMaxHeads = 256;             // heads one workgroup can count
constexpr int jt_stage_bytes(int nb) { return (kJtTok + 64 * nb) * kJStep * 2; }
constexpr size_t kJtLdsBytes = (size_t)kJtTeams * kJtStages * jt_stage_bytes(2);

// One tile: tokens c0 .. c0+63 of the n_items tokens of `head` (listed in slots), columns f0 .. f0 + 64*NB - 1 of its
// 128 query (0..127) and 128 key (128..255) columns.
template <int NB>
__device__ __forceinline__ void project_tile(const char *__restrict__ x, const char *__restrict__ w_q,
                                             const char *__restrict__ w_k, int H, int k, int Tn, int D,
                                             char *__restrict__ q_out, char *__restrict__ k_compact, int pos0, int Tc_cap,
                                             char *lds, const int *slots, int head, int n_items, int c0, int f0)
{
    constexpr int kStageBytes = jt_stage_bytes(NB);
    constexpr int kLoads = kStageBytes / 1024 / kJtWaves;                // direct loads per wave and stage: 2 + 2*NB
    const int tid = threadIdx.x, lane = tid & 63, w8 = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = w8 / kJtWaves, w = w8 % kJtWaves;
    const int r = lane & 31, hl = lane >> 5;
    const int wm = w & 1, wn = w >> 1;               // the wave's 32 tokens and 32*NB columns of the tile

    const unsigned int row_bytes = (unsigned int)D * 2u;
    // staging: direct load i of wave w fills rows 8*(w + 4i) .. +7 of its team's stage (rows 0..63 tokens, then the
    // weight rows); lane l's 16 bytes land in slot l%8 of row l/8, and piece p of row R belongs in slot
    // p ^ ((R >> 1) & 7): 16 consecutive rows read at one piece index touch 16 different 16-byte bank groups.
    // Groups of eight token rows past the end are not loaded: what LDS holds there feeds accumulator columns that are
    // never written.
    unsigned int src[kLoads];
#pragma unroll
    for (int i = 0; i < kLoads; ++i) {
        const int row = 8 * (w + kJtWaves * i) + (lane >> 3), piece = (lane & 7) ^ ((row >> 1) & 7);
        unsigned int at;
        if (i < 2) {                                 // rows 0..63: tokens
            const int it = min(c0 + row, n_items - 1);
            const int sl = slots[it / Tn];
            at = (unsigned int)((sl / k) * Tn + it % Tn);
        } else {
            at = (unsigned int)(row - kJtTok);
        }
        src[i] = at * row_bytes + piece * 16;
    }
    const bool skip0 = c0 + 8 * w >= n_items, skip1 = c0 + 8 * (w + kJtWaves) >= n_items;     // skip0 implies skip1
    const int n_steps = D / kJStep, first = team * ((n_steps + 1) / 2);
    const int my_steps = team == 0 ? (n_steps + 1) / 2 : n_steps / 2;        // the second team may have one stage less
    char *const ring = lds + team * (kJtStages * kStageBytes);
#if defined(__HIP_DEVICE_COMPILE__)
    const auto x_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(x), 0, 0x7fffffff, 0x00020000);
    const auto w_rs = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<char *>((f0 < kHeadDim ? w_q : w_k) + ((size_t)head * kHeadDim + (f0 & (kHeadDim - 1))) * row_bytes), 0,
        0x7fffffff, 0x00020000);
    auto stage = [&](int s, int buf) {
#pragma unroll
        for (int i = 0; i < kLoads; ++i) {
            if ((i == 0 && skip0) || (i == 1 && skip1)) continue;
            __builtin_amdgcn_raw_ptr_buffer_load_lds(
                i < 2 ? x_rs : w_rs,
                (__attribute__((address_space(3))) void *)(ring + buf * kStageBytes + (w + kJtWaves * i) * 1024), 16,
                (int)(src[i] + (unsigned int)(first + s) * (kJStep * 2)), 0, 0, 0);
        }
    };
    // waits until at most the loads of ONE younger stage are in flight
    auto older_landed = [&]() {
        if (skip0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads - 2) : "memory");
        else if (skip1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads - 1) : "memory");
        else asm volatile("s_waitcnt vmcnt(%0)" ::"n"(kLoads) : "memory");
    };
#else
    auto stage = [&](int, int) {};
    (void)skip0, (void)skip1, (void)first;
#endif
    f32x16 acc[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[nb][e] = 0.f;

    const int sw = (r >> 1) & 7;                     // fragments start on multiples of 16 rows
    if (my_steps > 0) stage(0, 0);
    if (my_steps > 1) stage(1, 1);
    int buf = 0;
    for (int s = 0; s < (n_steps + 1) / 2; ++s) {    // both teams: the same number of barriers
#if defined(__HIP_DEVICE_COMPILE__)
        // this wave's loads of stage s have landed (those of stage s + 1 may still be in flight), then everyone's have;
        // the barrier also frees the buffer that stage s - 1 was read from
        if (s + 1 < my_steps) older_landed();
        else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
#endif
        if (s + 2 < my_steps) stage(s + 2, buf == 0 ? 2 : buf - 1);          // buffer (s + 2) % 3
        if (s < my_steps) {
            const char *base = ring + buf * kStageBytes;
#pragma unroll
            for (int ks = 0; ks < kJStep / 16; ++ks) {
                const int piece = ((2 * ks + hl) ^ sw) << 4;
                Frag a[NB], b;
                b.raw = *reinterpret_cast<const u32x4 *>(base + (wm * 32 + r) * 128 + piece);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    a[nb].raw = *reinterpret_cast<const u32x4 *>(base + (kJtTok + wn * 32 * NB + nb * 32 + r) * 128 + piece);
#pragma unroll
                for (int nb = 0; nb < NB; ++nb)
                    acc[nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[nb].bf, b.bf, acc[nb], 0, 0, 0);
            }
        }
        buf = buf == 2 ? 0 : buf + 1;
    }
    // the second team's sums through the rings (no loads are in flight any more)
    __syncthreads();
    f32x4 *const other = reinterpret_cast<f32x4 *>(lds) + w * (NB * 4 * 64) + lane;
    if (team == 1) {
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4)
                other[(nb * 4 + v4) * 64] =
                    f32x4{acc[nb][v4 * 4], acc[nb][v4 * 4 + 1], acc[nb][v4 * 4 + 2], acc[nb][v4 * 4 + 3]};
    }
    __syncthreads();
    const int it = c0 + wm * 32 + r;
    if (team == 0 && it < n_items) {
        const int sl = slots[it / Tn], tok = it % Tn;
        char *orow = f0 < kHeadDim ? q_out + ((((size_t)(sl / k) * H + head) * Tn) + tok) * (kHeadDim * 2)
                                   : k_compact + ((size_t)sl * Tc_cap + pos0 + tok) * (kHeadDim * 2);
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
                const f32x4 add = other[(nb * 4 + v4) * 64];
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)(acc[nb][v4 * 4 + e] + add[e]);
                *reinterpret_cast<bf16x4 *>(orow + ((f0 & (kHeadDim - 1)) + wn * 32 * NB + nb * 32 + v4 * 8 + hl * 4) * 2) = o;
            }
    }
}

__global__ __launch_bounds__(kJtBlock) void project_tile_kernel(const char *__restrict__ x, const char *__restrict__ w_q,
                                                                const char *__restrict__ w_k,
                                                                const int32_t *__restrict__ rep, int B, int H, int k,
                                                                int Tn, int D, char *__restrict__ q_out,
                                                                char *__restrict__ k_compact, int pos0, int Tc_cap)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    __shared__ int slots[kJrMaxSlots];
    __shared__ int wave_sum[kJtWaves * kJtTeams];
    __shared__ int count[kJtMaxHeads];
    __shared__ int mine[2];
    const int tid = threadIdx.x, lane = tid & 63, w8 = tid >> 6;

    // tiles of every head, their running sum, and the one this workgroup stands for
    for (int h = tid; h < H; h += kJtBlock) count[h] = 0;
    __syncthreads();
    for (int i = tid; i < B * k; i += kJtBlock) {
        const int rh = rep[i];
        if (rh >= 0) atomicAdd(&count[min(rh, H - 1)], 1);
    }
    __syncthreads();
    const int n_tiles = tid < H ? (count[tid] * Tn + kJtTok - 1) / kJtTok : 0;
    int upto = n_tiles;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int other = __shfl_up(upto, o);
        upto += lane >= o ? other : 0;
    }
    if (lane == 63) wave_sum[w8] = upto;
    __syncthreads();
    int before = 0, total = 0;
#pragma unroll
    for (int v = 0; v < kJtWaves * kJtTeams; ++v) {
        before += v < w8 ? wave_sum[v] : 0;
        total += wave_sum[v];
    }
    const int parts = 4 * total <= kJtNarrow ? 4 : 2;
    const int items = parts * total, per_xcd = (items + 7) / 8;
    const int local = (int)(blockIdx.x >> 3), item = (int)(blockIdx.x & 7) * per_xcd + local;
    if (local >= per_xcd || item >= items) return;               // the same decision in every thread
    const int at = item / parts - before - (upto - n_tiles);     // tile number inside this thread's head
    if (at >= 0 && at < n_tiles) {
        mine[0] = tid;
        mine[1] = at;
    }
    __syncthreads();
    const int head = mine[0], c0 = mine[1] * kJtTok;
    const int n_items = list_slots<kJtWaves * kJtTeams>(rep, B * k, head, H, slots, wave_sum) * Tn;
    if (parts == 4)
        project_tile<1>(x, w_q, w_k, H, k, Tn, D, q_out, k_compact, pos0, Tc_cap, lds, slots, head, n_items, c0, item % 4 * 64);
    else
        project_tile<2>(x, w_q, w_k, H, k, Tn, D, q_out, k_compact, pos0, Tc_cap, lds, slots, head, n_items, c0, item % 2 * 128);
}

// Measurement aid: the matrix pipe alone.  Every wave (two per SIMD on every CU) loads six operand fragments from
// `buf` once and then issues rounds of eight independent v_mfma_f32_32x32x16_bf16 with nothing else in the loop.
// The rate depends on the operand VALUES (switching activity moves the clocks), hence operands from the caller's
// data rather than constants.
constexpr int kProbeBlocks = 512, kProbeMfmaPerRound = 8;
__global__ __launch_bounds__(kJBlock) void mfma_probe_kernel(const u32x4 *__restrict__ buf, unsigned long long n_pieces,
                                                             int rounds, float *__restrict__ sink)
{
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    Frag a[2], b[4];
#pragma unroll
    for (int i = 0; i < 6; ++i) {
        const unsigned long long at = (((unsigned long long)blockIdx.x * 8 + w) * 6 + i) * 64 + lane;
        (i < 2 ? a[i] : b[i - 2]).raw = buf[at % n_pieces];
    }
    f32x16 acc[kProbeMfmaPerRound];
#pragma unroll
    for (int i = 0; i < kProbeMfmaPerRound; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[i][e] = 0.f;
    for (int it = 0; it < rounds; ++it) {
#pragma unroll
        for (int i = 0; i < kProbeMfmaPerRound; ++i)
            acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i & 1].bf, b[i >> 1].bf, acc[i], 0, 0, 0);
    }
    float t = 0.f;
#pragma unroll
    for (int i = 0; i < kProbeMfmaPerRound; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e) t += acc[i][e];
    if (t == 123.456f) sink[0] = t;              // practically never true: keeps the MFMAs alive
}

}  // namespace

double mfma_probe_flops(int rounds)
{
    return (double)kProbeBlocks * (kJBlock / 64) * (double)rounds * kProbeMfmaPerRound * (2.0 * 32 * 32 * 16);
}

int launch_mfma_probe(const void *buf, size_t bytes, int rounds, float *sink, const KernelEvents &ev, hipStream_t stream)
{
    return (int)launch_kernel(mfma_probe_kernel, dim3(kProbeBlocks), dim3(kJBlock), 0, stream, ev,
                              static_cast<const u32x4 *>(buf), (unsigned long long)(bytes / 16), rounds, sink);
}

int launch_project_qk(const void *x, const void *w_q, const void *w_k, const int32_t *rep, int B, int H, int k, int Tn,
                      int D, void *q_out, void *k_compact, int pos0, int Tc_cap, const KernelEvents &ev,
                      hipStream_t stream)
{
    const char *xc = static_cast<const char *>(x), *wq = static_cast<const char *>(w_q), *wk = static_cast<const char *>(w_k);
    char *qo = static_cast<char *>(q_out), *ko = static_cast<char *>(k_compact);
    // Which kernel: by the number of tokens over all (row, slot) pairs, in time per call (before: 256-token tiles for
    // every size; D = 4096 unless noted).  A 256-token tile of one (row, slot) pair is a chain of D/64 stages however
    // few tokens it holds, so calls with few tokens took 77-86 us (170-215 us at D = 9216) at any size:
    //   B*Tn <= 8           one row of MFMA columns per head: B 1, 8 of 32 heads: 77 -> 13 us; B 1, 16 of 72, D 9216:
    //                       171 -> 28 us (33 us with the 64-token tiles)
    //   B*k*Tn <= most      64-token tiles, head-major: B 16, k 8, Tn 1 / 16 / 64 / 128: 80 / 82 / 82 / 85 -> 17 / 20 / 32 /
    //                       62 us; B 1, k 8, Tn 512 / 2043: 85 / 87 -> 21 / 60 us; B 4, k 16, D 9216, Tn 16 / 256:
    //                       175 / 215 -> 52 / 135 us; B 4, k 8, D 6656, Tn 512: 151 -> 95 us
    //   above               256-token tiles: B 16, k 8, Tn 256: 98 us (118 us with the small tiles)
    // From 16384 pairs' tokens on the small tiles take a third round of the chip.  It pays where the large tiles need a second
    // one, or are a long chain and do not fill theirs, or hold few tokens each; in us, large / small tiles:
    //   B 16, k 8 (128 large tiles), Tn 144, 160 and 192: D 4096 85 / 80, 88 / 82 and 88 / 84, D 3072 66 / 65 and (192) 68 / 68,
    //   D 2048 47.2 / 47.7, 47.8 / 48.0 and 49.1 / 50.6, D 1024 28 / 31 and (192) 30 / 33, D 512 19 / 24 and (192) 21 / 25
    //   B 1, k 8, Tn 2304 and 3072: D 2048 49.9 / 48.3 and 50.8 / 51.3
    //   B 16, k 10 (160), Tn 140, D 5120: 118 / 111
    //   B 16, k 16 (256), Tn 72 / 80 / 96: D 4096 100 / 82 and (96) 104 / 108, D 9216 238 / 195, 238 / 196 and 238 / 246
    //   B 16, k 32 (512), Tn 48: D 512 37 / 27, D 4096 202 / 90
    // Both small kernels list the pairs of a head in LDS (at most kJrMaxSlots of them).
    const long long items = (long long)B * k * Tn;
    const bool listed = (long long)B * k <= kJrMaxSlots;
    if (listed && (long long)B * Tn <= kJrTokens && H <= 0x7fffffff / kJrParts)
        return (int)launch_kernel(project_rows_kernel, dim3((unsigned int)H * kJrParts), dim3(kJrWaves * 64), 0, stream, ev,
                                  xc, wq, wk, rep, B, H, k, Tn, D, qo, ko, pos0, Tc_cap);
    // (the tile kernel addresses the activations and one head's weights with 32-bit byte offsets below 2 GiB)
    const long long n_large = (long long)B * k * ((Tn + kJTok - 1) / kJTok);
    const long long most = n_large > 256 ? 24576 : (D < 2048 ? 16384 : (D < 3072 || n_large > 200 ? 20480 : 24576));
    if (listed && items <= most && H <= kJtMaxHeads && (long long)B * Tn * D * 2 < 0x7fffffffLL &&
        (long long)kHeadDim * D * 2 < 0x7fffffffLL) {
        static DeviceFlags tile_lds_allowed;
        const hipError_t attr = allow_dynamic_lds(reinterpret_cast<const void *>(&project_tile_kernel), kJtLdsBytes,
                                                  tile_lds_allowed);
        if (attr != hipSuccess) return (int)attr;
        // an upper bound of the tiles: the heads' tokens rounded up to whole tiles
        const long long tiles = items / kJtTok + (H < B * k ? H : B * k);
        long long n_wg = 2 * tiles;
        if (n_wg < kJtNarrow) n_wg = 4 * tiles < kJtNarrow ? 4 * tiles : kJtNarrow;
        return (int)launch_kernel(project_tile_kernel, dim3((unsigned int)((n_wg + 7) / 8 * 8)), dim3(kJtBlock), kJtLdsBytes,
                                  stream, ev, xc, wq, wk, rep, B, H, k, Tn, D, qo, ko, pos0, Tc_cap);
    }
    static DeviceFlags lds_allowed;
    const hipError_t attr = allow_dynamic_lds(reinterpret_cast<const void *>(&project_kernel), kJLdsBytes, lds_allowed);
    if (attr != hipSuccess) return (int)attr;
    const int n_mt = (Tn + kJTok - 1) / kJTok;
    if ((long long)n_mt * k * B > 0x7fffffffLL) return (int)hipErrorInvalidConfiguration;
    return (int)launch_kernel(project_kernel, dim3((unsigned int)n_mt * k * B), dim3(kJBlock), kJLdsBytes, stream, ev, xc,
                              wq, wk, rep, H, k, Tn, D, n_mt, qo, ko, pos0, Tc_cap);
}

}  // namespace chai
