// Query / key projections of the representative heads only (Fig. 3, Section 3.5: clustered attention needs the
// query and key vectors of one head per cluster, so the columns of W_Q and W_K that belong to the other heads are
// never multiplied; the new keys go straight into the pruned K cache).  A dense contraction with reuse on both
// operands, so it runs on the matrix cores.
//
//   for batch row b, slot j, r = rep_heads[b][j] >= 0, token i < Tn:
//       q_out[b][r][i][:]            = bf16( x[b][i][:] . w_q[r*128 .. r*128+127][:]^T )
//       k_compact[b][j][pos0 + i][:] = bf16( x[b][i][:] . w_k[r*128 .. r*128+127][:]^T )
//
// Three kernels, chosen in launch_project_qk by the number of tokens; the first below is the one for prompts.  In all of them
// the product is formed transposed, C^T = W X^T: both operands are then read along the contraction axis (weights are stored
// one row per output feature), a lane owns one token and gets 4 consecutive output features per register quad; fp32
// accumulation, one rounding to bf16 at the end.
#include "chai_internal.h"

#include <hip/hip_ext.h>

#include <algorithm>
#include <cmath>
#include <iterator>
#include <type_traits>
#include <utility>

namespace chai {

namespace {

constexpr int kJBlock = 256;                 // threads (4 waves, one per SIMD: 2 along the tokens x 2 along the columns)
constexpr int kJTok = 256;                   // tokens per workgroup tile
constexpr int kJCol = 2 * kHeadDim;          // columns per workgroup tile: query + key columns of one head
constexpr int kJStep = 64;                   // contraction elements per stage; widths are multiples of it
constexpr int kJStageBytes = (kJTok + kJCol) * kJStep * 2;                 // 64 KB: activations, then weights; rows of 128 B
constexpr int kJLoads = kJStageBytes / 1024 / (kJBlock / 64);              // direct loads per wave and stage (16)
constexpr int kJOutBytes = 32 * kHeadDim * 2;                              // output staging of one wave: 32 tokens
constexpr size_t kJLdsBytes = 2 * (size_t)kJStageBytes + kJBlock / 64 * kJOutBytes;          // all 160 KB of a CU
constexpr int kJCus = 256;                   // workgroups of the large tiles: one per CU

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

union Frag {
    u32x4 raw;
    bf16x8 bf;
};

// f(integral_constant 0), f(1), .. f(N - 1)
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

// ---------------------------------------------------------------------------------------------------------
// Prompts.  A tile is 256 tokens x 256 columns, the 128 query and the 128 key columns of one representative, which share the
// activations.  Four waves, one per SIMD, own 128 x 128 of it each (all 256 accumulation registers): 16 products of 16 x 16 x 32
// per LDS fragment pair, half of the LDS reads that eight waves of 64 x 128 need.  Stages of 64 contraction steps, 64 KB, are
// loaded straight into LDS, two of them; a wave reads the fragments of one half of a stage while it multiplies the other, so
// that ONE barrier per stage, in its middle, frees the stage that has been read and hands over the one that has arrived.
//
// What bounds it: power.  With every CU multiplying N(0,1) data the chip runs at 1.6 to 1.8 GHz instead of 2.4, so that time is
// energy.  Measured on operands of this kind with nothing but products: 32 x 32 x 16 tiles 1790 TFLOP/s, 16 x 16 x 32 ones, which
// touch the accumulators half as often, 2060.  16 rows x 2043 tokens, 8 of 32 heads, D = 4096 (1024 tiles), per call:
//   eight waves of 64 x 128, 32 x 32 x 16, staged through registers            490 us
//   four waves of 128 x 128, loads straight to LDS, a workgroup per tile       477 (1.60 GHz, 172 000 cycles per tile of 131 000)
//   one workgroup per CU, the next tile loaded during the end of one, whole output rows stored (8-byte pieces took 22 000 cycles per
//   tile, rows through LDS take 7000)                                          460
//   16 x 16 x 32                                                               436
//   stages of 64 steps in cache lines of 128 bytes instead of 32 in half lines 415 (1.78 GHz; 350 if all loads hit L2, 312 without)
// and no difference: the order of the products, a fifth stage of 32.  Slower: the loads of a stage closer together (432, 457).
// All 256 ordinary registers are taken as well, and 39 more are kept in scratch (80 bytes per lane), where a tile ends and the next
// one's addresses are made; within a tile nothing is.
//
// One workgroup per CU takes several (batch row, token tile, slot) items one after the other.  Items are numbered slot first and
// dealt to the XCDs in contiguous ranges: the slots of a token tile read the same activations and find them in L2.
// ---------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kJBlock, 1) void project_kernel(const char *__restrict__ x, const char *__restrict__ w_q,
                                                             const char *__restrict__ w_k,
                                                             const int32_t *__restrict__ rep, int H, int k, int Tn, int D,
                                                             int n_mt, unsigned n_items, char *__restrict__ q_out,
                                                             char *__restrict__ k_compact, int pos0, int Tc_cap)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int r = lane & 15, g = lane >> 4;
    const int wm = w & 1, wn = w >> 1;               // wave's 128-token half, and query (0) or key (1) columns

    struct Item {
        int b, j, t0, head;
    };
    const unsigned xcd = blockIdx.x & 7u, each = n_items >> 3, rest = n_items & 7u;
    const unsigned hi = each * (xcd + 1) + min(xcd + 1, rest);
    // The items of this workgroup.  Only those whose slot is in use are numbered: with as many slots per row as workgroups per XCD, or
    // a divisor of it, a workgroup that went by the numbers of all would always meet the same slot, and the unused ones' workgroups
    // would stand idle (16 rows x 2043 tokens, 8 slots of 32 in use 1378 -> 442 us, level where all are).
    unsigned at = each * xcd + min(xcd, rest), next = at;    // the 64 items looked up last (those in use: `used`), and the next ones
    unsigned before = 0, mine = blockIdx.x >> 3;     // items in use before those; number of the one this workgroup takes next
    unsigned long long used = 0ull;
    auto next_item = [&](Item &it) __attribute__((always_inline)) {      // false: there is none
        unsigned slots = (unsigned)k, tiles = (unsigned)n_mt;
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+s"(slots), "+s"(tiles)); // what dividing by them takes is made here, not kept in registers all the time
#endif
        for (;;) {
            const unsigned n = (unsigned)__popcll(used);
            if (mine < before + n) break;
            before += n;
            used = 0ull;
            at = next;
            if (at >= hi) return false;
            next = at + 64;
            const unsigned item = min(at + lane, hi - 1), bm = item / slots;
            const int head = rep[(size_t)(bm / tiles) * k + (item - bm * slots)];
            used = __ballot(at + lane < hi && head >= 0);
        }
        unsigned long long left = used;
        for (unsigned i = before; i < mine; ++i) left &= left - 1ull;
        mine += gridDim.x >> 3;
        const unsigned item = at + (unsigned)__ffsll((long long)left) - 1u, bm = item / slots;
        it.j = (int)(item - bm * slots);
        it.b = (int)(bm / tiles);
        it.t0 = (int)(bm - (unsigned)it.b * tiles) * kJTok;
        it.head = min(rep[(size_t)it.b * k + it.j], H - 1);
        return true;
    };

    // staging: direct load i of wave w fills rows 8*(w + 4i) .. +7 of a stage (rows 0..255 tokens, 256..383 query and
    // 384..511 key rows of the weights); lane l's 16 bytes land in slot l%8 of row l/8, and piece p of row R belongs in
    // slot p ^ ((R >> 1) & 7): 16 consecutive rows read at one piece index touch 16 different 16-byte bank groups.
    const size_t row_bytes = (size_t)D * 2;
    auto piece16 = [&](int l) { return (unsigned)((l & 7) ^ ((l >> 4) + 4 * (w & 1))) * 16; };
    auto srow = [&](int l) { return 8 * w + (l >> 3); };
    unsigned xoff[8], woff[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) woff[i] = (unsigned)(srow(lane) + 32 * i) * (unsigned)row_bytes + piece16(lane);
    const char *xb = nullptr, *wqb = nullptr, *wkb = nullptr;
    auto load_from = [&](const Item &it) __attribute__((always_inline)) {
        int l = lane;
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+v"(l));                  // made here, too
#endif
#pragma unroll
        for (int i = 0; i < 8; ++i) xoff[i] = (unsigned)min(srow(l) + 32 * i, Tn - 1 - it.t0) * (unsigned)row_bytes + piece16(l);
        xb = x + ((size_t)it.b * Tn + it.t0) * row_bytes;
        wqb = w_q + (size_t)it.head * kHeadDim * row_bytes;
        wkb = w_k + (size_t)it.head * kHeadDim * row_bytes;
    };
#if defined(__HIP_DEVICE_COMPILE__)
    auto load = [&](int s, int buf_off, auto ic) {
        constexpr int i = decltype(ic)::value;
        const char *base = i < 8 ? xb : (i < 12 ? wqb : wkb);
        const auto rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(base), 0, -1, 0x00020000);
        auto *dst = (__attribute__((address_space(3))) void *)(lds + buf_off + (w + 4 * i) * 1024);
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, dst, 16, (int)(i < 8 ? xoff[i & 7] : woff[i & 3]), s * (kJStep * 2), 0, 0);
    };
    // every wave's loads but the youngest N have landed, and every wave has read what it reads before this point
    auto landed = [&](auto n) {
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(decltype(n)::value) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
    };
#else
    auto load = [&](int, int, auto) {};
    auto landed = [&](auto) {};
    (void)xb, (void)wqb, (void)wkb, (void)xoff, (void)woff;
#endif

    // fragments: 16 rows x 32 contraction elements (half a stage), lane's row r, 8 elements at 8*g.  Fragment i: 0 the first
    // 16 weight rows, 1 .. 8 the token rows, 9 .. 15 the other weight rows, which is the order the products need them in.
    const int sw = (r >> 1) & 7;
    const int a_row = (kJTok + wn * kHeadDim + r) * (kJStep * 2), b_row = (wm * 128 + r) * (kJStep * 2);
    const int piece[2] = {(g ^ sw) << 4, ((4 + g) ^ sw) << 4};
    Frag fa[2][8], fb[2][8];
    auto read = [&](auto half, auto ic, const char *base) {
        constexpr int i = decltype(ic)::value, h = decltype(half)::value, nb = i == 0 ? 0 : i - 8, tb = i - 1;
        if constexpr (i >= 1 && i <= 8) fb[h][tb].raw = *reinterpret_cast<const u32x4 *>(base + piece[h] + b_row + tb * 16 * (kJStep * 2));
        else fa[h][nb].raw = *reinterpret_cast<const u32x4 *>(base + piece[h] + a_row + nb * 16 * (kJStep * 2));
    };
    constexpr std::integral_constant<int, 0> lower{};
    constexpr std::integral_constant<int, 1> upper{};

    Item now, then;
    if (!next_item(now)) return;
    bool more = true;                                // `then`, whose stages are loaded behind those of `now`, exists
    const int n_steps = D / kJStep;
    load_from(now);
    int ls = 0;                                      // the stage to load next (of `now`, or of `then`)
    auto advance = [&]() __attribute__((always_inline)) {
        if (__builtin_expect(ls == n_steps, 0)) {
            more = next_item(then);
            if (more) load_from(then);
            ls = more ? 0 : n_steps - 1;             // past the last item: requested, not read
        }
    };
    for (int i = 0; i < 2; ++i) {
        advance();
        unroll<kJLoads>([&](auto ic) { load(ls, i * kJStageBytes, ic); });
        ++ls;
    }
    landed(std::integral_constant<int, kJLoads>{});
    unroll<16>([&](auto i) { read(lower, i, lds); });
    int cur = 0;                                     // byte offset of the present stage
    for (;;) {
        f32x4 acc[8][8];                             // [column block of 16][token block of 16]
        // Half a stage: 64 products, and between them 16 reads for the next half and, where the stage has been read, the loads
        // of the one after the next into its place.
        auto half = [&](auto hc, auto first) {
            constexpr int h = decltype(hc)::value;
            unroll<64>([&](auto nc) {
                constexpr int n = decltype(nc)::value, nb = n >> 3, tb = (nb & 1) ? 7 - (n & 7) : n & 7;
                const f32x4 c = decltype(first)::value ? f32x4{0.f, 0.f, 0.f, 0.f} : acc[nb][tb];
                acc[nb][tb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fa[h][nb].bf, fb[h][tb].bf, c, 0, 0, 0);
                if constexpr (n % 3 == 0 && n < 48)
                    read(std::integral_constant<int, 1 - h>{}, std::integral_constant<int, n / 3>{}, lds + (h == 0 ? cur : cur ^ kJStageBytes));
                if constexpr (h == 1 && n % 4 == 2) load(ls, cur, std::integral_constant<int, n / 4>{});
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        auto stage = [&](auto first) {
            half(lower, first);
            advance();
            landed(std::integral_constant<int, 0>{});
            half(upper, std::false_type{});
            ++ls;
            cur ^= kJStageBytes;
        };
        stage(std::true_type{});
        for (int s = 1; s < n_steps; ++s) stage(std::false_type{});

        // D[4*g + v][r]: this lane's token is t0 + wm*128 + tb*16 + r, its features nb*16 + 4*g .. +3.
        // 32 tokens at a time through LDS (piece p of token row R in slot p ^ (R & 15)), so that whole rows are stored.
        char *const strip = lds + 2 * kJStageBytes + w * kJOutBytes;
        const int left = Tn - now.t0 - wm * 128;             // tokens from this wave's first one on
        char *const rows = (wn == 0 ? q_out + (((size_t)now.b * H + now.head) * (size_t)Tn) * (kHeadDim * 2)
                                    : k_compact + (((size_t)now.b * k + now.j) * (size_t)Tc_cap + pos0) * (kHeadDim * 2)) +
                           (size_t)(now.t0 + wm * 128) * (kHeadDim * 2);
        int l = lane;
#if defined(__HIP_DEVICE_COMPILE__)
        asm volatile("" : "+v"(l));                  // addresses are made here, not kept in registers all the time
#endif
        const int wr = l & 15, wp = l >> 5, wh = (l >> 4 & 1) * 8, rd = l >> 4, rp = l & 15;
        unroll<4>([&](auto tc) {
#pragma unroll
            for (int t2 = 0; t2 < 2; ++t2)
#pragma unroll
                for (int nb = 0; nb < 8; ++nb) {
                    const f32x4 &d = acc[nb][2 * decltype(tc)::value + t2];
                    bf16x4 o;
#pragma unroll
                    for (int e = 0; e < 4; ++e) o[e] = (__bf16)d[e];
                    *reinterpret_cast<bf16x4 *>(strip + (t2 * 16 + wr) * (kHeadDim * 2) + (((nb * 2 + wp) ^ wr) << 4) + wh) = o;
                }
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_sched_barrier(0);
            u32x4 o[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = 4 * i + rd;
                o[i] = *reinterpret_cast<const u32x4 *>(strip + row * (kHeadDim * 2) + ((rp ^ (row & 15)) << 4));
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int row = decltype(tc)::value * 32 + 4 * i + rd;
                if (row < left) *reinterpret_cast<u32x4 *>(rows + (unsigned)(row * (kHeadDim * 2) + rp * 16)) = o[i];
            }
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_sched_barrier(0);
        });
        if (!more) break;
        now = then;
    }
#if defined(__HIP_DEVICE_COMPILE__)
    // the requests past the end have landed before LDS is given to another workgroup
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#endif
}

// The (row, slot) pairs that `head` represents, as indexes into rep, ascending: all workgroups of a head agree which
// tokens belong to which chunk.  Returns their number; B*k <= kJtMaxSlots.  Every thread of the workgroup calls it.
constexpr int kJtMaxSlots = 1024;
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
// At most eight tokens, where the streamed weights (below) do not pay: narrow products, and more heads than they have rounds
// for.  The call is bound by reading the representatives' weights once, or by its launch.  One workgroup
// per (head, 16 output features), the 16 rows of a 16 x 16 x 32 MFMA tile: it looks up which (row, slot) pairs the head
// represents -- none: done -- and gathers their tokens as the tile's columns.  The contraction is dealt to the 8 waves
// in blocks of 64 elements (the workgroup walks 1 KB of every weight row per round), operands go from memory straight
// into the MFMA registers -- a weight element is used by one workgroup only, LDS would be a detour --, kJrBlocks
// blocks ahead, and the waves' fp32 sums are added in wave order.  grid (H * 16).  1 row x 1 token, 1000 of 1000 heads, D = 512 295 us (streamed 660), 256
// of 256, D = 64 19.5 us (34.3).
// ---------------------------------------------------------------------------------------------------------
constexpr int kJrWaves = 8, kJrBlocks = 4;
constexpr int kJrTokens = 8;                 // tokens of all rows up to which this kernel is faster than 64-token tiles
constexpr int kJrParts = kJCol / 16;                 // workgroups per head

__global__ __launch_bounds__(kJrWaves * 64) void project_rows_kernel(const char *__restrict__ x,
                                                                     const char *__restrict__ w_q,
                                                                     const char *__restrict__ w_k,
                                                                     const int32_t *__restrict__ rep, int B, int H, int k,
                                                                     int Tn, int D, char *__restrict__ q_out,
                                                                     char *__restrict__ k_compact, int pos0, int Tc_cap)
{
    __shared__ int slots[kJtMaxSlots];
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
// A few tokens per head (the new tokens of a batch, a short block of one request): the call is bound by reading the
// representatives' weights once.  The 256 query and key columns of every head in use are cut into equal parts of 8 to 64 columns,
// as many as fill the CUs evenly (a unit of 8 weight rows is one direct load to LDS: eight lines of 128 bytes), so that 8 heads in
// use keep the chip as busy as 32.  Which heads those are, which part of which one it takes and where its tokens stand every wave
// finds out for itself: there is no barrier before the sums.  The contraction is dealt to the 8 waves in blocks of 64 elements;
// a wave streams its blocks of weights and of up to 32 tokens through a ring of its own in LDS and multiplies what has landed.  The
// waves' fp32 sums are added in wave order.
//
// What bounds it: launch, map look-up and ramp (5 to 6 us together: 8 heads of width 1024 take 6 us), then HBM.  Against the kernels
// before (at most 8 tokens: 16 weight rows per workgroup, fragments straight from memory, each of whose loads touched 16 half
// lines; more: 64 x 64 or 64 x 128 tiles of two teams of waves with a barrier per stage, which leave half of the CUs without work
// where 32 heads are in use), weights not in any cache: 16 rows x 1 token, 8 of 32 heads, D = 4096 20.1 -> 14.1 us (16.2 -> 11.3
// with weights that the memory-side cache holds); 1 x 1 12.0 -> 7.3; 1 x 32 18.6 -> 10.1; 16 x 4 24.4 -> 20.9; 2 x 1, 16 of 72, D = 9216
// 30.7 -> 23.0; 4 x 1 41.8 -> 30.4; 16 x 1, 8 of 52, D = 6656 29.0 -> 20.9.  Found on the way: fragments of the weights straight from
// memory, whole parts of 32 columns 17.2 us for the first of these; parts of 32 columns whatever is in use 13.2 there, but 14.0
// for 3 x 1, 8 of 52 (12.4) and 37.8 for 4 x 1, 16 of 72 (30.4).
// ---------------------------------------------------------------------------------------------------------
constexpr int kJsWaves = 8, kJsUnits = kJCol / 8, kJsFewUnits = 4, kJsMaxUnits = 8;      // units of a head, and most of a workgroup
constexpr int kJsWaveBytes = 20 * 1024;      // ring of a wave: two blocks at least
constexpr int kJsPass = 32;                  // the most tokens that are multiplied at a time
// ... with so many units: more than 16 leave room in the rings for six
constexpr int js_pass(int units) { return units <= kJsMaxUnits - 2 ? kJsPass : 16; }
constexpr size_t kJsLdsBytes = (size_t)kJsWaves * kJsWaveBytes;

// or over the wave, in every lane
__device__ __forceinline__ unsigned wave_or(unsigned x)
{
    unsigned z = x;
    z |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)z, 0x111, 0xf, 0xf, true);       // row_shr 1, 2, 4, 8
    z |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)z, 0x112, 0xf, 0xf, true);
    z |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)z, 0x114, 0xf, 0xf, true);
    z |= (unsigned)__builtin_amdgcn_update_dpp(0, (int)z, 0x118, 0xf, 0xf, true);       // lane 15 of a row has the row's
    return (unsigned)(__builtin_amdgcn_readlane((int)z, 15) | __builtin_amdgcn_readlane((int)z, 31) |
                      __builtin_amdgcn_readlane((int)z, 47) | __builtin_amdgcn_readlane((int)z, 63));
}

template <int MOST>
__global__ __launch_bounds__(kJsWaves * 64) void project_stream_kernel(const char *__restrict__ x, const char *__restrict__ w_q,
                                                                       const char *__restrict__ w_k,
                                                                       const int32_t *__restrict__ rep, int B, int H, int k,
                                                                       int Tn, int D, char *__restrict__ q_out,
                                                                       char *__restrict__ k_compact, int pos0, int Tc_cap)
{
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n_pairs = B * k, n_windows = (H + 63) / 64;

    // The first map entries are requested before anything else.
    constexpr int kAhead = MOST;
    int first[kAhead];
#pragma unroll
    for (int u = 0; u < kAhead; ++u) first[u] = u * 64 + lane < n_pairs ? rep[u * 64 + lane] : -1;
    auto each_pair = [&](auto f) __attribute__((always_inline)) {    // f(pair, its head or less than 0), 64 pairs at a time
#pragma unroll
        for (int u = 0; u < kAhead; ++u)
            if (u * 64 < n_pairs) f(u * 64 + lane, min(first[u], H - 1));
        for (int i0 = kAhead * 64; i0 < n_pairs; i0 += 64) f(i0 + lane, i0 + lane < n_pairs ? min(rep[i0 + lane], H - 1) : -1);
    };
    auto window = [&](int i) __attribute__((always_inline)) {        // which of the heads 64 i .. 64 i + 63 are in use
        unsigned lo = 0u, hi = 0u;
        each_pair([&](int, int r) {
            const unsigned bit = (r >> 6) == i ? 1u << (r & 31) : 0u;
            lo |= (r & 32) ? 0u : bit;
            hi |= (r & 32) ? bit : 0u;
        });
        return (unsigned long long)wave_or(hi) << 32 | wave_or(lo);
    };
    unsigned use_lo = 0u, use_hi = 0u;               // lane i: window i
    int used = 0;
    for (int i = 0; i < n_windows; ++i) {
        const unsigned long long heads = window(i);
        used += __popcll(heads);
        use_lo = lane == i ? (unsigned)heads : use_lo;
        use_hi = lane == i ? (unsigned)(heads >> 32) : use_hi;
    }
    // Units of a workgroup: as many as make (rounds of the chip) * (units + what a workgroup costs besides) least; none that would
    // take two passes for the tokens of a head that stands once in every row.  (One that stands in several slots of a row has more.)
    int units = 1;
    unsigned long long least = ~0ull;
    int parts = kJsUnits;
    const int most = B * Tn <= js_pass(MOST) ? MOST : min(MOST, kJsMaxUnits - 2);
    unroll<MOST>([&](auto i) {
        constexpr int u = i.value + 1, p = (kJsUnits + u - 1) / u;
        const unsigned long long cost = (unsigned long long)((used * p + kJCus - 1) / kJCus) * (unsigned)(u * D + 4096);
        if (u <= most && used * p <= (int)gridDim.x && cost < least) {
            least = cost;
            units = u;
            parts = p;
        }
    });
    const int rank = (int)blockIdx.x / parts, part = (int)blockIdx.x - rank * parts;
    if (rank >= used) return;                        // (all waves alike)
    int head = 0;
    for (int i = 0, before = 0; i < n_windows; ++i) {
        unsigned long long heads = i >= 64 ? window(i)
                                           : (unsigned long long)(unsigned)__builtin_amdgcn_readlane((int)use_hi, i) << 32 |
                                                 (unsigned)__builtin_amdgcn_readlane((int)use_lo, i);
        if (before + __popcll(heads) > rank) {
            for (; before < rank; ++before) heads &= heads - 1ull;
            head = i * 64 + __ffsll((long long)heads) - 1;
            break;
        }
        before += __popcll(heads);
    }
    head = __builtin_amdgcn_readfirstlane(head);
    // Pairs of this head, ascending: numbers p0 .. p0 + kJsPass - 1 of them to lanes 0 .. of `listed`; returns how many there are
    int listed = 0;
    auto list_pairs = [&](int p0) __attribute__((always_inline)) {
        int n = -p0;
        each_pair([&](int pair, int r) {
            const unsigned long long votes = __ballot(r == head);
            const int at = n + __popcll(votes & ((1ull << lane) - 1ull));
            const int sent = __builtin_amdgcn_ds_permute(r == head && at >= 0 && at < kJsPass ? at * 4 : 63 * 4, pair);
            const int more = n + __popcll(votes);
            if (lane >= n && lane < more) listed = sent;
            n = more;
        });
        return __builtin_amdgcn_readfirstlane(n) + p0;
    };
    const int n_items = list_pairs(0) * Tn;          // tokens of this head

    const int col = lane & 15, g = lane >> 4, r8 = lane >> 3;
    const unsigned int row_bytes = (unsigned int)D * 2u;
    const int f0 = part * units * 8, n_units = min(units, kJsUnits - part * units);      // features 0..127 query, 128..255 key
    const int n_mine = (D / 64 - w + kJsWaves - 1) / kJsWaves;                   // blocks of this wave: w, w + 8, ..
    char *const ring = lds + w * kJsWaveBytes;
    // piece p of row r of eight lands in slot p ^ (r >> 1), with 4 on top in every other group of eight rows: 16 rows read at one
    // piece touch 16 different 16-byte bank groups
    const int piece[2] = {((lane & 7) ^ (r8 >> 1)) * 16, ((lane & 7) ^ (4 + (r8 >> 1))) * 16};
    unsigned int woff[MOST];
#pragma unroll
    for (int i = 0; i < MOST; ++i) {
        const int f = min(f0 + 8 * i, kJCol - 8);    // (a unit is of queries or of keys)
        woff[i] = (unsigned int)((f & (kHeadDim - 1)) + r8) * row_bytes + piece[i & 1];
    }
#if defined(__HIP_DEVICE_COMPILE__)
    const size_t head_at = (size_t)head * kHeadDim * row_bytes;
    const auto q_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(w_q + head_at), 0, -1, 0x00020000);
    const auto k_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(w_k + head_at), 0, -1, 0x00020000);
    const auto x_rs = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(x), 0, -1, 0x00020000);
#endif

    // up to 8 XT tokens c0 .. with U units
    auto run = [&](int c0, auto u_, auto xt_) __attribute__((always_inline)) {
        constexpr int U = decltype(u_)::value, XT = decltype(xt_)::value, NB = (U + 1) / 2, TT = (XT + 1) / 2;
        constexpr int kLoads = U + XT, kBytes = kLoads * 1024, R = kJsWaveBytes / kBytes < 8 ? kJsWaveBytes / kBytes : 8;
        static_assert(R >= 2 && kJsWaves * NB * TT * 1024 <= kJsWaves * kJsWaveBytes, "a block ahead; the sums fit");
        unsigned int xoff[XT];
#pragma unroll
        for (int i = 0; i < XT; ++i) {
            const int it = min(c0 + 8 * i + r8, n_items - 1);        // tokens past the end repeat the last one, unused
            xoff[i] = (unsigned int)((__shfl(listed, it / Tn - c0 / Tn) / k) * Tn + it % Tn) * row_bytes + piece[i & 1];
        }
        auto fetch = [&](int s, int at) {
#if defined(__HIP_DEVICE_COMPILE__)
            const unsigned int off = (unsigned int)(w + s * kJsWaves) * 128u;
            auto load = [&](__amdgpu_buffer_rsrc_t rs, unsigned int from, int i) {
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (__attribute__((address_space(3))) void *)(ring + at * kBytes + i * 1024), 16,
                                                         (int)from, 0, 0, 0);
            };
#pragma unroll
            for (int i = 0; i < U; ++i) load(f0 + 8 * i < kHeadDim ? q_rs : k_rs, woff[i] + off, i);
#pragma unroll
            for (int i = 0; i < XT; ++i) load(x_rs, xoff[i] + off, U + i);
#endif
        };
        // all requests but those of the `younger` last blocks have landed
        auto landed = [&](int younger) {
#if defined(__HIP_DEVICE_COMPILE__)
            if (younger >= R - 1) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((R - 1) * kLoads) : "memory");
            else
                unroll<R - 1>([&](auto m) {
                    if (younger == m.value) asm volatile("s_waitcnt vmcnt(%0)" ::"n"(m.value * kLoads) : "memory");
                });
#endif
        };
        f32x4 acc[NB][TT];
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int t = 0; t < TT; ++t) acc[n][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int s = 0; s < R - 1; ++s)
            if (s < n_mine) fetch(s, s);
        int at = 0;
        for (int s = 0; s < n_mine; ++s) {
            if (s + R - 1 < n_mine) fetch(s + R - 1, at == 0 ? R - 1 : at - 1);
            landed(n_mine - 1 - s);
            const char *base = ring + at * kBytes;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int slot = ((4 * i + g) ^ ((col >> 1) & 7)) << 4;
                Frag a[NB], b[TT];                   // (rows past an odd number of units are of no column or token)
#pragma unroll
                for (int n = 0; n < NB; ++n) a[n].raw = *reinterpret_cast<const u32x4 *>(base + (n * 16 + col) * 128 + slot);
#pragma unroll
                for (int t = 0; t < TT; ++t) b[t].raw = *reinterpret_cast<const u32x4 *>(base + (U * 8 + t * 16 + (XT == 1 ? col & 7 : col)) * 128 + (XT == 1 ? ((4 * i + g) ^ ((col & 7) >> 1)) << 4 : slot));
#pragma unroll
                for (int n = 0; n < NB; ++n)
#pragma unroll
                    for (int t = 0; t < TT; ++t) acc[n][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[n].bf, b[t].bf, acc[n][t], 0, 0, 0);
            }
            at = at == R - 1 ? 0 : at + 1;
        }
        __syncthreads();
        f32x4 *const red = reinterpret_cast<f32x4 *>(lds);   // [wave][n][t][lane]
#pragma unroll
        for (int n = 0; n < NB; ++n)
#pragma unroll
            for (int t = 0; t < TT; ++t) red[((w * NB + n) * TT + t) * 64 + lane] = acc[n][t];
        __syncthreads();
        // lane l holds features f0 + 16 n + 4*(l/16) .. +3 of token l%16
        if (w < NB * TT) {
            const int n = w / TT, t = w % TT, item = c0 + t * 16 + col, f = f0 + n * 16 + g * 4;
            const int sl = __shfl(listed, min(item, n_items - 1) / Tn - c0 / Tn);
            if (item < min(n_items, c0 + 8 * XT) && n * 16 + g * 4 < U * 8) {
                f32x4 sum = red[(n * TT + t) * 64 + lane];
#pragma unroll
                for (int i = 1; i < kJsWaves; ++i) sum += red[((i * NB + n) * TT + t) * 64 + lane];
                const int tok = item % Tn;
                char *orow = f < kHeadDim ? q_out + ((((size_t)(sl / k) * H + head) * Tn) + tok) * (kHeadDim * 2)
                                          : k_compact + ((size_t)sl * Tc_cap + pos0 + tok) * (kHeadDim * 2);
                bf16x4 o;
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = (__bf16)sum[e];
                *reinterpret_cast<bf16x4 *>(orow + (f & (kHeadDim - 1)) * 2) = o;
            }
        }
        __syncthreads();
    };
    auto pass = [&](int c0, auto u_) __attribute__((always_inline)) {
        const int left = n_items - c0;
        if (left <= 8) run(c0, u_, std::integral_constant<int, 1>{});
        else if constexpr (js_pass(decltype(u_)::value) == 16) run(c0, u_, std::integral_constant<int, 2>{});
        else if (left <= 16) run(c0, u_, std::integral_constant<int, 2>{});
        else run(c0, u_, std::integral_constant<int, kJsPass / 8>{});
    };
    const int step = js_pass(n_units);
    for (int c0 = 0; c0 < n_items; c0 += step) {
        if (c0 != 0) list_pairs(c0 / Tn);
        unroll<MOST>([&](auto i) __attribute__((always_inline)) {
            if (n_units == i.value + 1) pass(c0, std::integral_constant<int, i.value + 1>{});
        });
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
    __shared__ int slots[kJtMaxSlots];
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

// Measurement aid: 32 x 32 x 16 products alone, the prefill kernels' shape (16 x 16 x 32 ones, project_kernel's, reach a sixth
// more on the same data: 2060 TFLOP/s where these reach 1790).  Every wave (two per SIMD on every CU) loads six operand fragments from
// `buf` once and then issues rounds of eight independent v_mfma_f32_32x32x16_bf16 with nothing else in the loop.
// The rate depends on the operand VALUES (switching activity moves the clocks), hence operands from the caller's
// data rather than constants.
constexpr int kProbeBlocks = 512, kProbeThreads = 512, kProbeMfmaPerRound = 8;
__global__ __launch_bounds__(kProbeThreads) void mfma_probe_kernel(const u32x4 *__restrict__ buf, unsigned long long n_pieces,
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
    return (double)kProbeBlocks * (kProbeThreads / 64) * (double)rounds * kProbeMfmaPerRound * (2.0 * 32 * 32 * 16);
}

int launch_mfma_probe(const void *buf, size_t bytes, int rounds, float *sink, const KernelEvents &ev, hipStream_t stream)
{
    return (int)launch_kernel(mfma_probe_kernel, dim3(kProbeBlocks), dim3(kProbeThreads), 0, stream, ev,
                              static_cast<const u32x4 *>(buf), (unsigned long long)(bytes / 16), rounds, sink);
}

// Which calls project_stream_kernel takes.  Its workgroups need a CU each, so that what they save by streaming is lost again where
// they are several rounds, and more tokens of a head than 16 cost it passes or units.  What decides is therefore how many heads are
// in use (if the rows' maps are independent: H (1 - (1 - k/H)^B), the maps themselves are on the device), how many tokens such a head
// has, and the width, against the kernel that the call takes otherwise: project_rows_kernel up to 8 tokens over all rows,
// 64-token tiles above.  The lines lie where the two were level over 14 000 calls drawn at random (1 to 64 tokens, 1 to 600 heads,
// widths 64 to 9216, weights in no cache).  Of 3706 further ones 1645 are streamed, 1.56 times as fast on average; 4.9 % of these measured
// more than 2 % slower than the other kernel, 1.2 % more than 5 %, 0.4 % more than 10 %.  Of the rest 4.2 % would gain 5 % or more.
// Other kernel / this one in us, D = 4096 unless noted:
// * up to 8 tokens: 1 x 1, 8 of 32 heads 12.0 / 7.3; 8 x 1, 72 of 72, D 9216 87.8 / 67.1; 4 x 1, 16 of 72, D 9216 41.8 / 30.4; 1 x 1, 128 of
//   128, D 512 38.5 / 18.2; but 256 of 256, D 64 19.5 / 34.3, and 64 of 64, D 8192 52.4 / 63.5 (below).
// * 9 to 32: 16 x 1, 8 of 32 20.1 / 14.1; 1 x 32, 8 of 32 18.6 / 10.1; 16 x 1, 10 of 72, D 9216 39.3 / 30.8; but 2 x 16, 72 of 72, D 1024
//   12.5 / 18.5, 1 x 32, 64 of 72, D 9216 55.1 / 65.0, 32 x 1, 12 of 256, D 1024 8.9 / 25.7, 16 x 1, 16 of 72, D 9216 45.5 / 46.7.
// * 33 to 64: 1 x 64, 8 of 32 20.8 / 14.5; 16 x 4, 8 of 32 24.0 / 21.4; 1 x 64, 16 of 72, D 9216 49.2 / 37.0; but 6 x 10, 16 of 72, D 9216 51.9 / 55.0, 2 x 32, 8 of 40, D
//   512 6.9 / 7.7.
// * where the call would be 256-token tiles (more pairs than are listed in LDS, or more heads than are counted there): 16 x 1, 72 of 72,
//   D 9216 1032 / 79; 64 x 1, 40 of 40, D 1024 285 / 46; but 2 x 1, 600 of 600, D 512 87 / 357, and every wave looks through all
//   pairs for every 64 heads: 1 x 1, 2000 of 2000, D 512 161 / 4990.
static bool project_streams(int B, int H, int k, int Tn, int D)
{
    const long long tokens = (long long)B * Tn, pairs = (long long)B * k;
    if (tokens > 64) return false;
    const double used = H * (1.0 - pow(1.0 - (double)k / H, B)), each = (double)(pairs * Tn) / used;
    const bool unlisted = pairs > kJtMaxSlots;
    if (unlisted || (H > kJtMaxHeads && tokens > kJrTokens)) {
        // No other kernel for few tokens: against 256-token tiles, by what either takes in us.  Here: launch and first ramp, the weights at
        // 5.5 TB/s (again for more than 32 tokens of a head) or a ramp for every further round, and the look through the maps in every
        // round, once per 64 heads and once per pass, 64 entries at a time beyond those that are requested at once.  There: rounds of
        // tiles, each a chain along the width.  (Out by a quarter at most over 450 calls but where both take 8 us.)
        const double rounds = ceil(used / 64 - 0.001), passes = ceil(each / kJsPass - 0.001), batches = pairs > 512 ? (pairs - 448) / 64.0 : 1.0;
        const double weights = used * D * 9.3e-5 * passes, ramps = 7.0 * (rounds - 1);
        const double here = 6.0 + (weights > ramps ? weights : ramps) + rounds * ((H + 63) / 64 + passes) * batches * 0.25;
        const double there = (double)((pairs + kJCus - 1) / kJCus) * (0.0225 * D + 5.0);
        return here < there;
    }
    if (H > kJtMaxHeads && used < 128.5) return used < 32.5 || D >= 256;     // (the other kernel starts 16 workgroups for every head there is)
    // Eight units leave the rings two blocks.  With rows that all begin on the same memory channels that is not enough.
    const bool eight = (used > 60.5 && used < 64.5) || (used > 102.5 && used < 128.5);
    if (eight && ((D % 8192 == 0 && tokens <= 16) || (D % 4096 == 0 && tokens <= 2))) return false;
    // at most so many heads in use, so many tokens of each, and at least this width
    struct Line {
        double used, each;
        int width;
    };
    static const Line to16[] = {{16, 16, 1024}, {32, 16, 1280}, {42, 4, 2048}, {42, 16, 2560}, {51, 4, 2048},
                                {64, 2, 2048},  {64, 4, 2560},  {51, 8, 4096}, {85, 2, 4096}};
    static const Line to32[] = {{16, 32, 1024}, {32, 16, 1280}, {32, 32, 2112}, {42, 8, 2048}, {42, 32, 2560}, {51, 4, 1536},
                                {51, 8, 2048},  {64, 4, 2048},  {85, 2, 2560},  {85, 4, 3072}, {128, 4, 5120}};
    static const Line to64[] = {{8, 64, 2048}, {16, 32, 2176}, {16, 64, 4096}, {32, 17, 2304}, {42, 8, 2560},
                                {64, 4, 2560}, {51, 8, 4096},  {85, 4, 3072},  {128, 2, 4096}};
    auto within = [&](const Line &l) { return used < l.used + 0.01 && each < l.each + 0.01 && D >= l.width; };
    if (tokens <= kJrTokens) {
        if (H <= 16) return D >= 2304;
        if (used < 8.5) return D >= 640;
        if (used < 42.5) return D >= 384;
        return H > kJtMaxHeads ? used < 320.5 && D >= 512 : D >= (used < 200.5 ? 256 : 448);
    }
    if (tokens <= 16) return std::any_of(std::begin(to16), std::end(to16), within);
    return tokens <= 32 ? std::any_of(std::begin(to32), std::end(to32), within) : std::any_of(std::begin(to64), std::end(to64), within);
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
    //   few tokens          project_stream_kernel, see there and project_streams; up to 8 project_rows_kernel where that one does not pay
    //   B*k*Tn <= most      64-token tiles, head-major: B 16, k 8, Tn 16 / 64 / 128: 82 / 82 / 85 -> 20 / 32 / 62 us; B 1, k 8, Tn
    //                       512 / 2043: 85 / 87 -> 21 / 60 us; B 4, k 16, D 9216, Tn 256: 215 -> 135 us; B 4, k 8, D 6656, Tn 512:
    //                       151 -> 95 us
    //   above               256-token tiles: B 16, k 8, Tn 256: 82 us (118 us with the small tiles)
    // From 16384 pairs' tokens on the small tiles take a third round of the chip.  It pays where the large tiles need a second
    // one, or are a long chain and do not fill theirs, or hold few tokens each; in us, large / small tiles:
    //   B 16, k 8 (128 large tiles), Tn 128: D 4096 74 / 61, D 2048 42 / 37, D 1024 26.0 / 25.2; Tn 144, 160 and 192: D 4096
    //   75 / 84, 76 / 84 and 75 / 88, (144) D 3072 58 / 68, (160) D 2048 43 / 50
    //   B 1, k 8, Tn 2304 and 3072: D 2048 42 / 50, D 4096 75 / 90; B 4, k 8, Tn 600 (96), D 6656: 118 / 127
    //   B 4, k 16, Tn 300 (128), D 9216: 199 / 182
    //   B 16, k 10 (160), Tn 140, D 6656: 146 / 137
    //   B 16, k 16 (256), Tn 72 / 80 / 96: (72) D 9216 227 / 194, D 4096 (80) 97 / 86 and (96) 98 / 114
    //   B 16, k 32 (512), Tn 48: D 512 42 / 27, D 4096 194 / 91
    // The small tiles and project_rows_kernel list the pairs of a head in LDS (at most kJtMaxSlots of them).
    const long long items = (long long)B * k * Tn;
    const bool listed = (long long)B * k <= kJtMaxSlots;
    if (project_streams(B, H, k, Tn, D)) {
        // one round of the chip, or two, or what the most units of a workgroup ask for
        const int heads = H < B * k ? H : B * k, most = heads * ((kJsUnits + kJsMaxUnits - 3) / (kJsMaxUnits - 2));
        const bool few = heads <= kJCus / (kJsUnits / kJsFewUnits);
        const int n_wg = few ? kJCus : (most > 2 * kJCus ? most : 2 * kJCus);
        auto *kernel = few ? project_stream_kernel<kJsFewUnits> : project_stream_kernel<kJsMaxUnits>;
        static DeviceFlags lds_allowed[2];
        const hipError_t attr = allow_dynamic_lds(reinterpret_cast<const void *>(kernel), kJsLdsBytes, lds_allowed[few ? 1 : 0]);
        if (attr != hipSuccess) return (int)attr;
        return (int)launch_kernel(kernel, dim3((unsigned int)n_wg), dim3(kJsWaves * 64), kJsLdsBytes, stream, ev, xc, wq, wk, rep, B, H, k, Tn,
                                  D, qo, ko, pos0, Tc_cap);
    }
    if (listed && (long long)B * Tn <= kJrTokens && H <= 0x7fffffff / kJrParts)
        return (int)launch_kernel(project_rows_kernel, dim3((unsigned int)H * kJrParts), dim3(kJrWaves * 64), 0, stream, ev,
                                  xc, wq, wk, rep, B, H, k, Tn, D, qo, ko, pos0, Tc_cap);
    // (the tile kernel addresses the activations and one head's weights with 32-bit byte offsets below 2 GiB)
    const long long n_large = (long long)B * k * ((Tn + kJTok - 1) / kJTok);
    const bool one_round = n_large <= 150 && D < 8192;
    const long long most = n_large > 256 ? 24576 : (D < 2048 || one_round ? 16384 : (D < 3072 || n_large > 200 ? 20480 : 24576));
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
    const unsigned int n_items = (unsigned int)n_mt * k * B;
    const bool one_each = n_items < kJCus || D < 2 * kJStep;    // (loads run two stages ahead, at most one item)
    return (int)launch_kernel(project_kernel, dim3(one_each ? (n_items + 7) / 8 * 8 : kJCus), dim3(kJBlock), kJLdsBytes,
                              stream, ev, xc, wq, wk, rep, H, k, Tn, D, n_mt, n_items, qo, ko, pos0, Tc_cap);
}

}  // namespace chai
