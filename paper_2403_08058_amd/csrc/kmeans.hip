// Cluster-membership kernels: the 5-token attention-score features (Section 3.3, with f(Q,K) = softmax(Q K^T)
// of Section 3.1) and K-Means over them (Section 3.5; clustering error of Section 3.2).
//
// The k-means result must be bit-identical to the sequential statement of the algorithm for the same feature
// bits, so every fp64 multiply, add, subtract and divide below is rounded on its own: this file is compiled
// with -ffp-contract=off, the pragma repeats it, and each sum runs in the stated index order inside ONE
// thread (threads split independent sums, never one sum).
#include "chai_internal.h"

#pragma clang fp contract(off)

namespace chai {

namespace {

// ---------------------------------------------------------------------------------------------------------
// Features: grid (H, B), one wave per head.  The 128-term fp64 dot product of a causal (i, j) pair is one chain of sums in element
// order.  Up to five positions (15 pairs) four neighbouring lanes share a pair: each converts and multiplies its 32 elements at the
// same time as the others, and then they continue the chain one after the other.  (One lane per pair did all of a pair's conversions
// and products itself: 6.3 us for 4 x 72 heads, the kernel alone, now 4.2; 300 x 128 heads, five positions 64.1 -> 36.7 us a call.)
// More positions have a lane per pair, which adds a product as soon as it is there: two lanes per pair of six or seven positions, or
// one that held all its products, took registers that cost more waves than they saved time (300 x 128 heads, seven positions 72.0 -> 87.7
// us, eight 77.4 -> 167.4).  A pair's last lane then has its score; lane p takes pair p's element of the softmax.
// ---------------------------------------------------------------------------------------------------------
__device__ __forceinline__ double from_lane_before(double x)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(x), 0x111, 0xf, 0xf, false);      // row_shr 1
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(x), 0x111, 0xf, 0xf, false);
    return __hiloint2double(hi, lo);
}

template <int SL>
__global__ __launch_bounds__(64) void feature_kernel(const void *__restrict__ q5, const void *__restrict__ k5,
                                                     int H, int n_tok, int bf16, long long qs, long long ks,
                                                     double scale, float *__restrict__ feat)
{
    constexpr int kElems = kHeadDim / SL;
    __shared__ double s[8][8], ex[8][8];
    const int h = blockIdx.x, b = blockIdx.y, lane = threadIdx.x;
    const size_t head = (size_t)b * H + h;

    // pair -> (i, j) with j <= i, row by row
    int i = 0, j = lane / SL;
    while (i < n_tok && j > i) { j -= i + 1; ++i; }
    // (of four lanes per pair nearly all have one: the others repeat a pair's loads)
    const int slice = lane % SL, si = SL > 1 ? min(i, n_tok - 1) : i, sj = SL > 1 ? min(j, n_tok - 1) : j;
    const size_t qo = head * (size_t)qs + (size_t)si * kHeadDim + slice * kElems;
    const size_t ko = head * (size_t)ks + (size_t)sj * kHeadDim + slice * kElems;
    double prod[SL > 1 ? kElems : 1], acc = 0.0;
    auto take = [&](int e, double p) {
        if constexpr (SL > 1) prod[e] = p;
        else acc = acc + p;
    };
    // 16-byte loads (rows start on 16-byte boundaries: the strides are multiples of 8 elements), all of a lane's requested at once
    if (SL > 1 || i < n_tok) {
        if (bf16) {
            const uint4 *qv = reinterpret_cast<const uint4 *>(static_cast<const unsigned short *>(q5) + qo);
            const uint4 *kv = reinterpret_cast<const uint4 *>(static_cast<const unsigned short *>(k5) + ko);
            uint4 qr[kElems / 8], kr[kElems / 8];
#pragma unroll
            for (int c8 = 0; c8 < kElems / 8; ++c8) {
                qr[c8] = qv[c8];
                kr[c8] = kv[c8];
            }
#pragma unroll
            for (int c8 = 0; c8 < kElems / 8; ++c8) {
                const unsigned int aw[4] = {qr[c8].x, qr[c8].y, qr[c8].z, qr[c8].w}, bw[4] = {kr[c8].x, kr[c8].y, kr[c8].z, kr[c8].w};
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const unsigned int abits = (e & 1) ? (aw[e >> 1] & 0xffff0000u) : (aw[e >> 1] << 16);
                    const unsigned int bbits = (e & 1) ? (bw[e >> 1] & 0xffff0000u) : (bw[e >> 1] << 16);
                    take(c8 * 8 + e, (double)__uint_as_float(abits) * (double)__uint_as_float(bbits));
                }
            }
        } else {
            const float4 *qv = reinterpret_cast<const float4 *>(static_cast<const float *>(q5) + qo);
            const float4 *kv = reinterpret_cast<const float4 *>(static_cast<const float *>(k5) + ko);
            constexpr int kPieces = (SL == 1 ? kElems / 2 : kElems) / 4;      // requested at once
#pragma unroll
            for (int c0 = 0; c0 < kElems / 4; c0 += kPieces) {
                float4 qr[kPieces], kr[kPieces];
#pragma unroll
                for (int c4 = 0; c4 < kPieces; ++c4) {
                    qr[c4] = qv[c0 + c4];
                    kr[c4] = kv[c0 + c4];
                }
#pragma unroll
                for (int c4 = 0; c4 < kPieces; ++c4) {
                    const float av[4] = {qr[c4].x, qr[c4].y, qr[c4].z, qr[c4].w}, bv[4] = {kr[c4].x, kr[c4].y, kr[c4].z, kr[c4].w};
#pragma unroll
                    for (int e = 0; e < 4; ++e) take((c0 + c4) * 4 + e, (double)av[e] * (double)bv[e]);
                }
            }
        }
        if (SL == 1) s[i][j] = scale * acc;
    }
    // stage st: the pair's lane number st goes on from where the lane before it has come to (what the others add up is not used)
    if constexpr (SL > 1) {
#pragma unroll
        for (int st = 0; st < SL; ++st) {
            if (st > 0) acc = from_lane_before(acc);
#pragma unroll
            for (int e = 0; e < kElems; ++e) acc = acc + prod[e];
        }
        if (i < n_tok && slice == SL - 1) s[i][j] = scale * acc;
        i = 0;
        j = lane;
        while (i < n_tok && j > i) { j -= i + 1; ++i; }
    }
    __syncthreads();
    // every pair's lane takes its own exponential and its own division (one lane per row took up to eight of each in a
    // row); the row sum is added in column order by all of them
    double e = 0.0;
    if (i < n_tok) {
        double m = s[i][0];
        for (int c = 1; c <= i; ++c) m = fmax(m, s[i][c]);
        e = exp(s[i][j] - m);
        ex[i][j] = e;
    }
    __syncthreads();
    float *f = feat + head * (size_t)(n_tok * n_tok);
    if (i < n_tok) {
        double z = 0.0;
        for (int c = 0; c <= i; ++c) z = z + ex[i][c];
        f[i * n_tok + j] = (float)(e / z);
    }
    if (lane < n_tok * n_tok && lane % n_tok > lane / n_tok) f[lane] = 0.0f;
}

__device__ __forceinline__ double sqdist(const float *__restrict__ x, const double *c, int F)
{
    double acc = 0.0;
    for (int f = 0; f < F; ++f) {
        const double diff = (double)x[f] - c[f];
        const double sq = diff * diff;
        acc = acc + sq;
    }
    return acc;
}

// ---------------------------------------------------------------------------------------------------------
// K-Means: grid (B), one workgroup per batch row, 2^n "slices" of lanes per head.  A handful of workgroups on an otherwise
// idle chip: its time is the length of the dependent chain of one pass, so a pass is two stretches with one barrier each:
//  * assignment: lane sl of a head scans the centres sl, sl + slices, .. (two distances at a time, each one sequential
//    fp64 sum), then the slices of the head, neighbours in one DPP row, agree on the smallest distance (lowest centre on
//    ties: what a single ascending scan picks); the head's bit goes into the member mask of its centre;
//  * update: one thread per (centre, coordinate) adds its members in head order, walking the bits of the mask.
// Whether a centre is empty every wave sees for itself from the masks, whether a head moved from a flag; masks and flag
// are doubled, the ones of the next pass are cleared during the update.  (Before: slice winners, assignments, counts,
// wave votes and member lists passed through LDS with eight barriers per pass, and one thread numbered the clusters in
// the end: 66 us for 72 heads, 16 centres, 9 passes; now 28 us.)
// Dynamic LDS (kmeans_layout): centres [k][FP] fp64, rows padded with zeros (a zero term leaves the sum unchanged),
// distances [H] fp64, masks [2][k][W] words, assignment [H], counts [k], labels [k], flags, and a copy of the features
// when it fits.
// ---------------------------------------------------------------------------------------------------------
constexpr int kRegF = 32;            // coordinates of a head that stay in registers
constexpr int kKmThreads = 1024;     // most threads of a workgroup
constexpr int kMaxSlices = 16;       // lanes of a DPP row

struct KmeansLayout {
    int FP, W, slices;               // padded coordinates, mask words per centre, lanes per head
    size_t dmin, mask, assign, count, label, flag, x, bytes;      // byte offsets (centres at 0)
    bool stage_x;
};

__host__ __device__ inline KmeansLayout kmeans_layout(int H, int F, int k)
{
    KmeansLayout L;
    L.FP = (F + 3) / 4 * 4;
    L.W = (H + 31) / 32;
    L.slices = 1;
    while (2 * L.slices <= k && 2 * L.slices * H <= kKmThreads && L.slices < kMaxSlices) L.slices *= 2;
    size_t at = sizeof(double) * (size_t)k * L.FP;
    L.dmin = at;   at += sizeof(double) * (size_t)H;
    L.mask = at;   at += sizeof(unsigned) * 2 * (size_t)k * L.W;
    L.assign = at; at += sizeof(int) * (size_t)H;
    L.count = at;  at += sizeof(int) * (size_t)k;
    L.label = at;  at += sizeof(int) * (size_t)k;
    L.flag = at;   at += sizeof(int) * 2;
    L.x = at;
    L.stage_x = at + sizeof(float) * (size_t)H * F <= 64 * 1024;
    if (L.stage_x) at += sizeof(float) * (size_t)H * F;
    L.bytes = at;
    return L;
}

// What a distance counts for in the choice of the nearest centre.  An ascending scan that starts with centre 0 and takes what
// is smaller passes a NaN by, and keeps centre 0 for good if that one is NaN: NaN is the largest value, or for centre 0
// the smallest, and the choice no longer depends on how the centres are dealt to the slices.
__device__ __forceinline__ double rank_distance(double d, int j)
{
    return d == d ? d : (j == 0 ? -HUGE_VAL : HUGE_VAL);
}

template <int CTRL>
__device__ __forceinline__ void take_nearer(double &d, int &j)
{
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(d), CTRL, 0xf, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(d), CTRL, 0xf, 0xf, false);
    const int oj = __builtin_amdgcn_update_dpp(0, j, CTRL, 0xf, 0xf, false);
    const double od = __hiloint2double(hi, lo);
    const bool other = od < d || (od == d && oj < j);       // never NaN: both lanes of a pair decide alike
    d = other ? od : d;
    j = other ? oj : j;
}

__global__ __launch_bounds__(kKmThreads) void kmeans_kernel(const float *__restrict__ feat, int H, int F, int k,
                                                            const int32_t *__restrict__ init_heads, int max_iter,
                                                            int32_t *__restrict__ h2c, int32_t *__restrict__ rep,
                                                            int32_t *__restrict__ ncl, int32_t *__restrict__ iters)
{
    extern __shared__ __attribute__((aligned(16))) char km_lds[];
    const KmeansLayout L = kmeans_layout(H, F, k);
    const int FP = L.FP, W = L.W, slices = L.slices;
    double *centre = reinterpret_cast<double *>(km_lds);
    double *dmin = reinterpret_cast<double *>(km_lds + L.dmin);
    unsigned *masks = reinterpret_cast<unsigned *>(km_lds + L.mask);
    int *assign = reinterpret_cast<int *>(km_lds + L.assign);
    int *count = reinterpret_cast<int *>(km_lds + L.count);
    int *label = reinterpret_cast<int *>(km_lds + L.label);
    int *flag = reinterpret_cast<int *>(km_lds + L.flag);
    float *x_lds = reinterpret_cast<float *>(km_lds + L.x);

    const int b = blockIdx.x, tid = threadIdx.x, n_thr = blockDim.x, lane = tid & 63;
    const float *Xg = feat + (size_t)b * H * F;
    const float *X = L.stage_x ? x_lds : Xg;                // same values either way
    if (L.stage_x)
        for (int i = tid; i < H * F; i += n_thr) x_lds[i] = Xg[i];
    for (int i = tid; i < k * FP; i += n_thr) {
        const int j = i / FP, f = i - j * FP;
        const int h0 = min(max(init_heads[(size_t)b * k + j], 0), H - 1);
        centre[i] = f < F ? (double)Xg[(size_t)h0 * F + f] : 0.0;
    }
    for (int i = tid; i < 2 * k * W; i += n_thr) masks[i] = 0u;
    if (tid < 2) flag[tid] = 0;

    // thread -> (head, slice), the same in every pass; the head's coordinates stay in registers when there are few enough
    const int my_h = tid / slices, sl = tid - my_h * slices;
    const bool owner = my_h < H;
    const bool in_regs = F <= kRegF;
    double xr[kRegF];
#pragma unroll
    for (int f = 0; f < kRegF; ++f) xr[f] = (in_regs && owner && f < F) ? (double)Xg[(size_t)my_h * F + f] : 0.0;
    int prev = -1;                                          // the head's centre in the pass before
    __syncthreads();

    int it = 0;
    for (;;) {
        unsigned *mask = masks + (it & 1) * (k * W);
        int *moved_flag = flag + (it & 1);
        ++it;
        int best = 0;
        double bd = 0.0;
        if (owner) {
            if (in_regs) {
                best = -1;
                for (int j = sl; j < k; j += 2 * slices) {
                    const int j2 = min(j + slices, k - 1);  // past the last centre: repeated, not used
                    const double *c0 = centre + (size_t)j * FP, *c1 = centre + (size_t)j2 * FP;
                    double a0 = 0.0, a1 = 0.0;
#pragma unroll
                    for (int f0 = 0; f0 < kRegF; f0 += 4) {
                        if (f0 < F) {
#pragma unroll
                            for (int f = f0; f < f0 + 4; ++f) {
                                const double e0 = xr[f] - c0[f], e1 = xr[f] - c1[f];
                                const double s0 = e0 * e0, s1 = e1 * e1;
                                a0 = a0 + s0;
                                a1 = a1 + s1;
                            }
                        }
                    }
                    a0 = rank_distance(a0, j);
                    a1 = rank_distance(a1, j2);
                    if (best < 0 || a0 < bd) { bd = a0; best = j; }
                    if (j + slices < k && a1 < bd) { bd = a1; best = j + slices; }
                }
            } else {
                best = -1;
                for (int j = sl; j < k; j += slices) {
                    const double dj = rank_distance(sqdist(X + (size_t)my_h * F, centre + (size_t)j * FP, F), j);
                    if (best < 0 || dj < bd) { bd = dj; best = j; }
                }
            }
        }
        if (slices > 1) take_nearer<0xB1>(bd, best);       // quad_perm [1,0,3,2]
        if (slices > 2) take_nearer<0x4E>(bd, best);       // quad_perm [2,3,0,1]
        if (slices > 4) take_nearer<0x141>(bd, best);      // row_half_mirror: the other quad, which agrees already
        if (slices > 8) take_nearer<0x140>(bd, best);      // row_mirror: the other eight
        if (owner && sl == 0) {
            assign[my_h] = best;
            dmin[my_h] = bd;
            atomicOr(&mask[best * W + (my_h >> 5)], 1u << (my_h & 31));
            if (best != prev) *moved_flag = 1;
        }
        const int before = prev;
        prev = best;
        __syncthreads();

        // Centres that received no head take, in ascending order, the farthest head of a cluster that can spare one.
        // Sequential by nature, but needed only when some centre is empty.
        bool empty = false;
        for (int j = lane; j < k; j += 64) {
            unsigned any = 0u;
            for (int i = 0; i < W; ++i) any |= mask[j * W + i];
            empty |= any == 0u;
        }
        int changed = *moved_flag;
        if (__any(empty)) {                                 // the same in every wave
            for (int j = tid; j < k; j += n_thr) {
                int n = 0;
                for (int i = 0; i < W; ++i) n += __popc(mask[j * W + i]);
                count[j] = n;
            }
            __syncthreads();
            if (tid == 0) {
                for (int j = 0; j < k; ++j) {
                    if (count[j] != 0) continue;
                    int pick = -1;
                    double far = 0.0;
                    for (int h = 0; h < H; ++h)
                        if (count[assign[h]] >= 2 && dmin[h] > far) { far = dmin[h]; pick = h; }
                    if (pick < 0) continue;
                    const int from = assign[pick];
                    count[from]--;
                    mask[from * W + (pick >> 5)] &= ~(1u << (pick & 31));
                    assign[pick] = j;
                    count[j] = 1;
                    mask[j * W + (pick >> 5)] |= 1u << (pick & 31);
                    dmin[pick] = 0.0;
                }
            }
            __syncthreads();
            // heads that moved for good: compared with the pass before, which the owners remember
            const int now = owner ? assign[my_h] : 0;
            changed = __syncthreads_or(owner && now != before);
            prev = now;
        }
        if (!changed || it >= max_iter) break;
        // update: one thread per (centre, coordinate), members added in head order, four requested at a time
        for (int i = tid; i < k * F; i += n_thr) {
            const int j = i / F, f = i - j * F;
            double acc = 0.0;
            int n = 0;
            for (int wd = 0; wd < W; ++wd) {
                unsigned left = mask[j * W + wd];
                n += __popc(left);
                while (left != 0u) {
                    float v[4];
                    int got = 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int h = wd * 32 + (left != 0u ? __ffs(left) - 1 : 0);
                        got += left != 0u;
                        left &= left - 1u;                  // 0 stays 0
                        v[u] = X[(size_t)h * F + f];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (u < got) acc = acc + (double)v[u];
                }
            }
            if (n != 0) centre[j * FP + f] = acc / (double)n;
        }
        unsigned *next = masks + (it & 1) * (k * W);
        for (int i = tid; i < k * W; i += n_thr) next[i] = 0u;
        if (tid == 0) flag[it & 1] = 0;
        __syncthreads();
    }

    // canonical labels: clusters numbered by their lowest member, which represents them
    const unsigned *mask = masks + ((it - 1) & 1) * (k * W);
    for (int j = tid; j < k; j += n_thr) {
        int low = H;
        for (int i = W - 1; i >= 0; --i) {
            const unsigned m = mask[j * W + i];
            if (m != 0u) low = i * 32 + __ffs(m) - 1;
        }
        count[j] = low;
    }
    __syncthreads();
    for (int j = tid; j < k; j += n_thr) {
        const int low = count[j];
        int rank = 0, used = 0;
        for (int i = 0; i < k; ++i) {
            rank += count[i] < low;
            used += count[i] < H;
        }
        label[j] = rank;
        if (low < H) rep[(size_t)b * k + rank] = low;
        if (j >= used) rep[(size_t)b * k + j] = -1;
        if (j == 0) ncl[b] = used;
    }
    __syncthreads();
    for (int h = tid; h < H; h += n_thr) h2c[(size_t)b * H + h] = label[assign[h]];
    if (tid == 0 && iters) iters[b] = it;
}

// ---------------------------------------------------------------------------------------------------------
// The same for features of whole positions (F a square) that fit LDS, up to 64 centres: with the same result bit for bit, and
// with less of what the kernel above is bound by.  A pass of that one (72 heads, 16 centres, 25 coordinates) takes 8400 cycles:
//  * 4200 for the distances, 3 fp64 operations per coordinate at 8 cycles each.  Here matrix instructions take them in fp32 first, 16
//    heads and 16 centres per wave, as s = |c|^2 / 2 - x c, and fp64 only those centres that can still be the nearest.  With
//    u = 2^-24 and M the largest |x|^2 (a centre is a mean of heads, or one: |c|^2 <= M, |x| |c| <= M) the F products of x c, each
//    rounded at most twice and of a centre rounded to fp32, are off by less than (2F + 2) u M, |c|^2 / 2 by (F + 2) u M, so that a
//    centre whose s exceeds the least by more than 2 (3F + 4) u M has the larger distance, in fp64 as well (whose own error is 2^-28
//    of this).  Twice that is allowed for, and 1e-30 for what underflows.  One centre left: it is the nearest.  Where a value is not
//    finite all centres are taken in fp64.
//  * 2900 for walking the members' bits, word by word.  Here every head ranks itself among its cluster's and the sum goes along a
//    list of members, four per word.
//  * 1200 for barriers and the look for empty centres.
// The numbering at the end ranks the centres by readlane in one wave; fp64 distances to the own centre, which the repair of empty
// centres asks for, are taken there.  A pass took 4700 cycles (sums 1950, distances 1500, empty centres and ranks 770), and the
// start 6000, most of it the latency of loading the features: 27.7 -> 19.2 us for 4 problems of 72 heads, 16 centres and 25
// coordinates; one launch alone over 300 problems of 128 heads, 16 centres and 64 coordinates 228 -> 52 us.  With all words of both
// masks requested at once (FEW) a call takes 5 to 8 % less: 4 x 72 heads in five, six and seven passes 14.7 -> 13.6, 16.9 -> 15.7 and 21.0
// -> 19.7, 8 x 128 in ten 28.4 -> 26.9.  Sixteen members of a sum requested at a time, and distances in two chains of products, were
// up to 4 % slower on more heads and no faster elsewhere.  What is bound by
// launching (up to 40 heads) takes what it did.  Where most passes need the 64-bit distances of all centres (problems of a few tight
// clusters) it is level with the general kernel: 71.9 and 71.6 us for 8 of 256 heads, 16 centres, 25 coordinates.
// Dynamic LDS (FastLayout): centres [k][FP] fp64, features [H][FP] fp32, centres [16 n][C32] fp32, masks, lists of members, ...
// ---------------------------------------------------------------------------------------------------------
constexpr int kFastCentres = 64;
typedef float km_f32x4 __attribute__((ext_vector_type(4)));
template <int F>
struct FastLayout {
    // coordinates per lane group of a matrix operand: F and the place of |c|^2, the last of the fourth group
    static constexpr int FP = (F + 3) / 4 * 4, G = (F / 4 + 1 + 3) / 4 * 4, C32 = 4 * G + 4;
    static_assert(4 * G > F, "room for |c|^2");
    int W, LS, tiles;                                        // mask words per centre, bytes of a list, tiles of 16 centres
    size_t x, c32, mask, list, assign, dmin, count, label, flag, bytes;
    __host__ __device__ FastLayout(int H, int k)
    {
        W = (H + 31) / 32;
        LS = (H + 3) / 4 * 4;
        tiles = (k + 15) / 16;
        size_t at = sizeof(double) * (size_t)k * FP;
        x = at;      at += sizeof(float) * (size_t)H * FP;
        c32 = at;    at += sizeof(float) * (size_t)tiles * 16 * C32;
        dmin = at;   at += sizeof(double) * (size_t)((H + 1) / 2 * 2);
        list = at;   at += (size_t)k * LS;
        mask = at;   at += sizeof(unsigned) * 2 * (size_t)k * W;
        assign = at; at += sizeof(int) * (size_t)H;
        count = at;  at += sizeof(int) * (size_t)k;
        label = at;  at += sizeof(int) * (size_t)k;
        flag = at;   at += sizeof(int) * 4;
        bytes = at;
    }
};

// op over the four lanes l, l ^ 16, l ^ 32, l ^ 48; all of them get it
template <typename T, typename Op>
__device__ __forceinline__ T over_groups(T x, Op op)
{
    static_assert(sizeof(T) == 4, "one register");
    auto bits = [](T v) { unsigned u; __builtin_memcpy(&u, &v, 4); return u; };
    auto value = [](unsigned u) { T v; __builtin_memcpy(&v, &u, 4); return v; };
    const auto a = __builtin_amdgcn_permlane32_swap(bits(x), bits(x), false, false);
    x = op(value(a[0]), value(a[1]));
    const auto b = __builtin_amdgcn_permlane16_swap(bits(x), bits(x), false, false);
    return op(value(b[0]), value(b[1]));
}

// FEW: at most 128 heads, four words of a mask
template <int F, bool FEW>
__global__ __launch_bounds__(kKmThreads) void kmeans_fast_kernel(const float *__restrict__ feat, int H, int k,
                                                                 const int32_t *__restrict__ init_heads, int max_iter,
                                                                 int32_t *__restrict__ h2c, int32_t *__restrict__ rep,
                                                                 int32_t *__restrict__ ncl, int32_t *__restrict__ iters)
{
    extern __shared__ __attribute__((aligned(16))) char km_lds[];
    constexpr int FP = FastLayout<F>::FP, G = FastLayout<F>::G, C32 = FastLayout<F>::C32;
    const FastLayout<F> L(H, k);
    const int W = L.W;
    double *centre = reinterpret_cast<double *>(km_lds);
    float *x_lds = reinterpret_cast<float *>(km_lds + L.x), *c32 = reinterpret_cast<float *>(km_lds + L.c32);
    double *dmin = reinterpret_cast<double *>(km_lds + L.dmin);
    unsigned char *list = reinterpret_cast<unsigned char *>(km_lds + L.list);
    unsigned *masks = reinterpret_cast<unsigned *>(km_lds + L.mask);
    int *assign = reinterpret_cast<int *>(km_lds + L.assign), *count = reinterpret_cast<int *>(km_lds + L.count);
    int *label = reinterpret_cast<int *>(km_lds + L.label), *flag = reinterpret_cast<int *>(km_lds + L.flag);

    const int b = blockIdx.x, tid = threadIdx.x, n_thr = blockDim.x, lane = tid & 63;
    const float *Xg = feat + (size_t)b * H * F;
    for (int j = tid; j < k; j += n_thr) label[j] = min(max(init_heads[(size_t)b * k + j], 0), H - 1);
    for (int i0 = tid; i0 < H * FP; i0 += 8 * n_thr) {      // (eight requests in flight: one by one the load takes 2 us)
        float v[8];
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = min(i0 + u * n_thr, H * FP - 1), h = i / FP, f = i - h * FP;
            v[u] = Xg[h * F + min(f, F - 1)];
        }
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int i = i0 + u * n_thr;
            if (i < H * FP) x_lds[i] = i % FP < F ? v[u] : 0.f;
        }
    }
    for (int i = tid; i < 2 * k * W; i += n_thr) masks[i] = 0u;
    for (int i = tid; i < k * L.LS / 4; i += n_thr) reinterpret_cast<unsigned *>(list)[i] = 0u;
    for (int i = tid; i < L.tiles * 16 * C32; i += n_thr) c32[i] = 0.f;
    if (tid < 4) flag[tid] = 0;
    __syncthreads();

    // wave -> 16 heads, a lane's own the one of its number in the group of 16; group g holds coordinates G g .. of it
    const int my_h = tid / 64 * 16 + (lane & 15), g = lane >> 4;
    const bool searching = tid / 64 * 16 < H, owner = my_h < H;      // (searching: this wave has heads)
    float xr[G];
    float x2 = 0.f;
#pragma unroll
    for (int t = 0; t < G; ++t) {
        const int f = G * g + t;
        xr[t] = f < FP ? x_lds[min(my_h, H - 1) * FP + min(f, FP - 1)] : 0.f;
        x2 = __builtin_fmaf(xr[t], xr[t], x2);
    }
    x2 = over_groups(x2, [](float p, float q) { return p + q; });
    if (g == 3) xr[G - 1] = -1.f;                            // times |c|^2 / 2
    // the largest |x|^2 of all heads, as the bits of a float (a NaN is larger than all others)
    if (g == 0 && owner) atomicMax(&flag[2], __float_as_int(x2) & 0x7fffffff);
    for (int i = tid; i < k * FP; i += n_thr) {
        const int j = i / FP, f = i - j * FP;
        const float v = x_lds[label[j] * FP + f];
        centre[i] = (double)v;
        c32[j * C32 + f] = v;
    }
    int prev = -1;                                          // the head's centre in the pass before
    __syncthreads();
    constexpr float kU = 5.9604645e-8f;
    const float slack = 4.f * (3 * F + 4) * kU * 1.01f * __int_as_float(flag[2]) + 1e-30f;

    // fp64 distance of this thread's head to centre j, as the general kernel takes it
    auto exact = [&](int j) {
        const float4 *xp = reinterpret_cast<const float4 *>(x_lds + my_h * FP);
        const double2 *cp = reinterpret_cast<const double2 *>(centre + j * FP);
        double a = 0.0;
#pragma unroll 4
        for (int t = 0; t < FP / 4; ++t) {                  // (past F both are 0)
            const float4 x = xp[t];
            const double2 c0 = cp[2 * t], c1 = cp[2 * t + 1];
            const double e0 = (double)x.x - c0.x, e1 = (double)x.y - c0.y, e2 = (double)x.z - c1.x, e3 = (double)x.w - c1.y;
            const double s0 = e0 * e0, s1 = e1 * e1, s2 = e2 * e2, s3 = e3 * e3;
            a = a + s0;
            a = a + s1;
            a = a + s2;
            a = a + s3;
        }
        return rank_distance(a, j);
    };
    int it = 0;
    for (;;) {
        unsigned *mask = masks + (it & 1) * (k * W);
        int *moved_flag = flag + (it & 1);
        ++it;
        for (int j = tid; j < k; j += n_thr) count[j] = 0;
        const int before = prev;
        if (searching) {
            // lane: centres 16 i + 4 g + 0 .. 3 of its head
            float s[kFastCentres / 16][4], least = INFINITY;
            bool sound = true;
#pragma unroll
            for (int i = 0; i < kFastCentres / 16; ++i) {
                if (i < L.tiles) {
                    float c[G], c2 = 0.f;
#pragma unroll
                    for (int t = 0; t < G; t += 4) {
                        const float4 v = *reinterpret_cast<const float4 *>(c32 + (i * 16 + (lane & 15)) * C32 + G * g + t);
                        c[t] = v.x; c[t + 1] = v.y; c[t + 2] = v.z; c[t + 3] = v.w;
                    }
#pragma unroll
                    for (int t = 0; t < G; ++t) c2 = __builtin_fmaf(c[t], c[t], c2);
                    c2 = over_groups(c2, [](float p, float q) { return p + q; });
                    if (g == 3) c[G - 1] = 0.5f * c2;
                    km_f32x4 acc = {0.f, 0.f, 0.f, 0.f};     // x c - |c|^2 / 2
#pragma unroll
                    for (int t = 0; t < G; ++t) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(c[t], xr[t], acc, 0, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const bool there = i * 16 + 4 * g + e < k;
                        sound = sound && (!there || fabsf(acc[e]) < INFINITY);       // false for NaN
                        s[i][e] = there ? -acc[e] : INFINITY;
                        least = fminf(least, s[i][e]);
                    }
                }
            }
            least = over_groups(least, [](float p, float q) { return fminf(p, q); });
            const float limit = least + slack;
            int near = sound && limit < INFINITY ? 0 : 1 << 16, best = kFastCentres;
#pragma unroll
            for (int i = kFastCentres / 16 - 1; i >= 0; --i) {
                if (i < L.tiles) {
#pragma unroll
                    for (int e = 3; e >= 0; --e) {
                        near += s[i][e] <= limit;
                        best = s[i][e] <= limit ? i * 16 + 4 * g + e : best;
                    }
                }
            }
            near = over_groups(near, [](int p, int q) { return p + q; });
            best = over_groups(best, [](int p, int q) { return min(p, q); });
            if (__any(owner && near != 1)) {
                double bd = HUGE_VAL;
                int by = kFastCentres;                       // loses against any
                if (owner && near != 1) {
#pragma unroll 1
                    for (int j = 4 * g; j < k; j += (j & 3) == 3 ? 13 : 1) {
                        float sj = INFINITY;
#pragma unroll
                        for (int i = 0; i < kFastCentres / 16; ++i)
#pragma unroll
                            for (int e = 0; e < 4; ++e) sj = i < L.tiles && j == i * 16 + 4 * g + e ? s[i][e] : sj;
                        if (near < 1 << 16 && !(sj <= limit)) continue;
                        const double dj = exact(j);
                        if (by == kFastCentres || dj < bd) {
                            bd = dj;
                            by = j;
                        }
                    }
                }
#pragma unroll
                for (int o = 16; o < 64; o <<= 1) {
                    const double od = __shfl_xor(bd, o);
                    const int oj = __shfl_xor(by, o);
                    const bool other = od < bd || (od == bd && oj < by);     // never NaN: all lanes of a head decide alike
                    bd = other ? od : bd;
                    by = other ? oj : by;
                }
                if (near != 1) best = by;
            }
            if (owner && g == 0) {
                assign[my_h] = best;
                atomicOr(&mask[best * W + (my_h >> 5)], 1u << (my_h & 31));
                if (best != prev) *moved_flag = 1;
            }
            prev = best;
        }
        __syncthreads();

        // members of a centre, and of those the ones below head h
        auto members = [&](int j, int h, int &below) {
            int n = 0;
            below = 0;
            for (int i0 = 0; i0 < W; i0 += 4) {
                unsigned word[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) word[u] = mask[j * W + min(i0 + u, W - 1)];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int i = i0 + u;
                    const unsigned m = i < W ? word[u] : 0u, low = i < (h >> 5) ? ~0u : (i == (h >> 5) ? (1u << (h & 31)) - 1u : 0u);
                    n += __popc(m);
                    below += __popc(m & low);
                }
            }
            return n;
        };
        // empty centres: as in the general kernel
        int rank, ignored, n_mine;
        bool empty;
        const int mine = max(min(prev, k - 1), 0);           // (lanes without a head: any centre)
        if constexpr (FEW) {                                 // all words of both centres requested at once
            unsigned own[4], seen[4], any = 0u;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                own[u] = mask[mine * W + min(u, W - 1)];
                seen[u] = mask[min(lane, k - 1) * W + min(u, W - 1)];
            }
            n_mine = rank = 0;
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const unsigned m = u < W ? own[u] : 0u, low = u < (my_h >> 5) ? ~0u : (u == (my_h >> 5) ? (1u << (my_h & 31)) - 1u : 0u);
                n_mine += __popc(m);
                rank += __popc(m & low);
                any |= seen[u];
            }
            empty = any == 0u;                               // (past the last centre: the last one's)
        } else {
            n_mine = members(mine, my_h, rank);
            empty = lane < k && members(lane, 0, ignored) == 0;
        }
        int changed = *moved_flag;
        if (__any(empty)) {                                 // the same in every wave
            if (owner && g == 0) dmin[my_h] = exact(prev);
            for (int j = tid; j < k; j += n_thr) label[j] = members(j, 0, ignored);
            __syncthreads();
            if (tid == 0) {
                for (int j = 0; j < k; ++j) {
                    if (label[j] != 0) continue;
                    int pick = -1;
                    double far = 0.0;
                    for (int h = 0; h < H; ++h)
                        if (label[assign[h]] >= 2 && dmin[h] > far) { far = dmin[h]; pick = h; }
                    if (pick < 0) continue;
                    const int from = assign[pick];
                    label[from]--;
                    mask[from * W + (pick >> 5)] &= ~(1u << (pick & 31));
                    assign[pick] = j;
                    label[j] = 1;
                    mask[j * W + (pick >> 5)] |= 1u << (pick & 31);
                    dmin[pick] = 0.0;
                }
            }
            __syncthreads();
            const int now = owner ? assign[my_h] : 0;
            changed = __syncthreads_or(owner && now != before);
            prev = now;
            n_mine = members(prev, my_h, rank);
        }
        if (!changed || it >= max_iter) break;
        // every head takes its place in the list of its cluster
        if (owner && g == 0) {
            list[prev * L.LS + rank] = (unsigned char)my_h;
            count[prev] = n_mine;
        }
        __syncthreads();
        // update: one thread per (centre, coordinate), members added in head order
        for (int i = tid; i < k * F; i += n_thr) {
            const int j = i / F, f = i - j * F, n = count[j];
            const unsigned *row = reinterpret_cast<const unsigned *>(list + j * L.LS);
            const int last = L.LS / 4 - 1;
            double acc = 0.0;
            for (int m = 0; m < n; m += 8) {                 // eight members requested at a time (whatever the list holds is a head)
                const unsigned w0 = row[m / 4], w1 = row[min(m / 4 + 1, last)];
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = x_lds[(((u < 4 ? w0 : w1) >> (8 * (u & 3))) & 0xffu) * FP + f];
#pragma unroll
                for (int u = 0; u < 8; ++u) acc = acc + (double)(m + u < n ? v[u] : -0.0f);      // (-0 changes no sum)
            }
            if (n != 0) {
                const double mean = acc / (double)n;
                centre[j * FP + f] = mean;
                c32[j * C32 + f] = (float)mean;
            }
        }
        unsigned *next = masks + (it & 1) * (k * W);
        for (int i = tid; i < k * W; i += n_thr) next[i] = 0u;
        if (tid == 0) flag[it & 1] = 0;
        __syncthreads();
    }

    // canonical labels: clusters numbered by their lowest member, which represents them
    if (tid < 64) {
        const unsigned *mask = masks + ((it - 1) & 1) * (k * W);
        int low = H;
        for (int i0 = 0; i0 < W; i0 += 4) {
            unsigned word[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) word[u] = mask[min(lane, k - 1) * W + min(i0 + u, W - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (i0 + u < W && word[u] != 0u) low = min(low, (i0 + u) * 32 + __ffs(word[u]) - 1);
        }
        if (lane >= k) low = H;
        int rank = 0;
        for (int i = 0; i < k; ++i) rank += __builtin_amdgcn_readlane(low, i) < low;
        const int used = __popcll(__ballot(low < H));
        if (lane < k) {
            label[lane] = rank;
            if (low < H) rep[(size_t)b * k + rank] = low;
            if (lane >= used) rep[(size_t)b * k + lane] = -1;
        }
        if (lane == 0) {
            ncl[b] = used;
            if (iters) iters[b] = it;
        }
    }
    __syncthreads();
    for (int h = tid; h < H; h += n_thr) h2c[(size_t)b * H + h] = label[assign[h]];
}

// ---------------------------------------------------------------------------------------------------------
// Clustering error of a given partition (Section 3.2): grid (B), 256 threads.  Means per (cluster, coordinate)
// by one thread each (members in head order), distance of every head to its cluster's mean by one thread each,
// then thread 0 adds the distances cluster by cluster, heads ascending: the order of the sequential statement.
// With rep_out, thread j also picks the member of cluster j nearest its mean (first of equals = lowest head,
// -1 for an empty slot).  Either output may be NULL.
// Dynamic LDS: means [k][F] fp64, distances [H] fp64, counts [k].
// ---------------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(kBlock) void cluster_error_kernel(const float *__restrict__ feat,
                                                               const int32_t *__restrict__ h2c, int H, int F, int k,
                                                               double *__restrict__ sse,
                                                               int32_t *__restrict__ rep_out)
{
    extern __shared__ double lds[];
    double *mean = lds;                          // [k][F]
    double *dist = mean + (size_t)k * F;         // [H]
    int *count = reinterpret_cast<int *>(dist + H);   // [k]
    const int b = blockIdx.x, tid = threadIdx.x;
    const float *X = feat + (size_t)b * H * F;
    const int32_t *lab = h2c + (size_t)b * H;

    for (int j = tid; j < k; j += kBlock) {
        int c = 0;
        for (int h = 0; h < H; ++h) c += lab[h] == j;
        count[j] = c;
    }
    __syncthreads();
    for (int i = tid; i < k * F; i += kBlock) {
        const int j = i / F, f = i - j * F;
        if (count[j] == 0) continue;
        double acc = 0.0;
        for (int h = 0; h < H; ++h)
            if (lab[h] == j) acc = acc + (double)X[(size_t)h * F + f];
        mean[i] = acc / (double)count[j];
    }
    __syncthreads();
    for (int h = tid; h < H; h += kBlock) {
        const int j = lab[h];
        dist[h] = (j >= 0 && j < k) ? sqdist(X + (size_t)h * F, mean + (size_t)j * F, F) : 0.0;
    }
    __syncthreads();
    if (rep_out != nullptr) {
        for (int j = tid; j < k; j += kBlock) {
            int best = -1;
            double best_d = 0.0;
            for (int h = 0; h < H; ++h)
                if (lab[h] == j && (best < 0 || dist[h] < best_d)) {
                    best = h;
                    best_d = dist[h];
                }
            rep_out[(size_t)b * k + j] = best;
        }
    }
    if (sse != nullptr && tid == 0) {
        double total = 0.0;
        for (int j = 0; j < k; ++j)
            for (int h = 0; h < H; ++h)
                if (lab[h] == j) total += dist[h];
        sse[b] = total;
    }
}

}  // namespace

int launch_score_features(const void *q5, const void *k5, int B, int H, int n_tok, int dtype, int64_t qs, int64_t ks,
                          float scale, float *feat, hipStream_t stream)
{
    auto *kernel = n_tok <= 5 ? feature_kernel<4> : feature_kernel<1>;       // 15 pairs of five positions, 21 of six
    return (int)launch_kernel(kernel, dim3(H, B), dim3(64), 0, stream, KernelEvents(), q5, k5, H, n_tok,
                              dtype == CHAI_BF16 ? 1 : 0, (long long)qs, (long long)ks, (double)scale, feat);
}

// Sizes that are accepted, next to H <= 256, F <= 64 and k*F <= 7168: a line that callers know, drawn on its own.  What the
// kernel allocates is kmeans_layout's, at most 73 976 bytes on this side of the line (244 heads, 25 coordinates, 240 centres).
bool assign_clusters_supported(int H, int F, int k)
{
    const long long s = 512 / H < 1 ? 1 : (512 / H > k ? k : 512 / H);
    return 8LL * k * F + 20LL * H + 12LL * H * s + 28LL * k <= 65472;
}

constexpr size_t kKmeansLds = 96 * 1024;     // most LDS of a workgroup (its CU has 160 KB)
constexpr size_t kPlainLds = 63 * 1024;      // most dynamic LDS without leave: 64 KB with what the kernels have besides (256 bytes)

template <int F>
static bool launch_fast(const float *feat, int B, int H, int k, const int32_t *init_heads, int max_iter, int32_t *h2c, int32_t *rep,
                        int32_t *ncl, int32_t *iters, hipStream_t stream, int &status)
{
    const FastLayout<F> L(H, k);
    if (L.bytes > kPlainLds || k > kFastCentres || H > 256) return false;
    // threads: the waves of all heads, and enough for the update to be one round where that is not much more
    int n_thr = (H + 15) / 16 * 64;
    const int update = (k * F + 63) / 64 * 64;
    if (n_thr < update) n_thr = update < 512 ? update : (n_thr < 512 ? 512 : n_thr);
    status = (int)launch_kernel(H <= 128 ? kmeans_fast_kernel<F, true> : kmeans_fast_kernel<F, false>, dim3(B), dim3(n_thr), L.bytes, stream, KernelEvents(), feat, H, k, init_heads,
                                max_iter, h2c, rep, ncl, iters);
    return true;
}

int launch_assign_clusters(const float *feat, int B, int H, int F, int k, const int32_t *init_heads, int max_iter,
                           int32_t *h2c, int32_t *rep, int32_t *ncl, int32_t *iters, hipStream_t stream)
{
    const KmeansLayout L = kmeans_layout(H, F, k);
    if (L.bytes > kKmeansLds) return (int)hipErrorInvalidConfiguration;
    // features of 3 to 8 positions: never slower there (the comment at the kernel); others would each need a kernel of their own,
    // and no prompt gives them
    int status = 0;
    auto fast = [&](auto *launch) { return launch(feat, B, H, k, init_heads, max_iter, h2c, rep, ncl, iters, stream, status); };
    if ((F == 9 && fast(launch_fast<9>)) || (F == 16 && fast(launch_fast<16>)) || (F == 25 && fast(launch_fast<25>)) ||
        (F == 36 && fast(launch_fast<36>)) || (F == 49 && fast(launch_fast<49>)) || (F == 64 && fast(launch_fast<64>)))
        return status;
    if (L.bytes > kPlainLds) {                              // the mask words of many centres over many heads
        static DeviceFlags lds_allowed;
        const hipError_t e = allow_dynamic_lds(reinterpret_cast<const void *>(&kmeans_kernel), kKmeansLds, lds_allowed);
        if (e != hipSuccess) return (int)e;
    }
    // threads: the lanes of all heads, and enough for the update to be one round where that is not much more
    int n_thr = (H * L.slices + 63) / 64 * 64;
    const int update = (k * F + 63) / 64 * 64;
    if (n_thr < update) n_thr = update < 512 ? update : (n_thr < 512 ? 512 : n_thr);
    return (int)launch_kernel(kmeans_kernel, dim3(B), dim3(n_thr), L.bytes, stream, KernelEvents(), feat, H, F, k, init_heads,
                              max_iter, h2c, rep, ncl, iters);
}

size_t cluster_error_lds_bytes(int H, int F, int k)
{
    return sizeof(double) * ((size_t)k * F + H) + sizeof(int) * (size_t)k;
}

int launch_cluster_error(const float *feat, const int32_t *h2c, int B, int H, int F, int k, double *sse,
                         int32_t *rep_out, hipStream_t stream)
{
    return (int)launch_kernel(cluster_error_kernel, dim3(B), dim3(kBlock), cluster_error_lds_bytes(H, F, k), stream,
                              KernelEvents(), feat, h2c, H, F, k, sse, rep_out);
}

}  // namespace chai
