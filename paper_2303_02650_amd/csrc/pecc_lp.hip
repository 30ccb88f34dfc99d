// Learned proposal for the perturbation step of SED (Sec. 5, Alg. 5): the
// solution-space exploring step relocates a few circles, and a small network
// scores candidate relocations (circle i, destination q) from local features
// so that the best-scored distinct circles are moved.
//
// Kernels
//   features_kernel   8 features per candidate, cell grid of side >= 4 in LDS,
//                     FP32 distances, FP64 where they cannot decide and
//                     for the overlaps
//   mlp_forward_kernel    8 -> 64 -> 64 -> 1 erf-GELU network on BF16 MFMA
//   mlp_grad_kernel       forward + backward of the mean BCE-with-logits loss,
//                         per-workgroup partial gradients (MFMA for every
//                         contraction), then grad_reduce_kernel sums them in a
//                         fixed order and, in a training step, updates
//   adam_kernel           Adam on FP32 master weights by itself
//   propose_kernel        top-k distinct circles by score (or the first k
//                         distinct candidates without usable scores) and the
//                         relocated layout
//   accept_kernel         keep the relocated-and-descended layout when its FP64
//                         energy is lower
//
// MFMA (gfx950, v_mfma_f32_16x16x32_bf16), per wave64 lane l, g = l / 16,
// r = l % 16:  A operand  A[r][8g + i],  B operand  B[8g + i][r]  (i < 8),
// result D[4g + i][r] (i < 4).  The network runs with neurons as the M
// dimension and rows (samples) as N, so a layer's result, lane (g, r) holding
// neurons 16t + 4g + i of row r for the four neuron tiles t, is already laid
// out as the next layer's B operand once the K slots are permuted to match:
// K slot (g, i') of chunk c is neuron 16 (2c + i' / 4) + 4g + i' % 4.  The
// weight fragments are read with that permutation, so no data moves between
// lanes.  The forward feeds the features and the first activations as BF16
// high + low pairs (x = hi + lo to about 2^-16), which keeps the logits near
// FP32 accuracy; the features' pair fits in the K slots the 8 inputs leave
// free.  Contractions over rows (weight gradients) go through a per-wave LDS
// stage that transposes rows into the K dimension.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "pecc_device.hpp"
#include "pecc_launch.hpp"
#include "pecc_lbfgs.hpp"

namespace pecc {
namespace {

constexpr int kFeat = 8, kHid = 64, kParams = 4801;
constexpr int oW1 = 0, oB1 = 512, oW2 = 576, oB2 = 4672, oW3 = 4736, oB3 = 4800;

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// Features
// ---------------------------------------------------------------------------
// Bound by vector issue: two points per candidate (the circle and its
// destination), each against the 3 x 3 cells of side 4 around it, 38 circles
// at packing density.  Those cost an FP32 distance and a sign bit per
// threshold, the bits collected per cell row and counted at the end; a circle
// that may overlap, or lies within a band of a threshold that the FP32
// distance cannot decide (distances of 2 and 4 are common in packings), is
// taken in FP64, the overlaps in the order of the cells.  512 threads share
// one sort of the circles; both points of a candidate run side by side.
// 128 x 4096 candidates at n = 1000: 48 us (127 us with every distance in
// FP64, a square root evaluated by the whole wave at nearly every circle).
constexpr int kFeatBlock = 512;
constexpr int kFeatChunk = 1024;     // candidates per workgroup
constexpr float kDensRadius = 4.0f;  // widest radius a feature looks at

struct FeatShared {
    float2 psort[kMaxN + 8];         // positions in cell order
    int cell_start[kMaxCells + 1];
    uint16_t cell_circ[kMaxN];
    uint16_t slot_tmp[kMaxN];
    uint16_t slot_of[kMaxN];         // place of a circle in the cell order
    int scan_tmp[kFeatBlock / 64];
};

// Overlap energy, neighbor count, boundary gap and density around the points
// p[0], p[1] over the circles except the one at place `own` (the circle that
// would move is lifted out).
__device__ __forceinline__ void feature_quads(const FeatShared &S, const Grid &g, double R, bool act,
                                              int own, const float2 (&p)[2], float *f)
{
#pragma clang fp contract(off)   // distances rounded operation by operation, like the oracle
    // thresholds on the squared distance; lo/hi: outside the FP32 distance's
    // error (4e-7 of it) on either side
    constexpr float kBand = 1e-6f;
    constexpr float kOver = 4.0f * (1.0f + kBand);
    constexpr float kNearLo = 5.29f * (1.0f - kBand), kNearHi = 5.29f * (1.0f + kBand);
    constexpr float kDensLo = 16.0f * (1.0f - kBand), kDensHi = 16.0f * (1.0f + kBand);
    int ra[2][3], rl[2][3];
    bool plain[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        int place;
        // a point that is not finite is near nothing
        const bool on = act && fabsf(p[q].x) < HUGE_VALF && fabsf(p[q].y) < HUGE_VALF;
        cell_rows(p[q], on, 0, g, S.cell_start, ra[q], rl[q], place);
        plain[q] = max(rl[q][0], max(rl[q][1], rl[q][2])) <= 32 && rl[q][0] + rl[q][1] + rl[q][2] <= 64;
    }
    int near[2] = {0, 0}, dens[2] = {0, 0};
    double e[2] = {0.0, 0.0};
    unsigned exact[2][3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int longest = wave_max_dpp(max(plain[0] ? rl[0][r] : 0, plain[1] ? rl[1][r] : 0));
        unsigned over[2] = {0, 0}, nlo[2] = {0, 0}, nhi[2] = {0, 0}, dlo[2] = {0, 0}, dhi[2] = {0, 0};
        // downwards, so that the bit shifted in last is the first candidate
        for (int k0 = (longest + 3) / 4 * 4 - 4; k0 >= 0; k0 -= 4) {
            float2 c[2][4];
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const float2 *src = S.psort + min(ra[q][r] + k0, kMaxN);
#pragma unroll
                for (int u = 0; u < 4; ++u) c[q][u] = src[u];
            }
#pragma unroll
            for (int u = 3; u >= 0; --u)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float dx = p[q].x - c[q][u].x, dy = p[q].y - c[q][u].y;
                    const float l2 = fmaf(dx, dx, dy * dy);
                    auto push = [&](unsigned &w, float limit) {
                        w = __builtin_amdgcn_alignbit(w, __float_as_uint(l2 - limit), 31);
                    };
                    push(over[q], kOver);
                    push(nlo[q], kNearLo);
                    push(nhi[q], kNearHi);
                    push(dlo[q], kDensLo);
                    push(dhi[q], kDensHi);
                }
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            unsigned keep = rl[q][r] < 32 ? (1u << rl[q][r]) - 1u : ~0u;
            const unsigned place = (unsigned)(own - ra[q][r]);
            if (place < 32u) keep &= ~(1u << place);
            if (!plain[q]) keep = 0;
            const unsigned ex = (over[q] | (nhi[q] & ~nlo[q]) | (dhi[q] & ~dlo[q])) & keep;
            exact[q][r] = ex;
            near[q] += __builtin_popcount(nlo[q] & keep & ~ex);
            dens[q] += __builtin_popcount(dlo[q] & keep & ~ex);
        }
    }
    auto visit = [&](int q, float2 c) {
#pragma clang fp contract(off)
        const double dx = (double)p[q].x - (double)c.x;
        const double dy = (double)p[q].y - (double)c.y;
        const double l2 = dx * dx + dy * dy;
        if (l2 < 4.0) {
            // FP64 root by Newton steps from the FP32 one (2 - l is 2 for any
            // l2 below the FP32 range's lower end)
            const float l2f = (float)l2;
            const float il = l2f > 1e-30f ? __builtin_amdgcn_rsqf(l2f) : 0.f;
            const double d = 2.0 - sqrt64_from32(l2, l2f * il, il);
            e[q] = e[q] + d * d;
        }
        near[q] += l2 < 5.29;
        dens[q] += l2 < 16.0;
    };
    unsigned long long mask[2];
    int cut[2], s1[2], s2[2], longest = 0;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        cut[q] = rl[q][0] + rl[q][1];
        s1[q] = ra[q][1] - rl[q][0];
        s2[q] = ra[q][2] - cut[q];
        mask[q] = (unsigned long long)exact[q][2];
        mask[q] = (mask[q] << (rl[q][1] & 63)) | exact[q][1];
        mask[q] = (mask[q] << (rl[q][0] & 63)) | exact[q][0];
        longest = max(longest, __builtin_popcountll(mask[q]));
    }
    longest = wave_max_dpp(longest);
    for (int k = 0; k < longest; ++k) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const bool has = mask[q] != 0;
            const int t = __builtin_ctzll(mask[q] | (1ull << 63));
            mask[q] &= mask[q] - 1;
            const float2 c = S.psort[has ? t + (t < rl[q][0] ? ra[q][0] : t < cut[q] ? s1[q] : s2[q]) : 0];
            if (has) visit(q, c);
        }
    }
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        if (!plain[q])               // a crowded neighborhood: candidate by candidate
            for (int r = 0; r < 3; ++r)
                for (int t = ra[q][r]; t < ra[q][r] + rl[q][r]; ++t)
                    if (t != own) visit(q, S.psort[t]);
        const double px = (double)p[q].x, py = (double)p[q].y;
        const double rho = sqrt(px * px + py * py);
        const double d0 = (rho + 1.0) - R;
        if (d0 > 0.0) e[q] = e[q] + d0 * d0;
        f[4 * q] = (float)(log10(e[q] + 1e-20) / 20.0 + 1.0);
        f[4 * q + 1] = (float)near[q];
        f[4 * q + 2] = (float)((R - 1.0 - rho) / R);
        f[4 * q + 3] = (float)((double)dens[q] / (16.0 * 3.14159265358979323846));
    }
}

template <int BLOCK>
__global__ __launch_bounds__(BLOCK) void features_kernel(
    const int32_t *__restrict__ offset, const float *__restrict__ Rf,
    const double *__restrict__ R64, const float *__restrict__ xy, int C,
    const int32_t *__restrict__ cand_circle, const float *__restrict__ cand_dest,
    float *__restrict__ feat)
{
    constexpr int kCpt = kMaxN / BLOCK;
    __shared__ FeatShared S;
    const int b = blockIdx.y, tid = threadIdx.x;
    const int o = offset[b];
    int n = offset[b + 1] - o;
    const bool bad = n < 0 || n > kMaxN;
    if (bad) n = 0;
    const double R = R64 ? R64[b] : (double)Rf[b];
    const float2 *p2 = reinterpret_cast<const float2 *>(xy) + o;
    const Grid g = make_grid(Rf[b], kDensRadius * (1.0f + kCellSafety));
    {
        float2 x[kCpt];
        int own[kCpt];
#pragma unroll
        for (int u = 0; u < kCpt; ++u) {
            const int i = tid + u * BLOCK;
            x[u] = i < n ? p2[i] : make_float2(0.f, 0.f);
            // a circle at NaN is near nothing, like one at infinity (whose
            // sign bits are known)
            if (x[u].x != x[u].x) x[u].x = HUGE_VALF;
            if (x[u].y != x[u].y) x[u].y = HUGE_VALF;
        }
        sort_cells<BLOCK, kCpt>(tid, x, n, g, S.cell_start, S.cell_circ, S.slot_tmp, S.psort,
                                         S.scan_tmp, own);
#pragma unroll
        for (int u = 0; u < kCpt; ++u)
            if (tid + u * BLOCK < n) S.slot_of[tid + u * BLOCK] = (uint16_t)own[u];
        __syncthreads();
    }
    const int c0 = blockIdx.x * kFeatChunk;
    const int c1 = min(C, c0 + kFeatChunk);
    // (a wave's first candidate, uniform: waves past the end have none)
    const int w0 = __builtin_amdgcn_readfirstlane(tid & ~(kWave - 1));
    for (int k0 = c0; k0 + w0 < c1; k0 += BLOCK) {
        // lanes past the end take the last candidate (the longest runs are
        // found across the lanes) and store nothing
        const int k = min(k0 + tid, c1 - 1);
        const int64_t gi = (int64_t)b * C + k;
        const int i = cand_circle[gi];
        const bool act = !bad && i >= 0 && i < n;
        float f[8];
        const float2 p[2] = {act ? p2[i] : make_float2(0.f, 0.f),
                             reinterpret_cast<const float2 *>(cand_dest)[gi]};
        feature_quads(S, g, R, act, act ? S.slot_of[i] : 0, p, f);
        if (!act) {
#pragma unroll
            for (int q = 0; q < 8; ++q) f[q] = __builtin_nanf("");
        }
        if (k0 + tid >= c1) continue;
        float4 *dst = reinterpret_cast<float4 *>(feat + gi * 8);
        dst[0] = make_float4(f[0], f[1], f[2], f[3]);
        dst[1] = make_float4(f[4], f[5], f[6], f[7]);
    }
}

// ---------------------------------------------------------------------------
// Network: weights in LDS as BF16 (round to nearest even of the FP32 master)
// ---------------------------------------------------------------------------
// Rows of 68 values: the fragments' 8-byte reads down 16 rows, and the
// transposed row of W2 written across 64 rows, would meet in one bank at 64.
constexpr int kRow2 = kHid + 4;

struct NetWeights {
    alignas(16) __bf16 w1[kHid * kFeat];     // [n][k]
    alignas(16) __bf16 w2[kHid * kRow2];     // [n][k]
    alignas(16) __bf16 w2t[kHid * kRow2];    // [k][n]  (backward)
    alignas(16) float b1[kHid];
    float b2[kHid], w3[kHid];             // w3 holds the BF16 values
    float b3;
};

template <int BLOCK>
__device__ void load_weights(const float *__restrict__ P, NetWeights &W, bool transpose)
{
    constexpr int kPer = (kParams + BLOCK - 1) / BLOCK;
    float in[kPer];                  // all in flight together
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int k = threadIdx.x + q * BLOCK;
        in[q] = P[k < kParams ? k : 0];
    }
#pragma unroll
    for (int q = 0; q < kPer; ++q) {
        const int k = threadIdx.x + q * BLOCK;
        const float v = in[q];
        if (k < oB1) {
            W.w1[k] = (__bf16)v;
        } else if (k < oW2) {
            W.b1[k - oB1] = v;
        } else if (k < oB2) {
            const int n = (k - oW2) / kHid, c = (k - oW2) % kHid;
            W.w2[n * kRow2 + c] = (__bf16)v;
            if (transpose) W.w2t[c * kRow2 + n] = (__bf16)v;
        } else if (k < oW3) {
            W.b2[k - oB2] = v;
        } else if (k < oB3) {
            W.w3[k - oW3] = (float)(__bf16)v;
        } else if (k < kParams) {
            W.b3 = v;
        }
    }
}

// erf(x) by the rational approximation 7.1.26 of Abramowitz and Stegun
// (Handbook of Mathematical Functions): erf(x) = 1 - (a1 t + ... + a5 t^5)
// exp(-x^2) with t = 1 / (1 + p x) for x >= 0, odd in x; at most 1.5e-7 from
// erf in exact arithmetic, about 6e-7 in FP32 with the hardware reciprocal
// and exponential.  gauss receives the exp(-x^2) it forms.  One reciprocal,
// one exponential and seven FMAs, against the library erff's longer
// piecewise evaluation.  Used where the derivative, which shares the
// exponential, is wanted too (training).
__device__ __forceinline__ float erf_as(float x, float &gauss)
{
    const float ax = fabsf(x);
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, ax, 1.0f));
    float q = fmaf(t, 1.061405429f, -1.453152027f);
    q = fmaf(t, q, 1.421413741f);
    q = fmaf(t, q, -0.284496736f);
    q = fmaf(t, q, 0.254829592f);
    gauss = __expf(-ax * ax);
    return copysignf(fmaf(-t * q, gauss, 1.0f), x);
}

// GELU(t) = t Phi(t) = 0.5 t (1 + erf(t / sqrt 2)) and its derivative
// Phi(t) + t phi(t), phi(t) = exp(-t^2 / 2) / sqrt(2 pi) (the same
// exponential as the erf's).
__device__ __forceinline__ float gelu(float t)
{
    float gs;
    return 0.5f * t * (1.0f + erf_as(t * 0.70710678118654752f, gs));
}

__device__ __forceinline__ float gelu_prime(float t)
{
    float gs;
    const float e = erf_as(t * 0.70710678118654752f, gs);
    return 0.5f * (1.0f + e) + t * 0.39894228040143268f * gs;
}

// GELU where its derivative is not wanted: log2 Phi(-|t|) is close to a
// parabola, so one exponential of a polynomial gives the tail.  Degree 6,
// the coefficients fitted (minimax over 0 <= |t| <= 8) for |t| Phi(-|t|):
// as written 5.5e-8 off in exact arithmetic (at 0.966), 8.9e-8 in FP32 with
// correctly rounded steps, besides the sum's own rounding; 2.6e-7 for 0.5 t (1
// + erf(t / sqrt 2)) by the rational approximation.  The network's 128
// activations per row are most of its vector work: 10 instructions each with
// one transcendental, 19 with two in that form.  The maximum keeps NaN.
__device__ __forceinline__ float gelu_fast(float t)
{
    const float c = fabsf(__builtin_amdgcn_fmed3f(t, -8.0f, 8.0f));
    float q = fmaf(c, 3.30928088e-05f, -7.69219594e-04f);
    q = fmaf(c, q, 8.08071624e-03f);
    q = fmaf(c, q, -5.34121022e-02f);
    q = fmaf(c, q, -4.58770961e-01f);
    q = fmaf(c, q, -1.15120173e+00f);
    q = fmaf(c, q, -9.99993086e-01f);
    return fmaf(-c, __builtin_amdgcn_exp2f(q), __builtin_elementwise_maximum(t, 0.0f));
}

__device__ __forceinline__ f32x4 mfma(bf16x8 a, bf16x8 b, f32x4 c)
{
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 cat(bf16x4 lo, bf16x4 hi)
{
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// A fragment of W1 for neuron tile t: row 16t + r, K slots 0..7 (g = 0) and
// again 8..15 (g = 1), which multiply the high and low BF16 parts of x.
__device__ __forceinline__ bf16x8 frag_w1(const NetWeights &W, int t, int g, int r)
{
    const bf16x8 v = *reinterpret_cast<const bf16x8 *>(&W.w1[(16 * t + r) * kFeat]);
    const bf16x8 z = {};
    return g < 2 ? v : z;
}

// A fragment of M (w2 or w2t) for output tile t and K chunk c under the
// permuted K order: slots i' < 4 are columns 32c + 4g + i', slots i' >= 4 are
// columns 32c + 16 + 4g + i' - 4.
__device__ __forceinline__ bf16x8 frag_perm(const __bf16 *M, int t, int c, int g, int r)
{
    const __bf16 *row = M + (16 * t + r) * kRow2 + 32 * c + 4 * g;
    return cat(*reinterpret_cast<const bf16x4 *>(row), *reinterpret_cast<const bf16x4 *>(row + 16));
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// The BF16 roundings of a pair of values and of their remainders: hi + lo
// carries them to about 2^-16 relative.
__device__ __forceinline__ void split2(float x, float y, unsigned &hi, unsigned &lo)
{
    hi = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{x, y}, bf16x2));
    const float xl = x - __uint_as_float(hi << 16), yl = y - __uint_as_float(hi & 0xffff0000u);
    lo = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2{xl, yl}, bf16x2));
}

// B fragments of chunk c from a result held as v[t][i] (neuron 16t + 4g + i):
// hi gets the BF16 rounding, lo the BF16 rounding of the remainder.
__device__ __forceinline__ void frag_chunk(const float (&v)[4][4], int c, bf16x8 &hi, bf16x8 &lo)
{
    u32x4 h, l;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        unsigned a, b;
        split2(v[2 * c + k / 2][2 * (k % 2)], v[2 * c + k / 2][2 * (k % 2) + 1], a, b);
        h[k] = a;
        l[k] = b;
    }
    hi = __builtin_bit_cast(bf16x8, h);
    lo = __builtin_bit_cast(bf16x8, l);
}

// Single BF16 rounding (the backward contractions).
__device__ __forceinline__ bf16x8 frag_chunk1(const float (&v)[4][4], int c)
{
    bf16x8 b;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        b[i] = (__bf16)v[2 * c][i];
        b[4 + i] = (__bf16)v[2 * c + 1][i];
    }
    return b;
}

// B fragment of the input layer: the 8 features of row r, their BF16
// high parts in the slots of g = 0 and the low parts in those of g = 1.
__device__ __forceinline__ bf16x8 frag_x(const float *__restrict__ X, int64_t row, int64_t rows,
                                         int g)
{
    u32x4 b = {0, 0, 0, 0};
    if (g < 2 && row < rows) {
        const float4 *p = reinterpret_cast<const float4 *>(X + row * kFeat);
        const float4 u = p[0], v = p[1];
        const float f[8] = {u.x, u.y, u.z, u.w, v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            unsigned hi, lo;
            split2(f[2 * i], f[2 * i + 1], hi, lo);
            b[i] = g == 0 ? hi : lo;
        }
    }
    return __builtin_bit_cast(bf16x8, b);
}

// Forward pass of 16 rows; a1/a2 get the pre-activations (neuron 16t+4g+i of
// this lane's row), h1b the BF16 high parts of h1 as B fragments, h2 the
// second activations; the return value is the logit of row r in every lane.
// TRAIN: the activation whose terms the derivative shares, and biases added to
// the products (the forward pass starts the products from them; a gradient's
// BF16 roundings would turn over with the last bit of an activation).
template <bool TRAIN>
__device__ __forceinline__ float forward16(const NetWeights &W, bf16x8 xb, int g, int r,
                                           float (&a1)[4][4], float (&a2)[4][4], bf16x8 (&h1b)[2],
                                           float (&h2)[4][4])
{
    float h1[4][4];
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const f32x4 bias = *reinterpret_cast<const f32x4 *>(&W.b1[16 * t + 4 * g]);
        const f32x4 d = mfma(frag_w1(W, t, g, r), xb, TRAIN ? f32x4{0.f, 0.f, 0.f, 0.f} : bias);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a1[t][i] = TRAIN ? d[i] + bias[i] : d[i];
            h1[t][i] = TRAIN ? gelu(a1[t][i]) : gelu_fast(a1[t][i]);
        }
    }
    bf16x8 h1l[2];
    frag_chunk(h1, 0, h1b[0], h1l[0]);
    frag_chunk(h1, 1, h1b[1], h1l[1]);
    float zp = 0.0f;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
        const bf16x8 w0 = frag_perm(W.w2, t, 0, g, r), w1 = frag_perm(W.w2, t, 1, g, r);
        const f32x4 bias = *reinterpret_cast<const f32x4 *>(&W.b2[16 * t + 4 * g]);
        f32x4 d = mfma(w0, h1b[0], TRAIN ? f32x4{0.f, 0.f, 0.f, 0.f} : bias);
        d = mfma(w1, h1b[1], d);
        d = mfma(w0, h1l[0], d);
        d = mfma(w1, h1l[1], d);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int nn = 16 * t + 4 * g + i;
            a2[t][i] = TRAIN ? d[i] + bias[i] : d[i];
            h2[t][i] = TRAIN ? gelu(a2[t][i]) : gelu_fast(a2[t][i]);
            zp += W.w3[nn] * h2[t][i];
        }
    }
    // sum over the four lane groups that share row r
    zp += __shfl_xor(zp, 16);
    zp += __shfl_xor(zp, 32);
    return zp + W.b3;
}

constexpr int kMlpBlock = 256;

// Bound by vector issue: per 16 rows 32 activations and the split of 24 values
// per lane against 20 matrix products.  The weight fragments and biases stay
// in registers over a wave's tiles (read from LDS per tile the kernel takes
// 70 us), the products start from the biases, and the bound of two waves per
// SIMD lets them land in vector registers (from accumulation registers every
// value is moved once more).  137 registers: three workgroups per CU.
// 524288 rows: 37 us, 63 us with the longer activation, added biases and a
// grid of four workgroups per CU, of which three were resident.
constexpr int kMlpPerCu = 3;

__global__ __launch_bounds__(kMlpBlock, 2) void mlp_forward_kernel(const float *__restrict__ P,
                                                                const float *__restrict__ X,
                                                                int64_t rows,
                                                                float *__restrict__ Z)
{
    __shared__ NetWeights W;
    load_weights<kMlpBlock>(P, W, false);
    __syncthreads();
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
    const int64_t waves = (int64_t)gridDim.x * (kMlpBlock / 64);
    const int64_t tiles = (rows + 15) / 16;
    for (int64_t tile = (int64_t)blockIdx.x * (kMlpBlock / 64) + (threadIdx.x >> 6); tile < tiles;
         tile += waves) {
        const int64_t row = tile * 16 + r;
        float a1[4][4], a2[4][4], h2[4][4];
        bf16x8 h1b[2];
        const float z = forward16<false>(W, frag_x(X, row, rows, g), g, r, a1, a2, h1b, h2);
        if (g == 0 && row < rows) Z[row] = z;
    }
}

// ---------------------------------------------------------------------------
// Backward
// ---------------------------------------------------------------------------
constexpr int kStageRow = 40;         // 32 rows and a pad against bank conflicts

struct WaveStage {                    // one per wave: 32 rows of the pair tile
    alignas(16) __bf16 da2[kHid][kStageRow];
    alignas(16) __bf16 h1[kHid][kStageRow];
    alignas(16) __bf16 da1[kHid][kStageRow];
    alignas(16) __bf16 x[16][kStageRow];     // features 8..15 stay zero
};

struct GradShared {
    NetWeights W;
    union {
        WaveStage stage[kMlpBlock / 64];
        float sum[kMlpBlock / 64][kParams + 1];   // the waves' sums after the row loop
    } u;
};

__device__ __forceinline__ float sum16(float v)   // over the 16 lanes of a group
{
    v += dpp<kDppXor1>(v);
    v += dpp<kDppXor2>(v);
    v += dpp<kDppHalfMirror>(v);
    v += dpp<kDppRowMirror>(v);
    return v;
}

// Bound by latency at a minibatch (8192 rows: one tile of 32 rows per wave):
// the weights' loads are in flight together, their transposed copy and the
// staged tiles are laid out without bank conflicts, and the waves' sums meet
// in LDS in one step instead of a read-modify-write chain of 130 values per
// lane and wave.  8192 rows: 12.7 us (32 us before); with the update in the
// reduction (4 us) a training step takes 15 us, 51 us before.
// Per workgroup: partial d(sum of row losses)/d params (not yet divided by
// rows) and the partial loss sum, written to part[blockIdx.x][0..kParams].
template <int TILES>
__global__ __launch_bounds__(kMlpBlock) void mlp_grad_kernel(const float *__restrict__ P,
                                                             const float *__restrict__ X,
                                                             const float *__restrict__ Y,
                                                             int64_t rows,
                                                             float *__restrict__ part,
                                                             int32_t *__restrict__ step)
{
    __shared__ GradShared S;
    load_weights<kMlpBlock>(P, S.W, true);
    const NetWeights &W = S.W;
    const int wv = threadIdx.x >> 6;
    const int lane = threadIdx.x & 63, g = lane >> 4, r = lane & 15;
    WaveStage &st = S.u.stage[wv];
    if constexpr (TILES == 1) {
        // the second 16 rows of the contractions stay zero
        for (int k = lane; k < (int)(sizeof(WaveStage) / 16); k += 64)
            reinterpret_cast<u32x4 *>(&st)[k] = u32x4{0, 0, 0, 0};
    } else {
        for (int k = lane; k < 16 * kStageRow; k += 64) (&st.x[0][0])[k] = (__bf16)0.0f;
    }
    __syncthreads();

    f32x4 gW2[4][4], gW1[4];
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        gW1[a] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int b = 0; b < 4; ++b) gW2[a][b] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    float gW3[4][4] = {}, gB2[4][4] = {}, gB1[4][4] = {};
    float gB3 = 0.0f, lsum = 0.0f;

    const int64_t waves = (int64_t)gridDim.x * (kMlpBlock / 64);
    const int64_t pairs = (rows + 16 * TILES - 1) / (16 * TILES);
    for (int64_t pt = (int64_t)blockIdx.x * (kMlpBlock / 64) + wv; pt < pairs; pt += waves) {
#pragma unroll
        for (int s = 0; s < TILES; ++s) {
            const int64_t row = (pt * TILES + s) * 16 + r;
            const bool valid = row < rows;
            const bf16x8 xb = frag_x(X, row, rows, g);
            float a1[4][4], a2[4][4], h2[4][4];
            bf16x8 h1b[2];
            const float z = forward16<true>(W, xb, g, r, a1, a2, h1b, h2);
            const float y = valid ? Y[row] : 0.0f;
            const float dz = valid ? 1.0f / (1.0f + __expf(-z)) - y : 0.0f;
            if (g == 0 && valid) {
                lsum += fmaxf(z, 0.0f) - z * y + log1pf(__expf(-fabsf(z)));
                gB3 += dz;
            }
            float da2[4][4];
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int nn = 16 * t + 4 * g + i;
                    gW3[t][i] += dz * h2[t][i];
                    da2[t][i] = dz * W.w3[nn] * gelu_prime(a2[t][i]);
                    gB2[t][i] += da2[t][i];
                }
            // dh1 = W2^T da2 (same permuted K order as the forward)
            const bf16x8 db0 = frag_chunk1(da2, 0), db1 = frag_chunk1(da2, 1);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                f32x4 d = mfma(frag_perm(W.w2t, t, 0, g, r), db0, f32x4{0.f, 0.f, 0.f, 0.f});
                d = mfma(frag_perm(W.w2t, t, 1, g, r), db1, d);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int nn = 16 * t + 4 * g + i;
                    const float da1 = d[i] * gelu_prime(a1[t][i]);
                    gB1[t][i] += da1;
                    st.da1[nn][16 * s + r] = (__bf16)da1;
                }
            }
#pragma unroll
            for (int t = 0; t < 4; ++t)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int nn = 16 * t + 4 * g + i;
                    st.da2[nn][16 * s + r] = (__bf16)da2[t][i];
                    st.h1[nn][16 * s + r] = (t & 1) ? h1b[t >> 1][4 + i] : h1b[t >> 1][i];
                }
            if (g == 0) {
#pragma unroll
                for (int f = 0; f < 8; ++f) st.x[f][16 * s + r] = xb[f];
            }
        }
        wave_sync();
        // dW2[n][k] += sum_rows da2[n][row] h1[k][row]; dW1[n][f] likewise with x
#pragma unroll
        for (int tn = 0; tn < 4; ++tn) {
            const bf16x8 a = *reinterpret_cast<const bf16x8 *>(&st.da2[16 * tn + r][8 * g]);
#pragma unroll
            for (int tk = 0; tk < 4; ++tk) {
                const bf16x8 b = *reinterpret_cast<const bf16x8 *>(&st.h1[16 * tk + r][8 * g]);
                gW2[tn][tk] = mfma(a, b, gW2[tn][tk]);
            }
            const bf16x8 a1f = *reinterpret_cast<const bf16x8 *>(&st.da1[16 * tn + r][8 * g]);
            const bf16x8 xf = *reinterpret_cast<const bf16x8 *>(&st.x[r][8 * g]);
            gW1[tn] = mfma(a1f, xf, gW1[tn]);
        }
        wave_sync();
    }

    // ---- workgroup reduction in a fixed order: every wave stores its sums,
    // the threads add them in the order of the waves
    __syncthreads();                  // the stages are dead; reuse as sum[][]
    float *sum = S.u.sum[wv];
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            gW3[t][i] = sum16(gW3[t][i]);
            gB2[t][i] = sum16(gB2[t][i]);
            gB1[t][i] = sum16(gB1[t][i]);
        }
    gB3 = sum16(gB3);
    lsum = sum16(lsum);
#pragma unroll
    for (int tn = 0; tn < 4; ++tn)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int nn = 16 * tn + 4 * g + i;
#pragma unroll
            for (int tk = 0; tk < 4; ++tk) sum[oW2 + nn * kHid + 16 * tk + r] = gW2[tn][tk][i];
            if (r < kFeat) sum[oW1 + nn * kFeat + r] = gW1[tn][i];
            if (r == 0) {
                sum[oW3 + nn] = gW3[tn][i];
                sum[oB2 + nn] = gB2[tn][i];
                sum[oB1 + nn] = gB1[tn][i];
            }
        }
    if (lane == 0) {
        sum[oB3] = gB3;
        sum[kParams] = lsum;
    }
    __syncthreads();
    float *dst = part + (int64_t)blockIdx.x * (kParams + 1);
    for (int k = threadIdx.x; k <= kParams; k += kMlpBlock) {
        float v = S.u.sum[0][k];
#pragma unroll
        for (int w = 1; w < kMlpBlock / 64; ++w) v += S.u.sum[w][k];
        dst[k] = v;
    }
    // the optimizer's step count, for the update that follows
    if (step && blockIdx.x == 0 && threadIdx.x == 0) *step += 1;
}

// ---------------------------------------------------------------------------
// Adam
// ---------------------------------------------------------------------------
// 1 - beta^t of both moments
__device__ __forceinline__ float2 adam_bias(const AdamArgs &a, int t)
{
    return make_float2((float)(1.0 - pow((double)a.b1, (double)t)),
                       (float)(1.0 - pow((double)a.b2, (double)t)));
}

// pk, m0, v0: the parameter and its moments before the step
__device__ __forceinline__ void adam_update(float *__restrict__ p, float *__restrict__ m,
                                            float *__restrict__ v, float pk, float m0, float v0,
                                            float gk, float2 bias, const AdamArgs &a, int k)
{
    const float mk = a.b1 * m0 + (1.0f - a.b1) * gk;
    const float vk = a.b2 * v0 + (1.0f - a.b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    p[k] = pk - a.lr * (mk / bias.x) / (sqrtf(vk / bias.y) + a.eps);
}

// grad[k] = (sum over workgroups) / rows; loss likewise.  ADAM: and the update
// of parameter k, with the count in *step.  Four waves take a quarter of the
// parts of 64 entries each, in order, 16 loads in flight, and the quarters are
// added in order (one thread per entry and one load at a time: 16 us for 64
// parts; 4 us for 128 in this form); a fifth computes the moments' factors
// meanwhile.
constexpr int kReduceSplit = 4;
constexpr int kReduceBlock = (kReduceSplit + 1) * kWave;

template <bool ADAM>
__global__ __launch_bounds__(kReduceBlock) void grad_reduce_kernel(
    const float *__restrict__ part, int nparts, int64_t rows, float *__restrict__ grad,
    float *__restrict__ loss, float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
    const int32_t *__restrict__ step, AdamArgs a)
{
    __shared__ float quarter[kReduceSplit][kWave];
    __shared__ float2 bias;
    const int lane = threadIdx.x & (kWave - 1), w = threadIdx.x / kWave;
    const int k = blockIdx.x * kWave + lane, kc = min(k, kParams);
    float pk = 0.f, m0 = 0.f, v0 = 0.f;
    if (w < kReduceSplit) {
        if (ADAM && w == 0 && k < kParams) { pk = p[k]; m0 = m[k]; v0 = v[k]; }
        const int w0 = nparts * w / kReduceSplit, w1 = nparts * (w + 1) / kReduceSplit;
        constexpr int kFly = 16;
        float s = 0.0f;
        for (int q0 = w0; q0 < w1; q0 += kFly) {
            float x[kFly];
#pragma unroll
            for (int q = 0; q < kFly; ++q) x[q] = part[(int64_t)min(q0 + q, w1 - 1) * (kParams + 1) + kc];
#pragma unroll
            for (int q = 0; q < kFly; ++q)
                if (q0 + q < w1) s += x[q];
        }
        quarter[w][lane] = s;
    } else if (ADAM && lane == 0) {
        bias = adam_bias(a, *step);
    }
    __syncthreads();
    if (w > 0 || k > kParams) return;
    float s = quarter[0][lane];
#pragma unroll
    for (int q = 1; q < kReduceSplit; ++q) s += quarter[q][lane];
    const float mean = rows > 0 ? s / (float)rows : 0.0f;
    if (k < kParams) {
        grad[k] = mean;
        if constexpr (ADAM) adam_update(p, m, v, pk, m0, v0, mean, bias, a, k);
    } else if (loss) {
        *loss = mean;
    }
}

// An update by itself: step counter on the device, t = *step + 1 is used,
// then stored.
__global__ void adam_kernel(float *__restrict__ p, float *__restrict__ m, float *__restrict__ v,
                            const float *__restrict__ g, const int32_t *__restrict__ step,
                            AdamArgs a, int count)
{
    const int k = blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= count) return;
    adam_update(p, m, v, p[k], m[k], v[k], g[k], adam_bias(a, *step + 1), a, k);
}

__global__ void step_bump_kernel(int32_t *step) { *step += 1; }

// ---------------------------------------------------------------------------
// Proposal: best candidate per circle by a 64-bit key (score, then lower
// candidate index), bitonic sort of the keys, first k taken.
// ---------------------------------------------------------------------------
constexpr int kPropBlock = 256;

__device__ __forceinline__ uint32_t ordered_bits(float s)
{
    s = s + 0.0f;                                  // -0 -> +0: equal scores tie
    const uint32_t u = __float_as_uint(s);
    return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

__global__ __launch_bounds__(kPropBlock) void propose_kernel(
    const int32_t *__restrict__ offset, const float *__restrict__ xy, int C,
    const int32_t *__restrict__ cand_circle, const float *__restrict__ cand_dest,
    const float *__restrict__ scores, int k, int32_t *__restrict__ selected,
    float *__restrict__ xy_out)
{
    __shared__ unsigned long long key[kMaxN];
    __shared__ int any_nan;
    const int b = blockIdx.x;
    const int o = offset[b];
    int n = offset[b + 1] - o;
    if (n < 0 || n > kMaxN) n = 0;
    const float2 *src = reinterpret_cast<const float2 *>(xy) + o;
    float2 *dst = reinterpret_cast<float2 *>(xy_out) + o;
    for (int i = threadIdx.x; i < n; i += kPropBlock) dst[i] = src[i];
    for (int i = threadIdx.x; i < kMaxN; i += kPropBlock) key[i] = 0ull;
    if (threadIdx.x == 0) any_nan = 0;
    __syncthreads();
    const int64_t base = (int64_t)b * C;
    if (scores) {
        for (int c = threadIdx.x; c < C; c += kPropBlock)
            if (scores[base + c] != scores[base + c]) any_nan = 1;
    }
    __syncthreads();
    const bool use = scores != nullptr && any_nan == 0;
    for (int c = threadIdx.x; c < C; c += kPropBlock) {
        const int i = cand_circle[base + c];
        if (i < 0 || i >= n) continue;
        const uint32_t hi = use ? ordered_bits(scores[base + c]) : 0x80000000u;
        const unsigned long long kk = ((unsigned long long)hi << 32) | (0xffffffffu - (uint32_t)c);
        atomicMax(&key[i], kk);
    }
    __syncthreads();
    for (int size = 2; size <= kMaxN; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            for (int t = threadIdx.x; t < kMaxN / 2; t += kPropBlock) {
                const int i = 2 * t - (t & (stride - 1));
                const int j = i + stride;
                const bool up = (i & size) == 0;
                const unsigned long long ki = key[i], kj = key[j];
                if ((ki > kj) == up) {
                    key[i] = kj;
                    key[j] = ki;
                }
            }
            __syncthreads();
        }
    }
    // ascending order: the best key is last
    for (int q = threadIdx.x; q < k; q += kPropBlock) {
        const unsigned long long kk = q < kMaxN ? key[kMaxN - 1 - q] : 0ull;
        int32_t c = -1;
        if (kk != 0ull) {
            c = (int32_t)(0xffffffffu - (uint32_t)(kk & 0xffffffffull));
            const int i = cand_circle[base + c];
            dst[i] = reinterpret_cast<const float2 *>(cand_dest)[base + c];
        }
        if (selected) selected[(int64_t)b * k + q] = c;
    }
}

// ---------------------------------------------------------------------------
// Acceptance: keep the new layout of instance b when e_new[b] < e_cur[b].
// ---------------------------------------------------------------------------
constexpr int kAcceptBlock = 256;

__global__ __launch_bounds__(kAcceptBlock) void accept_kernel(
    const int32_t *__restrict__ offset, float *__restrict__ xy_cur, double *__restrict__ e_cur,
    const float *__restrict__ xy_new, const double *__restrict__ e_new,
    int32_t *__restrict__ accepted)
{
    const int b = blockIdx.x;
    const int o = offset[b];
    int n = offset[b + 1] - o;
    if (n < 0 || n > kMaxN) n = 0;
    const double en = e_new[b], ec = e_cur[b];
    const bool take = en < ec;
    __syncthreads();                 // every thread has read e_cur[b]
    if (take) {
        const float2 *src = reinterpret_cast<const float2 *>(xy_new) + o;
        float2 *dst = reinterpret_cast<float2 *>(xy_cur) + o;
        for (int i = threadIdx.x; i < n; i += kAcceptBlock) dst[i] = src[i];
    }
    if (threadIdx.x == 0) {
        if (take) e_cur[b] = en;
        if (accepted) accepted[b] = take ? 1 : 0;
    }
}

// 16-row tiles of a wave's turn in the gradient: one while that leaves no more
// workgroups than CUs (a minibatch is a single turn, and half the turn's
// chain), two beyond, where the contractions over rows then fill their 32
// places.  8192 rows: 12.7 us with one, 16 us with two.
int mlp_tiles(int64_t rows) { return rows <= 256 * 4 * 16 ? 1 : 2; }

int mlp_grid(int64_t rows)
{
    const int per_wg_rows = (kMlpBlock / 64) * 16 * mlp_tiles(rows);
    const int64_t need = (rows + per_wg_rows - 1) / per_wg_rows;
    return (int)(need < 1 ? 1 : (need > 256 ? 256 : need));
}

void run_mlp_grad(const float *params, const float *X, const float *Y, int64_t rows, float *part,
                  int32_t *step, hipStream_t s)
{
    const int grid = mlp_grid(rows);
    if (mlp_tiles(rows) == 1)
        mlp_grad_kernel<1><<<grid, kMlpBlock, 0, s>>>(params, X, Y, rows, part, step);
    else
        mlp_grad_kernel<2><<<grid, kMlpBlock, 0, s>>>(params, X, Y, rows, part, step);
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_features(const int32_t *offset, const float *R, const double *R64,
                           const float *xy, int B, int C, const int32_t *cand_circle,
                           const float *cand_dest, float *feat, hipStream_t s)
{
    if (B <= 0 || C <= 0) return hipSuccess;
    dim3 grid((C + kFeatChunk - 1) / kFeatChunk, B);
    // half the threads where they cover the candidates of an instance and there
    // are more instances than CUs: 2048 instances with 64 candidates, n = 10
    // 17.7 us (21.8 with 512 threads), n = 1000 28.3 us (32.7); one instance of
    // n = 1000 sorts its circles faster with 512 (10.8 us, 11.2 with 256)
    if (C <= kFeatBlock / 2 && B > 256)
        features_kernel<kFeatBlock / 2><<<grid, kFeatBlock / 2, 0, s>>>(offset, R, R64, xy, C,
                                                                     cand_circle, cand_dest, feat);
    else
        features_kernel<kFeatBlock><<<grid, kFeatBlock, 0, s>>>(offset, R, R64, xy, C, cand_circle,
                                                                cand_dest, feat);
    return hipGetLastError();
}

hipError_t launch_mlp_forward(const float *params, const float *X, int64_t rows, float *Z,
                              hipStream_t s)
{
    if (rows <= 0) return hipSuccess;
    // at least two 16-row tiles per wave, and no more workgroups than are
    // resident: each loads the weights
    const int64_t need = (rows + 4 * 32 - 1) / (4 * 32);
    const int grid = (int)(need > kMlpPerCu * 256 ? kMlpPerCu * 256 : need);
    hipLaunchKernelGGL(mlp_forward_kernel, dim3(grid), dim3(kMlpBlock), 0, s, params, X, rows, Z);
    return hipGetLastError();
}

size_t mlp_grad_workspace_bytes(int64_t rows)
{
    // enough for every smaller row count too: the most workgroups once they
    // take two tiles
    const int parts = mlp_tiles(rows) == 1 ? mlp_grid(rows) : 256;
    return (size_t)parts * (kParams + 1) * sizeof(float);
}

hipError_t launch_mlp_grad(const float *params, const float *X, const float *Y, int64_t rows,
                           float *loss, float *grad, void *ws, hipStream_t s)
{
    const int grid = mlp_grid(rows);
    float *part = static_cast<float *>(ws);
    run_mlp_grad(params, X, Y, rows, part, nullptr, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    grad_reduce_kernel<false><<<kParams / kWave + 1, kReduceBlock, 0, s>>>(
        part, grid, rows, grad, loss, nullptr, nullptr, nullptr, nullptr, AdamArgs{});
    return hipGetLastError();
}

hipError_t launch_train_step(float *params, float *m, float *v, int32_t *step, const AdamArgs &a,
                             const float *X, const float *Y, int64_t rows, float *loss, float *grad,
                             void *ws, hipStream_t s)
{
    const int grid = mlp_grid(rows);
    float *part = static_cast<float *>(ws);
    run_mlp_grad(params, X, Y, rows, part, step, s);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    grad_reduce_kernel<true><<<kParams / kWave + 1, kReduceBlock, 0, s>>>(
        part, grid, rows, grad, loss, params, m, v, step, a);
    return hipGetLastError();
}

hipError_t launch_adam(float *params, float *m, float *v, const float *grad, int32_t *step,
                       const AdamArgs &a, hipStream_t s)
{
    hipLaunchKernelGGL(adam_kernel, dim3((kParams + 255) / 256), dim3(256), 0, s, params, m, v,
                       grad, step, a, kParams);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(step_bump_kernel, dim3(1), dim3(1), 0, s, step);
    return hipGetLastError();
}

hipError_t launch_propose(const int32_t *offset, const float *xy, int B, int C,
                          const int32_t *cand_circle, const float *cand_dest, const float *scores,
                          int k, int32_t *selected, float *xy_out, hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(propose_kernel, dim3(B), dim3(kPropBlock), 0, s, offset, xy, C,
                       cand_circle, cand_dest, scores, k, selected, xy_out);
    return hipGetLastError();
}

hipError_t launch_accept(const int32_t *offset, float *xy_cur, double *e_cur, const float *xy_new,
                         const double *e_new, int B, int32_t *accepted, hipStream_t s)
{
    if (B <= 0) return hipSuccess;
    hipLaunchKernelGGL(accept_kernel, dim3(B), dim3(kAcceptBlock), 0, s, offset, xy_cur, e_cur,
                       xy_new, e_new, accepted);
    return hipGetLastError();
}

}  // namespace pecc
