// L-BFGS building blocks shared by the descent kernels: the slot layout of
// the fused reduction, DPP wave reductions, the wave reduce-scatter, the
// Gram-matrix update rule, the pair terms and the pre-tested neighbor
// predicate.  gfx950 (wave64) only.
#pragma once
#include "pecc_device.hpp"

#include <type_traits>

namespace pecc {

// A place beyond everything: a pair term with it is zero.
constexpr float kFarCoord = 3.0e18f;      // (3e18)^2 * 2 is finite in FP32

constexpr int kMM = 10;                   // history slots (max m)
constexpr int kNB = 2 * kMM + 1;          // basis size: s_0..s_9, y_0..y_9, g
constexpr int kG = 2 * kMM;               // basis index of g

// Slots of the fused reduction.  gt: trial gradient, sc = xt - x, yc = gt - g.
constexpr int sGS(int j) { return j; }                      // gt . s_j
constexpr int sGY(int j) { return kMM + j; }                // gt . y_j
constexpr int sSS(int j) { return 2 * kMM + j - 1; }        // sc . s_j   (j >= 1)
constexpr int sSY(int j) { return 3 * kMM - 1 + j - 1; }    // sc . y_j   (j >= 1)
constexpr int sYS(int j) { return 4 * kMM - 2 + j - 1; }    // yc . s_j   (j >= 1)
constexpr int sYY(int j) { return 5 * kMM - 3 + j - 1; }    // yc . y_j   (j >= 1)
constexpr int sGG = 6 * kMM - 4;                            // gt . gt
constexpr int sScSc = sGG + 1;                              // sc . sc
constexpr int sScYc = sGG + 2;                              // sc . yc
constexpr int sYcYc = sGG + 3;                              // yc . yc
constexpr int sScG = sGG + 4;                               // sc . gt
constexpr int sYcG = sGG + 5;                               // yc . gt
constexpr int sE = sGG + 6;                                 // trial energy (radius rad)
constexpr int sE1 = sGG + 7;                                // trial energy of unit circles
static_assert(sE1 < kWave, "fused reduction must fit one slot per lane");

// Layout-identical mirror of pecc_descent_result, and its first 40 bytes.
struct DescentResultDev {
    int32_t status, iters, evals, rebuilds;
    int64_t pair_evals;
    float E32, gnorm;
    double E64;
    int32_t cell_evals, reserved;
};
struct DescentHead {
    int32_t status, iters, evals, rebuilds;
    int64_t pair_evals;
    float E32, gnorm;
    double E64;
};

// Writes the result of instance b: the head as one struct, then cell_evals
// and the reserved word.  (Kernels build the 40-byte head: a 48-byte local
// struct changes the descent kernel's register allocation -- spills, and in
// one instantiation a misaligned register pair the compiler rejects.)
__device__ __forceinline__ void store_result(DescentResultDev *out, int b, const DescentHead &r,
                                             int cell_evals)
{
    char *o = reinterpret_cast<char *>(out) + (size_t)b * sizeof(DescentResultDev);
    *reinterpret_cast<DescentHead *>(o) = r;
    *reinterpret_cast<int2 *>(o + sizeof(DescentHead)) = make_int2(cell_evals, 0);
}

// The result of an instance that is not descended (status BAD_INSTANCE,
// energies NaN, E64 = -1).  The constants pass through an empty asm so the
// compiler materialises them here, on this rare path, instead of keeping
// them in registers across the whole descent loop.
__device__ __forceinline__ void store_bad_instance(DescentResultDev *out, int b)
{
    float qnan = __builtin_nanf("");
    double m1 = -1.0;
    asm volatile("" : "+v"(qnan), "+v"(m1));
    DescentHead r = {};
    r.status = 7;
    r.E32 = qnan;
    r.gnorm = qnan;
    r.E64 = m1;
    store_result(out, b, r, 0);
}

// History elements: float2, or the same bits held as one 64-bit value (an
// aligned register pair, so that shifting the history moves pairs).
__device__ __forceinline__ float2 as_f2(float2 v) { return v; }
__device__ __forceinline__ float2 as_f2(double v) { return __builtin_bit_cast(float2, v); }
__device__ __forceinline__ double as_f64(float2 v) { return __hiloint2double(__float_as_int(v.y), __float_as_int(v.x)); }

// A circle's history pushed by one pair, in place (the value moves of the
// plain assignments are otherwise allocated to a second set of registers and
// copied back at the end of the loop body).  Early-clobbered: v is read last.
__device__ __forceinline__ void push_history(double (&H)[kMM], double v)
{
    asm("v_mov_b64 %0, %1\n\tv_mov_b64 %1, %2\n\tv_mov_b64 %2, %3\n\tv_mov_b64 %3, %4\n\t"
        "v_mov_b64 %4, %5\n\tv_mov_b64 %5, %6\n\tv_mov_b64 %6, %7\n\tv_mov_b64 %7, %8\n\t"
        "v_mov_b64 %8, %9\n\tv_mov_b64 %9, %10"
        : "+&v"(H[0]), "+&v"(H[1]), "+&v"(H[2]), "+&v"(H[3]), "+&v"(H[4]), "+&v"(H[5]), "+&v"(H[6]),
          "+&v"(H[7]), "+&v"(H[8]), "+&v"(H[9])
        : "v"(v));
}

// Products and sums of two products with their roundings written out.  Which
// product of a sum the compiler fuses is its choice, and it differs between
// instantiations of one kernel; these have the same bits in all of them.
//   mul_rounded  a * b, never fused
//   dot2         a b + c d as fma(a, b, c d)
template <typename T>
__device__ __forceinline__ T mul_rounded(T a, T b)
{
#pragma clang fp contract(off)
    return a * b;
}
__device__ __forceinline__ float dot2(float a, float b, float c, float d) { return fmaf(a, b, mul_rounded(c, d)); }
__device__ __forceinline__ double dot2(double a, double b, double c, double d) { return fma(a, b, mul_rounded(c, d)); }

// Value of reduction slot v summed over this thread's circles (v is a
// constant after unrolling, so the branches fold away): one FMA chain over
// the circles' coordinates, started by a product.
template <int CPT, typename HV>
__device__ __forceinline__ float slot_value(int v, const float2 (&gt)[CPT], const float2 (&sc)[CPT],
                                            const float2 (&yc)[CPT],
                                            const HV (&S)[CPT][kMM],
                                            const HV (&Y)[CPT][kMM], float e, float e1)
{
    if (v == sE) return e;
    if (v == sE1) return e1;
    float acc = 0.f;
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        float2 a, b;
        if (v < kMM) { a = gt[c]; b = as_f2(S[c][v]); }
        else if (v < 2 * kMM) { a = gt[c]; b = as_f2(Y[c][v - kMM]); }
        else if (v < 3 * kMM - 1) { a = sc[c]; b = as_f2(S[c][v - 2 * kMM + 1]); }
        else if (v < 4 * kMM - 2) { a = sc[c]; b = as_f2(Y[c][v - (3 * kMM - 1) + 1]); }
        else if (v < 5 * kMM - 3) { a = yc[c]; b = as_f2(S[c][v - (4 * kMM - 2) + 1]); }
        else if (v < 6 * kMM - 4) { a = yc[c]; b = as_f2(Y[c][v - (5 * kMM - 3) + 1]); }
        else if (v == sGG) { a = gt[c]; b = gt[c]; }
        else if (v == sScSc) { a = sc[c]; b = sc[c]; }
        else if (v == sScYc) { a = sc[c]; b = yc[c]; }
        else if (v == sYcYc) { a = yc[c]; b = yc[c]; }
        else if (v == sScG) { a = sc[c]; b = gt[c]; }
        else { a = yc[c]; b = gt[c]; }   // sYcG
        acc = c == 0 ? a.x * b.x : fmaf(a.x, b.x, acc);
        acc = fmaf(a.y, b.y, acc);
    }
    return acc;
}

// ---------------------------------------------------------------------------
// Cross-lane moves.  DPP (data-parallel primitives) patterns run at VALU
// rate; quad_perm and the row mirrors stay inside 16-lane rows, row_bcast
// crosses rows.  Lane builtins work on 32-bit integers, so floats travel as
// bit patterns.
// ---------------------------------------------------------------------------
constexpr int kDppXor1 = 0xB1;        // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;        // quad_perm [2,3,0,1]
constexpr int kDppRowMirror = 0x140;  // lane i <- 15-i inside a row
constexpr int kDppHalfMirror = 0x141; // lane i <- 7-i inside half a row
constexpr int kDppBcast15 = 0x142;    // lane 15 of row r -> row r+1
constexpr int kDppBcast31 = 0x143;    // lane 31 -> rows 2 and 3

template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ float dpp(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v),
                                                                 CTRL, ROW_MASK, 0xf, false));
}

__device__ __forceinline__ float uniform_first(float v)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, v)));
}
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, v), l));
}

__device__ __forceinline__ double lane_value64(double v, int l)
{
    const long long bits = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(bits & 0xffffffffLL), l);
    const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), l);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// Sum over the 64 lanes, returned wave-uniform.  Every wave adds in the same
// order, so every wave gets the same bits.
__device__ __forceinline__ float wave_sum_dpp(float v)
{
    v += dpp<kDppXor1>(v);
    v += dpp<kDppXor2>(v);
    v += dpp<kDppHalfMirror>(v);
    v += dpp<kDppRowMirror>(v);          // every lane of a row holds the row sum
    v += dpp<kDppBcast15, 0xa>(v);       // rows 1, 3 add rows 0, 2
    v += dpp<kDppBcast31, 0xc>(v);       // rows 2, 3 add lane 31 (rows 0 + 1)
    return lane_value(v, 63);
}

// The two halves of the two-loop recursion on the Gram matrix (ten pairs,
// lane l holding row l of it): per step one product, its lane's value to a
// scalar, one FMA on every lane, and the scalar written into the one lane of
// cf that keeps it (in the wait state between the product and its lane read).
//   down, j = 9 .. 0:  a = lane j of rho * acc;         acc -= a * b[j];  lane 10 + j of cf = a
//   up,   j = 0 .. 9:  a = lane 10 + j of cf - rho acc;  acc += a * b[j];  lane j of cf = a
// In asm because the language has no lane write here (a compare, a move and
// a select per step take twice the chain's own instructions).  The wait
// states are those of a VALU result read by v_readlane (one) and of an SGPR
// it wrote read by a VALU instruction (two).
#define PECC_LOOP_STEP(FIRST, FILL, SRC, S, SIGN, J)                                                  \
    FIRST "\n\t" FILL "\n\tv_readlane_b32 %[" S "], %[t], " #SRC "\n\ts_nop 1\n\tv_fma_f32 %[acc], " SIGN \
    "%[b" #J "], %[" S "], %[acc]\n\t"
#define PECC_LOOP_KEEP(S, L) "v_writelane_b32 %[cf], %[" S "], " #L
#define PECC_DOWN(FILL, S, J) PECC_LOOP_STEP("v_mul_f32 %[t], %[rho], %[acc]", FILL, J, S, "-", J)
#define PECC_UP(FILL, SRC, S, J) PECC_LOOP_STEP("v_fma_f32 %[t], -%[rho], %[acc], %[cf]", FILL, SRC, S, "", J)
#define PECC_LOOP_OPERANDS                                                                            \
    : [acc] "+&v"(acc), [cf] "+&v"(cf), [t] "=&v"(t), [s0] "=&s"(s0), [s1] "=&s"(s1)                    \
    : [rho] "v"(rho), [b0] "v"(b[0]), [b1] "v"(b[1]), [b2] "v"(b[2]), [b3] "v"(b[3]), [b4] "v"(b[4]), \
      [b5] "v"(b[5]), [b6] "v"(b[6]), [b7] "v"(b[7]), [b8] "v"(b[8]), [b9] "v"(b[9])
__device__ __forceinline__ void two_loop_down(const float *b, float rho, float &acc, float &cf)
{
    float t;
    int s0, s1;
    asm(PECC_DOWN("s_nop 0", "s0", 9)
        PECC_DOWN(PECC_LOOP_KEEP("s0", 19), "s1", 8)
        PECC_DOWN(PECC_LOOP_KEEP("s1", 18), "s0", 7)
        PECC_DOWN(PECC_LOOP_KEEP("s0", 17), "s1", 6)
        PECC_DOWN(PECC_LOOP_KEEP("s1", 16), "s0", 5)
        PECC_DOWN(PECC_LOOP_KEEP("s0", 15), "s1", 4)
        PECC_DOWN(PECC_LOOP_KEEP("s1", 14), "s0", 3)
        PECC_DOWN(PECC_LOOP_KEEP("s0", 13), "s1", 2)
        PECC_DOWN(PECC_LOOP_KEEP("s1", 12), "s0", 1)
        PECC_DOWN(PECC_LOOP_KEEP("s0", 11), "s1", 0)
        PECC_LOOP_KEEP("s1", 10) "\n\ts_nop 0"
        PECC_LOOP_OPERANDS);
    (void)t;
    (void)s0;
    (void)s1;
}
__device__ __forceinline__ void two_loop_up(const float *b, float rho, float &acc, float &cf)
{
    float t;
    int s0, s1;
    asm(PECC_UP("s_nop 0", 10, "s0", 0)
        PECC_UP(PECC_LOOP_KEEP("s0", 0), 11, "s1", 1)
        PECC_UP(PECC_LOOP_KEEP("s1", 1), 12, "s0", 2)
        PECC_UP(PECC_LOOP_KEEP("s0", 2), 13, "s1", 3)
        PECC_UP(PECC_LOOP_KEEP("s1", 3), 14, "s0", 4)
        PECC_UP(PECC_LOOP_KEEP("s0", 4), 15, "s1", 5)
        PECC_UP(PECC_LOOP_KEEP("s1", 5), 16, "s0", 6)
        PECC_UP(PECC_LOOP_KEEP("s0", 6), 17, "s1", 7)
        PECC_UP(PECC_LOOP_KEEP("s1", 7), 18, "s0", 8)
        PECC_UP(PECC_LOOP_KEEP("s0", 8), 19, "s1", 9)
        PECC_LOOP_KEEP("s1", 9) "\n\ts_nop 0"
        PECC_LOOP_OPERANDS);
    (void)t;
    (void)s0;
    (void)s1;
}

// Maximum of a non-negative int over the 64 lanes, returned wave-uniform
// (lanes a DPP pattern leaves out read 0, which no value is below).
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ int dppi(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, CTRL, ROW_MASK, 0xf, false);
}
__device__ __forceinline__ int wave_max_dpp(int v)
{
    v = max(v, dppi<kDppXor1>(v));
    v = max(v, dppi<kDppXor2>(v));
    v = max(v, dppi<kDppHalfMirror>(v));
    v = max(v, dppi<kDppRowMirror>(v));
    v = max(v, dppi<kDppBcast15, 0xa>(v));
    v = max(v, dppi<kDppBcast31, 0xc>(v));
    return __builtin_amdgcn_readlane(v, 63);
}

// Sum of an int over the 64 lanes (exact), returned wave-uniform.
__device__ __forceinline__ int wave_sum_int(int v)
{
    v += dppi<kDppXor1>(v);
    v += dppi<kDppXor2>(v);
    v += dppi<kDppHalfMirror>(v);
    v += dppi<kDppRowMirror>(v);
    v += dppi<kDppBcast15, 0xa>(v);
    v += dppi<kDppBcast31, 0xc>(v);
    return __builtin_amdgcn_readlane(v, 63);
}

// Inclusive prefix sum of an int over the 64 lanes (row shifts inside the
// 16-lane rows, then the row totals passed on).
__device__ __forceinline__ int wave_scan_dpp(int v)
{
    v += dppi<0x111>(v);                 // row_shr 1, 2, 4, 8
    v += dppi<0x112>(v);
    v += dppi<0x114>(v);
    v += dppi<0x118>(v);
    v += dppi<kDppBcast15, 0xa>(v);
    v += dppi<kDppBcast31, 0xc>(v);
    return v;
}

// The same sum for a double: each DPP step moves the two 32-bit halves.
template <int CTRL, int ROW_MASK = 0xf>
__device__ __forceinline__ double dpp64(double v)
{
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), CTRL, ROW_MASK, 0xf, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROW_MASK, 0xf, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

__device__ __forceinline__ double wave_sum_dpp(double v)
{
    v += dpp64<kDppXor1>(v);
    v += dpp64<kDppXor2>(v);
    v += dpp64<kDppHalfMirror>(v);
    v += dpp64<kDppRowMirror>(v);
    v += dpp64<kDppBcast15, 0xa>(v);
    v += dpp64<kDppBcast31, 0xc>(v);
    const long long b = __builtin_bit_cast(long long, v);
    const int lo = __builtin_amdgcn_readlane((int)(b & 0xffffffffLL), 63);
    const int hi = __builtin_amdgcn_readlane((int)(b >> 32), 63);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (long long)(unsigned)lo);
}

// Maximum of a non-negative double over the 64 lanes (NaN is passed over),
// returned wave-uniform.
__device__ __forceinline__ double wave_max_dpp(double v)
{
    v = fmax(v, dpp64<kDppXor1>(v));
    v = fmax(v, dpp64<kDppXor2>(v));
    v = fmax(v, dpp64<kDppHalfMirror>(v));
    v = fmax(v, dpp64<kDppRowMirror>(v));
    v = fmax(v, dpp64<kDppBcast15, 0xa>(v));
    v = fmax(v, dpp64<kDppBcast31, 0xc>(v));
    return lane_value64(v, 63);
}

// Slot held by lane L after wave_reduce_scatter: slot L.
__device__ __forceinline__ int lane_slot(int L) { return L; }

// Half swaps between two registers (gfx950 VALU permutes).  swap32: a keeps
// its lanes 0-31 and receives b's lanes 0-31 in lanes 32-63; b receives a's
// lanes 32-63 in lanes 0-31 and keeps its lanes 32-63.  swap16: the same on
// 16-lane rows (a keeps rows 0, 2 and receives b's rows 0, 2 in rows 1, 3; b
// receives a's rows 1, 3 and keeps its rows 1, 3).  Written as asm because
// the builtins return one register twice in this compiler; the two wait
// states cover a VALU write of an operand just before, once for all the
// pairs of a call (the wait states are idle issue cycles: a third of the
// stage's time while every pair had its own).
__device__ __forceinline__ void swap32(float (&a)[4], float (&b)[4])
{
    asm("s_nop 1\n\tv_permlane32_swap_b32 %0, %4\n\tv_permlane32_swap_b32 %1, %5\n\t"
        "v_permlane32_swap_b32 %2, %6\n\tv_permlane32_swap_b32 %3, %7"
        : "+v"(a[0]), "+v"(a[1]), "+v"(a[2]), "+v"(a[3]), "+v"(b[0]), "+v"(b[1]), "+v"(b[2]), "+v"(b[3]));
}
__device__ __forceinline__ void swap16(float &a0, float &b0, float &a1, float &b1)
{
    asm("s_nop 1\n\tv_permlane16_swap_b32 %0, %1\n\tv_permlane16_swap_b32 %2, %3"
        : "+v"(a0), "+v"(b0), "+v"(a1), "+v"(b1));
}

// Reduce-scatter of the 64 slot values over the wave: afterwards lane L
// holds the wave sum of slot L.  Each stage halves the values per lane by
// pairing slots that differ in one bit with lanes that differ in the same
// bit: bit 5 and bit 4 by half swaps (slot q and q + 32 swapped between the
// wave halves, then added: one swap and one add per pair), bits 3, 2, 1, 0
// by DPP inside 16-lane rows (row mirror, half mirror, xor 2, xor 1; the lane
// whose bit is set keeps the upper slot).  Slots are produced in groups of
// eight (u + 8k, k = 0..7) that the first three stages consume, so only a
// few values are live at once.
template <bool STREAM, int CPT, typename HV>
__device__ __forceinline__ float wave_reduce_scatter(const float2 (&gt)[CPT],
                                                     const float2 (&sc)[CPT],
                                                     const float2 (&yc)[CPT],
                                                     const HV (&S)[CPT][kMM],
                                                     const HV (&Y)[CPT][kMM], float e,
                                                     float e1)
{
    const int lane = threadIdx.x & (kWave - 1);
    const bool b3 = (lane & 8) != 0, b2 = (lane & 4) != 0, b1 = (lane & 2) != 0;
    const bool b0 = (lane & 1) != 0;
    float h[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
        float w[4], lo[4], hi[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            lo[k] = slot_value(u + 8 * k, gt, sc, yc, S, Y, e, e1);
            hi[k] = slot_value(u + 8 * k + 32, gt, sc, yc, S, Y, e, e1);
        }
        swap32(lo, hi);
#pragma unroll
        for (int k = 0; k < 4; ++k) w[k] = lo[k] + hi[k];   // lanes 0-31: slot u + 8k, lanes 32-63: + 32
        swap16(w[0], w[2], w[1], w[3]);
        // rows 0, 2: slot of w[k]; rows 1, 3: + 16
        const float v[2] = {w[0] + w[2], w[1] + w[3]};
        h[u] = (b3 ? v[1] : v[0]) + dpp<kDppRowMirror>(b3 ? v[0] : v[1]);
        // STREAM: the next group is not hoisted above here (few values live
        // at once; without it the groups overlap, which a lone wave per SIMD
        // needs against the eight cycles of a dependent VALU instruction)
        if constexpr (STREAM) __builtin_amdgcn_sched_barrier(0);
    }
    float t4[4];
#pragma unroll
    for (int v = 0; v < 4; ++v) t4[v] = (b2 ? h[v + 4] : h[v]) + dpp<kDppHalfMirror>(b2 ? h[v] : h[v + 4]);
    float t2[2];
#pragma unroll
    for (int v = 0; v < 2; ++v) t2[v] = (b1 ? t4[v + 2] : t4[v]) + dpp<kDppXor2>(b1 ? t4[v] : t4[v + 2]);
    return (b0 ? t2[1] : t2[0]) + dpp<kDppXor1>(b0 ? t2[0] : t2[1]);
}

// Which vector basis index a of the updated basis is: 0 = an old basis
// vector (index in *old), 1 = sc, 2 = yc, 3 = gt.
__device__ __forceinline__ int new_basis_kind(int a, bool push, int *old)
{
    if (a == kG) return 3;
    if (push) {
        if (a < kMM) {
            if (a == kMM - 1) return 1;
            *old = a + 1;
            return 0;
        }
        if (a == 2 * kMM - 1) return 2;
        *old = a + 1;
        return 0;
    }
    *old = a;
    return 0;
}

// Slot holding <kind-vector, old basis vector o>, kind in {1,2,3}.
__device__ __forceinline__ int slot_new_old(int kind, int o)
{
    const bool is_s = o < kMM;
    const int j = is_s ? o : o - kMM;
    if (kind == 3) return is_s ? sGS(j) : sGY(j);
    if (kind == 1) return is_s ? sSS(j) : sSY(j);
    return is_s ? sYS(j) : sYY(j);
}

__device__ __forceinline__ int slot_new_new(int ka, int kb)
{
    if (ka > kb) { const int t = ka; ka = kb; kb = t; }
    if (ka == 1 && kb == 1) return sScSc;
    if (ka == 1 && kb == 2) return sScYc;
    if (ka == 2 && kb == 2) return sYcYc;
    if (ka == 1 && kb == 3) return sScG;
    if (ka == 2 && kb == 3) return sYcG;
    return sGG;
}

// Where entry ent = a * kNB + l of the updated Gram matrix comes from:
// an old entry (index < 0x8000) or a reduction slot (0x8000 + slot).
__device__ __forceinline__ uint16_t gram_source(int ent, bool push)
{
    const int a = ent / kNB, l = ent - a * kNB;
    int oa = 0, ol = 0;
    const int ka = new_basis_kind(a, push, &oa);
    const int kl = new_basis_kind(l, push, &ol);
    if (ka == 0 && kl == 0) return (uint16_t)(oa * kNB + ol);
    int sl;
    if (ka == 0) sl = slot_new_old(kl, oa);
    else if (kl == 0) sl = slot_new_old(ka, ol);
    else sl = slot_new_new(ka, kl);
    return (uint16_t)(0x8000 + sl);
}

// Whole-instance descent with B as a ring: the slots that lane l (basis
// vector l in pair order of the UPDATED basis: s_0..s_9, y_0..y_9, g)
// takes its new Gram entries from, as byte addresses for ds_bpermute
// packed in one word: bits 0-7 <g, b_l> without a push, 8-15 <g, b_l>
// with a push, 16-23 <s, b_l> and 24-31 <y, b_l> of the pushed pair.  A
// push renumbers old pair j + 1 as pair j; the new pair is pair 9.
__device__ __forceinline__ uint32_t gram_perm_bytes(int l)
{
    const bool is_g = l >= kG, is_s = l < kMM;
    const int j = is_s ? l : (is_g ? 0 : l - kMM);
    auto slot = [&](int kind, bool push) -> int {   // kind 3: g, 1: s, 2: y
        const bool newp = push && j == kMM - 1;
        const int jo = push ? j + 1 : j;
        if (is_g) return kind == 3 ? sGG : kind == 1 ? sScG : sYcG;
        if (newp) {
            if (kind == 3) return is_s ? sScG : sYcG;
            if (kind == 1) return is_s ? sScSc : sScYc;
            return is_s ? sScYc : sYcYc;
        }
        if (kind == 3) return is_s ? sGS(jo) : sGY(jo);
        if (kind == 1) return is_s ? sSS(jo) : sSY(jo);
        return is_s ? sYS(jo) : sYY(jo);
    };
    return (uint32_t)(4 * slot(3, false)) | ((uint32_t)(4 * slot(3, true)) << 8) |
           ((uint32_t)(4 * slot(1, true)) << 16) | ((uint32_t)(4 * slot(2, true)) << 24);
}

// ---------------------------------------------------------------------------
// Counting sort of the n circles of one instance into grid cells, ascending
// circle index inside every cell, with the positions copied in that order:
//   cell_start [ncell + 1]  first slot of each cell
//   cell_circ  [n]          circle of each slot
//   psort      [n]          its position (the list build reads a cell row as
//                           one contiguous run of them, without the index)
//   own[u]                  slot of circle tid + u * BLOCK
// tmp: n entries of scratch (by slot, in arrival order); scan_tmp: BLOCK / 64
// ints.  The order inside a cell comes from ranking each circle among its
// cell's circles (one or two of them at the cutoff's cell size), which every
// circle does at once; sorting each cell by one thread left most lanes idle
// behind chains of dependent LDS accesses.  The scan sums the cells a
// thread owns, then the lanes by DPP: one barrier.  Ends with a barrier.
// ---------------------------------------------------------------------------
template <int BLOCK, int CPT>
__device__ __forceinline__ void sort_cells(int tid, const float2 (&x)[CPT], int n, const Grid &g,
                                           int *cell_start, uint16_t *cell_circ, uint16_t *tmp,
                                           float2 *psort, int *scan_tmp, int (&own)[CPT])
{
    constexpr int NW = BLOCK / kWave;
    const int ncell = g.nc * g.nc;
    for (int c = tid; c <= ncell; c += BLOCK) cell_start[c] = 0;
    __syncthreads();
    int cell[CPT], slot[CPT];
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        cell[u] = slot[u] = 0;
        if (tid + u * BLOCK < n) {
            cell[u] = cell_of(x[u], g);
            slot[u] = atomicAdd(&cell_start[cell[u]], 1);
        }
    }
    __syncthreads();
    // a thread's cells: up to four stay in registers (their reads in flight
    // together), more are read twice
    constexpr int kReg = 4;
    const int ch = (ncell + BLOCK - 1) / BLOCK;
    const int c0 = tid * ch, c1 = c0 + ch < ncell ? c0 + ch : ncell;
    int cnt4[kReg], sum = 0;
    if (ch <= kReg) {
#pragma unroll
        for (int q = 0; q < kReg; ++q) cnt4[q] = q < ch && c0 + q < ncell ? cell_start[c0 + q] : 0;
#pragma unroll
        for (int q = 0; q < kReg; ++q) sum += cnt4[q];
    } else {
        for (int c = c0; c < c1; ++c) sum += cell_start[c];
    }
    const int inc = wave_scan_dpp(sum);
    int run = inc - sum;
    if constexpr (NW > 1) {
        if ((tid & (kWave - 1)) == kWave - 1) scan_tmp[tid / kWave] = inc;
        __syncthreads();
        const int w = __builtin_amdgcn_readfirstlane(tid / kWave);
#pragma unroll
        for (int q = 0; q < NW - 1; ++q) run += q < w ? scan_tmp[q] : 0;
    }
    if (ch <= kReg) {
#pragma unroll
        for (int q = 0; q < kReg; ++q) {
            if (q < ch && c0 + q < ncell) cell_start[c0 + q] = run;
            run += cnt4[q];
        }
    } else {
        for (int c = c0; c < c1; ++c) {
            const int v = cell_start[c];
            cell_start[c] = run;
            run += v;
        }
    }
    if (tid == 0) cell_start[ncell] = n;
    __syncthreads();
    int a[CPT], z[CPT];
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        a[u] = cell_start[cell[u]];
        z[u] = cell_start[cell[u] + 1];
        if (tid + u * BLOCK < n) tmp[a[u] + slot[u]] = (uint16_t)(tid + u * BLOCK);
        else z[u] = a[u];
    }
    __syncthreads();
#pragma unroll
    for (int u = 0; u < CPT; ++u) {
        const int i = tid + u * BLOCK;
        int r = a[u];
        for (int t = a[u]; t < z[u]; t += 4) {       // four reads in flight
            int v[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = tmp[t + q < z[u] ? t + q : t];
#pragma unroll
            for (int q = 0; q < 4; ++q) r += (t + q < z[u] && v[q] < i) ? 1 : 0;
        }
        own[u] = r;
        if (i < n) {
            cell_circ[r] = (uint16_t)i;
            psort[r] = x[u];
        }
    }
    __syncthreads();
}

// Slots of the 3 x 3 cells around the cell of p: three cell rows (first slot,
// length; rows outside the grid are empty); own: the slot of p's circle, self
// receives its place in the run of the three rows.
__device__ __forceinline__ void cell_rows(float2 p, bool act, int own, const Grid &g,
                                          const int *cell_start, int (&ra)[3], int (&rl)[3],
                                          int &self)
{
    const int cx = cell_coord(p.x, g), cy = cell_coord(p.y, g);
    const int y0 = cy > 0 ? cy - 1 : 0, y1 = cy < g.nc - 1 ? cy + 1 : g.nc - 1;
    const int x0 = cx > 0 ? cx - 1 : 0, x1 = cx < g.nc - 1 ? cx + 1 : g.nc - 1;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const bool row = act && y0 + r <= y1;
        const int yy = y0 + r <= y1 ? y0 + r : y0;
        const int a = cell_start[yy * g.nc + x0];
        const int z = cell_start[yy * g.nc + x1 + 1];
        ra[r] = row ? a : 0;
        rl[r] = row ? z - a : 0;
    }
    self = cy > y0 ? rl[0] + own - ra[1] : own - ra[0];
}

// The lowest bit of a candidate mask taken: candidate k of three runs (k < n0:
// slot k + s0, k < n01: k + s1, else k + s2); j receives its circle.  False
// (and some circle) when the mask is empty.
__device__ __forceinline__ bool next_neighbor(unsigned &mask, int n0, int n01, int s0, int s1, int s2,
                                              const uint16_t *cell_circ, int &j)
{
    const bool has = mask != 0;
    const int k = __builtin_ctz(mask | (1u << 31));
    mask &= mask - 1;
    j = cell_circ[has ? k + (k < n0 ? s0 : k < n01 ? s1 : s2) : 0];
    return has;
}

__device__ __forceinline__ bool next_neighbor(unsigned long long &mask, int n0, int n01, int s0, int s1,
                                              int s2, const uint16_t *cell_circ, int &j)
{
    const bool has = mask != 0;
    const int k = __builtin_ctzll(mask | (1ull << 63));
    mask &= mask - 1;
    j = cell_circ[has ? k + (k < n0 ? s0 : k < n01 ? s1 : s2) : 0];
    return has;
}

// Which of the candidates of a thread's circles are neighbors (the predicate
// near64 with c2): one bit per candidate in the order of the circle's three
// runs ra, rl (at most 32 each, 64 in all; kmax: the wave's longest of each,
// uniform), the circle itself (place self) left out.  FP32 decides outside a
// band of 1e-6 c2 around c2 (the FP32 distance is within 4e-7);
// a wave with a candidate inside the band takes the FP64 predicate for all of
// its own.  CAND
// candidates of a row are read per turn, past a run's end from any readable
// position (psort has NMAX + 8).  NO_NAN: the circles' distances are numbers
// (so that a sign bit decides), two instructions fewer per candidate, and
// any cutoff (1e-30 covers squares below the normal range).
template <int CPT, int CAND, int NMAX, bool NO_NAN = false>
__device__ __forceinline__ void neighbor_masks(const float2 (&x)[CPT], const bool (&act)[CPT],
                                               const int (&self)[CPT], const int (&ra)[CPT][3],
                                               const int (&rl)[CPT][3], const int (&kmax)[3],
                                               const float2 *psort, double c2,
                                               unsigned long long (&mask)[CPT])
{
    const float c2f = (float)c2, band = NO_NAN ? c2f * 1e-6f + 1e-30f : c2f * 1e-6f;
    float dmin = 3.0e38f;
    auto scan = [&](auto exact) {
        unsigned mr[CPT][3];
#pragma unroll
        for (int r = 0; r < 3; ++r) {
#pragma unroll
            for (int c = 0; c < CPT; ++c) mr[c][r] = 0;
            for (int k0 = 0; k0 < kmax[r]; k0 += CAND) {
                float px[CPT][CAND], py[CPT][CAND];
                unsigned bits[CPT];
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const float2 *src = psort + min(ra[c][r] + k0, NMAX);
#pragma unroll
                    for (int u = 0; u < CAND; ++u) {
                        const float2 v = src[u];
                        px[c][u] = v.x;
                        py[c][u] = v.y;
                    }
                    bits[c] = 0;
                }
                if constexpr (NO_NAN && !decltype(exact)::value) {
#pragma unroll
                    for (int u = CAND - 1; u >= 0; --u)
#pragma unroll
                        for (int c = 0; c < CPT; ++c) {
                            const float dx = x[c].x - px[c][u], dy = x[c].y - py[c][u];
                            const float t = fmaf(dx, dx, fmaf(dy, dy, -c2f));
                            bits[c] = __builtin_amdgcn_alignbit(bits[c], __float_as_uint(t), 31);
                            dmin = fminf(dmin, fabsf(t));
                        }
                }
#pragma unroll
                for (int u = 0; u < (NO_NAN && !decltype(exact)::value ? 0 : CAND); ++u)
#pragma unroll
                    for (int c = 0; c < CPT; ++c) {
                        bool nb;
                        if constexpr (decltype(exact)::value) {
                            nb = near64(x[c], make_float2(px[c][u], py[c][u]), c2);
                        } else {
                            const float dx = x[c].x - px[c][u], dy = x[c].y - py[c][u];
                            const float t = dx * dx + dy * dy - c2f;
                            nb = t < 0.f;
                            dmin = fminf(dmin, fabsf(t));
                        }
                        bits[c] |= nb ? 1u << u : 0u;
                    }
#pragma unroll
                for (int c = 0; c < CPT; ++c) mr[c][r] |= bits[c] << k0;
            }
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            mask[c] = 0;
#pragma unroll
            for (int r = 2; r >= 0; --r) {
                const unsigned keep = rl[c][r] < 32 ? (1u << rl[c][r]) - 1u : ~0u;
                mask[c] = (mask[c] << rl[c][r]) | (unsigned long long)(mr[c][r] & keep);
            }
            mask[c] = act[c] ? mask[c] & ~(1ull << self[c]) : 0ull;
        }
    };
    scan(std::false_type{});
    if (__builtin_amdgcn_ballot_w64(dmin <= band)) scan(std::true_type{});
}

// Neighbor lists of a workgroup's circles (tid + c * BLOCK) into ELL slots,
// slot-major (list[t * NMAX + i]: byte offset of the t-th neighbor in the
// position array), in the order of the sorted cells, every list padded with
// far_off up to the longest of the wave; list_n: list lengths.  Neighbor: the
// predicate near64 with c2, decided in FP32 outside a band of 1e-6 c2 around
// it (the FP32 distance is within 4e-7).  Returns the wave's longest list (its
// pad length); up: listed neighbors with a higher index; *over is set when a
// list does not fit.
//
// Bound by instruction issue (two waves per SIMD): about 13 candidates per
// circle, but 20 to 30 for the wave's longest run, so the candidates' part is
// kept small -- an FP32 distance and one mask bit each, from consecutive
// sorted positions -- and everything that only a neighbor needs (its index,
// the list write) runs over the mask bits, at most 7 or 8 per wave.  The FP64
// predicate runs for the whole wave when any of its distances falls in the
// band (at n = 1000 about one wave in a thousand).  PAD: lists are padded to
// a multiple of it.  The candidate-by-candidate
// loop this replaces tested, masked and stored about 40 instructions per
// candidate: a 256 x n = 1000 descent 30.1 -> 28.1 ms, 448 SED candidates of
// n = 300 .. 1000 17.7 -> 16.8 ms, one start of n = 20 446 -> 405 us.
template <int BLOCK, int CPT, int ELL, int NMAX, int PAD>
__device__ __forceinline__ int build_lists(int tid, const float2 (&x)[CPT], const bool (&act)[CPT],
                                           const int (&own)[CPT], const Grid &g,
                                           const int *cell_start, const uint16_t *cell_circ,
                                           const float2 *psort, double c2, uint16_t *list,
                                           uint8_t *list_n, int far_off, int (&up)[CPT], int *over)
{
    // candidates of a row per turn: a row has about four, the wave's longest
    // seven; a lone wave per SIMD reads eight to wait for LDS once
    constexpr int kCand = CPT == 1 && BLOCK <= 256 ? 8 : 4;
    int ra[CPT][3], rl[CPT][3], self[CPT], cnt[CPT];
    int kmax[3] = {0, 0, 0};
    bool fits = true;              // three runs of at most 32, 64 candidates in all
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        cell_rows(x[c], act[c], own[c], g, cell_start, ra[c], rl[c], self[c]);
        cnt[c] = up[c] = 0;
#pragma unroll
        for (int r = 0; r < 3; ++r) kmax[r] = max(kmax[r], rl[c][r]);
        fits = fits && rl[c][0] + rl[c][1] + rl[c][2] <= 64;
    }
#pragma unroll
    for (int r = 0; r < 3; ++r) kmax[r] = wave_max_dpp(kmax[r]);
    int m = 0;
    if (max(kmax[0], max(kmax[1], kmax[2])) <= 32 && !__builtin_amdgcn_ballot_w64(!fits)) {
        unsigned long long mask[CPT];
        neighbor_masks<CPT, kCand, NMAX>(x, act, self, ra, rl, kmax, psort, c2, mask);
        // neighbors: one mask bit of every circle per turn; a turn's index
        // read is in flight while the next turn's bits are taken (its write
        // comes one turn later)
        int cut[CPT], sh1[CPT], sh2[CPT], jv[CPT];
        bool has[CPT];
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            cut[c] = rl[c][0] + rl[c][1];
            sh1[c] = ra[c][1] - rl[c][0];
            sh2[c] = ra[c][2] - cut[c];
            up[c] = 0;
        }
        // the wave's longest list
        int longest = 0;
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            cnt[c] = __builtin_popcountll(mask[c]);
            longest = max(longest, cnt[c]);
        }
        m = wave_max_dpp(longest);
#pragma unroll
        for (int c = 0; c < CPT; ++c)
            has[c] = next_neighbor(mask[c], rl[c][0], cut[c], ra[c][0], sh1[c], sh2[c], cell_circ, jv[c]);
        for (int q = 0; q < m; ++q) {
            int jq[CPT];
            bool hq[CPT];
#pragma unroll
            for (int c = 0; c < CPT; ++c) { jq[c] = jv[c]; hq[c] = has[c]; }
            if (q + 1 < m) {
#pragma unroll
                for (int c = 0; c < CPT; ++c)
                    has[c] = next_neighbor(mask[c], rl[c][0], cut[c], ra[c][0], sh1[c], sh2[c], cell_circ, jv[c]);
            }
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                const int i = tid + c * BLOCK;
                if (q < ELL) list[q * NMAX + i] = (uint16_t)(hq[c] ? jq[c] * (int)sizeof(float2) : far_off);
                up[c] += (hq[c] && jq[c] > i) ? 1 : 0;
            }
        }
    } else {
        // a crowded neighborhood: candidate by candidate
        int longest = 0;
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int i = tid + c * BLOCK;
#pragma unroll
            for (int r = 0; r < 3; ++r) {
                for (int t = ra[c][r]; t < ra[c][r] + rl[c][r]; ++t) {
                    if (t != own[c] && near64(x[c], psort[t], c2)) {
                        const int j = cell_circ[t];
                        if (cnt[c] < ELL) list[cnt[c] * NMAX + i] = (uint16_t)(j * (int)sizeof(float2));
                        ++cnt[c];
                        up[c] += j > i ? 1 : 0;
                    }
                }
            }
            longest = max(longest, cnt[c]);
        }
        m = wave_max_dpp(longest);
#pragma unroll
        for (int c = 0; c < CPT; ++c)
            for (int t = cnt[c]; t < min(m, ELL); ++t) list[t * NMAX + tid + c * BLOCK] = (uint16_t)far_off;
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c)
        if (act[c]) {
            if (cnt[c] > ELL) *over = 1;
            list_n[tid + c * BLOCK] = (uint8_t)min(cnt[c], ELL);
        }
    m = min(m, ELL);
    if (PAD > 1 && m % PAD != 0) {       // (ELL is a multiple of PAD)
#pragma unroll
        for (int c = 0; c < CPT; ++c)
            for (int q = m; q % PAD != 0; ++q) list[q * NMAX + tid + c * BLOCK] = (uint16_t)far_off;
        m += PAD - m % PAD;
    }
    return m;
}

// FP32 pair term of circle i (at q) with circle j (at pj): energy on the
// i < j side only, gradient of circle i always.  Branch-free (selects only):
// non-overlapping pairs give d = 0, coincident centres d = 2 rad with no
// gradient.  (With branches the compiler merges the accumulations into one
// store through a selected address and moves the accumulators to memory.)
__device__ __forceinline__ void pair_term32(float2 q, float2 pj, bool count_e, float two_r,
                                            float four_r2, float &e, float &e1, float &gx,
                                            float &gy)
{
    const float dx = q.x - pj.x, dy = q.y - pj.y;
    const float l2 = dot2(dx, dx, dy, dy);
    const bool ov = l2 < four_r2;
    const float il = (ov && l2 > 0.f) ? __builtin_amdgcn_rsqf(l2) : 0.f;
    const float d = ov ? two_r - l2 * il : 0.f;
    // the same pair for unit circles (rad <= the descent's radius): overlap
    // 2 - l, which is d - (two_r - 2) whenever it is positive
    const float d1 = fmaxf(d - (two_r - 2.f), 0.f);
    e += count_e ? d * d : 0.f;
    e1 += count_e ? d1 * d1 : 0.f;
    const float kf = -2.f * d * il;
    gx += kf * dx;
    gy += kf * dy;
}

// FP64 pair energies (descent objective, unit circles) of a pair i < j.
__device__ __forceinline__ void pair_term64(float2 q, float2 pj, double two_r64, double four_r2_64,
                                            double &eo, double &et)
{
    const double ex = (double)q.x - (double)pj.x, ey = (double)q.y - (double)pj.y;
    const double m2 = dot2(ex, ex, ey, ey);
    if (m2 < four_r2_64) {
        const double l = sqrt(m2);
        const double d = two_r64 - l;
        const double dt = m2 < 4.0 ? 2.0 - l : 0.0;
        eo += d * d;
        et += dt * dt;
    }
}

// sqrt(m2) in FP64 from FP32 estimates l32 ~ sqrt(m2) and il ~ 1/sqrt(m2)
// (both 0 when m2 is 0): two Newton steps l <- l + (m2 - l^2) * il / 2, the
// residual formed with one rounding.  With relative errors e of l32 and h
// of il, one step leaves about e^2 / 2 + e h (1e-14 from 1e-7) and the
// second one FP64 rounding: a square root without the FP64 reciprocal
// square root, whose seed is no better than il.
__device__ __forceinline__ double sqrt64_from32(double m2, float l32, float il)
{
    const double h = (double)(0.5f * il);
    double l = (double)l32;
    l = fma(fma(-l, l, m2), h, l);
    l = fma(fma(-l, l, m2), h, l);
    return l;
}

// The list sweep's FP32 pair term of circle i (at q) with circle j (at pj),
// as pair_term32 but with the gradient term divided by -2: gx, gy receive
// (d / l) (c_i - c_j), and the caller multiplies the sum by -2 -- a scaling
// by a power of two, exact, so the result has pair_term32's bits.  Returns
// the FP32 1/l (from max(l^2, FLT_MIN): coincident centres give d = 2 rad
// and a zero term without a test of their own) and l2, the seeds of
// pair_term64s.
__device__ __forceinline__ float pair_term32s(float2 q, float2 pj, bool count_e, float two_r,
                                              float four_r2, float &e, float &e1, float &gx,
                                              float &gy, float &l2o, bool want_e1 = true)
{
    const float dx = q.x - pj.x, dy = q.y - pj.y;
    const float l2 = dot2(dx, dx, dy, dy);
    const bool ov = l2 < four_r2;
    // + FLT_MIN: a finite inverse for coincident centres; a no-op (exact)
    // for any l2 above 2^-100
    const float il = __builtin_amdgcn_rsqf(l2 + 1.17549435e-38f);
    const float d = ov ? two_r - l2 * il : 0.f;
    const float dc = count_e ? d : 0.f;       // the overlap if this term counts the pair
    e = fmaf(dc, d, e);
    // the unit-circle energy (wave-uniform want_e1: only its caller's switch
    // into the FP64 regime reads it)
    if (want_e1) {
        const float d1 = fmaxf(dc - (two_r - 2.f), 0.f);
        e1 = fmaf(d1, d1, e1);
    }
    const float kf = d * il;
    gx += kf * dx;
    gy += kf * dy;
    l2o = l2;
    return il;
}

// pair_term64 with the square root from the FP32 seeds (l32 = l2 * il).
__device__ __forceinline__ void pair_term64s(float2 q, float2 pj, float l32, float il,
                                             double two_r64, double four_r2_64, double &eo,
                                             double &et)
{
    const double ex = (double)q.x - (double)pj.x, ey = (double)q.y - (double)pj.y;
    const double m2 = dot2(ex, ex, ey, ey);
    if (m2 < four_r2_64) {
        const double l = sqrt64_from32(m2, l32, il);
        const double d = two_r64 - l;
        const double dt = m2 < 4.0 ? 2.0 - l : 0.0;
        eo += d * d;
        et += dt * dt;
    }
}

}  // namespace pecc
