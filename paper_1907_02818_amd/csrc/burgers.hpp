// One cell of the upwinded Burgers step and of its gather-form adjoint, shared by every kernel
// that computes them.  Contraction into fused multiply-adds is switched off and written out, so
// that kernels which apply several steps of a time loop to cells held in registers round every
// cell like the kernels that apply one step, and the results are equal bit for bit.
#pragma once
#include "common.hpp"

namespace sadj {

// max(v, 0) and min(v, 0) as one instruction each: written as selects or library calls the compiler adds
// an instruction that quiets signalling NaN first, a tenth of the primal step's arithmetic.
__device__ __forceinline__ double pos_part(double v) { double r; asm("v_max_f64 %0, %1, 0" : "=v"(r) : "v"(v)); return r; }
__device__ __forceinline__ double neg_part(double v) { double r; asm("v_min_f64 %0, %1, 0" : "=v"(r) : "v"(v)); return r; }
__device__ __forceinline__ float pos_part(float v) { float r; asm("v_max_f32 %0, 0, %1" : "=v"(r) : "v"(v)); return r; }
__device__ __forceinline__ float neg_part(float v) { float r; asm("v_min_f32 %0, 0, %1" : "=v"(r) : "v"(v)); return r; }

// What a cell gives its neighbours: g_-(i) = C max(u_i,0) + D to the cell on its left, g_+(i) = -C min(u_i,0) + D to the one on its
// right.  The forward step is written with the same two: with d_l = u_i - u_{i-1}, d_r = u_{i+1} - u_i
//   r_i = u_i - C (max(u_i,0) d_l + min(u_i,0) d_r) + D (d_r - d_l) = u_i - g_- d_l + g_+ d_r,
// 8 operations a cell (d_l is its neighbour's d_r) where the formula as it stands takes 10.
template <class T> __device__ __forceinline__ T burgers_to_left(T u, T C, T D) { return fma_t(C, pos_part(u), D); }
template <class T> __device__ __forceinline__ T burgers_to_right(T u, T C, T D) { return fma_t(-C, neg_part(u), D); }

// Values that are not finite.  The formula multiplies the difference it does not use by 0, which gives NaN where that difference
// is not finite; the short forms below leave it out, and a NaN or an infinity beside a cell would get lost.  So:
//   - Where the short form of r_i is not finite the formula as it stands is evaluated.  The short form is finite only if u_{i-1}, u_i,
//     u_{i+1} all are: g_- d_l and g_+ d_r are not finite (0 times infinity included) as soon as one of them is not.
//   - The slope adds 0 times the value that it leaves out, and 0 u_i.  (Not the difference: of finite values it may overflow.)
// Neither changes a bit of a finite result.  The loops ask once per pass and wave whether this is needed.
template <class T> __device__ __forceinline__ T burgers_primal_formula(T um, T u0, T up, T C, T D)
{
#pragma clang fp contract(off)
    const T conv = fma_t(pos_part(u0), u0 - um, neg_part(u0) * (up - u0));
    return fma_t(D, fma_t(T(-2), u0, um) + up, fma_t(-C, conv, u0));
}

// r_i from (um, u0, up) = u[i-1], u[i], u[i+1].  CHECKED: for values that may not be finite.
template <bool CHECKED, class T> __device__ __forceinline__ T burgers_primal_cell(T um, T u0, T up, T C, T D)
{
#pragma clang fp contract(off)
    const T r = u0 + fma_t(burgers_to_right(u0, C, D), up - u0, -(burgers_to_left(u0, C, D) * (u0 - um)));
    if (CHECKED && !__builtin_isfinite(r)) return burgers_primal_formula(um, u0, up, C, D);
    return r;
}

// Sign bit of v set ? b : a, with a shift and a bit field insert per word (the shift written out: the compiler would make a comparison
// and selections of it).  Measured with two waves per SIMD: 11 cycles for a double, 13 to 21 with v_cmp and v_cndmask, the most where the
// selection reads VCC in its short form.
__device__ __forceinline__ unsigned sign_mask(int high) { unsigned m; asm("v_ashrrev_i32 %0, 31, %1" : "=v"(m) : "v"(high)); return m; }
__device__ __forceinline__ int by_mask(unsigned m, int a, int b) { return (int)((m & (unsigned)b) | (~m & (unsigned)a)); }
__device__ __forceinline__ double by_sign(double v, double a, double b)
{
    const unsigned m = sign_mask(__double2hiint(v));
    return __hiloint2double(by_mask(m, __double2hiint(a), __double2hiint(b)), by_mask(m, __double2loint(a), __double2loint(b)));
}
__device__ __forceinline__ float by_sign(float v, float a, float b)
{
    return __int_as_float(by_mask(sign_mask(__float_as_int(v)), __float_as_int(a), __float_as_int(b)));
}

// The upwind slope of values that are finite and not 0: |u| + (u > 0 ? d_l : d_r).  max(u,0) - min(u,0) is |u|.
template <class T> __device__ __forceinline__ T burgers_slope(T um, T u0, T up)
{
#pragma clang fp contract(off)
    const T dl = u0 - um, dr = up - u0;
    return __builtin_elementwise_abs(u0) + by_sign(u0, dl, dr);
}
// Of finite values, from that: both one-sided differences count where u = 0 (of either sign).
template <class T> __device__ __forceinline__ T burgers_slope_at_zero(T slope, T um, T u0, T up)
{
#pragma clang fp contract(off)
    return u0 == T(0) ? (u0 - um) + (up - u0) : slope;
}
// Of any values: values that are not finite count where they are not used, too.
template <class T> __device__ __forceinline__ T burgers_slope_in_full(T slope, T um, T u0, T up)
{
#pragma clang fp contract(off)
    const T unused = u0 > T(0) ? up : u0 < T(0) ? um : T(0);
    return burgers_slope_at_zero(fma_t(T(0), u0, fma_t(T(0), unused, slope)), um, u0, up);
}

// g_0 = 1 - 2D - C slope.  1 - 2D is the same for all cells, and what its rounding loses adds up over the steps of a loop.  fp64 rounds it
// once and spends one operation a cell: after 128 steps (C = 0.1, D = 0.05) lam is 3.4e-15 off, 3.6e-15 with the formula as it stands.
// In fp32 that form would be 3.0e-6 off instead of 2.9e-6, so 1 is added last, where the other two terms vary from cell to cell and
// so does the rounding: 2.0e-7, for one more operation.  (1 + g, and not lam + g lam: an infinite lam stays infinite.)
template <class T> __device__ __forceinline__ T burgers_centre(T slope, T C, T D)
{
#pragma clang fp contract(off)
    if constexpr (sizeof(T) == 8) return fma_t(-C, slope, T(1) - T(2) * D);
    else return T(1) + fma_t(-C, slope, T(-2) * D);
}

// One u_bar[j] of its three terms: iteration j+1 read u[j] as its left cell, j-1 as its right cell:
//   g_-(j+1) r_bar[j+1] + g_+(j-1) r_bar[j-1] + g_0(j) r_bar[j],
//   g_0(i) = 1 - 2D - C( |u_i| + [u_i>=0](u_i-u_{i-1}) + [u_i<=0](u_{i+1}-u_i) )
// from_left = g_+(j-1) r_bar[j-1]; r_bar zero where the iteration does not exist; in0: iteration j exists.
template <class T> __device__ __forceinline__ T burgers_adjoint_cell(T slope, T up, T from_left, T r0, T rp, T C, T D, bool in0)
{
#pragma clang fp contract(off)
    const T sides = fma_t(burgers_to_left(up, C, D), rp, from_left);
    return in0 ? fma_t(burgers_centre(slope, C, D), r0, sides) : sides;
}

// The same from the values at j-1, j, j+1.
template <class T> __device__ __forceinline__ T burgers_adjoint_terms(T um, T u0, T up, T rm, T r0, T rp, T C, T D, bool in0)
{
    const T slope = burgers_slope_in_full(burgers_slope(um, u0, up), um, u0, up);
    return burgers_adjoint_cell(slope, up, mul_rounded(burgers_to_right(um, C, D), rm), r0, rp, C, D, in0);
}

}  // namespace sadj
