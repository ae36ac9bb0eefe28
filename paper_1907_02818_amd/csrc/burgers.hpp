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

__device__ __forceinline__ double fused_mul_add(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fused_mul_add(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// r_i from (um, u0, up) = u[i-1], u[i], u[i+1].
template <class T> __device__ __forceinline__ T burgers_primal_cell(T um, T u0, T up, T C, T D)
{
#pragma clang fp contract(off)
    const T conv = fused_mul_add(pos_part(u0), u0 - um, neg_part(u0) * (up - u0));
    const T lap = fused_mul_add(T(-2), u0, um) + up;
    return fused_mul_add(D, lap, fused_mul_add(-C, conv, u0));
}

// The three terms of one u_bar[j]; (um, u0, up) = u[j-1], u[j], u[j+1], (rm, r0, rp) = r_bar at
// the same cells with zeros where the iteration does not exist:
//   g_-(i) = C max(u_i,0) + D,  g_+(i) = -C min(u_i,0) + D,
//   g_0(i) = 1 - 2D - C( [u_i>=0](u_i-u_{i-1}) + max(u_i,0) + [-u_i>=0](u_{i+1}-u_i) - min(u_i,0) )
template <class T> __device__ __forceinline__ T burgers_adjoint_terms(T um, T u0, T up, T rm, T r0, T rp, T C, T D, bool in0)
{
#pragma clang fp contract(off)
    const T dpos = u0 >= T(0) ? T(1) : T(0);
    const T dneg = -u0 >= T(0) ? T(1) : T(0);
    // dpos and dneg are 0 or 1: their products are exact, and fusing them changes no bit
    const T slope = fused_mul_add(dneg, up - u0, fused_mul_add(dpos, u0 - um, pos_part(u0))) - neg_part(u0);
    const T g0 = T(1) - C * slope - T(2) * D;
    const T from_right = (C * pos_part(up) + D) * rp;      // iteration j+1 read u[j] as its left cell
    const T from_left = (-C * neg_part(um) + D) * rm;      // iteration j-1 read u[j] as its right cell
    return from_right + (in0 ? g0 * r0 : T(0)) + from_left;
}

}  // namespace sadj
