// 1-D stencils: linear 3-point wave step and upwinded Burgers step, primal and
// gather-form adjoint (paper Sections 3.2, 4.1 in one dimension, and 4.2).
//
// Mapping to CDNA4.  A 64-lane wave owns a segment of 64*PX consecutive cells, PX
// cells (16 bytes) per lane.  Neighbour values travel between lanes with wave
// shuffles; the two cells beside the segment are loaded by lanes 0 and 63.  No LDS,
// no barrier, no atomics: each output cell is written by exactly one lane.
//
// Regions (Sections 3.3.3, 3.3.4).  The core waves cover the segments whose reads
// all lie in the primal iteration space I = [1, n-2]; they run an instantiation that
// is compiled without any guard.  The remainder waves cover the first and the last
// segment(s) with the guarded instantiation: a term is kept iff its primal iteration
// exists, unused values are replaced by zero with a select (never multiplied by zero),
// and loads are element-wise and clamped into the array.  Core and remainder are
// disjoint and unordered, so they share one dispatch: the first workgroups are core,
// the last one or two are remainder.
#include "burgers.hpp"
#include "common.hpp"
#include "launch.hpp"

namespace sadj {

struct Args1d {
    const void *a0, *a1, *a2;   // inputs (meaning depends on the kernel)
    void *o0, *o1;              // outputs
    long n;
    double C, D;
    double w[3];                // box stencil: gather weights at offsets -1, 0, +1
    long core_segs;             // core waves handle segments 1 .. core_segs
    long core_blocks;           // workgroups [0, core_blocks) are core, the rest remainder
    long rem_segs;              // remainder waves: index 0 -> segment 0, k>0 -> segment core_segs + k
};

constexpr int kWaves1d = 4;
constexpr bool kStreamStores = true;
enum Op1d { OP_ADJ_WAVE, OP_ADJ_WAVE_UPREV, OP_PRI_WAVE, OP_PRI_BURGERS, OP_ADJ_BURGERS, OP_ADJ_BOX, OP_PRI_BOX,
            OP_ADJ_BURGERS_ASSIGN, OP_PRI_BURGERS_KEEP_ENDS };

// Load PX consecutive cells starting at x.  Unguarded: one vector load.  Guarded:
// element-wise, indices clamped to [0, n-1].
template <class T, int PX, bool GUARD, bool STREAM = false>
__device__ __forceinline__ void load_cells(const T *p, long x, long n, T (&v)[PX])
{
    if (!GUARD) {
        const Vec<T, PX> t = STREAM ? ld_vec_stream<T, PX>(p + x) : ld_vec<T, PX>(p + x);
#pragma unroll
        for (int e = 0; e < PX; ++e) v[e] = t.v[e];
    } else {
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            const long i = x + e < n ? x + e : n - 1;
            v[e] = p[i];
        }
    }
}
// The cell beside a wave's segment; only lanes 0 and 63 use it, so only they load it.
template <class T, bool GUARD> __device__ __forceinline__ T load_cell(const T *p, long i, long n, int lane)
{
    if (GUARD) i = i < 0 ? 0 : (i > n - 1 ? n - 1 : i);
    T v = T(0);
    if (lane == 0 || lane == 63) v = p[i];
    return v;
}
template <class T, int PX, bool GUARD>
__device__ __forceinline__ void store_cells(T *p, long x, long n, const T (&v)[PX], const bool (&ok)[PX])
{
    if (!GUARD) {
        Vec<T, PX> t;
#pragma unroll
        for (int e = 0; e < PX; ++e) t.v[e] = v[e];
        if (kStreamStores) st_vec_stream<T, PX>(p + x, t);
        else st_vec<T, PX>(p + x, t);
    } else {
#pragma unroll
        for (int e = 0; e < PX; ++e)
            if (ok[e]) p[x + e] = v[e];
    }
}

// ------------------------------------------------------------------- wave, adjoint
// u_bar[j] += 2 r_bar[j] [j in I] + q[j-1] - 2 q[j] + q[j+1],  q = c*r_bar on I, else 0.
template <class T, int PX, bool GUARD, bool UPREV>
__device__ __forceinline__ void adj_wave1d_segment(const Args1d &a, long xs, int lane)
{
    constexpr int W = 64 * PX;
    const long n = a.n;
    const T *cg = static_cast<const T *>(a.a0);
    const T *rg = static_cast<const T *>(a.a1);
    T *ug = static_cast<T *>(a.o0);
    T *pg = static_cast<T *>(a.o1);
    const long x = xs + (long)lane * PX;
    const long hx = lane < 32 ? xs - 1 : xs + W;
    T cv[PX], rv[PX], uv[PX], pv[PX];
    load_cells<T, PX, GUARD, true>(cg, x, n, cv);
    load_cells<T, PX, GUARD, true>(rg, x, n, rv);
    load_cells<T, PX, GUARD, true>(ug, x, n, uv);
    if (UPREV) load_cells<T, PX, GUARD, true>(pg, x, n, pv);
    const T hc = load_cell<T, GUARD>(cg, hx, n, lane), hr = load_cell<T, GUARD>(rg, hx, n, lane);
    T q[PX], rr[PX];
    bool ok[PX];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
        const bool in = GUARD ? (x + e >= 1 && x + e <= n - 2) : true;
        ok[e] = GUARD ? (x + e < n) : true;
        rr[e] = in ? rv[e] : T(0);
        q[e] = in ? cv[e] * rv[e] : T(0);
    }
    const bool hin = GUARD ? (hx >= 1 && hx <= n - 2) : true;
    const T qh = hin ? hc * hr : T(0);
    T left, right;
    wave_neighbours<T, PX>(q, qh, lane, left, right);
    T out[PX], pout[PX];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
        const T l = e == 0 ? left : q[e - 1];
        const T r = e == PX - 1 ? right : q[e + 1];
        out[e] = uv[e] + ((T(-2) * q[e] + (l + r)) + T(2) * rr[e]);
        if (UPREV) pout[e] = pv[e] - rr[e];
    }
    store_cells<T, PX, GUARD>(ug, x, n, out, ok);
    if (UPREV) store_cells<T, PX, GUARD>(pg, x, n, pout, ok);
}

// -------------------------------------------------------------------- wave, primal
// r[i] = 2u[i] - u_prev[i] + c[i]*(u[i-1] - 2u[i] + u[i+1]) for i in I.
template <class T, int PX, bool GUARD>
__device__ __forceinline__ void pri_wave1d_segment(const Args1d &a, long xs, int lane)
{
    constexpr int W = 64 * PX;
    const long n = a.n;
    const T *ug = static_cast<const T *>(a.a0);
    const T *pg = static_cast<const T *>(a.a1);
    const T *cg = static_cast<const T *>(a.a2);
    T *rg = static_cast<T *>(a.o0);
    const long x = xs + (long)lane * PX;
    const long hx = lane < 32 ? xs - 1 : xs + W;
    T uv[PX], pv[PX], cv[PX];
    load_cells<T, PX, GUARD, true>(ug, x, n, uv);
    load_cells<T, PX, GUARD, true>(pg, x, n, pv);
    load_cells<T, PX, GUARD, true>(cg, x, n, cv);
    const T uh = load_cell<T, GUARD>(ug, hx, n, lane);
    T left, right;
    wave_neighbours<T, PX>(uv, uh, lane, left, right);
    T out[PX];
    bool ok[PX];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
        const T l = e == 0 ? left : uv[e - 1];
        const T r = e == PX - 1 ? right : uv[e + 1];
        ok[e] = GUARD ? (x + e >= 1 && x + e <= n - 2) : true;
        out[e] = T(2) * uv[e] - pv[e] + cv[e] * (T(-2) * uv[e] + (l + r));
    }
    store_cells<T, PX, GUARD>(rg, x, n, out, ok);
}

// ------------------------------------------------ three-point stencil, general weights
// primal   r[i] = c[i]*(w[-1] u[i-1] + w[0] u[i] + w[+1] u[i+1])            for i in I
// adjoint  u_bar[j] += W[-1] q[j-1] + W[0] q[j] + W[+1] q[j+1], q = c*r_bar on I, else 0,
// with W the mirrored table W[o] = w[-o] (paper Section 3.2: the worked example with
// weights (2,-3,4), whose outer weights trade places in the adjoint).  a.w holds the
// gather weights, i.e. w for the primal and W for the adjoint.
template <class T, int PX, bool GUARD, bool ADJ>
__device__ __forceinline__ void box1d_segment(const Args1d &a, long xs, int lane)
{
    constexpr int W = 64 * PX;
    const long n = a.n;
    const T wm = (T)a.w[0], w0 = (T)a.w[1], wp = (T)a.w[2];
    const T *g0 = static_cast<const T *>(a.a0);      // adjoint: c      primal: u
    const T *g1 = static_cast<const T *>(a.a1);      // adjoint: r_bar  primal: c
    T *og = static_cast<T *>(a.o0);
    const long x = xs + (long)lane * PX;
    const long hx = lane < 32 ? xs - 1 : xs + W;
    T v0[PX], v1[PX], vo[PX];
    load_cells<T, PX, GUARD, true>(g0, x, n, v0);
    load_cells<T, PX, GUARD, true>(g1, x, n, v1);
    if (ADJ) load_cells<T, PX, GUARD, true>(og, x, n, vo);
    T sh = load_cell<T, GUARD>(g0, hx, n, lane);
    if (ADJ) {
        const T h1 = load_cell<T, GUARD>(g1, hx, n, lane);
        const bool hin = GUARD ? (hx >= 1 && hx <= n - 2) : true;
        sh = hin ? sh * h1 : T(0);
    }
    T s[PX];
    bool ok[PX];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
        const bool in = GUARD ? (x + e >= 1 && x + e <= n - 2) : true;
        if (ADJ) { s[e] = in ? v0[e] * v1[e] : T(0); ok[e] = GUARD ? (x + e < n) : true; }
        else     { s[e] = v0[e]; ok[e] = in; }
    }
    T left, right;
    wave_neighbours<T, PX>(s, sh, lane, left, right);
    T out[PX];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
        const T l = e == 0 ? left : s[e - 1];
        const T r = e == PX - 1 ? right : s[e + 1];
        const T sum = (wm * l + w0 * s[e]) + wp * r;
        out[e] = ADJ ? vo[e] + sum : v1[e] * sum;
    }
    store_cells<T, PX, GUARD>(og, x, n, out, ok);
}

// ----------------------------------------------------------------- Burgers, primal
// KEEP_ENDS: the two end cells, which no iteration writes, receive the input's end values
// (boundary data held fixed from one state of a time loop to the next).
template <class T, int PX, bool GUARD, bool KEEP_ENDS = false>
__device__ __forceinline__ void pri_burgers_segment(const Args1d &a, long xs, int lane)
{
    constexpr int W = 64 * PX;
    const long n = a.n;
    const T C = (T)a.C, D = (T)a.D;
    const T *ug = static_cast<const T *>(a.a0);
    T *rg = static_cast<T *>(a.o0);
    const long x = xs + (long)lane * PX;
    const long hx = lane < 32 ? xs - 1 : xs + W;
    T uv[PX];
    load_cells<T, PX, GUARD, true>(ug, x, n, uv);
    const T uh = load_cell<T, GUARD>(ug, hx, n, lane);
    T left, right;
    wave_neighbours<T, PX>(uv, uh, lane, left, right);
    T out[PX];
    bool ok[PX];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
        const T um = e == 0 ? left : uv[e - 1];
        const T up = e == PX - 1 ? right : uv[e + 1];
        const T u0 = uv[e];
        const bool in = GUARD ? (x + e >= 1 && x + e <= n - 2) : true;
        ok[e] = (GUARD && KEEP_ENDS) ? (x + e < n) : in;
        const T val = burgers_primal_cell<true>(um, u0, up, C, D);
        out[e] = (GUARD && KEEP_ENDS) ? (in ? val : u0) : val;
    }
    store_cells<T, PX, GUARD>(rg, x, n, out, ok);
}

// ---------------------------------------------------------------- Burgers, adjoint
// u_bar[j] += g_-(j+1) r_bar[j+1] [j+1 in I] + g_0(j) r_bar[j] [j in I] + g_+(j-1) r_bar[j-1] [j-1 in I]
// The primal u is read at j-1, j, j+1 (shifted reads, Section 3.3.2).
// ASSIGN: u_bar[j] = (the three terms) instead of +=, for a time loop that recycles a
// buffer whose accumulated value is known to be zero (u_bar is then not read).
template <class T, int PX, bool GUARD, bool ASSIGN>
__device__ __forceinline__ void adj_burgers_segment(const Args1d &a, long xs, int lane)
{
    constexpr int W = 64 * PX;
    const long n = a.n;
    const T C = (T)a.C, D = (T)a.D;
    const T *ug = static_cast<const T *>(a.a0);
    const T *rg = static_cast<const T *>(a.a1);
    T *bg = static_cast<T *>(a.o0);
    const long x = xs + (long)lane * PX;
    const long hx = lane < 32 ? xs - 1 : xs + W;
    T uv[PX], rv[PX], bv[PX];
    load_cells<T, PX, GUARD, true>(ug, x, n, uv);
    load_cells<T, PX, GUARD, true>(rg, x, n, rv);
    if (!ASSIGN) load_cells<T, PX, GUARD, true>(bg, x, n, bv);
    const T uh = load_cell<T, GUARD>(ug, hx, n, lane);
    T rh = load_cell<T, GUARD>(rg, hx, n, lane);
    bool ok[PX], in[PX];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
        in[e] = GUARD ? (x + e >= 1 && x + e <= n - 2) : true;
        ok[e] = GUARD ? (x + e < n) : true;
        rv[e] = in[e] ? rv[e] : T(0);       // r_bar outside I is never used
    }
    if (GUARD) rh = (hx >= 1 && hx <= n - 2) ? rh : T(0);
    T ul, ur, rl, rr;
    wave_neighbours<T, PX>(uv, uh, lane, ul, ur);
    wave_neighbours<T, PX>(rv, rh, lane, rl, rr);
    T out[PX];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
        const T um = e == 0 ? ul : uv[e - 1];
        const T up = e == PX - 1 ? ur : uv[e + 1];
        const T rm = e == 0 ? rl : rv[e - 1];
        const T rp = e == PX - 1 ? rr : rv[e + 1];
        const T terms = burgers_adjoint_terms(um, uv[e], up, rm, rv[e], rp, C, D, in[e]);
        out[e] = ASSIGN ? terms : bv[e] + terms;
    }
    store_cells<T, PX, GUARD>(bg, x, n, out, ok);
}

// -------------------------------------------------------------------------- kernels
template <class T, int PX, bool GUARD, int OP>
__device__ __forceinline__ void run_segment(const Args1d &a, long xs, int lane)
{
    if (OP == OP_ADJ_WAVE) adj_wave1d_segment<T, PX, GUARD, false>(a, xs, lane);
    else if (OP == OP_ADJ_WAVE_UPREV) adj_wave1d_segment<T, PX, GUARD, true>(a, xs, lane);
    else if (OP == OP_PRI_WAVE) pri_wave1d_segment<T, PX, GUARD>(a, xs, lane);
    else if (OP == OP_PRI_BURGERS) pri_burgers_segment<T, PX, GUARD>(a, xs, lane);
    else if (OP == OP_PRI_BURGERS_KEEP_ENDS) pri_burgers_segment<T, PX, GUARD, true>(a, xs, lane);
    else if (OP == OP_ADJ_BOX) box1d_segment<T, PX, GUARD, true>(a, xs, lane);
    else if (OP == OP_PRI_BOX) box1d_segment<T, PX, GUARD, false>(a, xs, lane);
    else if (OP == OP_ADJ_BURGERS_ASSIGN) adj_burgers_segment<T, PX, GUARD, true>(a, xs, lane);
    else adj_burgers_segment<T, PX, GUARD, false>(a, xs, lane);
}

template <class T, int PX, int OP>
__global__ __launch_bounds__(64 * kWaves1d) void stencil1d_kernel(Args1d a)
{
    constexpr int W = 64 * PX;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long b = blockIdx.x;
    if (b < a.core_blocks) {                       // block-uniform; no barrier in this kernel
        const long local = b * kWaves1d + wave;
        if (local >= a.core_segs) return;
        run_segment<T, PX, false, OP>(a, (1 + local) * W, lane);
    } else {
        const long local = (b - a.core_blocks) * kWaves1d + wave;
        if (local >= a.rem_segs) return;
        const long seg = local == 0 ? 0 : a.core_segs + local;
        run_segment<T, PX, true, OP>(a, seg * W, lane);
    }
}

// Core: segments 1 .. s_hi (all reads inside I, whole vectors inside the array).
// Remainder: segment 0 and segments s_hi+1 .. nseg-1.
template <class T, int PX, int OP>
static hipError_t launch_1d(Args1d a, hipStream_t stream)
{
    constexpr int W = 64 * PX;
    const long n = a.n;
    const long nseg = (n + W - 1) / W;
    long s_hi = (n - 2) / W - 1;                  // last segment with xs + W <= n-2
    if (s_hi < 1) s_hi = 0;                       // no core segment
    a.core_segs = s_hi;
    a.core_blocks = (a.core_segs + kWaves1d - 1) / kWaves1d;
    a.rem_segs = 1 + (nseg - 1 - s_hi);
    const long rem_blocks = (a.rem_segs + kWaves1d - 1) / kWaves1d;
    dim3 grid((unsigned)(a.core_blocks + rem_blocks));
    hipLaunchKernelGGL((stencil1d_kernel<T, PX, OP>), grid, dim3(64 * kWaves1d), 0, stream, a);
    return hipGetLastError();
}

static inline bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

template <int OP>
static hipError_t dispatch_1d(int is_f64, const Args1d &a, hipStream_t stream)
{
    const bool al = aligned16(a.a0) && aligned16(a.a1) && aligned16(a.a2) && aligned16(a.o0) && aligned16(a.o1);
    if (is_f64) return al ? launch_1d<double, 2, OP>(a, stream) : launch_1d<double, 1, OP>(a, stream);
    return al ? launch_1d<float, 4, OP>(a, stream) : launch_1d<float, 1, OP>(a, stream);
}

hipError_t launch_adjoint_wave1d(int is_f64, long n, const void *c, const void *r_bar, void *u_bar,
                                 void *u_prev_bar, hipStream_t stream)
{
    Args1d a{};
    a.a0 = c; a.a1 = r_bar; a.o0 = u_bar; a.o1 = u_prev_bar; a.n = n;
    return u_prev_bar ? dispatch_1d<OP_ADJ_WAVE_UPREV>(is_f64, a, stream)
                      : dispatch_1d<OP_ADJ_WAVE>(is_f64, a, stream);
}
hipError_t launch_primal_wave1d(int is_f64, long n, const void *u, const void *u_prev, const void *c,
                                void *r, hipStream_t stream)
{
    Args1d a{};
    a.a0 = u; a.a1 = u_prev; a.a2 = c; a.o0 = r; a.n = n;
    return dispatch_1d<OP_PRI_WAVE>(is_f64, a, stream);
}
hipError_t launch_adjoint_burgers1d(int is_f64, long n, double C, double D, const void *u,
                                    const void *r_bar, void *u_bar, int assign, hipStream_t stream)
{
    Args1d a{};
    a.a0 = u; a.a1 = r_bar; a.o0 = u_bar; a.n = n; a.C = C; a.D = D;
    return assign ? dispatch_1d<OP_ADJ_BURGERS_ASSIGN>(is_f64, a, stream) : dispatch_1d<OP_ADJ_BURGERS>(is_f64, a, stream);
}
hipError_t launch_primal_burgers1d(int is_f64, long n, double C, double D, const void *u, void *r,
                                   hipStream_t stream, int keep_ends)
{
    Args1d a{};
    a.a0 = u; a.o0 = r; a.n = n; a.C = C; a.D = D;
    return keep_ends ? dispatch_1d<OP_PRI_BURGERS_KEEP_ENDS>(is_f64, a, stream) : dispatch_1d<OP_PRI_BURGERS>(is_f64, a, stream);
}

hipError_t launch_box1d(int adjoint, int is_f64, long n, const double *w, const void *in0, const void *in1,
                        void *out, hipStream_t stream)
{
    Args1d a{};
    a.a0 = in0; a.a1 = in1; a.o0 = out; a.n = n;
    a.w[0] = w[0]; a.w[1] = w[1]; a.w[2] = w[2];
    return adjoint ? dispatch_1d<OP_ADJ_BOX>(is_f64, a, stream) : dispatch_1d<OP_PRI_BOX>(is_f64, a, stream);
}

}  // namespace sadj
