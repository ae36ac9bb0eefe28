// Star stencils on grids that do not fill the chip, and on larger ones whose rows are no whole cache lines (plan_rows in ahead.hpp): a z-march
// whose requests run ahead of the arithmetic.
//
// The kernels of wave3d_adjoint.hip, wave3d_primal.hip and star3d.hip are built for grids of several 10^8 bytes, where memory
// is the bound and one plane in flight per workgroup keeps it busy.  On smaller grids a workgroup marches a few planes only
// and waits for each of them; what counts there is the time from a plane's request to the next plane's.  This march differs in
// three things:
//   - No condition on the plane index around any memory access: arrays are addressed through buffer resources, a plane that is
//     not wanted has a resource of zero bytes or lies beyond it (loads return zero, stores are dropped by the hardware's bounds check), and
//     cells outside the grid or outside I have an offset beyond any plane.  The wait counters therefore know exactly what is
//     outstanding, and D planes are really in flight; with a branch around a load or store the compiler waits for everything.
//     (All slots of the ring of requests are filled and emptied in one order, hence the scheduling barriers; the requests before the loop
//     are followed by as many stores, to nowhere, as those in it.)
//   - The R planes before and after a chunk add to the chunk's sums by their own cell only (a star has no corners): they
//     are read without halo, are not staged in LDS and need no barrier, and the R planes before the chunk are requested together.
//     A chunk of n planes costs n full steps and R cheap ones where the other kernels take n + 2R.
//   - Halo cells move as vectors, 16 bytes (fp32, small tiles: 8) per lane.
// Adjoint, u_bar only, GPU time in us, the kernels named above with the shapes they took before / this: fp64 radius 4
// 40^3 8.7 / 4.3, 80 x 96 x 112 16.6 / 8.5, 128^3 22.9 / 15.7, 200^3 64.9 / 43.3, 256^3 93.3 / 84.0; fp32 radius 4 40^3 6.5 / 4.1,
// 128^3 15.4 / 9.1, 256^3 53.2 / 43.6; fp64 radius 1 128^3 14.8 / 12.1, 200^3 54.1 / 40.4.  128^3 fp64 radius 4: star adjoint 26.6 /
// 16.3, star primal 22.8 / 12.4, wave primal 22.3 / 14.3 (the first of each in the kernels' shapes of larger grids).
// Two planes in flight: one measured 0 to 10 % slower; four, in fp64, up to six times as long.
// A step's own instructions: one resource per array and march instead of one per plane and access takes 40 scalar instructions in two steps
// instead of 115 to 175, next to 80 (radius 1) to 160 vector ones (fp64, 80 x 96 x 112 radius 4 with u_prev_bar 10.8 -> 10.5 us; fp32 star
// primal radius 4 536 x 36 x 176 13.2 -> 11.2; 140 drawn grids 1.01 times as fast, most of them bound by the launch or by memory).
// Registers: the tiles of whole rows leave 128 at radius 1 and 2.  One form spills five of them, the fp32 adjoint of radius 2 that accumulates u_prev_bar in
// rows that are no whole vectors; 300 x 350 x 405 292 -> 192 us all the same, against the tiles of larger grids.
#pragma once
#include "ahead.hpp"

namespace sadj {

// 3 w_0 s + sum_k w_k xs_k + sum_k w_k ys_k
template <class T, int R> __device__ __forceinline__ T wave_in_plane(T s, const T (&xs)[R], const T (&ys)[R])
{
    T t = mul_rounded(T(3.0 * star_w<R>(0)), s);
#pragma unroll
    for (int k = 1; k <= R; ++k) t = fma_t(T(star_w<R>(k)), xs[k - 1], t);
#pragma unroll
    for (int k = 1; k <= R; ++k) t = fma_t(T(star_w<R>(k)), ys[k - 1], t);
    return t;
}

// The same with the largest term last, whose size the other roundings then do not have (fp32 primal, error against 64 bits, centre first / last:
// radius 1 4.41e-8 / 4.26e-8, radius 4 5.01e-8 / 4.54e-8; wave3d_primal.hip 4.34e-8, 4.96e-8).  The adjoint's order is that of its other
// kernels, bit for bit.
template <class T, int R> __device__ __forceinline__ T wave_in_plane_small_first(T s, const T (&xs)[R], const T (&ys)[R])
{
    T t = fma_t(T(star_w<R>(R)), xs[R - 1], mul_rounded(T(star_w<R>(R)), ys[R - 1]));
#pragma unroll
    for (int k = R - 1; k >= 1; --k) t = fma_t(T(star_w<R>(k)), xs[k - 1], fma_t(T(star_w<R>(k)), ys[k - 1], t));
    return fma_t(T(3.0 * star_w<R>(0)), s, t);
}

// A value the compiler must have computed by now (it would otherwise compute it from a slot's registers after the slot's next
// request was issued, and copy the slot to keep both).
template <class T> __device__ __forceinline__ void computed(T &v) { asm volatile("" : "+v"(v)); }

// The same in registers other than those of `v`: of a request's slot a value is taken before the slot's next request, where the
// compiler would otherwise keep it in the slot's registers, request into others, and at the loop's end move (and so wait for) the newest.
__device__ __forceinline__ float taken(float v) { float r; asm volatile("v_mov_b32 %0, %1" : "=&v"(r) : "v"(v)); return r; }
__device__ __forceinline__ double taken(double v)
{
    return __hiloint2double(__float_as_int(taken(__int_as_float(__double2hiint(v)))), __float_as_int(taken(__int_as_float(__double2loint(v)))));
}

// The value of the lane before (AFTER: behind) this one, `edge` where at_edge: the neighbour in x without a way through LDS.
template <bool AFTER> __device__ __forceinline__ float beside(float v, float edge, bool at_edge)
{
    const float r = __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), AFTER ? 0x130 : 0x138, 0xf, 0xf, true));
    return at_edge ? edge : r;
}
template <bool AFTER> __device__ __forceinline__ double beside(double v, double edge, bool at_edge)
{
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), AFTER ? 0x130 : 0x138, 0xf, 0xf, true);
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), AFTER ? 0x130 : 0x138, 0xf, 0xf, true);
    return __hiloint2double(at_edge ? __double2hiint(edge) : hi, at_edge ? __double2loint(edge) : lo);
}

// ---- buffer access
typedef unsigned Dwords2 __attribute__((ext_vector_type(2)));
typedef unsigned Dwords4 __attribute__((ext_vector_type(4)));
constexpr unsigned kNowhere = 0x80000000u;          // an offset beyond every plane that takes this path (below 2^31 bytes)
constexpr int kCached = 0, kStreaming = 2;          // cache policy operand: none, non-temporal

// N cells at a byte offset; dwords at or beyond the resource's size read as zero.  Dword alignment is enough.
template <class T, int N, int POLICY> __device__ __forceinline__ Vec<T, N> buffer_load(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    Vec<T, N> v;
    if constexpr (sizeof(v) == 4) { const unsigned t = __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, POLICY); __builtin_memcpy(&v, &t, 4); }
    else if constexpr (sizeof(v) == 8) { const Dwords2 t = __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, POLICY); __builtin_memcpy(&v, &t, 8); }
    else { const Dwords4 t = __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, POLICY); __builtin_memcpy(&v, &t, 16); }
    return v;
}
template <class T, int N, int POLICY> __device__ __forceinline__ void buffer_store(__amdgpu_buffer_rsrc_t r, unsigned off, const Vec<T, N> &v)
{
    if constexpr (sizeof(v) == 4) { unsigned t; __builtin_memcpy(&t, &v, 4); __builtin_amdgcn_raw_buffer_store_b32(t, r, off, 0, POLICY); }
    else if constexpr (sizeof(v) == 8) { Dwords2 t; __builtin_memcpy(&t, &v, 8); __builtin_amdgcn_raw_buffer_store_b64(t, r, off, 0, POLICY); }
    else { Dwords4 t; __builtin_memcpy(&t, &v, 16); __builtin_amdgcn_raw_buffer_store_b128(t, r, off, 0, POLICY); }
}

// An array along a march: the byte offset of a cell in the plane that step k touches is its offset in a plane plus k planes, counted from
// the plane that step 0 touches (outside the array perhaps, where it is not wanted).  Steps from `first` on touch wanted planes, `count`
// of them from step 0 on; the others get a resource of zero bytes or offsets beyond it.  Two scalar instructions an access, where a
// resource for each plane takes ten.  A chunk (of a grid's z cut) and 16 planes more stay below 2^31 bytes, so that kNowhere stays beyond.
struct MarchedArray {
    char *base;
    int first;
    unsigned size;
    __device__ __forceinline__ MarchedArray(const void *array, int z0, int lo, int hi, unsigned bytes)
        : base(static_cast<char *>(const_cast<void *>(array)) + (long long)z0 * (long long)bytes), first(lo - z0),
          size(hi >= z0 ? (unsigned)(hi + 1 - z0) * bytes : 0u) {}
    __device__ __forceinline__ __amdgpu_buffer_rsrc_t at(int k) const
    {
        return __builtin_amdgcn_make_buffer_rsrc(base, 0, k >= first ? size : 0u, 0x00020000);
    }
};

enum class StarOp { WaveAdjoint, WavePrimal, StarAdjoint, StarPrimal };

// BX x BY: threads of a tile.  BX = 0: tiles of whole rows, of size.bx vectors, whose halo columns lie outside the grid.
template <class T, int R, int BX, int BY, int PX> struct AheadTile {
    static constexpr bool ROWS = BX == 0;
    static constexpr int NT = ROWS ? rows_threads(R) : BX * BY;
    static constexpr int HV = (R + PX - 1) / PX, HX = HV * PX;           // halo columns on a side, in vectors and in cells
    static constexpr int PLANE = ROWS ? NT * PX + 2 * HX * kRowsMaxY + 2 * R * (rows_max_x(R) * PX + 2 * HX) : (BX * PX + 2 * HX) * (BY + 2 * R);
    // halo vectors at most; slots per thread
    static constexpr int NH = ROWS ? 2 * R * rows_max_x(R) : 2 * R * BX + 2 * HV * BY, HS = (NH + NT - 1) / NT;
    static_assert(!ROWS || HS * NT <= 1024, "quotients by the reciprocal");
    RowsTile size;
    __device__ __forceinline__ int bx() const { return ROWS ? size.bx : BX; }
    __device__ __forceinline__ int by() const { return ROWS ? size.by : BY; }
    __device__ __forceinline__ int lx() const { return bx() * PX + 2 * HX; }
    __device__ __forceinline__ int rows(int h) const { return ROWS ? (h * size.reciprocal) >> 20 : h / BX; }
    // LDS coordinates of the first cell of halo vector tid + s * NT: rows above and below the tile, then columns beside it
    __device__ __forceinline__ bool halo_vector(int tid, int s, int &lx, int &ly) const
    {
        const int h = tid + s * NT;
        if (ROWS || h < 2 * R * bx()) {
            const int row = rows(h);
            lx = HX + (h - row * bx()) * PX;
            ly = row < R ? row : row + by();
        } else {
            const int h2 = h - 2 * R * bx(), k = h2 % (2 * HV);
            lx = (k < HV ? k : k + bx()) * PX;
            ly = R + h2 / (2 * HV);
        }
        return h < 2 * R * bx() + (ROWS ? 0 : 2 * HV * by());
    }
};

// One thread: PX consecutive cells of one row.  RAGGED: rows or arrays are not whole vectors, so a row's last vector may reach
// into the next row: its cells there are masked on loading and it is stored cell by cell.
// UPREV (wave adjoint): see wave3d_adjoint.hip.  D: planes in flight.  POLICY: of the arrays without reuse.
template <StarOp OP, class T, int R, int BX, int BY, int PX, int D, int UPREV, int POLICY, bool RAGGED>
__global__ __launch_bounds__((AheadTile<T, R, BX, BY, PX>::NT), 2) void star_ahead_kernel(AheadArgs args)
{
    using G = AheadTile<T, R, BX, BY, PX>;
    const G tile{args.rows};
    using V = Vec<T, PX>;
    constexpr int HS = G::HS, HX = G::HX;
    const int LX = tile.lx();
    constexpr bool ADJ = OP == StarOp::WaveAdjoint || OP == StarOp::StarAdjoint;
    constexpr bool WAVE = OP == StarOp::WaveAdjoint || OP == StarOp::WavePrimal;
    constexpr bool UPRIMAL = OP == StarOp::WavePrimal;
    constexpr bool MASK = ADJ && (RAGGED || R % PX != 0);           // vectors that straddle the edge of I
    constexpr bool PARTIAL = RAGGED || (!ADJ && R % PX != 0);       // vectors that are stored in part
    __shared__ __attribute__((aligned(16))) T sq[2 * G::PLANE];
    const March3dArgs &a = args.m;
    int tix, tiy, zs, ze;
    block_to_tile(a.map, blockIdx.x, tix, tiy, zs, ze);
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    if (!ADJ) {                                     // a primal's outputs are the planes of I
        zs = max(zs, R);
        ze = min(ze, nz - R);
        if (zs >= ze) return;
    }
    const int tid = threadIdx.x, ty = tile.rows(tid), tx = tid - ty * tile.bx();
    const unsigned bytes = (unsigned)nx * (unsigned)ny * (unsigned)sizeof(T);
    const int x0 = tix * tile.bx() * PX, y0 = tiy * tile.by();
    const bool idle = G::ROWS && ty >= tile.by();   // threads that whole rows leave over: cells outside the grid
    const int x = x0 + tx * PX, y = idle ? ny : y0 + ty;
    const int row_at = idle ? R * LX : (R + ty) * LX + tx * PX, own_at = idle ? 0 : row_at + HX;             // (0, 0) is a corner nobody reads
    auto in_I = [&](int xx, int yy) { return xx >= R && xx < nx - R && yy >= R && yy < ny - R; };
    auto in_grid = [&](int xx, int yy) { return xx >= 0 && xx < nx && yy >= 0 && yy < ny; };
    auto offset = [&](int xx, int yy) { return ((unsigned)yy * (unsigned)nx + (unsigned)xx) * (unsigned)sizeof(T); };
    // goff: the vector if any cell lies in the grid, ioff: if any lies in I; woff / poff: the vector if all cells that receive
    // output are there / its single cells if only some are
    bool in[PX], out[PX], any_I = false, all_out = true, any_out = false;
#pragma unroll
    for (int e = 0; e < PX; ++e) {
        in[e] = in_I(x + e, y);
        out[e] = ADJ ? in_grid(x + e, y) : in[e];
        any_I = any_I || in[e];
        all_out = all_out && out[e];
        any_out = any_out || out[e];
    }
    const unsigned goff = in_grid(x, y) ? offset(x, y) : kNowhere, ioff = any_I ? offset(x, y) : kNowhere;
    const unsigned woff = all_out ? offset(x, y) : kNowhere;
    unsigned poff[PX];
#pragma unroll
    for (int e = 0; e < PX; ++e) poff[e] = out[e] && !all_out ? offset(x + e, y) : kNowhere;
    const bool parts = PARTIAL && __any(any_out && !all_out);       // the same in all lanes of a wave
    const unsigned soff = ADJ ? ioff : goff;                         // source field: q on I, u on the grid
    unsigned hoff[HS];
    bool hin[HS][PX];
    int hl[HS];
#pragma unroll
    for (int s = 0; s < HS; ++s) {
        int lx, ly;
        const bool slot = tile.halo_vector(tid, s, lx, ly);
        const int hx = x0 - HX + lx, hy = y0 - R + ly;
        bool any = false;
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            hin[s][e] = slot && (ADJ ? in_I(hx + e, hy) : in_grid(hx + e, hy));
            any = any || hin[s][e];
        }
        hoff[s] = any ? offset(hx, hy) : kNowhere;
        hl[s] = slot ? ly * LX + lx : 0;
    }
    const T w0 = (T)args.w0;
    T wx[2 * R], wy[2 * R], wz[2 * R];
#pragma unroll
    for (int i = 0; i < 2 * R; ++i) { wx[i] = (T)args.w[0][i]; wy[i] = (T)args.w[1][i]; wz[i] = (T)args.w[2][i]; }
    // weight with which plane z adds to plane z + k (before) / z - k (after)
    auto z_weight_up = [&](int k) { return WAVE ? T(star_w<R>(k)) : wz[R - k]; };
    auto z_weight_down = [&](int k) { return WAVE ? T(star_w<R>(k)) : wz[R + k - 1]; };

    // The arrays along the march: step k has plane z = zs - R + k arrive and completes plane zo = z - R.  Source planes that exist: of I
    // (adjoint: q is zero elsewhere), of the grid (primal); halo cells of the chunk's planes only.
    const int z0 = zs - R, zlast = ze - 1 + R;
    const int src_lo = ADJ ? R : 0, src_hi = ADJ ? nz - R - 1 : nz - 1;
    const MarchedArray in0(a.in0, z0, src_lo, min(zlast, src_hi), bytes), in0h(a.in0, z0, src_lo, min(ze - 1, src_hi), bytes);
    const MarchedArray in1(a.in1, z0, src_lo, min(zlast, src_hi), bytes), in1h(a.in1, z0, src_lo, min(ze - 1, src_hi), bytes);
    const MarchedArray out0(a.out0, z0 - R, zs, ze - 1, bytes);
    // what the completing output plane is combined with: start value (wave adjoint), u_bar (star adjoint), c (primals); r_bar (UPREV 4), u_prev (wave primal)
    const MarchedArray with0(OP == StarOp::WaveAdjoint ? (UPREV >= 3 ? a.in2 : a.out0) : OP == StarOp::StarAdjoint ? a.out0 : UPRIMAL ? a.in2 : a.in1,
                             z0 - R, zs, ze - 1, bytes);
    const MarchedArray with1(a.in1, z0 - R, zs, ze - 1, bytes);
    // u_prev_bar of the arriving plane: where it is accumulated (UPREV 1) of I only; of the completing plane (UPREV 4)
    const MarchedArray prev(a.out1, z0, max(zs, UPREV == 1 ? R : 0), UPREV == 1 ? min(ze - 1, nz - R - 1) : ze - 1, bytes), prev4(a.out1, z0 - R, zs, ze - 1, bytes);

    // values in flight; s0 (, s1): the source field's factors; o0 (, o1): what the completing output plane is combined with
    // (wave adjoint: start value, UPREV 4: r_bar; star adjoint: u_bar; wave primal: c, u_prev; star primal: c);
    // pv: u_prev_bar of the arriving plane (UPREV 1)
    V s0[D], s1[D], o0[D], o1[D], pv[D], h0[D][HS], h1[D][HS];
    auto issue = [&](int k, int d) {
        const unsigned zoff = (unsigned)k * bytes;
        s0[d] = buffer_load<T, PX, kCached>(in0.at(k), soff + zoff);
        if (ADJ) {
            s1[d] = buffer_load<T, PX, kCached>(in1.at(k), soff + zoff);
            if (UPREV == 1) pv[d] = buffer_load<T, PX, POLICY>(prev.at(k), goff + zoff);
#pragma unroll
            for (int s = 0; s < HS; ++s) {
                h0[d][s] = buffer_load<T, PX, kCached>(in0h.at(k), hoff[s] + zoff);
                h1[d][s] = buffer_load<T, PX, kCached>(in1h.at(k), hoff[s] + zoff);
            }
        } else {
#pragma unroll
            for (int s = 0; s < HS; ++s) h0[d][s] = buffer_load<T, PX, kCached>(in0h.at(k), hoff[s] + zoff);
        }
    };
    auto issue_out = [&](int k, int d) {
        const unsigned off = (ADJ ? goff : ioff) + (unsigned)k * bytes;
        o0[d] = buffer_load<T, PX, POLICY>(with0.at(k), off);
        if (UPRIMAL || (OP == StarOp::WaveAdjoint && UPREV == 4)) o1[d] = buffer_load<T, PX, POLICY>(with1.at(k), off);
    };
    auto store_out = [&](__amdgpu_buffer_rsrc_t r, unsigned zoff, const V &o) {
        buffer_store<T, PX, POLICY>(r, woff + zoff, o);
        if (PARTIAL && parts) {
#pragma unroll
            for (int e = 0; e < PX; ++e) buffer_store<T, 1, POLICY>(r, poff[e] + zoff, Vec<T, 1>{{o.v[e]}});
        }
    };
    auto source = [&](T f0, T f1, bool inside) {
        if (!ADJ) return f0;
        const T q = mul_rounded(f0, f1);
        return MASK ? (inside ? q : T(0)) : q;
    };

    // acc[k]: running sum of output plane z - R + k, z the arriving plane; the last one, z + R, starts at zero.
    // hist[k] (wave primal): u of plane z - 1 - k
    T acc[PX][2 * R + 1], hist[PX][R];
#pragma unroll
    for (int e = 0; e < PX; ++e) {
#pragma unroll
        for (int k = 0; k <= 2 * R; ++k) acc[e][k] = T(0);
#pragma unroll
        for (int k = 0; k < R; ++k) hist[e][k] = T(0);
    }

    auto step = [&](int k, int d) {
        const int z = z0 + k, zo = z - R;
        const unsigned zoff = (unsigned)k * bytes;
        T *sb = sq + (k & 1) * G::PLANE;
        T own[PX], rr[PX], r2[PX];
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            own[e] = source(s0[d].v[e], s1[d].v[e], in[e]);
            if (OP == StarOp::WaveAdjoint) {
                rr[e] = MASK ? (in[e] ? s1[d].v[e] : T(0)) : s1[d].v[e];
                r2[e] = rr[e] + rr[e];
            }
        }
        if (z < ze) {
            V v;
#pragma unroll
            for (int e = 0; e < PX; ++e) v.v[e] = own[e];
            st_vec<T, PX>(sb + own_at, v);
#pragma unroll
            for (int s = 0; s < HS; ++s) {
#pragma unroll
                for (int e = 0; e < PX; ++e) v.v[e] = source(h0[d][s].v[e], h1[d][s].v[e], hin[s][e]);
                st_vec<T, PX>(sb + hl[s], v);
            }
        }
        if (OP == StarOp::WaveAdjoint && (UPREV == 1 || UPREV == 2)) {
            V o;
#pragma unroll
            for (int e = 0; e < PX; ++e) o.v[e] = (UPREV == 1 ? pv[d].v[e] : T(0)) - rr[e];
            store_out(prev.at(k), zoff, o);
        }
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            computed(own[e]);
            if (OP == StarOp::WaveAdjoint) computed(r2[e]);
        }
        issue(k + D, d);
        if (z < ze) {
            __syncthreads();
            T row[PX + 2 * HX];
            V col[2 * R + 1];
            const T *at = sb + row_at;
#pragma unroll
            for (int i = 0; i < PX + 2 * HX; i += PX) {
                if (i == HX) continue;
                const V t = ld_vec<T, PX>(at + i);
#pragma unroll
                for (int e = 0; e < PX; ++e) row[i + e] = t.v[e];
            }
#pragma unroll
            for (int e = 0; e < PX; ++e) row[HX + e] = own[e];
#pragma unroll
            for (int k = -R; k <= R; ++k)
                if (k != 0) col[R + k] = ld_vec<T, PX>(at + HX + k * LX);
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                if (WAVE) {
                    T xs[R], ys[R];
#pragma unroll
                    for (int k = 1; k <= R; ++k) {
                        xs[k - 1] = add_rounded(row[HX + e - k], row[HX + e + k]);
                        ys[k - 1] = add_rounded(col[R - k].v[e], col[R + k].v[e]);
                    }
                    const T t = UPRIMAL ? wave_in_plane_small_first<T, R>(own[e], xs, ys) : wave_in_plane<T, R>(own[e], xs, ys);
                    acc[e][R] = add_rounded(acc[e][R], OP == StarOp::WaveAdjoint ? add_rounded(r2[e], t) : t);
                } else if (R == 1) {
                    // one sum, from the planes before to the centre: seven roundings, where axes summed by themselves have nine and an in-plane sum,
                    // centre first, eight of larger values (fp32 primal, error against 64 bits, in-plane sum / each axis by itself / this: random
                    // weights 5.81e-8 / 5.82e-8 / 5.70e-8, one-sided ones 4.98e-8 / 5.21e-8 / 4.67e-8, 7-point Laplacian 7.07e-8 / 5.71e-8 / 4.68e-8;
                    // star3d.hip 5.89e-8, 5.41e-8, 6.28e-8; from one set of weights to another 0.77 to 1.19 times the in-plane sum's)
                    const T t = fma_t(wx[1], row[HX + e + 1], fma_t(wx[0], row[HX + e - 1], acc[e][1]));
                    acc[e][1] = fma_t(w0, own[e], fma_t(wy[1], col[2].v[e], fma_t(wy[0], col[0].v[e], t)));
                } else {
                    // each axis summed by itself: partial sums and with them their roundings are smaller (fp32 primal, error against 64
                    // bits, one sum / this: radius 2 2.50e-8 / 2.39e-8, radius 4 2.27e-8 / 2.07e-8; star3d.hip 2.43e-8, 2.12e-8)
                    T tx = mul_rounded(wx[R - 1], row[HX + e - 1]), ty = mul_rounded(wy[R - 1], col[R - 1].v[e]);
#pragma unroll
                    for (int k = 1; k <= R; ++k) {
                        if (k > 1) {
                            tx = fma_t(wx[R - k], row[HX + e - k], tx);
                            ty = fma_t(wy[R - k], col[R - k].v[e], ty);
                        }
                        tx = fma_t(wx[R + k - 1], row[HX + e + k], tx);
                        ty = fma_t(wy[R + k - 1], col[R + k].v[e], ty);
                    }
                    const T t = add_rounded(fma_t(w0, own[e], tx), ty);
                    acc[e][R] = add_rounded(acc[e][R], t);
                }
#pragma unroll
                for (int k = 1; k <= R; ++k) acc[e][R + k] = fma_t(z_weight_up(k), own[e], acc[e][R + k]);
            }
        }
#pragma unroll
        for (int e = 0; e < PX; ++e)
#pragma unroll
            for (int k = 1; k <= R; ++k) acc[e][R - k] = fma_t(z_weight_down(k), own[e], acc[e][R - k]);
        const bool zin = zo >= R && zo < nz - R;
        V o;
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            if (OP == StarOp::WaveAdjoint) {
                const T start = UPREV >= 3 ? (zin && in[e] ? T(0) - o0[d].v[e] : T(0)) : o0[d].v[e];
                o.v[e] = add_rounded(start, acc[e][0]);
            } else if (OP == StarOp::StarAdjoint) {
                o.v[e] = add_rounded(o0[d].v[e], acc[e][0]);
            } else if (OP == StarOp::WavePrimal) {
                o.v[e] = fma_t(o0[d].v[e], acc[e][0], fma_t(T(2), hist[e][R - 1], T(0) - o1[d].v[e]));
            } else {
                o.v[e] = mul_rounded(o0[d].v[e], acc[e][0]);
            }
        }
        store_out(out0.at(k), zoff, o);
        if (OP == StarOp::WaveAdjoint && UPREV == 4) {
#pragma unroll
            for (int e = 0; e < PX; ++e) o.v[e] = zin && in[e] ? T(0) - o1[d].v[e] : T(0);
            store_out(prev4.at(k), zoff, o);
        }
        issue_out(k + D, d);
#pragma unroll
        for (int e = 0; e < PX; ++e) {
#pragma unroll
            for (int k = 0; k < 2 * R; ++k) { acc[e][k] = acc[e][k + 1]; computed(acc[e][k]); }
            acc[e][2 * R] = T(0);
            if (UPRIMAL) {
#pragma unroll
                for (int k = R - 1; k > 0; --k) { hist[e][k] = hist[e][k - 1]; computed(hist[e][k]); }
                hist[e][0] = own[e];
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    // the R planes before the chunk, together
    V f0[R], f1[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
        f0[j] = buffer_load<T, PX, kCached>(in0.at(j), soff + (unsigned)j * bytes);
        if (ADJ) f1[j] = buffer_load<T, PX, kCached>(in1.at(j), soff + (unsigned)j * bytes);
    }
    __builtin_amdgcn_sched_barrier(0);
    // as many stores as in a step (here to nowhere), or the loop's waits would have to suit both counts
#pragma unroll
    for (int d = 0; d < D; ++d) {
        if (OP == StarOp::WaveAdjoint && (UPREV == 1 || UPREV == 2)) buffer_store<T, PX, POLICY>(prev.at(-1), kNowhere, V{});
        issue(R + d, d);
        buffer_store<T, PX, POLICY>(out0.at(-1), kNowhere, V{});
        if (OP == StarOp::WaveAdjoint && UPREV == 4) buffer_store<T, PX, POLICY>(prev4.at(-1), kNowhere, V{});
        issue_out(R + d, d);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int j = 0; j < R; ++j)
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            const T q = source(f0[j].v[e], f1[j].v[e], in[e]);
            // plane zs - R + j adds to planes zs .. zs + j
#pragma unroll
            for (int i = 0; i <= j; ++i) acc[e][R + i] = fma_t(z_weight_up(R - j + i), q, acc[e][R + i]);
            if (UPRIMAL) hist[e][R - 1 - j] = q;
        }
    if (G::ROWS) {                                   // halo columns, of both planes in LDS
        for (int i = tid; i < 2 * HX * tile.by(); i += G::NT) {
            const int row = i / (2 * HX), col = i % (2 * HX);
            T *at = sq + (R + row) * LX + (col < HX ? col : col + tile.bx() * PX);
            at[0] = at[G::PLANE] = T(0);
        }
    }
    const int end = zlast - z0;
    int k = R;
    for (; k + D - 1 <= end; k += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) step(k + d, d);
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d) {
        if (k + d > end) return;
        step(k + d, d);
    }
}

template <StarOp OP, class T, int R, int UPREV, int BX, int BY, int PX, int POLICY, bool RAGGED>
static hipError_t launch_ahead_kernel(const AheadArgs &a, unsigned pad, hipStream_t stream)
{
    hipLaunchKernelGGL((star_ahead_kernel<OP, T, R, BX, BY, PX, 2, UPREV, POLICY, RAGGED>), dim3(a.m.map.total_blocks),
                       dim3(AheadTile<T, R, BX, BY, PX>::NT), pad, stream, a);
    return hipGetLastError();
}

// Rows that are not whole vectors take the RAGGED instantiations; an array need only be aligned to its elements.
template <StarOp OP, class T, int R, int UPREV> static hipError_t launch_ahead(AheadShape shape, const AheadArgs &a, unsigned pad, hipStream_t stream)
{
    constexpr int PXV = 16 / sizeof(T);
    constexpr int RX = sizeof(T) == 8 ? 32 : 16, RY = sizeof(T) == 8 ? 16 : 32;      // threads of the ragged wide tile
    const bool whole = a.m.nx % (shape == AheadShape::Small ? 2 : PXV) == 0;
    switch (shape) {
    case AheadShape::Small:
        return whole ? launch_ahead_kernel<OP, T, R, UPREV, 16, 16, 2, kCached, false>(a, pad, stream)
                     : launch_ahead_kernel<OP, T, R, UPREV, 16, 16, 2, kCached, true>(a, pad, stream);
    case AheadShape::Wide:
        return whole ? launch_ahead_kernel<OP, T, R, UPREV, 32, 16, PXV, kCached, false>(a, pad, stream)
                     : launch_ahead_kernel<OP, T, R, UPREV, RX, RY, PXV, kCached, true>(a, pad, stream);
    case AheadShape::WideStream:
        return whole ? launch_ahead_kernel<OP, T, R, UPREV, 32, 16, PXV, kStreaming, false>(a, pad, stream)
                     : launch_ahead_kernel<OP, T, R, UPREV, RX, RY, PXV, kStreaming, true>(a, pad, stream);
    case AheadShape::Rows:                           // loops only, see plan_rows
        if constexpr (OP == StarOp::WaveAdjoint && UPREV >= 3)
            return whole ? launch_ahead_kernel<OP, T, R, UPREV, 0, 0, PXV, kCached, false>(a, pad, stream)
                         : launch_ahead_kernel<OP, T, R, UPREV, 0, 0, PXV, kCached, true>(a, pad, stream);
        else return hipErrorNotSupported;
    case AheadShape::RowsStream:
        return whole ? launch_ahead_kernel<OP, T, R, UPREV, 0, 0, PXV, kStreaming, false>(a, pad, stream)
                     : launch_ahead_kernel<OP, T, R, UPREV, 0, 0, PXV, kStreaming, true>(a, pad, stream);
    default: return hipErrorNotSupported;
    }
}

}  // namespace sadj
