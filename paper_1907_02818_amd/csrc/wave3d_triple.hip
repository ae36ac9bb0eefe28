// Three reverse steps of a time loop of radius-1 wave steps in one pass over the data: the two-step march of
// wave3d_pair.hip with one more stage.  With a = lam^{k+1}, b = lam^k, m the indicator of I and S the
// 7-point star,
//     a1 = b + 2 a m + S(c a m),   a2 = -a m + 2 a1 m + S(c a1 m),   a3 = -a1 m + 2 a2 m + S(c a2 m)
// and the pass reads a, b, c and writes a3 and -a2 m: 40 bytes per cell (fp64) for three steps.
//
// In step zi of the march stage 1 reads plane zi of q0 = c a m and completes a1 of plane zi-1, stage 2 reads
// q1 = c a1 m of plane zi-2 and completes a2 of plane zi-3, stage 3 reads q2 = c a2 m of plane zi-4 and
// completes a3 of plane zi-5.  A tile needs a2 on itself and the cells next to it (D1), a1 also two cells
// out (D2) and q0 three cells out (D3); distances are counted in cells along x plus along y, so
// the frames have cut corners.  The first threads own one frame cell each (fp32: two): D1 cells run stages 1
// and 2, D2 cells stage 1.  All three LDS planes are double-buffered and one barrier per step serves
// all.  Values outside I are replaced by zero with selects, never by a multiplication.
//
// What bounds it: registers first.  A spill costs more than its own traffic, because a reload waits for
// all loads in flight.  512 threads with 256 registers hold three sums per stage and owned cell because
// q1 and q2 go to LDS as soon as they are formed, c of older planes waits in LDS (all but 320 bytes of the
// 160 KB are used in fp64), and all LDS planes share one geometry.  Then memory: 512^3 fp64, a pass
// takes 1.02 ms = 5.2 TB/s on its 40 bytes per cell (a two-step pass 0.95 ms), 0.34 ms per step against 0.48.
#include "ahead3d.hpp"
#include "launch.hpp"
#include "tile3d.hpp"

#include <type_traits>

namespace sadj {

struct TripleArgs {
    const void *c, *a, *b;
    void *out_a, *out_b;
    int nx, ny, nz;
    TileMap map;
};

template <class T, int BX, int BY, int PY, int PX> struct TripleTile {
    static constexpr int TX = BX * PX, TY = BY * PY, NT = BX * BY;
    // all LDS planes have the geometry of the widest, origin (x0-3, y0-3), so that a cell has one address in
    // all of them (three geometries need more address registers than the kernel has)
    static constexpr int LX = TX + 6, PLANE = LX * (TY + 6);
    static constexpr int SIDE = 2 * TX + 2 * TY;
    static constexpr int N1 = SIDE, N2 = SIDE + 4, N3 = SIDE + 8;           // cells of D1, D2, D3
    static constexpr int NFRAME = N1 + N2 + N3;
    static constexpr int HS = (NFRAME + NT - 1) / NT;
    static constexpr int RS = (N1 + N2 + NT - 1) / NT;                      // slots whose cells run stage 1
    static_assert(N1 <= NT, "one cell that runs stage 2 per thread");

    // Frame slot s of thread tid -> coordinates in the q0 plane; false if the slot is unused.
    __device__ static __forceinline__ bool frame_cell(int tid, int s, int &lx, int &ly)
    {
        int h = tid + s * NT;
        const bool used = h < NFRAME;
        const int d = h < N1 ? 1 : h < N1 + N2 ? 2 : 3;
        h -= d == 1 ? 0 : d == 2 ? N1 : N1 + N2;
        int x, y;
        if (h < 2 * TX) {                       // rows d above and below
            x = h % TX;
            y = h < TX ? -d : TY - 1 + d;
        } else if (h < SIDE) {                  // columns d left and right
            h -= 2 * TX;
            x = (h & 1) ? TX - 1 + d : -d;
            y = h / 2;
        } else {                                // corners: d-1 cells each, i+1 out in x and d-1-i in y
            h -= SIDE;
            const int i = h >> 2;
            x = (h & 1) ? TX + i : -1 - i;
            y = (h & 2) ? TY + d - 2 - i : 1 - d + i;
        }
        lx = x + 3;
        ly = y + 3;
        return used;
    }
};

template <class T, int BX, int BY, int PY, int PX, bool GUARD>
__device__ __forceinline__ void triple_march(const TripleArgs &a, int tix, int tiy, int zs, int ze, T *__restrict__ sq0,
                                             T *__restrict__ sq1, T *__restrict__ sq2, Vec<T, PX> *__restrict__ cold, T *__restrict__ coldr)
{
    using G = TripleTile<T, BX, BY, PY, PX>;
    using V = Vec<T, PX>;
    constexpr int TX = G::TX, TY = G::TY, LX = G::LX, HS = G::HS, RS = G::RS;
    constexpr T W0 = T(3.0 * star_w<1>(0)), W1 = T(star_w<1>(1));
    const int tid = threadIdx.x;
    const int tx = tid % BX, ty = tid / BX;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const size_t plane = (size_t)nx * ny;
    const int x0 = tix * TX, y0 = tiy * TY;

    const T *__restrict__ cg = static_cast<const T *>(a.c);
    const T *__restrict__ ag = static_cast<const T *>(a.a);
    const T *__restrict__ bg = static_cast<const T *>(a.b);
    T *__restrict__ oag = static_cast<T *>(a.out_a);
    T *__restrict__ obg = static_cast<T *>(a.out_b);

    TileAddr<PX, PY, HS, GUARD> ad;
    ad.init(tx, ty, x0, y0, nx, ny, 1, 3, LX, 0 /* plane corner, never read */, (uint32_t)sizeof(T),
            [&](int s, int &lx, int &ly) { return G::frame_cell(tid, s, lx, ly); });
    const uint32_t dummy = ad.dummy;
    uint32_t ooff[PY];
    bool ouse[PY][PX], ostore[PY];
#pragma unroll
    for (int p = 0; p < PY; ++p) {
        ostore[p] = ad.own_grid[p];
        ooff[p] = ad.own_off[p];             // inside the grid, so that loads need no guard of their own
#pragma unroll
        for (int e = 0; e < PX; ++e) ouse[p][e] = ad.own_I[p][e];
    }
    // the thread's vector of row p in a plane: core tiles need the offset of the first row only
    auto row = [&](auto *base, int p) { return base + (GUARD ? 0 : (size_t)p * nx); };
    auto off = [&](int p) { return ooff[GUARD ? p : 0]; };
    uint32_t hoff[HS];
    uint32_t hpack = 0;
    bool huse[HS];
#pragma unroll
    for (int s = 0; s < HS; ++s) {
        huse[s] = ad.halo_I[s];
        hoff[s] = huse[s] ? ad.halo_off[s] : dummy;
        hpack |= (uint32_t)ad.halo_lds[s] << (16 * s);
    }
    static_assert(HS <= 2 && G::PLANE <= 65536, "two LDS indexes share a register");
    auto hlds = [&](int s) { return s == 0 ? hpack & 0xffffu : hpack >> 16; };
    // the frame cells of this thread that run stage 1 (D1, D2) and stage 2 (D1: slot 0, whole waves)
    bool ring1[RS], ruse[RS];
    const bool ring2 = tid < G::N1;
#pragma unroll
    for (int s = 0; s < RS; ++s) {
        ring1[s] = tid + s * G::NT < G::N1 + G::N2;
        ruse[s] = ring1[s] && huse[s];
    }
    const int own = (3 + ty * PY) * LX + 3 + tx * PX;

    // running sums of the three stages: index 0 = the plane that completes in this step
    T acc1[PY][PX][3], acc2[PY][PX][3], acc3[PY][PX][3], acc1r[RS][3], acc2r[3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        acc2r[k] = T(0);
#pragma unroll
        for (int s = 0; s < RS; ++s) acc1r[s][k] = T(0);
#pragma unroll
        for (int p = 0; p < PY; ++p)
#pragma unroll
            for (int e = 0; e < PX; ++e) acc1[p][e][k] = acc2[p][e][k] = acc3[p][e][k] = T(0);
    }
    // c and a1 m of the plane before (c of the two planes before that waits in LDS, where only its own thread
    // touches it)
    T c1[PY][PX], a1m[PY][PX], c1r[RS], sbr[RS];
#pragma unroll
    for (int i = 0; i < 2 * PY; ++i) cold[i * G::NT + tid] = V{};
    if (ring2) coldr[tid] = coldr[G::N1 + tid] = T(0);
#pragma unroll
    for (int s = 0; s < RS; ++s) c1r[s] = sbr[s] = T(0);
#pragma unroll
    for (int p = 0; p < PY; ++p)
#pragma unroll
        for (int e = 0; e < PX; ++e) c1[p][e] = a1m[p][e] = T(0);
    bool q1_valid = false, q2_valid = false;     // the planes of q1 and q2 that this step reads were staged by the last one

    V sa[PY], sc[PY], sb[PY];
    T sha[HS], shc[HS];
#pragma unroll
    for (int p = 0; p < PY; ++p) { sa[p] = V{}; sc[p] = V{}; sb[p] = V{}; }
#pragma unroll
    for (int s = 0; s < HS; ++s) sha[s] = shc[s] = T(0);

    auto plane_in_I = [&](int z) { return z >= 1 && z < nz - 1; };
    const int zi0 = zs - 3, zi1 = ze + 2;        // q0 planes that reach the outputs [zs, ze)
    auto a1_wanted = [&](int z) { return z >= zs - 2 && z <= ze + 1 && plane_in_I(z); };
    auto a2_wanted = [&](int z) { return z >= zs - 1 && z <= ze && plane_in_I(z); };

    // request what step z consumes: a and c of plane z (tile and frame), and, once the values of the step
    // before are used up, b of plane z-1 (tile, D1 and D2); `steady`: every condition on the plane
    // index holds
    auto issue = [&](int z, auto steady) {
        constexpr bool ST = decltype(steady)::value;
        if (ST || (z <= zi1 && plane_in_I(z))) {
            const T *cp = cg + (size_t)z * plane;
            const T *ap = ag + (size_t)z * plane;
#pragma unroll
            for (int p = 0; p < PY; ++p) {
                sc[p] = ld_vec_off<T, PX, false>(row(cp, p), off(p));
                sa[p] = ld_vec_off<T, PX, false>(row(ap, p), off(p));
            }
#pragma unroll
            for (int s = 0; s < HS; ++s) { shc[s] = ld_off(cp, hoff[s]); sha[s] = ld_off(ap, hoff[s]); }
        }
    };
    auto issue_b = [&](int z, auto steady) {
        constexpr bool ST = decltype(steady)::value;
        if (ST || a1_wanted(z)) {
            const T *bp = bg + (size_t)z * plane;
#pragma unroll
            for (int p = 0; p < PY; ++p) sb[p] = ld_vec_off<T, PX, false>(row(bp, p), off(p));
#pragma unroll
            for (int s = 0; s < RS; ++s) sbr[s] = ld_off(bp, hoff[s]);
        }
    };
    // the star of one staged plane at a thread's tile cells and its sums: planes before, at and after
    // (the thread's own values of q are read back: kept in registers from staging to here they cost spills)
    auto star = [&](const T *sp, T (&acc)[PY][PX][3]) {
        T q[PY][PX];
#pragma unroll
        for (int p = 0; p < PY; ++p)
#pragma unroll
            for (int e = 0; e < PX; ++e) q[p][e] = sp[own + p * LX + e];
#pragma unroll
        for (int p = 0; p < PY; ++p)
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                const T *at = sp + own + p * LX + e;
                const T left = e > 0 ? q[p][e - 1] : at[-1];
                const T right = e < PX - 1 ? q[p][e + 1] : at[1];
                const T up = p > 0 ? q[p - 1][e] : at[-LX];
                const T down = p < PY - 1 ? q[p + 1][e] : at[LX];
                acc[p][e][1] += W0 * q[p][e] + W1 * (left + right) + W1 * (up + down);
                acc[p][e][0] += W1 * q[p][e];
                acc[p][e][2] += W1 * q[p][e];
            }
    };
    auto star_ring = [&](const T *at, T (&acc)[3]) {
        const T q = at[0];
        acc[1] += W0 * q + W1 * (at[-1] + at[1]) + W1 * (at[-LX] + at[LX]);
        acc[0] += W1 * q;
        acc[2] += W1 * q;
    };

    issue(zi0, std::false_type{});
    issue_b(zi0 - 1, std::false_type{});
    int buf = 0;
    auto step = [&](int zi, auto steady) {
        constexpr bool ST = decltype(steady)::value;
        const bool zin = ST || (zi <= zi1 && plane_in_I(zi));
        // what this step reads (s0 is staged now), and where it leaves q1 and q2 for the next step: the buffers
        // that the step before last wrote and the last one read, which every thread has left at the barrier
        T *s0 = sq0 + buf * G::PLANE;
        const T *s1 = sq1 + buf * G::PLANE, *s2 = sq2 + buf * G::PLANE;
        T *n1 = sq1 + (buf ^ 1) * G::PLANE, *n2 = sq2 + (buf ^ 1) * G::PLANE;
        T am[PY][PX], cc[PY][PX], amr[RS], ccr[RS];
#pragma unroll
        for (int s = 0; s < RS; ++s) amr[s] = ccr[s] = T(0);
        if (zin) {
#pragma unroll
            for (int p = 0; p < PY; ++p)
#pragma unroll
                for (int e = 0; e < PX; ++e) {
                    const T cv = sc[p].v[e], av = sa[p].v[e];
                    cc[p][e] = cv;
                    am[p][e] = GUARD ? (ouse[p][e] ? av : T(0)) : av;
                    s0[own + p * LX + e] = GUARD ? (ouse[p][e] ? cv * av : T(0)) : cv * av;
                }
#pragma unroll
            for (int s = 0; s < HS; ++s) {
                const T qq = GUARD ? (huse[s] ? shc[s] * sha[s] : T(0)) : shc[s] * sha[s];
                s0[hlds(s)] = qq;
                if (s < RS) { ccr[s] = shc[s]; amr[s] = GUARD ? (huse[s] ? sha[s] : T(0)) : sha[s]; }
            }
        } else {
#pragma unroll
            for (int p = 0; p < PY; ++p)
#pragma unroll
                for (int e = 0; e < PX; ++e) cc[p][e] = am[p][e] = T(0);
        }
        issue(zi + 1, steady);
        __syncthreads();

        // ---- stage 3: q2 of plane zi-4; a3 of plane zi-5 is complete
        if (ST || q2_valid) star(s2, acc3);
        const int zo3 = zi - 5;
        if (ST || (zo3 >= zs && zo3 < ze)) {
            T *op = oag + (size_t)zo3 * plane;
#pragma unroll
            for (int p = 0; p < PY; ++p) {
                V o;
#pragma unroll
                for (int e = 0; e < PX; ++e) o.v[e] = acc3[p][e][0];
                if (!GUARD || ostore[p]) st_vec_off<T, PX, true>(row(op, p), off(p), o);
            }
        }

        // ---- stage 2: q1 of plane zi-2; a2 of plane zi-3 is complete
        if (ST || q1_valid) {
            star(s1, acc2);
            if (ring2) star_ring(s1 + hlds(0), acc2r);
        }
        const int zo2 = zi - 3;
        q2_valid = ST || a2_wanted(zo2);
#pragma unroll
        for (int p = 0; p < PY; ++p) {
            const V c3 = cold[(buf * PY + p) * G::NT + tid];
            V o, keep;
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                const T a2m = q2_valid && (!GUARD || ouse[p][e]) ? acc2[p][e][0] : T(0);
                if (q2_valid) n2[own + p * LX + e] = !GUARD || ouse[p][e] ? c3.v[e] * a2m : T(0);
                acc3[p][e][0] = acc3[p][e][1];
                acc3[p][e][1] = acc3[p][e][2] + T(2) * a2m;
                acc3[p][e][2] = -a1m[p][e];                                   // of plane zi-2
                acc2[p][e][0] = acc2[p][e][1];
                acc2[p][e][1] = acc2[p][e][2];
                acc2[p][e][2] = -am[p][e];                                    // of plane zi
                keep.v[e] = c1[p][e];
                o.v[e] = -a2m;
            }
            cold[(buf * PY + p) * G::NT + tid] = keep;
            if (ST || (zo2 >= zs && zo2 < ze))       // zero on planes outside I
                if (!GUARD || ostore[p]) st_vec_off<T, PX, true>(row(obg + (size_t)zo2 * plane, p), off(p), o);
        }
        if (ring2) {
            T *cr = coldr + buf * G::N1 + tid;
            if (q2_valid) n2[hlds(0)] = ruse[0] ? *cr * acc2r[0] : T(0);
            *cr = c1r[0];
        }
        acc2r[0] = acc2r[1]; acc2r[1] = acc2r[2]; acc2r[2] = -amr[0];

        // ---- stage 1: q0 of plane zi; a1 of plane zi-1 is complete
        if (zin) {
            star(s0, acc1);
#pragma unroll
            for (int s = 0; s < RS; ++s)
                if (ring1[s]) star_ring(s0 + hlds(s), acc1r[s]);
        }
        q1_valid = ST || a1_wanted(zi - 1);
#pragma unroll
        for (int p = 0; p < PY; ++p)
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                const T v = acc1[p][e][0] + sb[p].v[e];
                a1m[p][e] = q1_valid && (!GUARD || ouse[p][e]) ? v : T(0);
                if (q1_valid) n1[own + p * LX + e] = !GUARD || ouse[p][e] ? c1[p][e] * v : T(0);
                acc2[p][e][1] += T(2) * a1m[p][e];
                acc1[p][e][0] = acc1[p][e][1] + T(2) * am[p][e];
                acc1[p][e][1] = acc1[p][e][2];
                acc1[p][e][2] = T(0);
                c1[p][e] = cc[p][e];
            }
#pragma unroll
        for (int s = 0; s < RS; ++s) {
            const T v = acc1r[s][0] + sbr[s];
            const T a1 = q1_valid && ruse[s] ? v : T(0);
            if (q1_valid && ring1[s]) n1[hlds(s)] = ruse[s] ? c1r[s] * v : T(0);
            if (s == 0) acc2r[1] += T(2) * a1;
            acc1r[s][0] = acc1r[s][1] + T(2) * amr[s];
            acc1r[s][1] = acc1r[s][2];
            acc1r[s][2] = T(0);
            c1r[s] = ccr[s];
        }
        issue_b(zi, steady);
        buf ^= 1;
    };
    // steady steps: planes zi-4 .. zi+1 lie in I, the output planes zi-5 and zi-3 in this chunk
    const int lo = zs + 5, hi = min(ze + 1, nz - 3);
    int zi = zi0;
    for (; zi <= ze + 4 && zi < lo; ++zi) step(zi, std::false_type{});
    // (guarded fp64 tiles have no register left for a second copy of the step: it would spill, and a reload
    // waits for every load in flight)
    if constexpr (!GUARD || sizeof(T) == 4) {
        __builtin_amdgcn_s_waitcnt(0x0F70);      // enter the steady loop with nothing outstanding (vmcnt(0))
        for (; zi <= hi; ++zi) step(zi, std::true_type{});
    }
    for (; zi <= ze + 4; ++zi) step(zi, std::false_type{});
}

template <class T, int BX, int BY, int PY, int PX>
__global__ __launch_bounds__(BX *BY) void adj_wave3d_triple_kernel(TripleArgs a)
{
    using G = TripleTile<T, BX, BY, PY, PX>;
    __shared__ T sq0[2 * G::PLANE];
    __shared__ T sq1[2 * G::PLANE];
    __shared__ T sq2[2 * G::PLANE];
    __shared__ Vec<T, PX> cold[2 * PY * G::NT];
    __shared__ T coldr[2 * G::N1];
    int tix, tiy, zs, ze;
    block_to_tile(a.map, blockIdx.x, tix, tiy, zs, ze);
    // core tile: the tile and its frame lie in I in x and y
    const int x0 = tix * G::TX, y0 = tiy * G::TY;
    const bool core = x0 >= 4 && x0 + G::TX + 4 <= a.nx && y0 >= 4 && y0 + G::TY + 4 <= a.ny;
    if (core) triple_march<T, BX, BY, PY, PX, false>(a, tix, tiy, zs, ze, sq0, sq1, sq2, cold, coldr);
    else      triple_march<T, BX, BY, PY, PX, true>(a, tix, tiy, zs, ze, sq0, sq1, sq2, cold, coldr);
}

// The same on grids that do not fill the chip, with requests ahead as in adj_wave3d_pair_ahead_kernel in wave3d_pair.hip: no condition
// around any memory access, planes that are not wanted and cells outside I read as zero.  One row of cells per thread
// and one frame cell at most, so that c of the three planes before and the cells' own q stay in registers.  The sums are triple_march's, bit for bit.
// Two planes in flight; three 3 % (fp32) to 70 % (fp64, registers) slower.  What bounds it on the smaller grids is what its waves issue per
// step, about 0.8 us, for 8 planes beyond each chunk: neighbours in x come from the lanes beside, resources last for the march,
// waves without frame cells leave the frame out (fp32 197 x 68 x 260 247 -> 208 us, 200^3 491 -> 412; fp64 128^3 213 -> 195, 160^3 351 -> 326,
// 300 x 80 x 80 235 -> 208).  The stages' stars also run on the planes at a chunk's ends whose q is zero (12 of 57 stage runs of a chunk of 11
// planes): left out by a uniform condition the same time within 2 % on 15 grids, fp32 slower.  Requests after the barrier and the reads: 8 % slower.  fp32 keeps to 128 registers, so that
// two workgroups share a CU where there are more of them than CUs (64 x 400 x 400: 472 us with 140 registers, 447).
template <class T, int BX, int BY, int PX, int D> __global__ __launch_bounds__(BX *BY, sizeof(T) == 4 ? 4 : 2) void adj_wave3d_triple_ahead_kernel(TripleArgs a)
{
    using G = TripleTile<T, BX, BY, 1, PX>;
    using V = Vec<T, PX>;
    static_assert(G::HS == 1, "one frame cell per thread at most");
    constexpr int LX = G::TX + 8, PLANE = LX * (G::TY + 6);      // origin (x0-4, y0-3): a thread's cells are a whole vector
    constexpr T W0 = T(3.0 * star_w<1>(0)), W1 = T(star_w<1>(1));
    __shared__ __attribute__((aligned(16))) T sq0[2 * PLANE];
    __shared__ __attribute__((aligned(16))) T sq1[2 * PLANE];
    __shared__ __attribute__((aligned(16))) T sq2[2 * PLANE];
    int tix, tiy, zs, ze;
    block_to_tile(a.map, blockIdx.x, tix, tiy, zs, ze);
    const int tid = threadIdx.x, tx = tid % BX, ty = tid / BX;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const unsigned bytes = (unsigned)nx * (unsigned)ny * (unsigned)sizeof(T);
    const int x0 = tix * G::TX, y0 = tiy * G::TY;
    const int x = x0 + tx * PX, y = y0 + ty;
    auto in_I = [&](int xx, int yy) { return xx >= 1 && xx < nx - 1 && yy >= 1 && yy < ny - 1; };
    auto offset = [&](int xx, int yy) { return ((unsigned)yy * (unsigned)nx + (unsigned)xx) * (unsigned)sizeof(T); };
    bool in[PX], any_I = false;
#pragma unroll
    for (int e = 0; e < PX; ++e) { in[e] = in_I(x + e, y); any_I = any_I || in[e]; }
    const unsigned ioff = any_I ? offset(x, y) : kNowhere;
    const unsigned goff = x < nx && y < ny ? offset(x, y) : kNowhere;         // rows are whole vectors
    int lx, ly;
    const bool frame = G::frame_cell(tid, 0, lx, ly);
    // frame cells that run stage 1, and waves that hold some, and some that run stage 2 as well; others leave their part out
    const bool ring1 = tid < G::N1 + G::N2;
    const bool ring1_wave = __builtin_amdgcn_readfirstlane(tid) < G::N1 + G::N2, ring2_wave = __builtin_amdgcn_readfirstlane(tid) < G::N1;
    const bool hin = frame && in_I(x0 - 3 + lx, y0 - 3 + ly);
    const unsigned hoff = hin ? offset(x0 - 3 + lx, y0 - 3 + ly) : kNowhere, roff = ring1 ? hoff : kNowhere;
    const int hl = frame ? ly * LX + lx + 1 : 0;                              // (0, 0) is a cell nobody reads
    const int at = ring1 ? hl : LX + 1;                                       // the cell whose neighbours are read
    const int own = (3 + ty) * LX + 4 + tx * PX;
    const bool left_end = tx == 0, right_end = tx == BX - 1;                  // whose neighbour in x is a frame cell
    const int end = left_end ? own - 1 : right_end ? own + PX : own;

    const int zi0 = zs - 3, zi1 = ze + 2;        // q0 planes that reach the outputs [zs, ze)
    const int a1_lo = max(zs - 2, 1), a1_hi = min(ze + 1, nz - 2);            // planes of a1 and a2 that do and lie in I
    const int a2_lo = max(zs - 1, 1), a2_hi = min(ze, nz - 2);
    // step k: c and a of plane zi0 + k, b of the one before, out_b of two more before, out_a of another two
    const MarchedArray mc(a.c, zi0, max(zi0, 1), min(zi1, nz - 2), bytes), ma(a.a, zi0, max(zi0, 1), min(zi1, nz - 2), bytes);
    const MarchedArray mb(a.b, zi0 - 1, a1_lo, a1_hi, bytes);
    const MarchedArray oa(a.out_a, zi0 - 5, zs, ze - 1, bytes), ob(a.out_b, zi0 - 3, zs, ze - 1, bytes);

    // in flight: c and a of plane z on tile and frame, b of plane z - 1 on tile, D1 and D2
    V sc[D], sa[D], sb[D];
    Vec<T, 1> shc[D], sha[D], sbr[D];
    auto issue = [&](int k, int d) {
        const unsigned zoff = (unsigned)k * bytes;
        const auto rc = mc.at(k), ra = ma.at(k), rb = mb.at(k);
        sc[d] = buffer_load<T, PX, kCached>(rc, ioff + zoff);
        sa[d] = buffer_load<T, PX, kCached>(ra, ioff + zoff);
        shc[d] = buffer_load<T, 1, kCached>(rc, hoff + zoff);
        sha[d] = buffer_load<T, 1, kCached>(ra, hoff + zoff);
        sb[d] = buffer_load<T, PX, kCached>(rb, ioff + zoff);
        sbr[d] = buffer_load<T, 1, kCached>(rb, roff + zoff);
        __builtin_amdgcn_sched_barrier(0);
    };
    // what a plane's cells and a step's neighbours in y and, at a row's ends, in x add
    struct Beside { V up, down; T end; };
    auto read_beside = [&](const T *sp) { return Beside{ld_vec<T, PX>(sp + own - LX), ld_vec<T, PX>(sp + own + LX), sp[end]}; };
    auto star = [&](const V &q, const Beside &n, T (&acc)[PX][3]) {
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            const T left = e > 0 ? q.v[e > 0 ? e - 1 : 0] : beside<false>(q.v[PX - 1], n.end, left_end);
            const T right = e < PX - 1 ? q.v[e < PX - 1 ? e + 1 : 0] : beside<true>(q.v[0], n.end, right_end);
            acc[e][1] += W0 * q.v[e] + W1 * (left + right) + W1 * (n.up.v[e] + n.down.v[e]);
            acc[e][0] += W1 * q.v[e];
            acc[e][2] += W1 * q.v[e];
        }
    };
    struct BesideRing { T x, X, y, Y; };
    auto read_ring = [&](const T *at) { return BesideRing{at[-1], at[1], at[-LX], at[LX]}; };
    auto star_ring = [&](T q, const BesideRing &n, T (&acc)[3]) {
        acc[1] += W0 * q + W1 * (n.x + n.X) + W1 * (n.y + n.Y);
        acc[0] += W1 * q;
        acc[2] += W1 * q;
    };

    // as in triple_march; c1, c2, c3: c of the three planes before
    T acc1[PX][3], acc2[PX][3], acc3[PX][3], acc1r[3], acc2r[3], a1m[PX], c1[PX], c2[PX], c3[PX], c1r = T(0), c2r = T(0), c3r = T(0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        acc1r[k] = acc2r[k] = T(0);
#pragma unroll
        for (int e = 0; e < PX; ++e) acc1[e][k] = acc2[e][k] = acc3[e][k] = T(0);
    }
#pragma unroll
    for (int e = 0; e < PX; ++e) a1m[e] = c1[e] = c2[e] = c3[e] = T(0);
    V q1{}, q2{};                                // of the planes that this step reads from LDS
    T q1r = T(0);

    auto step = [&](int k, int d) {
        const unsigned zoff = (unsigned)k * bytes;
        const int buf = k & 1;
        T *s0 = sq0 + buf * PLANE;
        const T *s1 = sq1 + buf * PLANE, *s2 = sq2 + buf * PLANE;
        T *n1 = sq1 + (buf ^ 1) * PLANE, *n2 = sq2 + (buf ^ 1) * PLANE;
        T am[PX], cc[PX], cb[PX];
        V q0;
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            cc[e] = sc[d].v[e];
            am[e] = in[e] ? sa[d].v[e] : T(0);
            q0.v[e] = in[e] ? cc[e] * sa[d].v[e] : T(0);
        }
        T q0r = shc[d].v[0] * sha[d].v[0];
        st_vec<T, PX>(s0 + own, q0);
        s0[hl] = q0r;
#pragma unroll
        for (int e = 0; e < PX; ++e) { cc[e] = taken(cc[e]); cb[e] = taken(sb[d].v[e]); computed(am[e]); computed(q0.v[e]); }
        const T amr = taken(sha[d].v[0]), ccr = taken(shc[d].v[0]), cbr = taken(sbr[d].v[0]);
        computed(q0r);
        __builtin_amdgcn_sched_barrier(0);
        issue(k + D, d);
        __syncthreads();
        // all of a step's reads are requested before the first is waited for
        const Beside b2 = read_beside(s2), b1 = read_beside(s1);
        const BesideRing r1 = read_ring(s1 + at);
        const Beside b0 = read_beside(s0);
        const BesideRing r0 = read_ring(s0 + at);
        __builtin_amdgcn_sched_barrier(0);

        // ---- stage 3: q2 of plane z-4; a3 of plane z-5 is complete
        star(q2, b2, acc3);
        V o;
#pragma unroll
        for (int e = 0; e < PX; ++e) o.v[e] = acc3[e][0];
        buffer_store<T, PX, kCached>(oa.at(k), goff + zoff, o);

        // ---- stage 2: q1 of plane z-2; a2 of plane z-3 is complete
        star(q1, b1, acc2);
        const bool a2_wanted = (unsigned)(zi0 + k - 3 - a2_lo) < (unsigned)max(a2_hi + 1 - a2_lo, 0);
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            T neg = -acc2[e][0], q = c3[e] * acc2[e][0];
            computed(neg); computed(q);
            o.v[e] = (a2_wanted & in[e]) ? neg : T(0);                          // -a2 m
            q2.v[e] = (a2_wanted & in[e]) ? q : T(0);
            acc3[e][0] = acc3[e][1];
            acc3[e][1] = acc3[e][2] - T(2) * o.v[e];
            acc3[e][2] = -a1m[e];                                             // of plane z-2
            acc2[e][0] = acc2[e][1];
            acc2[e][1] = acc2[e][2];
            acc2[e][2] = -am[e];                                              // of plane z
        }
        st_vec<T, PX>(n2 + own, q2);
        if (ring2_wave) {
            star_ring(q1r, r1, acc2r);
            T q = c3r * acc2r[0];
            computed(q);
            n2[hl] = (a2_wanted & hin) ? q : T(0);
            acc2r[0] = acc2r[1]; acc2r[1] = acc2r[2]; acc2r[2] = -amr;
        }
        buffer_store<T, PX, kCached>(ob.at(k), goff + zoff, o);

        // ---- stage 1: q0 of plane z; a1 of plane z-1 is complete
        star(q0, b0, acc1);
        const bool a1_wanted = (unsigned)(zi0 + k - 1 - a1_lo) < (unsigned)max(a1_hi + 1 - a1_lo, 0);
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            T v = acc1[e][0] + cb[e], q = c1[e] * v;
            computed(v); computed(q);
            a1m[e] = (a1_wanted & in[e]) ? v : T(0);
            q1.v[e] = (a1_wanted & in[e]) ? q : T(0);
            acc2[e][1] += T(2) * a1m[e];
            acc1[e][0] = acc1[e][1] + T(2) * am[e];
            acc1[e][1] = acc1[e][2];
            acc1[e][2] = T(0);
            c3[e] = c2[e]; c2[e] = c1[e]; c1[e] = cc[e];
        }
        st_vec<T, PX>(n1 + own, q1);
        if (ring1_wave) {
            star_ring(q0r, r0, acc1r);
            T v = acc1r[0] + cbr, q = c1r * v;
            computed(v); computed(q);
            const T a1r = (a1_wanted & hin) ? v : T(0);
            q1r = (a1_wanted & hin) ? q : T(0);
            n1[hl] = q1r;
            acc2r[1] += T(2) * a1r;
            acc1r[0] = acc1r[1] + T(2) * amr;
            acc1r[1] = acc1r[2];
            acc1r[2] = T(0);
        }
        c3r = c2r; c2r = c1r; c1r = ccr;
        __builtin_amdgcn_sched_barrier(0);
    };

    // each request is followed by two stores, as in the loop (here to nowhere), or the loop's waits would have to suit both counts
#pragma unroll
    for (int d = 0; d < D; ++d) {
        issue(d, d);
        buffer_store<T, PX, kCached>(oa.at(-1), kNowhere, V{});
        buffer_store<T, PX, kCached>(ob.at(-1), kNowhere, V{});
        __builtin_amdgcn_sched_barrier(0);
    }
    // the first step reads planes of q1 and q2 that none has written
    st_vec<T, PX>(sq1 + own, q1);
    st_vec<T, PX>(sq2 + own, q2);
    sq1[hl] = T(0);
    sq2[hl] = T(0);
    const int steps = ze + 5 - zi0;
    int k = 0;
    for (; k + D <= steps; k += D) {
#pragma unroll
        for (int d = 0; d < D; ++d) step(k + d, d);
    }
#pragma unroll
    for (int d = 0; d < D - 1; ++d) {
        if (k + d >= steps) return;
        step(k + d, d);
    }
}

// Where the march with its requests ahead is taken: by the planes it marches against those of the wide tiles above, whose cells per workgroup are
// two (fp32: four) times as many, and by the bytes of the five arrays.  25 steps on 130 drawn grids, time in the wide tiles over time of this march, by
// the quotient of the planes: fp64 up to 300 MB, quotient to 2 1.00 to 1.29; 300 .. 1200 MB below 1.7 1.02 to 1.24, 1.7 .. 2 0.93 to 1.05;
// fp32 up to 260 MB, to 3.57 1.08 to 1.42; 260 .. 600 MB below 3.13 1.04 to 1.68, above 0.88 to 1.12.  Grids of few planes, whose chunks are short,
// gain less (6 x 676 x 588, quotient 2, 0.80) and keep the quotients 1.85 and 2.94.  The grid alone decides.
static bool triple_runs_ahead(int is_f64, int nx, int ny, int nz)
{
    const double plane = (double)nx * ny * (is_f64 ? 8 : 4), bytes = 5 * plane * nz;
    const bool cached = bytes <= (is_f64 ? 300e6 : 260e6);
    if (bytes > (is_f64 ? 1200e6 : 600e6) || (nz + 16) * plane >= 0x1p31) return false;       // the latter: see MarchedArray
    if (!cached && nz < 16) return false;
    TileMap wide, ahead;
    plan_march(wide, nx, ny, nz, is_f64 ? 64 : 128, 32, 4, LaunchOptions{});
    plan_march(ahead, nx, ny, nz, 64, 16, 4, LaunchOptions{});
    const int percent = nz < 16 ? (is_f64 ? 54 : 34) : cached ? (is_f64 ? 49 : 28) : is_f64 ? 59 : 32;
    return percent * march_planes(ahead, 8) < 100 * march_planes(wide, 8);
}

template <class T, int PX>
static hipError_t launch_triple(TripleArgs a, const LaunchOptions &opt, hipStream_t stream)
{
    constexpr int BX = 32, BY = 16, PY = 2;
    using G = TripleTile<T, BX, BY, PY, PX>;
    if (opt.ahead == 0 && triple_runs_ahead(sizeof(T) == 8, a.nx, a.ny, a.nz)) {
        plan_march(a.map, a.nx, a.ny, a.nz, 64, 16, 4, opt);
        hipLaunchKernelGGL((adj_wave3d_triple_ahead_kernel<T, BX, BY, 2, 2>), dim3(a.map.total_blocks), dim3(BX * BY), ahead_pad(opt), stream, a);
        return hipGetLastError();
    }
    // each chunk marches 8 planes beyond its own: plan as a march of radius 4
    plan_march(a.map, a.nx, a.ny, a.nz, G::TX, G::TY, 4, opt);
    hipLaunchKernelGGL((adj_wave3d_triple_kernel<T, BX, BY, PY, PX>), dim3(a.map.total_blocks), dim3(G::NT), 0, stream, a);
    return hipGetLastError();
}

// A chunk marches 5 planes beyond its own for two steps and 8 for three, and a plane of the three-step march
// takes about 1.1 (fp64) or 1.2 (fp32) times as long.  Short marches on small grids therefore take two
// steps per pass.  Priced and measured in the tiles without requests ahead: 25 steps, two (in 64 x 32 tiles, fp32
// 128 x 32) / three per pass, fp64 33 x 40 x 72 71 / 83 us, 128^3 309 / 265, 512^3 12.9 / 9.4 ms; fp32 128^3 192 / 221 us,
// 96 x 130 x 164 262 / 279, 160 x 180 x 200 451 / 406, 512^3 6.6 / 5.0 ms.  Two and three steps group the sums differently, so grid and type alone decide: options that
// cut the march another way must not change a bit.
int adjoint_wave3d_steps_per_pass(int is_f64, int nx, int ny, int nz)
{
    TileMap three;
    plan_march(three, nx, ny, nz, is_f64 ? 64 : 128, 32, 4, LaunchOptions{});
    return 20 * march_planes(three, 8) * (is_f64 ? 11 : 12) < 3 * adjoint_wave3d_pair_cost(is_f64, nx, ny, nz) ? 3 : 2;
}

hipError_t launch_adjoint_wave3d_triple(int is_f64, int nx, int ny, int nz, const void *c, const void *a, const void *b,
                                        void *out_a, void *out_b, const LaunchOptions &opt, hipStream_t stream)
{
    if (!adjoint_wave3d_pair_supported(is_f64, nx, c, a, b, out_a, out_b)) return hipErrorNotSupported;
    TripleArgs p{};
    p.c = c; p.a = a; p.b = b; p.out_a = out_a; p.out_b = out_b;
    p.nx = nx; p.ny = ny; p.nz = nz;
    return is_f64 ? launch_triple<double, 2>(p, opt, stream) : launch_triple<float, 4>(p, opt, stream);
}

}  // namespace sadj
