// Two reverse steps of a time loop of radius-1 wave steps in one pass over the data.
//
// What is computed.  A solver repeats u^{k+1} = 2 u^k - u^{k-1} + c * Lap(u^k) on I (paper
// Section 4.1; Section 4 notes that such solvers take many steps).  With a = lam^{k+1},
// b = lam^k and m the indicator of I, one reverse step in gather form (Sections 3.3.2-3.3.4) is
//     a' = b + 2 a m + S(q),   q = c a m,        b' = -a m
// where S is the 7-point star with the second-difference weights (symmetric, so the gather
// uses the same table).  Two steps in a row give
//     a'' = -a m + 2 a' m + S(q'),   q' = c a' m,   b'' = -a' m
// and a' itself is never needed in memory.  This kernel reads a, b, c once and writes a'' and
// b'' once: 40 bytes per cell (fp64) for two steps where two single-step launches move 80.
//
// How.  The z-march of the single-step adjoint (wave3d_adjoint.hip) run as a two-stage pipeline.
// Stage 1 stages plane z of q in LDS on the tile plus a frame of width 2 and keeps three running
// sums per cell for a' on the tile AND on the ring of cells around it (a thread owns PX x PY tile
// cells; the first 2 TX + 2 TY threads own one ring cell each).  A plane of a' is complete one
// step after its q plane arrived; b is added, q' = c a' m is formed on tile and ring and staged
// in a second LDS plane, from which stage 2 forms a'' on the tile with three more running sums.
// Both LDS planes are double-buffered and one barrier per step serves both stages: stage 2 works
// one step behind stage 1.  Values outside I are replaced by zero with selects, never by a
// multiplication, so NaN outside I cannot leak (Section 3.3.4: guarded remainder; tiles whose
// frame lies in I in x and y run an unguarded instantiation).
//
// The outputs must be arrays other than a and b: neighbouring workgroups read the frame of a and
// the ring of b while this one writes.
#include "launch.hpp"
#include "ahead.hpp"
#include "ahead3d.hpp"
#include "tile3d.hpp"

#include <type_traits>

namespace sadj {

struct PairArgs {
    const void *c, *a, *b;
    void *out_a, *out_b;
    int nx, ny, nz;
    TileMap map;
};

template <class T, int BX, int BY, int PY, int PX> struct PairTile {
    static constexpr int TX = BX * PX, TY = BY * PY, NT = BX * BY;
    static constexpr int LX1 = TX + 4, LY1 = TY + 4, PLANE1 = LX1 * LY1;   // q:  origin (x0-2, y0-2)
    static constexpr int LX2 = TX + 2, LY2 = TY + 2, PLANE2 = LX2 * LY2;   // q': origin (x0-1, y0-1)
    static constexpr int NRING = 2 * TX + 2 * TY;                           // ring cells without corners: a' is formed there
    static constexpr int NFRAME = NRING + 4 + 2 * TX + 2 * TY;              // + ring corners + the arms two cells out
    static constexpr int HS = (NFRAME + NT - 1) / NT;
    static_assert(NRING <= NT, "one ring cell per thread at most");

    // Frame slot s of thread tid -> coordinates in the q plane; false if the slot is unused.
    // Slots 0 .. NRING-1 are the ring (rows above and below, then the columns left and right),
    // then its four corners, then the rows and columns two cells out.
    __device__ static __forceinline__ bool frame_cell(int tid, int s, int &lx, int &ly)
    {
        int h = tid + s * NT;
        const bool used = h < NFRAME;
        if (h < 2 * TX) {
            lx = 2 + h % TX;
            ly = h < TX ? 1 : TY + 2;
        } else if (h < NRING) {
            h -= 2 * TX;
            lx = (h & 1) ? TX + 2 : 1;
            ly = 2 + h / 2;
        } else if (h < NRING + 4) {
            h -= NRING;
            lx = (h & 1) ? TX + 2 : 1;
            ly = (h & 2) ? TY + 2 : 1;
        } else if (h < NRING + 4 + 2 * TX) {
            h -= NRING + 4;
            lx = 2 + h % TX;
            ly = h < TX ? 0 : TY + 3;
        } else {
            h -= NRING + 4 + 2 * TX;
            lx = (h & 1) ? TX + 3 : 0;
            ly = 2 + h / 2;
        }
        return used;
    }
};

template <class T, int BX, int BY, int PY, int PX, bool GUARD>
__device__ __forceinline__ void pair_march(const PairArgs &a, int tix, int tiy, int zs, int ze, T *__restrict__ sq1,
                                           T *__restrict__ sq2)
{
    using G = PairTile<T, BX, BY, PY, PX>;
    using V = Vec<T, PX>;
    constexpr int TX = G::TX, TY = G::TY, LX1 = G::LX1, LX2 = G::LX2, HS = G::HS;
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
    ad.init(tx, ty, x0, y0, nx, ny, 1, 2, LX1, 0 /* plane corner, never read */, (uint32_t)sizeof(T),
            [&](int s, int &lx, int &ly) { return G::frame_cell(tid, s, lx, ly); });
    const uint32_t dummy = ad.dummy;
    uint32_t ooff[PY], coff[PY];
    bool ouse[PY][PX], ostore[PY];
#pragma unroll
    for (int p = 0; p < PY; ++p) {
        ostore[p] = ad.own_grid[p];
        ooff[p] = ad.own_off[p];
        bool any = false;
#pragma unroll
        for (int e = 0; e < PX; ++e) { ouse[p][e] = ad.own_I[p][e]; any = any || ouse[p][e]; }
        coff[p] = (!GUARD || any) ? ooff[p] : dummy;
    }
    uint32_t hoff[HS];
    int hlds[HS];
    bool huse[HS];
#pragma unroll
    for (int s = 0; s < HS; ++s) {
        huse[s] = ad.halo_I[s];
        hoff[s] = huse[s] ? ad.halo_off[s] : dummy;
        hlds[s] = ad.halo_lds[s];
    }
    // the ring cell of this thread (slot 0 of the first NRING threads); whole waves have one or none
    const bool ring = tid < G::NRING;
    int rlx, rly;
    G::frame_cell(tid, 0, rlx, rly);
    const int ring1 = rly * LX1 + rlx;                   // in the q plane
    const int ring2 = (rly - 1) * LX2 + (rlx - 1);       // in the q' plane
    const bool ruse = ring && huse[0];

    // running sums: index 0 = the plane that completes in this step
    T acc1[PY][PX][3], acc1r[3], acc2[PY][PX][3];
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        acc1r[k] = T(0);
#pragma unroll
        for (int p = 0; p < PY; ++p)
#pragma unroll
            for (int e = 0; e < PX; ++e) acc1[p][e][k] = acc2[p][e][k] = T(0);
    }
    // carried from the previous step: c and a m of its plane, and what stage 2 consumes one step late
    T c_prev[PY][PX], c_prev_r = T(0), am_prev[PY][PX], q2[PY][PX], q2r = T(0), a1m[PY][PX];
#pragma unroll
    for (int p = 0; p < PY; ++p)
#pragma unroll
        for (int e = 0; e < PX; ++e) c_prev[p][e] = am_prev[p][e] = q2[p][e] = a1m[p][e] = T(0);
    bool q2_valid = false;

    // values in flight for the next step
    V sa[PY], sc[PY], sb[PY];
    T sha[HS], shc[HS], sbr = T(0);
#pragma unroll
    for (int p = 0; p < PY; ++p) { sa[p] = V{}; sc[p] = V{}; sb[p] = V{}; }
#pragma unroll
    for (int s = 0; s < HS; ++s) sha[s] = shc[s] = T(0);

    auto plane_in_I = [&](int z) { return z >= 1 && z < nz - 1; };
    const int zi0 = zs - 2, zi1 = ze + 1;        // q planes that reach the outputs [zs, ze)
    // a' of plane z is wanted for z in [zs-1, ze] and only on I
    auto a1_wanted = [&](int z) { return z >= zs - 1 && z <= ze && plane_in_I(z); };

    // request what step z consumes: a and c of plane z (tile and frame), b of plane z-1 (tile and ring)
    // `steady` (a std::bool_constant): the caller knows that every condition on the plane index
    // holds, so the step has no branches on them (measured 2 % faster than the generic step alone)
    auto issue = [&](int z, auto steady) {
        constexpr bool ST = decltype(steady)::value;
        if (ST || (z <= zi1 && plane_in_I(z))) {
            const T *cp = cg + (size_t)z * plane;
            const T *ap = ag + (size_t)z * plane;
#pragma unroll
            for (int p = 0; p < PY; ++p) {
                sc[p] = ld_vec_off<T, PX, false>(cp, coff[p]);
                sa[p] = ld_vec_off<T, PX, false>(ap, coff[p]);
            }
#pragma unroll
            for (int s = 0; s < HS; ++s) { shc[s] = ld_off(cp, hoff[s]); sha[s] = ld_off(ap, hoff[s]); }
        }
        if (ST || a1_wanted(z - 1)) {
            const T *bp = bg + (size_t)(z - 1) * plane;
#pragma unroll
            for (int p = 0; p < PY; ++p) sb[p] = ld_vec_off<T, PX, false>(bp, coff[p]);
            if (ring) sbr = ld_off(bp, hoff[0]);
        }
    };

    issue(zi0, std::false_type{});
    int buf = 0;
    auto step = [&](int zi, auto steady) {
        constexpr bool ST = decltype(steady)::value;
        const bool zin = ST || (zi <= zi1 && plane_in_I(zi));
        T *s1 = sq1 + buf * G::PLANE1;
        T *s2 = sq2 + buf * G::PLANE2;
        T qo[PY][PX], am[PY][PX], cc[PY][PX], qr = T(0), amr = T(0), ccr = T(0);
        if (zin) {
#pragma unroll
            for (int p = 0; p < PY; ++p)
#pragma unroll
                for (int e = 0; e < PX; ++e) {
                    const T cv = sc[p].v[e], av = sa[p].v[e];
                    cc[p][e] = cv;
                    am[p][e] = GUARD ? (ouse[p][e] ? av : T(0)) : av;
                    qo[p][e] = GUARD ? (ouse[p][e] ? cv * av : T(0)) : cv * av;
                    s1[(2 + ty * PY + p) * LX1 + 2 + tx * PX + e] = qo[p][e];
                }
#pragma unroll
            for (int s = 0; s < HS; ++s) {
                const T qq = GUARD ? (huse[s] ? shc[s] * sha[s] : T(0)) : shc[s] * sha[s];
                s1[hlds[s]] = qq;
                if (s == 0) { qr = qq; ccr = shc[0]; amr = GUARD ? (huse[0] ? sha[0] : T(0)) : sha[0]; }
            }
        } else {
#pragma unroll
            for (int p = 0; p < PY; ++p)
#pragma unroll
                for (int e = 0; e < PX; ++e) cc[p][e] = am[p][e] = qo[p][e] = T(0);
        }
        const bool stage2 = ST || q2_valid;       // q' of plane zi-2 was formed in the previous step
        if (stage2) {
#pragma unroll
            for (int p = 0; p < PY; ++p)
#pragma unroll
                for (int e = 0; e < PX; ++e) s2[(1 + ty * PY + p) * LX2 + 1 + tx * PX + e] = q2[p][e];
            if (ring) s2[ring2] = q2r;
        }
        V cb[PY];
#pragma unroll
        for (int p = 0; p < PY; ++p) cb[p] = sb[p];
        const T cbr = sbr;
        issue(zi + 1, steady);
        __syncthreads();

        // ---- stage 2: q' of plane zi-2 -> a'' sums of planes zi-3, zi-2, zi-1
        if (stage2) {
#pragma unroll
            for (int p = 0; p < PY; ++p)
#pragma unroll
                for (int e = 0; e < PX; ++e) {
                    const T *at = s2 + (1 + ty * PY + p) * LX2 + 1 + tx * PX + e;
                    const T left = e > 0 ? q2[p][e - 1] : at[-1];
                    const T right = e < PX - 1 ? q2[p][e + 1] : at[1];
                    const T up = p > 0 ? q2[p - 1][e] : at[-LX2];
                    const T down = p < PY - 1 ? q2[p + 1][e] : at[LX2];
                    const T s = W0 * q2[p][e] + W1 * (left + right) + W1 * (up + down);
                    acc2[p][e][1] += s + T(2) * a1m[p][e];
                    acc2[p][e][0] += W1 * q2[p][e];
                    acc2[p][e][2] += W1 * q2[p][e];
                }
        }
#pragma unroll
        for (int p = 0; p < PY; ++p)
#pragma unroll
            for (int e = 0; e < PX; ++e) acc2[p][e][2] -= am_prev[p][e];      // -a m of plane zi-1
        const int zo2 = zi - 3;
        if (ST || (zo2 >= zs && zo2 < ze)) {
            T *op = oag + (size_t)zo2 * plane;
#pragma unroll
            for (int p = 0; p < PY; ++p) {
                V o;
#pragma unroll
                for (int e = 0; e < PX; ++e) o.v[e] = acc2[p][e][0];
                if (!GUARD || ostore[p]) st_vec_off<T, PX, true>(op, ooff[p], o);
            }
        }

        // ---- stage 1: q of plane zi -> a' sums of planes zi-1, zi, zi+1
        if (zin) {
#pragma unroll
            for (int p = 0; p < PY; ++p)
#pragma unroll
                for (int e = 0; e < PX; ++e) {
                    const T *at = s1 + (2 + ty * PY + p) * LX1 + 2 + tx * PX + e;
                    const T left = e > 0 ? qo[p][e - 1] : at[-1];
                    const T right = e < PX - 1 ? qo[p][e + 1] : at[1];
                    const T up = p > 0 ? qo[p - 1][e] : at[-LX1];
                    const T down = p < PY - 1 ? qo[p + 1][e] : at[LX1];
                    const T s = W0 * qo[p][e] + W1 * (left + right) + W1 * (up + down);
                    acc1[p][e][1] += s + T(2) * am[p][e];
                    acc1[p][e][0] += W1 * qo[p][e];
                    acc1[p][e][2] += W1 * qo[p][e];
                }
            if (ring) {
                const T *at = s1 + ring1;
                const T s = W0 * qr + W1 * (at[-1] + at[1]) + W1 * (at[-LX1] + at[LX1]);
                acc1r[1] += s + T(2) * amr;
                acc1r[0] += W1 * qr;
                acc1r[2] += W1 * qr;
            }
        }
        // a' of plane zi-1 is complete: form q' and -a' m from it
        const int zo1 = zi - 1;
        q2_valid = ST || a1_wanted(zo1);
        if (q2_valid) {
#pragma unroll
            for (int p = 0; p < PY; ++p)
#pragma unroll
                for (int e = 0; e < PX; ++e) {
                    const T a1 = acc1[p][e][0] + cb[p].v[e];
                    a1m[p][e] = GUARD ? (ouse[p][e] ? a1 : T(0)) : a1;
                    q2[p][e] = GUARD ? (ouse[p][e] ? c_prev[p][e] * a1 : T(0)) : c_prev[p][e] * a1;
                }
            const T a1r = acc1r[0] + cbr;
            q2r = GUARD ? (ruse ? c_prev_r * a1r : T(0)) : c_prev_r * a1r;
        } else {
#pragma unroll
            for (int p = 0; p < PY; ++p)
#pragma unroll
                for (int e = 0; e < PX; ++e) a1m[p][e] = q2[p][e] = T(0);
            q2r = T(0);
        }
        if (ST || (zo1 >= zs && zo1 < ze)) {         // b'' = -a' m; zero on planes outside I
            T *op = obg + (size_t)zo1 * plane;
#pragma unroll
            for (int p = 0; p < PY; ++p) {
                V o;
#pragma unroll
                for (int e = 0; e < PX; ++e) o.v[e] = -a1m[p][e];
                if (!GUARD || ostore[p]) st_vec_off<T, PX, true>(op, ooff[p], o);
            }
        }
        // next step
        acc1r[0] = acc1r[1]; acc1r[1] = acc1r[2]; acc1r[2] = T(0);
        c_prev_r = ccr;
#pragma unroll
        for (int p = 0; p < PY; ++p)
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                acc1[p][e][0] = acc1[p][e][1]; acc1[p][e][1] = acc1[p][e][2]; acc1[p][e][2] = T(0);
                acc2[p][e][0] = acc2[p][e][1]; acc2[p][e][1] = acc2[p][e][2]; acc2[p][e][2] = T(0);
                c_prev[p][e] = cc[p][e];
                am_prev[p][e] = am[p][e];
            }
        buf ^= 1;
    };
    // steady steps: planes zi-2 .. zi+1 lie in I, and the output planes zi-3 and zi-1 in this chunk
    const int lo = max(zs + 3, 3), hi = min(ze, nz - 3);
    int zi = zi0;
    for (; zi <= zi1 + 1 && zi < lo; ++zi) step(zi, std::false_type{});
    __builtin_amdgcn_s_waitcnt(0x0F70);          // enter the steady loop with nothing outstanding (vmcnt(0))
    for (; zi <= hi; ++zi) step(zi, std::true_type{});
    for (; zi <= zi1 + 1; ++zi) step(zi, std::false_type{});
}

template <class T, int BX, int BY, int PY, int PX>
__global__ __launch_bounds__(BX *BY) void adj_wave3d_pair_kernel(PairArgs a)
{
    using G = PairTile<T, BX, BY, PY, PX>;
    __shared__ T sq1[2 * G::PLANE1];
    __shared__ T sq2[2 * G::PLANE2];
    int tix, tiy, zs, ze;
    block_to_tile(a.map, blockIdx.x, tix, tiy, zs, ze);
    // core tile: the tile and its frame lie in I in x and y
    const int x0 = tix * G::TX, y0 = tiy * G::TY;
    const bool core = x0 >= 3 && x0 + G::TX + 3 <= a.nx && y0 >= 3 && y0 + G::TY + 3 <= a.ny;
    if (core) pair_march<T, BX, BY, PY, PX, false>(a, tix, tiy, zs, ze, sq1, sq2);
    else      pair_march<T, BX, BY, PY, PX, true>(a, tix, tiy, zs, ze, sq1, sq2);
}

// The same on grids that do not fill the chip, where a workgroup marches few planes and the time from a plane's request to the
// next plane's is what counts.  As in ahead3d.hpp all accesses go through buffer resources, without a condition around any of
// them: a plane that is not wanted has a resource of zero bytes and reads as zero, cells outside I have an offset beyond any plane.
// The waits (vmcnt 10 to 13, of 6 loads and 2 stores a plane) leave a plane's requests in flight for two steps; one instantiation
// serves core and remainder.  The sums are pair_march's, bit for bit.
// What bounds it is what its waves issue: 120 instructions a step, 0.5 us with two waves per SIMD (half of it vector ALU; half the cells per thread in
// twice the waves: the same; reading LDS while the next plane arrives: 0 to 7 % slower), then 3 us of start and first latency a launch.  Hence
// one resource per array and march, neighbours in x from the lanes beside, all LDS reads of a step together, and waves without ring cells
// that leave the ring out.  25 steps, with a resource per plane and access and all neighbours from LDS / now: fp32 96 x 130 x 164 186 / 163 us, 128^3 155 /
// 140, 300 x 80 x 80 184 / 160, 64^3 90 / 84; fp64 40 x 300 x 96 191 / 169.  Three planes in flight 8 % slower.
template <class T, int BX, int BY, int PX, int D>
__global__ __launch_bounds__(BX *BY) void adj_wave3d_pair_ahead_kernel(PairArgs a)
{
    using G = PairTile<T, BX, BY, 1, PX>;
    using V = Vec<T, PX>;
    static_assert(G::HS == 1, "one frame cell per thread at most");
    constexpr int LX = G::LX1;                   // both planes have the wider one's geometry, where a thread's cells are whole vectors
    constexpr T W0 = T(3.0 * star_w<1>(0)), W1 = T(star_w<1>(1));
    __shared__ __attribute__((aligned(16))) T sq1[2 * G::PLANE1];
    __shared__ __attribute__((aligned(16))) T sq2[2 * G::PLANE1];
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
    // this thread's frame cell, which is a ring cell for the first NRING threads
    int lx, ly;
    const bool frame = G::frame_cell(tid, 0, lx, ly), ring = tid < G::NRING;
    const bool hin = frame && in_I(x0 - 2 + lx, y0 - 2 + ly), rin = ring && hin;
    const unsigned hoff = hin ? offset(x0 - 2 + lx, y0 - 2 + ly) : kNowhere, roff = ring ? hoff : kNowhere;
    const bool ring_wave = __builtin_amdgcn_readfirstlane(tid) < G::NRING;    // waves without a ring cell skip what is theirs
    const int hl = frame ? ly * LX + lx : 0;                                  // (0, 0) is a corner nobody reads
    const int ring1 = ring ? hl : LX + 1;
    const int own = (2 + ty) * LX + 2 + tx * PX;
    const bool left_end = tx == 0, right_end = tx == BX - 1;                  // whose neighbour in x is a frame cell
    const int end = left_end ? own - 1 : right_end ? own + PX : own;

    const int zi0 = zs - 2, zi1 = ze + 1;        // q planes that reach the outputs [zs, ze)
    const int a1_lo = max(zs - 1, 1), a1_hi = min(ze, nz - 2);      // planes of a' that do and lie in I
    // step k: c and a of plane zi0 + k, b and out_b of the one before, out_a of two more before
    const MarchedArray mc(a.c, zi0, max(zi0, 1), min(zi1, nz - 2), bytes), ma(a.a, zi0, max(zi0, 1), min(zi1, nz - 2), bytes);
    const MarchedArray mb(a.b, zi0 - 1, a1_lo, a1_hi, bytes);
    const MarchedArray oa(a.out_a, zi0 - 3, zs, ze - 1, bytes), ob(a.out_b, zi0 - 1, zs, ze - 1, bytes);

    // in flight: c and a of plane z on tile and frame, b of plane z - 1 on tile and ring
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

    // as in pair_march
    T acc1[PX][3], acc1r[3], acc2[PX][3], c_prev[PX], c_prev_r = T(0), am_prev[PX], q2r = T(0);
    V q2, neg_a1m;
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        acc1r[k] = T(0);
#pragma unroll
        for (int e = 0; e < PX; ++e) acc1[e][k] = acc2[e][k] = T(0);
    }
#pragma unroll
    for (int e = 0; e < PX; ++e) c_prev[e] = am_prev[e] = q2.v[e] = neg_a1m.v[e] = T(0);

    auto step = [&](int k, int d) {
        const unsigned zoff = (unsigned)k * bytes;
        T *s1 = sq1 + (k & 1) * G::PLANE1;
        T *s2 = sq2 + (k & 1) * G::PLANE1;
        T am[PX], cc[PX], cb[PX];
        V qo;
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            cc[e] = sc[d].v[e];
            am[e] = in[e] ? sa[d].v[e] : T(0);
            qo.v[e] = in[e] ? cc[e] * sa[d].v[e] : T(0);
        }
        T qr = shc[d].v[0] * sha[d].v[0];
        st_vec<T, PX>(s1 + own, qo);
        s1[hl] = qr;
        st_vec<T, PX>(s2 + own, q2);
        if (ring_wave) s2[hl] = q2r;
#pragma unroll
        for (int e = 0; e < PX; ++e) { cc[e] = taken(cc[e]); cb[e] = taken(sb[d].v[e]); computed(am[e]); computed(qo.v[e]); }
        const T amr = taken(sha[d].v[0]), ccr = taken(shc[d].v[0]), cbr = taken(sbr[d].v[0]);
        computed(qr);
        __builtin_amdgcn_sched_barrier(0);
        issue(k + D, d);
        __syncthreads();

        // the star of plane z without its z neighbours' terms
        auto in_plane = [&](const V &q, const V &up, const V &down, T frame_cell, int e) {
            const T left = e > 0 ? q.v[e > 0 ? e - 1 : 0] : beside<false>(q.v[PX - 1], frame_cell, left_end);
            const T right = e < PX - 1 ? q.v[e < PX - 1 ? e + 1 : 0] : beside<true>(q.v[0], frame_cell, right_end);
            return W0 * q.v[e] + W1 * (left + right) + W1 * (up.v[e] + down.v[e]);
        };
        // all of a step's reads are requested before the first is waited for
        const V up2 = ld_vec<T, PX>(s2 + own - LX), down2 = ld_vec<T, PX>(s2 + own + LX);
        const T end2 = s2[end];
        const V up1 = ld_vec<T, PX>(s1 + own - LX), down1 = ld_vec<T, PX>(s1 + own + LX);
        const T end1 = s1[end], ring_x = s1[ring1 - 1], ring_X = s1[ring1 + 1], ring_y = s1[ring1 - LX], ring_Y = s1[ring1 + LX];
        __builtin_amdgcn_sched_barrier(0);
        // ---- stage 2: q' of plane z-2 -> a'' sums of planes z-3, z-2, z-1
        V o;
        {
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                acc2[e][1] += in_plane(q2, up2, down2, end2, e) - T(2) * neg_a1m.v[e];
                acc2[e][0] += W1 * q2.v[e];
                acc2[e][2] = W1 * q2.v[e] - am_prev[e];                       // -a m of plane z-1
                o.v[e] = acc2[e][0];
            }
        }
        buffer_store<T, PX, kCached>(oa.at(k), goff + zoff, o);

        // ---- stage 1: q of plane z -> a' sums of planes z-1, z, z+1
        {
#pragma unroll
            for (int e = 0; e < PX; ++e) {
                acc1[e][1] += in_plane(qo, up1, down1, end1, e) + T(2) * am[e];
                acc1[e][0] += W1 * qo.v[e];
                acc1[e][2] = W1 * qo.v[e];
            }
        }
        // a' of plane z-1 is complete: form q' and -a' m from it
        const bool wanted = (unsigned)(zi0 + k - 1 - a1_lo) < (unsigned)max(a1_hi + 1 - a1_lo, 0);
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            T neg_a1 = -acc1[e][0] - cb[e], q = c_prev[e] * -neg_a1;
            computed(neg_a1); computed(q);
            neg_a1m.v[e] = (wanted & in[e]) ? neg_a1 : T(0);
            q2.v[e] = (wanted & in[e]) ? q : T(0);
        }
        if (ring_wave) {
            const T s = W0 * qr + W1 * (ring_x + ring_X) + W1 * (ring_y + ring_Y);
            acc1r[1] += s + T(2) * amr;
            acc1r[0] += W1 * qr;
            acc1r[2] = W1 * qr;
            T q = c_prev_r * (acc1r[0] + cbr);
            computed(q);
            q2r = (wanted & rin) ? q : T(0);
            acc1r[0] = acc1r[1]; acc1r[1] = acc1r[2];
        }
        buffer_store<T, PX, kCached>(ob.at(k), goff + zoff, neg_a1m);
        c_prev_r = ccr;
#pragma unroll
        for (int e = 0; e < PX; ++e) {
            acc1[e][0] = acc1[e][1]; acc1[e][1] = acc1[e][2];
            acc2[e][0] = acc2[e][1]; acc2[e][1] = acc2[e][2];
            c_prev[e] = cc[e];
            am_prev[e] = am[e];
        }
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
    const int steps = zi1 + 2 - zi0;
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

// Beyond the grids of the march above, tiles of 64 x 32 (fp32: 128 x 32) cells, one workgroup per CU; on the smallest fp64 grids, whose
// chunks the 5 planes that a workgroup marches beyond its own dominate, 64 x 16 cells, whose march step takes 0.72 of the
// time.  25 steps, default / small tiles: fp64 24^3 125 / 101 us, 64^3 134 / 110, 128^3 309 / 307.  (fp32 grids like these, and fp64 ones of 16 planes
// or more, take the march above.)
// The cost decides where passes take three steps, which round differently.  It stays what it was when the default and the small
// tiles (fp32: 0.79 of the step, two workgroups per CU) were all there was, so that a grid's results do as well.
struct PairPlan {
    TileMap map;
    bool small;            // the 64 x 16 tiles cost less
    long cost;             // planes marched in default tiles, times 100
};

static PairPlan plan_pair(int is_f64, int nx, int ny, int nz, const LaunchOptions &opt)
{
    // each chunk marches 5 planes beyond its own: planned as a march of radius 2
    PairPlan p{};
    plan_march(p.map, nx, ny, nz, is_f64 ? 64 : 128, 32, 2, opt);
    p.cost = 100 * march_planes(p.map, 5);
    if (opt.zchunk == 0 && opt.lds_pad == 0 && p.map.zchunk < 8) {
        const int per_cu = is_f64 ? 1 : 2;
        TileMap m;
        plan_march(m, nx, ny, nz, 64, 16, 2, opt, per_cu);
        const long cost = (is_f64 ? 72 : 79) * march_planes(m, 5, per_cu);
        if (cost < p.cost) p = {is_f64 ? m : p.map, true, cost};
    }
    return p;
}

long adjoint_wave3d_pair_cost(int is_f64, int nx, int ny, int nz)
{
    return plan_pair(is_f64, nx, ny, nz, LaunchOptions{}).cost;
}

// Where the march with its requests ahead is taken, by the bytes of the five arrays, which it relies on finding in the last-level cache
// (drawn grids, time in the shapes above over its time): fp32 up to 130 MB 1.15 to 1.35; against the default tiles, which the
// last passes of a three-step sweep would take, 130 .. 230 MB 1.05 and more, 230 .. 300 MB 0.95 (0.93); fp64 30 .. 60 MB 1.24, default tiles up
// to 230 MB 1.22 (1.12), 230 .. 300 MB 1.09 (0.98); fp64 in small tiles below 30 MB 1.00 to 1.17 from 16 planes on, 0.89 to 1.1 with fewer: a
// chunk of one or two planes leaves no request to run ahead of.  fp32 grids of more bytes that would cost less in 64 x 16 tiles
// (few rows of 10^5 cells, whose default tiles are half empty) take it too: 6 x 16 x 200000, 9 steps, without / with requests ahead 466 / 452 us.
static bool pair_runs_ahead(int is_f64, int nx, int ny, int nz, const PairPlan &plan)
{
    const double plane = (double)nx * ny * (is_f64 ? 8 : 4), bytes = 5 * plane * nz;
    if ((nz + 16) * plane >= 0x1p31) return false;                  // see MarchedArray
    if (!is_f64) return bytes <= 230e6 || plan.small;
    return bytes <= 230e6 && (!plan.small || bytes >= 30e6 || nz >= 16);
}

template <class T, int PX>
static hipError_t launch_pair(PairArgs a, const LaunchOptions &opt, hipStream_t stream)
{
    constexpr int BX = 32, BY = 16, PY = 2;
    using G = PairTile<T, BX, BY, PY, PX>;
    const size_t al = PX * sizeof(T);
    const void *arrays[5] = {a.c, a.a, a.b, a.out_a, a.out_b};
    for (const void *p : arrays)
        if (reinterpret_cast<uintptr_t>(p) % al != 0) return hipErrorNotSupported;
    if (a.nx % PX != 0) return hipErrorNotSupported;
    const PairPlan plan = plan_pair(sizeof(T) == 8, a.nx, a.ny, a.nz, opt);
    a.map = plan.map;
    if (opt.ahead == 0 && pair_runs_ahead(sizeof(T) == 8, a.nx, a.ny, a.nz, plan_pair(sizeof(T) == 8, a.nx, a.ny, a.nz, LaunchOptions{}))) {
        plan_march(a.map, a.nx, a.ny, a.nz, 64, 16, 2, opt);
        hipLaunchKernelGGL((adj_wave3d_pair_ahead_kernel<T, BX, BY, 2, 2>), dim3(a.map.total_blocks), dim3(BX * BY), ahead_pad(opt), stream, a);
        return hipGetLastError();
    }
    if constexpr (sizeof(T) == 8) {
        if (plan.small) {
            using S = PairTile<T, BX, BY, 1, 2>;
            const unsigned spad = one_workgroup_per_cu_pad(sizeof(T) * 2 * (S::PLANE1 + S::PLANE2), opt.lds_pad);
            hipLaunchKernelGGL((adj_wave3d_pair_kernel<T, BX, BY, 1, 2>), dim3(a.map.total_blocks), dim3(S::NT), spad, stream, a);
            return hipGetLastError();
        }
    }
    const size_t lds = sizeof(T) * 2 * (G::PLANE1 + G::PLANE2);
    const unsigned pad = one_workgroup_per_cu_pad(lds, opt.lds_pad);
    hipLaunchKernelGGL((adj_wave3d_pair_kernel<T, BX, BY, PY, PX>), dim3(a.map.total_blocks), dim3(G::NT), pad, stream, a);
    return hipGetLastError();
}

// whole vectors per lane: nx a multiple of the vector length and every array aligned to it
bool adjoint_wave3d_pair_supported(int is_f64, int nx, const void *c, const void *p0, const void *p1, const void *p2,
                                   const void *p3)
{
    const size_t al = 16;
    const int px = is_f64 ? 2 : 4;
    const void *arrays[5] = {c, p0, p1, p2, p3};
    for (const void *p : arrays)
        if (reinterpret_cast<uintptr_t>(p) % al != 0) return false;
    return nx % px == 0;
}

hipError_t launch_adjoint_wave3d_pair(int is_f64, int nx, int ny, int nz, const void *c, const void *a, const void *b,
                                      void *out_a, void *out_b, const LaunchOptions &opt, hipStream_t stream)
{
    PairArgs p{};
    p.c = c; p.a = a; p.b = b; p.out_a = out_a; p.out_b = out_b;
    p.nx = nx; p.ny = ny; p.nz = nz;
    return is_f64 ? launch_pair<double, 2>(p, opt, stream) : launch_pair<float, 4>(p, opt, stream);
}

}  // namespace sadj
