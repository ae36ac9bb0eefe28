// Time loops of the Burgers step: several steps per pass over the data, forward and reverse
// (paper Sections 3.1 and 4.2: the nonlinear stencil's adjoint reads the primal states).
//
// A wave holds a window of 64*PXL consecutive cells in registers, PXL per lane, and applies m steps to
// it.  A cell's value after k steps depends on k cells to either side, so `halo` cells at either end of
// the window are recomputed by the neighbouring windows and only the 64*PXL - 2 halo between
// them are stored: halo 16, 8 in passes of up to 8 steps over stored states, and 16, 24 or 32 in passes that recompute up to 8, 12 or 16
// states.  No LDS, no barrier: neighbours travel by whole-wave lane shifts (DPP).
//
// Windows that lie in I = [1, n-2] run without guards; the others clamp their loads into the array
// and mask with selects.  A window belongs to one wave, so the branch between the two is uniform.
//
// What bounds it (fp64; one launch per step before).  Forward with every state stored: memory, 8 + 8/m bytes
// per cell and step instead of 16; 10^7 cells, 16 steps: 245 us, 5.5 TB/s.  Reverse over stored states:
// memory, 8 + 16/m bytes instead of 24; a sweep of 16 steps of 10^7 cells 284 us.  Reverse from a
// checkpoint: 24/m bytes, the m states are recomputed in registers and the vector ALUs are the bound; so is the forward sweep
// that stores checkpoints only.  Per four fp64 cells a forward step takes 38 instructions and a reverse one 64 (43 and 103 before
// both were written with g_- and g_+, see burgers.hpp): 3 10^6 cells, 128 steps, every 16th kept, forward 164 -> 155 us, reverse
// 616 -> 532, and -> 486 with passes of 16 steps.  75 -> 64 with the upwind difference taken by the sign bit, one question for zeros a pass
// and full passes without a condition per step: gradient 662 -> 623 us, fp32 420 -> 386 (up to 5 % more or less from box to box, with the shader clock).
// The vector ALUs issue for 41 us at 2.4 GHz in a pass of 3 10^6 cells of 56 to 61 us, whose last round of windows is partly filled, for 230 in one of 2^24 cells
// of 270 to 300; this load leaves a clock of about 2.1 GHz.  Windows that refresh their ends from their neighbours through LDS, every 4 or 8 steps,
// compute 16 and 11 % fewer cells and measured 0 and 2 % faster (fp32 8 % slower): the waits at the barriers take what the cells save.
#include "burgers.hpp"
#include "burgers_plan.hpp"
#include "launch.hpp"

namespace sadj {

struct BurgersForwardArgs {
    const void *src;        // the state the pass starts from
    void *rows;             // receives the states after steps first, first+every, ... in consecutive rows of n cells
    void *last;             // receives the state after step m (nullable)
    long first, every;
    long n;
    double C, D;
    int m;
    int hold;               // 1: the end cells keep their values; 0: every state is stored (first = every = 1) and
                            // the end cells of every row are given, never written
};

struct BurgersReverseArgs {
    const void *src;        // state t
    const void *rows;       // states t+first, t+first+every, ... (the others are recomputed)
    const void *lam_in;
    void *lam_out;
    long n;
    double C, D;
    int m, first, every;
    int halo;               // cells recomputed on either side of a window, states all in memory
};

constexpr int kLoopWaves = 4;         // windows per workgroup
constexpr int kAhead = 4;             // states in flight in a pass over stored states
constexpr int kLoopH = 16;            // cells recomputed on either side of a window
constexpr int kShortH = 8;            // the same in short passes over stored states
static_assert(kLoopH >= kForwardSteps && kLoopH >= kReverseSteps && kShortH >= kShortSteps, "halo of a pass");

// Cells that a window stores, of the 64 * PXL that it holds.
__host__ __device__ constexpr int own_cells(int PXL, int halo) { return 64 * PXL - 2 * halo; }

// Whole-wave lane shifts (DPP).  shift: the value of the lane to the left (right), `edge` in lane 0
// (63); rotate: the same with lanes 0 and 63 taken as neighbours.
template <bool RIGHT> __device__ __forceinline__ int lane_shift(int v, int edge)
{
    return __builtin_amdgcn_update_dpp(edge, v, RIGHT ? 0x130 : 0x138, 0xf, 0xf, false);
}
template <bool RIGHT> __device__ __forceinline__ int lane_rotate(int v)
{
    return __builtin_amdgcn_update_dpp(0, v, RIGHT ? 0x134 : 0x13c, 0xf, 0xf, true);
}
template <bool RIGHT> __device__ __forceinline__ float lane_shift(float v, float edge)
{
    return __int_as_float(lane_shift<RIGHT>(__float_as_int(v), __float_as_int(edge)));
}
template <bool RIGHT> __device__ __forceinline__ float lane_rotate(float v) { return __int_as_float(lane_rotate<RIGHT>(__float_as_int(v))); }
template <bool RIGHT> __device__ __forceinline__ double lane_shift(double v, double edge)
{
    return __hiloint2double(lane_shift<RIGHT>(__double2hiint(v), __double2hiint(edge)),
                            lane_shift<RIGHT>(__double2loint(v), __double2loint(edge)));
}
template <bool RIGHT> __device__ __forceinline__ double lane_rotate(double v)
{
    return __hiloint2double(lane_rotate<RIGHT>(__double2hiint(v)), lane_rotate<RIGHT>(__double2loint(v)));
}

// min(|a|, |b|, least), NaN if one of them is.  Of doubles the upper words, taken as floats, which keeps their order; one below 2^-1015
// is no normal float, one of 2^1017 or more may be NaN.
__device__ __forceinline__ float least_magnitude(float a, float b, float least)
{
    float r;
    asm("v_minimum3_f32 %0, |%1|, |%2|, %3" : "=v"(r) : "v"(a), "v"(b), "v"(least));
    return r;
}
__device__ __forceinline__ float least_magnitude(double a, double b, float least)
{
    return least_magnitude(__int_as_float(__double2hiint(a)), __int_as_float(__double2hiint(b)), least);
}
constexpr float kLeastNormal = 0x1p-126f;

// A lane's PXL cells of one row, in runs of RUN consecutive cells.  SPREAD: a run is one 16-byte access
// and the lanes' runs lie side by side, so that every access of a wave is one piece of memory; else the
// lane's cells are one run, which needs half the lane shifts.  Rows of an odd length start at
// addresses that are multiples of the element size only, and the vector type says so.
template <class T, int PXL, bool GUARD, bool SPREAD> struct Lane {
    static constexpr int W = 64 * PXL;
    static constexpr int PXV = PXL * sizeof(T) < 16 ? PXL : 16 / (int)sizeof(T);
    static constexpr int RUN = SPREAD ? PXV : PXL, RUNS = PXL / RUN;
    typedef T VT __attribute__((ext_vector_type(PXV), aligned(sizeof(T))));
    long x0, lo, hi;                  // first cell of the lane's first run; cells lo .. hi-1 are the window's own
    long n;
    int lane, halo;                   // cells recomputed on either side, a multiple of RUN
    bool in[PXL];

    __device__ __forceinline__ Lane(long w, int lane_, long n_, int halo_) : n(n_), lane(lane_), halo(halo_)
    {
        const int V = own_cells(PXL, halo);
        x0 = w * V - halo + (long)lane * RUN;
        lo = w * V;
        hi = (w + 1) * V < n ? (w + 1) * V : n;
#pragma unroll
        for (int e = 0; e < PXL; ++e) in[e] = GUARD ? (cell(e) >= 1 && cell(e) <= n - 2) : true;
    }
    __device__ __forceinline__ long cell(int e) const { return x0 + e / RUN * (64 * RUN) + e % RUN; }

    template <bool STREAM = false> __device__ __forceinline__ void load(const T *p, T (&v)[PXL]) const
    {
        if (!GUARD) {
#pragma unroll
            for (int h = 0; h < PXL; h += PXV) {
                const VT *q = reinterpret_cast<const VT *>(p + cell(h));
                const VT t = STREAM ? __builtin_nontemporal_load(q) : *q;
#pragma unroll
                for (int e = 0; e < PXV; ++e) v[h + e] = t[e];
            }
        } else {
#pragma unroll
            for (int e = 0; e < PXL; ++e) {
                long i = cell(e);
                i = i < 0 ? 0 : (i > n - 1 ? n - 1 : i);
                v[e] = p[i];
            }
        }
    }
    // ends: the end cells of the array are stored as well
    __device__ __forceinline__ void store(T *p, const T (&v)[PXL], bool ends) const
    {
        if (!GUARD) {
            // whole runs are the window's own or not
#pragma unroll
            for (int h = 0; h < PXL; h += PXV) {
                const int r = h / RUN;
                VT t;
#pragma unroll
                for (int e = 0; e < PXV; ++e) t[e] = v[h + e];
                if ((r > 0 || lane >= halo / RUN) && (r < RUNS - 1 || lane < 64 - halo / RUN))
                    __builtin_nontemporal_store(t, reinterpret_cast<VT *>(p + cell(h)));
            }
        } else {
#pragma unroll
            for (int e = 0; e < PXL; ++e)
                if (cell(e) >= lo && cell(e) < hi && (ends || in[e])) p[cell(e)] = v[e];
        }
    }
    // The cells before (after) each run; any value beyond the window, which only reaches cells that are discarded.
    __device__ __forceinline__ void before(const T (&v)[PXL], T (&left)[RUNS]) const
    {
#pragma unroll
        for (int r = 0; r < RUNS; ++r) {
            const T end = v[r * RUN + RUN - 1];
            left[r] = r > 0 ? lane_shift<false>(end, lane_rotate<false>(v[r > 0 ? r * RUN - 1 : 0])) : lane_rotate<false>(end);
        }
    }
    __device__ __forceinline__ void after(const T (&v)[PXL], T (&right)[RUNS]) const
    {
#pragma unroll
        for (int r = 0; r < RUNS; ++r) {
            const T first = v[r * RUN];
            right[r] = r < RUNS - 1 ? lane_shift<true>(first, lane_rotate<true>(v[r < RUNS - 1 ? (r + 1) * RUN : 0])) : lane_rotate<true>(first);
        }
    }
    __device__ __forceinline__ void beside(const T (&v)[PXL], T (&left)[RUNS], T (&right)[RUNS]) const
    {
        before(v, left);
        after(v, right);
    }
    template <bool CHECKED> __device__ __forceinline__ void primal_step(T (&u)[PXL], T C, T D) const
    {
        T ul[RUNS], ur[RUNS], next[PXL];
        beside(u, ul, ur);
#pragma unroll
        for (int e = 0; e < PXL; ++e) {
            const T val = burgers_primal_cell<CHECKED>(e % RUN == 0 ? ul[e / RUN] : u[e - 1], u[e], e % RUN == RUN - 1 ? ur[e / RUN] : u[e + 1], C, D);
            next[e] = in[e] ? val : u[e];
        }
#pragma unroll
        for (int e = 0; e < PXL; ++e) u[e] = next[e];
    }
    // Whether a value of the window (any lane's) is not finite: a lane's sum is not if one of its cells is not (or if it overflows, which
    // costs a second pass and changes nothing).  Additions, because a class test per cell needs a scalar operation each.
    __device__ __forceinline__ bool not_finite(const T (&u)[PXL]) const
    {
        T sum[PXL];
#pragma unroll
        for (int e = 0; e < PXL; ++e) sum[e] = u[e];
#pragma unroll
        for (int k = PXL / 2; k > 0; k /= 2)
#pragma unroll
            for (int e = 0; e < k; ++e) sum[e] = add_rounded(sum[e], sum[e + k]);
        return __any(!__builtin_isfinite(sum[0]));
    }
    // Of the cells of several states, one state after the other: whether one (any lane's) may be zero is then asked once.
    __device__ __forceinline__ float least_of(const T (&u)[PXL], float least) const
    {
#pragma unroll
        for (int e = 0; e < PXL; e += 2) least = least_magnitude(u[e], u[e + 1], least);
        return least;
    }
    static __device__ __forceinline__ bool maybe_zero(float least) { return __any(!(least >= kLeastNormal)); }
    // CHECKED: for states that may not be finite.  zero (the same in all lanes): cells of u may be zero.
    template <bool CHECKED> __device__ __forceinline__ void reverse_step(const T (&u)[PXL], T (&lam)[PXL], T C, T D, bool zero) const
    {
        T ul[RUNS], ur[RUNS], lr[RUNS], left[RUNS], slope[PXL], give[PXL], next[PXL];
        beside(u, ul, ur);
#pragma unroll
        for (int e = 0; e < PXL; ++e) {
            lam[e] = in[e] ? lam[e] : T(0);                                // lam outside I is never used
            slope[e] = burgers_slope(e % RUN == 0 ? ul[e / RUN] : u[e - 1], u[e], e % RUN == RUN - 1 ? ur[e / RUN] : u[e + 1]);
            give[e] = mul_rounded(burgers_to_right(u[e], C, D), lam[e]);
        }
        // u = 0 exactly is rare but in fields that are zero over a stretch
        if (CHECKED || zero) {
#pragma unroll
            for (int e = 0; e < PXL; ++e) {
                const T um = e % RUN == 0 ? ul[e / RUN] : u[e - 1], up = e % RUN == RUN - 1 ? ur[e / RUN] : u[e + 1];
                slope[e] = CHECKED ? burgers_slope_in_full(slope[e], um, u[e], up) : burgers_slope_at_zero(slope[e], um, u[e], up);
            }
        }
        before(give, left);
        after(lam, lr);
#pragma unroll
        for (int e = 0; e < PXL; ++e) {
            const bool first = e % RUN == 0, end = e % RUN == RUN - 1;
            next[e] = burgers_adjoint_cell(slope[e], end ? ur[e / RUN] : u[e + 1], first ? left[e / RUN] : give[e - 1], lam[e],
                                           end ? lr[e / RUN] : lam[e + 1], C, D, in[e]);
        }
#pragma unroll
        for (int e = 0; e < PXL; ++e) lam[e] = next[e];
    }
};

// What follows is computed from `lane` anew: in code that is rarely reached, addresses kept from before would cost that code registers.
template <class T> __device__ __forceinline__ void computed_here(T &v) { asm volatile("" : "+v"(v)); }

// The value that lane `from` (uniform) holds, in all lanes.
__device__ __forceinline__ float lane_value(float v, int from) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), from)); }
__device__ __forceinline__ double lane_value(double v, int from)
{
    return __hiloint2double(__builtin_amdgcn_readlane(__double2hiint(v), from), __builtin_amdgcn_readlane(__double2loint(v), from));
}

// A pass over one window.  Returns whether the checked form is needed: a cell that is not finite stays so and makes its neighbours'
// next values so, in either form of the step, so if the last state is finite all were.
template <bool CHECKED, class T, int PXL, bool GUARD, bool SPREAD>
__device__ __forceinline__ bool burgers_forward_window(const BurgersForwardArgs &a, long w, int lane)
{
    if (CHECKED) computed_here(lane);
    const Lane<T, PXL, GUARD, SPREAD> L(w, lane, a.n, kLoopH);
    const T C = (T)a.C, D = (T)a.D;
    T u[PXL];
    L.load(static_cast<const T *>(a.src), u);
    T *row = static_cast<T *>(a.rows);
    long next = a.first;
    // Given end cells of the m rows: lanes 0 .. 15 fetch cell 0, lanes 16 .. 31 cell n-1 of row 0 .. 15 before the
    // loop.  Fetched where they are needed, each step of an end window would wait for memory
    // (16 stored steps of 10^6 fp32 cells: 29 us instead of 13).
    T ends = T(0);
    if (GUARD && !a.hold && lane < 32) ends = row[(long)min(lane & 15, a.m - 1) * a.n + (lane < 16 ? 0 : a.n - 1)];
    static_assert(kForwardSteps <= 16, "a lane per given end cell");
    for (int s = 0; s < a.m;) {
        const int stop = next < a.m ? (int)next : a.m;
        if (!CHECKED) {
            for (; s + 2 <= stop; s += 2) {       // by twos: the cells need no moves between registers
                L.template primal_step<false>(u, C, D);
                L.template primal_step<false>(u, C, D);
            }
        }
        for (; s < stop; ++s) L.template primal_step<CHECKED>(u, C, D);
        if (s != next) continue;
        if (GUARD && !a.hold) {
#pragma unroll
            for (int e = 0; e < PXL; ++e) {
                const T left = lane_value(ends, s - 1), right = lane_value(ends, s + 15);
                u[e] = L.cell(e) == 0 ? left : L.cell(e) == a.n - 1 ? right : u[e];
            }
        }
        L.store(row, u, a.hold);
        row += a.n;
        next += a.every;
    }
    if (a.last) L.store(static_cast<T *>(a.last), u, true);
    return !CHECKED && L.not_finite(u);
}

template <class T, int PXL, bool SPREAD> __global__ __launch_bounds__(64 * kLoopWaves) void burgers_forward_kernel(BurgersForwardArgs a)
{
    constexpr int W = 64 * PXL, V = own_cells(PXL, kLoopH);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long w = (long)blockIdx.x * kLoopWaves + wave, x0 = w * V - kLoopH;
    if (w * V >= a.n) return;
    const bool inside = x0 >= 1 && x0 + W - 1 <= a.n - 2;
    const bool again = inside ? burgers_forward_window<false, T, PXL, false, SPREAD>(a, w, lane) : burgers_forward_window<false, T, PXL, true, SPREAD>(a, w, lane);
    // rare: the pass is done again from its source, which it never writes
    if (__builtin_expect(again, 0)) burgers_forward_window<true, T, PXL, true, SPREAD>(a, w, lane);
}

// The end cells of all rows that a pass reads: cell 0 in lanes 0 .. 15, cell n-1 in lanes 16 .. 31 (src where there is no such row).
template <class T> __device__ __forceinline__ T end_cells(const BurgersReverseArgs &a, int lane)
{
    static_assert(kRecomputeSteps <= 16 && kReverseSteps <= 16, "a lane per end cell");
    const int row = lane & 15;
    const bool read = row > 0 && a.first + (row - 1) * a.every < a.m;
    const T *p = read ? static_cast<const T *>(a.rows) + (row - 1) * a.n : static_cast<const T *>(a.src);
    return p[(lane & 16) == 0 ? 0 : a.n - 1];
}

// Reverse steps over m states that are all in memory (rows follows src, first = every = 1), m % kAhead == REM.
// The requests follow the length of the pass: an earlier form issued those of 15 steps always, re-reading the
// last state for the missing ones, and a sweep of 5 steps over 4 10^6 fp32 cells took 60 us instead of 38, of 3 steps
// over 10^6 fp64 cells 29 instead of 17.
// Returns false, as burgers_reverse_recompute does, if a state may not have been finite: a cell of I whose u is not finite has a
// slope that is not, so its lam is not finite after that step and stays so.  The end cells have no lam of their own;
// windows that hold one look at them in the rows that the pass reads (recomputed states keep them).
template <class T, int PXL, bool GUARD, int REM>
__device__ __forceinline__ bool burgers_reverse_stored(const BurgersReverseArgs &a, long w, int lane)
{
    const Lane<T, PXL, GUARD, true> L(w, lane, a.n, a.halo);
    const T C = (T)a.C, D = (T)a.D;
    const T *src = static_cast<const T *>(a.src);
    T lam[PXL], u[kAhead][PXL];
    L.load(static_cast<const T *>(a.lam_in), lam);
    const T ends = GUARD ? end_cells<T>(a, lane) : T(0);
    stored_reverse_schedule<kAhead, REM>(
        a.m, [&](int t, int slot) { L.template load<true>(src + (long)t * a.n, u[slot]); },
        [&](int slot) {
            L.template reverse_step<false>(u[slot], lam, C, D, L.maybe_zero(L.least_of(u[slot], __builtin_inff())));
            __builtin_amdgcn_sched_barrier(0);       // steps interleaved with each other need half as many registers again
        });
    L.store(static_cast<T *>(a.lam_out), lam, true);
    return !(L.not_finite(lam) || (GUARD && __any(!__builtin_isfinite(ends))));
}

// Reverse steps from a checkpoint: the states are recomputed forward from state t into registers, except
// where a further checkpoint is met.
// FULL: all M steps.  Forward and reverse steps of a state share values that would occupy registers in between: computed_here
// keeps them apart.
template <class T, int PXL, bool GUARD, int M, bool FULL>
__device__ __forceinline__ bool burgers_reverse_recompute(const BurgersReverseArgs &a, long w, int lane)
{
    const Lane<T, PXL, GUARD, false> L(w, lane, a.n, 2 * M);
    const T C = (T)a.C, D = (T)a.D;
    T lam[PXL], u[M][PXL];
    L.load(static_cast<const T *>(a.src), u[0]);
    L.load(static_cast<const T *>(a.lam_in), lam);
    const T ends = GUARD ? end_cells<T>(a, lane) : T(0);
    const T *row = static_cast<const T *>(a.rows);
    int next = a.first;
    float least = L.least_of(u[0], __builtin_inff());
#pragma unroll
    for (int s = 1; s < M; ++s) {
        if (!FULL && s >= a.m) continue;
        if (s == next) {
            L.load(row, u[s]);
            row += a.n;
            next += a.every;
        } else {
#pragma unroll
            for (int e = 0; e < PXL; ++e) u[s][e] = u[s - 1][e];
            L.template primal_step<false>(u[s], C, D);
        }
        least = L.least_of(u[s], least);
    }
    const bool zero = L.maybe_zero(least);
#pragma unroll
    for (int s = M - 1; s >= 0; --s) {
        if (FULL) {
#pragma unroll
            for (int e = 0; e < PXL; ++e) computed_here(u[s][e]);
        }
        if (FULL || s < a.m) L.template reverse_step<false>(u[s], lam, C, D, zero);
        __builtin_amdgcn_sched_barrier(0);           // nor are steps to be interleaved
    }
    L.store(static_cast<T *>(a.lam_out), lam, true);
    return !(L.not_finite(lam) || (GUARD && __any(!__builtin_isfinite(ends))));
}

// A pass of either kind over states that may not be finite: for each reverse step its state anew from the row before it, in the
// checked forms, and the lanes store the cells that they stored before.  Loops instead of a pass in registers: small beside the
// code above, which runs 4 to 6 % slower with tests between its steps or a second copy of itself (3 10^6 cells, fp64 and fp32).  As it
// is the tests cost a reverse sweep 0.4 % in fp64 and 1.3 to 1.8 % in fp32 (10^6 and 3 10^6 cells).
template <class T, int PXL, bool SPREAD>
__device__ __forceinline__ void burgers_reverse_not_finite(const BurgersReverseArgs &a, long w, int lane, int halo)
{
    computed_here(lane);
    const Lane<T, PXL, true, SPREAD> L(w, lane, a.n, halo);
    const T C = (T)a.C, D = (T)a.D;
    T lam[PXL], u[PXL];
    L.load(static_cast<const T *>(a.lam_in), lam);
#pragma unroll 1
    for (int s = a.m - 1; s >= 0; --s) {
        const int rows = s < a.first ? 0 : (s - a.first) / a.every + 1;       // that hold states up to s, src not counted
        L.load(rows == 0 ? static_cast<const T *>(a.src) : static_cast<const T *>(a.rows) + (rows - 1) * a.n, u);
#pragma unroll 1
        for (int t = rows == 0 ? 0 : a.first + (rows - 1) * a.every; t < s; ++t) L.template primal_step<true>(u, C, D);
        L.template reverse_step<true>(u, lam, C, D, true);
    }
    L.store(static_cast<T *>(a.lam_out), lam, true);
}

// REM: number of steps modulo kAhead of a pass over stored states; -M: up to M states are recomputed.  FULL: M steps, known at compile
// time, so that lam needs no moves where the steps' branches would join: 4 instructions of 68 a step.  The waves per SIMD are those
// that fit without it, but for fp64 passes of 8 steps (134 registers, 3 waves; held to 128 they spill: 433 / 468 us for 97 steps of 3 10^6
// cells).  In wide windows of floats passes of 8 steps take the form with conditions (295 us; FULL 311, held to 128 registers 330), and so do
// those of 12, which FULL spills three registers of (153 without; 6 10^5 cells, 120 steps, every 12th kept 103 / 107 us, 2 10^6, 96, 24th 203 / 208).
template <class T, int PXL, int REM, bool FULL>
__global__ __launch_bounds__(64 * kLoopWaves, REM == -12 ? 3 : REM == -16 ? 2 : 1) void burgers_reverse_kernel(BurgersReverseArgs a)
{
    const int halo = REM >= 0 ? a.halo : -2 * REM, W = 64 * PXL, V = own_cells(PXL, halo);
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const long w = (long)blockIdx.x * kLoopWaves + wave, x0 = w * V - halo;
    if (w * V >= a.n) return;
    const bool inside = x0 >= 1 && x0 + W - 1 <= a.n - 2;
    bool done;
    if (__builtin_expect(inside, 1)) {
        if constexpr (REM >= 0) done = burgers_reverse_stored<T, PXL, false, REM>(a, w, lane);
        else done = burgers_reverse_recompute<T, PXL, false, -REM, FULL>(a, w, lane);
    } else {
        if constexpr (REM >= 0) done = burgers_reverse_stored<T, PXL, true, REM>(a, w, lane);
        else done = burgers_reverse_recompute<T, PXL, true, -REM, false>(a, w, lane);
    }
    if (__builtin_expect(!done, 0)) burgers_reverse_not_finite<T, PXL, (REM >= 0)>(a, w, lane, halo);
}

// Cells per lane: wide windows recompute the least (own cells of 256 in fp64: 224, in a reverse pass of 16 recomputed states 192; of 512
// in fp32: 480 and 448) and are taken where every SIMD of the chip gets one; shorter arrays are spread over more SIMDs in narrow
// windows (96 and 64 of 128).  Narrow / wide, us, 16 stored forward steps and a reverse sweep of 64 steps from every 16th state:
// fp64 10^5 cells 11.8 / 14.0 and 40.5 / 43.5, 2.3 10^5 12.0 / 12.5 and 54.4 / 53.2, 5 10^5 22.4 / 21.4 and 84.9 / 75.2, 10^6 40.9 / 36.8 and
// 147 / 124; fp32 10^5 11.1 / 14.5 and 36.8 / 55.0, 3 10^5 11.7 / 14.7 and 52.0 / 57.6, 5 10^5 12.6 / 15.2 and 64.0 / 63.2, 7 10^5 18.1 / 17.5 and
// 90.3 / 66.6, 2 10^6 47.0 / 39.9 and 168 / 139.
template <class T> static bool wide_windows(long n)
{
    return n >= 1024L * own_cells(32 / (int)sizeof(T), kLoopH);
}

static dim3 loop_grid(int PXL, int halo, long n)
{
    const long windows = ceil_div(n, own_cells(PXL, halo));
    return dim3((unsigned)ceil_div(windows, kLoopWaves));
}

template <class T, bool SPREAD> static hipError_t forward_T(const BurgersForwardArgs &a, hipStream_t stream)
{
    constexpr int WIDE = 32 / (int)sizeof(T), NARROW = 2;
    const dim3 block(64 * kLoopWaves);
    if (wide_windows<T>(a.n)) hipLaunchKernelGGL((burgers_forward_kernel<T, WIDE, SPREAD>), loop_grid(WIDE, kLoopH, a.n), block, 0, stream, a);
    else hipLaunchKernelGGL((burgers_forward_kernel<T, NARROW, SPREAD>), loop_grid(NARROW, kLoopH, a.n), block, 0, stream, a);
    return hipGetLastError();
}

template <class T, int REM, bool FULL = false> static hipError_t reverse_T(const BurgersReverseArgs &a, hipStream_t stream)
{
    constexpr int WIDE = 32 / (int)sizeof(T), NARROW = 2;
    constexpr bool WIDE_FULL = FULL && !(sizeof(T) == 4 && REM == -12);     // see burgers_reverse_kernel
    const dim3 block(64 * kLoopWaves);
    if (wide_windows<T>(a.n))
        hipLaunchKernelGGL((burgers_reverse_kernel<T, WIDE, REM, WIDE_FULL>), loop_grid(WIDE, REM >= 0 ? a.halo : -2 * REM, a.n), block, 0, stream, a);
    else
        hipLaunchKernelGGL((burgers_reverse_kernel<T, NARROW, REM, FULL>), loop_grid(NARROW, REM >= 0 ? a.halo : -2 * REM, a.n), block, 0, stream, a);
    return hipGetLastError();
}

template <class T> static hipError_t reverse_stored_T(const BurgersReverseArgs &a, hipStream_t stream)
{
    static_assert(kAhead == 4, "a case per remainder");
    switch (a.m % kAhead) {
    case 0: return reverse_T<T, 0>(a, stream);
    case 1: return reverse_T<T, 1>(a, stream);
    case 2: return reverse_T<T, 2>(a, stream);
    default: return reverse_T<T, 3>(a, stream);
    }
}

template <class T> static hipError_t reverse_recompute_T(const BurgersReverseArgs &a, hipStream_t stream)
{
    switch (recompute_kernel(a.m)) {
    case 8: return sizeof(T) == 8 && a.m == 8 ? reverse_T<T, -8, sizeof(T) == 8>(a, stream) : reverse_T<T, -8>(a, stream);
    case 12: return a.m == 12 ? reverse_T<T, -12, true>(a, stream) : reverse_T<T, -12>(a, stream);
    default: return a.m == 16 ? reverse_T<T, -16, true>(a, stream) : reverse_T<T, -16>(a, stream);
    }
}

namespace {

struct LoopOps {
    int is_f64;
    long n;
    double C, D;
    hipStream_t stream;

    int forward(const char *src, char *rows, long first, long every, int m, char *last, bool hold) const
    {
        const BurgersForwardArgs a{src, rows, last, first, every, n, C, D, m, hold ? 1 : 0};
        if (every == 1) return is_f64 ? forward_T<double, true>(a, stream) : forward_T<float, true>(a, stream);
        return is_f64 ? forward_T<double, false>(a, stream) : forward_T<float, false>(a, stream);
    }
    int reverse(const char *src, const char *rows, int first, int every, int m, const char *lam_in, char *lam_out) const
    {
        // Nothing to keep between steps: the single-step kernel computes no cell twice.  It moves one cell per lane
        // where an array is not 16-byte aligned, which costs more (16 10^6 cells fp64 80 us, the window 63).
        const uintptr_t at = reinterpret_cast<uintptr_t>(src) | reinterpret_cast<uintptr_t>(lam_in) | reinterpret_cast<uintptr_t>(lam_out);
        if (m == 1 && at % 16 == 0) return launch_adjoint_burgers1d(is_f64, n, C, D, src, lam_in, lam_out, 1, stream);
        const BurgersReverseArgs a{src, rows, lam_in, lam_out, n, C, D, m, first, every, m <= kShortSteps ? kShortH : kLoopH};
        if (every == 1) return is_f64 ? reverse_stored_T<double>(a, stream) : reverse_stored_T<float>(a, stream);
        return is_f64 ? reverse_recompute_T<double>(a, stream) : reverse_recompute_T<float>(a, stream);
    }
    int reverse_first(const char *u, const char *lam_in, char *lam_out) const
    {
        return launch_adjoint_burgers1d(is_f64, n, C, D, u, lam_in, lam_out, 0, stream);
    }
};

}  // namespace

hipError_t launch_burgers_history_forward(int is_f64, long n, long nsteps, double C, double D, void *states, hipStream_t stream)
{
    LoopOps ops{is_f64, n, C, D, stream};
    return (hipError_t)plan_burgers_history_forward(ops, static_cast<char *>(states), (size_t)n * (is_f64 ? 8 : 4), nsteps);
}
hipError_t launch_burgers_history_reverse(int is_f64, long n, long nsteps, double C, double D, const void *states, void *const (&lam)[2],
                                          hipStream_t stream)
{
    LoopOps ops{is_f64, n, C, D, stream};
    char *const l[2] = {static_cast<char *>(lam[0]), static_cast<char *>(lam[1])};
    return (hipError_t)plan_burgers_history_reverse(ops, static_cast<const char *>(states), (size_t)n * (is_f64 ? 8 : 4), nsteps, l);
}
hipError_t launch_burgers_ckpt_forward(int is_f64, long n, long nsteps, long every, double C, double D, void *ckpt, void *work,
                                       void *u_final, hipStream_t stream)
{
    LoopOps ops{is_f64, n, C, D, stream};
    return (hipError_t)plan_burgers_ckpt_forward(ops, static_cast<char *>(ckpt), static_cast<char *>(work), static_cast<char *>(u_final),
                                                 (size_t)n * (is_f64 ? 8 : 4), nsteps, every);
}
hipError_t launch_burgers_ckpt_reverse(int is_f64, long n, long nsteps, long every, double C, double D, const void *ckpt, void *work,
                                       void *const (&lam)[2], hipStream_t stream)
{
    if (every == 1) return launch_burgers_history_reverse(is_f64, n, nsteps, C, D, ckpt, lam, stream);
    LoopOps ops{is_f64, n, C, D, stream};
    char *const l[2] = {static_cast<char *>(lam[0]), static_cast<char *>(lam[1])};
    const bool wide = is_f64 ? wide_windows<double>(n) : wide_windows<float>(n);
    BurgersCkptReverse<LoopOps> plan{ops, static_cast<const char *>(ckpt), static_cast<char *>(work), (size_t)n * (is_f64 ? 8 : 4), every,
                                     recompute_steps(n, wide ? (is_f64 ? 256 : 512) : 128, every)};
    return (hipError_t)plan.run(nsteps, l);
}

}  // namespace sadj
