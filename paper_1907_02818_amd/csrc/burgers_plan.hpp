// Order of launches of the Burgers time loops: which runs of steps share a pass over the data, where
// the states between passes go, and which buffers the adjoint alternates between.  Host code
// without any device call, so that the order can be replayed on a CPU; `Ops` makes the launches:
//   int forward(src, rows, first, every, m, last, hold)   m steps from the state at src; the state
//        after step s = first, first+every, ... goes to rows, rows+1, ..., the state after step m
//        also to `last` (null: not wanted)
//   int reverse(src, rows, first, every, m, lam_in, lam_out)   m reverse steps in assign mode over
//        the states t, t+1, ..., t+m-1: state t is at src, state t+first at rows, t+first+every at
//        rows+1, ..., the others are recomputed
//   int reverse_first(u, lam_in, lam_out)   one reverse step, accumulated into lam_out
// Rows and lam buffers are byte pointers, a row is `row` bytes; 0 is success, anything else ends
// the plan and is returned.
#pragma once
#include <cstddef>

namespace sadj {

// Steps that one pass can take (bounded by the cells it recomputes beside its window).
constexpr int kForwardSteps = 16;     // forward: one cell per step and side
constexpr int kReverseSteps = 15;     // reverse, all states in memory: one cell per step and side
constexpr int kShortSteps = 8;        // longest of the passes over states in memory that recompute half as many cells
constexpr size_t kUnevenRow = (size_t)96 << 20;
constexpr int kRecomputeSteps = 16;   // reverse from a checkpoint: two cells per step and side

inline long ceil_div(long a, long b) { return (a + b - 1) / b; }

// Order of memory requests and steps of a reverse pass over m states that are all in memory, m % AHEAD == REM:
// load(t, slot) requests state t into one of AHEAD register sets, step(slot) applies the state in it;
// m-1, m-2, ..., 0 are applied in this order.  Each state is requested once, AHEAD steps early, and no request
// is behind a condition, so that the wait before a step leaves the later ones outstanding.
template <int AHEAD, int REM, class Load, class Step>
__attribute__((always_inline)) constexpr void stored_reverse_schedule(int m, const Load &load, const Step &step)
{
    if (m < AHEAD) {
#pragma unroll
        for (int j = 0; j < REM; ++j) load(m - 1 - j, j);
#pragma unroll
        for (int j = 0; j < REM; ++j) step(j);
        return;
    }
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) load(m - 1 - j, j);
#pragma unroll
    for (int j = 0; j < REM; ++j) {
        step(j);
        load(m - 1 - AHEAD - j, j);
    }
    int t = m - 1 - REM - AHEAD;                                 // the state to be requested next
    for (; t >= 0; t -= AHEAD)
#pragma unroll
        for (int j = 0; j < AHEAD; ++j) {
            step((REM + j) % AHEAD);
            load(t - j, (REM + j) % AHEAD);
        }
#pragma unroll
    for (int j = 0; j < AHEAD; ++j) step((REM + j) % AHEAD);
}

// The kernel that takes a pass of m recomputed steps: it holds 8, 12 or 16 states in registers (fp64: 116, 148 and 180 of them, 4, 3 and 2
// waves per SIMD; in passes of exactly 8, 12 or 16 steps 134, 166 and 198, 3, 3 and 2 waves) and recomputes two cells per state and side.
inline int recompute_kernel(int m) { return m <= 8 ? 8 : m <= 12 ? 12 : 16; }

// Longest pass of a checkpointed reverse sweep (8, 12 or 16 steps) on n cells in windows of `window`: the one whose passes cost
// least per step.  A pass costs its launch, about 60 instructions in each of 10^6 cells, and per cell 20 instructions' time for
// its loads and stores, 9 instructions for each state that it recomputes and 17 for each reverse step, times window / own cells;
// fewer waves per SIMD cost 3 and 5 %.  (A reverse step takes 16 by now, and passes of exactly 8 steps have three waves; with these weights one choice in twenty
// would be another, between lengths that the model puts within 3 % of each other.  The choices below are still the fastest, or within 2 % of it.)
// Long passes spare launches and, where they cover a checkpoint interval, the launches that
// would find the states inside it; short ones recompute fewer cells beside their windows.  Reverse sweeps with 8 / 12 / 16 at most: fp64
// 3 10^6 cells, 128 steps, every 16th kept 520 / 533 / 451 us; 1.7 10^7, 64, 16th 1399 / 1399 / 1345; 1.2 10^6, 185, 6th 342 / 292 / 288;
// 6 10^6, 64, 8th 427 / 425 / 521; fp32 3 10^6, 128, 16th 385 / 384 / 307; 10^6, 128, 12th 217 / 147 / 146; 8 10^6, 64, 8th 344 / 344 / 352.
inline int recompute_steps(long n, int window, long every)
{
    int best = 8;
    double best_cost = 0;
    for (int most = 8; most <= kRecomputeSteps; most += 4) {
        double steps, passes, work;
        auto pass = [&](int m, long kept) {                      // kept: states found in memory, the first one among them
            const int states = recompute_kernel(m);
            const double cells = (double)window / (window - 4 * states), waves = states == 8 ? 1 : states == 12 ? 1.03 : 1.05;
            return (9.0 * (m - kept) + 17.0 * m) * cells * waves;
        };
        if (every <= most) {
            steps = (double)(most / every * every);
            passes = 1;
            work = pass((int)steps, most / every);
        } else {
            const long parts = ceil_div(every, most), size = ceil_div(every, parts);
            steps = (double)every;
            passes = (double)(parts + ceil_div(parts - 1, kForwardSteps / size));
            work = parts * pass((int)size, 1) + 9.0 * 1.14 * (parts - 1) * size;
        }
        const double cost = (passes * (60e6 + 20 * (double)n) + work * (double)n) / steps;
        if (most == 8 || cost < best_cost) { best = most; best_cost = cost; }
    }
    return best;
}

// nsteps forward steps that store every state (row t at base + t*row, row 0 given).
template <class Ops> int plan_burgers_history_forward(Ops &ops, char *base, size_t row, long nsteps)
{
    const long passes = ceil_div(nsteps, kForwardSteps);
    for (long t = 0, i = 0; i < passes; ++i) {
        const long m = ceil_div(nsteps - t, passes - i);
        if (int e = ops.forward(base + (size_t)t * row, base + (size_t)(t + 1) * row, 1, 1, (int)m, nullptr, false)) return e;
        t += m;
    }
    return 0;
}

// Reverse sweep over nsteps states in consecutive rows (state t at base + t*row); the result is in
// lam[nsteps % 2].  After the first step, which accumulates into lam[1], every pass reads one of
// the two buffers and writes the other, so the number of passes has the parity of the steps left.
// The passes are of equal length, but where one short pass and single steps do, those are taken: a single
// step has no window ends to compute twice.  Not for rows that the last-level cache (256 MB) cannot hold two
// of, where a single step reads and writes lam in memory.  8 steps after the first one as 4 + 4 / 7 + 1: 10^6 fp32
// cells 18.6 / 15.9 us, 4 10^6 53.0 / 48.2, 16 10^6 (64 MB rows) 179 / 166, 16 10^6 fp64 cells (128 MB) 323 / 339.
template <class Ops> int plan_burgers_history_reverse(Ops &ops, const char *base, size_t row, long nsteps, char *const (&lam)[2])
{
    if (nsteps <= 0) return 0;
    if (int e = ops.reverse_first(base + (size_t)(nsteps - 1) * row, lam[0], lam[1])) return e;
    long left = nsteps - 1;
    if (left == 0) return 0;
    long passes = ceil_div(left, kReverseSteps);
    passes += (passes ^ left) & 1;
    for (int cur = 1; passes > 0; --passes, cur ^= 1) {
        const long uneven = left - (passes - 1);
        const long m = uneven <= kShortSteps && row <= kUnevenRow ? uneven : ceil_div(left, passes);
        left -= m;
        const char *src = base + (size_t)left * row;
        if (int e = ops.reverse(src, src + row, 1, 1, (int)m, lam[cur], lam[cur ^ 1])) return e;
    }
    return 0;
}

// Forward sweep that stores the states every, 2*every, ... in rows 1, 2, ... of ckpt (row 0 given) and the
// last one in u_final (nullable); work: two rows.
template <class Ops> int plan_burgers_ckpt_forward(Ops &ops, char *ckpt, char *work, char *u_final, size_t row, long nsteps, long every)
{
    // passes that end at a checkpoint: several intervals each where they are short, else equal parts of one
    const long step = every <= kForwardSteps ? kForwardSteps / every * every : ceil_div(every, ceil_div(every, kForwardSteps));
    const char *cur = ckpt;
    int w = 0;
    for (long t = 0; t < nsteps;) {
        long end = t + step;
        if (every > kForwardSteps && end > (t / every + 1) * every) end = (t / every + 1) * every;
        if (end > nsteps) end = nsteps;
        char *last = end == nsteps ? u_final : nullptr;
        if (end % every != 0 && !last) { last = work + (size_t)w * row; w ^= 1; }
        const long next = t / every + 1;                         // the first checkpoint after t
        if (int e = ops.forward(cur, ckpt + (size_t)next * row, next * every - t, every, (int)(end - t), last, true)) return e;
        cur = end % every == 0 ? ckpt + (size_t)(end / every) * row : last;
        t = end;
    }
    return 0;
}

// Reverse sweep from checkpoints (state j*every in row j of ckpt, every >= 2); the result is in
// lam[nsteps % 2].  work: every-1 rows, for states at which a pass starts and, where the number of
// passes has the wrong parity, for the adjoint between the last two passes.
template <class Ops> struct BurgersCkptReverse {
    Ops &ops;
    const char *ckpt;
    char *work;
    size_t row;
    long every;
    int most;                           // longest pass, see recompute_steps

    const char *ckpt_row(long j) const { return ckpt + (size_t)j * row; }

    // Number of passes over the states 0 .. hi-1 with at most `most` steps each.
    long count(long hi, int most) const
    {
        if (every <= most) return ceil_div(hi, most / every * every);
        return hi / every * ceil_div(every, most) + ceil_div(hi % every, most);
    }

    // State t, t >= t0 = the checkpoint before it: steps t0 -> t with the last state in `to`.
    int state_to(long t, char *to)
    {
        const long t0 = t / every * every;
        const char *cur = ckpt_row(t0 / every);
        long left = t - t0;
        int w = 1;                                               // rows 1 and 2 between passes (every > 16 here)
        while (left > 0) {
            const long m = left < kForwardSteps ? left : (long)kForwardSteps;
            left -= m;
            char *dst = left == 0 ? to : work + (size_t)w * row;
            if (int e = ops.forward(cur, nullptr, every + m, every, (int)m, dst, true)) return e;
            cur = dst;
            w ^= 3;
        }
        return 0;
    }

    int run(long nsteps, char *const (&lam)[2])
    {
        if (nsteps <= 0) return 0;
        const long top = nsteps - 1;
        const char *u = ckpt_row(top / every);
        if (top % every != 0) {
            if (int e = state_to(top, work)) return e;
            u = work;
        }
        if (int e = ops.reverse_first(u, lam[0], lam[1])) return e;
        if (top == 0) return 0;
        long passes = count(top, most);
        if (passes == 1 && top % 2 == 0) {                       // one pass would have to write the buffer it reads
            most = (int)(top / 2);
            passes = count(top, most);
        }
        const bool detour = (passes - top) % 2 != 0;             // the last pass but one leaves lam in a row of work
        char *in = lam[1];
        int cur = 1;
        auto pass = [&](const char *src, long t, long m) {
            --passes;
            char *out = lam[cur ^ 1];
            if (detour && passes == 1) out = work + (size_t)(every - 2) * row;
            else cur ^= 1;
            const long next = t / every + 1;
            const int e = ops.reverse(src, ckpt_row(next), (int)(next * every - t < m ? next * every - t : m), every, (int)m, in, out);
            in = out;
            return e;
        };
        for (long hi = top; hi > 0;) {
            if (every <= most) {
                const long span = most / every * every, t = (hi - 1) / span * span;
                if (int e = pass(ckpt_row(t / every), t, hi - t)) return e;
                hi = t;
                continue;
            }
            const long t0 = (hi - 1) / every * every, parts = ceil_div(hi - t0, most), size = ceil_div(hi - t0, parts);
            // the states at which the parts after the first one start: rows 0, 1, ... of work
            const long group = kForwardSteps / size;
            for (long k = 0; k + 1 < parts; k += group) {
                const long g = parts - 1 - k < group ? parts - 1 - k : group;
                const char *src = k == 0 ? ckpt_row(t0 / every) : work + (size_t)(k - 1) * row;
                if (int e = ops.forward(src, work + (size_t)k * row, size, size, (int)(g * size), nullptr, true)) return e;
            }
            for (long k = parts - 1; k >= 0; --k) {
                const char *src = k == 0 ? ckpt_row(t0 / every) : work + (size_t)(k - 1) * row;
                const long t = t0 + k * size;
                if (t >= hi) return -1;
                if (int e = pass(src, t, hi - t)) return e;
                hi = t;
            }
        }
        return 0;
    }
};

}  // namespace sadj
