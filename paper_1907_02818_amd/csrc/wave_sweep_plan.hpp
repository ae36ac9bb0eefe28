// Order of launches of a reverse sweep of wave steps, some of which share a pass over the data.  Host code without
// any device call, so that the order can be replayed on a CPU.
#pragma once

namespace sadj {

// Order of launches of a reverse sweep of wave steps that may use a fourth array.
// Buffers 0..2 are the caller's lam arrays, 3 is the work array.  A state is the pair (A, B) of
// buffers that hold lam^{k+1} and lam^k.  A single step updates B in place and assigns -A m to
// a buffer F outside {A, B}: (A, B) -> (B, F).  A pass over two or three steps writes both results to the
// two buffers outside {A, B}: (A, B) -> (F, G).  After the first step (which accumulates into
// lam2 and is always single) the state is (1, 2); the sweep must end in (n%3, (n+1)%3).  The
// body alternates passes of `most` steps (1,2) -> (0,3) -> (1,2) ...; the last few steps are chosen by
// exhaustive dynamic programming so that the end state is met with as few launches as possible
// (every launch moves five words per cell, however many steps it takes).
struct WaveStepLaunch { int steps, a, b, o0, o1; };   // single: o0 = F;  pass: o0 <- lam^{k+1-steps}, o1 <- lam^{k-steps}

constexpr int kTailMax = 12;

struct WaveSweepPlan {
    bool plain = true;                 // single steps rotating the caller's three buffers, work unused
    long body = 0;                     // else: passes alternating (1,2) -> (0,3) -> (1,2) ..., then the tail
    int tail_len = 0;
    WaveStepLaunch tail[kTailMax];
};

inline int state_id(int a, int b) { return a * 4 + b; }

// Launches for steps 1 .. nsteps-1 (step 0 is not part of the plan).
inline WaveSweepPlan plan_wave_sweep(long nsteps, int most)
{
    WaveSweepPlan plan;
    const long m = nsteps - 1;
    if (m < 2) return plan;
    const int ta = (int)(nsteps % 3), tb = (int)((nsteps + 1) % 3);
    const int tmax = (int)(m < kTailMax ? m : kTailMax);
    // best[t][state]: fewest launches on a way from state to the target in exactly t steps, none: kNone
    constexpr int kNone = 1000;
    int best[kTailMax + 1][16], choice[kTailMax + 1][16][3];
    for (int t = 0; t <= tmax; ++t)
        for (int s = 0; s < 16; ++s) best[t][s] = kNone;
    best[0][state_id(ta, tb)] = 0;
    for (int t = 1; t <= tmax; ++t)
        for (int a = 0; a < 4; ++a)
            for (int b = 0; b < 4; ++b) {
                if (a == b) continue;
                int fr[2], nf = 0;
                for (int f = 0; f < 4; ++f)
                    if (f != a && f != b) fr[nf++] = f;
                int &bst = best[t][state_id(a, b)];
                int *ch = choice[t][state_id(a, b)];
                for (int i = 0; i < 2; ++i) {
                    const int v = best[t - 1][state_id(b, fr[i])] + 1;
                    if (v < bst) { bst = v; ch[0] = 1; ch[1] = fr[i]; ch[2] = -1; }
                    for (int k = 2; k <= most && k <= t; ++k) {
                        const int w = best[t - k][state_id(fr[i], fr[1 - i])] + 1;
                        if (w < bst) { bst = w; ch[0] = k; ch[1] = fr[i]; ch[2] = fr[1 - i]; }
                    }
                }
            }
    auto body_state = [](long passes, int &a, int &b) { if (passes % 2 == 0) { a = 1; b = 2; } else { a = 0; b = 3; } };
    long total = -1;
    int t = 0, a = 1, b = 2;
    for (long q = m / most; q >= 0 && m - most * q <= tmax; --q) {
        body_state(q, a, b);
        const int launches = best[m - most * q][state_id(a, b)];
        if (launches < kNone && (total < 0 || q + launches < total)) { total = q + launches; plan.body = q; }
    }
    if (total < 0) return plan;        // plain stays set: single steps over three buffers
    plan.plain = false;
    t = (int)(m - most * plan.body);
    body_state(plan.body, a, b);
    while (t > 0) {
        const int *ch = choice[t][state_id(a, b)];
        plan.tail[plan.tail_len++] = {ch[0], a, b, ch[1], ch[2]};
        if (ch[0] == 1) { a = b; b = ch[1]; }
        else            { a = ch[1]; b = ch[2]; }
        t -= ch[0];
    }
    return plan;
}

}  // namespace sadj
