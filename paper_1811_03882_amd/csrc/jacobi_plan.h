// How dn_jacobi splits its iterations over launches of the tiled kernel
// (jacobi.hip).  Plain host C++.  Internal to the library.
#pragma once

namespace dnk {

constexpr int JT_W = 8, JT_COLS = 128;  // waves of a patch, its columns

struct JacobiPlan { int rows, launches; bool in_place; };

// Workgroups of a patch height and iterations per launch; 0 if the rim leaves
// nothing to write.
inline long jacobi_groups(int n, int m, int rows, int t)
{
    const int wx = m <= JT_COLS ? JT_COLS : JT_COLS - 2 * t, wy = n <= rows ? rows : rows - 2 * t;
    if (wx <= 0 || wy <= 0) return 0;
    return ((long)(m + wx - 1) / wx) * ((n + wy - 1) / wy);
}

// Limits of a launch: 65535 workgroups down, fewer than 2^32 threads across.
constexpr int JT_MAX_Y = 65535, JT_MAX_X = (1 << 23) - 1;
// Grids the tiled kernel takes with a rim of one: jacobi_plan() finds a plan.
inline bool jacobi_tiled(int n, int m) { return n < (1 << 19) && m <= (JT_COLS - 2) * JT_MAX_X; }

// Rows per wave and launches for `iters` iterations: the least launches x
// (launch + t x iteration) over patch heights and iterations per launch t.  The
// model ranks the choices: 6.5 us a launch with its loads and stores; an iteration
// 0.15 us of barrier and LDS latency and, per workgroup a CU runs at once, 96
// clocks of issue a row (two waves on each SIMD, 12 instructions for two columns).
// It leaves out what patches at the grid's edge do more, for which a launch waits:
// 1000x1500 at 64 iterations takes 92 us where it says 71, on the plan it
// chooses, 96-row patches and 16 iterations (256 workgroups).
// A grid that fits in one patch needs no rim and no partner buffer: one launch,
// in place (at most 4096 iterations each, so that a launch stays short).
inline JacobiPlan jacobi_plan(int n, int m, int iters)
{
    JacobiPlan best{0, 0, false};
    double cost = 1e300;
    for (int r = 4; r <= 16; r += 4) {
        const int rows = r * JT_W;
        if (n <= rows && m <= JT_COLS) return JacobiPlan{r, (iters - 1) / 4096 + 1, true};
        for (int t = 1; t <= 24 && t <= iters; ++t) {
            const long g = jacobi_groups(n, m, rows, t);
            if (g == 0) break;
            if (n > rows && (n - 1) / (rows - 2 * t) >= JT_MAX_Y) break;
            if (m > JT_COLS && (m - 1) / (JT_COLS - 2 * t) >= JT_MAX_X) break;
            // an even number of launches ends in the buffer it began in; an odd
            // one (a single launch, or one for each of an odd number of
            // iterations, where none is left for another) is followed by a copy
            long launches = ((long)iters + t - 1) / t;
            if (launches > 1 && launches < iters) launches += launches & 1;
            const double copy = launches == 1 ? 6.5 : (launches & 1) ? 6.5 + 3.2e-6 * n * m : 0.0;
            const double per_cu = (double)((g + 255) / 256);
            const double us = launches * (6.5 + (double)iters / launches * (0.15 + 0.0457 * r * per_cu)) + copy;
            if (us < cost) {
                cost = us;
                best = JacobiPlan{r, (int)launches, false};
            }
        }
    }
    return best;
}

// Iterations of launch k of the plan, `done` of `iters` before it: equal shares,
// the larger ones first.
inline int jacobi_share(const JacobiPlan &p, int iters, int done, int k)
{
    return (iters - done - 1) / (p.launches - k) + 1;
}

}  // namespace dnk
