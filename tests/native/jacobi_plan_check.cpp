// Host driver of tests/test_jacobi_plan_cpu.py: for every grid and iteration
// count, the launches of the plan (jacobi_plan.h) are ones that the tiled
// kernel's launch accepts and their iterations add up.

#include <climits>
#include <cstdio>
#include <vector>

#include "jacobi_plan.h"

using namespace dnk;

static long plans = 0;

static bool check(int n, int m, int iters)
{
    ++plans;
    const JacobiPlan p = jacobi_plan(n, m, iters);
    const int rows = p.rows * JT_W;
    bool ok = p.rows >= 4 && p.rows <= 16 && p.rows % 4 == 0 && p.launches >= 1 && p.launches <= iters;
    ok = ok && (!p.in_place || (n <= rows && m <= JT_COLS));
    int done = 0;
    for (int k = 0; ok && k < p.launches; ++k) {
        const int t = jacobi_share(p, iters, done, k);
        const int hx = m <= JT_COLS ? 0 : t, hy = n <= rows ? 0 : t;
        ok = t >= 1 && t <= iters - done && 2 * hx < JT_COLS && 2 * hy < rows;
        if (!ok) break;
        const long gx = hx ? ((long)m + JT_COLS - 2 * hx - 1) / (JT_COLS - 2 * hx) : 1;
        const long gy = hy ? ((long)n + rows - 2 * hy - 1) / (rows - 2 * hy) : 1;
        // HIP's limits: 65535 blocks down, fewer than 2^32 threads across
        ok = gy <= 65535 && gx * 64 * JT_W < (1L << 32) && (!p.in_place || gx * gy == 1);
        done += t;
        // the shares are equal from here on: the rest of a long run is like this one
        if (ok && k == 1000) {
            const int left = p.launches - k - 1;
            ok = left <= iters - done && (long)left * t >= iters - done;
            done = iters;
            break;
        }
    }
    ok = ok && done == iters;
    if (!ok) printf("%d x %d, %d iterations: rows %d, launches %d, in place %d; %d iterations dealt out\n", n, m, iters,
                    p.rows, p.launches, (int)p.in_place, done);
    return ok;
}

int main()
{
    std::vector<int> sides;
    for (long s = 1; s < 60000; s = s * 9 / 8 + 1) sides.push_back((int)s);
    for (int s : {32, 64, 96, 127, 128, 129, 130, 1000, 1500, 19900, 22100, 24000, 25200, 400000, (1 << 19) - 1}) sides.push_back(s);
    std::vector<int> iters;
    for (int i = 1; i <= 130; ++i) iters.push_back(i);
    for (int i : {255, 256, 257, 1000, 1001, 4095, 4096, 4097, 100001, INT_MAX - 4095, INT_MAX - 4094, INT_MAX - 1, INT_MAX}) iters.push_back(i);
    // the widest grids (up to 2^40 points)
    for (int n : {1, 2, 3, 33, 300})
        for (long m : {1L << 29, 1056964000L, 1056965000L, 1100000000L, (1L << 31) - 1})
            for (int i : iters)
                if (jacobi_tiled(n, (int)m) && !check(n, (int)m, i)) return 1;
    for (int n : sides)
        for (int m : sides)
            for (int i : iters)
                if (!check(n, m, i)) return 1;
    printf("ok %ld plans\n", plans);
    return 0;
}
