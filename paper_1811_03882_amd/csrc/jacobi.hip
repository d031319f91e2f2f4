// Jacobi iteration for the Laplace equation (second workload of the paper's
// transfer rule: the sample program solved with Jacobi's method, Sec. 4).
//
// One iteration: every interior point of the [n][m] FP64 grid becomes the
// average of its four neighbours from the previous iterate, summed in the
// order up + down + left + right (contraction off, so the result is the
// same in every rounding as the plain definition); the boundary stays fixed.
// HBM-bound: each iteration reads one grid and writes one.  A thread owns a
// column segment of STRIP rows, keeps the vertical neighbours in registers
// and reads the horizontal ones through the L1, so every element leaves HBM
// about once per iteration.  The largest change of the iteration is reduced
// per wave and folded into one global maximum (non-negative doubles order
// like their bit patterns).
#include "dn_kernels.h"

#pragma clang fp contract(off)

namespace dnk {

// one iteration per launch (the per-iteration transfer mode, and grids too tall
// or too wide for the tiled kernel's launch below)
constexpr int JAC_BX = 64, JAC_BY = 4, JAC_STRIP = 8;

__global__ void __launch_bounds__(JAC_BX * JAC_BY) jacobi_step(const double *__restrict__ u, double *__restrict__ v,
                                                              int n, int m, unsigned long long *max_change)
{
    const int j = blockIdx.x * JAC_BX + (threadIdx.x % JAC_BX);
    const int i0 = (blockIdx.y * JAC_BY + threadIdx.x / JAC_BX) * JAC_STRIP;
    double ch = 0.0;
    if (j < m && i0 < n) {
        const bool edge_col = j == 0 || j == m - 1;
        double up = i0 > 0 ? u[(size_t)(i0 - 1) * m + j] : 0.0;
        double mid = u[(size_t)i0 * m + j];
        for (int r = 0; r < JAC_STRIP; ++r) {
            const int i = i0 + r;
            if (i >= n) break;
            const double down = i + 1 < n ? u[(size_t)(i + 1) * m + j] : 0.0;
            double out = mid;
            if (!edge_col && i > 0 && i < n - 1) {
                const double left = u[(size_t)i * m + j - 1], right = u[(size_t)i * m + j + 1];
                double s = up + down;
                s = s + left;
                s = s + right;
                out = 0.25 * s;
                ch = fmax(ch, fabs(out - mid));
            }
            v[(size_t)i * m + j] = out;
            up = mid;
            mid = down;
        }
    }
    if (max_change) {
        // wave maximum, then one atomic per wave
        for (int off = 32; off > 0; off >>= 1) ch = fmax(ch, __shfl_xor(ch, off));
        if ((threadIdx.x & 63) == 0) atomicMax(max_change, (unsigned long long)__double_as_longlong(ch));
    }
}

__global__ void jacobi_zero(unsigned long long *p) { *p = 0ull; }

// ---------------------------------------------------------------- several iterations per launch
// One launch per iteration is bound by the launch itself on small grids (7.7 us
// per iteration at 1000x1500, whose 24 MB take 5 us from HBM and less from
// cache) and by memory on large ones.  Here a workgroup loads a patch of 8*R x
// 128 points once, runs t iterations on it in registers and writes back the
// part whose values do not depend on anything outside the patch: all but a rim
// of t points on the sides that have grid beyond them.  Neighbouring patches
// overlap by that rim, so the extra work is the price of t - 1 passes over
// memory and t - 1 launches.
//   * A wave owns R rows of the patch, a lane two neighbouring columns:
//     vertical neighbours are registers, horizontal ones the lane's other
//     column or one whole-wave DPP shift, and only the first and last row of a
//     wave go through LDS (two buffers by turns: one barrier per iteration).
//   * Every value is formed by the same four operations in the same order as in
//     jacobi_step, so the result has the same bits for any R, t and tiling.
// Bound by instruction issue and the launches.  Measured, 64 iterations of
// 1000x1500: 491 us one launch per iteration, 92 us as four launches of 16 on
// 96-row patches.

template <int CTRL> __device__ __forceinline__ double wave_shift(double v)
{
    const unsigned long long b = (unsigned long long)__double_as_longlong(v);
    const unsigned lo = __builtin_amdgcn_update_dpp(0, (int)(unsigned)b, CTRL, 0xf, 0xf, true);
    const unsigned hi = __builtin_amdgcn_update_dpp(0, (int)(unsigned)(b >> 32), CTRL, 0xf, 0xf, true);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// The wave's place in its patch and what stays fixed there.
struct JacobiWave {
    int wave, lane, i0, n;
    bool fixed0, fixed1;  // the lane's columns lie on or outside the grid's boundary
    bool out0, out1;      // the lane's columns are written by this workgroup
    int ilo, ihi;         // and rows [ilo, ihi)
};

// One iteration on the wave's rows c[r][0..1].  EDGE: the patch touches the
// grid's boundary (fixed values) or reaches past it.  WANT: returns the
// largest change among the points this workgroup writes.
template <int R, bool EDGE, bool WANT>
__device__ __forceinline__ double jacobi_once(double (&c)[R][2], double (*b)[JT_W][JT_COLS], const JacobiWave &w)
{
    double ch = 0.0;
    *reinterpret_cast<double2 *>(&b[0][w.wave][2 * w.lane]) = make_double2(c[0][0], c[0][1]);
    *reinterpret_cast<double2 *>(&b[1][w.wave][2 * w.lane]) = make_double2(c[R - 1][0], c[R - 1][1]);
    __syncthreads();
    // past the patch's first and last wave: any value, it reaches only the rim
    const double2 up = *reinterpret_cast<const double2 *>(&b[1][max(w.wave - 1, 0)][2 * w.lane]);
    const double2 dn = *reinterpret_cast<const double2 *>(&b[0][min(w.wave + 1, JT_W - 1)][2 * w.lane]);
    double u0 = up.x, u1 = up.y;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double m0 = c[r][0], m1 = c[r][1];
        const double d0 = r + 1 < R ? c[r + 1][0] : dn.x, d1 = r + 1 < R ? c[r + 1][1] : dn.y;
        const double l0 = wave_shift<0x138>(m1);  // lane - 1's second column
        const double r1 = wave_shift<0x130>(m0);  // lane + 1's first column
        double s0 = u0 + d0, s1 = u1 + d1;
        s0 = s0 + l0;
        s1 = s1 + m0;
        s0 = s0 + m1;
        s1 = s1 + r1;
        s0 = 0.25 * s0;
        s1 = 0.25 * s1;
        if (EDGE) {
            const bool row = w.i0 + r <= 0 || w.i0 + r >= w.n - 1;
            s0 = row || w.fixed0 ? m0 : s0;
            s1 = row || w.fixed1 ? m1 : s1;
        }
        if (WANT && w.i0 + r >= w.ilo && w.i0 + r < w.ihi) {
            if (w.out0) ch = fmax(ch, fabs(s0 - m0));
            if (w.out1) ch = fmax(ch, fabs(s1 - m1));
        }
        c[r][0] = s0;
        c[r][1] = s1;
        u0 = m0;
        u1 = m1;
    }
    return ch;
}

// hx, hy: rim of the patch on its vertical / horizontal sides (0: the grid
// fits in that direction).  u == v only with a single workgroup.
template <int R>
__global__ void __launch_bounds__(64 * JT_W, 2) jacobi_tile(const double *u, double *v, int n, int m, int t, int hx, int hy,
                                                            unsigned long long *max_change)
{
    constexpr int ROWS = R * JT_W;
    __shared__ double rim[2][2][JT_W][JT_COLS];
    JacobiWave w;
    w.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    w.lane = threadIdx.x & 63;
    w.n = n;
    const int j0 = (int)blockIdx.x * (JT_COLS - 2 * hx) - hx, ib = (int)blockIdx.y * (ROWS - 2 * hy) - hy;
    const int j = j0 + 2 * w.lane;
    w.i0 = ib + w.wave * R;
    // points outside the grid only ever meet fixed ones: load any point there
    double c[R][2];
    const int ja = min(max(j, 0), m - 1), jb = min(max(j + 1, 0), m - 1);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const double *p = u + (size_t)min(max(w.i0 + r, 0), n - 1) * m;
        c[r][0] = p[ja];
        c[r][1] = p[jb];
    }
    // what this workgroup writes: the patch without its rim
    w.ilo = max(0, ib + hy);
    w.ihi = min(n, ib + ROWS - hy);
    const int jlo = max(0, j0 + hx), jhi = min(m, j0 + JT_COLS - hx);
    w.out0 = j >= jlo && j < jhi;
    w.out1 = j + 1 >= jlo && j + 1 < jhi;
    w.fixed0 = j <= 0 || j >= m - 1;
    w.fixed1 = j + 1 <= 0 || j + 1 >= m - 1;
    const bool edge = ib <= 0 || ib + ROWS >= n || j0 <= 0 || j0 + JT_COLS >= m;
    double ch = 0.0;
    const int plain = max_change ? t - 1 : t;
    if (edge) {
        for (int it = 0; it < plain; ++it) jacobi_once<R, true, false>(c, rim[it & 1], w);
    } else {
        for (int it = 0; it < plain; ++it) jacobi_once<R, false, false>(c, rim[it & 1], w);
    }
    if (max_change) ch = jacobi_once<R, true, true>(c, rim[plain & 1], w);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        if (w.i0 + r < w.ilo || w.i0 + r >= w.ihi) continue;
        double *q = v + (size_t)(w.i0 + r) * m + j;
        if (w.out0) q[0] = c[r][0];
        if (w.out1) q[1] = c[r][1];
    }
    if (max_change) {
        // one atomic per workgroup: they queue up at the one address, about 10 ns
        // each.  One per wave made flat grids, which have more waves here than on
        // the kernel of one iteration, slower than on that kernel (3 x 1000000, 16
        // iterations: 899 us against 869; 195 with one per workgroup)
        __shared__ double most[JT_W];
        for (int off = 32; off > 0; off >>= 1) ch = fmax(ch, __shfl_xor(ch, off));
        if (w.lane == 0) most[w.wave] = ch;
        __syncthreads();
        if (threadIdx.x == 0) {
            for (int k = 1; k < JT_W; ++k) ch = fmax(ch, most[k]);
            if (ch > 0.0) atomicMax(max_change, (unsigned long long)__double_as_longlong(ch));
        }
    }
}

hipError_t launch_jacobi_step(const double *u, double *v, int n, int m, unsigned long long *max_change, hipStream_t s)
{
    if (max_change) hipLaunchKernelGGL(jacobi_zero, dim3(1), dim3(1), 0, s, max_change);
    dim3 grid((m + JAC_BX - 1) / JAC_BX, (n + JAC_BY * JAC_STRIP - 1) / (JAC_BY * JAC_STRIP));
    hipLaunchKernelGGL(jacobi_step, grid, dim3(JAC_BX * JAC_BY), 0, s, u, v, n, m, max_change);
    return hipGetLastError();
}

template <int R>
static hipError_t go_jacobi(const double *u, double *v, int n, int m, int t, unsigned long long *max_change, hipStream_t s)
{
    constexpr int ROWS = R * JT_W;
    const int hx = m <= JT_COLS ? 0 : t, hy = n <= ROWS ? 0 : t;
    if (t < 1 || 2 * hx >= JT_COLS || 2 * hy >= ROWS) return hipErrorInvalidValue;
    const long gx = hx ? ((long)m + JT_COLS - 2 * hx - 1) / (JT_COLS - 2 * hx) : 1;
    const long gy = hy ? ((long)n + ROWS - 2 * hy - 1) / (ROWS - 2 * hy) : 1;
    if (gy > JT_MAX_Y || gx > JT_MAX_X || (u == v && gx * gy > 1)) return hipErrorInvalidValue;
    if (max_change) hipLaunchKernelGGL(jacobi_zero, dim3(1), dim3(1), 0, s, max_change);
    hipLaunchKernelGGL(jacobi_tile<R>, dim3((unsigned)gx, (unsigned)gy), dim3(64 * JT_W), 0, s, u, v, n, m, t, hx, hy, max_change);
    return hipGetLastError();
}

hipError_t launch_jacobi_tile(int rows, const double *u, double *v, int n, int m, int t, unsigned long long *max_change, hipStream_t s)
{
    switch (rows) {
    case 4: return go_jacobi<4>(u, v, n, m, t, max_change, s);
    case 8: return go_jacobi<8>(u, v, n, m, t, max_change, s);
    case 12: return go_jacobi<12>(u, v, n, m, t, max_change, s);
    case 16: return go_jacobi<16>(u, v, n, m, t, max_change, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace dnk
