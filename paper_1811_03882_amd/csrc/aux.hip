// Memory-bound kernels around the convolutions: FP64 batch-norm fold and
// weight packing (load time), input ingest and output egress (once per
// forward), standalone max pool and residual add (per-layer mode and the
// layers that cannot be fused), and the amax reduction used for FP8
// calibration.  All activations are NHWC with 16-byte padded channels; every
// kernel moves whole 16-byte segments where the layout allows it.
#include "dn_kernels.h"
#include "seg.h"

namespace dnk {

// ---------------------------------------------------------------- fold + pack
// One block per padded output channel.  FP64: scale = gamma / sqrt(var + eps),
// w' = w * scale, b' = (b - mean) * scale + beta (b' = b without BN).  The
// packed row is [k_pad] with k = (cb*R*S + r*S + s)*CB + ci, c = cb*CB + ci,
// CB = kblock_ch(dt, cin_p, R*S) (compact: k = r*16 + s*CP + c,
// CP = first_cp(cin)),
// zeros in every padding.
// Mode 2 packs the backward-data conv of a forward conv (stride 1 over the
// output gradient): here cout / cin are the forward conv's cin / cout, the
// raw array is the forward [cin][cout][R][S] one, and the packed weight is
// w'[co][c][r][s] = w[c][co][R-1-r][S-1-s] * scale[c] with the forward BN
// scale of channel c (FP64), bias 0.
// FP8 rows get scale s = max|w'| / 448 and store e4m3(w' / s).

template <int DT>
__global__ void __launch_bounds__(256) fold_pack(int mode, const double *w, const double *bias, const double *mean,
                                                 const double *var, const double *gamma, const double *beta,
                                                 double eps, int has_bn, int cout, int cin, int R, int S,
                                                 int cin_p, int k_pad, void *wout, float *bout, float *sout)
{
    const int co = blockIdx.x;
    const int RS = R * S;
    double sc = 1.0, bb = 0.0;
    if (co < cout && mode != 2) {
        if (has_bn) {
            sc = gamma[co] / sqrt(var[co] + eps);
            bb = (bias[co] - mean[co]) * sc + beta[co];
        } else {
            bb = bias[co];
        }
    }
    auto wval = [&](int k) -> double {
        int c, r, s;
        if (mode == 1) {  // k = r*16 + s*CP + c
            const int cp = first_cp(cin);
            r = k / 16;
            const int e = k - r * 16;
            s = e / cp;
            c = e - s * cp;
            if (co >= cout || r >= R || s >= S || c >= cin) return 0.0;
        } else {        // k = (cb*R*S + r*S + s)*CB + ci, c = cb*CB + ci
            const int CB = kblock_ch(DT, cin_p, RS);
            const int blk = k / CB, cb = blk / RS, tap = blk - cb * RS;
            c = cb * CB + (k - blk * CB);
            if (co >= cout || c >= cin) return 0.0;
            r = tap / S;
            s = tap - r * S;
        }
        if (mode == 2) {
            const double g = has_bn ? gamma[c] / sqrt(var[c] + eps) : 1.0;
            return w[(((size_t)c * cout + co) * R + (R - 1 - r)) * S + (S - 1 - s)] * g;
        }
        return w[(((size_t)co * cin + c) * R + r) * S + s] * sc;
    };
    double qs = 1.0;
    if (DT == FP8) {
        __shared__ double red[256];
        double mx = 0.0;
        for (int k = threadIdx.x; k < k_pad; k += blockDim.x) mx = fmax(mx, fabs(wval(k)));
        red[threadIdx.x] = mx;
        __syncthreads();
        for (int off = 128; off > 0; off >>= 1) {
            if ((int)threadIdx.x < off) red[threadIdx.x] = fmax(red[threadIdx.x], red[threadIdx.x + off]);
            __syncthreads();
        }
        qs = red[0] > 0.0 ? red[0] / 448.0 : 1.0;
    }
    for (int k = threadIdx.x; k < k_pad; k += blockDim.x) {
        const double v = wval(k);
        const size_t o = (size_t)co * k_pad + k;
        if (DT == F32) ((float *)wout)[o] = (float)v;
        else if (DT == BF16) ((uint16_t *)wout)[o] = f2bf((float)v);
        else ((uint8_t *)wout)[o] = (uint8_t)f2e4m3((float)(v / qs));
    }
    if (threadIdx.x == 0) {
        bout[co] = (float)bb;
        sout[co] = (float)qs;
    }
}

hipError_t launch_fold_pack(int dt, int mode, const double *w, const double *bias, const double *mean,
                            const double *var, const double *gamma, const double *beta, double eps,
                            int has_bn, int cout, int cin, int R, int S, int cin_p, int k_pad,
                            int cout_p, void *wout, float *bout, float *sout, hipStream_t s)
{
    dim3 g(cout_p), b(256);
    switch (dt) {
    case F32: hipLaunchKernelGGL(fold_pack<F32>, g, b, 0, s, mode, w, bias, mean, var, gamma, beta, eps, has_bn, cout, cin, R, S, cin_p, k_pad, wout, bout, sout); break;
    case BF16: hipLaunchKernelGGL(fold_pack<BF16>, g, b, 0, s, mode, w, bias, mean, var, gamma, beta, eps, has_bn, cout, cin, R, S, cin_p, k_pad, wout, bout, sout); break;
    case FP8: hipLaunchKernelGGL(fold_pack<FP8>, g, b, 0, s, mode, w, bias, mean, var, gamma, beta, eps, has_bn, cout, cin, R, S, cin_p, k_pad, wout, bout, sout); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- ingest
// NCHW FP32 -> NHWC storage type.  One thread per (pixel, 16-byte segment):
// consecutive threads read consecutive pixels of one channel plane.

// x8 set: the source is 8-bit pixels, value q / 255 (x unused).
template <int DT>
__global__ void __launch_bounds__(256) ingest(const float *x, const unsigned char *x8, int n, int c, int hw, int cp,
                                              float inv_scale, void *y)
{
    constexpr int E = Seg<DT>::N;
    const int nseg = cp / E;
    const size_t total = (size_t)n * hw * nseg;
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total) return;
    const int p = (int)(t % hw);
    const size_t rest = t / hw;
    const int sg = (int)(rest % nseg);
    const int img = (int)(rest / nseg);
    float f[E];
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int ch = sg * E + e;
        const size_t i = ((size_t)img * c + ch) * hw + p;
        f[e] = ch < c ? (x8 ? __fdiv_rn((float)x8[i], 255.0f) : x[i]) * inv_scale : 0.0f;
    }
    ((uint4 *)y)[((size_t)img * hw + p) * nseg + sg] = Seg<DT>::enc(f);
}

hipError_t launch_ingest(int dt, const float *x, int n, int c, int h, int w, int cp, float inv_scale,
                         void *y, hipStream_t s, const unsigned char *x8)
{
    const size_t total = (size_t)n * h * w * (cp / seg_el(dt));
    if (total == 0) return hipSuccess;
    dim3 g((unsigned)((total + 255) / 256)), b(256);
    switch (dt) {
    case F32: hipLaunchKernelGGL(ingest<F32>, g, b, 0, s, x, x8, n, c, h * w, cp, inv_scale, y); break;
    case BF16: hipLaunchKernelGGL(ingest<BF16>, g, b, 0, s, x, x8, n, c, h * w, cp, inv_scale, y); break;
    case FP8: hipLaunchKernelGGL(ingest<FP8>, g, b, 0, s, x, x8, n, c, h * w, cp, inv_scale, y); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- egress
// NHWC storage type -> NCHW FP32; thread per (pixel, segment), consecutive
// threads write consecutive pixels of a channel plane.  IT is the type of the
// thread index: 32-bit (a short division sequence) whenever the thread count
// fits, 64-bit otherwise.

template <int DT, typename IT>
__global__ void __launch_bounds__(256) egress(const void *x, int n, int c, int hw, int cp, float scale, float *y)
{
    constexpr int E = Seg<DT>::N;
    const int nseg = (c + E - 1) / E, cseg = cp / E;
    const IT total = (IT)n * hw * nseg;
    const IT t = (IT)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total) return;
    const int p = (int)(t % (IT)hw);
    const IT rest = t / (IT)hw;
    const int sg = (int)(rest % (IT)nseg);
    const int img = (int)(rest / (IT)nseg);
    float f[E];
    Seg<DT>::dec(((const uint4 *)x)[((size_t)img * hw + p) * cseg + sg], f);
#pragma unroll
    for (int e = 0; e < E; ++e) {
        const int ch = sg * E + e;
        if (ch < c) y[((size_t)img * c + ch) * hw + p] = f[e] * scale;
    }
}

hipError_t launch_egress(int dt, const void *x, int n, int c, int h, int w, int cp, float scale,
                         float *y, hipStream_t s)
{
    const size_t total = (size_t)n * h * w * ((c + seg_el(dt) - 1) / seg_el(dt));
    if (total == 0) return hipSuccess;
    dim3 g((unsigned)((total + 255) / 256)), b(256);
    const bool small = total + 256 < (1ull << 32);
#define DN_EGRESS(D)                                                                              \
    do {                                                                                          \
        if (small) hipLaunchKernelGGL((egress<D, unsigned>), g, b, 0, s, x, n, c, h * w, cp, scale, y); \
        else hipLaunchKernelGGL((egress<D, size_t>), g, b, 0, s, x, n, c, h * w, cp, scale, y);         \
    } while (0)
    switch (dt) {
    case F32: DN_EGRESS(F32); break;
    case BF16: DN_EGRESS(BF16); break;
    case FP8: DN_EGRESS(FP8); break;
    default: return hipErrorInvalidValue;
    }
#undef DN_EGRESS
    return hipGetLastError();
}

// ---------------------------------------------------------------- max pool
// -inf outside the input; window starts at i*stride - (size-1)/2.  Values are
// decoded, compared and re-encoded, which is exact (no new values appear).
// SZ = 2: windows of two, which start inside the input, with their four loads
// in flight together (a position past the edge reads the last one instead, a
// duplicate that changes no maximum).  Bound by the latency of a thread's
// loads: one after the other behind their edge tests, 64 x 13 x 13 x 512 BF16
// took 9.8 us at stride 1, with the four in flight 7.9 (22 MB: 4.3 us at the
// rate of a large copy).  SZ = 0: any size.

template <int DT, typename IT, int SZ>
__global__ void __launch_bounds__(256) maxpool(const void *x, void *y, int n, int h, int w, int cp, int size,
                                               int stride, int ho, int wo)
{
    constexpr int E = Seg<DT>::N;
    const int nseg = cp / E;
    const IT total = (IT)n * ho * wo * nseg;
    const IT t = (IT)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= total) return;
    const int sg = (int)(t % (IT)nseg);
    const size_t p = t / (IT)nseg;
    const int j = (int)((IT)p % (IT)wo);
    const IT q = (IT)p / (IT)wo;
    const int i = (int)(q % (IT)ho);
    const int img = (int)(q / (IT)ho);
    float m[E];
#pragma unroll
    for (int e = 0; e < E; ++e) m[e] = -INFINITY;
    if constexpr (SZ == 2) {
        const int y0 = i * stride, x0 = j * stride;
        const int dy = y0 + 1 < h ? w * nseg : 0, dx = x0 + 1 < w ? nseg : 0;
        const uint4 *px = (const uint4 *)x + (((size_t)img * h + y0) * w + x0) * nseg + sg;
        const uint4 r[4] = {px[0], px[dx], px[dy], px[dy + dx]};
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            float f[E];
            Seg<DT>::dec(r[k], f);
#pragma unroll
            for (int e = 0; e < E; ++e) m[e] = fmaxf(m[e], f[e]);
        }
        ((uint4 *)y)[p * nseg + sg] = Seg<DT>::enc(m);
        return;
    }
    const int off = (size - 1) / 2;
    for (int u = 0; u < size; ++u) {
        const int yy = i * stride - off + u;
        if (yy < 0 || yy >= h) continue;
        for (int v = 0; v < size; ++v) {
            const int xx = j * stride - off + v;
            if (xx < 0 || xx >= w) continue;
            float f[E];
            Seg<DT>::dec(((const uint4 *)x)[(((size_t)img * h + yy) * w + xx) * nseg + sg], f);
#pragma unroll
            for (int e = 0; e < E; ++e) m[e] = fmaxf(m[e], f[e]);
        }
    }
    ((uint4 *)y)[p * nseg + sg] = Seg<DT>::enc(m);
}

hipError_t launch_maxpool(int dt, const void *x, void *y, int n, int h, int w, int cp, int size,
                          int stride, int ho, int wo, hipStream_t s)
{
    const size_t total = (size_t)n * ho * wo * (cp / seg_el(dt));
    if (total == 0) return hipSuccess;
    dim3 g((unsigned)((total + 255) / 256)), b(256);
    const bool small = total + 256 < (1ull << 32);
    // the window's first element is inside the input, and its offsets fit an int
    const bool two = size == 2 && (ho - 1) * stride < h && (wo - 1) * stride < w && (size_t)w * cp < (1u << 30);
#define DN_MAXPOOL(D)                                                                                            \
    do {                                                                                                        \
        if (small && two) hipLaunchKernelGGL((maxpool<D, unsigned, 2>), g, b, 0, s, x, y, n, h, w, cp, size, stride, ho, wo); \
        else if (small) hipLaunchKernelGGL((maxpool<D, unsigned, 0>), g, b, 0, s, x, y, n, h, w, cp, size, stride, ho, wo); \
        else hipLaunchKernelGGL((maxpool<D, size_t, 0>), g, b, 0, s, x, y, n, h, w, cp, size, stride, ho, wo);   \
    } while (0)
    switch (dt) {
    case F32: DN_MAXPOOL(F32); break;
    case BF16: DN_MAXPOOL(BF16); break;
    case FP8: DN_MAXPOOL(FP8); break;
    default: return hipErrorInvalidValue;
    }
#undef DN_MAXPOOL
    return hipGetLastError();
}

// ---------------------------------------------------------------- residual add

template <int DT>
__global__ void __launch_bounds__(256) add_seg(const uint4 *a, float sa, const uint4 *b, float sb, uint4 *y,
                                               float inv_sy, size_t nseg)
{
    constexpr int E = Seg<DT>::N;
    const size_t t = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nseg) return;
    float fa[E], fb[E];
    Seg<DT>::dec(a[t], fa);
    Seg<DT>::dec(b[t], fb);
#pragma unroll
    for (int e = 0; e < E; ++e) fa[e] = (fa[e] * sa + fb[e] * sb) * inv_sy;
    y[t] = Seg<DT>::enc(fa);
}

hipError_t launch_add(int dt, const void *a, float sa, const void *b, float sb, void *y, float inv_sy,
                      size_t count, hipStream_t s)
{
    const size_t nseg = count / seg_el(dt);
    if (nseg == 0) return hipSuccess;
    dim3 g((unsigned)((nseg + 255) / 256)), bl(256);
    const uint4 *A = (const uint4 *)a, *B = (const uint4 *)b;
    uint4 *Y = (uint4 *)y;
    switch (dt) {
    case F32: hipLaunchKernelGGL(add_seg<F32>, g, bl, 0, s, A, sa, B, sb, Y, inv_sy, nseg); break;
    case BF16: hipLaunchKernelGGL(add_seg<BF16>, g, bl, 0, s, A, sa, B, sb, Y, inv_sy, nseg); break;
    case FP8: hipLaunchKernelGGL(add_seg<FP8>, g, bl, 0, s, A, sa, B, sb, Y, inv_sy, nseg); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------- amax
// |x| >= 0, so the IEEE bit pattern orders like an unsigned integer and the
// block maxima combine with a 32-bit atomic max.

__global__ void __launch_bounds__(256) amax_kernel(const float *x, size_t n, unsigned *out)
{
    __shared__ float red[256];
    float m = 0.0f;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        m = fmaxf(m, fabsf(x[i]));
    red[threadIdx.x] = m;
    __syncthreads();
    for (int off = 128; off > 0; off >>= 1) {
        if ((int)threadIdx.x < off) red[threadIdx.x] = fmaxf(red[threadIdx.x], red[threadIdx.x + off]);
        __syncthreads();
    }
    if (threadIdx.x == 0) atomicMax(out, __float_as_uint(red[0]));
}

hipError_t launch_amax(const float *x, size_t count, float *out, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    size_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(amax_kernel, dim3((unsigned)blocks), dim3(256), 0, s, x, count, (unsigned *)out);
    return hipGetLastError();
}

__global__ void zero_kernel(float *p, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0.0f;
}

hipError_t launch_zero_f32(float *p, size_t count, hipStream_t s)
{
    if (count == 0) return hipSuccess;
    hipLaunchKernelGGL(zero_kernel, dim3((unsigned)((count + 255) / 256)), dim3(256), 0, s, p, count);
    return hipGetLastError();
}

// ---------------------------------------------------------------- MFMA peak probe
// Measurement only: every wave keeps eight independent accumulator chains of
// one MFMA instruction busy (no memory traffic), so the achieved rate is the
// matrix-core throughput at the clock the chip actually runs.  The chains are
// written as one asm block so that the compiler cannot insert copies between
// dependent instructions; each accumulator is reused only after seven others.
typedef float pf4 __attribute__((ext_vector_type(4)));
typedef int pi8 __attribute__((ext_vector_type(8)));
typedef unsigned pu4 __attribute__((ext_vector_type(4)));

template <int DT>
__global__ void __launch_bounds__(256) mfma_peak_kernel(float *out, int iters)
{
    pf4 c0 = {0.f, 0.f, 0.f, 0.f}, c1 = c0, c2 = c0, c3 = c0, c4 = c0, c5 = c0, c6 = c0, c7 = c0;
    const unsigned v = 0x3c003c00u + threadIdx.x;  // small finite operands
    for (int it = 0; it < iters; ++it) {
        if constexpr (DT == BF16) {
            const pu4 a = {v, v + 1, v + 2, v + 3};
            asm volatile(
                "v_mfma_f32_16x16x32_bf16 %0, %8, %8, %0\n\t"
                "v_mfma_f32_16x16x32_bf16 %1, %8, %8, %1\n\t"
                "v_mfma_f32_16x16x32_bf16 %2, %8, %8, %2\n\t"
                "v_mfma_f32_16x16x32_bf16 %3, %8, %8, %3\n\t"
                "v_mfma_f32_16x16x32_bf16 %4, %8, %8, %4\n\t"
                "v_mfma_f32_16x16x32_bf16 %5, %8, %8, %5\n\t"
                "v_mfma_f32_16x16x32_bf16 %6, %8, %8, %6\n\t"
                "v_mfma_f32_16x16x32_bf16 %7, %8, %8, %7"
                : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3), "+v"(c4), "+v"(c5), "+v"(c6), "+v"(c7)
                : "v"(a));
        } else if constexpr (DT == FP8) {
            const pi8 a = {(int)v, (int)v, (int)v, (int)v, (int)v, (int)v, (int)v, (int)v};
            asm volatile(
                "v_mfma_f32_16x16x128_f8f6f4 %0, %8, %8, %0\n\t"
                "v_mfma_f32_16x16x128_f8f6f4 %1, %8, %8, %1\n\t"
                "v_mfma_f32_16x16x128_f8f6f4 %2, %8, %8, %2\n\t"
                "v_mfma_f32_16x16x128_f8f6f4 %3, %8, %8, %3\n\t"
                "v_mfma_f32_16x16x128_f8f6f4 %4, %8, %8, %4\n\t"
                "v_mfma_f32_16x16x128_f8f6f4 %5, %8, %8, %5\n\t"
                "v_mfma_f32_16x16x128_f8f6f4 %6, %8, %8, %6\n\t"
                "v_mfma_f32_16x16x128_f8f6f4 %7, %8, %8, %7"
                : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3), "+v"(c4), "+v"(c5), "+v"(c6), "+v"(c7)
                : "v"(a));
        } else {
            const float a = __uint_as_float(0x3f800000u + threadIdx.x);
            asm volatile(
                "v_mfma_f32_16x16x4_f32 %0, %8, %8, %0\n\t"
                "v_mfma_f32_16x16x4_f32 %1, %8, %8, %1\n\t"
                "v_mfma_f32_16x16x4_f32 %2, %8, %8, %2\n\t"
                "v_mfma_f32_16x16x4_f32 %3, %8, %8, %3\n\t"
                "v_mfma_f32_16x16x4_f32 %4, %8, %8, %4\n\t"
                "v_mfma_f32_16x16x4_f32 %5, %8, %8, %5\n\t"
                "v_mfma_f32_16x16x4_f32 %6, %8, %8, %6\n\t"
                "v_mfma_f32_16x16x4_f32 %7, %8, %8, %7"
                : "+v"(c0), "+v"(c1), "+v"(c2), "+v"(c3), "+v"(c4), "+v"(c5), "+v"(c6), "+v"(c7)
                : "v"(a));
        }
    }
    const float r = c0[0] + c1[1] + c2[2] + c3[3] + c4[0] + c5[1] + c6[2] + c7[3];
    out[(size_t)blockIdx.x * blockDim.x + threadIdx.x] = r;
}

double mfma_peak_flops_per_launch(int dt, int blocks, int iters)
{
    const double per = dt == FP8 ? 16.0 * 16 * 128 * 2 : dt == BF16 ? 16.0 * 16 * 32 * 2 : 16.0 * 16 * 4 * 2;
    return (double)blocks * 4 /* waves */ * iters * 8 /* MFMAs per iteration */ * per;
}

hipError_t launch_mfma_peak(int dt, float *out, int blocks, int iters, hipStream_t s)
{
    switch (dt) {
    case F32: hipLaunchKernelGGL(mfma_peak_kernel<F32>, dim3(blocks), dim3(256), 0, s, out, iters); break;
    case BF16: hipLaunchKernelGGL(mfma_peak_kernel<BF16>, dim3(blocks), dim3(256), 0, s, out, iters); break;
    case FP8: hipLaunchKernelGGL(mfma_peak_kernel<FP8>, dim3(blocks), dim3(256), 0, s, out, iters); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace dnk
