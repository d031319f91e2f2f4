// Device code shared by the convolution kernels (conv.hip, conv_pipe.hip):
// storage conversions, the MFMA step, tile order, epilogues and the global ->
// LDS transfer.  Internal to the library.
#pragma once

#include "dn_kernels.h"

namespace dnk {

typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f16v __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef int i32x8 __attribute__((ext_vector_type(8)));

// ---------------------------------------------------------------- conversions

__device__ __forceinline__ uint16_t f2bf(float f)
{
    return __builtin_bit_cast(uint16_t, (__bf16)f);  // v_cvt_pk_bf16_f32: round to nearest even
}
__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }
__device__ __forceinline__ uint8_t f2e4m3(float f)
{
    f = fminf(fmaxf(f, -448.0f), 448.0f);  // saturate
    return (uint8_t)(__builtin_amdgcn_cvt_pk_fp8_f32(f, f, 0, false) & 0xFF);
}
__device__ __forceinline__ float e4m32f(uint32_t b) { return __builtin_amdgcn_cvt_f32_fp8((int)b, 0); }

template <int DT> __device__ __forceinline__ float load_el(const void *p, size_t i)
{
    if constexpr (DT == F32) return ((const float *)p)[i];
    else if constexpr (DT == BF16) return bf2f(((const uint16_t *)p)[i]);
    else return e4m32f(((const uint8_t *)p)[i]);
}
template <int DT> __device__ __forceinline__ void store_el(void *p, size_t i, float v)
{
    if constexpr (DT == F32) ((float *)p)[i] = v;
    else if constexpr (DT == BF16) ((uint16_t *)p)[i] = f2bf(v);
    else ((uint8_t *)p)[i] = f2e4m3(v);
}
// four consecutive elements (i a multiple of 4), storage type -> FP32, one load
template <int DT> __device__ __forceinline__ void load4(const void *p, size_t i, float *v)
{
    if constexpr (DT == F32) {
        const float4 t = *reinterpret_cast<const float4 *>((const float *)p + i);
        v[0] = t.x; v[1] = t.y; v[2] = t.z; v[3] = t.w;
    } else if constexpr (DT == BF16) {
        const uint2 t = *reinterpret_cast<const uint2 *>((const uint16_t *)p + i);
        v[0] = bf2f((uint16_t)(t.x & 0xFFFFu)); v[1] = bf2f((uint16_t)(t.x >> 16));
        v[2] = bf2f((uint16_t)(t.y & 0xFFFFu)); v[3] = bf2f((uint16_t)(t.y >> 16));
    } else {
        const unsigned t = *reinterpret_cast<const unsigned *>((const uint8_t *)p + i);
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = e4m32f((t >> (8 * j)) & 0xFFu);
    }
}
// four consecutive channels, FP32 values -> storage type, one store
template <int DT> __device__ __forceinline__ void store4(void *y, size_t idx, const float *v)
{
    if constexpr (DT == F32) {
        *reinterpret_cast<float4 *>((float *)y + idx) = make_float4(v[0], v[1], v[2], v[3]);
    } else if constexpr (DT == BF16) {
        *reinterpret_cast<uint2 *>((uint16_t *)y + idx) =
            make_uint2((unsigned)f2bf(v[0]) | ((unsigned)f2bf(v[1]) << 16), (unsigned)f2bf(v[2]) | ((unsigned)f2bf(v[3]) << 16));
    } else {
        *reinterpret_cast<unsigned *>((uint8_t *)y + idx) = (unsigned)f2e4m3(v[0]) | ((unsigned)f2e4m3(v[1]) << 8) |
                                                            ((unsigned)f2e4m3(v[2]) << 16) | ((unsigned)f2e4m3(v[3]) << 24);
    }
}

// ---------------------------------------------------------------- MFMA step

template <int DT> struct Tr;
// SPL: 16-byte segments per lane per MFMA K-step; KSPT: K-steps per 128-byte K-tile.
template <> struct Tr<F32> { static constexpr int SPL = 1, KSPT = 2; };
template <> struct Tr<BF16> { static constexpr int SPL = 1, KSPT = 2; };
template <> struct Tr<FP8> { static constexpr int SPL = 2, KSPT = 1; };

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

template <int DT> __device__ __forceinline__ void mma(f4 &acc, const u32x4_t *a, const u32x4_t *b)
{
    if constexpr (DT == F32) {
        const float af[4] = {__uint_as_float(a[0].x), __uint_as_float(a[0].y), __uint_as_float(a[0].z), __uint_as_float(a[0].w)};
        const float bf[4] = {__uint_as_float(b[0].x), __uint_as_float(b[0].y), __uint_as_float(b[0].z), __uint_as_float(b[0].w)};
#pragma unroll
        for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_16x16x4f32(af[j], bf[j], acc, 0, 0, 0);
    } else if constexpr (DT == BF16) {
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a[0]), __builtin_bit_cast(bf16x8, b[0]), acc, 0, 0, 0);
    } else {
        const i32x8 av = {(int)a[0].x, (int)a[0].y, (int)a[0].z, (int)a[0].w, (int)a[1].x, (int)a[1].y, (int)a[1].z, (int)a[1].w};
        const i32x8 bv = {(int)b[0].x, (int)b[0].y, (int)b[0].z, (int)b[0].w, (int)b[1].x, (int)b[1].y, (int)b[1].z, (int)b[1].w};
        // format 0 = e4m3 for both operands, no block scaling
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(av, bv, acc, 0, 0, 0, 0, 0, 0);
    }
}

// Blocks are dealt to the 8 XCDs round-robin; renumber them so that each XCD
// receives a contiguous run of tiles (neighbouring tiles share A rows / B
// columns in that XCD's L2).
__device__ __forceinline__ int xcd_remap(int bid, int G)
{
    const int per = (G + 7) >> 3;
    const int xcd = bid & 7, loc = bid >> 3;
    const int tall = G - (per - 1) * 8;
    return xcd < tall ? xcd * per + loc : tall * per + (xcd - tall) * (per - 1) + loc;
}

// Logical tile id -> (M tile, N tile).  N tiles are taken in groups of four;
// within a group the id runs over (M tile, N tile in group), N fastest.  The
// run of ids one XCD receives is then a block of about 8 M tiles x 4 N tiles
// rather than 4 x 8 when N has 8 tiles, which balances the input rows and
// weight columns its L2 has to hold.
__device__ __forceinline__ void tile_mn(int logical, int mt, int ntn, int &mi, int &ni)
{
    constexpr int GN = 4;
    const int ngf = ntn / GN;            // complete groups
    const int gtiles = mt * GN;
    if (logical < ngf * gtiles) {
        const int g = logical / gtiles, r = logical - g * gtiles;
        mi = r / GN;
        ni = g * GN + (r - (r / GN) * GN);
    } else {
        const int w = ntn - ngf * GN, r = logical - ngf * gtiles;
        mi = r / w;
        ni = ngf * GN + (r - (r / w) * w);
    }
}

// Leaky: v for v > 0, else v * slope.  For 0 <= slope <= 1 that is exactly
// max(v, v * slope) (signed zeros and NaN included), two instructions.
__device__ __forceinline__ float activate(float v, int act, float slope)
{
    if (act != 1) return v;
    if (slope >= 0.0f && slope <= 1.0f) return fmaxf(v, v * slope);
    return v > 0.0f ? v : v * slope;
}

// The same function as one select: with lin_slope = slope for leaky and 1 for
// linear, v > 0 ? v : v * lin_slope equals activate(v, act, slope) bit for bit
// (for any slope; signed zeros and NaN included), without a branch on act.
__device__ __forceinline__ float act_slope(int act, float slope) { return act == 1 ? slope : 1.0f; }
__device__ __forceinline__ float activate_sel(float v, float lin_slope) { return v > 0.0f ? v : v * lin_slope; }

// The value an output takes once stored (rounded to the storage type).
template <int DT> __device__ __forceinline__ float stored_value(float v)
{
    if constexpr (DT == F32) return v;
    else if constexpr (DT == BF16) return bf2f(f2bf(v));
    else return e4m32f(f2e4m3(v));
}

// Index (2*dy + dx) of the first maximal stored output of a 2x2 window whose
// accumulators are acc[0..3] in row-major window order: the branch the
// max-pool gradient follows.
// The output is activate(acc * scl + bias) * post, as in the caller's epilogue:
// monotone in acc, so the largest stored value is the stored value of the
// largest accumulator, and the first element that reaches it is looked for
// among three.  A NaN is never larger than anything, and stays the choice where
// it comes first.
template <int DT> __device__ __forceinline__ unsigned char window_argmax(const float *acc, float scl, float bias,
                                                                        int act, float slope, float post)
{
    const auto stored = [&](float v) { return stored_value<DT>(activate(v * scl + bias, act, slope) * post); };
    const float m = stored(fmaxf(fmaxf(acc[0], acc[1]), fmaxf(acc[2], acc[3])));
    const unsigned char tail = stored(acc[1]) == m ? 1 : stored(acc[2]) == m ? 2 : 3;
    return stored(acc[0]) < m ? tail : 0;
}

// ---------------------------------------------------------------- the kernel

// Global-memory accesses go through explicit address-space-1 pointers so that
// the compiler emits global (not flat) loads: their completion is tracked by
// vmcnt alone and the LDS traffic of the current K-tile is not serialised
// behind the prefetch of the next one.
#define GLOBAL __attribute__((address_space(1)))
typedef u32x4_t u32x4;

__device__ __forceinline__ u32x4 gload16(const void *base, size_t byte_off)
{
    return *(const GLOBAL u32x4 *)((const GLOBAL char *)base + byte_off);
}

// Epilogue shared by the implicit-GEMM kernels.  MFMA 16x16 output layout:
// lane holds column (lane & 15) and rows 4*(lane >> 4) + i, i = 0..3; rowb /
// colb are this lane's first row / column.  With split-K the raw FP32
// partial sums go to the scratch plane of this split instead; when the last
// split finishes the tile in the same launch (a.tile_count set) they are
// device-scope stores, written through to where every XCD reads them.
// acc[g][f] holds rows rowb + g*RSTR + (0..3) of column colb + f*CSTR (16x16
// blocks: RSTR = CSTR = 16; 32x32 blocks split into four row quads: RSTR = 8,
// CSTR = 32).  Every quad starts at a multiple of 4, so with a fused pool it is
// one 2x2 window.
template <int DT, int FM, int FN, int RSTR = 16, int CSTR = 16>
__device__ __forceinline__ void conv_epilogue(const ConvArgs &a, f4 (&acc)[FM][FN], int rowb, int colb)
{
    if (a.splits > 1) {
        float *P = a.partial + (size_t)blockIdx.z * a.M * a.cout_p;
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
            const int col = colb + fn * CSTR;
            if (col >= a.cout_p) continue;
#pragma unroll
            for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int m = rowb + fm * RSTR + i;
                    if (m >= a.M) continue;
                    float *q = P + (size_t)m * a.cout_p + col;
                    if (a.tile_count) __hip_atomic_store(q, acc[fm][fn][i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    else *q = acc[fm][fn][i];
                }
        }
        return;
    }
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        const int col = colb + fn * CSTR;
        if (col >= a.cout_p) continue;
        const float bias = a.bias[col];
        const float scl = (DT == FP8) ? a.wscale[col] * a.in_scale : 1.0f;
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
            const int mb = rowb + fm * RSTR;
            if (mb >= a.M) continue;
            if (a.pool) {
                // rows mb..mb+3 are one 2x2 window (M is a multiple of 4 here); pooling
                // the accumulators is exact: scale > 0, and bias, activation and
                // rounding are monotone
                const float mx = fmaxf(fmaxf(acc[fm][fn][0], acc[fm][fn][1]), fmaxf(acc[fm][fn][2], acc[fm][fn][3]));
                store_el<DT>(a.y, (size_t)(mb >> 2) * a.cout_p + col, activate(mx * scl + bias, a.act, a.slope) * a.out_inv_scale);
                if (a.argmax) {
                    const float w4[4] = {acc[fm][fn][0], acc[fm][fn][1], acc[fm][fn][2], acc[fm][fn][3]};
                    a.argmax[(size_t)(mb >> 2) * a.cout_p + col] = window_argmax<DT>(w4, scl, bias, a.act, a.slope, a.out_inv_scale);
                }
            } else {
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = activate(acc[fm][fn][i] * scl + bias, a.act, a.slope);
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int m = mb + i;
                    if (m >= a.M) break;
                    float o = v[i];
                    if (a.res) o += load_el<DT>(a.res, (size_t)m * a.cout_p + col) * a.res_scale;
                    store_el<DT>(a.y, (size_t)m * a.cout_p + col, o * a.out_inv_scale);
                }
            }
        }
    }
}

// 16-byte device-scope load (the buffer instruction's SC1 bit): it misses in
// the caches that other XCDs' stores do not reach.  off: bytes from base.
__device__ __forceinline__ f4 load16_dev(const float *base, unsigned off)
{
    const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, (short)0, 0x7fffffff, 0x00020000);
    return __builtin_bit_cast(f4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)off, 0, 16));
}

// Four channels col..col+3 of output pixel m as NCHW FP32: the value a consumer
// of the stored tensor would read, in the caller's layout.
template <int DT> __device__ __forceinline__ void store4_nchw(float *y, int C, int HW, float scale, unsigned m, int col, const float *v)
{
    const unsigned n = m / (unsigned)HW, p = m - n * (unsigned)HW;
    float *q = y + ((size_t)n * C + col) * HW + p;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float s = stored_value<DT>(v[i]);
        if (col + i < C) q[(size_t)i * HW] = DT == FP8 ? s * scale : s;
    }
}

// Split-K finish of one output group: rows (2x2 windows when pooled) `ro`,
// channels col..col+3 (cout_p is a multiple of 4): the partial sums added in
// split order, then the same epilogue as the unsplit path, one vector store.
// Both finishes below call it, so they round alike.  The separate finish
// reads each split's partials with one 16-byte load as it adds them; the
// in-kernel finish (DEV) issues the device-scope loads of all splits first,
// so that they are in flight together, then adds them in the same order.
template <int DT, bool DEV = false> __device__ __forceinline__ void splitk_finish4(const ConvArgs &a, size_t ro, int col)
{
    float bias[4], scl[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        bias[j] = a.bias[col + j];
        scl[j] = (DT == FP8) ? a.wscale[col + j] * a.in_scale : 1.0f;
    }
    const size_t plane = (size_t)a.M * a.cout_p;
    auto total = [&](size_t m, float *t) {
        t[0] = t[1] = t[2] = t[3] = 0.0f;
        if constexpr (DEV) {
            f4 v[SPLITK_FUSED_MAX];
#pragma unroll
            for (int z = 0; z < SPLITK_FUSED_MAX; ++z)
                if (z < a.splits) v[z] = load16_dev(a.partial, (unsigned)((z * plane + m * a.cout_p + col) * sizeof(float)));
#pragma unroll
            for (int z = 0; z < SPLITK_FUSED_MAX; ++z)
                if (z < a.splits) { t[0] += v[z][0]; t[1] += v[z][1]; t[2] += v[z][2]; t[3] += v[z][3]; }
        } else {
            for (int z = 0; z < a.splits; ++z) {
                const float4 p = *reinterpret_cast<const float4 *>(a.partial + z * plane + m * a.cout_p + col);
                t[0] += p.x; t[1] += p.y; t[2] += p.z; t[3] += p.w;
            }
        }
    };
    float o[4], t[4];
    if (a.pool) {
        float w4[4][4];  // [column][window element]
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = -INFINITY;
        for (int q = 0; q < 4; ++q) {
            total(ro * 4 + q, t);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                w4[j][q] = t[j];
                o[j] = fmaxf(o[j], activate(t[j] * scl[j] + bias[j], a.act, a.slope));
            }
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] *= a.out_inv_scale;
        if (a.argmax) {
#pragma unroll
            for (int j = 0; j < 4; ++j) a.argmax[ro * a.cout_p + col + j] = window_argmax<DT>(w4[j], scl[j], bias[j], a.act, a.slope, a.out_inv_scale);
        }
    } else {
        total(ro, t);
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = activate(t[j] * scl[j] + bias[j], a.act, a.slope);
        if (a.res) {
            float r[4];
            load4<DT>(a.res, ro * a.cout_p + col, r);
#pragma unroll
            for (int j = 0; j < 4; ++j) o[j] += r[j] * a.res_scale;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] *= a.out_inv_scale;
    }
    if (a.nchw) store4_nchw<DT>(a.nchw, a.nchw_c, a.Ho * a.Wo, a.nchw_scale, (unsigned)ro, col, o);
    else store4<DT>(a.y, ro * a.cout_p + col, o);
}

// In-kernel split-K finish (a.tile_count set).  Each split's workgroup of an
// output tile, once its partial plane is written, counts itself in the tile's
// counter; the last of the a.splits workgroups to arrive sums the tile's
// partials in split order and runs the epilogue, then sets the counter back
// to zero for the next launch that uses it.  The L2 caches of the XCDs are
// not coherent with each other: the partials travel by device-scope stores,
// all complete (vmcnt 0) before the workgroup counts itself, and device-scope
// loads issued after the count is seen, so no cache-wide write-back or
// invalidate is needed.
template <int DT, int BM, int BN, int NT>
__device__ __forceinline__ void splitk_tail(const ConvArgs &a, int m0, int n0, void *lds)
{
    // one word of the caller's LDS, whose last reads are behind the barrier below
    int *s_last = reinterpret_cast<int *>(lds);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned *cnt = a.tile_count + blockIdx.x;
        const int last = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (unsigned)(a.splits - 1);
        if (last) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        *s_last = last;
    }
    __syncthreads();
    if (!*s_last) return;
    const int rows = a.pool ? BM / 4 : BM;
    const int r0 = a.pool ? m0 / 4 : m0;
    const int rend = a.pool ? a.M / 4 : a.M;
    constexpr int CQ = BN / 4;
    for (int i = threadIdx.x; i < rows * CQ; i += NT) {
        const int r = r0 + i / CQ, col = n0 + (i % CQ) * 4;
        if (r < rend && col < a.cout_p) splitk_finish4<DT, true>(a, (size_t)r, col);
    }
}

#define DN_OOB 0x80000000u

__device__ __forceinline__ void lds_barrier() { asm volatile("s_barrier" ::: "memory"); }

template <int N> __device__ __forceinline__ void wait_vm()
{
    // s_waitcnt vmcnt(N) with expcnt / lgkmcnt left at their maxima (no wait)
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

typedef int i32x4 __attribute__((ext_vector_type(4)));

// Buffer resource (V#) for raw 32-bit-offset loads: base, stride 0,
// num_records = size in bytes (loads at or past it return zeros).
__device__ __forceinline__ i32x4 make_rsrc(const void *base, unsigned bytes)
{
    const unsigned long long b = (unsigned long long)base;
    return i32x4{(int)(unsigned)b, (int)(unsigned)(b >> 32), (int)bytes, 0x00020000};
}

// One 16-byte-per-lane global -> LDS transfer.  Issued as inline assembly so
// that the compiler does not see an LDS write in flight: it would otherwise
// drain every outstanding transfer (vmcnt(0)) before each LDS read, and the
// pipeline below could not keep K-tiles in flight.  Completion is tracked by
// the explicit vmcnt waits + barrier of the main loop.
// m0 is reserved for the compiler's own LDS-DMA / message use, none of which
// this file emits; listing it as clobbered keeps any such use correct.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma16(const i32x4 &rsrc, unsigned voff, const void *lds_dst)
{
    // the destination is wave-uniform by construction; say so to the compiler
    const unsigned m0v = __builtin_amdgcn_readfirstlane(
        (unsigned)(size_t)(const __attribute__((address_space(3))) void *)lds_dst);
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds"
                 :
                 : "s"(m0v), "v"(voff), "s"(rsrc)
                 : "memory", "m0");
}
#pragma clang diagnostic pop

// Division by a runtime divisor d >= 1 without the integer-divide sequence:
// q = umulhi(n, ceil(2^32 / d)) is exact whenever n * d < 2^32 (true for
// every LDS index here).
struct FastDiv {
    unsigned m, d;
    __device__ explicit FastDiv(unsigned d_) : m(d_ > 1 ? 0xFFFFFFFFu / d_ + 1u : 0u), d(d_) {}
    __device__ __forceinline__ unsigned div(unsigned n) const { return d > 1 ? __umulhi(n, m) : n; }
};

}  // namespace dnk
