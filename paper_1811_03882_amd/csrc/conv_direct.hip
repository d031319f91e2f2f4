// Direct convolutions for layers of few channels: the network's first layer,
// reading the NCHW image itself (conv_first), and the halo kernels, whose input
// windows sit in LDS (conv_halo, conv_halo2).  The operation, the K order (but
// for the first layer's) and the epilogue are conv.hip's.
#include <algorithm>
#include <type_traits>

#include "conv_dev.h"

namespace dnk {

// Dynamic LDS above the default per-kernel limit must be enabled per kernel.
template <typename K> static void allow_lds(K kernel, size_t bytes)
{
    if (bytes > 64 * 1024) (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// ---------------------------------------------------------------- first layer
// The network's first convolution reads the caller's NCHW FP32 image itself
// (the ingest is fused).  A th x 64 output tile (th = 16, or 8 when the window
// of 16 rows would not fit in LDS) stages its input window in LDS as NHWC in
// the storage type, channels padded to CP = 4, 8 or 16 with zeros.  The packed
// weights use the K order k = r*16 + s*CP + c (CP*S <= 16), so the 16 K
// elements of filter row r for output pixel (ho, wo) are the window pixels
// (ho*stride + r, wo*stride + s), s < S: a contiguous span of the window, read
// straight into the MFMA operand (read units past S are zero, matching zero
// weights).  The weights are operand A and stay in registers for the tile;
// pixels are operand B, so a lane's accumulator holds four consecutive output
// channels of one pixel and leaves with one vector store.  With POOL a
// 16-pixel block is four 2x2 windows on lanes 4w..4w+3, reduced by two quad
// shuffles.

constexpr int FT_W = 64;   // conv output columns per workgroup tile

__host__ __device__ constexpr int first_kstep(int dt) { return dt == FP8 ? 128 : (dt == BF16 ? 32 : 16); }
int first_kpad(int dt, int R) { return (R * 16 + first_kstep(dt) - 1) / first_kstep(dt) * first_kstep(dt); }

// CP floats -> one window pixel in the storage type (CP*esize bytes at dst)
// (sc is 1 except for FP8, so only FP8 multiplies)
template <int DT, int CP> __device__ __forceinline__ void put_pixel(unsigned char *dst, const float *v, float sc)
{
    constexpr int NW = CP * esize(DT) / 4;  // 32-bit words
    unsigned w[NW];
#pragma unroll
    for (int i = 0; i < NW; ++i) {
        if constexpr (DT == F32) {
            w[i] = __float_as_uint(v[i]);
        } else if constexpr (DT == BF16) {
            w[i] = (unsigned)f2bf(v[2 * i]) | ((unsigned)f2bf(v[2 * i + 1]) << 16);
        } else {
            w[i] = (unsigned)f2e4m3(v[4 * i] * sc) | ((unsigned)f2e4m3(v[4 * i + 1] * sc) << 8) |
                   ((unsigned)f2e4m3(v[4 * i + 2] * sc) << 16) | ((unsigned)f2e4m3(v[4 * i + 3] * sc) << 24);
        }
    }
    if constexpr (NW == 1) {
        *reinterpret_cast<unsigned *>(dst) = w[0];
    } else if constexpr (NW == 2) {
        *reinterpret_cast<uint2 *>(dst) = make_uint2(w[0], w[1]);
    } else {
#pragma unroll
        for (int q = 0; q < NW / 4; ++q)
            reinterpret_cast<u32x4 *>(dst)[q] = u32x4{w[4 * q], w[4 * q + 1], w[4 * q + 2], w[4 * q + 3]};
    }
}


// s * v + c for a wave-uniform s (24-bit operands) as one v_mad_u32_u24.
// Written out because, for v in {0, 1}, the compiler turns the multiply into
// a select plus an add (two instructions).
__device__ __forceinline__ unsigned mad_u24(int s, int v, int c)
{
    unsigned r;
    asm("v_mad_u32_u24 %0, %1, %2, %3" : "=v"(r) : "s"(s), "v"(v), "v"(c));
    return r;
}
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

// MODE FIRST_ARGMAX (with POOL): also store each window's argmax code
// (a.argmax); FIRST_NCHW: the result leaves as a.nchw.  A template flag so that
// the plain instantiations, bound by instruction issue, carry none of that code.
enum { FIRST_PLAIN = 0, FIRST_ARGMAX = 1, FIRST_NCHW = 2 };
template <int DT, bool POOL, int CP, int MODE = FIRST_PLAIN, int NBM = FIRST_MAX_COUT / 16>
__global__ void __launch_bounds__(256) conv_first(FirstArgs a)
{
    constexpr bool AM = MODE == FIRST_ARGMAX;
    constexpr int ES = esize(DT), SEG = seg_el(DT);
    constexpr int SPL = Tr<DT>::SPL, KSTEP = first_kstep(DT);
    constexpr int KPL = KSTEP / 4;                               // K elements per lane per step
    constexpr int PIXB = CP * ES;                                // bytes per window pixel
    constexpr int UB = PIXB < 16 ? PIXB : 16;                    // LDS read unit
    constexpr int UPS = 16 / UB;                                 // read units per 16-byte segment
    constexpr int MAXKS = DT == FP8 ? 1 : (DT == BF16 ? 2 : 4);  // K-steps for R <= FIRST_MAX_R
    constexpr int MAXNB = NBM;  // 16-channel output blocks this instance handles at most
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const int LH = (a.th - 1) * a.stride + a.R, LW = (FT_W - 1) * a.stride + a.S;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 15, lgrp = lane >> 4;
    // tiles in (image, row band, column) order, dealt to the XCDs in
    // contiguous runs: the halo rows a tile shares with the band above were
    // read through the same L2 shortly before
    const int ntx = (a.Wo + FT_W - 1) / FT_W, nty = (a.Ho + a.th - 1) / a.th;
    const int logical = xcd_remap(blockIdx.x, gridDim.x);
    const int n = logical / (ntx * nty), trem = logical - n * (ntx * nty);
    const int th0 = (trem / ntx) * a.th, tw0 = (trem % ntx) * FT_W;
    const int hi0 = th0 * a.stride - a.pad, wi0 = tw0 * a.stride - a.pad;
    const int KS = a.k_pad / KSTEP;

    // ---- stage the window: thread per pixel, PB pixels (all their channel
    // loads) in flight per thread, (row, col) advanced incrementally.  The
    // image's C planes are one buffer resource: a pixel outside the image
    // gets an offset past its size and the channels C..CP-1 lie past it too,
    // so both read as zero without a branch.
    {
        constexpr int PB = CP == 4 ? 5 : (CP == 8 ? 3 : 2);
        const int npix = LH * LW;
        const unsigned plane = (unsigned)a.H * (unsigned)a.W;
        auto stage = [&](auto u8tag) {
            constexpr bool U8 = decltype(u8tag)::value;
            constexpr unsigned EB = U8 ? 1 : 4;  // bytes per input element
            const void *img = U8 ? (const void *)(a.x8 + (size_t)n * a.C * plane) : (const void *)(a.x + (size_t)n * a.C * plane);
            const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void *)img, (short)0, (int)(a.C * plane * EB), 0x00020000);
            int lr = tid / LW, lc = tid % LW;
            const int dlr = 256 / LW, dlc = 256 % LW;
            for (int base = 0; base < npix; base += 256 * PB) {
                float v[PB][CP];
#pragma unroll
                for (int j = 0; j < PB; ++j) {
                    const int hi = hi0 + lr, wi = wi0 + lc;
                    const bool ok = base + j * 256 + tid < npix && (unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W;
                    const unsigned off = ok ? (unsigned)(hi * a.W + wi) * EB : 0x80000000u;
#pragma unroll
                    for (int c = 0; c < CP; ++c) {
                        if constexpr (U8)
                            v[j][c] = __fdiv_rn((float)__builtin_amdgcn_raw_buffer_load_b8(rs, (int)off, (int)(c * plane), 0), 255.0f);
                        else
                            v[j][c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (int)off, (int)(c * plane * 4), 0));
                    }
                    lc += dlc; lr += dlr;
                    if (lc >= LW) { lc -= LW; ++lr; }
                }
#pragma unroll
                for (int j = 0; j < PB; ++j) {
                    const int p = base + j * 256 + tid;
                    if (p < npix) put_pixel<DT, CP>(lds_raw + (size_t)p * PIXB, v[j], a.in_inv_scale);
                }
            }
        };
        if (a.x8) stage(std::true_type{});
        else stage(std::false_type{});
    }

    // (64-bit indices: blocks x 256 threads pass 2^31 with 8.4 M small images)
    for (size_t i = (size_t)blockIdx.x * 256 + tid; i < (size_t)a.nzero; i += (size_t)gridDim.x * 256) a.zero[i] = 0u;

    // 16 zero bytes after the window: read units past row R or tap S read here
    const int zaddr = (LH * LW * PIXB + 15) & ~15;
    if (tid == 0) *reinterpret_cast<u32x4 *>(lds_raw + zaddr) = u32x4{0u, 0u, 0u, 0u};

    const int nb_count = (a.cout_p + 15) / 16;
    // ---- A fragments (weights) for every 16-channel block, kept in registers
    u32x4 aw[MAXNB][MAXKS][SPL];
#pragma unroll
    for (int nb = 0; nb < MAXNB; ++nb)
#pragma unroll
        for (int ks = 0; ks < MAXKS; ++ks)
#pragma unroll
            for (int j = 0; j < SPL; ++j) {
                aw[nb][ks][j] = u32x4{0u, 0u, 0u, 0u};
                if (nb < nb_count && nb * 16 + lrow < a.cout_p && ks < KS) {
                    const size_t off = ((size_t)(nb * 16 + lrow) * a.k_pad + ks * KSTEP + lgrp * KPL) * ES + j * 16;
                    aw[nb][ks][j] = gload16(a.w, off);
                }
            }
    __syncthreads();

    // per-lane epilogue constants, loaded once.  POOL: pixels are MFMA operand A,
    // so a lane holds one channel (nb*16 + lrow) of the four pixels of one 2x2
    // window and pools in registers.  Otherwise: weights are operand A and a
    // lane holds channels nb*16 + 4*lgrp + (0..3) of one pixel.  The output
    // scale (1 except FP8) folds into scale and bias for BF16 / FP32.
    const float ofold = DT == FP8 ? 1.0f : a.out_inv_scale;
    float bias4[MAXNB][4], scl4[MAXNB][4];
#pragma unroll
    for (int nb = 0; nb < MAXNB; ++nb)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int ch = POOL ? nb * 16 + lrow : nb * 16 + 4 * lgrp + i;
            const bool live = nb < nb_count && ch < a.cout_p;
            bias4[nb][i] = live ? a.bias[ch] * ofold : 0.0f;
            scl4[nb][i] = (DT == FP8 && live) ? a.wscale[ch] * a.in_scale : ofold;
        }
    const float opost = DT == FP8 ? a.out_inv_scale : 1.0f;
    const float lsl = act_slope(a.act, a.slope);
    // this image's output; offsets inside one image fit in 31 bits (checked at launch)
    const int Hy = POOL ? a.Ho >> 1 : a.Ho, Wy = POOL ? a.Wo >> 1 : a.Wo;
    unsigned char *yimg = reinterpret_cast<unsigned char *>(a.y) + (size_t)n * Hy * Wy * a.cout_p * ES;
    // the lane's part of its pixel position; the block's part is wave-uniform
    int lho, lwo;
    if (POOL) {
        lho = (lrow & 3) >> 1;
        lwo = 2 * (lrow >> 2) + (lrow & 1);
    } else {
        lho = 0;
        lwo = lrow;
    }
    const int lpx = (lho * LW + lwo) * a.stride * PIXB;
    // ---- the read units of this lane's K segments: a unit is live inside
    // filter row R and tap S.  Its LDS address for the block at byte offset
    // bpx is bpx * live + ua (one 24-bit multiply-add; LDS addresses are below
    // 2^24): the block's pixel plus the lane's pixel and unit offset where
    // live, the zero area where not.
    // the window's LDS address, so that a unit's address needs no further add
    const int lds_base = (int)(unsigned)(size_t)(const __attribute__((address_space(3))) unsigned char *)lds_raw;
    int ua[MAXKS][SPL][UPS], ulive[MAXKS][SPL][UPS];
#pragma unroll
    for (int ks = 0; ks < MAXKS; ++ks)
#pragma unroll
        for (int j = 0; j < SPL; ++j)
#pragma unroll
            for (int u = 0; u < UPS; ++u) {
                const int k0 = ks * KSTEP + lgrp * KPL + j * SEG;
                const int r = k0 / 16, rb = (k0 % 16) * ES + u * UB;  // byte within the run
                const int s = rb / PIXB;
                const bool live = ks < KS && r < a.R && s < a.S;
                ulive[ks][j][u] = live ? 1 : 0;
                ua[ks][j][u] = lds_base + (live ? lpx + (r * LW + s) * PIXB + rb % PIXB : zaddr);
            }
    auto read_b = [&](int bpx, u32x4 (&bf)[MAXKS][SPL]) {
#pragma unroll
        for (int ks = 0; ks < MAXKS; ++ks)
#pragma unroll
            for (int j = 0; j < SPL; ++j) {
                unsigned wv[4];
#pragma unroll
                for (int u = 0; u < UPS; ++u) {
                    const unsigned addr = mad_u24(bpx, ulive[ks][j][u], ua[ks][j][u]);
                    if constexpr (UB == 16) {
                        const u32x4 t = *(const __attribute__((address_space(3))) u32x4 *)(size_t)addr;
                        wv[0] = t.x; wv[1] = t.y; wv[2] = t.z; wv[3] = t.w;
                    } else if constexpr (UB == 8) {
                        const u32x2 t = *(const __attribute__((address_space(3))) u32x2 *)(size_t)addr;
                        wv[2 * u] = t.x; wv[2 * u + 1] = t.y;
                    } else {
                        wv[u] = *(const __attribute__((address_space(3))) unsigned *)(size_t)addr;
                    }
                }
                bf[ks][j] = u32x4{wv[0], wv[1], wv[2], wv[3]};
            }
    };

    if constexpr (POOL) {
        // Wave w takes, in every band of two output rows, the 16-pixel blocks
        // at columns 8w and 8w + 32 (four 2x2 windows each).  Lane (lgrp,
        // lrow) stores channel nb*16 + lrow of window lgrp: a wave-uniform
        // offset plus a lane constant, through a buffer resource the size of
        // the image's output, so that a window past the right edge (offset
        // moved past the size) is dropped without a branch.
        const __amdgpu_buffer_rsrc_t ry =
            __builtin_amdgcn_make_buffer_rsrc((void *)yimg, (short)0, (int)((size_t)Hy * Wy * a.cout_p * ES), 0x00020000);
        const __amdgpu_buffer_rsrc_t ram = __builtin_amdgcn_make_buffer_rsrc(
            AM ? (void *)(a.argmax + (size_t)n * Hy * Wy * a.cout_p) : nullptr, (short)0, AM ? Hy * Wy * a.cout_p : 0, 0x00020000);
        const unsigned lane_off = (unsigned)((lgrp * a.cout_p + lrow) * ES);
        const int bands = min(a.th >> 1, Hy - (th0 >> 1));
        for (int band = 0; band < bands; ++band) {
            const int hp = (th0 >> 1) + band;
#pragma unroll
            for (int hf = 0; hf < 2; ++hf) {
                const int bwo = 8 * (wave + 4 * hf);
                const int bpx = (2 * band * LW + bwo) * a.stride * PIXB;
                u32x4 bf[MAXKS][SPL];
                read_b(bpx, bf);
                const int wpb = (tw0 >> 1) + (bwo >> 1);
                const bool wok = wpb + lgrp < Wy;
#pragma unroll
                for (int nb = 0; nb < MAXNB; ++nb) {
                    if (nb >= nb_count) break;
                    // acc[i]: channel nb*16 + lrow of pixel 4*lgrp + i = quadrant i of window lgrp.
                    // The max is taken on the accumulators: scale > 0, bias, activation
                    // and rounding are monotone, so this equals pooling the outputs.
                    f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < MAXKS; ++ks) mma<DT>(acc, bf[ks], aw[nb][ks]);
                    const int col = nb * 16 + lrow;
                    const float mx = fmaxf(fmaxf(acc[0], acc[1]), fmaxf(acc[2], acc[3]));
                    const float o = activate_sel(mx * scl4[nb][0] + bias4[nb][0], lsl) * opost;
                    const bool ok = wok && col < a.cout_p;
                    const int soff = ((hp * Wy + wpb) * a.cout_p + nb * 16) * ES;
                    const int voff = ok ? (int)lane_off : (int)0x80000000u;
                    if constexpr (MODE == FIRST_NCHW) {
                        const float s = stored_value<DT>(o);
                        if (ok && col < a.nchw_c)
                            a.nchw[(((size_t)n * a.nchw_c + col) * Hy + hp) * Wy + wpb + lgrp] = DT == FP8 ? s * a.nchw_scale : s;
                        continue;
                    }
                    if constexpr (DT == F32) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o), ry, voff, soff, 0);
                    else if constexpr (DT == BF16) __builtin_amdgcn_raw_buffer_store_b16(f2bf(o), ry, voff, soff, 0);
                    else __builtin_amdgcn_raw_buffer_store_b8(f2e4m3(o), ry, voff, soff, 0);
                    if constexpr (AM) {
                        const float w4[4] = {acc[0], acc[1], acc[2], acc[3]};
                        __builtin_amdgcn_raw_buffer_store_b8(window_argmax<DT>(w4, scl4[nb][0], bias4[nb][0], a.act, a.slope, opost), ram,
                                                             ok ? lgrp * a.cout_p + lrow : (int)0x80000000u,
                                                             (hp * Wy + wpb) * a.cout_p + nb * 16, 0);
                    }
                }
            }
        }
    } else {
        const int blocks = a.th * FT_W / 16;  // 16-pixel MFMA blocks per tile
        for (int b = wave; b < blocks; b += 4) {
            const int bho = b / (FT_W / 16), bwo = (b % (FT_W / 16)) * 16;
            const int bpx = (bho * LW + bwo) * a.stride * PIXB;
            u32x4 bf[MAXKS][SPL];
            read_b(bpx, bf);
            // K steps past k_pad multiply zero weights by zero data: no branches
#pragma unroll
            for (int nb = 0; nb < MAXNB; ++nb) {
                if (nb >= nb_count) break;
                // acc[i]: channel ch0 + i of this lane's pixel
                f4 acc = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < MAXKS; ++ks) mma<DT>(acc, aw[nb][ks], bf[ks]);
                const int ch0 = nb * 16 + 4 * lgrp;
                float v[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = activate_sel(acc[i] * scl4[nb][i] + bias4[nb][i], lsl) * opost;
                const int ho = th0 + bho, wo = tw0 + bwo + lrow;
                if (ho < a.Ho && ch0 < a.cout_p && wo < a.Wo) {
                    if constexpr (MODE == FIRST_NCHW) store4_nchw<DT>(a.nchw + (size_t)n * a.nchw_c * a.Ho * a.Wo, a.nchw_c, a.Ho * a.Wo, a.nchw_scale, (unsigned)(ho * a.Wo + wo), ch0, v);
                    else store4<DT>(yimg, (ho * a.Wo + wo) * a.cout_p + ch0, v);
                }
            }
        }
    }
}

static size_t first_lds_for(int C, int R, int S, int stride, int th, int dt)
{
    const int LH = (th - 1) * stride + R, LW = (FT_W - 1) * stride + S;
    return (((size_t)LH * LW * first_cp(C) * esize(dt) + 15) & ~(size_t)15) + 16;  // window + 16 zero bytes
}
// 32 output rows per tile where that window stays small enough for the
// workgroups per CU the registers allow (fewer halo rows and per-tile set-up
// per output), else 16, else 8.
static int first_tile_h(int dt, int C, int R, int S, int stride)
{
    if (first_lds_for(C, R, S, stride, 32, dt) <= 20 * 1024) return 32;
    return first_lds_for(C, R, S, stride, 16, dt) <= FIRST_LDS_MAX ? 16 : 8;
}
// Fewer rows, down to 4, while the tiles do not give every CU one: a small batch
// is bound by the longest tile, not by the halo rows (32x32, batch 1, FP32: 8.6
// us on two tiles of 16 rows, 5.4 us on eight of 4).
static int first_tile_h(int dt, const FirstArgs &a)
{
    int th = first_tile_h(dt, a.C, a.R, a.S, a.stride);
    while (th > 4 && (long)((a.Wo + FT_W - 1) / FT_W) * ((a.Ho + th - 1) / th) * a.batch < 256) th /= 2;
    return th;
}
size_t first_lds_bytes(int dt, int C, int R, int S, int stride)
{
    return first_lds_for(C, R, S, stride, first_tile_h(dt, C, R, S, stride), dt);
}

hipError_t launch_conv_first(int dt, const FirstArgs &a, hipStream_t s)
{
    FirstArgs b = a;
    b.th = first_tile_h(dt, a);
    const size_t lds = first_lds_for(a.C, a.R, a.S, a.stride, b.th, dt);
    // one image's input planes (up to the padded channel count) and output
    // are addressed through buffer resources with 31-bit offsets
    if (lds > FIRST_LDS_MAX || a.R > FIRST_MAX_R || a.C > 16 || first_cp(a.C) * a.S > 16 || a.cout_p > FIRST_MAX_COUT ||
        a.stride > 2 || (a.cout_p & 3) || (size_t)a.Ho * a.Wo * a.cout_p * esize(dt) >= (1u << 31) ||
        (size_t)first_cp(a.C) * a.H * a.W * 4 >= (1u << 31))
        return hipErrorInvalidValue;
    const long nblk = (long)((a.Wo + FT_W - 1) / FT_W) * ((a.Ho + b.th - 1) / b.th) * a.batch;
    if (nblk >= (1L << 31)) return hipErrorInvalidValue;
    dim3 grid((unsigned)nblk);
#define DN_FIRST_CP(D, P, C, M)                                                                      \
    do {                                                                                             \
        if (b.cout_p <= 16) {                                                                        \
            allow_lds(conv_first<D, P, C, M, 1>, lds);                                               \
            hipLaunchKernelGGL((conv_first<D, P, C, M, 1>), grid, dim3(256), lds, s, b);             \
        } else {                                                                                     \
            allow_lds(conv_first<D, P, C, M>, lds);                                                  \
            hipLaunchKernelGGL((conv_first<D, P, C, M>), grid, dim3(256), lds, s, b);                \
        }                                                                                            \
    } while (0)
#define DN_FIRST_P(D, P, M)                                                                          \
    do {                                                                                             \
        const int cp = first_cp(a.C);                                                                \
        if (cp == 4) DN_FIRST_CP(D, P, 4, M);                                                        \
        else if (cp == 8) DN_FIRST_CP(D, P, 8, M);                                                   \
        else DN_FIRST_CP(D, P, 16, M);                                                               \
    } while (0)
#define DN_FIRST(D)                                                                                  \
    do {                                                                                             \
        if (b.nchw) {                                                                                \
            if (b.pool) DN_FIRST_P(D, true, FIRST_NCHW);                                             \
            else DN_FIRST_P(D, false, FIRST_NCHW);                                                   \
        } else if (b.pool) {                                                                         \
            DN_FIRST_P(D, true, FIRST_PLAIN);                                                        \
        } else {                                                                                     \
            DN_FIRST_P(D, false, FIRST_PLAIN);                                                       \
        }                                                                                            \
    } while (0)
    if (b.argmax && (!b.pool || dt == FP8)) return hipErrorInvalidValue;
    if (b.argmax) {  // the input-gradient pass (F32 / BF16)
        if (dt == F32) DN_FIRST_P(F32, true, FIRST_ARGMAX);
        else DN_FIRST_P(BF16, true, FIRST_ARGMAX);
        return hipGetLastError();
    }
    switch (dt) {
    case F32: DN_FIRST(F32); break;
    case BF16: DN_FIRST(BF16); break;
    case FP8: DN_FIRST(FP8); break;
    default: return hipErrorInvalidValue;
    }
#undef DN_FIRST
#undef DN_FIRST_P
#undef DN_FIRST_CP
    return hipGetLastError();
}

// ---------------------------------------------------------------- halo kernel
// Small convolutions (K = R*S*Cin_p up to HALO_KMAX elements, Cout <= 64):
// one workgroup owns a TH x 32 output tile and every output channel.  Its
// input window (tile + filter halo) is read from HBM once into LDS, NHWC,
// each pixel padded to an odd number of 16-byte chunks so that the 16 lanes
// of a fragment read hit distinct banks; the weights [cout_p][K] sit in LDS
// as well (rows padded the same way).  The whole K loop then runs out of
// LDS: a lane's A-fragment segment is the 16-byte channel chunk (tap, c0) of
// its pixel, read directly from the window, so no input element is fetched
// once per filter tap as in the gathered implicit GEMM.

constexpr int HT_W = 32;
constexpr int HALO_KMAX_BYTES = 1280;  // K * element size (the offset table holds 20 MFMA K-steps)

int halo_lds_bytes(int dt, const ConvArgs &a, int th)
{
    const int ES = esize(dt), SEG = seg_el(dt);
    const int kstep = 4 * (dt == FP8 ? 32 : (dt == BF16 ? 8 : 4));
    const int K = a.R * a.S * a.cin_p;
    const int ku = (K + kstep - 1) / kstep * kstep;
    const int cps = a.cin_p / SEG, pst = cps | 1;
    const int wch = ku * ES / 16, wst = wch | 1;
    const int lh = (th - 1) * a.stride + a.R, lw = (HT_W - 1) * a.stride + a.S;
    const int coutp = (a.cout_p + 15) / 16 * 16;
    return (lh * lw * pst + coutp * wst + 1) * 16;  // window, weights, one zero chunk
}

constexpr int HALO_LDS_MAX = 96 * 1024;

bool halo_ok(int dt, const ConvArgs &a)
{
    return kblock_ch(dt, a.cin_p, a.R * a.S) == a.cin_p && a.R * a.S * a.cin_p * esize(dt) <= HALO_KMAX_BYTES &&
           a.cout_p <= 64 && a.stride <= 2 && (size_t)a.Ho * a.Wo * a.cout_p < (1u << 31) &&
           (size_t)a.H * a.W * a.cin_p * esize(dt) < (1u << 31) &&
           halo_lds_bytes(dt, a, 8) <= HALO_LDS_MAX;
}


// AM (with POOL): also store each window's argmax code (a.argmax).
template <int DT, bool POOL, int TH, int NB, bool AM = false>
__global__ void __launch_bounds__(256) conv_halo(ConvArgs a)
{
    constexpr int ES = esize(DT), SEG = seg_el(DT);
    constexpr int SPL = Tr<DT>::SPL;
    constexpr int KPL = 4 * SPL * SEG / 4;                 // K elements per lane per MFMA step
    constexpr int KSTEP = 4 * KPL;
    constexpr int BLOCKS = TH * HT_W / 16, NBW = BLOCKS / 4;  // MFMA blocks per tile / per wave
    constexpr int MAXNB = NB;                                 // 16-channel output blocks
    static_assert(KPL == SPL * SEG, "lane K chunk");
    extern __shared__ __align__(16) unsigned char halo_raw[];
    u32x4 *win = reinterpret_cast<u32x4 *>(halo_raw);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 15, lgrp = lane >> 4;
    const int n = blockIdx.z, th0 = blockIdx.y * TH, tw0 = blockIdx.x * HT_W;
    const int K = a.R * a.S * a.cin_p;
    const int KS = (K + KSTEP - 1) / KSTEP;
    const int cps = a.cin_p / SEG, pst = cps | 1;
    const int wch = KS * KSTEP * ES / 16, wst = wch | 1;
    const int LH = (TH - 1) * a.stride + a.R, LW = (HT_W - 1) * a.stride + a.S;
    u32x4 *wlds = win + LH * LW * pst;
    constexpr int nb_count = NB;
    const u32x4 z4 = {0u, 0u, 0u, 0u};
    const int zchunk = LH * LW * pst + NB * 16 * wst;  // reads past K land on this zero chunk
    if (tid == 0) win[zchunk] = z4;

    // ---- input window -> LDS (8 loads in flight per thread)
    {
        const int hi0 = th0 * a.stride - a.pad, wi0 = tw0 * a.stride - a.pad;
        const int tot = LH * LW * cps;
        const FastDiv by_cps(cps), by_lw(LW);
        const unsigned char *ximg = reinterpret_cast<const unsigned char *>(a.x) + (size_t)n * a.H * a.W * a.cin_p * ES;
        for (int base = 0; base < tot; base += 256 * 8) {
            u32x4 v[8];
            int dst[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const int e = base + j * 256 + tid;
                const int px = by_cps.div(e), ch = e - px * cps;
                const int lr = by_lw.div(px), lc = px - lr * LW;
                const int hi = hi0 + lr, wi = wi0 + lc;
                const bool ok = e < tot && (unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W;
                const unsigned off = ok ? (unsigned)(((hi * a.W + wi) * a.cin_p + ch * SEG) * ES) : 0u;
                v[j] = ok ? gload16(ximg, off) : z4;
                dst[j] = e < tot ? px * pst + ch : -1;
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (dst[j] >= 0) win[dst[j]] = v[j];
        }
        // weights: rows [cout_p][KS*KSTEP] (K beyond k_pad reads as zero)
        const int wtot = nb_count * 16 * wch;
        const FastDiv by_wch(wch);
        for (int e = tid; e < wtot; e += 256) {
            const int row = by_wch.div(e), ch = e - row * wch;
            const bool ok = row < a.cout_p && (ch + 1) * 16 <= a.k_pad * ES;
            wlds[row * wst + ch] = ok ? gload16(a.w, (size_t)row * a.k_pad * ES + ch * 16) : z4;
        }
    }
    __syncthreads();

    // ---- window offsets (in chunks) of every 16-byte K segment, -1 beyond K:
    // table[(ks*4 + lane group)*SPL + j], one division per entry per workgroup
    __shared__ int toff_tab[20 * 4 * 2];
    for (int e = tid; e < KS * 4 * SPL; e += 256) {
        const int j = e % SPL, g = (e / SPL) % 4, ks = e / (4 * SPL);
        const int k = ks * KSTEP + g * KPL + j * SEG;
        int o = -1;
        if (k < K) {
            const int tap = k / a.cin_p, c0 = k - tap * a.cin_p;
            const int r = tap / a.S, sx = tap - r * a.S;
            o = (r * LW + sx) * pst + c0 / SEG;
        }
        toff_tab[e] = o;
    }
    __syncthreads();

    // ---- this wave's blocks: pixel of lane (A row) per block
    int pbase[NBW];
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
        const int b = wave + 4 * i;
        int hl, wl;
        if (POOL) {
            const int rp = b / (HT_W / 8), wg = b % (HT_W / 8);
            hl = 2 * rp + ((lrow >> 1) & 1);
            wl = 2 * (wg * 4 + (lrow >> 2)) + (lrow & 1);
        } else {
            hl = b / (HT_W / 16);
            wl = (b % (HT_W / 16)) * 16 + lrow;
        }
        pbase[i] = (hl * a.stride * LW + wl * a.stride) * pst;
    }

    f4 acc[NBW][MAXNB];
#pragma unroll
    for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int j = 0; j < MAXNB; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

    for (int ks = 0; ks < KS; ++ks) {
        int toff[SPL];
#pragma unroll
        for (int j = 0; j < SPL; ++j) toff[j] = toff_tab[(ks * 4 + lgrp) * SPL + j];
        u32x4 bfr[MAXNB][SPL];
#pragma unroll
        for (int nb = 0; nb < MAXNB; ++nb)
#pragma unroll
            for (int j = 0; j < SPL; ++j)
                bfr[nb][j] = nb < nb_count ? wlds[(nb * 16 + lrow) * wst + (ks * KSTEP + lgrp * KPL + j * SEG) / SEG] : z4;
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            u32x4 af[SPL];
#pragma unroll
            for (int j = 0; j < SPL; ++j) af[j] = win[toff[j] >= 0 ? pbase[i] + toff[j] : zchunk];
#pragma unroll
            for (int nb = 0; nb < MAXNB; ++nb)
                if (nb < nb_count) mma<DT>(acc[i][nb], af, bfr[nb]);
        }
    }

    // ---- epilogue: bias, activation, [residual], [2x2 max], round, NHWC store
    // (offsets inside one image fit in 32 bits: checked by halo_ok)
    const int Hp = a.Ho >> 1, Wp = a.Wo >> 1;
    const size_t img = POOL ? (size_t)Hp * Wp * a.cout_p : (size_t)a.Ho * a.Wo * a.cout_p;
    unsigned char *yimg = reinterpret_cast<unsigned char *>(a.y) + (size_t)n * img * ES;
    const unsigned char *rimg = a.res ? reinterpret_cast<const unsigned char *>(a.res) + (size_t)n * img * ES : nullptr;
#pragma unroll
    for (int nb = 0; nb < MAXNB; ++nb) {
        if (nb >= nb_count) break;
        const int col = nb * 16 + lrow;
        if (col >= a.cout_p) continue;
        const float bias = a.bias[col];
        const float scl = (DT == FP8) ? a.wscale[col] * a.in_scale : 1.0f;
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
            const int b = wave + 4 * i;
            if (POOL) {
                // a lane's four rows are one 2x2 window: pool the accumulators
                // (scale > 0; bias, activation and rounding are monotone)
                const float mx = fmaxf(fmaxf(acc[i][nb][0], acc[i][nb][1]), fmaxf(acc[i][nb][2], acc[i][nb][3]));
                const float o = activate(mx * scl + bias, a.act, a.slope) * a.out_inv_scale;
                const int rp = b / (HT_W / 8), wg = b % (HT_W / 8);
                const int hp = (th0 >> 1) + rp, wp = (tw0 >> 1) + wg * 4 + lgrp;
                if (hp < Hp && wp < Wp) {
                    store_el<DT>(yimg, (hp * Wp + wp) * a.cout_p + col, o);
                    if constexpr (AM) {
                        const float w4[4] = {acc[i][nb][0], acc[i][nb][1], acc[i][nb][2], acc[i][nb][3]};
                        a.argmax[(size_t)n * img + (hp * Wp + wp) * a.cout_p + col] = window_argmax<DT>(w4, scl, bias, a.act, a.slope, a.out_inv_scale);
                    }
                }
            } else {
                float v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) v[q] = activate(acc[i][nb][q] * scl + bias, a.act, a.slope);
                const int ho = th0 + b / (HT_W / 16);
                if (ho < a.Ho) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int wo = tw0 + (b % (HT_W / 16)) * 16 + 4 * lgrp + q;
                        if (wo >= a.Wo) continue;
                        const int o = (ho * a.Wo + wo) * a.cout_p + col;
                        float r = v[q];
                        if (rimg) r += load_el<DT>(rimg, o) * a.res_scale;
                        store_el<DT>(yimg, o, r * a.out_inv_scale);
                    }
                }
            }
        }
    }
}

template <int DT, bool POOL, int TH, bool AM = false>
static hipError_t go_halo(const ConvArgs &a, dim3 grid, size_t lds, hipStream_t s)
{
    switch ((a.cout_p + 15) / 16) {
    case 1: allow_lds(conv_halo<DT, POOL, TH, 1, AM>, lds); hipLaunchKernelGGL((conv_halo<DT, POOL, TH, 1, AM>), grid, dim3(256), lds, s, a); break;
    case 2: allow_lds(conv_halo<DT, POOL, TH, 2, AM>, lds); hipLaunchKernelGGL((conv_halo<DT, POOL, TH, 2, AM>), grid, dim3(256), lds, s, a); break;
    case 3: allow_lds(conv_halo<DT, POOL, TH, 3, AM>, lds); hipLaunchKernelGGL((conv_halo<DT, POOL, TH, 3, AM>), grid, dim3(256), lds, s, a); break;
    case 4: allow_lds(conv_halo<DT, POOL, TH, 4, AM>, lds); hipLaunchKernelGGL((conv_halo<DT, POOL, TH, 4, AM>), grid, dim3(256), lds, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int DT>
static hipError_t go_halo_dt(const ConvArgs &a, int th, dim3 grid, size_t lds, hipStream_t s)
{
    if constexpr (DT != FP8) {
        if (a.pool && a.argmax)  // the input-gradient pass
            return th == 16 ? go_halo<DT, true, 16, true>(a, grid, lds, s) : go_halo<DT, true, 8, true>(a, grid, lds, s);
    }
    if (th == 16) return a.pool ? go_halo<DT, true, 16>(a, grid, lds, s) : go_halo<DT, false, 16>(a, grid, lds, s);
    return a.pool ? go_halo<DT, true, 8>(a, grid, lds, s) : go_halo<DT, false, 8>(a, grid, lds, s);
}

hipError_t launch_conv_halo(int dt, const ConvArgs &a, hipStream_t s)
{
    if (!halo_ok(dt, a)) return hipErrorInvalidValue;
    // 16-row tiles when two workgroups still fit in a CU's LDS and there are
    // enough of them for every CU, else 8 rows (208x208x16 -> 32, FP32, batch 1:
    // 18.4 us on 91 tiles of 16 rows, 11.7 on 182 of 8)
    const long tiles16 = (long)((a.Wo + HT_W - 1) / HT_W) * ((a.Ho + 15) / 16) * a.batch;
    const int th = halo_lds_bytes(dt, a, 16) <= 80 * 1024 && tiles16 >= 256 ? 16 : 8;
    dim3 grid((a.Wo + HT_W - 1) / HT_W, (a.Ho + th - 1) / th, a.batch);
    const size_t lds = halo_lds_bytes(dt, a, th);
    switch (dt) {
    case F32: return go_halo_dt<F32>(a, th, grid, lds, s);
    case BF16: return go_halo_dt<BF16>(a, th, grid, lds, s);
    case FP8: return go_halo_dt<FP8>(a, th, grid, lds, s);
    default: return hipErrorInvalidValue;
    }
}

// ---------------------------------------------------------------- persistent halo kernel
// The halo kernel's operation and reduction order (every output element is one
// 16x16 MFMA chain over the same K steps, in order, with the same K subset per
// lane as the GEMM tiles), restructured so that loads overlap the products:
//   * two workgroups per CU each loop over TH x 32 output tiles (every
//     output channel);
//   * each wave keeps the weights of its output channels (NBP 16-channel
//     blocks of NG groups) in registers for the whole run (no per-tile weight
//     staging) and owns a part of each tile's 16-pixel MFMA blocks (NQ parts,
//     NG * NQ = 4 waves); one fragment read from LDS feeds one MFMA per
//     channel block;
//   * a block is 16 consecutive pixels of one output row, so the 16 lanes of
//     a fragment read hit 16 distinct LDS banks (odd chunk pitch per pixel);
//     a wave owns blocks in vertical pairs, so with a fused 2x2 pool each
//     window's four outputs sit in one lane's accumulators (rows r and r+1,
//     two neighbouring columns);
//   * input windows travel global -> LDS directly (buffer_load ... lds) into
//     NBUF buffers, so the windows of the next NBUF-1 tiles are in flight
//     while one is multiplied (one barrier per tile);
//   * tiles are dealt out in runs of consecutive tiles per XCD, so the halo
//     rows and columns that neighbouring tiles share are read through the
//     same L2;
//   * stores are counted, and the wait for a window leaves them in flight; an
//     unpooled tile stores four channels of a pixel per lane and instruction
//     (two bytes per lane before).  Input gradient of the nine-layer net, batch
//     16, BF16, whose convs with argmax codes and to the image run here: 763 ->
//     729 us.
// Bound by issue and latency with two waves per SIMD (counters at 104x104x32 ->
// 64 + pool, batch 64: matrix cores busy 33 %, VALU 39 %, waves waiting 44 %).

// Output rows per tile: 16, or 8 for four 16-channel blocks (whose
// accumulators and weights would not leave room for 16 rows).
__host__ __device__ constexpr int h2_th(int nb) { return nb >= 4 ? 8 : 16; }
// K steps whose weights a wave keeps in registers (BF16 / FP32: 10, FP8: 5).
__host__ __device__ constexpr int h2_ksmax(int dt) { return dt == FP8 ? 5 : 10; }
constexpr int H2_MAXBLK = 16;  // 1 KB window blocks one wave transfers per tile (at most)

// Chunk pitch of a window pixel: odd (the 16 lanes of a fragment read, 16
// consecutive pixels, hit distinct banks) and at least one chunk longer than
// the pixel's channels (the padding chunk, loaded as zeros, is what K
// segments past K read).
__host__ __device__ constexpr int h2_pitch(int cps) { return (cps & 1) ? cps + 2 : cps + 1; }
// 16-channel blocks per wave: every block up to 3, two of four.
__host__ __device__ constexpr int h2_nbp(int nb) { return nb == 4 ? 2 : nb; }
// Tile row of block i of pixel part q of rpw rows: a part's blocks are its rows
// one after the other, each in two column halves.
__device__ __forceinline__ constexpr int h2_row(int q, int rpw, int i) { return q * rpw + (i >> 1); }

// s_waitcnt vmcnt(at most n) for a wave-uniform run-time n: the largest of a few
// constants not above it.
__device__ __forceinline__ void wait_vm_upto(int n)
{
    if (n >= 32) {
        if (n >= 48) { if (n >= 60) wait_vm<60>(); else wait_vm<48>(); }
        else { if (n >= 40) wait_vm<40>(); else wait_vm<32>(); }
    } else if (n >= 16) {
        if (n >= 24) { if (n >= 28) wait_vm<28>(); else wait_vm<24>(); }
        else { if (n >= 20) wait_vm<20>(); else wait_vm<16>(); }
    } else if (n >= 8) {
        if (n >= 12) { if (n >= 14) wait_vm<14>(); else wait_vm<12>(); }
        else { if (n >= 10) wait_vm<10>(); else wait_vm<8>(); }
    } else {
        if (n >= 4) { if (n >= 6) wait_vm<6>(); else wait_vm<4>(); }
        else if (n >= 2) wait_vm<2>();
        else wait_vm<0>();
    }
}

template <int N>
struct Int {
    static constexpr int value = N;
};

// 16-byte units of a window buffer, rounded to whole 1 KB transfers.
__host__ __device__ constexpr int h2_wslots(int lh, int lw, int cps) { return (lh * lw * h2_pitch(cps) + 63) / 64 * 64; }

// CPS > 0: a 3x3 stride-1 filter over CPS 16-byte chunks of channels, so that
// the window's layout is known at compile time: a fragment's address is one
// lane register per K step plus a constant, a window transfer's one addition
// (rows outside the image fall outside the buffer by themselves; columns are
// tested only in tiles at the left or right edge).  CPS = 0: any shape.
template <int DT, bool POOL, int NB, bool AM = false, int CPS = 0>
__global__ void __launch_bounds__(256, 2) conv_halo2(ConvArgs a, int nbuf)
{
    constexpr int ES = esize(DT), SEG = seg_el(DT);
    constexpr int SPL = Tr<DT>::SPL;
    constexpr int KPL = SPL * SEG, KSTEP = 4 * KPL;
    constexpr int NBP = h2_nbp(NB), NG = NB / NBP, NQ = 4 / NG;
    constexpr int TH = h2_th(NB), BLOCKS = TH * HT_W / 16, BPW = BLOCKS / NQ, RPW = BPW / 2;
    constexpr bool FIX = CPS > 0;
    constexpr bool TAPS = FIX && CPS * SEG == KSTEP;  // a K step is one filter tap
    constexpr int KSM = FIX ? (9 * CPS * SEG + KSTEP - 1) / KSTEP : h2_ksmax(DT);
    constexpr int MAXBLK = FIX ? (h2_wslots(TH + 2, HT_W + 2, FIX ? CPS : 1) / 64 + 3) / 4 : H2_MAXBLK;
    static_assert(NG * NBP == NB && RPW % 2 == 0 && RPW * NQ == TH, "wave split");
    extern __shared__ __align__(16) unsigned char halo_raw[];
    u32x4 *lds = reinterpret_cast<u32x4 *>(halo_raw);

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wg = wave % NG, wq = wave / NG;  // channel group, pixel part
    const int lrow = lane & 15, lgrp = lane >> 4;
    const int FR = FIX ? 3 : a.R, FS = FIX ? 3 : a.S, SD = FIX ? 1 : a.stride;
    const int cps = FIX ? CPS : a.cin_p / SEG, cin_p = cps * SEG, pst = h2_pitch(cps);
    const int K = FR * FS * cin_p;
    const int KS = (K + KSTEP - 1) / KSTEP;
    const int LH = (TH - 1) * SD + FR, LW = (HT_W - 1) * SD + FS;
    const int npx = LH * LW;
    const int wslots = h2_wslots(LH, LW, cps), nblk = wslots / 64;  // 16-byte slots per buffer
    const int ntw = (a.Wo + HT_W - 1) / HT_W, nth = (a.Ho + TH - 1) / TH;
    const int per_img = ntw * nth, total = a.batch * per_img;
    const unsigned img_bytes = (unsigned)((size_t)a.H * a.W * cin_p * ES);
    const u32x4 z4 = {0u, 0u, 0u, 0u};

    // this workgroup's tiles: XCD (blockIdx % 8) owns a run of consecutive tiles
    const int xcd = blockIdx.x & 7, li = blockIdx.x >> 3, per_xcd = gridDim.x >> 3;
    const int run = (total + 7) / 8;
    const int t_end = min(total, (xcd + 1) * run);
    const int t0 = xcd * run + li;
    if (t0 >= t_end) return;  // whole workgroup
    const int my_tiles = (t_end - t0 + per_xcd - 1) / per_xcd;

    // tile position (image, row, column) and its step from one of this
    // workgroup's tiles to the next: divided out once, then added with carries
    struct Pos { int n, ti, tj; };
    const int step_n = per_xcd / per_img, step_r = per_xcd - step_n * per_img, step_i = step_r / ntw, step_j = step_r - step_i * ntw;
    auto next = [&](Pos &q) {
        q.tj += step_j;
        if (q.tj >= ntw) { q.tj -= ntw; ++q.ti; }
        q.ti += step_i;
        if (q.ti >= nth) { q.ti -= nth; ++q.n; }
        q.n += step_n;
    };
    Pos cur;  // the tile multiplied next
    cur.n = t0 / per_img;
    cur.ti = (t0 - cur.n * per_img) / ntw;
    cur.tj = t0 - cur.n * per_img - cur.ti * ntw;
    Pos ahead = cur;  // the tile whose window goes out next
    int abuf = 0;

    // window slots this wave transfers: blocks wave, wave + 4, ...; lane L
    // of a block fills slot 64*block + L = pixel * pst + chunk (chunks past
    // the pixel's channels are padding and load zeros)
    const int dw = nblk > wave ? (nblk - wave + 3) / 4 : 0;
    const FastDiv by_pst(pst), by_lw(LW);
    constexpr unsigned DEAD = 0xC0000000u;  // past any buffer this runs on, also with a tile's offset added
    int s_lr[MAXBLK], s_lc[MAXBLK], s_off[MAXBLK];
#pragma unroll
    for (int q = 0; q < MAXBLK; ++q) {
        const int sl = (wave + 4 * q) * 64 + lane;
        const int px = by_pst.div(sl), ch = sl - px * pst;
        const int lr = by_lw.div(px), lc = px - lr * LW;
        const bool live = q < dw && ch < cps && px < npx;
        s_lr[q] = live ? lr : -(1 << 20);
        s_lc[q] = lc;
        s_off[q] = (lc * cin_p + ch * SEG) * ES;
        if constexpr (FIX) s_off[q] = live ? s_off[q] + lr * a.W * cin_p * ES : (int)DEAD;
    }
    auto issue = [&] {  // the window at `ahead` into buffer abuf
        const int hi0 = ahead.ti * TH * SD - a.pad, wi0 = ahead.tj * HT_W * SD - a.pad;
        i32x4 rs = make_rsrc(reinterpret_cast<const unsigned char *>(a.x) + (size_t)ahead.n * img_bytes, img_bytes);
        // wave-uniform by construction; keep it in scalar registers
        rs.x = __builtin_amdgcn_readfirstlane(rs.x);
        rs.y = __builtin_amdgcn_readfirstlane(rs.y);
        rs.z = __builtin_amdgcn_readfirstlane(rs.z);
        rs.w = __builtin_amdgcn_readfirstlane(rs.w);
        u32x4 *dst = lds + abuf * wslots;
        if constexpr (FIX) {
            const int toff = (hi0 * a.W + wi0) * cin_p * ES;
            const bool inside = wi0 >= 0 && wi0 + LW <= a.W;
#pragma unroll
            for (int q = 0; q < MAXBLK; ++q) {
                if (q >= dw) break;  // wave-uniform
                unsigned off = (unsigned)(s_off[q] + toff);
                if (!inside && (unsigned)(wi0 + s_lc[q]) >= (unsigned)a.W) off = DN_OOB;
                dma16(rs, off, dst + (wave + 4 * q) * 64);
            }
        } else {
#pragma unroll
            for (int q = 0; q < MAXBLK; ++q) {
                if (q >= dw) break;  // wave-uniform
                const int hi = hi0 + s_lr[q], wi = wi0 + s_lc[q];
                const bool ok = (unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W;
                const unsigned off = ok ? (unsigned)((hi * a.W + wi0) * cin_p * ES + s_off[q]) : DN_OOB;
                dma16(rs, off, dst + (wave + 4 * q) * 64);
            }
        }
        next(ahead);
        abuf = abuf + 1 == nbuf ? 0 : abuf + 1;
    };
    // the first nbuf - 1 windows go out before anything else
    for (int k = 0; k < nbuf - 1 && k < my_tiles; ++k) issue();

    // weights of this wave's output channels, all K steps, in registers
    u32x4 wr[NBP][KSM][SPL];
#pragma unroll
    for (int nb = 0; nb < NBP; ++nb)
#pragma unroll
        for (int ks = 0; ks < KSM; ++ks)
#pragma unroll
            for (int j = 0; j < SPL; ++j) {
                const int ch = (wg * NBP + nb) * 16 + lrow;
                const int k = ks * KSTEP + lgrp * KPL + j * SEG;
                wr[nb][ks][j] = (ks < KS && ch < a.cout_p) ? gload16(a.w, ((size_t)ch * a.k_pad + k) * ES) : z4;
            }
    // byte offset, relative to the lane's pixel, of the 16-byte chunk that
    // holds this lane's K segment j of step ks; segments past K read the
    // pixel's own padding chunk (always zero)
    int toffb[KSM][SPL];
#pragma unroll
    for (int ks = 0; ks < KSM; ++ks)
#pragma unroll
        for (int j = 0; j < SPL; ++j) {
            const int k = ks * KSTEP + lgrp * KPL + j * SEG;
            int o = cps;
            if (k < K) {
                const int tap = k / cin_p, c0 = k - tap * cin_p;
                const int r = tap / FS, sx = tap - r * FS;
                o = (r * LW + sx) * pst + c0 / SEG;
            }
            toffb[ks][j] = o * 16;
            // FIX: the LDS address for the wave's first block (constant offsets lead to the others)
            if constexpr (FIX)
                toffb[ks][j] += (int)(unsigned)(size_t)(const __attribute__((address_space(3))) unsigned char *)halo_raw +
                                (h2_row(wq, RPW, 0) * LW + lrow) * pst * 16;
        }
    // this wave's blocks: block i is tile row h2_row(wq, RPW, i), columns
    // 16 * (i & 1) + (0..15); lane lrow reads the A row of pixel lrow
    int pbb[BPW];
#pragma unroll
    for (int i = 0; i < BPW; ++i)
        pbb[i] = (h2_row(wq, RPW, i) * SD * LW + (16 * (i & 1) + lrow) * SD) * pst * 16;
    // pooled: a lane's accumulators are one channel of four pixels (pixels are
    // MFMA operand A); else four channels of one pixel (weights are operand A)
    constexpr int CH = POOL ? 1 : 4;
    float bias[NBP][CH], scl[NBP][CH];
#pragma unroll
    for (int nb = 0; nb < NBP; ++nb)
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int col = (wg * NBP + nb) * 16 + (POOL ? lrow : 4 * lgrp + i);
            bias[nb][i] = col < a.cout_p ? a.bias[col] : 0.0f;
            scl[nb][i] = (DT == FP8 && col < a.cout_p) ? a.wscale[col] * a.in_scale : 1.0f;
        }
    const int Hp = a.Ho >> 1, Wp = a.Wo >> 1;
    const size_t img = POOL ? (size_t)Hp * Wp * a.cout_p : (size_t)a.Ho * a.Wo * a.cout_p;
    const float lsl = act_slope(a.act, a.slope);

    int cbuf = 0;
    int st1 = 0, st2 = 0, st3 = 0;  // vector stores this wave issued for tiles k - 1, k - 2, k - 3
    for (int k = 0; k < my_tiles; ++k) {
        // this wave's transfers of tile k landed.  Vector memory operations
        // complete in order, so whatever was issued after them may stay in
        // flight: the transfers of the next tiles and the stores of the last
        // nbuf - 1 (waiting for those too exposed their way to memory in every
        // tile).  The count never exceeds what was issued.
        wait_vm_upto(min(nbuf - 2, my_tiles - 1 - k) * dw + st1 + (nbuf > 2 ? st2 : 0) + (nbuf > 3 ? st3 : 0));
        // the barrier: every wave's transfers landed and every wave is done
        // with tile k - 1's buffer
        lds_barrier();
        if (k + nbuf - 1 < my_tiles) issue();
        const int n = cur.n, th0 = cur.ti * TH, tw0 = cur.tj * HT_W;

        f4 acc[BPW][NBP];
#pragma unroll
        for (int i = 0; i < BPW; ++i)
#pragma unroll
            for (int nb = 0; nb < NBP; ++nb) acc[i][nb] = f4{0.f, 0.f, 0.f, 0.f};
        const int woff = cbuf * wslots * 16;
        // the second column half of a tile at the right edge can lie outside
        // altogether: no work for it (one block in eight at 104 columns)
        const bool half = tw0 + 16 >= a.Wo;
        if constexpr (TAPS) {
            // window row by window row: a fragment read once serves every
            // output row whose filter covers it (up to three), and each output
            // still adds its taps in order
            using lds16 = const __attribute__((address_space(3))) u32x4;
            const auto *q = (const __attribute__((address_space(3))) unsigned char *)(size_t)(unsigned)(toffb[0][0] + woff);
            auto taps = [&](auto halves) {
#pragma unroll
                for (int ir = 0; ir < RPW + 2; ++ir)
#pragma unroll
                    for (int sx = 0; sx < 3; ++sx)
#pragma unroll
                        for (int c = 0; c < halves.value; ++c) {
                            const u32x4 f[1] = {*(lds16 *)(q + (ir * (HT_W + 2) + sx + 16 * c) * h2_pitch(FIX ? CPS : 1) * 16)};
#pragma unroll
                            for (int r = 0; r < 3; ++r) {
                                const int row = ir - r;
                                if (row < 0 || row >= RPW) continue;
#pragma unroll
                                for (int nb = 0; nb < NBP; ++nb) {
                                    if constexpr (POOL) mma<DT>(acc[2 * row + c][nb], f, wr[nb][3 * r + sx]);
                                    else mma<DT>(acc[2 * row + c][nb], wr[nb][3 * r + sx], f);
                                }
                            }
                        }
            };
            if (half) taps(Int<1>());
            else taps(Int<2>());
        } else if constexpr (FIX) {
            auto steps = [&](auto halves) {
                constexpr int ST = 3 - halves.value;  // every block, or the first column halves
#pragma unroll
                for (int ks = 0; ks < KSM; ++ks) {
                    u32x4 af[BPW][SPL];
#pragma unroll
                    for (int j = 0; j < SPL; ++j) {
                        const auto *q = (const __attribute__((address_space(3))) unsigned char *)(size_t)(unsigned)(toffb[ks][j] + woff);
#pragma unroll
                        for (int i = 0; i < BPW; i += ST)
                            af[i][j] = *(const __attribute__((address_space(3))) u32x4 *)(q + ((i >> 1) * (HT_W + 2) + 16 * (i & 1)) * h2_pitch(FIX ? CPS : 1) * 16);
                    }
#pragma unroll
                    for (int i = 0; i < BPW; i += ST)
#pragma unroll
                        for (int nb = 0; nb < NBP; ++nb) {
                            if constexpr (POOL) mma<DT>(acc[i][nb], af[i], wr[nb][ks]);
                            else mma<DT>(acc[i][nb], wr[nb][ks], af[i]);
                        }
                }
            };
            if (half) steps(Int<1>());
            else steps(Int<2>());
        } else {
            const unsigned char *wbuf = halo_raw + woff;
            const unsigned char *blk[BPW];
#pragma unroll
            for (int i = 0; i < BPW; ++i) blk[i] = wbuf + pbb[i];
#pragma unroll
            for (int ks = 0; ks < KSM; ++ks) {
                if (ks < KS) {
                    u32x4 af[BPW][SPL];
#pragma unroll
                    for (int i = 0; i < BPW; ++i)
#pragma unroll
                        for (int j = 0; j < SPL; ++j) af[i][j] = *reinterpret_cast<const u32x4 *>(blk[i] + toffb[ks][j]);
#pragma unroll
                    for (int i = 0; i < BPW; ++i)
#pragma unroll
                        for (int nb = 0; nb < NBP; ++nb) {
                            if constexpr (POOL) mma<DT>(acc[i][nb], af[i], wr[nb][ks]);
                            else mma<DT>(acc[i][nb], wr[nb][ks], af[i]);
                        }
                }
            }
        }

        // epilogue: bias, activation, [residual], [2x2 max], round, NHWC store.
        // Stores go through a buffer resource the size of the image's output: an
        // element past the right edge or the channels gets an offset past it,
        // which the store drops, so every wave issues a number it can count.
        unsigned char *yimg = reinterpret_cast<unsigned char *>(a.y) + (size_t)n * img * ES;
        const unsigned char *rimg = a.res ? reinterpret_cast<const unsigned char *>(a.res) + (size_t)n * img * ES : nullptr;
        const __amdgpu_buffer_rsrc_t ry = __builtin_amdgcn_make_buffer_rsrc((void *)yimg, (short)0, (int)(img * ES), 0x00020000);
        int stores = 0;
        if constexpr (POOL) {
            const __amdgpu_buffer_rsrc_t ram = __builtin_amdgcn_make_buffer_rsrc(
                AM ? (void *)(a.argmax + (size_t)n * img) : nullptr, (short)0, AM ? (int)img : 0, 0x00020000);
#pragma unroll
            for (int nb = 0; nb < NBP; ++nb) {
                const int col = (wg * NBP + nb) * 16 + lrow;
                // blocks i (row 2k) and i + 2 (row 2k + 1) of the same column
                // half: lane column pairs (4*lgrp + 2j, + 1) are the windows.
                // The store offset is a wave-uniform part (window row, the
                // block's first window) plus a lane part.
#pragma unroll
                for (int i = 0; i < BPW; ++i) {
                    if (i & 2) continue;
                    if ((i & 1) && half) continue;  // wave-uniform
                    const int hp = (th0 + h2_row(wq, RPW, i)) >> 1;
                    if (hp >= Hp) continue;  // wave-uniform
                    const int wpb = (tw0 + 16 * (i & 1)) >> 1;
                    const int soff = (hp * Wp + wpb) * a.cout_p;
#pragma unroll
                    for (int j = 0; j < 2; ++j) {
                        const float w4[4] = {acc[i][nb][2 * j], acc[i][nb][2 * j + 1], acc[i + 2][nb][2 * j],
                                             acc[i + 2][nb][2 * j + 1]};
                        const float mx = fmaxf(fmaxf(w4[0], w4[1]), fmaxf(w4[2], w4[3]));
                        float o = activate_sel(mx * scl[nb][0] + bias[nb][0], lsl);
                        if constexpr (DT == FP8) o *= a.out_inv_scale;  // 1 for the other types
                        const bool ok = wpb + 2 * lgrp + j < Wp && col < a.cout_p;
                        const int loff = (2 * lgrp + j) * a.cout_p + col;
                        const int voff = ok ? loff * ES : (int)DN_OOB;
                        if constexpr (DT == F32) __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(o), ry, voff, soff * ES, 0);
                        else if constexpr (DT == BF16) __builtin_amdgcn_raw_buffer_store_b16(f2bf(o), ry, voff, soff * ES, 0);
                        else __builtin_amdgcn_raw_buffer_store_b8(f2e4m3(o), ry, voff, soff * ES, 0);
                        if constexpr (AM)
                            __builtin_amdgcn_raw_buffer_store_b8(
                                window_argmax<DT>(w4, scl[nb][0], bias[nb][0], a.act, a.slope, a.out_inv_scale), ram,
                                ok ? loff : (int)DN_OOB, soff, 0);
                    }
                    stores += AM ? 4 : 2;
                }
            }
        } else {
#pragma unroll
            for (int nb = 0; nb < NBP; ++nb) {
                const int ch = (wg * NBP + nb) * 16 + 4 * lgrp;  // cout_p is a multiple of 4
#pragma unroll
                for (int i = 0; i < BPW; ++i) {
                    const int ho = th0 + h2_row(wq, RPW, i);
                    if (ho >= a.Ho || ((i & 1) && half)) continue;  // wave-uniform
                    const int wob = tw0 + 16 * (i & 1);
                    const int soff = (ho * a.Wo + wob) * a.cout_p;
                    const bool ok = wob + lrow < a.Wo && ch < a.cout_p;
                    const int loff = lrow * a.cout_p + ch;
                    float v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) v[q] = activate_sel(acc[i][nb][q] * scl[nb][q] + bias[nb][q], lsl);
                    if (rimg) {
                        float r[4] = {0.0f, 0.0f, 0.0f, 0.0f};
                        if (ok) load4<DT>(rimg, (size_t)soff + loff, r);
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] += r[q] * a.res_scale;
                    }
                    if constexpr (DT == FP8) {
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[q] *= a.out_inv_scale;
                    }
                    const int voff = ok ? loff * ES : (int)DN_OOB;
                    if constexpr (DT == F32) {
                        __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(v[0]), __float_as_uint(v[1]), __float_as_uint(v[2]), __float_as_uint(v[3])}, ry, voff, soff * ES, 0);
                    } else if constexpr (DT == BF16) {
                        __builtin_amdgcn_raw_buffer_store_b64(u32x2{(unsigned)f2bf(v[0]) | ((unsigned)f2bf(v[1]) << 16), (unsigned)f2bf(v[2]) | ((unsigned)f2bf(v[3]) << 16)}, ry, voff, soff * ES, 0);
                    } else {
                        __builtin_amdgcn_raw_buffer_store_b32((unsigned)f2e4m3(v[0]) | ((unsigned)f2e4m3(v[1]) << 8) | ((unsigned)f2e4m3(v[2]) << 16) | ((unsigned)f2e4m3(v[3]) << 24), ry, voff, soff * ES, 0);
                    }
                    ++stores;
                }
            }
        }
        st3 = st2;
        st2 = st1;
        st1 = stores;
        next(cur);
        cbuf = cbuf + 1 == nbuf ? 0 : cbuf + 1;
    }
}

constexpr size_t H2_LDS_MAX = 76 * 1024;  // two workgroups per CU

// Window slots (16 bytes) of one LDS buffer of the persistent halo kernel at
// the tile of nb 16-channel blocks.
static int halo2_wslots(int dt, const ConvArgs &a, int nb)
{
    const int th = h2_th(nb);
    const int lh = (th - 1) * a.stride + a.R, lw = (HT_W - 1) * a.stride + a.S;
    return h2_wslots(lh, lw, a.cin_p / seg_el(dt));
}

// The 16-channel blocks a layer runs with: its own, or four, the last ones
// empty, in BF16 with three blocks or where two windows of the 16-row tiles do
// not fit.
static int halo2_blocks(int dt, const ConvArgs &a)
{
    const int nb = (a.cout_p + 15) / 16;
    const bool four = dt == BF16 && (nb == 3 || (nb < 3 && 2 * (size_t)halo2_wslots(dt, a, nb) * 16 > H2_LDS_MAX));
    return four ? 4 : nb;
}

// Window buffers: as many as fit (up to 4), at least 2.
static int halo2_nbuf(size_t per)
{
    int nb = 4;
    while (nb > 2 && nb * per > H2_LDS_MAX) --nb;
    return nb;
}

bool halo2_ok(int dt, const ConvArgs &a, bool as_four)
{
    const int kstep = dt == FP8 ? 128 : (dt == BF16 ? 32 : 16);
    const int K = a.R * a.S * a.cin_p;
    const int nb = as_four ? halo2_blocks(dt, a) : (a.cout_p + 15) / 16;
    const int ws = halo2_wslots(dt, a, nb);
    return kblock_ch(dt, a.cin_p, a.R * a.S) == a.cin_p && nb <= 4 && nb != 3 && (K + kstep - 1) / kstep <= h2_ksmax(dt) &&
           a.stride <= 2 && (size_t)a.Ho * a.Wo * a.cout_p * esize(dt) < (1u << 31) &&
           (size_t)a.H * a.W * a.cin_p * esize(dt) < (1u << 31) && ws / 64 <= 4 * H2_MAXBLK &&
           2 * (size_t)ws * 16 <= H2_LDS_MAX;
}

// The instance for a shape: CPS of those with the window's layout built in, or 0.
static int halo2_fix(int dt, const ConvArgs &a)
{
    const bool fix = dt == BF16 && a.R == 3 && a.S == 3 && a.stride == 1 &&
                     (size_t)(a.H + a.pad + 64) * a.W * a.cin_p * esize(dt) < (1u << 30);
    return fix && (a.cin_p == 16 || a.cin_p == 32) ? a.cin_p / seg_el(BF16) : 0;
}

long halo2_tiles(int dt, const ConvArgs &a, bool *fixed)
{
    const int th = h2_th(halo2_blocks(dt, a));
    if (fixed) *fixed = halo2_fix(dt, a) != 0;
    return (long)a.batch * ((a.Ho + th - 1) / th) * ((a.Wo + HT_W - 1) / HT_W);
}

template <int DT, bool POOL, bool AM, int CPS>
static hipError_t go_halo2(const ConvArgs &a, int grid, int nbuf, size_t lds, hipStream_t s)
{
    const int nb = halo2_blocks(DT, a);
    if constexpr (CPS != 4) {  // two windows of 18 x 34 pixels of 4 chunks are past H2_LDS_MAX
        switch (nb) {
        case 1: allow_lds(conv_halo2<DT, POOL, 1, AM, CPS>, lds); hipLaunchKernelGGL((conv_halo2<DT, POOL, 1, AM, CPS>), dim3(grid), dim3(256), lds, s, a, nbuf); return hipGetLastError();
        case 2: allow_lds(conv_halo2<DT, POOL, 2, AM, CPS>, lds); hipLaunchKernelGGL((conv_halo2<DT, POOL, 2, AM, CPS>), dim3(grid), dim3(256), lds, s, a, nbuf); return hipGetLastError();
        default: break;
        }
    }
    if (nb != 4) return hipErrorInvalidValue;
    allow_lds(conv_halo2<DT, POOL, 4, AM, CPS>, lds);
    hipLaunchKernelGGL((conv_halo2<DT, POOL, 4, AM, CPS>), dim3(grid), dim3(256), lds, s, a, nbuf);
    return hipGetLastError();
}

// BF16 3x3 stride-1 layers of 16 and 32 channels, the shapes in use, run the
// instances with the window's layout built in (images below 1 GB, padding below
// them included: their transfers mark dead slots by an offset past that).  The general form issues
// 535 vector instructions a wave and tile besides the MFMAs, more than the
// MFMAs take: tile positions divided out (150), window addresses (84), fragment
// addresses (72).  64 images of 104 x 104 x 32 -> 64 channels, pooled: 38.5 us
// before, 30 with these, 28.4 with window rows read once (32 channels), 28.1 with
// the empty column halves left out.
template <int DT, bool POOL, bool AM>
static hipError_t go_halo2(const ConvArgs &a, int grid, int nbuf, size_t lds, hipStream_t s)
{
    if constexpr (DT == BF16) {
        const int cps = halo2_fix(DT, a);
        if (cps == 2) return go_halo2<DT, POOL, AM, 2>(a, grid, nbuf, lds, s);
        if (cps == 4) return go_halo2<DT, POOL, AM, 4>(a, grid, nbuf, lds, s);
    }
    return go_halo2<DT, POOL, AM, 0>(a, grid, nbuf, lds, s);
}

template <int DT>
static hipError_t go_halo2_dt(const ConvArgs &a, int grid, int nbuf, size_t lds, hipStream_t s)
{
    if constexpr (DT != FP8) {
        if (a.pool && a.argmax) return go_halo2<DT, true, true>(a, grid, nbuf, lds, s);
    }
    return a.pool ? go_halo2<DT, true, false>(a, grid, nbuf, lds, s) : go_halo2<DT, false, false>(a, grid, nbuf, lds, s);
}

hipError_t launch_conv_halo2(int dt, const ConvArgs &a, hipStream_t s)
{
    if (!halo2_ok(dt, a, true)) return hipErrorInvalidValue;
    const long tiles = halo2_tiles(dt, a, nullptr);
    const size_t per = (size_t)halo2_wslots(dt, a, halo2_blocks(dt, a)) * 16;
    const int nbuf = halo2_nbuf(per);
    const size_t lds = nbuf * per;
    // two workgroups per CU, a multiple of 8 (the tile runs are per XCD)
    const long want = std::min<long>(tiles, 512L);
    const int grid = (int)std::max<long>(8, (want + 7) / 8 * 8);
    switch (dt) {
    case F32: return go_halo2_dt<F32>(a, grid, nbuf, lds, s);
    case BF16: return go_halo2_dt<BF16>(a, grid, nbuf, lds, s);
    case FP8: return go_halo2_dt<FP8>(a, grid, nbuf, lds, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace dnk
