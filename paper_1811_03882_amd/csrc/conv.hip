// Implicit-GEMM convolution for gfx950 (CDNA4) with a fused epilogue.
//
// GEMM view (M = batch*Ho*Wo output pixels, N = output channels,
// K = R*S*Cin_pad):  Y[m][j] = sum_k A[m][k] * B[k][j].
// A is never materialised: each 128-byte K-slice of an A row is gathered from
// the NHWC input as eight 16-byte segments, each lying inside one filter tap
// (r, s) because channels are padded to 16 bytes, and staged in LDS.  The K
// order is k = (cb*R*S + r*S + s)*CB + ci (c = cb*CB + ci, CB = kblock_ch()):
// tap-major for narrow layers, channel-block-major for wide ones.  B is the
// packed weight matrix [cout_p][k_pad] (K contiguous).  Products run on MFMA
// with FP32 accumulation:
//   FP32  v_mfma_f32_16x16x4_f32        (4 issues per 16-wide K step)
//   BF16  v_mfma_f32_16x16x32_bf16
//   FP8   v_mfma_f32_16x16x128_f8f6f4   (OCP e4m3 operands)
// Every lane supplies its row (A) / column (B) of a 16x16 block with the same
// K subset for both operands, so each dot product covers every k once.
//
// Epilogue (per output element, FP32): acc * (FP8 weight scale * input scale)
// + folded bias -> leaky or linear -> [+ residual] -> [max over the four rows
// of a 2x2 pooling window] -> round to the storage type -> NHWC store.
// Pooling after the activation and after rounding are both exact because the
// activation and the rounding are monotone non-decreasing.
#include <algorithm>
#include <type_traits>

#include "conv_dev.h"

namespace dnk {

// Separate split-K finish: one thread per output group.
template <int DT>
__global__ void __launch_bounds__(256) splitk_reduce(ConvArgs a)
{
    const size_t rows = a.pool ? (size_t)(a.M >> 2) : (size_t)a.M;
    const int cq = a.cout_p >> 2;
    const size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= rows * cq) return;
    splitk_finish4<DT>(a, idx / cq, (int)(idx % cq) * 4);
}

// Position of one lane's 16-byte K segment in the packed K order, advanced
// K-tile by K-tile (a workgroup loads its K-tiles in increasing order): the
// filter tap (r, s) and input channel c0 of k = kt*BKE + sc*SEG, with the
// divisions done once at the first K-tile instead of at every one.
// Tap-major order: k = tap*cin_p + c.  Channel-block-major (cbsh >= 0):
// blocks of CB = 2^cbsh channels, every tap of a block before the next block;
// a K-tile lies inside one block (BKE divides CB).  The segment is inside K
// when r < R and c0 < cin_p.
struct KPos {
    int r, s, c0, off, cbase;  // off, cbase: offset in and start of the channel block
    __device__ __forceinline__ void init(int k0, int cin_p, int RS, int S, int cbsh)
    {
        int tap;
        if (cbsh < 0) {
            tap = k0 / cin_p;
            c0 = k0 - tap * cin_p;
            off = cbase = 0;
        } else {
            const int blk = k0 >> cbsh, cb = blk / RS;
            tap = blk - cb * RS;
            cbase = cb << cbsh;
            off = k0 & ((1 << cbsh) - 1);
            c0 = cbase + off;
        }
        r = tap / S;
        s = tap - r * S;
    }
    __device__ __forceinline__ void next(int bke, int cin_p, int R, int S, int cbsh)
    {
        if (cbsh < 0) {
            c0 += bke;
            while (c0 >= cin_p) {
                c0 -= cin_p;
                if (++s == S) { s = 0; ++r; }
            }
        } else {
            off += bke;
            if (off >= (1 << cbsh)) {
                off -= 1 << cbsh;
                if (++s == S) {
                    s = 0;
                    if (++r == R) { r = 0; cbase += 1 << cbsh; }
                }
            }
            c0 = cbase + off;
        }
    }
};

template <int DT, int BM, int BN, int WM, int WN>
__global__ void __launch_bounds__(64 * WM * WN) conv_igemm(ConvArgs a)
{
    constexpr int NT = 64 * WM * WN;
    constexpr int ES = esize(DT), SEG = seg_el(DT), BKE = bk_el(DT);
    constexpr int RSTEP = NT / 8;                       // rows covered per load pass
    constexpr int AR = BM / RSTEP;                      // A rows per thread
    constexpr int BR = (BN + RSTEP - 1) / RSTEP;        // B rows per thread
    constexpr int WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
    constexpr int SPL = Tr<DT>::SPL, KSPT = Tr<DT>::KSPT;
    static_assert(BM % RSTEP == 0 && WTM % 16 == 0 && WTN % 16 == 0, "tile shape");

    __shared__ u32x4 sA[2][BM * 8];
    __shared__ u32x4 sB[2][BN * 8];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM;

    const int ntn = (a.cout_p + BN - 1) / BN;
    const int logical = xcd_remap(blockIdx.x, gridDim.x);
    int mi, ni;
    tile_mn(logical, gridDim.x / ntn, ntn, mi, ni);
    const int m0 = mi * BM, n0 = ni * BN;

    // ---- per-row gather state for A (fixed for the whole K loop)
    const int sc = tid & 7;
    const int rbase = tid >> 3;
    int a_pix[AR], a_hi[AR], a_wi[AR];
#pragma unroll
    for (int i = 0; i < AR; ++i) {
        const int m = m0 + rbase + i * RSTEP;
        a_pix[i] = 0; a_hi[i] = -(1 << 28); a_wi[i] = 0;
        if (m < a.M) {
            int n, ho, wo;
            if (a.pool) {
                const int q = m & 3, win = m >> 2, wp2 = a.Wo >> 1, hp2 = a.Ho >> 1;
                const int wp = win % wp2, t = win / wp2;
                ho = 2 * (t % hp2) + (q >> 1); wo = 2 * wp + (q & 1); n = t / hp2;
            } else {
                wo = m % a.Wo; const int t = m / a.Wo; ho = t % a.Ho; n = t / a.Ho;
            }
            a_pix[i] = n * a.H * a.W;
            a_hi[i] = ho * a.stride - a.pad;
            a_wi[i] = wo * a.stride - a.pad;
        }
    }
    bool b_ok[BR];
    size_t b_off[BR];
#pragma unroll
    for (int i = 0; i < BR; ++i) {
        const int row = rbase + i * RSTEP, n = n0 + row;
        b_ok[i] = row < BN && n < a.cout_p;
        b_off[i] = ((size_t)(b_ok[i] ? n : 0) * a.k_pad + sc * SEG) * ES;
    }

    const int nkt = a.k_pad / BKE;
    const int kt0 = blockIdx.z * a.ktiles_per_split;
    const int kt1 = min(nkt, kt0 + a.ktiles_per_split);
    const int RS = a.R * a.S;
    const int cbsh = kblock_ch(DT, a.cin_p, RS) == a.cin_p ? -1 : 7 - (ES >> 1);  // log2 of a 128-byte block
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    KPos kp;
    kp.init(kt0 * BKE + sc * SEG, a.cin_p, RS, a.S, cbsh);
    long long a_base[AR];  // element offset of each row's tap (0, 0), channel 0 (meaningful where in range)
#pragma unroll
    for (int i = 0; i < AR; ++i) a_base[i] = ((long long)a_pix[i] + (long long)a_hi[i] * a.W + a_wi[i]) * a.cin_p;

    u32x4 ra[AR], rb[BR];
    f4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

    const int lrow = lane & 15, lgrp = lane >> 4;

// Issue the global loads of K-tile KT into ra / rb (no wait).  KT must be the
// K-tile after the previous call's (kp advances one K-tile per call).
#define DN_GLOAD(KT)                                                                           \
    do {                                                                                       \
        const int r_ = kp.r, s_ = kp.s;                                                        \
        const bool kv_ = r_ < a.R && kp.c0 < a.cin_p;                                          \
        const long long toff_ = ((long long)r_ * a.W + s_) * a.cin_p + kp.c0;                  \
        _Pragma("unroll") for (int i = 0; i < AR; ++i) {                                       \
            const int hi_ = a_hi[i] + r_, wi_ = a_wi[i] + s_;                                  \
            const bool ok_ = kv_ && (unsigned)hi_ < (unsigned)a.H && (unsigned)wi_ < (unsigned)a.W; \
            const size_t off_ = ok_ ? (size_t)(a_base[i] + toff_) * ES : 0;                    \
            ra[i] = ok_ ? gload16(a.x, off_) : zero4;                                          \
        }                                                                                      \
        const size_t kb_ = (size_t)(KT) * BKE * ES;                                            \
        _Pragma("unroll") for (int i = 0; i < BR; ++i)                                         \
            rb[i] = b_ok[i] ? gload16(a.w, b_off[i] + kb_) : zero4;                            \
        kp.next(BKE, a.cin_p, a.R, a.S, cbsh);                                                 \
    } while (0)

// Write ra / rb into LDS stage BUF (rows swizzled: segment s of row r sits at s ^ (r & 7)).
#define DN_SSTORE(BUF)                                                                         \
    do {                                                                                       \
        _Pragma("unroll") for (int i = 0; i < AR; ++i) {                                       \
            const int row_ = rbase + i * RSTEP;                                                \
            sA[BUF][row_ * 8 + (sc ^ (row_ & 7))] = ra[i];                                     \
        }                                                                                      \
        _Pragma("unroll") for (int i = 0; i < BR; ++i) {                                       \
            const int row_ = rbase + i * RSTEP;                                                \
            if (row_ < BN) sB[BUF][row_ * 8 + (sc ^ (row_ & 7))] = rb[i];                      \
        }                                                                                      \
    } while (0)

    if (kt0 < kt1) {
        DN_GLOAD(kt0);
        DN_SSTORE(0);
    }
    __syncthreads();
    for (int kt = kt0; kt < kt1; ++kt) {
        const int buf = (kt - kt0) & 1;
        const bool more = kt + 1 < kt1;
        if (more) DN_GLOAD(kt + 1);
#pragma unroll
        for (int ks = 0; ks < KSPT; ++ks) {
            u32x4 af[FM][SPL], bfr[FN][SPL];
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) {
                const int row = wm * WTM + fm * 16 + lrow;
#pragma unroll
                for (int j = 0; j < SPL; ++j) {
                    const int seg = ks * 4 * SPL + lgrp * SPL + j;
                    af[fm][j] = sA[buf][row * 8 + (seg ^ (row & 7))];
                }
            }
#pragma unroll
            for (int fn = 0; fn < FN; ++fn) {
                const int row = wn * WTN + fn * 16 + lrow;
#pragma unroll
                for (int j = 0; j < SPL; ++j) {
                    const int seg = ks * 4 * SPL + lgrp * SPL + j;
                    bfr[fn][j] = sB[buf][row * 8 + (seg ^ (row & 7))];
                }
            }
#pragma unroll
            for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                for (int fn = 0; fn < FN; ++fn) mma<DT>(acc[fm][fn], af[fm], bfr[fn]);
        }
        // keep the LDS stores of the next tile behind this tile's MFMAs, so the
        // wait for its global loads overlaps the matrix work
        __builtin_amdgcn_sched_barrier(0);
        if (more) DN_SSTORE(buf ^ 1);
        __syncthreads();
    }
#undef DN_GLOAD
#undef DN_SSTORE

    conv_epilogue<DT, FM, FN>(a, acc, m0 + wm * WTM + 4 * lgrp, n0 + wn * WTN + lrow);
    if (a.splits > 1 && a.tile_count) splitk_tail<DT, BM, BN, NT>(a, m0, n0, sA);
}

// ---------------------------------------------------------------- LDS-DMA variant
// Same GEMM, but the K-tiles travel global -> LDS directly
// (buffer_load_dwordx4 ... lds: lane L of a wave instruction writes bytes
// [16L, 16L + 16) of a 1 KB LDS block, i.e. row L/8, physical segment L%8 of
// an 8-row group).  No VGPR staging, so NS-1 K-tiles can be in flight while
// one is multiplied.  Out-of-range taps and rows use an offset past the
// buffer's size, for which the buffer load returns zeros.
// SPR = 16-byte segments per LDS row (8: 128-byte K-tile, 4: 64-byte K-tile,
// which halves a stage so that four stages of a 256x256 tile fit in LDS).
// Row r stores logical segment s at physical segment s ^ swz(r); swz makes
// the 16 lanes of an MFMA fragment read hit distinct banks.
template <int SPR> __device__ __forceinline__ int seg_swz(int row)
{
    return SPR == 8 ? (row & 7) : ((row >> 2) & 3);
}

// MF = 16: 16x16 MFMA blocks (every dtype); MF = 32: 32x32x16 BF16 blocks,
// which take twice the passes of a 16x16x32 block for twice the products
// (the same rate) but read each 1 KB operand fragment for twice the work, so
// a tile needs half the LDS reads per product.  A 32x32 fragment: lane l holds row l%32 and K
// elements [8*(l/32), 8*(l/32) + 8) of the 16-element step, i.e. one 16-byte
// segment; the result quad q of a lane covers rows 8q + 4*(l/32) + (0..3).
template <int DT, int BM, int BN, int WM, int WN, int NS, int SPR, int MF = 16>
__global__ void __launch_bounds__(64 * WM * WN) conv_igemm_dl(ConvArgs a)
{
    constexpr int NW = WM * WN;
    constexpr int ES = esize(DT), SEG = seg_el(DT);
    constexpr int BKE = SPR * SEG;                      // K elements per tile
    constexpr int RPI = 64 / SPR;                       // rows filled by one wave-wide transfer
    constexpr int RSTEP = RPI * NW;
    constexpr int AGRP = BM / RPI, BGRP = BN / RPI;     // row groups (one transfer each) per tile
    constexpr int AR = (AGRP + NW - 1) / NW, BR = (BGRP + NW - 1) / NW;  // transfers per wave (max)
    constexpr int LPT = AR + BR;
    constexpr int WTM = BM / WM, WTN = BN / WN, FM = WTM / MF, FN = WTN / MF;
    constexpr int SPL = Tr<DT>::SPL;
    constexpr int KSPT = MF == 16 ? SPR / (4 * SPL) : SPR / 2;  // MFMA K-steps per tile
    static_assert(MF == 16 || (MF == 32 && DT == BF16), "32x32 blocks are BF16 only");
    static_assert(KSPT >= 1 && (MF == 32 || KSPT * 4 * SPL == SPR), "K-tile / MFMA step mismatch");
    static_assert(BM % RPI == 0 && BN % RPI == 0 && WTM % MF == 0 && WTN % MF == 0, "tile shape");
    typedef std::conditional_t<MF == 16, f4, f16v> accT;
    static_assert(NS >= 2 && NS <= 4 && LPT * (NS - 2) < 64, "pipeline depth");

    __shared__ u32x4 sA[NS][BM * SPR];
    __shared__ u32x4 sB[NS][BN * SPR];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave % WM, wn = wave / WM;
    const int ntn = (a.cout_p + BN - 1) / BN;
    const int logical = xcd_remap(blockIdx.x, gridDim.x);
    int mi, ni;
    tile_mn(logical, gridDim.x / ntn, ntn, mi, ni);
    const int m0 = mi * BM, n0 = ni * BN;
    // transfers this wave issues per K-tile (waves share the row groups round-robin)
    const int my_a = (AGRP - wave + NW - 1) / NW, my_b = (BGRP - wave + NW - 1) / NW;
    const int my_lpt = my_a + my_b;

    // lane L of a transfer fills row L/SPR, physical segment L%SPR of its row
    // group; with the swizzle that is the logical segment below
    const int rbase = wave * RPI + lane / SPR;          // this lane's row in the wave's first group
    const int sc = (lane % SPR) ^ seg_swz<SPR>(rbase);
    int a_pix[AR], a_hi[AR], a_wi[AR];
#pragma unroll
    for (int i = 0; i < AR; ++i) {
        const int m = m0 + rbase + i * RSTEP;
        a_pix[i] = 0; a_hi[i] = -(1 << 28); a_wi[i] = 0;
        if (m < a.M) {
            int n, ho, wo;
            if (a.pool) {
                const int q = m & 3, win = m >> 2, wp2 = a.Wo >> 1, hp2 = a.Ho >> 1;
                const int wp = win % wp2, t = win / wp2;
                ho = 2 * (t % hp2) + (q >> 1); wo = 2 * wp + (q & 1); n = t / hp2;
            } else {
                wo = m % a.Wo; const int t = m / a.Wo; ho = t % a.Ho; n = t / a.Ho;
            }
            a_pix[i] = n * a.H * a.W;
            a_hi[i] = ho * a.stride - a.pad;
            a_wi[i] = wo * a.stride - a.pad;
        }
    }
    unsigned b_off[BR];
#pragma unroll
    for (int i = 0; i < BR; ++i) {
        const int n = n0 + rbase + i * RSTEP;
        b_off[i] = n < a.cout_p ? (unsigned)(((size_t)n * a.k_pad + sc * SEG) * ES) : DN_OOB;
    }
    const i32x4 rx = make_rsrc(a.x, a.x_bytes);
    const i32x4 rw = make_rsrc(a.w, a.w_bytes);

    const int nkt = a.k_pad / BKE;
    const int tpk = bk_el(DT) / BKE;                    // tiles per 128-byte split-K unit
    const int kt0 = blockIdx.z * a.ktiles_per_split * tpk;
    const int kt1 = min(nkt, kt0 + a.ktiles_per_split * tpk);
    const int RS = a.R * a.S;
    // channel-block-major K order uses a power-of-two block (32 / 64 / 128 channels)
    const int cbsh = kblock_ch(DT, a.cin_p, RS) == a.cin_p ? -1 : 7 - (ES >> 1);
    KPos kp;  // this lane's K segment of the next K-tile to issue (issued in increasing order)
    kp.init(kt0 * BKE + sc * SEG, a.cin_p, RS, a.S, cbsh);
    long long a_base[AR];  // element offset of each row's tap (0, 0), channel 0 (meaningful where in range)
#pragma unroll
    for (int i = 0; i < AR; ++i) a_base[i] = ((long long)a_pix[i] + (long long)a_hi[i] * a.W + a_wi[i]) * a.cin_p;

    auto issue = [&](int kt, int st) {
        const int r = kp.r, s = kp.s;
        const bool kv = r < a.R && kp.c0 < a.cin_p;
        const long long toff = ((long long)r * a.W + s) * a.cin_p + kp.c0;
#pragma unroll
        for (int i = 0; i < AR; ++i) {
            if (AGRP % NW != 0 && i == AR - 1 && i >= my_a) break;  // wave-uniform
            const int hi = a_hi[i] + r, wi = a_wi[i] + s;
            const bool ok = kv && (unsigned)hi < (unsigned)a.H && (unsigned)wi < (unsigned)a.W;
            const unsigned off = ok ? (unsigned)((a_base[i] + toff) * ES) : DN_OOB;
            dma16(rx, off, &sA[st][(wave + i * NW) * 64]);
        }
        const unsigned kb = (unsigned)(kt * BKE * ES);
#pragma unroll
        for (int i = 0; i < BR; ++i) {
            if (BGRP % NW != 0 && i == BR - 1 && i >= my_b) break;  // wave-uniform
            const unsigned off = b_off[i] == DN_OOB ? DN_OOB : b_off[i] + kb;
            dma16(rw, off, &sB[st][(wave + i * NW) * 64]);
        }
        kp.next(BKE, a.cin_p, a.R, a.S, cbsh);
    };

    accT acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = accT{};
    const int lrow = lane & 15, lgrp = lane >> 4;

#pragma unroll
    for (int st = 0; st < NS - 1; ++st)
        if (kt0 + st < kt1) issue(kt0 + st, st);

    int cs = 0;  // stage holding tile kt
    for (int kt = kt0; kt < kt1; ++kt) {
        // this wave's transfers of tile kt landed; later tiles may stay in flight
        const int after = min(NS - 2, kt1 - 1 - kt);  // tiles issued after kt so far
        if (after == 0) wait_vm<0>();
        else if (my_lpt == LPT) { if (after >= 2) wait_vm<LPT * 2>(); else wait_vm<LPT>(); }
        else if (my_lpt == LPT - 1) { if (after >= 2) wait_vm<(LPT - 1) * 2>(); else wait_vm<LPT - 1>(); }
        else { if (after >= 2) wait_vm<(LPT > 1 ? LPT - 2 : 0) * 2>(); else wait_vm<(LPT > 1 ? LPT - 2 : 0)>(); }
        lds_barrier();  // every wave's transfers landed; every wave is done with tile kt-1
        if (kt + NS - 1 < kt1) issue(kt + NS - 1, cs == 0 ? NS - 1 : cs - 1);
        if constexpr (MF == 32) {
            const int r32 = lane & 31, h = lane >> 5;
#pragma unroll
            for (int ks = 0; ks < KSPT; ++ks) {
                const int seg = ks * 2 + h;
                u32x4 af[FM], bfr[FN];
#pragma unroll
                for (int fm = 0; fm < FM; ++fm) {
                    const int row = wm * WTM + fm * 32 + r32;
                    af[fm] = sA[cs][row * SPR + (seg ^ seg_swz<SPR>(row))];
                }
#pragma unroll
                for (int fn = 0; fn < FN; ++fn) {
                    const int row = wn * WTN + fn * 32 + r32;
                    bfr[fn] = sB[cs][row * SPR + (seg ^ seg_swz<SPR>(row))];
                }
#pragma unroll
                for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                    for (int fn = 0; fn < FN; ++fn)
                        acc[fm][fn] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, af[fm]),
                                                                             __builtin_bit_cast(bf16x8, bfr[fn]),
                                                                             acc[fm][fn], 0, 0, 0);
            }
        } else {
#pragma unroll
        for (int ks = 0; ks < KSPT; ++ks) {
            u32x4 af[FM][SPL], bfr[FN][SPL];
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) {
                const int row = wm * WTM + fm * 16 + lrow;
#pragma unroll
                for (int j = 0; j < SPL; ++j) {
                    const int seg = ks * 4 * SPL + lgrp * SPL + j;
                    af[fm][j] = sA[cs][row * SPR + (seg ^ seg_swz<SPR>(row))];
                }
            }
#pragma unroll
            for (int fn = 0; fn < FN; ++fn) {
                const int row = wn * WTN + fn * 16 + lrow;
#pragma unroll
                for (int j = 0; j < SPL; ++j) {
                    const int seg = ks * 4 * SPL + lgrp * SPL + j;
                    bfr[fn][j] = sB[cs][row * SPR + (seg ^ seg_swz<SPR>(row))];
                }
            }
#pragma unroll
            for (int fm = 0; fm < FM; ++fm)
#pragma unroll
                for (int fn = 0; fn < FN; ++fn) mma<DT>(acc[fm][fn], af[fm], bfr[fn]);
        }
        }
        cs = cs + 1 == NS ? 0 : cs + 1;
    }
    if constexpr (MF == 32) {
        f4 q4[FM * 4][FN];
#pragma unroll
        for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int fn = 0; fn < FN; ++fn)
                    q4[fm * 4 + q][fn] = f4{acc[fm][fn][4 * q], acc[fm][fn][4 * q + 1], acc[fm][fn][4 * q + 2], acc[fm][fn][4 * q + 3]};
        conv_epilogue<DT, FM * 4, FN, 8, 32>(a, q4, m0 + wm * WTM + 4 * (lane >> 5), n0 + wn * WTN + (lane & 31));
    } else {
        conv_epilogue<DT, FM, FN>(a, acc, m0 + wm * WTM + 4 * lgrp, n0 + wn * WTN + lrow);
    }
    if (a.splits > 1 && a.tile_count) splitk_tail<DT, BM, BN, 64 * NW>(a, m0, n0, sA);
}

// ---------------------------------------------------------------- dispatch

static const TileCfg kTiles[] = {
    {64, 64, 2, 2},    // 0
    {128, 64, 2, 2},   // 1
    {128, 128, 2, 2},  // 2
    {256, 128, 2, 2},  // 3
    {256, 256, 2, 4},  // 4
    {128, 256, 2, 4},  // 5
    {256, 16, 4, 1},   // 6
    {256, 32, 4, 1},   // 7
    {64, 128, 1, 4},   // 8
    {64, 32, 2, 2},    // 9
    {256, 256, 2, 2},  // 10: 4 waves of 128x128
    {192, 256, 1, 4},  // 11: 57 M-tiles x 4 for M = 64*169
    {128, 256, 1, 4},  // 12
    // LDS-DMA pipeline variants (bm, bn, waves_m, waves_n; stages in dispatch)
    {256, 128, 2, 2},  // 13: 3 stages
    {128, 128, 2, 2},  // 14: 4 stages
    {256, 256, 2, 4},  // 15: 2 stages
    {192, 256, 1, 4},  // 16: 2 stages
    {128, 256, 2, 4},  // 17: 3 stages
    {256, 128, 2, 4},  // 18: 3 stages, 8 waves
    // 64-byte K-tiles (FP32 / BF16; FP8 falls back to 128-byte tiles)
    {256, 256, 2, 4},  // 19: 4 stages, 8 waves
    {192, 256, 1, 4},  // 20: 4 stages
    {128, 256, 2, 4},  // 21: 4 stages, 8 waves
    {256, 128, 2, 2},  // 22: 4 stages
    // 31 x 8 = 248 tiles for M = 64*169, N = 1024 (one round on 256 CUs)
    {352, 128, 2, 4},  // 23: 2 stages, 8 waves
    {352, 128, 2, 2},  // 24: 2 stages, 4 waves
    {352, 128, 2, 8},  // 25: 2 stages, 16 waves (4 per SIMD)
    {256, 256, 2, 8},  // 26: 2 stages, 16 waves
    // 32x32x16 BF16 blocks (other dtypes run the same tile with 16x16 blocks)
    {384, 128, 4, 2, 32},  // 27: 29 x 8 = 232 tiles for M = 64*169; 2 stages, 8 waves of 96x64
    {384, 128, 4, 4, 32},  // 28: 2 stages, 16 waves of 96x32
    {256, 256, 2, 4, 32},  // 29: 2 stages, 8 waves of 128x64
    {256, 256, 4, 4, 32},  // 30: 2 stages, 16 waves of 64x64
    {256, 128, 4, 2, 32},  // 31: 3 stages, 8 waves of 64x64
    {128, 128, 2, 2, 32},  // 32: 4 stages, 4 waves of 64x64
    {352, 128, 11, 1, 32}, // 33: 2 stages, 11 waves of 32x128
    // 64-byte K-tiles, 4 stages (three K-tiles in flight)
    {352, 128, 2, 8},      // 34: 16 waves
    {384, 128, 4, 2, 32},  // 35: 8 waves of 96x64
    {384, 128, 4, 4, 32},  // 36: 16 waves of 96x32
    {256, 256, 4, 4, 32},  // 37: 16 waves of 64x64
    {352, 128, 11, 1, 32}, // 38: 11 waves of 32x128
    // half-height tiles sized so that two workgroups share a CU (LDS <= 80 KB):
    // the second workgroup computes while the first waits for its K-tile
    {176, 128, 1, 8},      // 39: 2 stages, 8 waves of 176x16
    {176, 128, 1, 4},      // 40: 2 stages, 4 waves of 176x32
    {192, 128, 2, 2, 32},  // 41: 2 stages, 4 waves of 96x64
    {192, 128, 2, 4, 32},  // 42: 2 stages, 8 waves of 96x32
    // small LDS-DMA tiles for small-M layers: deep pipelines in 48-64 KB, so
    // two or three workgroups share a CU and keep more K-tiles in flight
    {64, 64, 2, 2},        // 43: 4 stages, 4 waves of 32x32
    {64, 64, 2, 2},        // 44: 3 stages
    {128, 64, 2, 2},       // 45: 4 stages, 4 waves of 64x32
    {64, 128, 2, 2},       // 46: 4 stages, 4 waves of 32x64
    {64, 32, 2, 2},        // 47: 4 stages, 4 waves of 32x16
    // pipelined kernel (conv_pipe.hip) where pipe_ok(), else tile 2's kernel
    {256, 256, 2, 4},      // 48: 2 stages, 8 waves of 128x64
    {192, 256, 2, 4},      // 49: 2 stages, 8 waves of 96x64
    {128, 128, 2, 4},      // 50: 2 stages, 8 waves of 64x32, two workgroups per CU
    {96, 128, 2, 2},       // 51: 2 stages, 4 waves of 48x64, two workgroups per CU
    {64, 128, 2, 2},       // 52: 3 stages, 4 waves of 32x64, two workgroups per CU
    {128, 64, 2, 2},       // 53: 2 stages, 4 waves of 64x32, three workgroups per CU
    {96, 64, 2, 2},        // 54: 2 stages, 4 waves of 48x32, three workgroups per CU
    {64, 64, 2, 2},        // 55: 3 stages, 4 waves of 32x32, three workgroups per CU
    {64, 32, 2, 2},        // 56: 3 stages, 4 waves of 32x16, four workgroups per CU
    {192, 128, 4, 2},      // 57: 2 stages, 8 waves of 48x64, two workgroups per CU
};
static_assert(sizeof(kTiles) / sizeof(kTiles[0]) == PIPE_TILE + PIPE_TILES, "the pipelined tiles are the table's last");

int tile_count() { return (int)(sizeof(kTiles) / sizeof(kTiles[0])); }
TileCfg tile_cfg(int i) { return kTiles[i]; }

size_t splitk_counters(int M, int cout_p)
{
    size_t most = 0;
    for (int i = 0; i < tile_count(); ++i) {
        const TileCfg t = kTiles[i];
        most = std::max(most, (size_t)((M + t.bm - 1) / t.bm) * ((cout_p + t.bn - 1) / t.bn));
    }
    return most;
}

template <int DT, int BM, int BN, int WM, int WN>
static hipError_t go(const ConvArgs &a, hipStream_t s)
{
    const int mt = (a.M + BM - 1) / BM, nt = (a.cout_p + BN - 1) / BN;
    dim3 grid(mt * nt, 1, a.splits);
    hipLaunchKernelGGL((conv_igemm<DT, BM, BN, WM, WN>), grid, dim3(64 * WM * WN), 0, s, a);
    return hipGetLastError();
}

template <int DT, int BM, int BN, int WM, int WN, int NS, int SPR = 8, int MF = 16>
static hipError_t go_dl(ConvArgs a, hipStream_t s)
{
    if constexpr (MF == 32 && DT != BF16) {
        return go_dl<DT, BM, BN, WM, WN, NS, SPR, 16>(a, s);  // 32x32 blocks: BF16 only
    } else {
        // buffer offsets are 32-bit: the LDS-DMA kernels need tensors below 2 GiB
        const size_t xb = (size_t)a.batch * a.H * a.W * a.cin_p * esize(DT);
        const size_t wb = (size_t)a.cout_p * a.k_pad * esize(DT);
        if (xb >= DN_OOB || wb >= DN_OOB) return go<DT, 128, 128, 2, 2>(a, s);  // register-staged path
        a.x_bytes = (unsigned)xb;
        a.w_bytes = (unsigned)wb;
        const int mt = (a.M + BM - 1) / BM, nt = (a.cout_p + BN - 1) / BN;
        dim3 grid(mt * nt, 1, a.splits);
        if constexpr (DT == FP8 && SPR == 4) {
            return go_dl<DT, BM, BN, WM, WN, NS == 4 ? 2 : NS, 8, MF>(a, s);  // FP8 K-steps need 128-byte tiles
        } else {
            hipLaunchKernelGGL((conv_igemm_dl<DT, BM, BN, WM, WN, NS, SPR, MF>), grid, dim3(64 * WM * WN), 0, s, a);
        }
        return hipGetLastError();
    }
}

template <int DT>
static hipError_t dispatch(int tile, const ConvArgs &a, hipStream_t s)
{
    switch (tile) {
    case 0: return go<DT, 64, 64, 2, 2>(a, s);
    case 1: return go<DT, 128, 64, 2, 2>(a, s);
    case 2: return go<DT, 128, 128, 2, 2>(a, s);
    case 3: return go<DT, 256, 128, 2, 2>(a, s);
    case 4: return go<DT, 256, 256, 2, 4>(a, s);
    case 5: return go<DT, 128, 256, 2, 4>(a, s);
    case 6: return go<DT, 256, 16, 4, 1>(a, s);
    case 7: return go<DT, 256, 32, 4, 1>(a, s);
    case 8: return go<DT, 64, 128, 1, 4>(a, s);
    case 9: return go<DT, 64, 32, 2, 2>(a, s);
    case 10: return go<DT, 256, 256, 2, 2>(a, s);
    case 11: return go<DT, 192, 256, 1, 4>(a, s);
    case 12: return go<DT, 128, 256, 1, 4>(a, s);
    case 13: return go_dl<DT, 256, 128, 2, 2, 3>(a, s);
    case 14: return go_dl<DT, 128, 128, 2, 2, 4>(a, s);
    case 15: return go_dl<DT, 256, 256, 2, 4, 2>(a, s);
    case 16: return go_dl<DT, 192, 256, 1, 4, 2>(a, s);
    case 17: return go_dl<DT, 128, 256, 2, 4, 3>(a, s);
    case 18: return go_dl<DT, 256, 128, 2, 4, 3>(a, s);
    case 19: return go_dl<DT, 256, 256, 2, 4, 4, 4>(a, s);
    case 20: return go_dl<DT, 192, 256, 1, 4, 4, 4>(a, s);
    case 21: return go_dl<DT, 128, 256, 2, 4, 4, 4>(a, s);
    case 22: return go_dl<DT, 256, 128, 2, 2, 4, 4>(a, s);
    case 23: return go_dl<DT, 352, 128, 2, 4, 2>(a, s);
    case 24: return go_dl<DT, 352, 128, 2, 2, 2>(a, s);
    case 25: return go_dl<DT, 352, 128, 2, 8, 2>(a, s);
    case 26: return go_dl<DT, 256, 256, 2, 8, 2>(a, s);
    case 27: return go_dl<DT, 384, 128, 4, 2, 2, 8, 32>(a, s);
    case 28: return go_dl<DT, 384, 128, 4, 4, 2, 8, 32>(a, s);
    case 29: return go_dl<DT, 256, 256, 2, 4, 2, 8, 32>(a, s);
    case 30: return go_dl<DT, 256, 256, 4, 4, 2, 8, 32>(a, s);
    case 31: return go_dl<DT, 256, 128, 4, 2, 3, 8, 32>(a, s);
    case 32: return go_dl<DT, 128, 128, 2, 2, 4, 8, 32>(a, s);
    case 33: return go_dl<DT, 352, 128, 11, 1, 2, 8, 32>(a, s);
    case 34: return go_dl<DT, 352, 128, 2, 8, 4, 4>(a, s);
    case 35: return go_dl<DT, 384, 128, 4, 2, 4, 4, 32>(a, s);
    case 36: return go_dl<DT, 384, 128, 4, 4, 4, 4, 32>(a, s);
    case 37: return go_dl<DT, 256, 256, 4, 4, 4, 4, 32>(a, s);
    case 38: return go_dl<DT, 352, 128, 11, 1, 4, 4, 32>(a, s);
    case 39: return go_dl<DT, 176, 128, 1, 8, 2>(a, s);
    case 40: return go_dl<DT, 176, 128, 1, 4, 2>(a, s);
    case 41: return go_dl<DT, 192, 128, 2, 2, 2, 8, 32>(a, s);
    case 42: return go_dl<DT, 192, 128, 2, 4, 2, 8, 32>(a, s);
    case 43: return go_dl<DT, 64, 64, 2, 2, 4>(a, s);
    case 44: return go_dl<DT, 64, 64, 2, 2, 3>(a, s);
    case 45: return go_dl<DT, 128, 64, 2, 2, 4>(a, s);
    case 46: return go_dl<DT, 64, 128, 2, 2, 4>(a, s);
    case 47: return go_dl<DT, 64, 32, 2, 2, 4>(a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conv(int dt, int tile, const ConvArgs &a, hipStream_t s)
{
    if (a.tile_count && (a.splits > SPLITK_FUSED_MAX ||
                         (size_t)a.splits * a.M * a.cout_p * sizeof(float) > 0x7fffffffu))
        return hipErrorInvalidValue;  // beyond the in-kernel finish's loads
    if (tile == HALO_TILE) return a.splits > 1 ? hipErrorInvalidValue : launch_conv_halo(dt, a, s);
    if (tile == HALO2_TILE) return a.splits > 1 ? hipErrorInvalidValue : launch_conv_halo2(dt, a, s);
    if (tile >= PIPE_TILE && tile < PIPE_TILE + PIPE_TILES) {
        if (pipe_ok(dt, a)) return launch_conv_pipe(dt, tile - PIPE_TILE, a, s);
        tile = 2;
    }
    switch (dt) {
    case F32: return dispatch<F32>(tile, a, s);
    case BF16: return dispatch<BF16>(tile, a, s);
    case FP8: return dispatch<FP8>(tile, a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_splitk_reduce(int dt, const ConvArgs &a, hipStream_t s)
{
    if (a.cout_p & 3) return hipErrorInvalidValue;  // channel padding keeps cout_p a multiple of 4
    const size_t rows = a.pool ? (size_t)(a.M >> 2) : (size_t)a.M;
    const size_t n = rows * (size_t)(a.cout_p >> 2);
    const unsigned blocks = (unsigned)((n + 255) / 256);
    switch (dt) {
    case F32: hipLaunchKernelGGL(splitk_reduce<F32>, dim3(blocks), dim3(256), 0, s, a); break;
    case BF16: hipLaunchKernelGGL(splitk_reduce<BF16>, dim3(blocks), dim3(256), 0, s, a); break;
    case FP8: hipLaunchKernelGGL(splitk_reduce<FP8>, dim3(blocks), dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace dnk
