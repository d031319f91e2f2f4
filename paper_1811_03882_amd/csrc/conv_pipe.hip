// Pipelined implicit-GEMM convolution for layers whose padded channels are a
// multiple of 128 bytes.  The operation, the packed K order and the order of
// every output's sum are those of conv_igemm / conv_igemm_dl (conv.hip):
// tiles of both families give the same bits at the same split count.
//
// What bounded conv_igemm_dl on wide layers is LDS read bandwidth: its waves of
// 176x16 outputs read 12 KB of fragments for 11 MFMAs, 1536 LDS clocks per
// K-tile of the 176x128 tile against 709 matrix clocks.  The register-staged
// small tiles were bound by the round trip of each K-tile's loads.  Here
//   * wave tiles are as square as the registers allow (96x64, 48x64, 64x32), which
//     brings LDS reads below the matrix time;
//   * the fragments of the next half K-tile are read while this half is
//     multiplied, and the transfers of a later K-tile are issued between rows of
//     products, so one barrier per K-tile is left and nothing waits right
//     behind it;
//   * addresses cost two vector instructions per 1 KB transfer.
// Measured on MI355X, BF16, batch 64: 13x13x1024 -> 1024, 3x3: 207 -> 153 us
// (984 -> 1330 TFLOP/s; an 8192^3 library product reaches 1190 here).  Shader
// counters of the 192x256 tile: matrix cores busy 73 % of the cycles of the 228
// CUs that have a tile (52 % before), no bank conflicts, engine clock 1.9 GHz
// against 2.1 at lower matrix load: what is left is mostly the power limit.
// Batch 16, 2704 rows: 134 -> 75 us, bound by how 2704x1024 divides into tiles
// for 256 CUs.  16x16x256 -> 512 at batch 16: 28.4 -> 17.1 us.  FP8 13x13x512 ->
// 1024 at batch 32: 48 -> 34 us.
#include <type_traits>
#include <utility>

#include "conv_dev.h"

namespace dnk {

// Every 128-byte K-tile then lies inside one filter tap and one 128-byte
// channel block, so the tap is wave-uniform: a row's address is a lane
// constant plus a scalar, and its validity one bit of a per-row tap mask
// computed before the K loop.
bool pipe_ok(int dt, const ConvArgs &a)
{
    const size_t xb = ((size_t)a.batch * a.H * a.W + (size_t)a.pad * (a.W + 1)) * a.cin_p * esize(dt);
    const size_t wb = (size_t)a.cout_p * a.k_pad * esize(dt);
    return (a.cin_p * esize(dt)) % 128 == 0 && a.R * a.S <= 31 && a.k_pad == a.R * a.S * a.cin_p && xb < DN_OOB && wb < DN_OOB;
}

// dma16 (conv_dev.h) with a scalar offset and the LDS address as base + constant.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
template <int LOFF> __device__ __forceinline__ void dma16s(const i32x4 &rsrc, unsigned voff, unsigned soff, unsigned lds)
{
    asm volatile("s_add_u32 m0, %0, %4\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds), "v"(voff), "s"(rsrc), "s"(soff), "i"(LOFF)
                 : "memory", "m0", "scc");
}
#pragma clang diagnostic pop

// Epilogue of the swapped product (weights as MFMA operand A, pixels as B):
// lane holds pixel rowb + fm*16 and channels colb + fn*16 + (0..3), so every
// store is one vector of four channels.
template <int DT, int FM, int FN>
__device__ __forceinline__ void pipe_epilogue(const ConvArgs &a, f4 (&acc)[FM][FN], int rowb, int colb)
{
    if (a.splits > 1) {
        float *P = a.partial + (size_t)blockIdx.z * a.M * a.cout_p;
        const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc((void *)a.partial, (short)0, 0x7fffffff, 0x00020000);
#pragma unroll
        for (int fm = 0; fm < FM; ++fm) {
            const int m = rowb + fm * 16;
            if (m >= a.M) continue;
#pragma unroll
            for (int fn = 0; fn < FN; ++fn) {
                const int col = colb + fn * 16;
                if (col >= a.cout_p) continue;
                if (a.tile_count) {  // device scope: the tile's last split reads them in this launch
                    const size_t off = ((size_t)blockIdx.z * a.M * a.cout_p + (size_t)m * a.cout_p + col) * sizeof(float);
                    __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, acc[fm][fn]), rp, (int)off, 0, 16);
                } else {
                    *reinterpret_cast<f4 *>(P + (size_t)m * a.cout_p + col) = acc[fm][fn];
                }
            }
        }
        return;
    }
    float bi[FN][4], scl[FN][4];
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        const int col = colb + fn * 16;
        const bool ok = col < a.cout_p;
        const float4 bias = ok ? *reinterpret_cast<const float4 *>(a.bias + col) : float4{0.f, 0.f, 0.f, 0.f};
        bi[fn][0] = bias.x; bi[fn][1] = bias.y; bi[fn][2] = bias.z; bi[fn][3] = bias.w;
#pragma unroll
        for (int i = 0; i < 4; ++i) scl[fn][i] = 1.0f;
        if constexpr (DT == FP8) {
            const float4 ws = ok ? *reinterpret_cast<const float4 *>(a.wscale + col) : float4{0.f, 0.f, 0.f, 0.f};
            scl[fn][0] = ws.x * a.in_scale; scl[fn][1] = ws.y * a.in_scale; scl[fn][2] = ws.z * a.in_scale; scl[fn][3] = ws.w * a.in_scale;
        }
    }
    // Pixel by pixel, so that the stores to one cache line follow each other:
    // every workgroup of a wide layer ends at once, and with the channel blocks
    // outermost the counters showed 2.4 times the output's bytes written (54 MB
    // for 22 at 13x13x1024, batch 64; 22 in this order, and 3 % off the layer's
    // time; FP8 13x13x512 -> 1024, batch 32: 34.1 -> 32.8 us).
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) {
        const int m = rowb + fm * 16;
        if (m >= a.M) continue;
        unsigned c01[FN], c23[FN];  // BF16 pairs
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
            const int col = colb + fn * 16;
            const bool ok = col < a.cout_p;
            const size_t o = (size_t)m * a.cout_p + col;
            float v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] = activate(acc[fm][fn][i] * scl[fn][i] + bi[fn][i], a.act, a.slope);
            if (a.res && ok) {
                float r[4];
                load4<DT>(a.res, o, r);
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] += r[i] * a.res_scale;
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) v[i] *= a.out_inv_scale;
            if (a.nchw) {
                if (ok) store4_nchw<DT>(a.nchw, a.nchw_c, a.Ho * a.Wo, a.nchw_scale, (unsigned)m, col, v);
            } else if constexpr (DT == BF16 && FN % 2 == 0) {
                c01[fn] = (unsigned)f2bf(v[0]) | ((unsigned)f2bf(v[1]) << 16);
                c23[fn] = (unsigned)f2bf(v[2]) | ((unsigned)f2bf(v[3]) << 16);
                if (fn & 1) {
                    // lanes of the first and third 16 take their neighbours' (the
                    // next 16 lanes') four channels of block fn - 1, those give
                    // theirs of block fn for them: eight channels a lane, one store
                    const auto lo = __builtin_amdgcn_permlane16_swap(c01[fn - 1], c01[fn], false, false);
                    const auto hi = __builtin_amdgcn_permlane16_swap(c23[fn - 1], c23[fn], false, false);
                    const int g = (threadIdx.x >> 4) & 3;
                    const int col8 = colb - 4 * g + (fn - 1 + (g & 1)) * 16 + (g >> 1) * 8;
                    if (col8 < a.cout_p)  // cout_p is a multiple of 8
                        *reinterpret_cast<u32x4 *>(reinterpret_cast<unsigned char *>(a.y) + ((size_t)m * a.cout_p + col8) * 2) =
                            u32x4{lo[0], hi[0], lo[1], hi[1]};
                }
            } else if (ok) {
                store4<DT>(a.y, o, v);
            }
        }
    }
}

// The pooled tiles' unsplit epilogue: a lane's four accumulators are the window
// of one channel, as in conv_epilogue, but window by window, so that the stores
// to one cache line follow each other here too (nine-layer net, BF16, batch 64,
// with two such layers: 519 -> 510 us).
template <int DT, int FM, int FN>
__device__ __forceinline__ void pipe_epilogue_pool(const ConvArgs &a, f4 (&acc)[FM][FN], int rowb, int colb)
{
    float bias[FN], scl[FN];
#pragma unroll
    for (int fn = 0; fn < FN; ++fn) {
        const int col = colb + fn * 16;
        bias[fn] = col < a.cout_p ? a.bias[col] : 0.0f;
        scl[fn] = (DT == FP8 && col < a.cout_p) ? a.wscale[col] * a.in_scale : 1.0f;
    }
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) {
        const int mb = rowb + fm * 16;
        if (mb >= a.M) continue;
#pragma unroll
        for (int fn = 0; fn < FN; ++fn) {
            const int col = colb + fn * 16;
            if (col >= a.cout_p) continue;
            const float w4[4] = {acc[fm][fn][0], acc[fm][fn][1], acc[fm][fn][2], acc[fm][fn][3]};
            const float mx = fmaxf(fmaxf(w4[0], w4[1]), fmaxf(w4[2], w4[3]));
            const size_t o = (size_t)(mb >> 2) * a.cout_p + col;
            store_el<DT>(a.y, o, activate(mx * scl[fn] + bias[fn], a.act, a.slope) * a.out_inv_scale);
            if (a.argmax) a.argmax[o] = window_argmax<DT>(w4, scl[fn], bias[fn], a.act, a.slope, a.out_inv_scale);
        }
    }
}

// s_waitcnt vmcnt(N) lgkmcnt(0), expcnt left at its maximum (no wait)
template <int N> __device__ __forceinline__ void wait_vm_lgkm0()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4));
}

template <int DT, int BM, int BN, int WM, int WN, int NS, int WPE, bool POOL>
__global__ void __launch_bounds__(64 * WM * WN, WPE) conv_pipe(ConvArgs a)
{
    constexpr int NW = WM * WN, ES = esize(DT), SEG = seg_el(DT), BKE = bk_el(DT);
    constexpr int AR = BM / 8 / NW, BR = BN / 8 / NW, LPT = AR + BR;  // 1 KB transfers per wave and K-tile
    constexpr int WTM = BM / WM, WTN = BN / WN, FM = WTM / 16, FN = WTN / 16;
    constexpr int SPL = Tr<DT>::SPL;
    constexpr int FA = (FM + 1) / 2;  // FP8 (one MFMA step per K-tile): A blocks of the first half
    static_assert(BM % (8 * NW) == 0 && BN % (8 * NW) == 0 && WTM % 16 == 0 && WTN % 16 == 0, "tile shape");
    static_assert(NS >= 2 && NS <= 4 && LPT * (NS - 2) < 64, "pipeline depth");

    __shared__ u32x4 sA[NS * BM * 8];
    __shared__ u32x4 sB[NS * BN * 8];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wm = wave % WM, wn = wave / WM;
    const int ntn = (a.cout_p + BN - 1) / BN;
    const int logical = xcd_remap(blockIdx.x, gridDim.x);
    int mi, ni;
    tile_mn(logical, gridDim.x / ntn, ntn, mi, ni);
    const int m0 = mi * BM, n0 = ni * BN;

    // lane L of a transfer fills row L/8, physical segment L%8 of its 8-row
    // group; the swizzle puts logical segment (L%8) ^ (row & 7) there.  A's
    // buffer starts pad rows and columns before x, so that the lane part of an
    // address (pixel) and its scalar part (tap, channel block) are both
    // non-negative; taps outside the image get an offset past the buffer.
    const int lr8 = lane >> 3, sc = (lane & 7) ^ lr8;
    unsigned a_off[AR], a_bad[AR];  // byte offset of the row's pixel; its taps outside the image
#pragma unroll
    for (int i = 0; i < AR; ++i) {
        const int m = m0 + (wave + i * NW) * 8 + lr8;
        a_off[i] = 0;
        a_bad[i] = 0xffffffffu;
        if (m < a.M) {
            int n, ho, wo;
            if (POOL) {
                const int q = m & 3, win = m >> 2, wp2 = a.Wo >> 1, hp2 = a.Ho >> 1;
                const int wp = win % wp2, t = win / wp2;
                ho = 2 * (t % hp2) + (q >> 1); wo = 2 * wp + (q & 1); n = t / hp2;
            } else {
                wo = m % a.Wo; const int t = m / a.Wo; ho = t % a.Ho; n = t / a.Ho;
            }
            const int hi = ho * a.stride - a.pad, wi = wo * a.stride - a.pad;
            a_off[i] = (unsigned)((((n * a.H + ho * a.stride) * a.W + wo * a.stride) * a.cin_p + sc * SEG) * ES);
            unsigned cm = 0;
            for (int s = 0; s < a.S; ++s) cm |= ((unsigned)(wi + s) < (unsigned)a.W ? 1u : 0u) << s;
            for (int r = 0; r < a.R; ++r)
                if ((unsigned)(hi + r) < (unsigned)a.H) a_bad[i] &= ~(cm << (r * a.S));
        }
    }
    unsigned b_off[BR];
#pragma unroll
    for (int i = 0; i < BR; ++i) {
        const int n = n0 + (wave + i * NW) * 8 + lr8;
        b_off[i] = n < a.cout_p ? (unsigned)((n * a.k_pad + sc * SEG) * ES) : DN_OOB;
    }
    const unsigned lead = (unsigned)(a.pad * (a.W + 1) * a.cin_p * ES);
    const i32x4 rx = make_rsrc((const char *)a.x - lead, a.x_bytes + lead);
    const i32x4 rw = make_rsrc(a.w, a.w_bytes);

    const int nkt = a.k_pad / BKE;
    const int kt0 = blockIdx.z * a.ktiles_per_split;
    const int nk = min(nkt, kt0 + a.ktiles_per_split) - kt0;  // K-tiles of this split (may be <= 0)
    // the next K-tile to transfer (scalar): tap t, column ts of it, byte
    // offset toff of the tap and channel block, byte offset kb in a B row
    const int RS = a.R * a.S, rowb = (a.W - a.S) * a.cin_p * ES;  // from a filter row's end to the next row's start
    int t = kt0 % RS, ts = t % a.S, kb = kt0 * 128;
    int toff = ((t / a.S) * a.W + ts) * a.cin_p * ES + (kt0 / RS) * 128;
    auto step = [&] {
        kb += 128;
        ++t;
        toff += a.cin_p * ES;
        if (++ts == a.S) { ts = 0; toff += rowb; }
        if (t == RS) { t = 0; toff += 128 - a.R * a.W * a.cin_p * ES; }
    };
    const unsigned ldsA = (unsigned)(size_t)(const __attribute__((address_space(3))) void *)sA + wave * 1024;
    const unsigned ldsB = (unsigned)(size_t)(const __attribute__((address_space(3))) void *)sB + wave * 1024;
    // transfers [LO, HI) of the LPT of the next K-tile, into stage st
    auto xfer = [&](auto lo, auto hi, int st) {
        constexpr int LO = decltype(lo)::value, HI = decltype(hi)::value;
        [&]<int... I>(std::integer_sequence<int, I...>) {
            ([&] {
                constexpr int i = LO + I;
                if constexpr (i < AR) dma16s<i * NW * 1024>(rx, ((a_bad[i] << (31 - t)) & DN_OOB) | a_off[i], (unsigned)toff, ldsA + st * (BM * 128));
                else dma16s<(i - AR) * NW * 1024>(rw, b_off[i - AR], (unsigned)kb, ldsB + st * (BN * 128));
            }(), ...);
        }(std::make_integer_sequence<int, (HI > LO ? HI - LO : 0)>{});
    };

    f4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f4{0.f, 0.f, 0.f, 0.f};

    const int lrow = lane & 15, lgrp = lane >> 4;
    // 16-byte index of this lane's segment of MFMA step 0 in the wave's first
    // A / B block; step 1 (BF16 / FP32) is the index ^ 4, the second segment
    // of an FP8 operand the index ^ 1
    const int sw = (lgrp * SPL) ^ (lrow & 7);
    const int ia = (wm * WTM + lrow) * 8 + sw, ib = (wn * WTN + lrow) * 8 + sw;
    auto read = [&](u32x4 (&f)[SPL], const u32x4 *s, int i) {
#pragma unroll
        for (int j = 0; j < SPL; ++j) f[j] = s[i ^ j];
    };
    auto product = [&](f4 &c, const u32x4 *af, const u32x4 *bf) {
        if constexpr (POOL) mma<DT>(c, af, bf);
        else mma<DT>(c, bf, af);  // swapped: a lane then holds four channels of one pixel
    };
    // Half-step boundary of K-tile k: this wave's fragments of tile k are in
    // registers and its transfers of tile k + 1 have landed; behind the
    // barrier so have all waves', so tile k's stage can take tile k + NS.
    auto turn = [&](bool steady) {
        __builtin_amdgcn_sched_barrier(0);
        if (steady) wait_vm_lgkm0<LPT * (NS - 2)>();
        else wait_vm_lgkm0<0>();
        lds_barrier();
        __builtin_amdgcn_sched_barrier(0);
    };

    if (nk > 0) {
        const int pre = min(nk, NS);
        for (int k = 0; k < pre; ++k) {
            xfer(std::integral_constant<int, 0>{}, std::integral_constant<int, LPT>{}, k);
            step();
        }
        if (nk >= NS) wait_vm<LPT * (NS - 1)>();
        else wait_vm<0>();
        lds_barrier();
    }
    // One half of a K-tile: rows [R0, R1) of products on fragments that are in
    // registers, one row of FN products at a time; between the rows go the LDS
    // reads of the next half's fragments (rd(q), q < NRD, in the first two
    // thirds of the rows) and, with MORE, the transfers of the K-tile that
    // takes the freed stage, so that neither leaves the matrix cores idle.
    auto half = [&](auto r0, auto r1, auto nrd, auto more, int st, auto &&mul, auto &&rd) {
        constexpr int R0 = decltype(r0)::value, R1 = decltype(r1)::value, NRD = decltype(nrd)::value, NR = R1 - R0;
        constexpr int RR = (2 * NR + 2) / 3;  // rows that take reads
        [&]<int... I>(std::integer_sequence<int, I...>) {
            ([&] {
                if constexpr (I < RR) {
#pragma unroll
                    for (int q = I * NRD / RR; q < (I + 1) * NRD / RR; ++q) rd(q);
                }
                if constexpr (decltype(more)::value)
                    xfer(std::integral_constant<int, I * LPT / NR>{}, std::integral_constant<int, (I + 1) * LPT / NR>{}, st);
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int j = 0; j < FN; ++j) mul(R0 + I, j);
                __builtin_amdgcn_s_setprio(0);
                __builtin_amdgcn_sched_barrier(0);
            }(), ...);
        }(std::make_integer_sequence<int, NR>{});
        if constexpr (decltype(more)::value) step();
    };
    typedef std::integral_constant<int, 0> c0;
    typedef std::integral_constant<int, FA> cA;
    typedef std::integral_constant<int, FM> cM;

    int st = 0, k = 0;
    if constexpr (DT == FP8) {
        // one MFMA step per K-tile: the halves are rows [0, FA) and [FA, FM);
        // the B fragments of the next K-tile wait in bn during the second
        u32x4 fa[FM][SPL], b[FN][SPL], bn[FN][SPL];
        if (nk > 0) {
#pragma unroll
            for (int i = 0; i < FA; ++i) read(fa[i], sA + i * 128, ia);
#pragma unroll
            for (int j = 0; j < FN; ++j) read(b[j], sB + j * 128, ib);
        }
        auto mul = [&](int i, int j) { product(acc[i][j], fa[i], b[j]); };
        auto tile = [&](auto more) {
            constexpr bool MORE = decltype(more)::value;
            const int nx = st + 1 == NS ? 0 : st + 1;
            half(c0{}, cA{}, std::integral_constant<int, FM - FA>{}, std::false_type{}, st, mul,
                 [&](int q) { read(fa[FA + q], sA + st * (BM * 8) + (FA + q) * 128, ia); });
            turn(MORE || k + NS - 1 < nk);
            // (after the last K-tile these reads bring an old stage, which nothing uses)
            half(cA{}, cM{}, std::integral_constant<int, FA + FN>{}, more, st, mul, [&](int q) {
                if (q < FN) read(bn[q], sB + nx * (BN * 8) + q * 128, ib);
                else read(fa[q - FN], sA + nx * (BM * 8) + (q - FN) * 128, ia);
            });
#pragma unroll
            for (int j = 0; j < FN; ++j)
#pragma unroll
                for (int q = 0; q < SPL; ++q) b[j][q] = bn[j][q];
            st = nx;
        };
        for (; k + NS < nk; ++k) tile(std::true_type{});
        for (; k < nk; ++k) tile(std::false_type{});
    } else {
        // two MFMA steps per K-tile: each half runs one on all rows
        u32x4 a0[FM][1], b0[FN][1], a1[FM][1], b1[FN][1];
        if (nk > 0) {
#pragma unroll
            for (int i = 0; i < FM; ++i) read(a0[i], sA + i * 128, ia);
#pragma unroll
            for (int j = 0; j < FN; ++j) read(b0[j], sB + j * 128, ib);
        }
        typedef std::integral_constant<int, FM + FN> cR;
        auto mul0 = [&](int i, int j) { product(acc[i][j], a0[i], b0[j]); };
        auto mul1 = [&](int i, int j) { product(acc[i][j], a1[i], b1[j]); };
        auto tile = [&](auto more) {
            constexpr bool MORE = decltype(more)::value;
            const int nx = st + 1 == NS ? 0 : st + 1;
            half(c0{}, cM{}, cR{}, std::false_type{}, st, mul0, [&](int q) {
                if (q < FN) read(b1[q], sB + st * (BN * 8) + q * 128, ib ^ 4);
                else read(a1[q - FN], sA + st * (BM * 8) + (q - FN) * 128, ia ^ 4);
            });
            turn(MORE || k + NS - 1 < nk);
            // (after the last K-tile these reads bring an old stage, which nothing uses)
            half(c0{}, cM{}, cR{}, more, st, mul1, [&](int q) {
                if (q < FN) read(b0[q], sB + nx * (BN * 8) + q * 128, ib);
                else read(a0[q - FN], sA + nx * (BM * 8) + (q - FN) * 128, ia);
            });
            st = nx;
        };
        for (; k + NS < nk; ++k) tile(std::true_type{});
        for (; k < nk; ++k) tile(std::false_type{});
    }
    __syncthreads();

    if constexpr (POOL) {
        if (a.splits > 1) conv_epilogue<DT, FM, FN>(a, acc, m0 + wm * WTM + 4 * lgrp, n0 + wn * WTN + lrow);
        else pipe_epilogue_pool<DT, FM, FN>(a, acc, m0 + wm * WTM + 4 * lgrp, n0 + wn * WTN + lrow);
    } else pipe_epilogue<DT, FM, FN>(a, acc, m0 + wm * WTM + lrow, n0 + wn * WTN + 4 * lgrp);
    if (a.splits > 1 && a.tile_count) splitk_tail<DT, BM, BN, 64 * NW>(a, m0, n0, sA);
}

template <int DT, int BM, int BN, int WM, int WN, int NS, int WPE>
static hipError_t go_pipe(ConvArgs a, hipStream_t s)
{
    a.x_bytes = (unsigned)((size_t)a.batch * a.H * a.W * a.cin_p * esize(DT));
    a.w_bytes = (unsigned)((size_t)a.cout_p * a.k_pad * esize(DT));
    const int mt = (a.M + BM - 1) / BM, nt = (a.cout_p + BN - 1) / BN;
    const dim3 grid(mt * nt, 1, a.splits), block(64 * WM * WN);
    if (a.pool) hipLaunchKernelGGL((conv_pipe<DT, BM, BN, WM, WN, NS, WPE, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((conv_pipe<DT, BM, BN, WM, WN, NS, WPE, false>), grid, block, 0, s, a);
    return hipGetLastError();
}

template <int DT> static hipError_t dispatch_pipe(int i, const ConvArgs &a, hipStream_t s)
{
    switch (i) {
    case 0: if constexpr (pipe_own(DT, 0)) return go_pipe<DT, 256, 256, 2, 4, 2, 2>(a, s); else return go_pipe<DT, 192, 256, 2, 4, 2, 2>(a, s);
    case 1: return go_pipe<DT, 192, 256, 2, 4, 2, 2>(a, s);
    case 2: return go_pipe<DT, 128, 128, 2, 4, 2, 4>(a, s);
    case 3: return go_pipe<DT, 96, 128, 2, 2, 2, 2>(a, s);
    case 4: return go_pipe<DT, 64, 128, 2, 2, 3, 2>(a, s);
    case 5: return go_pipe<DT, 128, 64, 2, 2, 2, 3>(a, s);
    case 6: return go_pipe<DT, 96, 64, 2, 2, 2, 3>(a, s);
    case 7: return go_pipe<DT, 64, 64, 2, 2, 3, 3>(a, s);
    case 8: return go_pipe<DT, 64, 32, 2, 2, 3, 4>(a, s);
    case 9: return go_pipe<DT, 192, 128, 4, 2, 2, DT == FP8 ? 2 : 4>(a, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_conv_pipe(int dt, int i, const ConvArgs &a, hipStream_t s)
{
    if (!pipe_ok(dt, a)) return hipErrorInvalidValue;
    switch (dt) {
    case F32: return dispatch_pipe<F32>(i, a, s);
    case BF16: return dispatch_pipe<BF16>(i, a, s);
    case FP8: return dispatch_pipe<FP8>(i, a, s);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace dnk
