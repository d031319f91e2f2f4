// Gradient through a 2x2/2 pool fused into its conv and through that conv's
// few channels, in one kernel: the backward-data conv whose input, the
// full-size gradient of the conv's output, exists only as the LDS window of a
// tile.  unpool_bwd (backward.hip) followed by a halo conv writes and re-reads
// that gradient, the largest tensor of the pass: 16 images of 416x416x16 in
// BF16 are 89 MB, four times the pooled gradient they come from.
//
// A workgroup owns 16 x 32 pixels of the result (at most 16 channels).  It
// forms its window from the pooled gradient, the pooled outputs (their sign is
// the leaky branch) and the windows' argmax codes, each read once plus the
// rim, with the arithmetic of unpool_bwd: the same rounded values.  The
// products then run as in conv_halo2: the same K order, so the same bits.  For
// the gradient of the image the rounded values leave as NCHW FP32, which the
// egress kernel would otherwise do.
// Measured, 416x416 at batch 16, BF16: 3 <- 16 channels 35 us (unpool,
// conv and egress: 121), 208x208, 16 <- 32 channels 25 us (52).
#include <type_traits>

#include "conv_dev.h"

namespace dnk {

constexpr int UP_TH = 16, UP_TW = 32;
constexpr int up_pitch(int cps) { return (cps & 1) ? cps + 2 : cps + 1; }  // odd, one zero chunk past the channels
constexpr int UP_KSMAX = 10;

static size_t up_lds(int dt, const UnpoolConvArgs &a)
{
    return (size_t)(UP_TH + a.R - 1) * (UP_TW + a.S - 1) * up_pitch(a.cp / seg_el(dt)) * 16;
}

bool unpool_conv_ok(int dt, const UnpoolConvArgs &a)
{
    if (dt != F32 && dt != BF16) return false;
    const int kstep = dt == BF16 ? 32 : 16, K = a.R * a.S * a.cp;
    const size_t big = (size_t)1 << 31;
    return a.cout_p <= 16 && kblock_ch(dt, a.cp, a.R * a.S) == a.cp && (K + kstep - 1) / kstep <= UP_KSMAX &&
           up_lds(dt, a) <= 64 * 1024 && a.batch <= 65535 && (a.Ho + UP_TH - 1) / UP_TH <= 65535 &&
           (size_t)a.Hp * a.Wp * a.cp * esize(dt) < big && (size_t)a.Ho * a.Wo * 16 * 4 < big;
}

// KSM: MFMA steps whose weights a wave holds (registers decide how many workgroups
// share a CU and hide each other's loads: five with 5 steps, four with 10).
template <int DT, bool IMAGE, int KSM>
__global__ void __launch_bounds__(256, KSM == 5 ? 5 : 4) conv_unpool(UnpoolConvArgs a)
{
    constexpr int ES = esize(DT), SEG = seg_el(DT), KSTEP = 4 * SEG;
    constexpr int BPW = UP_TH * UP_TW / 16 / 4;  // 16-pixel blocks per wave
    extern __shared__ __align__(16) unsigned char up_raw[];
    u32x4 *win = reinterpret_cast<u32x4 *>(up_raw);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lrow = lane & 15, lgrp = lane >> 4;
    const int n = blockIdx.z, th0 = blockIdx.y * UP_TH, tw0 = blockIdx.x * UP_TW;
    const int K = a.R * a.S * a.cp, KS = (K + KSTEP - 1) / KSTEP;
    const int cps = a.cp / SEG, pst = up_pitch(cps);
    const int LH = UP_TH + a.R - 1, LW = UP_TW + a.S - 1;
    const u32x4 z4 = {0u, 0u, 0u, 0u};

    // weights of the (at most 16) output channels, every K step
    // (lanes past the last channel repeat it: their results go nowhere)
    u32x4 wr[KSM][1];
    const unsigned wrow = (unsigned)(min(lrow, a.cout_p - 1) * a.k_pad + lgrp * SEG) * ES;
#pragma unroll
    for (int ks = 0; ks < KSM; ++ks) {
        wr[ks][0] = z4;
        if (ks < KS) wr[ks][0] = gload16(a.w, wrow + ks * KSTEP * ES);
    }

    // ---- the window: one item per pooled pixel and 16-byte segment, which
    // holds the 2x2 pixels of the full-size gradient (pixels outside the image
    // are zero, and belong to pooled pixels outside it)
    {
        const int hi0 = th0 - a.pad, wi0 = tw0 - a.pad;
        const int pi0 = hi0 >> 1, pj0 = wi0 >> 1;  // floor
        const int PR = ((hi0 + LH - 1) >> 1) - pi0 + 1, PC = ((wi0 + LW - 1) >> 1) - pj0 + 1;
        const int items = PR * PC * cps;
        const size_t img = (size_t)n * a.Hp * a.Wp * a.cp;
        const unsigned char *dyi = reinterpret_cast<const unsigned char *>(a.dy) + img * ES;
        const unsigned char *poi = reinterpret_cast<const unsigned char *>(a.pooled) + img * ES;
        const unsigned char *ami = a.argmax + img;
        constexpr int U = 2;  // items in flight per thread
        const FastDiv by_cps(cps), by_pc(PC);
        const int wbase = wave * 64;
        for (int base = tid; base < items + tid; base += 256 * U) {
            const int wfirst = base - tid + wbase;  // the wave's first item (uniform): past the last, nothing to do
            u32x4 dy[U], po[U];
            unsigned am[U][2];
            int y0[U], x0[U], sg[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int e = base + u * 256;
                const int px = by_cps.div(e);
                sg[u] = e - px * cps;
                const int pr = by_pc.div(px), pi = pi0 + pr, pj = pj0 + px - pr * PC;
                y0[u] = e < items ? 2 * pi - hi0 : -8;
                x0[u] = 2 * pj - wi0;
                const bool in = e < items && (unsigned)pi < (unsigned)a.Hp && (unsigned)pj < (unsigned)a.Wp;
                const unsigned o = in ? (unsigned)((pi * a.Wp + pj) * a.cp + sg[u] * SEG) : 0u;
                dy[u] = in ? gload16(dyi, (size_t)o * ES) : z4;
                po[u] = in ? gload16(poi, (size_t)o * ES) : z4;
                if constexpr (SEG == 8) {
                    const uint2 c = in ? *reinterpret_cast<const uint2 *>(ami + o) : make_uint2(0u, 0u);
                    am[u][0] = c.x;
                    am[u][1] = c.y;
                } else {
                    am[u][0] = in ? *reinterpret_cast<const unsigned *>(ami + o) : 0u;
                    am[u][1] = 0u;
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (wfirst + u * 256 >= items) continue;
                // the gradient of each element's window maximum, rounded as stored
                unsigned g[SEG];
#pragma unroll
                for (int e = 0; e < SEG; ++e) {
                    float d, p;
                    if constexpr (DT == F32) {
                        d = __uint_as_float(dy[u][e]);
                        p = __uint_as_float(po[u][e]);
                    } else {
                        d = bf2f((uint16_t)(dy[u][e >> 1] >> (16 * (e & 1))));
                        p = bf2f((uint16_t)(po[u][e >> 1] >> (16 * (e & 1))));
                    }
                    d *= (a.mask < 0.0f || p > 0.0f) ? 1.0f : a.mask;
                    if constexpr (DT == F32) g[e] = __float_as_uint(d);
                    else g[e] = f2bf(d);
                }
                // element e of window position k: g[e] where the code is k, else zero.
                // The codes' two bits, spread over each element, split g in four.
                u32x4 v[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    unsigned gq, lo, hi;
                    if constexpr (DT == F32) {
                        gq = g[q];
                        lo = (unsigned)((int)(am[u][0] << (31 - 8 * q)) >> 31);
                        hi = (unsigned)((int)(am[u][0] << (30 - 8 * q)) >> 31);
                    } else {
                        typedef short s2 __attribute__((ext_vector_type(2)));
                        gq = g[2 * q] | (g[2 * q + 1] << 16);
                        const unsigned c = __builtin_amdgcn_perm(0u, am[u][q >> 1], q & 1 ? 0x0C030C02u : 0x0C010C00u);
                        lo = __builtin_bit_cast(unsigned, (s2)(__builtin_bit_cast(s2, c) << (short)15) >> (short)15);
                        hi = __builtin_bit_cast(unsigned, (s2)(__builtin_bit_cast(s2, c) << (short)14) >> (short)15);
                    }
                    const unsigned bottom = gq & hi, top = gq ^ bottom;
                    v[3][q] = bottom & lo;
                    v[2][q] = bottom ^ v[3][q];
                    v[1][q] = top & lo;
                    v[0][q] = top ^ v[1][q];
                }
                const int at = (y0[u] * LW + x0[u]) * pst + sg[u];
                const bool yt = (unsigned)y0[u] < (unsigned)LH, yb = (unsigned)(y0[u] + 1) < (unsigned)LH;
                const bool xl = (unsigned)x0[u] < (unsigned)LW, xr = (unsigned)(x0[u] + 1) < (unsigned)LW;
                if (yt && xl) win[at] = v[0];
                if (yt && xr) win[at + pst] = v[1];
                if (yb && xl) win[at + LW * pst] = v[2];
                if (yb && xr) win[at + LW * pst + pst] = v[3];
            }
        }
        if (K < KS * KSTEP)
            for (int px = tid; px < LH * LW; px += 256) win[px * pst + cps] = z4;  // read by K segments past K
    }
    // offset, relative to the lane's pixel, of lane group g's K segment of step
    // ks: the divisions once per workgroup and entry
    __shared__ int toff_tab[KSM * 4];
    if (tid < KSM * 4) {
        const int k = (tid >> 2) * KSTEP + (tid & 3) * SEG;
        int o = cps;
        if (k < K) {
            const int tap = k / a.cp, c0 = k - tap * a.cp, r = tap / a.S, sx = tap - r * a.S;
            o = (r * LW + sx) * pst + c0 / SEG;
        }
        toff_tab[tid] = o;
    }
    __syncthreads();

    int toff[KSM];
#pragma unroll
    for (int ks = 0; ks < KSM; ++ks) toff[ks] = toff_tab[ks * 4 + lgrp];
    f4 acc[BPW];
#pragma unroll
    for (int i = 0; i < BPW; ++i) acc[i] = f4{0.f, 0.f, 0.f, 0.f};
    int pb[BPW];  // block i: tile row 4*wave + i/2, columns 16*(i & 1) + (0..15)
#pragma unroll
    for (int i = 0; i < BPW; ++i) pb[i] = ((4 * wave + (i >> 1)) * LW + 16 * (i & 1) + lrow) * pst;
#pragma unroll
    for (int ks = 0; ks < KSM; ++ks) {
        if (ks < KS)
#pragma unroll
        for (int i = 0; i < BPW; ++i) {
            const u32x4 af[1] = {win[pb[i] + toff[ks]]};
            if constexpr (IMAGE) mma<DT>(acc[i], af, wr[ks]);  // lane: channel lrow of four pixels
            else mma<DT>(acc[i], wr[ks], af);                  // lane: four channels of pixel lrow
        }
    }

    // ---- linear, zero bias (as the conv kernels add it), rounded to the storage type
#pragma unroll
    for (int i = 0; i < BPW; ++i) {
        const int ho = th0 + 4 * wave + (i >> 1);
        if (ho >= a.Ho) continue;  // wave-uniform
        float v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) v[q] = acc[i][q] + 0.0f;
        if constexpr (IMAGE) {
            const int wo = tw0 + 16 * (i & 1) + 4 * lgrp;
            if (lrow >= a.C) continue;
            float *y = reinterpret_cast<float *>(a.y) + (((size_t)n * a.C + lrow) * a.Ho + ho) * a.Wo + wo;
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = stored_value<DT>(v[q]);
            if ((a.Wo & 3) == 0) {  // the row starts on 16 bytes: whole vectors, all inside or all outside
                if (wo < a.Wo) *reinterpret_cast<float4 *>(y) = make_float4(v[0], v[1], v[2], v[3]);
            } else {
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (wo + q < a.Wo) y[q] = v[q];
            }
        } else {
            const int wo = tw0 + 16 * (i & 1) + lrow, ch = 4 * lgrp;
            if (wo < a.Wo && ch < a.cout_p)
                store4<DT>(reinterpret_cast<unsigned char *>(a.y) + (size_t)n * a.Ho * a.Wo * a.cout_p * ES, (size_t)(ho * a.Wo + wo) * a.cout_p + ch, v);
        }
    }
}

template <int DT, bool IMAGE> static hipError_t go_unpool(const UnpoolConvArgs &a, hipStream_t s)
{
    const dim3 grid((a.Wo + UP_TW - 1) / UP_TW, (a.Ho + UP_TH - 1) / UP_TH, a.batch);
    const int kstep = 4 * seg_el(DT), KS = (a.R * a.S * a.cp + kstep - 1) / kstep;
    if (KS <= 5) hipLaunchKernelGGL((conv_unpool<DT, IMAGE, 5>), grid, dim3(256), up_lds(DT, a), s, a);
    else hipLaunchKernelGGL((conv_unpool<DT, IMAGE, UP_KSMAX>), grid, dim3(256), up_lds(DT, a), s, a);
    return hipGetLastError();
}

hipError_t launch_conv_unpool(int dt, const UnpoolConvArgs &a, hipStream_t s)
{
    if (!unpool_conv_ok(dt, a) || (a.image && (a.C > 16 || ((uintptr_t)a.y & 15)))) return hipErrorInvalidValue;
    if (dt == F32) return a.image ? go_unpool<F32, true>(a, s) : go_unpool<F32, false>(a, s);
    return a.image ? go_unpool<BF16, true>(a, s) : go_unpool<BF16, false>(a, s);
}

}  // namespace dnk
