// Detection post-processing of a region-layer output, on the device.
//
// The workload's detection program turns the last layer's output into boxes
// (Sec. 5.1.1).  The rule (a reading; the paper gives none): each grid cell
// holds A anchors x (5 + C) channels: tx, ty, tw, th, to, then C class
// logits.  Box centre ((j + sigmoid(tx)) / W, (i + sigmoid(ty)) / H), size
// (anchor_w * exp(tw) / W, anchor_h * exp(th) / H), class scores
// sigmoid(to) * softmax(logits).  Per image and class, candidates with
// score >= thresh are ranked by score (descending, ties by box index
// (i*W + j)*A + a) and kept greedily unless a kept box overlaps them with
// IoU > nms_thresh, at most max_det per class.
//
// Two kernels: decode (one thread per box) writes every box and every class score to the
// workspace; nms (one workgroup per image and class) collects the class's
// candidates, sorts them and runs the greedy suppression, one kept box per
// step.  Both are latency-bound, not traffic-bound (64 images x 845 boxes x 20
// classes move 5.4 MB): decode therefore has every logit load of a box in
// flight at once, and nms sorts the candidates alone, not the class's boxes,
// and forms their overlaps before the greedy pass.  At those sizes with about 20
// candidates a class (166 at most): 66 -> 25 us for both kernels.
// Arithmetic is FP32 with contraction off, in the order the definition
// states, so threshold and overlap decisions are reproducible.
#include "dn_kernels.h"

#include <algorithm>
#include <mutex>

#pragma clang fp contract(off)

namespace dnk {

__device__ __forceinline__ float sigm(float x) { return 1.0f / (1.0f + expf(-x)); }

// CM > 0: at most CM classes, all logits of the box in registers (loads in
// flight together, one exponential each); threads in box order, so that scores
// and boxes leave in whole lines.  CM = 0: any number, read three times; threads
// in plane order, so that these reads are whole lines (200 classes, 8 x 2028 boxes:
// 142 us, 187 in box order).  The sums run in the same order either way.
template <int CM>
__global__ void __launch_bounds__(CM > 0 ? 64 : 256) detect_decode(DetectArgs a)
{
    const int HW = a.H * a.W, B = HW * a.A;
    const int t = blockIdx.x * blockDim.x + threadIdx.x;  // (n, box) or (n, anchor, cell)
    if (t >= a.N * B) return;
    const int n = t / B, r = t - n * B;
    const int cell = CM > 0 ? r / a.A : r % HW, anc = CM > 0 ? r - cell * a.A : r / HW;
    const int b = cell * a.A + anc;  // box index
    const int i = cell / a.W, j = cell - i * a.W;
    const float *p = a.y + ((size_t)n * a.A * (5 + a.C) + (size_t)anc * (5 + a.C)) * HW + cell;
    float e[CM > 0 ? CM : 1];
    if constexpr (CM > 0) {
#pragma unroll
        for (int k = 0; k < CM; ++k) e[k] = k < a.C ? p[(size_t)(5 + k) * HW] : -INFINITY;
    }
    const float bx = ((float)j + sigm(p[0])) / (float)a.W;
    const float by = ((float)i + sigm(p[(size_t)HW])) / (float)a.H;
    const float bw = (a.anchors[2 * anc] * expf(p[2 * (size_t)HW])) / (float)a.W;
    const float bh = (a.anchors[2 * anc + 1] * expf(p[3 * (size_t)HW])) / (float)a.H;
    const float obj = sigm(p[4 * (size_t)HW]);
    float mx = -INFINITY, sum = 0.0f;
    float *sc = a.score + (size_t)n * a.C * B + b;
    if constexpr (CM > 0) {
#pragma unroll
        for (int k = 0; k < CM; ++k) mx = fmaxf(mx, e[k]);
#pragma unroll
        for (int k = 0; k < CM; ++k)
            if (k < a.C) {
                e[k] = expf(e[k] - mx);
                sum += e[k];
            }
#pragma unroll
        for (int k = 0; k < CM; ++k)
            if (k < a.C) sc[(size_t)k * B] = obj * (e[k] / sum);
    } else {
        for (int k = 0; k < a.C; ++k) mx = fmaxf(mx, p[(size_t)(5 + k) * HW]);
        for (int k = 0; k < a.C; ++k) sum += expf(p[(size_t)(5 + k) * HW] - mx);
        for (int k = 0; k < a.C; ++k) sc[(size_t)k * B] = obj * (expf(p[(size_t)(5 + k) * HW] - mx) / sum);
    }
    reinterpret_cast<float4 *>(a.box)[(size_t)n * B + b] = make_float4(bx, by, bw, bh);
}

__device__ __forceinline__ float box_iou(float4 p, float4 q)
{
    const float l1 = p.x - p.z / 2.0f, r1 = p.x + p.z / 2.0f, t1 = p.y - p.w / 2.0f, d1 = p.y + p.w / 2.0f;
    const float l2 = q.x - q.z / 2.0f, r2 = q.x + q.z / 2.0f, t2 = q.y - q.w / 2.0f, d2 = q.y + q.w / 2.0f;
    const float iw = fmaxf(0.0f, fminf(r1, r2) - fmaxf(l1, l2));
    const float ih = fmaxf(0.0f, fminf(d1, d2) - fmaxf(t1, t2));
    const float inter = iw * ih;
    const float uni = p.z * p.w + q.z * q.w - inter;
    return uni > 0.0f ? inter / uni : 0.0f;
}

__device__ __forceinline__ float lane_of(float v, int i)  // lane i's v, i wave-uniform
{
    return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(v), i));
}
__device__ __forceinline__ unsigned long long lane_of(unsigned long long v, int i)
{
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)v, i);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(v >> 32), i);
    return ((unsigned long long)hi << 32) | lo;
}

// A box's edges and area, as box_iou() forms them.
struct Edges { float l, r, t, d, area; };
__device__ __forceinline__ Edges edges_of(float4 p)
{
    return Edges{p.x - p.z / 2.0f, p.x + p.z / 2.0f, p.y - p.w / 2.0f, p.y + p.w / 2.0f, p.z * p.w};
}
// box_iou(p, q) > thresh for the wave's live lanes.  The quotient is needed
// exactly only where it lies within rounding of the threshold: inter against
// thresh * uni (relative error below 1e-6) decides every other lane, and the
// division runs only if some lane is undecided.  slack: 1e-30, or infinite (every
// lane undecided) for thresholds from 0 to 1e-30, to which a quotient too small
// for a float rounds down.
__device__ __forceinline__ bool overlaps(const Edges &p, const Edges &q, float thresh, float slack, bool live)
{
    const float iw = fmaxf(0.0f, fminf(p.r, q.r) - fmaxf(p.l, q.l));
    const float ih = fmaxf(0.0f, fminf(p.d, q.d) - fmaxf(p.t, q.t));
    const float inter = iw * ih;
    const float uni = p.area + q.area - inter;
    const float part = thresh * uni, diff = inter - part;
    const bool sure = uni > 0.0f && fabsf(diff) > 4e-6f * fabsf(part) + slack;
    bool over = diff > 0.0f;
    if (__any(live && !sure)) over = (uni > 0.0f ? inter / uni : 0.0f) > thresh;
    return live && over;
}

// m <= 64*Q <= 256 candidates, the whole workgroup.  A candidate's place in the
// order is the number of larger keys (one pass over the keys in LDS, no
// exchanges).  Row i of the overlap matrix is one test of the wave's lanes
// against candidate i and a ballot: rows are independent, so the four waves
// share them, and the greedy pass that is left, a chain of one step per kept
// box, only masks bits that one wave holds in registers.
template <int Q>
__device__ __forceinline__ void nms_small(const DetectArgs &a, unsigned long long *key, int m, const float4 *bx,
                                          size_t obase, int *count)
{
    unsigned long long *skey = key + 256;                                     // [64*Q] sorted
    float4 *sbox = reinterpret_cast<float4 *>(skey + 64 * Q);                 // [64*Q]
    unsigned long long *rows = reinterpret_cast<unsigned long long *>(sbox + 64 * Q);  // [64*Q][Q]
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid >= m && tid < m + 8 && tid < 256) key[tid] = 0ull;  // below every key: whole groups of 8 can be read
    __syncthreads();
    if (tid < m) {
        const unsigned long long kv = key[tid];
        const float4 box = bx[~(unsigned)(kv & 0xFFFFFFFFull)];
        int rank = 0;
        for (int e = 0; e < m; e += 8) {
            unsigned long long o[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) o[q] = key[e + q];
#pragma unroll
            for (int q = 0; q < 8; ++q) rank += o[q] > kv ? 1 : 0;
        }
        skey[rank] = kv;
        sbox[rank] = box;
    }
    __syncthreads();
    float4 box[Q];
    Edges ed[Q];
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        box[q] = q * 64 + lane < m ? sbox[q * 64 + lane] : make_float4(0.0f, 0.0f, 0.0f, 0.0f);
        ed[q] = edges_of(box[q]);
    }
    const float slack = a.nms_thresh >= 0.0f && a.nms_thresh < 1e-30f ? INFINITY : 1e-30f;
#pragma unroll
    for (int p = 0; p < Q; ++p) {
        for (int i = wave; i < 64 && p * 64 + i < m; i += 4) {
            const Edges e = {lane_of(ed[p].l, i), lane_of(ed[p].r, i), lane_of(ed[p].t, i), lane_of(ed[p].d, i), lane_of(ed[p].area, i)};
#pragma unroll
            for (int q = p; q < Q; ++q) {  // only later candidates matter
                if (q * 64 >= m) break;
                const unsigned long long over = __ballot(overlaps(e, ed[q], a.nms_thresh, slack, q * 64 + lane < m));
                if (lane == 0) rows[(size_t)(p * 64 + i) * Q + q] = over;
            }
        }
    }
    __syncthreads();
    if (tid >= 64) return;
    unsigned long long row[Q][Q], left[Q];  // the lane's rows; candidates neither kept nor suppressed
#pragma unroll
    for (int p = 0; p < Q; ++p) {
        const bool in = p * 64 + lane < m;
#pragma unroll
        for (int q = p; q < Q; ++q) row[p][q] = in && q * 64 < m ? rows[(size_t)(p * 64 + lane) * Q + q] : 0ull;
        const int c = m - p * 64;
        left[p] = c >= 64 ? ~0ull : (c > 0 ? (1ull << c) - 1 : 0ull);
    }
    int kept = 0, place[Q];  // place: the lane's candidates' places among the kept
#pragma unroll
    for (int p = 0; p < Q; ++p) {
        place[p] = -1;
        while (left[p] && kept < a.max_det) {
            const int i = __ffsll(left[p]) - 1;
            if (lane == i) place[p] = kept;
            ++kept;
#pragma unroll
            for (int q = p; q < Q; ++q) left[q] &= ~lane_of(row[p][q], i);
            left[p] &= ~(1ull << i);
        }
    }
#pragma unroll
    for (int p = 0; p < Q; ++p)
        if (place[p] >= 0) {
            const unsigned long long kv = skey[p * 64 + lane];
            float *d = a.dets + (obase + place[p]) * 5;
            d[0] = __uint_as_float((unsigned)(kv >> 32));
            d[1] = box[p].x; d[2] = box[p].y; d[3] = box[p].z; d[4] = box[p].w;
            a.det_index[obase + place[p]] = (int)~(unsigned)(kv & 0xFFFFFFFFull);
        }
    if (lane == 0) *count = kept;
}
constexpr size_t NMS_SMALL_LDS = 256 * 8 + 256 * (8 + 16 + 4 * 8);  // key, skey, sbox, rows at Q = 4

// Sort key: score bits (scores are >= 0, so their bits order like the
// values) above the complemented box index, descending = score desc, index asc.
// Keys differ, so the order they were collected in does not matter.
__global__ void __launch_bounds__(256) detect_nms(DetectArgs a)
{
    extern __shared__ __align__(16) unsigned char nms_raw[];
    const int B = a.H * a.W * a.A;
    int PB = 1;
    while (PB < B) PB <<= 1;
    unsigned long long *key = reinterpret_cast<unsigned long long *>(nms_raw);   // [PB]
    float4 *cbox = reinterpret_cast<float4 *>(nms_raw + (size_t)PB * 8);        // [PB]
    unsigned char *keep = nms_raw + (size_t)PB * 24;                              // [PB]
    __shared__ int ncand;
    const int n = blockIdx.x / a.C, k = blockIdx.x - (blockIdx.x / a.C) * a.C;
    const int tid = threadIdx.x, lane = tid & 63;
    const float *sc = a.score + ((size_t)n * a.C + k) * B;
    if (tid == 0) ncand = 0;
    __syncthreads();
    // candidates -> key[0 .. m), in no particular order; 4 score loads in flight
    for (int e0 = tid; e0 < B + tid; e0 += 1024) {
        float s[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) s[q] = e0 + q * 256 < B ? sc[e0 + q * 256] : 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = e0 + q * 256;
            const bool c = e < B && s[q] >= a.thresh;
            const unsigned long long vote = __ballot(c);
            if (vote == 0) continue;
            int base = 0;
            if (lane == 0) base = atomicAdd(&ncand, __popcll(vote));
            base = __shfl(base, 0);
            if (c) key[base + __popcll(vote & ((1ull << lane) - 1))] = ((unsigned long long)__float_as_uint(s[q]) << 32) | (unsigned)(~(unsigned)e);
        }
    }
    __syncthreads();
    const int m = ncand;
    const float4 *bx = reinterpret_cast<const float4 *>(a.box) + (size_t)n * B;
    const size_t obase = ((size_t)n * a.C + k) * a.max_det;
    if (m <= 256) {
        int *count = a.counts + (size_t)n * a.C + k;
        if (m <= 64) nms_small<1>(a, key, m, bx, obase, count);
        else if (m <= 128) nms_small<2>(a, key, m, bx, obase, count);
        else nms_small<4>(a, key, m, bx, obase, count);
        return;
    }
    // more: bitonic sort of the next power of two in LDS, descending
    int P = 512;
    while (P < m) P <<= 1;
    for (int e = m + tid; e < P; e += 256) key[e] = 0ull;
    for (int size = 2; size <= P; size <<= 1) {
        for (int stride = size >> 1; stride > 0; stride >>= 1) {
            __syncthreads();
            for (int e = tid; e < P / 2; e += 256) {
                const int lo = 2 * e - (e & (stride - 1));
                const int hi = lo + stride;
                const bool desc = (lo & size) == 0;
                const unsigned long long x = key[lo], y = key[hi];
                if ((x < y) == desc) {
                    key[lo] = y;
                    key[hi] = x;
                }
            }
        }
    }
    __syncthreads();
    for (int e = tid; e < m; e += 256) {
        cbox[e] = bx[~(unsigned)(key[e] & 0xFFFFFFFFull)];
        keep[e] = 1;
    }
    __syncthreads();
    int kept = 0;
    for (int i = 0; i < m && kept < a.max_det; ++i) {
        if (!keep[i]) continue;  // uniform: keep[] is only written before the barrier below
        const float4 bi = cbox[i];
        if (tid == 0) {
            const unsigned bidx = ~(unsigned)(key[i] & 0xFFFFFFFFull);
            float *d = a.dets + (obase + kept) * 5;
            d[0] = __uint_as_float((unsigned)(key[i] >> 32));
            d[1] = bi.x; d[2] = bi.y; d[3] = bi.z; d[4] = bi.w;
            a.det_index[obase + kept] = (int)bidx;
        }
        ++kept;
        for (int j = i + 1 + tid; j < m; j += 256)
            if (keep[j] && box_iou(bi, cbox[j]) > a.nms_thresh) keep[j] = 0;
        __syncthreads();
    }
    if (tid == 0) a.counts[(size_t)n * a.C + k] = kept;
}

size_t detect_nms_lds(int boxes)
{
    int P = 1;
    while (P < boxes) P <<= 1;
    return std::max((size_t)P * 25, NMS_SMALL_LDS);
}

// ---------------------------------------------------------------- fixed scratch
// The decoded scores and boxes of dn_detect_noalloc live here instead of in a
// caller workspace.  Each GPU the library runs on holds its own copy for the
// life of the process; calls on one GPU share it.  In host code the array's
// name is not a device address: its address is taken once per device with
// hipGetSymbolAddress (that device current) and only that address is used.
static __device__ __align__(256) unsigned char scratch[DETECT_NOALLOC_BYTES];

hipError_t detect_scratch(void **ptr)
{
    constexpr int MAX_DEVICES = 64;
    static std::mutex mu;
    static void *addr[MAX_DEVICES] = {};
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> g(mu);
    if (!addr[dev]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        addr[dev] = p;
    }
    *ptr = addr[dev];
    return hipSuccess;
}

hipError_t launch_detect(const DetectArgs &a, hipStream_t s)
{
    const int B = a.H * a.W * a.A;
    const long total = (long)a.N * B;
    const dim3 g((unsigned)((total + 63) / 64)), b(64);  // one wave: spread over the CUs
    if (a.C <= 24) hipLaunchKernelGGL(detect_decode<24>, g, b, 0, s, a);
    else if (a.C <= 96) hipLaunchKernelGGL(detect_decode<96>, g, b, 0, s, a);
    else hipLaunchKernelGGL(detect_decode<0>, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a);
    const size_t lds = detect_nms_lds(B);
    if (lds > 64 * 1024)
        (void)hipFuncSetAttribute((const void *)detect_nms, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    hipLaunchKernelGGL(detect_nms, dim3((unsigned)(a.N * a.C)), dim3(256), lds, s, a);
    return hipGetLastError();
}

}  // namespace dnk
