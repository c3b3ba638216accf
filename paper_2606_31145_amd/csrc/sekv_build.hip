// Prefill-side cache builder for gfx950: the step before the decode path (Sec. 3.1 and
// Sec. 3.2).  Three kernels:
//
//   segment_kernel   surprisal segmentation of one sequence per workgroup: mu and sigma
//                    of the sequence's surprisal in one fixed summation order (1024
//                    strided float64 partials, then halving), boundaries where
//                    H_t > mu + alpha sigma, the local window, runs between neighbouring
//                    anchors shorter than min_span back to full resolution; anchors and
//                    spans listed in token order.  Integer results, exact.
//   gather_kernel    anchor rows of the token keys/values into the anchor arrays, and the
//                    surprisal-weighted mean key and value of every span (eq.
//                    surprisal_weight; float32 accumulation), |S| and ln|S|.
//   svd_kernel       (sekv_svd.h) one (sequence, KV head, span, side) per workgroup: a randomized
//                    truncated SVD of the span's |S| x d matrix (eq. key_svd); the factors
//                    go into the span's block of the factor arena, stored with the rank
//                    rounded up to the 16-byte granule (the extra components zero).

#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include "sekv_internal.h"
#include "sekv_build_internal.h"

namespace sekv {

// defined in sekv_svd_inst.hip, one object per (element bytes, head_dim)
hipError_t launch_svd_2_128(const BuildArgs &a, unsigned items, bool wide, hipStream_t s);
hipError_t launch_svd_2_64(const BuildArgs &a, unsigned items, bool wide, hipStream_t s);
hipError_t launch_svd_4_128(const BuildArgs &a, unsigned items, bool wide, hipStream_t s);
hipError_t launch_svd_4_64(const BuildArgs &a, unsigned items, bool wide, hipStream_t s);

namespace {

constexpr unsigned kWideSides = 512;    // span sides up to which each gets four waves
constexpr int kSegThreads = 1024;
constexpr int BT = 256;                 // builder threads per workgroup
constexpr int kMaxL = 40;               // largest sketch width

__device__ inline float ld_elem(const void *base, size_t i, int elem) {
    if (elem == 2) {
        const uint16_t u = reinterpret_cast<const uint16_t *>(base)[i];
        return __uint_as_float(uint32_t(u) << 16);
    }
    return reinterpret_cast<const float *>(base)[i];
}

__device__ inline void st_elem(void *base, size_t i, float v, int elem) {
    if (elem == 2) {
        uint32_t u = __float_as_uint(v);
        u += 0x7FFFu + ((u >> 16) & 1u);                 // round to nearest even
        reinterpret_cast<uint16_t *>(base)[i] = uint16_t(u >> 16);
    } else {
        reinterpret_cast<float *>(base)[i] = v;
    }
}

// ---------------------------------------------------------------------------
// segmentation
// ---------------------------------------------------------------------------

// Exclusive scan of cnt[0, kSegThreads) in place (Hillis-Steele); returns the total.
__device__ int block_scan(int *cnt, int *tmp, int tid) {
    int v = cnt[tid];
    for (int off = 1; off < kSegThreads; off <<= 1) {
        tmp[tid] = v;
        __syncthreads();
        if (tid >= off) v += tmp[tid - off];
        __syncthreads();
    }
    tmp[tid] = v;                                       // inclusive
    __syncthreads();
    const int total = tmp[kSegThreads - 1];
    cnt[tid] = tid > 0 ? tmp[tid - 1] : 0;
    __syncthreads();
    return total;
}

// Sum of the values in the fixed order of the segmentation rule.
__device__ double fixed_order_sum(double mine, double *part, int tid) {
    part[tid] = mine;
    __syncthreads();
    for (int h = kSegThreads / 2; h >= 1; h >>= 1) {
        if (tid < h) part[tid] = part[tid] + part[tid + h];
        __syncthreads();
    }
    const double s = part[0];
    __syncthreads();
    return s;
}

__global__ void __launch_bounds__(kSegThreads) segment_kernel(SegArgs a) {
    __shared__ double part[kSegThreads];
    __shared__ int cnt[kSegThreads], tmp[kSegThreads];
    const int tid = threadIdx.x, b = blockIdx.x;
    int n = a.n_tokens[b];
    n = n < 0 ? 0 : (n > a.N ? a.N : n);
    const float *H = a.surprisal + size_t(b) * a.N;
    unsigned char *flag = a.ws_flag + size_t(b) * a.N;
    unsigned char *inspan = a.ws_inspan + size_t(b) * a.N;
    int32_t *pos = a.ws_pos + size_t(b) * (a.N + 2);
    int32_t *anchor_idx = a.anchor_idx + size_t(b) * a.N;
    int32_t *span_start = a.span_start + size_t(b) * a.N;
    int32_t *span_len = a.span_len + size_t(b) * a.N;
    if (n == 0) {
        if (tid == 0) { a.n_anchors[b] = 0; a.n_spans[b] = 0; }
        return;
    }
    // 1. mu and sigma, each sum in the fixed order; no fused multiply-add anywhere
    double thr;
    {
#pragma clang fp contract(off)
        double acc = 0.0;
        for (int t = tid; t < n; t += kSegThreads) acc = acc + double(H[t]);
        const double mu = fixed_order_sum(acc, part, tid) / double(n);
        double acc2 = 0.0;
        for (int t = tid; t < n; t += kSegThreads) {
            const double dv = double(H[t]) - mu;
            const double sq = dv * dv;
            acc2 = acc2 + sq;
        }
        const double sigma = sqrt(fixed_order_sum(acc2, part, tid) / double(n));
        const double as = a.alpha * sigma;
        thr = mu + as;
    }
    // 2. boundary and window flags; inspan cleared
    for (int t = tid; t < n; t += kSegThreads) {
        flag[t] = (double(H[t]) > thr || t >= n - a.window) ? 1 : 0;
        inspan[t] = 0;
    }
    __syncthreads();
    // 3. positions of the flagged tokens, in order, between sentinels -1 and n
    const int chunk = (n + kSegThreads - 1) / kSegThreads;
    const int t0 = tid * chunk, t1 = min(n, t0 + chunk);
    int c = 0;
    for (int t = t0; t < t1; ++t) c += flag[t];
    cnt[tid] = c;
    __syncthreads();
    const int m = block_scan(cnt, tmp, tid);
    {
        int w = cnt[tid];
        for (int t = t0; t < t1; ++t)
            if (flag[t]) pos[1 + w++] = t;
    }
    if (tid == 0) { pos[0] = -1; pos[m + 1] = n; }
    __syncthreads();
    // 4. the m + 1 gaps between consecutive positions: long ones are spans
    const int ng = m + 1;
    const int gchunk = (ng + kSegThreads - 1) / kSegThreads;
    const int g0 = tid * gchunk, g1 = min(ng, g0 + gchunk);
    c = 0;
    for (int i = g0; i < g1; ++i) c += (pos[i + 1] - pos[i] - 1 >= a.min_span) ? 1 : 0;
    cnt[tid] = c;
    __syncthreads();
    const int ns = block_scan(cnt, tmp, tid);
    {
        int w = cnt[tid];
        for (int i = g0; i < g1; ++i) {
            const int s = pos[i] + 1, L = pos[i + 1] - pos[i] - 1;
            if (L >= a.min_span) {
                span_start[w] = s;
                span_len[w] = L;
                ++w;
                for (int t = s; t < s + L; ++t) inspan[t] = 1;
            }
        }
    }
    __syncthreads();
    // 5. anchors: every token outside the spans, in order
    c = 0;
    for (int t = t0; t < t1; ++t) c += inspan[t] ? 0 : 1;
    cnt[tid] = c;
    __syncthreads();
    const int na = block_scan(cnt, tmp, tid);
    {
        int w = cnt[tid];
        for (int t = t0; t < t1; ++t)
            if (!inspan[t]) anchor_idx[w++] = t;
    }
    if (tid == 0) { a.n_anchors[b] = na; a.n_spans[b] = ns; }
}

// ---------------------------------------------------------------------------
// anchors and summaries
// ---------------------------------------------------------------------------

// Tokens of sequence b, clamped to [0, N] as the segmentation clamps them.
__device__ inline int seq_tokens(const BuildArgs &a, int b) {
    const int n = a.n_tokens[b];
    return n < 0 ? 0 : min(n, a.N);
}

// An anchor index or span outside the sequence's tokens: the row or span is skipped.
__device__ inline void flag_table(const BuildArgs &a) {
    __hip_atomic_fetch_or(a.error, kErrSelRange, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// grid = B * Hkv * rows workgroups; workgroup (pair, y) copies anchor rows
// [64 y, 64 y + 64) and summarises span y.
__global__ void __launch_bounds__(BT) gather_kernel(BuildArgs a, int rows) {
    const int pair = blockIdx.x / rows, b = pair / a.Hkv, g = pair % a.Hkv;
    const int y = blockIdx.x % rows, tid = threadIdx.x;
    const int d = a.d, e = a.elem;
    const size_t tok0 = size_t(pair) * a.N;                 // row of token 0 of (b, g)
    const int nt = seq_tokens(a, b);
    int na = a.n_anchors[b];
    na = na < 0 ? 0 : min(na, min(a.A_max, a.N));
    int ns = a.n_spans[b];
    ns = ns < 0 ? 0 : min(ns, min(a.M_max, a.N));
    // anchor rows
    for (int i = tid; i < 64 * d; i += BT) {
        const int r = y * 64 + i / d, col = i % d;
        if (r < na) {
            const int t = a.anchor_idx[size_t(b) * a.N + r];
            if (t >= 0 && t < nt) {
                const size_t dst = (size_t(pair) * a.A_max + r) * d + col;
                st_elem(a.anchor_k, dst, ld_elem(a.keys, (tok0 + t) * d + col, e), e);
                st_elem(a.anchor_v, dst, ld_elem(a.values, (tok0 + t) * d + col, e), e);
            } else if (col == 0) {
                flag_table(a);
            }
        }
    }
    // span y: surprisal-weighted means; |S| and ln|S| once per sequence (g == 0)
    if (y >= ns) return;
    const int s0 = a.span_start[size_t(b) * a.N + y];
    int L = a.span_len_seg[size_t(b) * a.N + y];
    if (s0 < 0 || L < 1 || s0 + L > nt) {
        if (tid == 0 && g == 0) flag_table(a);
        return;
    }
    __shared__ float red[2][BT];
    __shared__ float hs;
    // weight normaliser sum_t H_t over the span (float64 then float32)
    {
        double acc = 0.0;
        for (int t = tid; t < L; t += BT) acc += double(a.surprisal[size_t(b) * a.N + s0 + t]);
        red[0][tid] = float(acc);
        __syncthreads();
        if (tid == 0) {
            double s = 0.0;
            for (int i = 0; i < BT; ++i) s += double(red[0][i]);
            hs = float(s);
        }
        __syncthreads();
    }
    const float tot = hs;
    const bool uniform = !(tot > 0.0f);
    // thread: column col, token parity par (two tokens streams), then one pass through LDS
    const int col = tid % d, par = tid / d, npar = BT / d;
    float ak = 0.0f, av = 0.0f;
    for (int t = par; t < L; t += npar) {
        const float w = uniform ? 1.0f / float(L) : a.surprisal[size_t(b) * a.N + s0 + t] / tot;
        ak += w * ld_elem(a.keys, (tok0 + s0 + t) * d + col, e);
        av += w * ld_elem(a.values, (tok0 + s0 + t) * d + col, e);
    }
    red[0][tid] = ak;
    red[1][tid] = av;
    __syncthreads();
    if (par == 0) {
        float sk = 0.0f, sv = 0.0f;
        for (int p = 0; p < npar; ++p) { sk += red[0][p * d + col]; sv += red[1][p * d + col]; }
        const size_t dst = (size_t(pair) * a.M_max + y) * d + col;
        st_elem(a.sum_k, dst, sk, e);
        st_elem(a.sum_v, dst, sv, e);
    }
    if (g == 0 && tid == 0) {
        a.span_len_out[size_t(b) * a.M_max + y] = L;
        a.span_logsize[size_t(b) * a.M_max + y] = log(double(L));
    }
}

}  // namespace

hipError_t launch_segment(const SegArgs &a, int batch, hipStream_t stream) {
    if (batch <= 0) return hipSuccess;
    hipLaunchKernelGGL(segment_kernel, dim3(unsigned(batch)), dim3(kSegThreads), 0, stream, a);
    return hipGetLastError();
}

hipError_t launch_build(const BuildArgs &a, int batch, hipStream_t stream) {
    if (batch <= 0) return hipSuccess;
    if (a.d > 128 || a.l > kMaxL || a.l < 2 || a.R > kMaxL) return hipErrorInvalidValue;
    const unsigned pairs = unsigned(batch * a.Hkv);
    const int rows = max(max((a.A_max + 63) / 64, a.M_max), 1);
    hipLaunchKernelGGL(gather_kernel, dim3(pairs * unsigned(rows)), dim3(BT), 0, stream, a, rows);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess || a.M_max == 0) return err;
    // four waves per span side while the sides (an upper bound: M_max per pair) leave CUs
    // without one
    const unsigned items = pairs * unsigned(a.M_max);
    const bool wide = items * 2 <= kWideSides;
    if (a.elem == 2)
        return a.d == 128 ? launch_svd_2_128(a, items, wide, stream) : launch_svd_2_64(a, items, wide, stream);
    return a.d == 128 ? launch_svd_4_128(a, items, wide, stream) : launch_svd_4_64(a, items, wide, stream);
}

}  // namespace sekv
