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

// Span sides up to which each gets four waves.  The wide variant holds one workgroup a CU at d 128,
// so past 256 sides it takes two rounds; a lone wave takes one round up to 1024.  us at d 128, sketch 40,
// one wave / four: bfloat16 192 sides 517 / 306, 304 515 / 512, 400 528 / 531, 544 530 / 698; float32 304 876 / 640,
// 544 884 / 824, 752 884 / 1031; d 64, sketch 24: 400 234 / 230, 544 243 / 312 and 369 / 292, 377 / 363.
constexpr unsigned kWideSides = 512;
constexpr int kSegThreads = 1024;
constexpr int BT = 256;                 // builder threads per workgroup
constexpr int kMaxL = 40;               // largest sketch width

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

// Exclusive prefix of each thread's v over the workgroup (kSegThreads threads); *total gets
// the sum.  `part`: one int per wave.
__device__ int block_scan(int v, int *part, int tid, int *total) {
    const int lane = tid & 63, wave = tid >> 6;
    int x = v;
    for (int off = 1; off < 64; off <<= 1) {
        const int y = __shfl_up(x, off, 64);
        if (lane >= off) x += y;
    }
    if (lane == 63) part[wave] = x;
    __syncthreads();
    int base = 0, sum = 0;
    for (int w = 0; w < kSegThreads / 64; ++w) {
        const int p = part[w];
        if (w < wave) base += p;
        sum += p;
    }
    __syncthreads();
    *total = sum;
    return base + x - v;
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

// One workgroup per sequence.  Bound by the latency of one CU's loads: three passes over the
// surprisal (the two sums, whose order is fixed, and the flags), each with kAhead loads in
// flight per thread.  Flags stay in registers as 64-token ballots, and spans and anchors come
// from the list of flagged positions alone: 131072 tokens took 380 us with byte flags
// in memory that each thread read back token by token.
__global__ void __launch_bounds__(kSegThreads) segment_kernel(SegArgs a) {
    constexpr int kAhead = 16;
    __shared__ double part[kSegThreads];
    __shared__ int wsum[kSegThreads / 64];
    const int tid = threadIdx.x, b = blockIdx.x, lane = tid & 63, wave = tid >> 6;
    int n = a.n_tokens[b];
    n = n < 0 ? 0 : (n > a.N ? a.N : n);
    const float *H = a.surprisal + size_t(b) * a.N;
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
        for (int t0 = tid; t0 < n; t0 += kAhead * kSegThreads) {
            float h[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) h[u] = t0 + u * kSegThreads < n ? H[t0 + u * kSegThreads] : 0.0f;
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (t0 + u * kSegThreads < n) acc = acc + double(h[u]);
        }
        const double mu = fixed_order_sum(acc, part, tid) / double(n);
        double acc2 = 0.0;
        for (int t0 = tid; t0 < n; t0 += kAhead * kSegThreads) {
            float h[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) h[u] = t0 + u * kSegThreads < n ? H[t0 + u * kSegThreads] : 0.0f;
#pragma unroll
            for (int u = 0; u < kAhead; ++u)
                if (t0 + u * kSegThreads < n) {
                    const double dv = double(h[u]) - mu;
                    const double sq = dv * dv;
                    acc2 = acc2 + sq;
                }
        }
        const double sigma = sqrt(fixed_order_sum(acc2, part, tid) / double(n));
        const double as = a.alpha * sigma;
        thr = mu + as;
    }
    // 2. positions of the flagged tokens (boundaries and the local window), in order, between
    //    sentinels -1 and n.  A thread owns 64 consecutive tokens of a tile of 65536: its
    //    wave forms the 64 ballots, one group of 64 tokens after another.
    constexpr int kTileTokens = 64 * kSegThreads;
    int m = 0;
    for (int t0 = 0; t0 < n; t0 += kTileTokens) {
        const int w0 = t0 + wave * 64 * 64;                  // the wave's first token
        uint64_t mine = 0;
        for (int g0 = 0; g0 < 64 && w0 + g0 * 64 < n; g0 += kAhead) {
            float h[kAhead];
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int t = w0 + (g0 + u) * 64 + lane;
                h[u] = t < n ? H[t] : 0.0f;
            }
#pragma unroll
            for (int u = 0; u < kAhead; ++u) {
                const int t = w0 + (g0 + u) * 64 + lane;
                const uint64_t word = __ballot(t < n && (double(h[u]) > thr || t >= n - a.window));
                if (lane == g0 + u) mine = word;
            }
        }
        int total;
        int at = m + block_scan(__popcll(mine), wsum, tid, &total);
        const int first = w0 + lane * 64;
        for (uint64_t x = mine; x; x &= x - 1) pos[1 + at++] = first + __builtin_ctzll(x);
        m += total;
    }
    if (tid == 0) { pos[0] = -1; pos[m + 1] = n; }
    __syncthreads();
    // 3. the m + 1 gaps between consecutive positions: long ones are spans; the tokens of the
    //    others, and the position that ends each gap but the last, are anchors
    const int ng = m + 1;
    const int gchunk = (ng + kSegThreads - 1) / kSegThreads;
    const int g0 = min(ng, tid * gchunk), g1 = min(ng, g0 + gchunk);
    int cs = 0, ca = 0;
    for (int i = g0; i < g1; ++i) {
        const int L = pos[i + 1] - pos[i] - 1;
        if (L >= a.min_span) ++cs;
        else ca += L;
        if (i < m) ++ca;
    }
    int ns, na;
    int ws = block_scan(cs, wsum, tid, &ns);
    int wa = block_scan(ca, wsum, tid, &na);
    // A run of anchors longer than kGapAlone is written by the whole wave: one lane alone makes the
    // kernel 3.7 ms long for a sequence of 131072 tokens under a min_span past them, the wave 0.14 ms.
    // Below, a lane's own run is at most half a wave's step.
    constexpr int kGapAlone = 32;
    for (int u = 0; u < gchunk; ++u) {
        const int i = g0 + u;
        const bool on = i < g1;
        const int p0 = on ? pos[i] : 0, p1 = on ? pos[i + 1] : 0, L = p1 - p0 - 1;
        const bool anchors = on && L < a.min_span;
        for (uint64_t gaps = __ballot(anchors && L > kGapAlone); gaps; gaps &= gaps - 1) {
            const int src = __builtin_ctzll(gaps);
            const int first = __shfl(p0, src, 64) + 1, n_gap = __shfl(L, src, 64), at = __shfl(wa, src, 64);
            for (int t = lane; t < n_gap; t += 64) anchor_idx[at + t] = first + t;
        }
        if (anchors) {
            if (L <= kGapAlone)
                for (int t = 0; t < L; ++t) anchor_idx[wa + t] = p0 + 1 + t;
            wa += L;
        } else if (on) {
            span_start[ws] = p0 + 1;
            span_len[ws] = L;
            ++ws;
        }
        if (on && i < m) anchor_idx[wa++] = p1;
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

// Sixteen bytes of stored values as float32.
template <int ELEM>
__device__ inline void unpack16(const uint4 &v, float (&f)[16 / ELEM]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if constexpr (ELEM == 2) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xFFFF0000u);
        } else {
            f[i] = __uint_as_float(w[i]);
        }
    }
}

// grid = B * Hkv * per workgroups: of a pair's, the first ab copy 64 anchor rows each, the others
// summarise one span each.  Both move 16-byte pieces, a row per D ELEM / 16
// lanes; a span's rows go round the workgroup with kAhead of them per thread in flight, so
// the tokens are read at the rate of memory (128K x 4: 2.1 GB; 2.25 ms with one 2-byte load
// after another per thread).
template <int ELEM, int D>
__global__ void __launch_bounds__(BT) gather_kernel(BuildArgs a, int ab, int per) {
    constexpr int VEC = 16 / ELEM, LPR = D / VEC, RPP = BT / LPR;    // values, lanes per row, rows per pass
    constexpr int kAhead = 4;
    const int pair = blockIdx.x / per, b = pair / a.Hkv, g = pair % a.Hkv;
    const int y = int(blockIdx.x % per) - ab, tid = threadIdx.x;
    const int rg = tid / LPR, col = tid % LPR;
    const uint4 *K = static_cast<const uint4 *>(a.keys) + size_t(pair) * a.N * LPR;
    const uint4 *V = static_cast<const uint4 *>(a.values) + size_t(pair) * a.N * LPR;
    const int nt = seq_tokens(a, b);
    if (y < 0) {
        int na = a.n_anchors[b];
        na = na < 0 ? 0 : min(na, min(a.A_max, a.N));
        const int r0 = (y + ab) * 64;
        for (int r = r0 + rg; r < min(na, r0 + 64); r += RPP) {
            const int t = a.anchor_idx[size_t(b) * a.N + r];
            if (t >= 0 && t < nt) {
                const size_t dst = (size_t(pair) * a.A_max + r) * LPR + col;
                static_cast<uint4 *>(a.anchor_k)[dst] = K[size_t(t) * LPR + col];
                static_cast<uint4 *>(a.anchor_v)[dst] = V[size_t(t) * LPR + col];
            } else if (col == 0) {
                flag_table(a);
            }
        }
        return;
    }
    // span y: surprisal-weighted means; |S| and ln|S| once per sequence (g == 0)
    int ns = a.n_spans[b];
    ns = ns < 0 ? 0 : min(ns, min(a.M_max, a.N));
    if (y >= ns) return;
    const int s0 = a.span_start[size_t(b) * a.N + y];
    const int L = a.span_len_seg[size_t(b) * a.N + y];
    if (s0 < 0 || L < 1 || s0 + L > nt) {
        if (tid == 0 && g == 0) flag_table(a);
        return;
    }
    __shared__ float red[2][RPP][D];
    __shared__ double wtot[BT / 64];
    const float *H = a.surprisal + size_t(b) * a.N + s0;
    // weight normaliser sum_t H_t over the span (float64, then float32)
    {
        double acc = 0.0;
        for (int t = tid; t < L; t += BT) acc += double(H[t]);
        for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off, 64);
        if ((tid & 63) == 0) wtot[tid >> 6] = acc;
        __syncthreads();
    }
    const float tot = float((wtot[0] + wtot[1]) + (wtot[2] + wtot[3]));
    const bool uniform = !(tot > 0.0f);
    K += size_t(s0) * LPR + col;
    V += size_t(s0) * LPR + col;
    float ak[VEC], av[VEC];
#pragma unroll
    for (int i = 0; i < VEC; ++i) ak[i] = av[i] = 0.0f;
    for (int t0 = rg; t0 < L; t0 += kAhead * RPP) {
        uint4 kv[kAhead], vv[kAhead];
        float w[kAhead];
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            const int t = t0 + u * RPP, tc = min(t, L - 1);
            kv[u] = K[size_t(tc) * LPR];
            vv[u] = V[size_t(tc) * LPR];
            w[u] = t < L ? (uniform ? 1.0f / float(L) : H[tc] / tot) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kAhead; ++u) {
            if (t0 + u * RPP < L) {
                float f[VEC];
                unpack16<ELEM>(kv[u], f);
#pragma unroll
                for (int i = 0; i < VEC; ++i) ak[i] += w[u] * f[i];
                unpack16<ELEM>(vv[u], f);
#pragma unroll
                for (int i = 0; i < VEC; ++i) av[i] += w[u] * f[i];
            }
        }
    }
#pragma unroll
    for (int i = 0; i < VEC; ++i) {
        red[0][rg][col * VEC + i] = ak[i];
        red[1][rg][col * VEC + i] = av[i];
    }
    __syncthreads();
    for (int i = tid; i < 2 * D; i += BT) {
        const int side = i / D, c = i % D;
        float s = 0.0f;
        for (int p = 0; p < RPP; ++p) s += red[side][p][c];
        st_elem(side ? a.sum_v : a.sum_k, (size_t(pair) * a.M_max + y) * D + c, s, ELEM);
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
    const int blocks = (a.A_max + 63) / 64;             // of anchor rows
    auto gather = [&](int ab, int per) {
        const dim3 grid(pairs * unsigned(per));
        if (a.elem == 2) {
            if (a.d == 128) hipLaunchKernelGGL((gather_kernel<2, 128>), grid, dim3(BT), 0, stream, a, ab, per);
            else hipLaunchKernelGGL((gather_kernel<2, 64>), grid, dim3(BT), 0, stream, a, ab, per);
        } else {
            if (a.d == 128) hipLaunchKernelGGL((gather_kernel<4, 128>), grid, dim3(BT), 0, stream, a, ab, per);
            else hipLaunchKernelGGL((gather_kernel<4, 64>), grid, dim3(BT), 0, stream, a, ab, per);
        }
    };
    // anchors and spans in one launch while it has fewer than 2^32 threads, HIP's limit, else one each
    if (uint64_t(pairs) * uint64_t(blocks + a.M_max) * BT < uint64_t(1) << 32) {
        gather(blocks, blocks + a.M_max);
    } else {
        gather(blocks, blocks);
        if (a.M_max > 0) gather(0, a.M_max);
    }
    hipError_t err = hipGetLastError();
    if (err != hipSuccess || a.M_max == 0) return err;
    // four waves per span side while the sides (an upper bound: M_max per pair, the counts are on
    // the device) are few
    const unsigned items = pairs * unsigned(a.M_max);
    const bool wide = items * 2 <= kWideSides;
    if (a.elem == 2)
        return a.d == 128 ? launch_svd_2_128(a, items, wide, stream) : launch_svd_2_64(a, items, wide, stream);
    return a.d == 128 ? launch_svd_4_128(a, items, wide, stream) : launch_svd_4_64(a, items, wide, stream);
}

}  // namespace sekv
