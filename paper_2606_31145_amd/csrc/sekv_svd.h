// Randomized truncated SVD of one span side (one (sequence, KV head, span, side) per
// workgroup): the span's |S| x d matrix X (eq. key_svd, rank r = min(|S|, d, R_max)).
//
//   sketch     Y = X Omega with a d x l test matrix; G = Y^T Y (float64), P = Y^T X (float32)
//   factor     G = R^T R by Cholesky with diagonal pivoting, stopped where the remaining
//              pivots fall below 1e-8 of the largest diagonal (a rank-deficient sketch keeps
//              k < l columns); C = R^-T in the same loop, so Q = Y C^T is an orthonormal basis
//              of the sketch's range and B = Q^T X = C P; M = B B^T (float64)
//   iterate    each subspace iteration sketches again with an orthonormal basis of P's (and
//              B's) row space, C_P P with C_P the inverse factor of P P^T
//   diagonal   M = E diag(sigma^2) E^T by one-sided Jacobi on the columns of M's Cholesky
//              factor (W W^T = M; W J has orthogonal columns E diag(sigma))
//   output     T = C^T E; a last pass over X forms U = Y T; V diag(sigma) = P^T T
//
// What bounds it: a span side is a long chain of small steps (three passes over 30 to 300 KB
// of L2-resident tokens, two to four 40 x 40 factorisations, 200 to 250 Jacobi rounds), and a
// layer has tens of thousands of them.  So a side runs in ONE wave (its steps need no
// workgroup barrier) and eight sides share a CU, two waves a SIMD.  Counted over a 128K x 4 layer, a
// wave spends 30 % of its cycles in vector instructions, 44 % waiting for one to issue (its own
// dependences, and the other wave) and 18 % for memory or LDS; the matrix cores are busy 40 % of
// the time.  That leaves 20 KB of LDS and 256 registers a side, hence: no copy of B, X or P is kept (M is formed
// tile by tile, the last pass forms P again), and LDS holds either the pass's tiles or one
// 40 x 40 matrix.  The dense products run on the matrix cores: bf16 MFMA where the operands
// are bf16 values (X, Omega) or exact three-way bf16 splits of float32 values (Y), float64
// MFMA for the Gram matrices and everything that multiplies C, E or T, so no sum is formed
// at a lower precision than its result needs.  Operands are used in the register layout
// that the product before left them in (contraction indices are permuted on both sides
// alike), so between products nothing moves through LDS except the transposed reads of X.
// A layer with too few span sides to fill the chip uses four waves per side instead, which
// share the passes.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sekv_internal.h"
#include "sekv_build_internal.h"

namespace sekv {
namespace {

constexpr int kMaxL = 40;                       // largest sketch width
template <bool B> struct Bool { static constexpr bool value = B; };

typedef double d4_t __attribute__((ext_vector_type(4)));
typedef float f4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf8_t __attribute__((ext_vector_type(8)));
typedef short s4_t __attribute__((ext_vector_type(4)));

__device__ inline d4_t mfma64(double a, double b, d4_t c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline f4_t mfma32(float a, float b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}
__device__ inline f4_t mfma_k32(const uint4 &a, const uint4 &b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8_t, a), __builtin_bit_cast(bf8_t, b), c, 0,
                                                   0, 0);
}
__device__ inline f4_t mfma_k16(const uint2 &a, const uint2 &b, f4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s4_t, a), __builtin_bit_cast(s4_t, b), c, 0, 0,
                                                     0);
}

// Four rows of one column of a bf16 tile in LDS: within 16 lanes, lane i names 4 columns
// 4 (i % 4) of row slot i / 4 and receives column i of the four row slots.
__device__ inline uint2 lds_tr4(const uint16_t *p) {
    typedef __attribute__((address_space(3))) s4_t *lds_p;
    const s4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(reinterpret_cast<lds_p>(reinterpret_cast<uintptr_t>(p)));
    return __builtin_bit_cast(uint2, v);
}

// LDS accesses of one wave complete in order; this keeps the compiler from moving one
// across the point where another lane's value is needed.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// A copy of a lane index that the compiler cannot see through: address arithmetic on it
// stays in its phase instead of being kept in registers across the others.
__device__ inline int opaque(int v) {
    int t;
    asm volatile("v_mov_b32 %0, %1" : "=v"(t) : "v"(v));
    return t;
}

// Four float32 values as bf16 pieces whose sum is exact: hi + mid + lo (8 bits each).
__device__ inline void split3(const float (&y)[4], uint2 &hi, uint2 &mid, uint2 &lo) {
    uint32_t h[4], m[4], l[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        h[i] = __float_as_uint(y[i]);
        const float r1 = y[i] - __uint_as_float(h[i] & 0xFFFF0000u);
        m[i] = __float_as_uint(r1);
        l[i] = __float_as_uint(r1 - __uint_as_float(m[i] & 0xFFFF0000u));
    }
    constexpr uint32_t kHigh = 0x07060302u;     // the high halves of two words
    hi = make_uint2(__builtin_amdgcn_perm(h[1], h[0], kHigh), __builtin_amdgcn_perm(h[3], h[2], kHigh));
    mid = make_uint2(__builtin_amdgcn_perm(m[1], m[0], kHigh), __builtin_amdgcn_perm(m[3], m[2], kHigh));
    lo = make_uint2(__builtin_amdgcn_perm(l[1], l[0], kHigh), __builtin_amdgcn_perm(l[3], l[2], kHigh));
}

__device__ inline uint32_t bf16_rne(float f) {
    uint32_t q = __float_as_uint(f);
    q += 0x7FFFu + ((q >> 16) & 1u);
    return q >> 16;
}

template <int ELEM>
__device__ inline void st_val(void *base, size_t i, float v) {
    if constexpr (ELEM == 2) reinterpret_cast<uint16_t *>(base)[i] = uint16_t(bf16_rne(v));
    else reinterpret_cast<float *>(base)[i] = v;
}

// float64 values across lanes
__device__ inline double lane_get(double v, int lane) {           // lane: uniform
    const int64_t u = __double_as_longlong(v);
    const uint32_t lo = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(u)), lane));
    const uint32_t hi = uint32_t(__builtin_amdgcn_readlane(int(uint32_t(uint64_t(u) >> 32)), lane));
    return __longlong_as_double(int64_t((uint64_t(hi) << 32) | lo));
}
template <int CTRL>
__device__ inline double wave_rot(double v) {                     // wave_rol:1 / wave_ror:1
    const int64_t u = __double_as_longlong(v);
    const int lo = int(uint32_t(u)), hi = int(uint32_t(uint64_t(u) >> 32));
    const uint32_t rl = uint32_t(__builtin_amdgcn_update_dpp(lo, lo, CTRL, 0xF, 0xF, false));
    const uint32_t rh = uint32_t(__builtin_amdgcn_update_dpp(hi, hi, CTRL, 0xF, 0xF, false));
    return __longlong_as_double(int64_t((uint64_t(rh) << 32) | rl));
}
constexpr int kWaveRol = 0x134;     // lane i takes lane i + 1's value (63 takes 0's)
constexpr int kWaveRor = 0x13C;     // lane i takes lane i - 1's value (0 takes 63's)
__device__ inline double lane_fetch(double v, int addr) {         // addr: 4 * lane
    const int64_t u = __double_as_longlong(v);
    const uint32_t lo = uint32_t(__builtin_amdgcn_ds_bpermute(addr, int(uint32_t(u))));
    const uint32_t hi = uint32_t(__builtin_amdgcn_ds_bpermute(addr, int(uint32_t(uint64_t(u) >> 32))));
    return __longlong_as_double(int64_t((uint64_t(hi) << 32) | lo));
}

// Largest 32-bit key over the wave, in every lane.
__device__ inline uint32_t wave_max_u32(uint32_t x) {
    x = max(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0xB1, 0xF, 0xF, false)));    // xor 1
    x = max(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x4E, 0xF, 0xF, false)));    // xor 2
    x = max(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x124, 0xF, 0xF, false)));   // row_ror:4
    x = max(x, uint32_t(__builtin_amdgcn_update_dpp(0, int(x), 0x128, 0xF, 0xF, false)));   // row_ror:8
    const auto a = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    x = max(uint32_t(a[0]), uint32_t(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return max(uint32_t(b[0]), uint32_t(b[1]));
}

// 1 / sqrt(x) for x > 0: the hardware's approximation (relative error about 5e-8) and one
// third-order correction.
__device__ inline double rsqrt64(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y * e, fma(0.375, e, 0.5), y);
}

// ---------------------------------------------------------------------------
// Cholesky with diagonal pivoting of the symmetric positive semi-definite n x n matrix in
// g (one wave; lane i owns column i), destroyed.  A step takes the largest remaining diagonal
// entry p (compared on the sign, exponent and 14 mantissa bits, the lane in the 6 bits left of a
// word: a near-maximum serves as well, ties to the lower index; whole doubles gave the same errors
// over 40 build configurations and cost 1 % of a layer) and forms row j of R, A ~ R^T R:
//   R[j][i] = (A[p][i] - sum_{m < j} R[m][p] R[m][i]) / R[j][p].
// It stops when the largest remaining entry is not above tau times the largest initial one;
// returns the number of steps k.  Row j of the result is stored at g's row p (nobody needs
// the rows in pivot order; piv[j] = p), rows that were no pivot are zero.
//   INV: row j of C = R^-T over the original indices (C A C^T = I on the pivots).  C follows
//        the same recurrence from the columns of the identity, and a column needs R's entries
//        before its pivot step and C's from it on, so the two share the storage.
//   not INV: row j of R over the original indices.
// Panels of 8 steps: within one, rows are kept in registers and a step subtracts the panel's
// terms itself (at most 7, their factors by v_readlane); after it the remaining rows of g take
// all 8 terms by float64 MFMA.  A step is then about 55 vector instructions and one LDS round
// trip; with every sum read back from LDS (a left-looking loop over all rows) it was 2400
// cycles, and the four factorisations of a span side 190 of its 435 us.
// ---------------------------------------------------------------------------
template <int NL, int LS, bool INV>
__device__ __forceinline__ int chol(double (*g)[LS], int *piv, int n, double tau, int lane) {
    constexpr int NT = NL / 16;
    const int li = min(lane, NL - 1), c16 = lane & 15, q = lane >> 4;
    double dg = lane < n ? g[li][li] : -1.0;
    bool taken = lane >= n;
    double floor_ = 0.0;
    int k = 0;
    for (int jb = 0;; jb += 8) {
        double w[8];
        int pr[8];
        bool fresh = false;                          // became a pivot in this panel
        bool stop = false;
#pragma unroll
        for (int jj = 0; jj < 8; ++jj) {
            w[jj] = 0.0;
            pr[jj] = 0;
            if (stop || jb + jj >= n) { stop = true; continue; }
            // everything up to the new row before the test that may end the loop, in one
            // block: the reciprocal root fills the reduction's wait states, the row's LDS read
            // is under way during the factors' reads
            const uint32_t hi = uint32_t(uint64_t(__double_as_longlong(dg)) >> 32);
            const bool live = !taken && dg > 0.0;
            const uint32_t key = wave_max_u32(live ? (hi & ~63u) | uint32_t(63 - lane) : 0u);
            const double ry = rsqrt64(live ? dg : 1.0);
            const uint32_t ku = uint32_t(__builtin_amdgcn_readfirstlane(int(key)));
            const int p = min(63 - int(ku & 63u), NL - 1);
            const double va = g[p][li];
            const double v = lane_get(dg, p), rinv = lane_get(ry, p);
            double acc = (taken || lane == p) ? 0.0 : va, acc2 = 0.0;
            if (INV && taken && !fresh) acc = va;
#pragma unroll
            for (int m = 0; m < jj; ++m) {
                if (m & 1) acc2 = fma(-lane_get(w[m], p), w[m], acc2);
                else acc = fma(-lane_get(w[m], p), w[m], acc);
            }
            double res = (acc + acc2) * rinv;
            if (!INV && taken) res = 0.0;
            if (lane == p) res = INV ? rinv : v * rinv;
            if (jb + jj == 0) floor_ = tau * v;
            if (ku == 0 || !(v > floor_)) { stop = true; continue; }
            pr[jj] = p;
            if (INV)
#pragma unroll
                for (int m = 0; m < jj; ++m)
                    if (lane == p) w[m] = 0.0;       // column p holds C from here on
            w[jj] = res;
            if (!taken) dg = fma(-res, res, dg);
            if (lane == p) taken = fresh = true;
            if (lane == 0) piv[jb + jj] = p;
            k = jb + jj + 1;
        }
        wave_sync();                                  // g's rows have been read
#pragma unroll
        for (int jj = 0; jj < 8; ++jj)
            if (jb + jj < k && lane < NL) g[pr[jj]][lane] = w[jj];
        wave_sync();
        // rows without a pivot take the panel's terms.  With INV, the panel's pivot columns
        // hold C from here on: what is above their own step (older rows) becomes zero, and
        // the rows without a pivot restart from the identity's zero
        const uint64_t tm = __ballot(taken), fm = __ballot(fresh);
        if (stop || jb + 8 >= n) {
            if (INV) {
                for (uint64_t old = tm & ~fm & ((uint64_t(1) << n) - 1); old; old &= old - 1)
                    if (fresh) g[__builtin_ctzll(old)][lane] = 0.0;
                wave_sync();
            }
            break;
        }
        double op[2][NT], om_[2][NT];
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            const int row = q == 0 ? pr[4 * kk] : q == 1 ? pr[4 * kk + 1] : q == 2 ? pr[4 * kk + 2] : pr[4 * kk + 3];
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                op[kk][t] = g[row][16 * t + c16];
                om_[kk][t] = ((tm >> (16 * t + c16)) & 1) ? 0.0 : -op[kk][t];
            }
        }
#pragma unroll
        for (int it = 0; it < NT; ++it) {
            const uint32_t fr = uint32_t(fm >> (16 * it + q));           // bit 4 e: row q + 4 e is the panel's
#pragma unroll
            for (int jt = 0; jt < NT; ++jt) {
                const bool restart = INV && ((fm >> (16 * jt + c16)) & 1);
                d4_t s;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s[e] = g[16 * it + q + 4 * e][16 * jt + c16];
                    if (restart && !((fr >> (4 * e)) & 1)) s[e] = 0.0;
                }
                s = mfma64(om_[0][it], op[0][jt], s);
                s = mfma64(om_[1][it], op[1][jt], s);
#pragma unroll
                for (int e = 0; e < 4; ++e) g[16 * it + q + 4 * e][16 * jt + c16] = s[e];
            }
        }
        wave_sync();
    }
    if (k < n) {
        const uint64_t tm = __ballot(taken && lane < n);
        for (int m = 0; m < NL; ++m)
            if (lane < NL && (!((tm >> m) & 1) || (INV && !taken))) g[m][lane] = 0.0;
        wave_sync();
    }
    return k;
}

// ---------------------------------------------------------------------------
// One-sided Jacobi: rotates the columns of W (an n x n matrix, n even)
// until they are pairwise orthogonal (column m starts as row piv[m] of g, m < k); then writes the normalised columns E and their
// norms in descending order: g[i][c] = E[i][c], sig[c] (both zero past column n).
//
// Columns sit at positions 0 .. n - 1 and every rotation also exchanges the two: rounds over
// the pairs (0,1), (2,3), ... and (1,2), (3,4), ... alternate, and n rounds bring every two
// columns together once (the odd-even transposition order).  Lane 20 g + s holds rows
// RW g .. of positions 2s and 2s + 1, so the even rounds are local and an odd round moves one
// column by one lane and back (wave rotations by DPP).  What leaves a group of 20 lanes at an
// end meets the identity (c, s) = (0, 1) there and comes back with its sign changed, in all
// three row groups alike; E's columns have arbitrary signs.
//
// V's rows are W's columns seen through M once more, so a pair that keeps the dot product ga and
// squared norms al, be leaves two rows of V with the product |ga| / min(al, be): its cosine times
// the ratio of the singular values.  A pair rotates unless its cosine is below 1e-18 (what float32
// holds of the angle), and the sweeps stop after one in which no |ga| / min(al, be) was above 1e-6
// (the next one's are about the square of it).  With cosines alone, to 1e-10, the rows' product was
// 5e-8 at singular values of 1/500 and grew with the ratio.  The angle's tangent is formed in
// float32 from ratios in [-1, 1] (an error of 1e-7 of an angle is one more small angle later),
// cosine and sine in float64: a float64 tangent, or sweeps until one rotates nothing, changed
// neither the orthogonality of U and V nor a first step's error against 64 bits in four digits (40
// build configurations, up to 16 seeds) and made a 128K x 4 layer 2 and 4 % longer.
// Per round and lane: 14 FMAs for the dot products, 56 for
// the rotation, 28 DPP moves, about 60 for the angle.
// ---------------------------------------------------------------------------
template <int NL, int LS>
__device__ __forceinline__ void jacobi_columns(double (*g)[LS], const int *piv, int k, double *sig, double *nrm,
                                               int n, int sweeps, int lane) {
    constexpr int RW = NL > 32 ? 14 : 11;                      // rows per lane (3 RW >= largest n)
    const int np = n / 2, grp = lane / 20, s = lane % 20;
    const bool active = grp < 3 && s < np, last = s == np - 1;
    const int pa = active && 2 * s < k ? piv[2 * s] : 0, pb = active && 2 * s + 1 < k ? piv[2 * s + 1] : 0;
    double a[RW], b[RW];
#pragma unroll
    for (int e = 0; e < RW; ++e) {
        const int i = RW * grp + e;
        a[e] = active && i < n && 2 * s < k ? g[pa][i] : 0.0;
        b[e] = active && i < n && 2 * s + 1 < k ? g[pb][i] : 0.0;
    }
    wave_sync();
    const int f0 = 4 * s, f1 = 4 * (20 + s), f2 = 4 * (40 + s);
    auto total = [&](double x) { return (lane_fetch(x, f0) + lane_fetch(x, f1)) + lane_fetch(x, f2); };
    auto dot = [&](const double (&x)[RW], const double (&y)[RW]) {
        double t[2] = {0.0, 0.0};
#pragma unroll
        for (int e = 0; e < RW; ++e) t[e & 1] = fma(x[e], y[e], t[e & 1]);
        return total(t[0] + t[1]);
    };
    bool wide = false;
    // x, y: the pair's columns (lower and higher position), al and be their squared norms;
    // rotates and exchanges them where `on`, leaves x alone elsewhere
    auto rotate = [&](double (&x)[RW], double (&y)[RW], double &al, double &be, bool on) {
        const double ga = dot(x, y);
        const double g2 = ga * ga, ab = al * be;
        const bool rot = on && g2 > 1e-36 * ab;
        wide |= on && fabs(ga) > 1e-6 * fmin(al, be);
        // t = sign(be - al) 2 ga / (|be - al| + sqrt((be - al)^2 + 4 ga^2)), from ratios to al + be
        const double rho = __builtin_amdgcn_rcp(al + be);
        const float dd = float((be - al) * rho), gg = float(2.0 * ga * rho);
        const float h = fabsf(dd) + __builtin_amdgcn_sqrtf(fmaf(dd, dd, gg * gg));
        const float tf = copysignf(1.0f, dd) * gg * __builtin_amdgcn_rcpf(h);
        const double t = rot ? double(tf) : 0.0;
        double c = rsqrt64(fma(t, t, 1.0)), sn = t * c;
        const double na = fma(-t, ga, al), nb = fma(t, ga, be);
        if (!on) { c = 0.0; sn = 1.0; }
#pragma unroll
        for (int e = 0; e < RW; ++e) {
            const double xe = x[e], ye = y[e];
            x[e] = fma(sn, xe, c * ye);
            y[e] = fma(c, xe, -(sn * ye));
        }
        const double nx = on ? nb : al, ny = on ? na : be;
        al = nx;
        be = ny;
    };
    for (int sweep = 0; sweep < sweeps; ++sweep) {
        wide = false;
        double al = dot(a, a), be = dot(b, b);
        for (int it = 0; it < np; ++it) {
            rotate(a, b, al, be, active);
#pragma unroll
            for (int e = 0; e < RW; ++e) a[e] = wave_rot<kWaveRol>(a[e]);
            al = wave_rot<kWaveRol>(al);
            rotate(b, a, be, al, active && !last);
#pragma unroll
            for (int e = 0; e < RW; ++e) a[e] = wave_rot<kWaveRor>(a[e]);
            al = wave_rot<kWaveRor>(al);
        }
        if (__ballot(wide) == 0) break;
    }
    // norms, their descending order (ties to the lower position), E
    const double al = dot(a, a), be = dot(b, b);
    if (lane < NL) nrm[lane] = -1.0;
    wave_sync();
    if (active && grp == 0) { nrm[2 * s] = al; nrm[2 * s + 1] = be; }
    for (int i = 0; i < NL; ++i)
        if (lane < NL) g[i][lane] = 0.0;
    if (lane < NL) sig[lane] = 0.0;
    wave_sync();
    int ra = 0, rb = 0;
    for (int m = 0; m < n; ++m) {
        const double o = nrm[m];
        ra += (o > al || (o == al && m < 2 * s)) ? 1 : 0;
        rb += (o > be || (o == be && m < 2 * s + 1)) ? 1 : 0;
    }
    const double ia = al > 0.0 ? rsqrt64(al) : 0.0, ib = be > 0.0 ? rsqrt64(be) : 0.0;
    // NaN norms compare with nothing: keep every index inside the matrix
    ra = min(ra, NL - 1);
    rb = min(rb, NL - 1);
    if (active) {
#pragma unroll
        for (int e = 0; e < RW; ++e) {
            const int i = RW * grp + e;
            if (i < n) {
                g[i][ra] = a[e] * ia;
                g[i][rb] = b[e] * ib;
            }
        }
        if (grp == 0) {
            sig[ra] = al > 0.0 ? al * ia : 0.0;
            sig[rb] = be > 0.0 ? be * ib : 0.0;
        }
    }
    wave_sync();
}

// Phase marks of the diagnostic trace (builds with SEKV_PHASE_TRACE): slot 0 holds the
// span length, then one s_memrealtime stamp per mark, for the first trace_items items.
enum : int {
    kSvStart = 1, kSvPass = 2, kSvGram = 3, kSvChol = 4, kSvIter = 5, kSvPass2 = 6, kSvChol2 = 7,
    kSvGram2 = 8, kSvCholM = 9, kSvJacobi = 10, kSvT = 11, kSvEnd = 14,
};
#ifdef SEKV_PHASE_TRACE
#define SV_STAMP(SLOT)                                                                         \
    do {                                                                                       \
        if (threadIdx.x == 0 && a.trace && item_ < a.trace_items)                              \
            a.trace[item_ * kTraceSlots + (SLOT)] = int64_t(__builtin_amdgcn_s_memrealtime()); \
    } while (0)
#else
#define SV_STAMP(SLOT) do {} while (0)
#endif

// LDS of one workgroup.  g holds one 40 x 40 matrix at a time (padded to whole tiles, zero
// there): G, then C; M, then C2 C or R, then E.  With one wave, the tiles of the passes and T
// take the same bytes.
template <int ELEM, int D, int NT, int NW>
struct SvdLds {
    static constexpr int NL = 16 * NT, LS = NL + 1;
    static constexpr int KR = NL < kMaxL ? NL : kMaxL;         // rows of the test matrix
    static constexpr int OS = D + 8;                           // its row stride (16-byte rows)
    static constexpr int XS = D * ELEM + 16, XB = 16 * XS;      // row stride and bytes of a wave's X tile
    static constexpr int TS = KR + 1;
    static constexpr int kG = NL * LS * 8, kOm = KR * OS * 2, kT = KR * TS * 8;
    static constexpr int kAcc = (4 * NT * (D / 16) + 4 * NT * (NT + 1)) * 256;   // a wave's sums
    // byte offsets
    static constexpr int om = NW == 1 ? 0 : kG;
    static constexpr int xs = NW == 1 ? (kOm + 15) / 16 * 16 : kG + (kOm + 15) / 16 * 16;
    static constexpr int xf = NW == 1 ? (kT + 15) / 16 * 16 : xs;
    static constexpr int red = xs + NW * XB;
    static constexpr int tiles = (xs > xf ? xs : xf) + XB;
    static constexpr int body = NW > 1 ? red + kAcc : kG > tiles ? kG : tiles;
    __attribute__((aligned(16))) unsigned char b[(body + 15) / 16 * 16];
    double sig[NL];
    union {
        double nrm[NL];
        int piv[NL];
    };
};

template <int ELEM, int D, int NT, int NW>
__global__ void __launch_bounds__(64 * NW, (ELEM == 2 && NW == 1) ? 2 : 1) svd_kernel(BuildArgs a) {
    using SM = SvdLds<ELEM, D, NT, NW>;
    constexpr int NL = SM::NL, LS = SM::LS, KR = SM::KR, OS = SM::OS, TS = SM::TS;
    constexpr int DT = D / 16;
    constexpr int NG = NT * (NT + 1) / 2;
    __shared__ SM sm;
    static_assert(NW > 1 || ELEM != 2 || sizeof(SM) <= 20 * 1024, "eight one-wave sides per CU");
    const int tid = threadIdx.x, lane = tid & 63, wave = NW == 1 ? 0 : tid >> 6;
    int c16 = lane & 15, q = lane >> 4;
    auto phase = [&]() __attribute__((always_inline)) {
        const int t = opaque(lane);
        c16 = t & 15;
        q = t >> 4;
    };
#ifdef SEKV_PHASE_TRACE
    const int64_t item_ = int64_t(blockIdx.y) * gridDim.x + blockIdx.x;
#endif
    const int side = blockIdx.y;                              // 0 keys, 1 values
    const int pair = blockIdx.x / a.M_max, S = blockIdx.x % a.M_max;
    const int b = pair / a.Hkv;
    int ns = a.n_spans[b];
    ns = ns < 0 ? 0 : min(ns, min(a.M_max, a.N));
    if (S >= ns) return;
    const int s0 = a.span_start[size_t(b) * a.N + S];
    const int L = a.span_len_seg[size_t(b) * a.N + S];
    int n_tok = a.n_tokens[b];
    n_tok = n_tok < 0 ? 0 : min(n_tok, a.N);
    if (s0 < 0 || L < 1 || s0 + L > n_tok) return;              // flagged by the gather kernel
    constexpr int gran = 16 / ELEM;
    const int r = min(min(L, D), a.R);                        // rank kept (eq. key_svd)
    const int rs = (r + gran - 1) / gran * gran;              // stored rank
    const int l = max(2, min(a.l, D) & ~1);                   // sketch width (even, for pairing)
    const unsigned char *X = static_cast<const unsigned char *>(side == 0 ? a.keys : a.values) +
                             (size_t(pair) * a.N + s0) * D * ELEM;
    // block layout: U_K | sigma_K | Vt_K | U_V | sigma_V | Vt_V, both sides of rank rs
    const int64_t boff = a.block_off[size_t(pair) * a.M_max + S];
    const int64_t side_elems = int64_t(L + 1 + D) * rs;
    const int64_t need = 2 * side_elems * ELEM;
    if (boff < 0 || (boff & 15) || boff + need > a.factors_bytes) {
        if (tid == 0) __hip_atomic_fetch_or(a.error, kErrBlockRange, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        return;
    }
    unsigned char *blk = static_cast<unsigned char *>(a.factors) + boff + (side ? side_elems * ELEM : 0);
    const int64_t s_off = int64_t(L) * rs, v_off = s_off + rs;    // in elements; U at 0
#ifdef SEKV_PHASE_TRACE
    if (tid == 0 && a.trace && item_ < a.trace_items) a.trace[item_ * kTraceSlots] = L;
#endif
    SV_STAMP(kSvStart);

    double(*const g)[LS] = reinterpret_cast<double(*)[LS]>(sm.b);
    double(*const tp)[TS] = reinterpret_cast<double(*)[TS]>(sm.b);
    uint16_t(*const om)[OS] = reinterpret_cast<uint16_t(*)[OS]>(sm.b + SM::om);
    unsigned char *const xs_raw = sm.b + SM::xs + wave * SM::XB;
    unsigned char *const xf_raw = NW == 1 ? sm.b + SM::xf : xs_raw;

    // the caller's test matrix into om (bfloat16, transposed; rows past l zero)
    for (int c0 = 16 * wave; c0 < D; c0 += 16 * NW) {
        float v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = lane < l ? a.omega[size_t(c0 + u) * a.l + lane] : 0.0f;
        if (lane < KR)
#pragma unroll
            for (int u = 0; u < 16; ++u) om[lane][c0 + u] = uint16_t(bf16_rne(v[u]));
    }
    __syncthreads();

    // 16 rows of X from token t on, as the A (or B) operand of a product over d: lane (c16, q)
    // takes token t + c16, and 16-byte pieces of it; rows past the span are zero
    constexpr int NX = D * ELEM / 64;                           // 16-byte pieces per lane
    auto load_x = [&](uint4 (&x)[NX], int t) __attribute__((always_inline)) {
        const unsigned char *row = X + size_t(t + c16) * D * ELEM + q * 16;
#pragma unroll
        for (int m = 0; m < NX; ++m)
            x[m] = t + c16 < L ? *reinterpret_cast<const uint4 *>(row + m * 64) : make_uint4(0u, 0u, 0u, 0u);
    };
    // the same rows into a tile in LDS, for products over the tokens
    auto store_x = [&](unsigned char *tile, const uint4 (&x)[NX]) __attribute__((always_inline)) {
        unsigned char *row = tile + c16 * SM::XS + q * 16;
#pragma unroll
        for (int m = 0; m < NX; ++m) *reinterpret_cast<uint4 *>(row + m * 64) = x[m];
    };
    // piece m of test-matrix row 16 nt + c16 that meets piece m of X
    auto load_om = [&](int nt, int m) __attribute__((always_inline)) -> uint4 {
        const uint16_t *row = om[min(16 * nt + c16, KR - 1)];
        if constexpr (ELEM == 2) return *reinterpret_cast<const uint4 *>(row + 32 * m + 8 * q);
        else {
            const uint2 v = *reinterpret_cast<const uint2 *>(row + 16 * m + 4 * q);
            return make_uint4(v.x, v.y, 0u, 0u);
        }
    };
    auto om_f = [&](const uint4 &o, int j) __attribute__((always_inline)) -> float {
        const uint32_t w = j < 2 ? o.x : o.y;
        return __uint_as_float((j & 1) ? (w & 0xFFFF0000u) : (w << 16));
    };
    auto x_f = [&](const uint4 &x, int j) __attribute__((always_inline)) -> float {
        return __uint_as_float(j == 0 ? x.x : j == 1 ? x.y : j == 2 ? x.z : x.w);
    };

    // T, zero outside its storage
    auto t_at = [&](int row, int comp) __attribute__((always_inline)) -> double {
        const double v = tp[min(row, KR - 1)][min(comp, KR - 1)];
        return row < KR ? v : 0.0;
    };
    // the upper tiles of a symmetric matrix into g, both halves, zero past l
    auto put_sym = [&](const d4_t (&m)[NG]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0, ij = 0; i < NT; ++i)
#pragma unroll
            for (int j = i; j < NT; ++j, ++ij)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = 16 * i + q + 4 * e, col = 16 * j + c16;
                    const double v = row < l && col < l ? m[ij][e] : 0.0;
                    g[row][col] = v;
                    if (i != j) g[col][row] = v;
                }
        wave_sync();
    };
    // P stays in registers through the factorisations, or the output pass forms it again
    constexpr bool kKeepP = ELEM == 4 || NW > 1;
    f4_t pacc[NT][DT];                  // P tiles (rows: sketch columns 16 nt + 4 q + r; column: 16 ct + c16)
    // P += Y^T X for the 16 tokens in `tile`; y: rows tokens 4 q + e, which is the contraction index
    auto add_p = [&](const f4_t (&y)[NT], const unsigned char *tile) __attribute__((always_inline)) {
        if constexpr (ELEM == 2) {
            uint2 yh[NT], ym[NT], yl[NT];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                const float yy[4] = {y[nt][0], y[nt][1], y[nt][2], y[nt][3]};
                split3(yy, yh[nt], ym[nt], yl[nt]);
            }
            const uint16_t *xs = reinterpret_cast<const uint16_t *>(tile) + (4 * q + c16 / 4) * (D + 8) +
                                 4 * (c16 % 4);
#pragma unroll
            for (int ct = 0; ct < DT; ++ct) {
                const uint2 xb = lds_tr4(xs + 16 * ct);
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    pacc[nt][ct] = mfma_k16(yl[nt], xb, pacc[nt][ct]);
                    pacc[nt][ct] = mfma_k16(ym[nt], xb, pacc[nt][ct]);
                    pacc[nt][ct] = mfma_k16(yh[nt], xb, pacc[nt][ct]);
                }
            }
        } else {
            const float *xs = reinterpret_cast<const float *>(tile) + 4 * q * (D + 4) + c16;
#pragma unroll
            for (int ct = 0; ct < DT; ++ct)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float xv = xs[e * (D + 4) + 16 * ct];
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) pacc[nt][ct] = mfma32(y[nt][e], xv, pacc[nt][ct]);
                }
        }
    };
    // V^T rows (T^T P) / sigma, zero past the kept components.  M was formed from the same P, so the
    // rows are orthonormal to the rounding of their storage whatever their singular value.  As
    // X^T U in float32 sums (which needs no P) they were not: two rows' product was up to 0.15 for
    // singular values down to 1e-4 of the largest (now 2.4e-3, bfloat16's own rounding), and 1.8e-3
    // instead of 1.2e-3 (root mean square) after a plain sketch.  A 128K x 4 layer: 8.58 against 8.93 ms.
    auto put_v = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            if (16 * ct >= rs) continue;
            double tv[NT][4];
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 4; ++e) tv[nt][e] = t_at(16 * nt + 4 * q + e, 16 * ct + c16);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) {
                d4_t v = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) v = mfma64(tv[nt][e], double(pacc[nt][dt][e]), v);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int comp = 16 * ct + q + 4 * e;
                    const double s = sm.nrm[comp];
                    if (comp < rs)
                        st_val<ELEM>(blk, size_t(v_off) + size_t(comp) * D + 16 * dt + c16,
                                     s > 0.0 ? float(v[e] / s) : 0.0f);
                }
            }
        }
    };
    // a pass over X with the test matrix in om: P = Y^T X into pacc, and with GRAM G = Y^T Y
    // (what is returned puts it into g)
    auto sketch = [&](auto gram_c) __attribute__((always_inline)) {
        constexpr bool GRAM = decltype(gram_c)::value;
        phase();
        d4_t gacc[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) gacc[i] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int ct = 0; ct < DT; ++ct) pacc[nt][ct] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
        uint4 xn[NX];
        load_x(xn, 16 * wave);
        for (int t0 = 16 * wave; t0 < L; t0 += 16 * NW) {
            f4_t y[NT];
            {
                uint4 x[NX];
#pragma unroll
                for (int m = 0; m < NX; ++m) x[m] = xn[m];
                load_x(xn, t0 + 16 * NW);
                store_x(xs_raw, x);
                // Y tile: rows tokens 4 q + r, column 16 nt + c16
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    y[nt] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int m = 0; m < NX; ++m) {
                        const uint4 o = load_om(nt, m);
                        if constexpr (ELEM == 2) y[nt] = mfma_k32(x[m], o, y[nt]);
                        else
#pragma unroll
                            for (int j = 0; j < 4; ++j) y[nt] = mfma32(x_f(x[m], j), om_f(o, j), y[nt]);
                    }
                    __builtin_amdgcn_sched_barrier(0);      // one tile of the test matrix at a time
                }
            }
#pragma unroll
            for (int i = 0, ij = 0; i < NT; ++i)
#pragma unroll
                for (int j = i; j < NT; ++j, ++ij)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if constexpr (GRAM) gacc[ij] = mfma64(double(y[i][e]), double(y[j][e]), gacc[ij]);
            wave_sync();
            add_p(y, xs_raw);
            wave_sync();
        }
        if constexpr (NW > 1) {
            // the other waves' sums into wave 0, one wave after another
            uint32_t *red = reinterpret_cast<uint32_t *>(sm.b + SM::red);
            for (int w = 1; w < NW; ++w) {
                __syncthreads();
                if (wave == w) {
                    int at = lane;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int ct = 0; ct < DT; ++ct)
#pragma unroll
                            for (int e = 0; e < 4; ++e, at += 64) red[at] = __float_as_uint(pacc[nt][ct][e]);
                    double *rd = reinterpret_cast<double *>(red + 256 * NT * DT);
#pragma unroll
                    for (int i = 0; i < (GRAM ? NG : 0); ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) rd[(4 * i + e) * 64 + lane] = gacc[i][e];
                }
                __syncthreads();
                if (wave == 0) {
                    int at = lane;
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                        for (int ct = 0; ct < DT; ++ct)
#pragma unroll
                            for (int e = 0; e < 4; ++e, at += 64) pacc[nt][ct][e] += __uint_as_float(red[at]);
                    const double *rd = reinterpret_cast<const double *>(red + 256 * NT * DT);
#pragma unroll
                    for (int i = 0; i < (GRAM ? NG : 0); ++i)
#pragma unroll
                        for (int e = 0; e < 4; ++e) gacc[i][e] += rd[(4 * i + e) * 64 + lane];
                }
            }
        }
        return [=]() __attribute__((always_inline)) { put_sym(gacc); };
    };
    // C as the operand of products over its rows: cr[i][nt] = C[4 i + q][16 nt + c16]
    constexpr int K4 = KR / 4;
    double cr[K4][NT];
    // M = B B^T with B = C P (C in g), then C into cr and M into g.  B^T tiles come out of the
    // product in the layout that the next product reads, one 16-column strip of B at a time.
    auto gram_b = [&]() __attribute__((always_inline)) {
        phase();
        d4_t macc[NG];
#pragma unroll
        for (int i = 0; i < NG; ++i) macc[i] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
        for (int ct = 0; ct < DT; ++ct) {
            d4_t bt[NT];
#pragma unroll
            for (int lt = 0; lt < NT; ++lt) bt[lt] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int lt = 0; lt < NT; ++lt)
                        bt[lt] = mfma64(double(pacc[nt][ct][e]), g[16 * lt + c16][16 * nt + 4 * q + e], bt[lt]);
                __builtin_amdgcn_sched_barrier(0);          // one tile of C's operands at a time
            }
#pragma unroll
            for (int i = 0, ij = 0; i < NT; ++i)
#pragma unroll
                for (int j = i; j < NT; ++j, ++ij)
#pragma unroll
                    for (int e = 0; e < 4; ++e) macc[ij] = mfma64(bt[i][e], bt[j][e], macc[ij]);
            wave_sync();                                    // C is read anew for each strip
            __builtin_amdgcn_sched_barrier(0);
        }
        // (where P is used again, its float64 copies are made anew: 192 registers)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int ct = 0; ct < DT; ++ct) asm volatile("" : "+v"(pacc[nt][ct]));
#pragma unroll
        for (int i = 0; i < K4; ++i)
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) cr[i][nt] = g[4 * i + q][16 * nt + c16];
        wave_sync();
        put_sym(macc);
    };

    // subspace iterations: the next test matrix is an orthonormal basis of P's row space,
    // C_P P with C_P the inverse Cholesky factor of P P^T (pivots down to the rounding of
    // float64: P's own float32 sums bound what its small directions are worth).  P = R^T B, so
    // this is B's row space too, without G, its factor and B; in a model of both (numpy, float32 sums,
    // bfloat16 test matrices, spectra from flat to 10^(-i/4)) the two bases give the same error
    // of the rank-32 factors.
    // (A span of at most l tokens is spanned by its sketch already: X Omega has the rank of X for
    // a generic Omega, and an iteration would change nothing but the rounding.)
    const int power = L <= l ? 0 : a.power;
    for (int it = 0; it < power; ++it) {
        sketch(Bool<false>{});
        __syncthreads();
        if (wave == 0) {
            SV_STAMP(kSvPass);
            phase();
            {
                // N = P P^T (float64) from 16-column strips of P, turned in LDS
                constexpr int SS = NL + 4;                      // strip row stride
                d4_t nacc[NG];
#pragma unroll
                for (int i = 0; i < NG; ++i) nacc[i] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int ct = 0; ct < DT; ++ct) {
                    float(*const ts)[SS] = reinterpret_cast<float(*)[SS]>(sm.b + (ct & 1) * 16 * SS * 4);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) *reinterpret_cast<f4_t *>(&ts[c16][16 * nt + 4 * q]) = pacc[nt][ct];
                    wave_sync();
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        double pd[NT];
#pragma unroll
                        for (int lt = 0; lt < NT; ++lt) pd[lt] = double(ts[4 * e + q][16 * lt + c16]);
#pragma unroll
                        for (int i = 0, ij = 0; i < NT; ++i)
#pragma unroll
                            for (int j = i; j < NT; ++j, ++ij) nacc[ij] = mfma64(pd[i], pd[j], nacc[ij]);
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
                wave_sync();
                put_sym(nacc);
            }
            SV_STAMP(kSvGram);
            chol<NL, LS, true>(g, sm.piv, l, 1e-16, opaque(lane));
            SV_STAMP(kSvChol);
            phase();
            // the basis; C_P's operand is in registers before om takes g's place
            double cp[NT][NT][4];
#pragma unroll
            for (int lt = 0; lt < NT; ++lt)
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int e = 0; e < 4; ++e) cp[lt][nt][e] = g[16 * lt + c16][16 * nt + 4 * q + e];
            wave_sync();
#pragma unroll
            for (int ct = 0; ct < DT; ++ct) {
                d4_t o[NT];
#pragma unroll
                for (int lt = 0; lt < NT; ++lt) o[lt] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
#pragma unroll
                        for (int lt = 0; lt < NT; ++lt)
                            o[lt] = mfma64(double(pacc[nt][ct][e]), cp[lt][nt][e], o[lt]);
#pragma unroll
                for (int lt = 0; lt < NT; ++lt) {
                    const int row = 16 * lt + c16;
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (row < KR)
                            om[row][16 * ct + q + 4 * e] = uint16_t(row < l ? bf16_rne(float(o[lt][e])) : 0u);
                }
                __builtin_amdgcn_sched_barrier(0);
            }
            SV_STAMP(kSvIter);
        }
        __syncthreads();
    }
    // the last pass; its test matrix stays in registers for the output pass
    auto put_g = sketch(Bool<true>{});
    phase();
    uint4 omk[NT][NX];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt)
#pragma unroll
        for (int m = 0; m < NX; ++m) omk[nt][m] = load_om(nt, m);
    __syncthreads();
    if (wave == 0) {
        put_g();
        SV_STAMP(kSvPass2);
        const int k = chol<NL, LS, true>(g, sm.piv, l, 1e-8, opaque(lane));
        SV_STAMP(kSvChol2);
        gram_b();
        SV_STAMP(kSvGram2);
        const int km = chol<NL, LS, false>(g, sm.piv, l, 1e-30, opaque(lane));
        SV_STAMP(kSvCholM);
        jacobi_columns<NL, LS>(g, sm.piv, km, sm.sig, sm.nrm, l, a.sweeps, opaque(lane));
        SV_STAMP(kSvJacobi);
        // components below 1e-5 of the largest singular value are numerically undetermined: zero
        if (lane < NL) {
            const double s = sm.sig[lane], top = sm.sig[0];
            sm.nrm[lane] = (lane < k && lane < r && s * s > 1e-10 * (top * top)) ? s : 0.0;
        }
        wave_sync();
        if (lane < rs) st_val<ELEM>(blk, size_t(s_off) + lane, float(sm.nrm[lane]));
        // T = C^T E
        phase();
        d4_t t[NT][NT];
#pragma unroll
        for (int ot = 0; ot < NT; ++ot)
#pragma unroll
            for (int ct = 0; ct < NT; ++ct) {
                t[ot][ct] = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int k4 = 0; k4 < K4; ++k4)
                    t[ot][ct] = mfma64(cr[k4][ot], g[4 * k4 + q][16 * ct + c16], t[ot][ct]);
            }
        wave_sync();
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            const int comp = 16 * ct + c16;
            const bool keep = sm.nrm[comp] > 0.0;
#pragma unroll
            for (int ot = 0; ot < NT; ++ot)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int row = 16 * ot + q + 4 * e;
                    if (row < KR && comp < KR) tp[row][comp] = keep ? t[ot][ct][e] : 0.0;
                }
        }
        wave_sync();
        if constexpr (kKeepP) put_v();
        SV_STAMP(kSvT);
    }
    __syncthreads();

    // output pass: U = Y T, 16 tokens at a time.  A lone wave with bfloat16 storage has no registers
    // to keep P in (that takes one wave per SIMD): the pass forms it again beside U, operation
    // for operation as the sketch did, so it has the same bits, and V follows at the end
    phase();
    bool keep[NT];
#pragma unroll
    for (int ct = 0; ct < NT; ++ct) keep[ct] = sm.nrm[16 * ct + c16] > 0.0;
    if constexpr (!kKeepP)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int ct = 0; ct < DT; ++ct) pacc[nt][ct] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
    uint4 xn[NX];
    load_x(xn, 16 * wave);
    for (int t0 = 16 * wave; t0 < L; t0 += 16 * NW) {
        // Y^T tile: rows sketch columns 16 nt + 4 q + r, column token c16
        f4_t yt[NT];
        {
            uint4 x[NX];
#pragma unroll
            for (int m = 0; m < NX; ++m) x[m] = xn[m];
            load_x(xn, t0 + 16 * NW);
            if constexpr (!kKeepP) store_x(xf_raw, x);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                yt[nt] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int m = 0; m < NX; ++m) {
                    if constexpr (ELEM == 2) yt[nt] = mfma_k32(omk[nt][m], x[m], yt[nt]);
                    else
#pragma unroll
                        for (int j = 0; j < 4; ++j) yt[nt] = mfma32(om_f(omk[nt][m], j), x_f(x[m], j), yt[nt]);
                }
            }
            if constexpr (!kKeepP) {
                f4_t y[NT];
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    y[nt] = f4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                    for (int m = 0; m < NX; ++m) y[nt] = mfma_k32(x[m], omk[nt][m], y[nt]);
                }
                wave_sync();
                add_p(y, xf_raw);
                wave_sync();
            }
        }
#pragma unroll
        for (int ct = 0; ct < NT; ++ct) {
            if (16 * ct >= rs) continue;
            // U tile: rows tokens q + 4 r, column component 16 ct + c16 (a component that was not
            // kept is zero also where the sketch is infinite or NaN)
            const int comp = 16 * ct + c16;
            d4_t u = d4_t{0.0, 0.0, 0.0, 0.0};
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int e = 0; e < 4; ++e) u = mfma64(double(yt[nt][e]), t_at(16 * nt + 4 * q + e, comp), u);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int t = t0 + q + 4 * e;
                if (t < L && comp < rs) st_val<ELEM>(blk, size_t(t) * rs + comp, keep[ct] ? float(u[e]) : 0.0f);
            }
        }
    }
    if constexpr (!kKeepP) put_v();
    SV_STAMP(kSvEnd);
}

}  // namespace
}  // namespace sekv
