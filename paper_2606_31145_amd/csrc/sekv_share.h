// The share item with bfloat16 storage, on the matrix cores (included by sekv_step.h, inside its
// namespaces).
//
// What bounds it: with two waves per SIMD a share item is as long as its chain of instructions
// and barriers, not its FLOPs: with fp32 FMAs and lane reductions an anchor block of 128 rows took
// about 1000 instructions a wave and 6 us, a zoomed span 8 barriers and 7 to 12 us; a 128K x 4 step
// issued 9.5 M vector instructions and a wave waited 49 % of its cycles.  (Now 6.1 M, and 54 % of
// fewer cycles: 32.4 M instead of 39.5 M.)  Here
// each wave works alone on its own rows with its own online softmax (no workgroup barrier
// between the selection and the partial), and every product is an MFMA:
//   scores  = rows x q       A: 16 rows of keys, straight from memory; B: the query, head n % G in
//                            column n.  bf16 products are exact, sums fp32.
//   values += rows^T x p     A: the rows turned by transposing LDS reads; B: the weights as
//                            three bf16 pieces whose sum is exactly the fp32 weight, piece s of
//                            head h in column s G + h, so the 16 columns that G <= 5 heads leave
//                            empty hold the pieces; the pieces' sums are added at the end.
// A product's result has its column in the lane (lane % 16) and rows 4 q + e, which is just the
// layout that the next product reads its weights in (contraction index permuted on both
// sides), so scores -> weights -> values stay in registers.  A zoom chains four of them:
// w = sigma_K (Vt_K q), scores = U_K w, y = U_V^T p, values += Vt_V^T (sigma_V y), with w and y
// split into three pieces as well: no fp32 value loses a bit on its way.
// Measured against fp32 FMAs on packed lanes, whole steps: 32K context, 8 heads of 4 queries,
// top 8: 23.0 -> 19.9 us; batch 32 of it in a graph of layers 661 -> 410 us; 128K x 4 33.4 ->
// 29.3 us; adaptive ranks with groups of 8 52.7 -> 30.9 us.  Mean error against 64 bits over
// 14 shapes of fp32 output: 2.46e-7 -> 2.32e-7.  fp32 storage stays on the FMAs of sekv_step.h: split
// like this its rows would take three times the registers (the fp32 matrix instruction, which takes
// them whole, is not tried yet).

typedef float f4v __attribute__((ext_vector_type(4)));

__device__ inline f4v mfma_bf16_k32(const uint4 &a, const uint4 &b, f4v c) {
    typedef __bf16 b8v __attribute__((ext_vector_type(8)));
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8v, a), __builtin_bit_cast(b8v, b), c, 0, 0, 0);
}
__device__ inline f4v mfma_bf16_k16(const uint2 &a, const uint2 &b, f4v c) {
    typedef short s4v __attribute__((ext_vector_type(4)));
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s4v, a), __builtin_bit_cast(s4v, b), c, 0, 0, 0);
}
// Four rows of one column of a bf16 tile in LDS: within 16 lanes, lane i names 4 columns
// 4 (i % 4) of row slot i / 4 and receives column i of the four row slots.
__device__ inline uint2 lds_turn4(const unsigned char *p) {
    typedef short s4v __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s4v *lds_p;
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                                         reinterpret_cast<lds_p>(reinterpret_cast<uintptr_t>(p))));
}
// LDS accesses of one wave complete in order; this keeps the compiler from moving one
// across the point where another lane's value is needed.
__device__ inline void wave_fence() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// One wave's view of a share item: lane roles and the online softmax of its rows.
template <int D, int G>
struct Wave {
    static constexpr int KC = D / 32;               // 16-byte pieces of a row per lane
    static constexpr int DT = D / 16;
    static constexpr int NU = (3 * G + 15) / 16;    // column tiles of (piece, head): 1, or 2 with G = 8
    static constexpr int RS = D * 2 + 16;           // row stride of a turned tile
    int c16, q, h;                                  // column, row group, the column's head
    int s0;                                         // piece in column tile 0 (>= 3: an empty column)
    unsigned char *wb;                              // the wave's LDS
    uint4 qB[KC];                                   // the query as B operand
    float m, l;                                     // running maximum and sum of head h (this lane's rows)
    f4v o[NU][DT];                                  // values: row 16 dt + 4 q + e, column (piece, head)
};

// The pieces of four fp32 values that this lane's column of tile u holds.
template <int D, int G>
__device__ inline uint2 pieces4(const Wave<D, G> &W, const float (&v)[4], int u) {
    const int s = W.s0 + u * (16 / G);
    uint32_t w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float x = v[i];
        const float t1 = x - __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
        x = s >= 1 ? t1 : x;
        const float t2 = x - __uint_as_float(__float_as_uint(x) & 0xFFFF0000u);
        x = s >= 2 ? t2 : x;
        w[i] = s >= 3 ? 0u : __float_as_uint(x);
    }
    constexpr uint32_t kHigh = 0x07060302u;         // the high halves of two words
    return make_uint2(__builtin_amdgcn_perm(w[1], w[0], kHigh), __builtin_amdgcn_perm(w[3], w[2], kHigh));
}

// Sum over the pieces (the columns of one head); every column of the head gets it.
template <int G, int NU>
__device__ inline f4v piece_sum(const f4v (&x)[NU]) {
    f4v r = x[0];
    if constexpr (NU > 1) r += x[1];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float v = r[e];
        v += dpp_mov<kDppRor8>(v);
        if constexpr (G <= 4) v += dpp_mov<kDppRor4>(v);
        if constexpr (G <= 2) v += dpp_mov<0x122>(v);
        if constexpr (G <= 1) v += dpp_mov<0x121>(v);
        r[e] = v;
    }
    return r;
}

// Weights of N base-2 scores of this lane (-inf: no such row) in place, relative to the new
// maximum; returns the factor for what was accumulated before.
template <int D, int G, int N>
__device__ inline float soft_step(Wave<D, G> &W, float (&s)[N]) {
    float mx = s[0];
#pragma unroll
    for (int i = 1; i < N; ++i) mx = fmaxf(mx, s[i]);
    mx = lane_reduce<4, 6, OpMax>(mx);
    const float mn = fmaxf(W.m, mx);
    const float base = mn == -INFINITY ? 0.0f : mn;
    const float so = __builtin_amdgcn_exp2f(W.m - base);
    float sum = 0.0f;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        s[i] = __builtin_amdgcn_exp2f(s[i] - base);
        sum += s[i];
    }
    W.l = W.l * so + sum;
    W.m = mn;
    return so;
}

template <int D, int G>
__device__ inline void scale_values(Wave<D, G> &W, float so) {
    if (__ballot(so != 1.0f) == 0) return;
#pragma unroll
    for (int u = 0; u < W.NU; ++u)
#pragma unroll
        for (int dt = 0; dt < W.DT; ++dt) W.o[u][dt] *= so;
}

// Sixteen rows (row-major, RB bytes apart) from `row0` of n, clamped to the last one, in the
// key layout: lane (c16, q) holds row c16's 16-byte pieces q, q + 4, ...
template <int D, int G>
__device__ inline void load16(const Wave<D, G> &W, uint4 (&v)[D / 32], const unsigned char *base, int row0, int n) {
    const unsigned char *p = base + size_t(min(row0 + W.c16, n - 1)) * (D * 2) + W.q * 16;
#pragma unroll
    for (int k = 0; k < D / 32; ++k) v[k] = ld16(p + k * 64);
}
// Their products with the query: a sum per 32 components, then those in pairs
template <int D, int G>
__device__ inline f4v row_dots(const Wave<D, G> &W, const uint4 (&v)[D / 32]) {
    f4v d[D / 32];
#pragma unroll
    for (int k = 0; k < D / 32; ++k) d[k] = mfma_bf16_k32(v[k], W.qB[k], f4v{0.0f, 0.0f, 0.0f, 0.0f});
    if constexpr (D == 128) return (d[0] + d[1]) + (d[2] + d[3]);
    else return d[0] + d[1];
}

// Those rows into the wave's LDS, to be turned; rows from `live` on hold anything (a NaN
// would outlive its zero weight) and become zeros.
template <int D, int G>
__device__ inline void turn16(const Wave<D, G> &W, uint4 (&v)[D / 32], int sub, int live) {
    unsigned char *p = W.wb + (16 * sub + W.c16) * W.RS + W.q * 16;
    if (live < 16)
#pragma unroll
        for (int k = 0; k < D / 32; ++k)
            if (W.c16 >= live) v[k] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
    for (int k = 0; k < D / 32; ++k) *reinterpret_cast<uint4 *>(p + k * 64) = v[k];
}
// values += rows^T x weights for the 32 (16) rows in the wave's LDS; w: the lane's weights of
// rows 4 q + e and 16 + 4 q + e
template <int D, int G>
__device__ inline void add_rows32(Wave<D, G> &W, const float (&w)[8]) {
    uint4 b[W.NU];
#pragma unroll
    for (int u = 0; u < W.NU; ++u) {
        const float lo[4] = {w[0], w[1], w[2], w[3]}, hi[4] = {w[4], w[5], w[6], w[7]};
        const uint2 x = pieces4(W, lo, u), y = pieces4(W, hi, u);
        b[u] = make_uint4(x.x, x.y, y.x, y.y);
    }
    const unsigned char *p = W.wb + (4 * W.q + W.c16 / 4) * W.RS + (W.c16 % 4) * 8;
#pragma unroll
    for (int dt = 0; dt < W.DT; ++dt) {
        const uint2 x = lds_turn4(p + dt * 32), y = lds_turn4(p + 16 * W.RS + dt * 32);
        const uint4 a = make_uint4(x.x, x.y, y.x, y.y);
#pragma unroll
        for (int u = 0; u < W.NU; ++u) W.o[u][dt] = mfma_bf16_k32(a, b[u], W.o[u][dt]);
    }
}
template <int D, int G>
__device__ inline void add_rows16(Wave<D, G> &W, const float (&w)[4]) {
    uint2 b[W.NU];
#pragma unroll
    for (int u = 0; u < W.NU; ++u) b[u] = pieces4(W, w, u);
    const unsigned char *p = W.wb + (4 * W.q + W.c16 / 4) * W.RS + (W.c16 % 4) * 8;
#pragma unroll
    for (int dt = 0; dt < W.DT; ++dt) {
        const uint2 a = lds_turn4(p + dt * 32);
#pragma unroll
        for (int u = 0; u < W.NU; ++u) W.o[u][dt] = mfma_bf16_k16(a, b[u], W.o[u][dt]);
    }
}

// One part of a zoomed span: the 16-token tiles part, part + parts, ... of it.
template <int D, int G, int R, bool RANKED>
__device__ __forceinline__ void zoom_part(const Params &p, Wave<D, G> &W, int L, int rk, int rv, int64_t off, int part,
                                          int parts) {
    constexpr int KC = D / 32, NU = Wave<D, G>::NU;
    constexpr bool K32 = R >= 32;                       // contraction over 32 components at a time
    constexpr int KK = K32 ? R / 32 : 1;                // 32- (or 16-) component steps
    constexpr int CT = R == 64 ? 2 : R == 32 ? 4 : 8;   // token tiles at a time (registers)
    constexpr int US = R * 2 + 16;                      // row stride of the turned U_V rows
    if constexpr (RANKED) {
        rk = __builtin_amdgcn_readfirstlane(rk);
        rv = __builtin_amdgcn_readfirstlane(rv);
    } else {
        rk = R;
        rv = R;
    }
    const int c16 = W.c16, q = W.q;
    const unsigned char *UK = p.factors + off;
    const unsigned char *sK = UK + size_t(L) * rk * 2;
    const unsigned char *VtK = sK + size_t(rk) * 2;
    const unsigned char *UV = VtK + size_t(rk) * D * 2;
    const unsigned char *sV = UV + size_t(L) * rv * 2;
    const unsigned char *VtV = sV + size_t(rv) * 2;
    const uint4 zero4 = make_uint4(0u, 0u, 0u, 0u);
    const int ntile = (L + 15) / 16;

    // rows of Vt_K: row i of tile t is the component that makes a lane's results (rows 4 q + e of
    // the tiles) the consecutive components its score operand needs
    constexpr int VT = K32 ? 2 : 1;                     // tiles of one step
    uint4 vk[VT][KC];
    auto load_vk = [&](int step) {
#pragma unroll
        for (int t = 0; t < VT; ++t) {
            const int comp = K32 ? 32 * step + 8 * (c16 / 4) + 4 * t + c16 % 4 : c16;
#pragma unroll
            for (int k = 0; k < KC; ++k)
                vk[t][k] = comp < rk ? ld16(VtK + uint32_t(comp * D * 2 + k * 64 + q * 16)) : zero4;
        }
    };
    load_vk(0);
    uint4 sk[KK];                                       // sigma_K of those components
#pragma unroll
    for (int k = 0; k < KK; ++k) {
        sk[k] = zero4;
        if constexpr (K32) {
            if (32 * k + 8 * q < rk) sk[k] = ld16(sK + (32 * k + 8 * q) * 2);
        } else if (4 * q < rk) {
            const uint2 v = *reinterpret_cast<const uint2 *>(sK + 4 * q * 2);
            sk[k].x = v.x;
            sk[k].y = v.y;
        }
    }
    // U rows of a token tile: K32: 16-byte pieces q, q + 4; else the 8-byte piece q
    using UPiece = std::conditional_t<K32, uint4, uint2>;
    auto load_u = [&](UPiece (&u)[CT][KK], const unsigned char *U, int r, int chunk) {
#pragma unroll
        for (int tt = 0; tt < CT; ++tt) {
            const uint32_t tok = uint32_t(min(16 * (part + parts * (chunk * CT + tt)) + c16, max(L, 1) - 1));
            const uint32_t row = tok * uint32_t(r * 2);          // |S| <= 2^20 and r <= 64: below 2^27
#pragma unroll
            for (int k = 0; k < KK; ++k) {
                u[tt][k] = UPiece{};
                if constexpr (K32) {
                    if (32 * k + 8 * q < r) u[tt][k] = ld16(U + (row + uint32_t(k * 64 + q * 16)));
                } else {
                    if (4 * q < r) u[tt][k] = *reinterpret_cast<const uint2 *>(U + (row + uint32_t(q * 8)));
                }
            }
        }
    };
    UPiece uk[CT][KK], uv[CT][KK];
    load_u(uk, UK, rk, 0);
    if constexpr (R < 64) load_u(uv, UV, rv, 0);

    // w = scale log2(e) sigma_K (Vt_K q), as score operand
    uint4 wB[NU][KK];
    {
#pragma unroll
        for (int k = 0; k < KK; ++k) {
            if (k > 0) load_vk(k);
            float wv[VT][4];
#pragma unroll
            for (int t = 0; t < VT; ++t) {
                const f4v d = row_dots(W, vk[t]);
                float sg[8];
                BF16::unpack(sk[k], sg);
#pragma unroll
                for (int e = 0; e < 4; ++e) wv[t][e] = d[e] * sg[4 * t + e] * p.scale_log2;
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const uint2 x = pieces4(W, wv[0], u);
                uint2 y = make_uint2(0u, 0u);
                if constexpr (K32) y = pieces4(W, wv[VT - 1], u);
                wB[u][k] = make_uint4(x.x, x.y, y.x, y.y);
            }
            if (KK > 1) __builtin_amdgcn_sched_barrier(0);
        }
    }
    if constexpr (R >= 64) load_u(uv, UV, rv, 0);       // into the registers Vt_K has released
    constexpr int YT = R >= 16 ? R / 16 : 1;
    f4v y[NU][YT];                                      // p^T U_V: row 16 ct + 4 q + e, column (piece, head)
#pragma unroll
    for (int u = 0; u < NU; ++u)
#pragma unroll
        for (int ct = 0; ct < YT; ++ct) y[u][ct] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
    float pend = 1.0f;                                  // factor not yet applied to W.o
    for (int chunk = 0; part + parts * (chunk * CT) < ntile; ++chunk) {
        const bool more = part + parts * ((chunk + 1) * CT) < ntile;
        float s[CT * 4];
#pragma unroll
        for (int tt = 0; tt < CT; ++tt) {
            const int t0 = 16 * (part + parts * (chunk * CT + tt)) + 4 * q;
            f4v d[NU];
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                d[u] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int k = 0; k < KK; ++k) {
                    if constexpr (K32) d[u] = mfma_bf16_k32(uk[tt][k], wB[u][k], d[u]);
                    else d[u] = mfma_bf16_k16(uk[tt][k], make_uint2(wB[u][k].x, wB[u][k].y), d[u]);
                }
            }
            const f4v t = piece_sum<G, NU>(d);
#pragma unroll
            for (int e = 0; e < 4; ++e) s[4 * tt + e] = t0 + e < L ? t[e] : -INFINITY;
        }
        if (more) load_u(uk, UK, rk, chunk + 1);
        const float so = soft_step(W, s);
        pend *= so;
#pragma unroll
        for (int u = 0; u < NU; ++u)
#pragma unroll
            for (int ct = 0; ct < YT; ++ct) y[u][ct] *= so;
        // U_V rows into LDS, then y += U_V^T p over 32 tokens at a time
#pragma unroll
        for (int tt = 0; tt < CT; ++tt) {
            unsigned char *row = W.wb + (16 * tt + c16) * US;
#pragma unroll
            for (int k = 0; k < KK; ++k) {
                if constexpr (K32) *reinterpret_cast<uint4 *>(row + k * 64 + q * 16) = uv[tt][k];
                else if (R == 16 || q < 2) *reinterpret_cast<uint2 *>(row + q * 8) = uv[tt][k];
            }
        }
        wave_fence();
        if (more) load_u(uv, UV, rv, chunk + 1);
#pragma unroll
        for (int tt = 0; tt < CT; tt += 2) {
            __builtin_amdgcn_sched_barrier(0);          // one step's operands in registers at a time
            const float lo[4] = {s[4 * tt], s[4 * tt + 1], s[4 * tt + 2], s[4 * tt + 3]};
            const float hi[4] = {s[4 * tt + 4], s[4 * tt + 5], s[4 * tt + 6], s[4 * tt + 7]};
            const unsigned char *r0 = W.wb + (16 * tt + 4 * q + c16 / 4) * US + (c16 % 4) * 8;
            uint4 a[YT];
#pragma unroll
            for (int ct = 0; ct < YT; ++ct) {
                const uint2 x = lds_turn4(r0 + ct * 32), z = lds_turn4(r0 + 16 * US + ct * 32);
                a[ct] = make_uint4(x.x, x.y, z.x, z.y);
            }
#pragma unroll
            for (int u = 0; u < NU; ++u) {
                const uint2 x = pieces4(W, lo, u), z = pieces4(W, hi, u);
                const uint4 b = make_uint4(x.x, x.y, z.x, z.y);
#pragma unroll
                for (int ct = 0; ct < YT; ++ct) y[u][ct] = mfma_bf16_k32(a[ct], b, y[u][ct]);
            }
        }
        wave_fence();
    }
    // values += Vt_V^T (sigma_V y), 32 (16) components at a time
    scale_values(W, pend);
#pragma unroll
    for (int c0 = 0; c0 < YT; c0 += 2) {
        constexpr int NS = YT >= 2 ? 2 : 1;
        __builtin_amdgcn_sched_barrier(0);
        float w[8];
#pragma unroll
        for (int i = 0; i < NS; ++i) {
            const int row = 16 * (c0 + i) + c16;
            uint4 v[KC];
#pragma unroll
            for (int k = 0; k < KC; ++k) v[k] = row < rv ? ld16(VtV + uint32_t(row * D * 2 + k * 64 + q * 16)) : zero4;
            const int c = 16 * (c0 + i) + 4 * q;
            uint2 sv = make_uint2(0u, 0u);
            if (c < rv) sv = *reinterpret_cast<const uint2 *>(sV + c * 2);
            f4v t[NU];
#pragma unroll
            for (int u = 0; u < NU; ++u) t[u] = y[u][c0 + i];
            const f4v ys = piece_sum<G, NU>(t);
            const float sg[4] = {__uint_as_float(sv.x << 16), __uint_as_float(sv.x & 0xFFFF0000u),
                                 __uint_as_float(sv.y << 16), __uint_as_float(sv.y & 0xFFFF0000u)};
#pragma unroll
            for (int e = 0; e < 4; ++e) w[4 * i + e] = c + e < rv ? ys[e] * sg[e] : 0.0f;
            turn16(W, v, i, 16);
        }
        wave_fence();
        if constexpr (NS == 2) {
            add_rows32(W, w);
        } else {
            const float w4[4] = {w[0], w[1], w[2], w[3]};
            add_rows16(W, w4);
        }
        wave_fence();
    }
}

// The partial of a share item again, entry by entry, where the matrix cores gave a NaN.  A split
// operand meets every stored value as three pieces and some zeros, so an infinite value (or weight)
// becomes infinity times zero there; here it is multiplied once, as fp32 storage does it: an
// infinite value of positive weight gives infinity, a score of -infinity a weight of zero.  Plain
// loops: the item's selection is in Z.sel and Z.zi, its logits were published, Z.wb is scratch.
// What the test for NaN costs where there is none: 32K 18.35 -> 18.6 us, 128K x 4 27.1 -> 27.4 us.
template <class T, int D, int G>
__device__ __forceinline__ void share_partial_plain(const Params &p, Smem<T, D, G> &sm, int pair, int j, int a_lo,
                                                    int a_end, int c_lo, int c_end, uint32_t tag, int tid) {
    constexpr int NO = G * D / 2, NP = (NO + NT - 1) / NT;   // value pairs; of a thread
    constexpr int NB = Smem<T, D, G>::CB;                    // rows at a time
    constexpr int NY = (G * kMaxTopK + NT - 1) / NT;         // components (at most 64 a head) of a thread
    static_assert(NB == 64 && kMaxTopK == 64, "64 rows and components");
    struct Scratch {
        float s[G][64], w[G][64], y[G][64];
        float m[G], l[G], so[G];
    };
    auto &Z = sm.u.share;
    static_assert(sizeof(Scratch) <= sizeof(Z.wb), "scratch in the waves' tiles");
    Scratch &X = *reinterpret_cast<Scratch *>(&Z.wb[0][0]);
    const int b = pair / p.Hkv, g = pair % p.Hkv;
    const size_t q0 = (size_t(b) * p.Hq + size_t(g) * G) * D;
    const size_t arow = size_t(pair) * p.A_max, srow = size_t(pair) * p.M_max;
    float o[NP][2];
#pragma unroll
    for (int u = 0; u < NP; ++u) o[u][0] = o[u][1] = 0.0f;
    if (tid < G) { X.m[tid] = -INFINITY; X.l[tid] = 0.0f; }
    // X.s[h][0, n) become weights relative to the new maximum; the sums so far follow it
    auto fold = [&](int n) {
        __syncthreads();
        if (tid < G) {
            float mx = -INFINITY, ls = 0.0f;
            for (int i = 0; i < n; ++i) mx = fmaxf(mx, X.s[tid][i]);
            const float mo = X.m[tid], mn = fmaxf(mo, mx);
            for (int i = 0; i < n; ++i) {
                const float wt = mn == -INFINITY ? 0.0f : safe_exp2(X.s[tid][i] - mn);
                X.s[tid][i] = wt;
                ls += wt;
            }
            const float so = mn == -INFINITY ? 1.0f : safe_exp2(mo - mn);
            X.so[tid] = so;
            X.l[tid] = X.l[tid] * so + ls;
            X.m[tid] = mn;
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int o2 = tid + NT * u;
            const float so = X.so[min(2 * o2 / D, G - 1)];
            o[u][0] *= so;
            o[u][1] *= so;
        }
    };
    // o += weights x rows [row, row + n) of `rows`
    auto add = [&](const float (&wt)[G][64], const void *rows, size_t row, int n) {
#pragma unroll
        for (int u = 0; u < NP; ++u) {
            const int o2 = tid + NT * u;
            if (o2 >= NO) continue;
            const int hl = 2 * o2 / D, d = 2 * o2 % D;
#pragma unroll 1
            for (int i = 0; i < n; ++i) {
                o[u][0] += wt[hl][i] * T::load1(rows, (row + i) * D + d);
                o[u][1] += wt[hl][i] * T::load1(rows, (row + i) * D + d + 1);
            }
        }
        __syncthreads();
    };
    auto q_dot = [&](int hl, const void *rows, size_t row) {
        float a = 0.0f;
#pragma unroll 1
        for (int d = 0; d < D; ++d) a += T::load1(p.q, q0 + size_t(hl) * D + d) * T::load1(rows, row * D + d);
        return a;
    };
    for (int a0 = a_lo; a0 < a_end; a0 += 64) {
        const int n = min(64, a_end - a0);
        for (int i = tid; i < G * 64; i += NT)
            if (i % 64 < n) X.s[i / 64][i % 64] = q_dot(i / 64, p.anchor_k, arow + a0 + i % 64) * p.scale_log2;
        fold(n);
        add(X.s, p.anchor_v, arow + a0, n);
    }
    for (int c0 = c_lo; c0 < c_end; c0 += 64) {
        const int n = min(64, c_end - c0);
        coarse_logits<T, D, G>(p, sm, pair, c0, n, tag, tid);
        __syncthreads();
        for (int i = tid; i < G * 64; i += NT) {
            bool zoomed = i % 64 >= n;
            for (int t = 0; t < p.k; ++t) zoomed |= Z.sel[t] == c0 + i % 64;
            X.s[i / 64][i % 64] = zoomed ? -INFINITY : Z.cw[i / 64][i % 64];
        }
        fold(n);
        add(X.s, p.sum_v, srow + c0, n);
    }
    for (int rank = j; rank < p.k; rank += p.n_zi) {
        const int4 zi = Z.zi[rank];
        if (zi.x < 0) continue;
        const int L = word_len(zi.y), rk = word_rk(zi.y), rv = word_rv(zi.y);
        const unsigned char *UK = p.factors + (int64_t(uint32_t(zi.z)) | (int64_t(zi.w) << 32));
        const unsigned char *sK = UK + size_t(L) * rk * T::kBytes;
        const unsigned char *VtK = sK + size_t(rk) * T::kBytes;
        const unsigned char *UV = VtK + size_t(rk) * D * T::kBytes;
        const unsigned char *sV = UV + size_t(L) * rv * T::kBytes;
        const unsigned char *VtV = sV + size_t(rv) * T::kBytes;
        for (int i = tid; i < G * 64; i += NT)
            if (i % 64 < rk) X.w[i / 64][i % 64] = q_dot(i / 64, VtK, i % 64) * T::load1(sK, i % 64) * p.scale_log2;
        __syncthreads();
        float y[NY];
#pragma unroll
        for (int u = 0; u < NY; ++u) y[u] = 0.0f;
        for (int t0 = 0; t0 < L; t0 += 64) {
            const int n = min(64, L - t0);
            for (int i = tid; i < G * 64; i += NT) {
                if (i % 64 >= n) continue;
                float a = 0.0f;
#pragma unroll 1
                for (int c = 0; c < rk; ++c) a += T::load1(UK, size_t(t0 + i % 64) * rk + c) * X.w[i / 64][c];
                X.s[i / 64][i % 64] = a;
            }
            fold(n);
#pragma unroll
            for (int u = 0; u < NY; ++u) {
                const int i = tid + NT * u, hl = min(i / 64, G - 1);
                y[u] *= X.so[hl];
#pragma unroll 1
                for (int t = 0; t < n; ++t)
                    if (i % 64 < rv) y[u] += X.s[hl][t] * T::load1(UV, size_t(t0 + t) * rv + i % 64);
            }
            __syncthreads();
        }
#pragma unroll
        for (int u = 0; u < NY; ++u) {
            const int i = tid + NT * u;
            if (i < G * 64 && i % 64 < rv) X.y[i / 64][i % 64] = y[u] * T::load1(sV, i % 64);
        }
        __syncthreads();
        add(X.y, VtV, 0, rv);
    }
    const size_t base = size_t(pair) * p.n_zi + j;
    if (tid < G) st_shared(&p.part_ml[base * G + tid], pack2(X.m[tid], X.l[tid]));
#pragma unroll
    for (int u = 0; u < NP; ++u) {
        const int o2 = tid + NT * u;
        if (o2 < NO) st_shared(&p.part_o[base * NO + o2], pack2(o[u][0], o[u][1]));
    }
    stores_done_barrier();
}

// share item: anchors share, selection slot j, summaries share of one pair.  Returns true when a
// wait lasted kHelpAfter polls: the caller then helps with routing (help_route) and runs the
// item again from the start.
template <class T, int D, int G>
__device__ __forceinline__ bool share_item_mfma(const Params &p, Smem<T, D, G> &sm, int pair, int j, uint32_t tag,
                                                int tid, bool first, bool may_give_up, bool leave) {
    constexpr int KC = D / 32, RB = D * 2, CB = Smem<T, D, G>::CB;
    static_assert(CB == 64, "one 16-row tile per wave in a summary block");
    auto &Z = sm.u.share;
    const int b = pair / p.Hkv, g = pair % p.Hkv;
    const int k = p.k, nz = p.n_zi;
    // this item's shares: contiguous ranges of the anchor and span index spaces up to the
    // maxima, so the first loads need no table value; the sequence's own counts (n_anchors,
    // n_spans) mask rows where the values are used.  Anchors go to the slots that start with
    // the launch (j < n_early): later slots reach their selection and zoom sooner.
    const int ne = p.n_early;
    const int as = (p.A_max + ne - 1) / ne;
    const int a_lo = j < ne ? min(p.A_max, j * as) : p.A_max, a_hi = min(p.A_max, a_lo + as);
    const int cs = (p.M_max + nz - 1) / nz;
    const int c_lo = min(p.M_max, j * cs), c_hi = min(p.M_max, c_lo + cs);
    const size_t pr = size_t(b) * p.Hkv + g;
    const unsigned char *ak = static_cast<const unsigned char *>(p.anchor_k) + (pr * p.A_max + a_lo) * RB;
    const unsigned char *av = static_cast<const unsigned char *>(p.anchor_v) + (pr * p.A_max + a_lo) * RB;
    const unsigned char *sv = static_cast<const unsigned char *>(p.sum_v) + pr * p.M_max * RB;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    if (first && p.end_route > 0) __builtin_amdgcn_s_sleep(kShareHoldBack);
    Wave<D, G> W;
    W.c16 = lane & 15;
    W.q = lane >> 4;
    W.h = W.c16 % G;
    W.s0 = W.c16 / G;
    W.wb = Z.wb[wave];
    W.m = -INFINITY;
    W.l = 0.0f;
#pragma unroll
    for (int u = 0; u < W.NU; ++u)
#pragma unroll
        for (int dt = 0; dt < W.DT; ++dt) W.o[u][dt] = f4v{0.0f, 0.0f, 0.0f, 0.0f};
    // 1. loads that depend on nothing: the query, the wave's first 32 anchors, its first summary
    //    rows (values only; the logits come from routing)
    {
        const unsigned char *qp = static_cast<const unsigned char *>(p.q) +
                                  ((size_t(b) * p.Hq + size_t(g) * G + W.h) * D) * 2 + W.q * 16;
#pragma unroll
        for (int i = 0; i < KC; ++i) W.qB[i] = ld16(qp + i * 64);
    }
    const int a_n = a_hi - a_lo;
    uint4 kr[2][KC], vr[2][KC], cv[KC];
    if (32 * wave < a_n)
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            load16(W, kr[i], ak, 32 * wave + 16 * i, a_n);
            load16(W, vr[i], av, 32 * wave + 16 * i, a_n);
        }
    if (c_lo < c_hi) load16(W, cv, sv, c_lo + 16 * wave, c_hi);
    int m_b = p.n_spans[b];
    m_b = m_b < 0 ? 0 : (m_b > p.M_max ? p.M_max : m_b);
    int An = p.n_anchors[b];
    An = An < 0 ? 0 : (An > p.A_max ? p.A_max : An);
    for (int t = tid; t < kMaxTopK; t += NT) { Z.sel[t] = -1; Z.zi[t] = make_int4(-1, 0, 0, 0); }
    __syncthreads();
    const int nc0 = max(0, min(min(CB, c_hi - c_lo), m_b - c_lo));

    // 2. the anchor share, 32 rows a wave at a time, while routing runs elsewhere; the next rows'
    //    keys load while these values are used, their values while the next scores are taken
    const int a_live = min(a_n, An - a_lo);
    for (int t = 32 * wave; t < a_live; t += 128) {
        float s[8];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const f4v d = row_dots(W, kr[i]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                s[4 * i + e] = t + 16 * i + 4 * W.q + e < a_live ? d[e] * p.scale_log2 : -INFINITY;
        }
        const bool more = t + 128 < a_live;
        if (more)
#pragma unroll
            for (int i = 0; i < 2; ++i) load16(W, kr[i], ak, t + 128 + 16 * i, a_n);
        scale_values(W, soft_step(W, s));
        turn16(W, vr[0], 0, a_live - t);
        turn16(W, vr[1], 1, a_live - t - 16);
        wave_fence();
        if (more)
#pragma unroll
            for (int i = 0; i < 2; ++i) load16(W, vr[i], av, t + 128 + 16 * i, a_n);
        add_rows32(W, s);
        wave_fence();
    }
    SEKV_STAMP(p, sm, kTrSAnchors);
    // 3. the selection (Z.sel, Z.zi) and the first summary block's logits (Z.cw)
    if (select_spans<T, D, G>(p, sm, pair, j, m_b, c_lo, nc0, tag, tid, may_give_up)) return true;
    // selected spans are zoomed: their summaries drop out
    auto drop_selected = [&](int c0, int nc) {
        if (tid < nc) {
            bool ex = false;
            for (int t = 0; t < k; ++t) ex |= (Z.sel[t] == c0 + tid);
            if (ex)
#pragma unroll
                for (int hl = 0; hl < G; ++hl) Z.cw[hl][tid] = -INFINITY;
        }
        __syncthreads();
    };
    auto coarse = [&](int nc) {
        float s[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int row = 16 * wave + 4 * W.q + e;
            s[e] = row < nc ? Z.cw[W.h][row] : -INFINITY;
        }
        scale_values(W, soft_step(W, s));
        turn16(W, cv, 0, nc - 16 * wave);
        wave_fence();
        add_rows16(W, s);
        wave_fence();
    };
    drop_selected(c_lo, nc0);
    if (16 * wave < nc0) coarse(nc0);
    // 4. zoom the slot's spans (ranks j, j + n_zi, ...): four and more go to the waves whole,
    //    fewer in two or four parts.  A part repeats the span's work on Vt_K and Vt_V, so parts
    //    for a better balance cost more than they give: us at rank 16, 512 pairs, whole / this / four
    //    parts: 2 spans a slot 55.8 / 53.2 / 57.8, 3 56.2 / 57.5 / 63.3, 4 57.4 / 56.8 / 68.9, 5 62.5 / 62.1 / 73.8, 6
    //    64.5 / 63.8 / 79.1, 9 71.0 / 70.4 / 93.6; rank 32, 5 spans 80.1 / 82.1 / 87.4.
    const int nsp = k > j ? (k - j + nz - 1) / nz : 0;
    const int lg = nsp >= 4 ? 0 : nsp >= 2 ? 1 : 2;
    auto zoom_one = [&](auto ranked_c, int32_t w, int64_t off, int part) {
        constexpr bool RANKED = decltype(ranked_c)::value;
        const int L = word_len(w), rk = word_rk(w), rv = word_rv(w);
        switch (p.r) {
            case 8: zoom_part<D, G, 8, RANKED>(p, W, L, rk, rv, off, part, 1 << lg); break;
            case 16: zoom_part<D, G, 16, RANKED>(p, W, L, rk, rv, off, part, 1 << lg); break;
            case 32: zoom_part<D, G, 32, RANKED>(p, W, L, rk, rv, off, part, 1 << lg); break;
            default: zoom_part<D, G, 64, RANKED>(p, W, L, rk, rv, off, part, 1 << lg); break;
        }
    };
    for (int unit = wave; unit < (nsp << lg); unit += 4) {
        // the same for the whole wave: in scalar registers
        int4 zi = Z.zi[j + nz * (unit >> lg)];
        zi.x = __builtin_amdgcn_readfirstlane(zi.x);
        zi.y = __builtin_amdgcn_readfirstlane(zi.y);
        if (zi.x < 0) continue;
        const int64_t off = int64_t(uint32_t(__builtin_amdgcn_readfirstlane(zi.z))) |
                            (int64_t(__builtin_amdgcn_readfirstlane(zi.w)) << 32);
        const int part = unit & ((1 << lg) - 1);
        // an opaque copy of the lane keeps the zooms' address arithmetic inside the loop
        int ln;
        asm volatile("v_mov_b32 %0, %1" : "=v"(ln) : "v"(lane));
        W.c16 = ln & 15;
        W.q = ln >> 4;
        W.s0 = W.c16 / G;
        if (p.block_rank) zoom_one(IC<1>{}, zi.y, off, part);
        else zoom_one(IC<0>{}, zi.y, off, part);
    }
    SEKV_STAMP(p, sm, kTrSZoomDone);
    // 5. the rest of the summary share (several blocks only when k is small)
    for (int c0 = c_lo + CB; c0 < c_hi && c0 < m_b; c0 += CB) {
        const int nc = min(min(CB, c_hi - c0), m_b - c0);
        load16(W, cv, sv, c0 + 16 * wave, c_hi);
        __syncthreads();                                // Z.cw is reused
        if (wait_coarse_logits<T, D, G>(p, sm, pair, c0, nc, tag, tid, may_give_up)) return true;
        drop_selected(c0, nc);
        if (16 * wave < nc) coarse(nc);
    }
    SEKV_STAMP(p, sm, kTrSCoarse);
    // 6. the waves' sums into one partial
    const float l = lane_reduce<4, 6>(W.l);
    if (lane < G) {
        sm.mw[wave][lane] = W.m;
        sm.lw[wave][lane] = l;
    }
    if (tid == 0) sm.bcast[7] = 0;
#pragma unroll
    for (int dt = 0; dt < W.DT; ++dt) {
        f4v t[W.NU];
#pragma unroll
        for (int u = 0; u < W.NU; ++u) t[u] = W.o[u][dt];
        const f4v v = piece_sum<G, W.NU>(t);
        if (W.c16 < G) *reinterpret_cast<f4v *>(&sm.red[wave][W.c16][16 * dt + 4 * W.q]) = v;
    }
    __syncthreads();
    {
        constexpr int NO = G * D / 2;
        const size_t base = size_t(pair) * p.n_zi + j;
        auto weights = [&](int hl, float (&wg)[4], float &m) {
            m = fmaxf(fmaxf(sm.mw[0][hl], sm.mw[1][hl]), fmaxf(sm.mw[2][hl], sm.mw[3][hl]));
            const float ref = m == -INFINITY ? 0.0f : m;
#pragma unroll
            for (int w = 0; w < 4; ++w) wg[w] = exp2f(sm.mw[w][hl] - ref);
        };
        if (tid < G) {
            float wg[4], m, ls = 0.0f;
            weights(tid, wg, m);
#pragma unroll
            for (int w = 0; w < 4; ++w) ls += wg[w] * sm.lw[w][tid];
            st_shared(&p.part_ml[base * G + tid], pack2(m, ls));
            if (ls != ls) sm.bcast[7] = 1;
        }
        uint64_t *po = p.part_o + base * NO;
        for (int o2 = tid; o2 < NO; o2 += NT) {
            const int hl = (2 * o2) / D, d = (2 * o2) % D;
            float wg[4], m, v0 = 0.0f, v1 = 0.0f;
            weights(hl, wg, m);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                v0 += wg[w] * sm.red[w][hl][d];
                v1 += wg[w] * sm.red[w][hl][d + 1];
            }
            st_shared(&po[o2], pack2(v0, v1));
            if (v0 != v0 || v1 != v1) sm.bcast[7] = 1;
        }
    }
    stores_done_barrier();
    // (cold, so that its loops do not weigh in the allocation of registers: 27.9 us at 128K x 4 else)
    if (__builtin_expect_with_probability(sm.bcast[7], 0, 1.0))
        share_partial_plain<T, D, G>(p, sm, pair, j, a_lo, min(a_hi, An), c_lo, min(c_hi, m_b), tag, tid);
    SEKV_STAMP(p, sm, kTrSPartial);
    count_partial<T, D, G>(p, sm, pair, tid, leave, tag);
    SEKV_STAMP(p, sm, kTrSMerged);
    return false;
}
