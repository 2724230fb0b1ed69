// The expert network and the router in f32 arithmetic, for any widths and both activation types: the f32 layers whose widths
// are no multiples of four (the others have r3_f32.hip), and the bf16 shapes that the bf16 MFMA kernels do not take.  Tiles run on
// the f32 matrix instruction (16x16x4): products and sums are those of an f32 FMA chain (bf16 operands are widened, so their
// products are exact).
//
// What bounds it: the f32 matrix pipe (154 TFLOP/s is what a large library product reaches here) where a
// shape has work, launch and load latency where it has not.  Operands go through registers into a
// double-buffered LDS tile of 32 k, the next tile's loads in flight while the current one is multiplied; the
// f32 instruction takes 32 cycles, so the fragment reads (16 bytes per lane and 16 k from a row-major tile,
// 4 bytes from a k-major one) are far from being felt.  Tiles are 128 x 128 (4 waves of 64 x 64) where
// that still gives every compute unit two of them, else 64 x 64 (4 waves of 32 x 32).
// Measured on T=3001 d=1000 E=64 K=6 F=704 bf16: 193 ms with one thread per output element, 4.2 ms here.
#include <algorithm>

#include "r3_f32.h"
#include "r3_kernels.h"
#include "r3_plain_tiles.h"

namespace r3 {

// ---------------------------------------------------------------------------
// Row-tiled contractions over the expert-sorted rows (listed in r3_f32.h; FFN1's P: gate | up halves).
// `in0` holds the rows; FFN1 with perm != NULL reads row r as in0[perm[r] / K], and with gates != NULL
// scales H by the gate of the row's slot.
// ---------------------------------------------------------------------------
template <class C, int MODE, typename T, bool VEC>
__global__ void __launch_bounds__(C::NT)
plain_rows_kernel(int d, int E, int F, const int32_t *__restrict__ offsets, const T *__restrict__ in0,
                  const T *__restrict__ in1, const int32_t *__restrict__ perm, int K, const float *__restrict__ gates,
                  const T *__restrict__ W0, const T *__restrict__ W1, const T *__restrict__ FAin,
                  const T *__restrict__ FBin, T *__restrict__ out0, T *__restrict__ out1, T *__restrict__ out2) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    constexpr int BF = MODE == PLAIN_FFN1 ? C::BP / 2 : C::BP;            // output features per tile
    const int NOUT = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) ? F : d;
    const int KK = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) ? d : F;      // width of the row operand
    const int npt = (NOUT + BF - 1) / BF;
    const RowTile t = find_row_tile<false>(offsets, E, C::BQ, blockIdx.x, npt);
    if (t.e < 0) return;
    const int p0 = t.col * BF, rows = t.row1 - t.row0;
    const T *w0 = W0 + (int64_t)t.e * d * F;
    const T *w1 = (MODE == PLAIN_FFN1 || MODE == PLAIN_DXP) ? W1 + (int64_t)t.e * d * F : nullptr;

    // the thread's rows of the row operand do not change over k
    constexpr int NQ = C::BQ * C::BK / 4 / C::NT, RSTEP = C::NT / (C::BK / 4);
    const T *qrow[NQ], *qrow1[MODE == PLAIN_DXP ? NQ : 1];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
        const int r = threadIdx.x / (C::BK / 4) + i * RSTEP;
        const int row = t.row0 + min(r, rows - 1);
        const int src = (MODE == PLAIN_FFN1 && perm) ? perm[row] / K : row;
        qrow[i] = in0 + (int64_t)src * KK;
        if constexpr (MODE == PLAIN_DXP) qrow1[i] = in1 + (int64_t)row * KK;
    }
    PlainAcc<C> acc;
    plain_zero<C>(acc);
    auto none = [](int) {};
    const int nk = (KK + C::BK - 1) / C::BK;
    auto fq = [&](int i, int, int k) { return load4<T, VEC>(qrow[i] + k, KK - k); };
    if constexpr (MODE == PLAIN_FFN1) {
        // P columns: per wave WTP / 2 features of W_gate, then the same features of W_up, so that a lane holds
        // both pre-activations of its (row, feature) pairs
        auto fp = [&](int, int k, int c) {
            const int w = c / C::WTP, cc = c % C::WTP, f = p0 + w * (C::WTP / 2) + cc % (C::WTP / 2);
            return load4<T, VEC>((cc < C::WTP / 2 ? w0 : w1) + (int64_t)k * F + f, k < d ? F - f : 0);
        };
        plain_mainloop<C, true, false>(acc, nk, fp, fq, none, lds);
    } else if constexpr (MODE == PLAIN_DOWN) {
        auto fp = [&](int, int k, int c) { return load4<T, VEC>(w0 + (int64_t)k * d + p0 + c, k < F ? d - p0 - c : 0); };
        plain_mainloop<C, true, false>(acc, nk, fp, fq, none, lds);
    } else {
        auto fp = [&](int, int r, int k) { return load4<T, VEC>(w0 + (int64_t)(p0 + r) * KK + k, p0 + r < NOUT ? KK - k : 0); };
        plain_mainloop<C, false, false>(acc, nk, fp, fq, none, lds);
        if constexpr (MODE == PLAIN_DXP) {
            auto fq1 = [&](int i, int, int k) { return load4<T, VEC>(qrow1[i] + k, KK - k); };
            auto fp1 = [&](int, int r, int k) { return load4<T, VEC>(w1 + (int64_t)(p0 + r) * KK + k, p0 + r < NOUT ? KK - k : 0); };
            plain_mainloop<C, false, false>(acc, nk, fp1, fq1, none, lds);
        }
    }
    plain_results<C>([&](int tp, int tq, int p, int q) {
        if (q >= rows) return;
        const int row = t.row0 + q;
        if constexpr (MODE == PLAIN_FFN1) {
            if (tp >= C::TP / 2) return;
            const int f = p0 + p / C::WTP * (C::WTP / 2) + p % C::WTP;
            if (f >= F) return;
            const float gq = gates ? gates[perm[row]] : 1.0f;
            float h[4], fa[4], fb[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float a = acc[tp][tq][i], b = acc[tp + C::TP / 2][tq][i];
                const float sg = sigmoidf_(a);
                h[i] = gq * (a * sg * b);
                fa[i] = b * sg * (1.0f + a * (1.0f - sg));
                fb[i] = a * sg;
            }
            const int64_t o = (int64_t)row * F + f;
            store4<T, VEC>(out0 + o, h, F - f);
            if (out1) store4<T, VEC>(out1 + o, fa, F - f);
            if (out2) store4<T, VEC>(out2 + o, fb, F - f);
        } else {
            const int c = p0 + p;
            if (c >= NOUT) return;
            const int64_t o = (int64_t)row * NOUT + c;
            float v[4] = {acc[tp][tq][0], acc[tp][tq][1], acc[tp][tq][2], acc[tp][tq][3]};
            if constexpr (MODE == PLAIN_DH) {
                const float4 a = load4<T, VEC>(FAin + o, F - c), b = load4<T, VEC>(FBin + o, F - c);
                float va[4] = {v[0] * a.x, v[1] * a.y, v[2] * a.z, v[3] * a.w};
                float vb[4] = {v[0] * b.x, v[1] * b.y, v[2] * b.z, v[3] * b.w};
                store4<T, VEC>(out0 + o, va, F - c);
                store4<T, VEC>(out1 + o, vb, F - c);
            } else {
                store4<T, VEC>(out0 + o, v, NOUT - c);
            }
        }
    });
}

// ---------------------------------------------------------------------------
// The three weight gradients of every expert in one launch, out[q][p] (+)= sum_r Qs[r][q] Ps[r][p] over the
// expert's rows:  dW_down: Qs = H, Ps = dYp (or dy through perm);  dW_gate, dW_up: Qs = the token rows,
// Ps = dA, dB.  A row operand with a perm is the un-permuted matrix and row r is its row perm[r] / K.
// ---------------------------------------------------------------------------
template <typename T>
struct PlainWgrad {
    const T *Qs, *Ps;
    const int32_t *qperm, *pperm;
    float *out;
    int NQ, NP, tiles;   // tiles: per expert
};
template <typename T>
struct PlainWgrad3 {
    PlainWgrad<T> g[3];
};

template <class C, typename T, bool VEC>
__global__ void __launch_bounds__(C::NT)
plain_wgrad_kernel(int E, int K, const int32_t *__restrict__ offsets, PlainWgrad3<T> all, int accumulate) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int per = all.g[0].tiles + all.g[1].tiles + all.g[2].tiles;
    const int e = blockIdx.x / per;
    int rem = blockIdx.x - e * per, which = 0;
    while (rem >= all.g[which].tiles) rem -= all.g[which++].tiles;
    const PlainWgrad<T> g = all.g[which];
    const int npt = (g.NP + C::BP - 1) / C::BP;
    const int qt = rem / npt, q0 = qt * C::BQ, p0 = (rem - qt * npt) * C::BP;
    const int r0 = offsets[e], n = offsets[e + 1] - r0;
    // a thread's k-rows of a tile: one of the gathered matrix's rows each, fetched a tile ahead
    constexpr int NPL = C::BP * C::BK / 4 / C::NT, NQL = C::BQ * C::BK / 4 / C::NT;
    constexpr int PSTEP = C::NT / (C::BP / 4), QSTEP = C::NT / (C::BQ / 4);
    int prow[NPL], qrow[NQL], pnext[NPL] = {}, qnext[NQL] = {};
    auto pre = [&](int kt) {
#pragma unroll
        for (int i = 0; i < NPL; ++i) {
            prow[i] = pnext[i];
            const int r = r0 + min(kt * C::BK + (int)threadIdx.x / (C::BP / 4) + i * PSTEP, max(n - 1, 0));
            pnext[i] = n > 0 && g.pperm ? g.pperm[r] / K : r;
        }
#pragma unroll
        for (int i = 0; i < NQL; ++i) {
            qrow[i] = qnext[i];
            const int r = r0 + min(kt * C::BK + (int)threadIdx.x / (C::BQ / 4) + i * QSTEP, max(n - 1, 0));
            qnext[i] = n > 0 && g.qperm ? g.qperm[r] / K : r;
        }
    };
    pre(0);   // (plain_mainloop shifts once more before it loads tile 0)
    auto fp = [&](int i, int k, int c) {
        return load4<T, VEC>(g.Ps + (int64_t)prow[i] * g.NP + p0 + c, k < n ? g.NP - p0 - c : 0);
    };
    auto fq = [&](int i, int k, int c) {
        return load4<T, VEC>(g.Qs + (int64_t)qrow[i] * g.NQ + q0 + c, k < n ? g.NQ - q0 - c : 0);
    };
    PlainAcc<C> acc;
    plain_zero<C>(acc);
    plain_mainloop<C, true, true>(acc, (n + C::BK - 1) / C::BK, fp, fq, [&](int kt) { pre(kt + 1); }, lds);
    float *o = g.out + (int64_t)e * g.NQ * g.NP;
    plain_results<C>([&](int tp, int tq, int p, int q) {
        if (q0 + q >= g.NQ || p0 + p >= g.NP) return;
        const int64_t at = (int64_t)(q0 + q) * g.NP + p0 + p;
        float v[4] = {acc[tp][tq][0], acc[tp][tq][1], acc[tp][tq][2], acc[tp][tq][3]};
        if (accumulate) {
            const float4 old = load4<float, VEC>(o + at, g.NP - p0 - p);
            v[0] += old.x; v[1] += old.y; v[2] += old.z; v[3] += old.w;
        }
        store4<float, VEC>(o + at, v, g.NP - p0 - p);
    });
}

// ---------------------------------------------------------------------------
// Router: logits s[t][e] = sum_c x[t][c] W_r[c][e] (+ bias), and the parts of dW_r.
// ---------------------------------------------------------------------------
template <class C, typename T, bool VECX, bool VECE>
__global__ void __launch_bounds__(C::NT)
plain_logits_kernel(int Tn, int d, int E, const T *__restrict__ x, const T *__restrict__ Wr, const float *__restrict__ bias,
                    float *__restrict__ logits) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int npt = (E + C::BP - 1) / C::BP;
    const int qt = blockIdx.x / npt, t0 = qt * C::BQ, p0 = (blockIdx.x - qt * npt) * C::BP;
    auto fp = [&](int, int k, int c) { return load4<T, VECE>(Wr + (int64_t)k * E + p0 + c, k < d ? E - p0 - c : 0); };
    auto fq = [&](int, int r, int k) { return load4<T, VECX>(x + (int64_t)min(t0 + r, Tn - 1) * d + k, d - k); };
    PlainAcc<C> acc;
    plain_zero<C>(acc);
    plain_mainloop<C, true, false>(acc, (d + C::BK - 1) / C::BK, fp, fq, [](int) {}, lds);
    plain_results<C>([&](int tp, int tq, int p, int q) {
        if (t0 + q >= Tn || p0 + p >= E) return;
        float v[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = acc[tp][tq][i] + (bias && p0 + p + i < E ? bias[p0 + p + i] : 0.0f);
        store4<float, VECE>(logits + (int64_t)(t0 + q) * E + p0 + p, v, E - p0 - p);
    });
}

template <class C, typename T, bool VECX, typename IdxT>
__global__ void __launch_bounds__(C::NT) plain_dwr_kernel(PlainDwr<T, IdxT> a) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    plain_dwr_tile<C, T, VECX>(a, blockIdx.x, lds);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
namespace {

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
constexpr int kFill = 512;   // 128 x 128 tiles from two per compute unit on; below, four times as many 64 x 64 ones

template <class K>
void allow_lds(K kernel, int bytes) {
    (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

template <class C, int MODE, typename T, bool VEC>
void rows_launch(int S, int d, int E, int F, const int32_t *offsets, const T *in0, const T *in1, const int32_t *perm, int K,
                 const float *gates, const T *W0, const T *W1, const T *FA, const T *FB, T *o0, T *o1, T *o2, hipStream_t s) {
    const int NOUT = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) ? F : d, BF = MODE == PLAIN_FFN1 ? C::BP / 2 : C::BP;
    auto k = plain_rows_kernel<C, MODE, T, VEC>;
    allow_lds(k, C::LDS);
    k<<<(unsigned)(max_row_tiles(S, E, C::BQ) * ceil_div(NOUT, BF)), C::NT, C::LDS, s>>>(d, E, F, offsets, in0, in1, perm, K, gates,
                                                                                     W0, W1, FA, FB, o0, o1, o2);
}

template <int MODE, typename T>
hipError_t rows_any(int S, int d, int E, int F, const int32_t *offsets, const void *in0, const void *in1, int Tn,
                    const int32_t *perm, int K, const float *gates, const void *W0, const void *W1, const void *FA, const void *FB, void *o0,
                    void *o1, void *o2, hipStream_t s) {
    const bool vec = d % 4 == 0 && F % 4 == 0;
#define R3_ROWS(C, V)                                                                                                   \
    rows_launch<C, MODE, T, V>(S, d, E, F, offsets, (const T *)in0, (const T *)in1, perm, K, gates, (const T *)W0,      \
                               (const T *)W1, (const T *)FA, (const T *)FB, (T *)o0, (T *)o1, (T *)o2, s)
    if constexpr (sizeof(T) == 4) {
        if (vec)
            return f32_rows(MODE, S, d, E, F, offsets, (const T *)in0, (const T *)in1, Tn, perm, K, gates, (const T *)W0,
                            (const T *)W1, (const T *)FA, (const T *)FB, (T *)o0, (T *)o1, (T *)o2, s);
        R3_ROWS(PlainSmall, false);
    } else {
        const int NOUT = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) ? F : d;
        const bool big = ceil_div(S, 128) * ceil_div(NOUT, MODE == PLAIN_FFN1 ? 64 : 128) >= kFill;
        if (vec && big) R3_ROWS(PlainBig, true);
        else if (vec) R3_ROWS(PlainSmall, true);
        else R3_ROWS(PlainSmall, false);
    }
#undef R3_ROWS
    return hipGetLastError();
}

template <int MODE>
hipError_t rows_by_act(int act, int S, int d, int E, int F, const int32_t *offsets, const void *in0, const void *in1,
                       int Tn, const int32_t *perm, int K, const float *gates, const void *W0, const void *W1, const void *FA,
                       const void *FB, void *o0, void *o1, void *o2, hipStream_t s) {
    return act == R3_BF16 ? rows_any<MODE, bf16_t>(S, d, E, F, offsets, in0, in1, Tn, perm, K, gates, W0, W1, FA, FB, o0, o1, o2, s)
                          : rows_any<MODE, float>(S, d, E, F, offsets, in0, in1, Tn, perm, K, gates, W0, W1, FA, FB, o0, o1, o2, s);
}

template <class C, typename T, bool VEC>
void wgrad_launch(int E, int K, const int32_t *offsets, PlainWgrad3<T> all, int accumulate, hipStream_t s) {
    int per = 0;
    for (auto &g : all.g) per += g.tiles = (int)(g.out ? ceil_div(g.NQ, C::BQ) * ceil_div(g.NP, C::BP) : 0);
    auto k = plain_wgrad_kernel<C, T, VEC>;
    allow_lds(k, C::LDS);
    k<<<(unsigned)((int64_t)E * per), C::NT, C::LDS, s>>>(E, K, offsets, all, accumulate);
}

template <typename T>
hipError_t wgrads_any(int d, int E, int F, int Tn, int K, const int32_t *offsets, const T *H, const T *dYrows,
                      const int32_t *dyperm, const T *xrows, const int32_t *xperm, const T *dA, const T *dB, float *dWg,
                      float *dWu, float *dWd, int accumulate, hipStream_t s) {
    const bool vec = d % 4 == 0 && F % 4 == 0;
    // (gathered rows by 32-bit offsets: a token matrix below 2 GB)
    if constexpr (sizeof(T) == 4)
        if (vec && ((!dyperm && !xperm) || (int64_t)Tn * d * 4 < (1ll << 31) - 16))
            return f32_wgrads(d, E, F, Tn, K, offsets, H, dYrows, dyperm, xrows, xperm, dA, dB, dWg, dWu, dWd, accumulate, s);
    PlainWgrad3<T> all = {{{H, dYrows, nullptr, dyperm, dWd, F, d, 0},
                           {xrows, dA, xperm, nullptr, dWg, d, F, 0},
                           {xrows, dB, xperm, nullptr, dWu, d, F, 0}}};
    const bool big = 3 * (int64_t)E * ceil_div(d, 128) * ceil_div(F, 128) >= kFill;
    if (vec && big) wgrad_launch<PlainBig, T, true>(E, K, offsets, all, accumulate, s);
    else if (vec) wgrad_launch<PlainSmall, T, true>(E, K, offsets, all, accumulate, s);
    else wgrad_launch<PlainSmall, T, false>(E, K, offsets, all, accumulate, s);
    return hipGetLastError();
}

template <typename T, typename IdxT>
void dwr_any(int Tn, int d, int E, int K, const T *x, const float *dz, const IdxT *idx, int64_t stride, float *part,
             hipStream_t s) {
    typedef PlainSmall C;
    const PlainDwr<T, IdxT> a = {Tn, d, E, K, plain_dwr_rows(Tn, d, E), x, dz, idx, stride, part};
    auto k = d % 4 == 0 ? plain_dwr_kernel<C, T, true, IdxT> : plain_dwr_kernel<C, T, false, IdxT>;
    allow_lds(k, C::LDS);
    k<<<plain_dwr_blocks(Tn, d, E), C::NT, C::LDS, s>>>(a);
}

template <typename T>
hipError_t logits_any(int Tn, int d, int E, const T *x, const T *Wr, const float *bias, float *logits, hipStream_t s) {
    typedef PlainSmall C;
    const unsigned grid = (unsigned)(ceil_div(Tn, C::BQ) * ceil_div(E, C::BP));
    const bool vx = d % 4 == 0, ve = E % 4 == 0;
#define R3_LOGITS(VX, VE)                                                                             \
    do {                                                                                              \
        allow_lds(plain_logits_kernel<C, T, VX, VE>, C::LDS);                                         \
        plain_logits_kernel<C, T, VX, VE><<<grid, C::NT, C::LDS, s>>>(Tn, d, E, x, Wr, bias, logits); \
    } while (0)
    if (vx && ve) R3_LOGITS(true, true);
    else if (vx) R3_LOGITS(true, false);
    else if (ve) R3_LOGITS(false, true);
    else R3_LOGITS(false, false);
#undef R3_LOGITS
    return hipGetLastError();
}

}  // namespace

hipError_t plain_router_logits(int T, int d, int E, int act, const void *x, const void *Wr, const float *bias, float *logits,
                               hipStream_t s) {
    ProfScope ps(PROF_LOGITS, s);
    return act == R3_BF16 ? logits_any(T, d, E, (const bf16_t *)x, (const bf16_t *)Wr, bias, logits, s)
                          : logits_any(T, d, E, (const float *)x, (const float *)Wr, bias, logits, s);
}

hipError_t plain_ffn2(int S, int d, int E, int F, int act, const void *H, const int32_t *offsets, const void *Wd, void *Yp,
                      hipStream_t s) {
    ProfScope ps(PROF_FFN2, s);
    return rows_by_act<PLAIN_DOWN>(act, S, d, E, F, offsets, H, nullptr, 0, nullptr, 1, nullptr, Wd, nullptr, nullptr, nullptr, Yp,
                                   nullptr, nullptr, s);
}

hipError_t plain_ffn1(int S, int d, int E, int F, int act, const void *rows, int T, const int32_t *perm, int K,
                      const int32_t *offsets, const void *Wg, const void *Wu, void *H, void *FA, void *FB, const float *gates,
                      hipStream_t s) {
    ProfScope ps(PROF_FFN1, s);
    return rows_by_act<PLAIN_FFN1>(act, S, d, E, F, offsets, rows, nullptr, T, perm, K, gates, Wg, Wu, nullptr, nullptr, H, FA, FB,
                                   s);
}

hipError_t plain_dh(int S, int d, int E, int F, int act, const void *dYp, const int32_t *offsets, const void *Wd,
                    const void *FA, const void *FB, void *dA, void *dB, hipStream_t s) {
    ProfScope ps(PROF_DH, s);
    return rows_by_act<PLAIN_DH>(act, S, d, E, F, offsets, dYp, nullptr, 0, nullptr, 1, nullptr, Wd, nullptr, FA, FB, dA, dB,
                                 nullptr, s);
}

hipError_t plain_dxp(int S, int d, int E, int F, int act, const void *dA, const void *dB, const int32_t *offsets,
                     const void *Wg, const void *Wu, void *dXp, hipStream_t s) {
    ProfScope ps(PROF_DXP, s);
    return rows_by_act<PLAIN_DXP>(act, S, d, E, F, offsets, dA, dB, 0, nullptr, 1, nullptr, Wg, Wu, nullptr, nullptr, dXp, nullptr,
                                  nullptr, s);
}

hipError_t plain_wgrads(int d, int E, int F, int T, int K, int act, const int32_t *offsets, const void *H, const void *dYrows,
                        const int32_t *dyperm, const void *xrows, const int32_t *xperm, const void *dA, const void *dB,
                        float *dWg, float *dWu, float *dWd, int accumulate, hipStream_t s) {
    ProfScope ps(PROF_WGRAD, s);
    return act == R3_BF16
               ? wgrads_any<bf16_t>(d, E, F, T, K, offsets, (const bf16_t *)H, (const bf16_t *)dYrows, dyperm, (const bf16_t *)xrows,
                                    xperm, (const bf16_t *)dA, (const bf16_t *)dB, dWg, dWu, dWd, accumulate, s)
               : wgrads_any<float>(d, E, F, T, K, offsets, (const float *)H, (const float *)dYrows, dyperm, (const float *)xrows,
                                   xperm, (const float *)dA, (const float *)dB, dWg, dWu, dWd, accumulate, s);
}

// tokens per part of dW_r: enough parts to give every compute unit a tile, at least 64 tokens each
int plain_dwr_rows(int T, int d, int E) {
    const int64_t tiles = ceil_div(d, 64) * ceil_div(E, 64);
    const int64_t ns = std::max<int64_t>(1, std::min<int64_t>(ceil_div(T, 64), ceil_div(256, tiles)));
    return (int)(ceil_div(ceil_div(T, ns), 32) * 32);
}

unsigned plain_dwr_blocks(int T, int d, int E) {
    return (unsigned)(ceil_div(T, plain_dwr_rows(T, d, E)) * ceil_div(d, PlainSmall::BQ) * ceil_div(E, PlainSmall::BP));
}

void plain_dwr_parts(int T, int d, int E, int K, int act, const void *x, const float *dz, const void *idx, int idx_dtype,
                     int64_t stride, float *part, hipStream_t s) {
    if (idx_dtype == R3_IDX_U8) {
        if (act == R3_BF16) dwr_any(T, d, E, K, (const bf16_t *)x, dz, (const uint8_t *)idx, stride, part, s);
        else dwr_any(T, d, E, K, (const float *)x, dz, (const uint8_t *)idx, stride, part, s);
    } else {
        if (act == R3_BF16) dwr_any(T, d, E, K, (const bf16_t *)x, dz, (const uint16_t *)idx, stride, part, s);
        else dwr_any(T, d, E, K, (const float *)x, dz, (const uint16_t *)idx, stride, part, s);
    }
}

}  // namespace r3
