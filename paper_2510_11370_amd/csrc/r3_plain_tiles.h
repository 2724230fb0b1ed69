// The tiles of r3_plain.hip: operands through registers into a double-buffered LDS tile, any widths, f32 matrix instruction.
#pragma once
#include "r3_common.h"

namespace r3 {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

template <int BP_, int BQ_>
struct PlainCfg {
    static constexpr int BP = BP_, BQ = BQ_, BK = 32, NT = 256;
    static constexpr int WTP = BP / 2, WTQ = BQ / 2, TP = WTP / 16, TQ = WTQ / 16;   // 2 x 2 waves
    static constexpr int KP = BK + 4;                 // floats per row of a row-major tile (reads spread over the banks)
    static constexpr int PBYTES = (BP * KP > BK * (BP + 4) ? BP * KP : BK * (BP + 4)) * 4;
    static constexpr int QBYTES = (BQ * KP > BK * (BQ + 4) ? BQ * KP : BK * (BQ + 4)) * 4;
    static constexpr int STAGE = PBYTES + QBYTES;
    static constexpr int LDS = 2 * STAGE;
};
typedef PlainCfg<128, 128> PlainBig;
typedef PlainCfg<64, 64> PlainSmall;

// four consecutive elements as floats; elements at or past `n` (counted from p) read as zero.  VEC: p is
// aligned to four elements and n is a multiple of four or <= 0
template <typename T, bool VEC>
__device__ __forceinline__ float4 load4(const T *p, int n) {
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if constexpr (VEC) {
        if (n > 0) {
            if constexpr (sizeof(T) == 4) {
                v = *(const float4 *)p;
            } else {
                const uint2 u = *(const uint2 *)p;
                v = make_float4(__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
                                __uint_as_float(u.y & 0xffff0000u));
            }
        }
    } else {
        if (n > 0) v.x = Elem<T>::ld(p);
        if (n > 1) v.y = Elem<T>::ld(p + 1);
        if (n > 2) v.z = Elem<T>::ld(p + 2);
        if (n > 3) v.w = Elem<T>::ld(p + 3);
    }
    return v;
}
template <typename T, bool VEC>
__device__ __forceinline__ void store4(T *p, const float (&v)[4], int n) {
    if constexpr (VEC) {
        if (n > 0) {
            if constexpr (sizeof(T) == 4) *(float4 *)p = make_float4(v[0], v[1], v[2], v[3]);
            else *(uint2 *)p = make_uint2(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]));
        }
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i)
            if (i < n) Elem<T>::st(p + i, v[i]);
    }
}

template <class C> using PlainAcc = f32x4_t[C::TP][C::TQ];

// D[p][q] = sum_k P[p][k] Q[q][k] over k in [0, nk * BK).  A k-major operand's loader is called as
// f(i, k, column), a row-major one's as f(i, row, k), for the thread's i-th piece of the tile (i is a constant
// after unrolling); both return four consecutive values (zero outside the matrix).  pre(kt) runs one k-tile before tile kt is loaded (index fetches).
template <class C, bool PTR, bool QTR, class FP, class FQ, class Pre>
__device__ __forceinline__ void plain_mainloop(PlainAcc<C> &acc, int nk, FP fp, FQ fq, Pre pre, char *lds) {
    constexpr int NP = C::BP * C::BK / 4 / C::NT, NQ = C::BQ * C::BK / 4 / C::NT;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wp = wave & 1, wq = wave >> 1;
    float4 rp[NP], rq[NQ];
    auto gload = [&](int kt) {
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int id = tid + i * C::NT;
            if constexpr (PTR) rp[i] = fp(i, kt * C::BK + id / (C::BP / 4), id % (C::BP / 4) * 4);
            else rp[i] = fp(i, id / (C::BK / 4), kt * C::BK + id % (C::BK / 4) * 4);
        }
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int id = tid + i * C::NT;
            if constexpr (QTR) rq[i] = fq(i, kt * C::BK + id / (C::BQ / 4), id % (C::BQ / 4) * 4);
            else rq[i] = fq(i, id / (C::BK / 4), kt * C::BK + id % (C::BK / 4) * 4);
        }
    };
    auto lstore = [&](int stage) {
        float *pb = (float *)(lds + stage * C::STAGE), *qb = (float *)(lds + stage * C::STAGE + C::PBYTES);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const int id = tid + i * C::NT;
            if constexpr (PTR) *(float4 *)(pb + id / (C::BP / 4) * (C::BP + 4) + id % (C::BP / 4) * 4) = rp[i];
            else *(float4 *)(pb + id / (C::BK / 4) * C::KP + id % (C::BK / 4) * 4) = rp[i];
        }
#pragma unroll
        for (int i = 0; i < NQ; ++i) {
            const int id = tid + i * C::NT;
            if constexpr (QTR) *(float4 *)(qb + id / (C::BQ / 4) * (C::BQ + 4) + id % (C::BQ / 4) * 4) = rq[i];
            else *(float4 *)(qb + id / (C::BK / 4) * C::KP + id % (C::BK / 4) * 4) = rq[i];
        }
    };
    // a lane's four k of a 16-k group are 4 (lane / 16) .. + 3, for both operands alike (the order of the
    // sum over k is free): 16 contiguous bytes of a row-major tile
    const int r16 = lane & 15, k4 = 4 * (lane >> 4);
    auto frag = [&](const float *b, bool tr, int pitch, int row, int k, float (&f)[4]) {
        if (tr) {
#pragma unroll
            for (int i = 0; i < 4; ++i) f[i] = b[(k + i) * pitch + row];
        } else {
            const float4 v = *(const float4 *)(b + row * pitch + k);
            f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
        }
    };
    if (nk <= 0) return;
    pre(0);
    gload(0);
    pre(1);
    lstore(0);
    __syncthreads();
    for (int kt = 0; kt < nk; ++kt) {
        const bool more = kt + 1 < nk;
        if (more) {
            gload(kt + 1);
            pre(kt + 2);
        }
        const float *pb = (const float *)(lds + (kt & 1) * C::STAGE);
        const float *qb = (const float *)(lds + (kt & 1) * C::STAGE + C::PBYTES);
#pragma unroll
        for (int g = 0; g < C::BK / 16; ++g) {
            float a[C::TP][4], b[C::TQ][4];
#pragma unroll
            for (int i = 0; i < C::TP; ++i)
                frag(pb, PTR, PTR ? C::BP + 4 : C::KP, wp * C::WTP + 16 * i + r16, 16 * g + k4, a[i]);
#pragma unroll
            for (int j = 0; j < C::TQ; ++j)
                frag(qb, QTR, QTR ? C::BQ + 4 : C::KP, wq * C::WTQ + 16 * j + r16, 16 * g + k4, b[j]);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < C::TP; ++i)
#pragma unroll
                    for (int j = 0; j < C::TQ; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
        }
        if (more) lstore((kt + 1) & 1);
        __syncthreads();
    }
}

template <class C>
__device__ __forceinline__ void plain_zero(PlainAcc<C> &acc) {
#pragma unroll
    for (int i = 0; i < C::TP; ++i)
#pragma unroll
        for (int j = 0; j < C::TQ; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
}
// the lane's results: f(tp, tq, p, q), acc[tp][tq][0..3] = D[p .. p + 3][q] (tile-local)
template <class C, class F>
__device__ __forceinline__ void plain_results(F f) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int tq = 0; tq < C::TQ; ++tq)
#pragma unroll
        for (int tp = 0; tp < C::TP; ++tp)
            f(tp, tq, (wave & 1) * C::WTP + 16 * tp + 4 * (lane >> 4), (wave >> 1) * C::WTQ + 16 * tq + (lane & 15));
}

// Parts of dW_r[c][e] = sum_t x[t][c] ds[t][e] over `rows` tokens each, ds[t][idx[t][j]] = dz[t][j] looked up as the tile is
// loaded.  One tile; `block` as the grid of plain_dwr_blocks() counts them.
template <typename T, typename IdxT>
struct PlainDwr {
    int Tn, d, E, K, rows;
    const T *x;
    const float *dz;
    const IdxT *idx;
    int64_t stride;
    float *part;
};
template <class C, typename T, bool VECX, typename IdxT>
__device__ __forceinline__ void plain_dwr_tile(const PlainDwr<T, IdxT> &g, int block, char *lds) {
    const int Tn = g.Tn, d = g.d, E = g.E, K = g.K, rows = g.rows;
    const T *__restrict__ x = g.x;
    const float *__restrict__ dz = g.dz;
    const IdxT *__restrict__ idx = g.idx;
    const int64_t stride = g.stride;
    const int npt = (E + C::BP - 1) / C::BP, nqt = (d + C::BQ - 1) / C::BQ;
    const int sp = block / (npt * nqt), rem = block - sp * npt * nqt;
    const int qt = rem / npt, q0 = qt * C::BQ, p0 = (rem - qt * npt) * C::BP;
    const int t0 = sp * rows, n = min(rows, Tn - t0);
    auto fp = [&](int, int k, int c) {
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if (k < n)
            for (int j = 0; j < K; ++j) {
                const int e = min((int)idx[(int64_t)(t0 + k) * stride + j], E - 1) - p0 - c;
                const float z = dz[(int64_t)(t0 + k) * K + j];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    if (e == i) v[i] = z;
            }
        return make_float4(v[0], v[1], v[2], v[3]);
    };
    auto fq = [&](int, int k, int c) { return load4<T, VECX>(x + (int64_t)(t0 + min(k, n - 1)) * d + q0 + c, k < n ? d - q0 - c : 0); };
    PlainAcc<C> acc;
    plain_zero<C>(acc);
    plain_mainloop<C, true, true>(acc, (n + C::BK - 1) / C::BK, fp, fq, [](int) {}, lds);
    float *o = g.part + (int64_t)sp * d * E;
    plain_results<C>([&](int tp, int tq, int p, int q) {
        if (q0 + q >= d || p0 + p >= E) return;
        float v[4] = {acc[tp][tq][0], acc[tp][tq][1], acc[tp][tq][2], acc[tp][tq][3]};
        store4<float, false>(o + (int64_t)(q0 + q) * E + p0 + p, v, E - p0 - p);
    });
}

}  // namespace r3
