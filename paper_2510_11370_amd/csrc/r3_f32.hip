// The expert network of the f32 layer on the f32 matrix instruction (16x16x4), for widths that are multiples of four
// (16-byte rows); all other widths and the bf16 layers without a matrix path have the tiles of r3_plain.hip.  Products and
// sums are those of an f32 FMA chain, in the same order of k as there.  SwiGLU, down projection and dXp of wide layers, and weight gradients that
// fill larger tiles, go to the bf16 instruction at f32 precision instead (r3_f32_split.h; the rules are at split_rows() below).
//
// What bounds it: the f32 matrix pipe, 256 FLOP per cycle and compute unit (157 TFLOP/s at 2.4 GHz); for layers of a few
// hundred rows the chain of loads and MFMAs of one tile.  An operand tile (32 k) goes from memory straight to LDS, 1 KB per
// wave and load, into the place its lane belongs to: the XOR swizzle that keeps the fragment reads free of bank conflicts is
// applied to the source address, and the buffer's bounds and an offset outside it give the zeros of ragged edges.  No
// operand passes the registers, so several small work-groups share a compute unit and cover each other's waits, which is
// why the tiles are small: 64 x 64 keeps both the row padding and the last round of tiles short.
#include <algorithm>
#include <type_traits>

#include "r3_f32.h"
#include "r3_f32_split.h"
#include "r3_finish.h"
#include "r3_kernels.h"
#include "r3_mfma2.h"
#include "r3_plain_tiles.h"

namespace r3 {
namespace {

// 4 waves as 2 (P) x 2 (Q), each TP x TQ tiles of 16 x 16; NST tiles of 32 k in LDS, NST - 1 on the way
template <int TP_, int TQ_, int NST_>
struct F32Cfg {
    static constexpr bool SPLIT = false;
    static constexpr int TP = TP_, TQ = TQ_, NST = NST_, NT = 256, BK = 32, MINW = 1;
    static constexpr int BP = 32 * TP, BQ = 32 * TQ, PBYTES = BP * BK * 4, STAGE = (BP + BQ) * BK * 4, LDS = NST * STAGE;
    static constexpr int LOADS = TP + TQ;   // loads per wave and k-tile (a load of four waves is 4 KB)
};
typedef F32Cfg<2, 2, 2> F32Tile;     // 32 KB of LDS: five work-groups on a compute unit, which cover what is not prefetched (four where the
                                     // weight gradients share their grid with the parts of dW_r, whose padded tiles take 36 KB)
typedef F32Cfg<1, 1, 4> F32Short;    // few tiles: four times as many, half the chain each, loads three k-tiles ahead (F32WgradOp: one)
typedef F32Cfg<2, 1, 4> F32Short1;   // the same for the SwiGLU, whose P tile holds both weights

// the same on the bf16 instruction (r3_f32_split.h); the last for the SwiGLU
typedef SplitCfg<4, 4, 1, 2> Split128;
typedef SplitCfg<2, 2, 2, 1> Split64;
typedef SplitCfg<1, 1, 2, 1> Split32;
typedef SplitCfg<2, 1, 2, 1> Split32x1;

template <class C> using F32Acc = f32x4_t[C::TP][C::TQ];

// Row-major operand tile [R rows][32 k]: a row is 128 B, its 16-byte chunk c sits at c ^ ((row >> 1) & 7).
template <int R>
struct F32Rows {
    Src src;
    int voff[R / 32], kc, KK, frag;
    // the row of the tile that this lane's i-th load belongs to
    static __device__ __forceinline__ int load_row(int i) { return 8 * ((int)(threadIdx.x >> 6) + 4 * i) + ((threadIdx.x & 63) >> 3); }
    __device__ __forceinline__ void init(const float *base, uint64_t bytes, int KK_, int wave_row) {
        const int lane = threadIdx.x & 63;
        src = Src{(const char *)base, bytes, 128};
        KK = KK_;
        kc = 4 * ((lane & 7) ^ ((load_row(0) >> 1) & 7));   // (32 rows on: the same swizzle)
        const int row = wave_row + (lane & 15);
        frag = row * 128 + (((lane >> 4) ^ ((row >> 1) & 7)) << 4);
    }
    __device__ __forceinline__ void set_row(int i, int row) { voff[i] = (row * KK + kc) * 4; }
    __device__ __forceinline__ void issue(int kt, uint32_t tile) const {
        const rsrc_t r = src_rsrc(src, kt);
        const bool in = kt * 32 + kc < KK;
#pragma unroll
        for (int i = 0; i < R / 32; ++i)
            lds_load16(r, tile + 1024 * ((threadIdx.x >> 6) + 4 * i), in ? voff[i] : kOutsideWindow);
    }
    // four consecutive k of row `wave_row + 16 t + lane % 16`, 16-k group g: k = 16 g + 4 (lane / 16) ..
    __device__ __forceinline__ void read(const char *tile, int t, int g, float (&f)[4]) const {
        const float4 v = *(const float4 *)(tile + (frag ^ (g << 6)) + t * 2048);
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
};

// k-major operand tile [32 k][R features], R = 64 or 32.  Its blocks of 16 features are spread so that the four k of a
// fragment read (4 apart) meet different banks: R = 64, block b of k at b ^ ((k >> 2) & 3); R = 32, two k-rows to the 256
// bytes of all banks, b ^ ((k >> 2) & 1) with k in row k ^ ((k >> 3) & 1).
template <int R>
struct F32Cols {
    static constexpr int ROWB = R * 4, KPL = 1024 / ROWB;   // bytes of a k-row; k-rows per load
    Src src;
    int koff[R / 32], coff, fr[R == 64 ? 1 : 2];
    // the k-row of the tile that this lane's i-th load belongs to
    static __device__ __forceinline__ int load_k(int i) {
        const int j = (threadIdx.x >> 6) + 4 * i, lane = threadIdx.x & 63;
        const int row = KPL * j + lane / (R / 4);
        return R == 64 ? row : row ^ (j & 1);
    }
    // base: first k-row, first feature; ld: floats per k-row; wave_block: the wave's first block of 16 features
    __device__ __forceinline__ void init(const float *base, uint64_t bytes, int ld, int wave_block) {
        const int lane = threadIdx.x & 63, hi = lane >> 4;
        src = Src{(const char *)base, bytes, (uint32_t)(32 * ld * 4)};
        const int slot = lane % (R / 4);
        coff = (R == 64 ? slot ^ (((threadIdx.x >> 6) & 3) << 2) : slot ^ (((lane >> 5) & 1) << 2)) * 16;
#pragma unroll
        for (int i = 0; i < R / 32; ++i) koff[i] = load_k(i) * ld * 4;
        if constexpr (R == 64) {
            fr[0] = 4 * hi * ROWB + ((wave_block ^ hi) << 6) + (lane & 15) * 4;
        } else {   // k = 4 hi + s sits in row 4 hi + (s ^ (hi >> 1))
            const int b = 4 * hi * ROWB + ((wave_block ^ (hi & 1)) << 6) + (lane & 15) * 4;
            fr[0] = b + (hi >> 1) * ROWB;
            fr[1] = b + (1 - (hi >> 1)) * ROWB;
        }
    }
    __device__ __forceinline__ void issue(int kt, uint32_t tile) const {
        const rsrc_t r = src_rsrc(src, kt);
#pragma unroll
        for (int i = 0; i < R / 32; ++i) lds_load16(r, tile + 1024 * ((threadIdx.x >> 6) + 4 * i), koff[i] + coff);
    }
    // one load of k-rows gathered from the whole matrix (src.step = 0): byte offset of this lane's row, < 0: none
    __device__ __forceinline__ void issue_row(int i, uint32_t tile, int row_off) const {
        lds_load16(src_rsrc(src, 0), tile + 1024 * ((threadIdx.x >> 6) + 4 * i), row_off < 0 ? kOutsideWindow : row_off + coff);
    }
    // four consecutive k (as F32Rows::read) of the wave's features 16 t + lane % 16
    __device__ __forceinline__ void read(const char *tile, int t, int g, float (&f)[4]) const {
#pragma unroll
        for (int s = 0; s < 4; ++s)
            f[s] = *(const float *)(tile + ((R == 64 ? fr[0] + s * ROWB : fr[s & 1] + (s & 2) * ROWB) ^ (t << 6)) + g * 16 * ROWB);
    }
};

// the wave's loads of all but `stages` k-tiles have landed, its LDS reads are done; then the waves meet
template <class C, int STAGES>
__device__ __forceinline__ void f32_wait() {
    constexpr int vm = STAGES * C::LOADS;
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(vm) : "memory");
}

template <class C>
__device__ __forceinline__ void f32_mul(F32Acc<C> &acc, const float (&a)[C::TP][4], const float (&b)[C::TQ][4]) {
#pragma unroll
    for (int s = 0; s < 4; ++s)
#pragma unroll
        for (int i = 0; i < C::TP; ++i)
#pragma unroll
            for (int j = 0; j < C::TQ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
}

// acc[p][q] += sum_k P[p][k] Q[q][k] over nk tiles of 32 k.  issue(kt, LDS address): the wave's C::LOADS loads of k-tile kt
// (zeros past the end).  rp(i, g, f, tile) / rq: fragment reads.  A k-tile is two groups of 16 k; a group is read while the
// one before it is multiplied, so that a k-tile opens with MFMAs that wait for nothing of it.
template <class C, class Issue, class RP, class RQ>
__device__ __forceinline__ void f32_loop(F32Acc<C> &acc, int nk, Issue issue, RP rp, RQ rq, char *lds) {
    const uint32_t at = lds_addr(lds);
    float a[2][C::TP][4], b[2][C::TQ][4];
    auto read = [&](const char *st, int g) {
#pragma unroll
        for (int i = 0; i < C::TP; ++i) rp(st, i, g, a[g][i]);
#pragma unroll
        for (int j = 0; j < C::TQ; ++j) rq(st + C::PBYTES, j, g, b[g][j]);
    };
#pragma unroll
    for (int p = 0; p < C::NST - 1; ++p) issue(p, at + p * C::STAGE);
    f32_wait<C, C::NST - 2>();
    int slot = 0;
    for (int kt = 0; kt < nk; ++kt) {
        const char *st = lds + slot * C::STAGE;
        const int prev = slot == 0 ? C::NST - 1 : slot - 1;
        issue(kt + C::NST - 1, at + prev * C::STAGE);   // into the tile that was left last
        read(st, 0);
        if (kt) f32_mul<C>(acc, a[1], b[1]);
        __builtin_amdgcn_sched_barrier(0);
        read(st, 1);
        f32_mul<C>(acc, a[0], b[0]);
        f32_wait<C, C::NST - 2>();
        slot = slot + 1 == C::NST ? 0 : slot + 1;
    }
    if (nk > 0) f32_mul<C>(acc, a[1], b[1]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the loads past the end, before the space is used again or left
}

template <class C>
__device__ __forceinline__ void f32_zero(F32Acc<C> &acc) {
#pragma unroll
    for (int i = 0; i < C::TP; ++i)
#pragma unroll
        for (int j = 0; j < C::TQ; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
}

// ---------------------------------------------------------------------------
// Row-tiled contractions over the expert-sorted rows (the operands of plain_rows_kernel).
// ---------------------------------------------------------------------------
struct F32RowArgs {
    int d, E, F;
    const int32_t *offsets;
    const float *in0, *in1;
    int T;
    const int32_t *perm;
    int K;
    const float *gates, *W0, *W1, *FA, *FB;
    float *out0, *out1, *out2;
};

// four consecutive features of a row of the result (SwiGLU: v of the gate's weight, w of the other's; gate: of the row's slot, or 1)
template <int MODE>
__device__ __forceinline__ void f32_rows_store(const float *__restrict__ FA, const float *__restrict__ FB, float *__restrict__ out0,
                                               float *__restrict__ out1, float *__restrict__ out2, int64_t o, float gate, float4 v, float4 w) {
    if constexpr (MODE == PLAIN_FFN1) {
        const float va[4] = {v.x, v.y, v.z, v.w}, vb[4] = {w.x, w.y, w.z, w.w};
        float h[4], fa[4], fb[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float a = va[i], b = vb[i];
            const float sg = sigmoidf_(a);
            h[i] = gate * (a * sg * b);
            fa[i] = b * sg * (1.0f + a * (1.0f - sg));
            fb[i] = a * sg;
        }
        *(float4 *)(out0 + o) = make_float4(h[0], h[1], h[2], h[3]);
        if (out1) *(float4 *)(out1 + o) = make_float4(fa[0], fa[1], fa[2], fa[3]);
        if (out2) *(float4 *)(out2 + o) = make_float4(fb[0], fb[1], fb[2], fb[3]);
    } else if constexpr (MODE == PLAIN_DH) {
        const float4 a = *(const float4 *)(FA + o), b = *(const float4 *)(FB + o);
        v = make_float4(gate * v.x, gate * v.y, gate * v.z, gate * v.w);
        *(float4 *)(out0 + o) = make_float4(v.x * a.x, v.y * a.y, v.z * a.z, v.w * a.w);
        *(float4 *)(out1 + o) = make_float4(v.x * b.x, v.y * b.y, v.z * b.z, v.w * b.w);
    } else {
        *(float4 *)(out0 + o) = v;
    }
}

// one tile; `block` of f32_rows_grid()
template <class C, int MODE>
__device__ __forceinline__ void f32_rows_tile(const F32RowArgs &g, int block, char *lds) {
    const int d = g.d, E = g.E, F = g.F, T = g.T, K = g.K;
    const int32_t *__restrict__ offsets = g.offsets, *__restrict__ perm = g.perm;
    const float *__restrict__ in0 = g.in0, *__restrict__ in1 = g.in1, *__restrict__ gates = g.gates, *__restrict__ W0 = g.W0,
                *__restrict__ W1 = g.W1, *__restrict__ FAin = g.FA, *__restrict__ FBin = g.FB;
    float *__restrict__ out0 = g.out0, *__restrict__ out1 = g.out1, *__restrict__ out2 = g.out2;
    static_assert(MODE != PLAIN_FFN1 || C::TP == 2, "one tile of each weight");
    constexpr int BF = MODE == PLAIN_FFN1 ? C::BP / 2 : C::BP;            // output features per tile
    const int NOUT = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) ? F : d;
    const int KK = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) ? d : F;      // width of the row operand
    const int npt = (NOUT + BF - 1) / BF;
    const RowTile t = find_row_tile<true>(offsets, E, C::BQ, block, npt);
    if (t.e < 0) return;
    const int p0 = t.col * BF, rows = t.row1 - t.row0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wp = wave & 1, wq = wave >> 1;
    const uint64_t wbytes = (uint64_t)d * F * 4;
    const float *w0 = W0 + (int64_t)t.e * d * F;

    const bool gather = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) && perm;
    F32Rows<C::BQ> Q;
    Q.init(gather ? in0 : in0 + (int64_t)t.row0 * KK, gather ? (uint64_t)T * KK * 4 : (uint64_t)rows * KK * 4, KK, wq * 16 * C::TQ);
#pragma unroll
    for (int i = 0; i < C::BQ / 32; ++i) {
        const int r = min(Q.load_row(i), rows - 1);
        Q.set_row(i, gather ? perm[t.row0 + r] / K : r);
    }
    F32Acc<C> acc;
    f32_zero<C>(acc);
    const int nk = (KK + C::BK - 1) / C::BK;
    auto rq = [&](const char *tile, int j, int g, float (&f)[4]) { Q.read(tile, j, g, f); };
    if constexpr (MODE == PLAIN_FFN1) {
        const float *w1 = W1 + (int64_t)t.e * d * F;
        F32Cols<32> G, U;   // the same 32 features of both weights, so that a lane holds both pre-activations
        G.init(w0 + p0, wbytes - p0 * 4u, F, wp);
        U.init(w1 + p0, wbytes - p0 * 4u, F, wp);
        f32_loop<C>(acc, nk, [&](int kt, uint32_t a) { G.issue(kt, a); U.issue(kt, a + 4096); Q.issue(kt, a + C::PBYTES); },
                    [&](const char *tile, int i, int g, float (&f)[4]) { G.read(tile + i * 4096, 0, g, f); }, rq, lds);
    } else if constexpr (MODE == PLAIN_DOWN) {
        F32Cols<C::BP> P;
        P.init(w0 + p0, wbytes - p0 * 4u, d, wp * C::TP);
        f32_loop<C>(acc, nk, [&](int kt, uint32_t a) { P.issue(kt, a); Q.issue(kt, a + C::PBYTES); },
                    [&](const char *tile, int i, int g, float (&f)[4]) { P.read(tile, i, g, f); }, rq, lds);
    } else {
        F32Rows<C::BP> P;
        const uint64_t pbytes = (uint64_t)(NOUT - p0) * KK * 4;
        P.init(w0 + (int64_t)p0 * KK, pbytes, KK, wp * 16 * C::TP);
#pragma unroll
        for (int i = 0; i < C::BP / 32; ++i) P.set_row(i, min(P.load_row(i), NOUT - p0 - 1));
        auto rp = [&](const char *tile, int i, int g, float (&f)[4]) { P.read(tile, i, g, f); };
        if constexpr (MODE == PLAIN_DH) {
            f32_loop<C>(acc, nk, [&](int kt, uint32_t a) { P.issue(kt, a); Q.issue(kt, a + C::PBYTES); }, rp, rq, lds);
        } else {   // one reduction over both halves: dA Wg^T, then dB Wu^T
            const Src p1{(const char *)(W1 + (int64_t)t.e * d * F + (int64_t)p0 * KK), pbytes, 128};
            const Src q1{(const char *)(in1 + (int64_t)t.row0 * KK), Q.src.nbytes, 128};
            const Src p0s = P.src, q0s = Q.src;
            f32_loop<C>(acc, 2 * nk,
                        [&](int kt, uint32_t a) {
                            const bool second = kt >= nk;
                            P.src = second ? p1 : p0s;
                            Q.src = second ? q1 : q0s;
                            P.issue(second ? kt - nk : kt, a);
                            Q.issue(second ? kt - nk : kt, a + C::PBYTES);
                        },
                        rp, rq, lds);
        }
    }
    // a lane's results: four consecutive features of one row per 16 x 16 tile
#pragma unroll
    for (int tq = 0; tq < C::TQ; ++tq) {
        const int q = wq * 16 * C::TQ + 16 * tq + (lane & 15);
        if (q >= rows) continue;
        const int row = t.row0 + q;
        const f32x4_t *v = &acc[0][tq];
        const float gate = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) && gates ? gates[perm[row]] : 1.0f;
        if constexpr (MODE == PLAIN_FFN1) {
            const int f = p0 + 16 * wp + 4 * (lane >> 4);
            if (f >= F) continue;
            const f32x4_t b = acc[1][tq];
            f32_rows_store<MODE>(FAin, FBin, out0, out1, out2, (int64_t)row * NOUT + f, gate, make_float4((*v)[0], (*v)[1], (*v)[2], (*v)[3]),
                                 make_float4(b[0], b[1], b[2], b[3]));
        } else {
#pragma unroll
            for (int tp = 0; tp < C::TP; ++tp) {
                const int c = p0 + wp * 16 * C::TP + 16 * tp + 4 * (lane >> 4);
                if (c >= NOUT) continue;
                const f32x4_t r = acc[tp][tq];
                f32_rows_store<MODE>(FAin, FBin, out0, out1, out2, (int64_t)row * NOUT + c, gate, make_float4(r[0], r[1], r[2], r[3]), float4());
            }
        }
    }
}

// the same with a split tile (not dH)
template <class C, int MODE>
__device__ __forceinline__ void split_rows_tile(const F32RowArgs &g, int block, char *lds) {
    constexpr bool ONE = MODE == PLAIN_FFN1;
    constexpr int BP = C::BP, BQ = C::BQ, BF = ONE ? BP / 2 : BP;
    typedef SplitWave<C, ONE> W;
    const int NOUT = ONE ? g.F : g.d, KK = ONE ? g.d : g.F;
    const RowTile t = find_row_tile<true>(g.offsets, g.E, BQ, block, (NOUT + BF - 1) / BF);
    if (t.e < 0) return;
    const int p0 = t.col * BF, rows = t.row1 - t.row0, nk = (KK + 31) / 32;
    const int lane = threadIdx.x & 63, u = threadIdx.x & 127;
    const int64_t we = (int64_t)t.e * g.d * g.F;
    const uint64_t wbytes = (uint64_t)g.d * g.F * 4;

    const bool gather = ONE && g.perm;
    SplitRows<BQ> Q;
    Q.init(gather ? g.in0 : g.in0 + (int64_t)t.row0 * KK, gather ? (uint64_t)g.T * KK * 4 : (uint64_t)rows * KK * 4, KK, u);
#pragma unroll
    for (int i = 0; i < Q.N; ++i) {
        const int r = min(Q.row(u, i), rows - 1);
        Q.set_row(i, gather ? g.perm[t.row0 + r] / g.K : r);
    }
    SplitAcc<C> acc;
    if constexpr (ONE) {   // the same features of both weights, so that a lane holds both pre-activations
        SplitCols<BP, true> P;
        P.init(((threadIdx.x >> 6) == 0 ? g.W0 : g.W1) + we + p0, wbytes - p0 * 4u, g.F, u);
        split_loop<C, W>(acc, nk, KK, P, Q, lds);
    } else if constexpr (MODE == PLAIN_DOWN) {
        SplitCols<BP, false> P;
        P.init(g.W0 + we + p0, wbytes - p0 * 4u, g.d, u);
        split_loop<C, W>(acc, nk, KK, P, Q, lds);
    } else {   // one reduction over both halves: dA Wg^T, then dB Wu^T
        static_assert(MODE == PLAIN_DXP, "");
        SplitRows<BP> P;
        const uint64_t pbytes = (uint64_t)(NOUT - p0) * KK * 4;
        P.init(g.W0 + we + (int64_t)p0 * KK, pbytes, KK, u);
#pragma unroll
        for (int i = 0; i < P.N; ++i) P.set_row(i, min(P.row(u, i), NOUT - p0 - 1));
        const SplitPair<SplitRows<BP>> P2{P, Src{(const char *)(g.W1 + we + (int64_t)p0 * KK), pbytes, 128}, nk};
        const SplitPair<SplitRows<BQ>> Q2{Q, Src{(const char *)(g.in1 + (int64_t)t.row0 * KK), Q.src.nbytes, 128}, nk};
        split_loop<C, W>(acc, 2 * nk, 2 * KK, P2, Q2, lds);
    }
#pragma unroll
    for (int j = 0; j < C::TQ; ++j) {
        const int q = W::qrow(j) + (lane & 15), row = t.row0 + q;
        if (q >= rows) continue;
        const float gate = ONE && g.gates ? g.gates[g.perm[row]] : 1.0f;
        auto quad = [&](int i) { return make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]); };
#pragma unroll
        for (int i = 0; i < (ONE ? C::TP / 2 : C::TP); ++i) {
            const int c = p0 + W::prow(i) + 4 * (lane >> 4);
            if (c >= NOUT) continue;
            f32_rows_store<MODE>(g.FA, g.FB, g.out0, g.out1, g.out2, (int64_t)row * NOUT + c, gate, quad(i), quad(ONE ? C::TP / 2 + i : i));
        }
    }
}

// ---------------------------------------------------------------------------
// The three weight gradients of every expert in one launch (as plain_wgrad_kernel).
// ---------------------------------------------------------------------------
// A k-major operand of which k-row r is row r0 + r of a matrix, or (GATHER) row perm[r0 + r] / K of it.  The entries of perm are fetched a
// k-tile before the loads that need them.  The compiler counts their loads but not the tiles', and waits for everything in flight
// before it uses an entry: so the gathered operand's loads go out first, when the tiles before have been waited for (with two tiles in LDS) or
// at most two are on the way (with four: one is left ahead), and a plain operand has no such registers.  With the choice made in the loop
// a tile's own loads were drained before the MFMAs: training, us, 2048 tokens top-4, 512 x 1024, 16 experts 763 | 748 now, 4096 top-2, 256 x 256, 8 experts,
// Zipf 274 | 217.  Entries by scalar loads, which have a counter of their own, take 8 selects a load: 217, and 8192 tokens, 128 x 256 189 | 203.
template <int R, bool GATHER>
struct F32WgradOp {
    F32Cols<R> op;
    const int32_t *perm;
    int n, ld, K, next[R / 32];
    __device__ __forceinline__ void init(const float *m, const int32_t *perm_, int64_t nrows, int r0, int n_, int ld_, int K_, int col0,
                                         int wave_block) {
        perm = GATHER ? perm_ + r0 : nullptr;
        n = n_; ld = ld_; K = K_;
        const int64_t first = GATHER ? 0 : (int64_t)r0 * ld;
        op.init(m + first + col0, (uint64_t)((GATHER ? nrows : n) * ld - col0) * 4, ld, wave_block);
        if constexpr (GATHER) {
            op.src.step = 0;
            fetch(0);
        }
    }
    __device__ __forceinline__ void fetch(int kt) {
#pragma unroll
        for (int i = 0; i < R / 32; ++i) next[i] = perm[min(kt * 32 + op.load_k(i), n - 1)];
    }
    __device__ __forceinline__ void issue(int kt, uint32_t tile) {
        if constexpr (!GATHER) {
            op.issue(kt, tile);
        } else {
            int off[R / 32];   // (every entry is used before the first load goes out)
#pragma unroll
            for (int i = 0; i < R / 32; ++i) off[i] = kt * 32 + op.load_k(i) < n ? next[i] / K * (ld * 4) : -1;
#pragma unroll
            for (int i = 0; i < R / 32; ++i) op.issue_row(i, tile, off[i]);
            fetch(kt + 1);
        }
    }
};

struct F32Wgrad {
    const float *Qs, *Ps;
    const int32_t *qperm, *pperm;
    float *out;
    int NQ, NP, tiles;   // tiles: per expert
};
struct F32Wgrad3 {
    F32Wgrad g[3];
};

template <class C>
__device__ __forceinline__ void f32_wgrad_tile(int E, int T, int K, const int32_t *__restrict__ offsets, const F32Wgrad3 &all,
                                               int accumulate, int block, char *lds) {
    const int per = all.g[0].tiles + all.g[1].tiles + all.g[2].tiles;
    const int e = block / per, t0 = all.g[0].tiles, t1 = t0 + all.g[1].tiles;
    int rem = block - e * per;
    const F32Wgrad g = rem < t0 ? all.g[0] : rem < t1 ? all.g[1] : all.g[2];
    rem -= rem < t0 ? 0 : rem < t1 ? t0 : t1;
    const int npt = (g.NP + C::BP - 1) / C::BP;
    const int qt = rem / npt, q0 = qt * C::BQ, p0 = (rem - qt * npt) * C::BP;
    const int r0 = offsets[e], n = offsets[e + 1] - r0;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, wp = wave & 1, wq = wave >> 1;
    F32Acc<C> acc;
    f32_zero<C>(acc);
    if (n > 0) {
        auto loop = [&](auto pg, auto qg) {
            F32WgradOp<C::BP, decltype(pg)::value> P;
            F32WgradOp<C::BQ, decltype(qg)::value> Q;
            P.init(g.Ps, g.pperm, T, r0, n, g.NP, K, p0, wp * C::TP);
            Q.init(g.Qs, g.qperm, T, r0, n, g.NQ, K, q0, wq * C::TQ);
            auto issue = [&](int kt, uint32_t a) {
                if constexpr (decltype(qg)::value) Q.issue(kt, a + C::PBYTES);
                P.issue(kt, a);
                if constexpr (!decltype(qg)::value) Q.issue(kt, a + C::PBYTES);
            };
            f32_loop<C>(acc, (n + C::BK - 1) / C::BK, issue, [&](const char *tile, int i, int gr, float (&f)[4]) { P.op.read(tile, i, gr, f); },
                        [&](const char *tile, int j, int gr, float (&f)[4]) { Q.op.read(tile, j, gr, f); }, lds);
        };
        if (g.pperm) loop(std::true_type{}, std::false_type{});        // dW_down from dy
        else if (g.qperm) loop(std::false_type{}, std::true_type{});   // dW_gate, dW_up from x
        else loop(std::false_type{}, std::false_type{});
    }
    float *o = g.out + (int64_t)e * g.NQ * g.NP;
#pragma unroll
    for (int tq = 0; tq < C::TQ; ++tq) {
        const int q = q0 + wq * 16 * C::TQ + 16 * tq + (lane & 15);
        if (q >= g.NQ) continue;
#pragma unroll
        for (int tp = 0; tp < C::TP; ++tp) {
            const int p = p0 + wp * 16 * C::TP + 16 * tp + 4 * (lane >> 4);
            if (p >= g.NP) continue;
            float4 *at = (float4 *)(o + (int64_t)q * g.NP + p);
            float4 v = make_float4(acc[tp][tq][0], acc[tp][tq][1], acc[tp][tq][2], acc[tp][tq][3]);
            if (accumulate) {
                const float4 old = *at;
                v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w;
            }
            *at = v;
        }
    }
}

template <class C>
__device__ __forceinline__ void split_wgrad_tile(int E, int T, int K, const int32_t *__restrict__ offsets, const F32Wgrad3 &all,
                                                 int accumulate, int block, char *lds) {
    typedef SplitWave<C, false> W;
    const int per = all.g[0].tiles + all.g[1].tiles + all.g[2].tiles;
    const int e = block / per, t0 = all.g[0].tiles, t1 = t0 + all.g[1].tiles;
    int rem = block - e * per;
    const F32Wgrad g = rem < t0 ? all.g[0] : rem < t1 ? all.g[1] : all.g[2];
    rem -= rem < t0 ? 0 : rem < t1 ? t0 : t1;
    const int npt = (g.NP + C::BP - 1) / C::BP;
    const int qt = rem / npt, q0 = qt * C::BQ, p0 = (rem - qt * npt) * C::BP;
    const int r0 = offsets[e], n = offsets[e + 1] - r0;
    const int lane = threadIdx.x & 63, u = threadIdx.x & 127;
    SplitAcc<C> acc;
    auto plain = [&](const float *m, int ld, int col0) {
        SplitCols<C::BP, false> op;
        op.init(m + (int64_t)r0 * ld + col0, (uint64_t)((int64_t)n * ld - col0) * 4, ld, u);
        return op;
    };
    auto gathered = [&](const float *m, int ld, int col0, const int32_t *perm) {
        SplitGather<C::BP> op;
        op.init(m + col0, (uint64_t)((int64_t)T * ld - col0) * 4, ld, u, perm + r0, n, K);
        return op;
    };
    static_assert(C::BP == C::BQ, "");
    const int nk = (n + 31) / 32;
    if (g.pperm) split_loop<C, W>(acc, nk, n, gathered(g.Ps, g.NP, p0, g.pperm), plain(g.Qs, g.NQ, q0), lds);
    else if (g.qperm) split_loop<C, W>(acc, nk, n, plain(g.Ps, g.NP, p0), gathered(g.Qs, g.NQ, q0, g.qperm), lds);
    else split_loop<C, W>(acc, nk, n, plain(g.Ps, g.NP, p0), plain(g.Qs, g.NQ, q0), lds);
    float *o = g.out + (int64_t)e * g.NQ * g.NP;
#pragma unroll
    for (int j = 0; j < C::TQ; ++j) {
        const int q = q0 + W::qrow(j) + (lane & 15);
        if (q >= g.NQ) continue;
#pragma unroll
        for (int i = 0; i < C::TP; ++i) {
            const int p = p0 + W::prow(i) + 4 * (lane >> 4);
            if (p >= g.NP) continue;
            float4 *at = (float4 *)(o + (int64_t)q * g.NP + p);
            float4 v = make_float4(acc[i][j][0], acc[i][j][1], acc[i][j][2], acc[i][j][3]);
            if (accumulate) {
                const float4 old = *at;
                v.x += old.x; v.y += old.y; v.z += old.z; v.w += old.w;
            }
            *at = v;
        }
    }
}

// either kind of tile
template <class C, int MODE>
__device__ __forceinline__ void rows_tile(const F32RowArgs &a, int block, char *lds) {
    if constexpr (C::SPLIT) split_rows_tile<C, MODE>(a, block, lds);
    else f32_rows_tile<C, MODE>(a, block, lds);
}
template <class C>
__device__ __forceinline__ void wgrad_tile(int E, int T, int K, const int32_t *__restrict__ offsets, const F32Wgrad3 &all, int accumulate,
                                           int block, char *lds) {
    if constexpr (C::SPLIT) split_wgrad_tile<C>(E, T, K, offsets, all, accumulate, block, lds);
    else f32_wgrad_tile<C>(E, T, K, offsets, all, accumulate, block, lds);
}

// ---------------------------------------------------------------------------
// Launches.  What does not wait for each other shares one: a layer of few tokens is a chain of launches, and a larger one
// fills one kernel's last round of tiles with the next one's.  After the one-call forward:  the gate's backward, W_r^T and dH, which reads dy's
// rows by itself and scales its results by the gates;  then the parts of dW_r, dXp and all weight gradients;  then the rest of the router beside
// dx.  T=256 d=128 E=8 K=2 F=256, kernels of a forward + backward: 58 us with a launch each, 50.7 in five launches of the backward (g dy written out
// for dH), 44.7 in these three; T=2048 d=512 E=16 K=4 F=1024: 815, 767 (595 with split tiles), 588.
// ---------------------------------------------------------------------------
template <class C, int MODE>
__global__ void __launch_bounds__(C::NT, C::MINW) f32_rows_kernel(F32RowArgs a) {
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS];
    rows_tile<C, MODE>(a, blockIdx.x, lds);
}

template <class C>
__global__ void __launch_bounds__(C::NT, C::MINW)
f32_wgrad_kernel(int E, int T, int K, const int32_t *__restrict__ offsets, F32Wgrad3 all, int accumulate) {
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS];
    wgrad_tile<C>(E, T, K, offsets, all, accumulate, blockIdx.x, lds);
}

constexpr int max_int(int a, int b) { return a > b ? a : b; }

// dz of the masked softmax from the gated rows that the forward left: w_j = <dy_t, Yp[row_j]> = g_j dg_j, dz_j = w_j - g_j sum_i w_i.
// A wave per token, four rows of Yp in flight.
struct F32Gate {
    int T, d, K;
    const float *dy, *Yp, *gates;
    const int32_t *inv_perm;
    float *dz, *dzrow;
};
__device__ __forceinline__ void f32_gate_tokens(const F32Gate &a, int block) {
    const int t = 4 * block + ((int)threadIdx.x >> 6), lane = threadIdx.x & 63, vecs = a.d / 4, K = a.K;
    if (t >= a.T) return;
    const int mine = lane < K ? a.inv_perm[(int64_t)t * K + lane] : 0;
    const float g = lane < K ? a.gates[(int64_t)t * K + lane] : 0.0f;
    const float4 *dy = (const float4 *)(a.dy + (int64_t)t * a.d);
    float w = 0.0f, mix = 0.0f;
    for (int j0 = 0; j0 < K; j0 += 4) {
        const float4 *y[4];
        float dot[4] = {};
#pragma unroll
        for (int u = 0; u < 4; ++u) y[u] = (const float4 *)(a.Yp + (int64_t)__shfl(mine, min(j0 + u, K - 1), 64) * a.d);
        for (int c = lane; c < vecs; c += 64) {
            const float4 b = dy[c];
            float4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) v[u] = y[u][c];
#pragma unroll
            for (int u = 0; u < 4; ++u) dot[u] = fmaf(b.x, v[u].x, fmaf(b.y, v[u].y, fmaf(b.z, v[u].z, fmaf(b.w, v[u].w, dot[u]))));
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const float sum = wave_sum(dot[u]);
            if (j0 + u < K) mix += sum;
            if (j0 + u == lane) w = sum;
        }
    }
    if (lane < K) {
        const float v = w - g * mix;
        a.dz[(int64_t)t * K + lane] = v;
        if (a.dzrow) a.dzrow[mine] = v;
    }
}

// [0, nt): W_r^T; [nt, ng): the gate's backward; from `first` on (a multiple of 8, so that the rows' tiles keep their XCDs) dH
template <class C>
__global__ void __launch_bounds__(C::NT, C::MINW)
f32_dh_kernel(F32RowArgs a, F32Gate gate, RouterFinish<float> wrt, int nt, int ng, int first) {
    __shared__ __attribute__((aligned(1024))) char lds[C::LDS];
    static_assert(sizeof(RouterFinishLds<float>) <= sizeof(lds), "");
    const int b = blockIdx.x;
    if (b >= first) rows_tile<C, PLAIN_DH>(a, b - first, lds);
    else if (b < nt) router_finish_block<C::NT>(wrt, b, *(RouterFinishLds<float> *)lds);
    else if (b < ng) f32_gate_tokens(gate, b - nt);
}

// [0, first): parts of dW_r; [first, second): dXp; then the weight gradients
template <class CR, class CW, typename IdxT>
__global__ void __launch_bounds__(CR::NT, max_int(CR::MINW, CW::MINW))
f32_grads_kernel(F32RowArgs a, int E, int T, int K, const int32_t *__restrict__ offsets, F32Wgrad3 all, int accumulate,
                 PlainDwr<float, IdxT> w, int nw, int first, int second) {
    __shared__ __attribute__((aligned(1024))) char lds[max_int(max_int(CR::LDS, CW::LDS), PlainSmall::LDS)];
    const int b = blockIdx.x;
    if (b >= second) wgrad_tile<CW>(E, T, K, offsets, all, accumulate, b - second, lds);
    else if (b >= first) rows_tile<CR, PLAIN_DXP>(a, b - first, lds);
    else if (b < nw) plain_dwr_tile<PlainSmall, float, true>(w, b, lds);
}

int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
// Tiles of 64 x 64 or of 32 x 32 outputs.  Row-tiled kernels: 32 x 32 below 512 tiles of the larger kind, and where an expert has
// fewer than 64 rows on average.  us, 64 x 64 | 32 x 32: dXp of 256 x 2 rows, 128 features out of 256 x 2 (16 tiles) 16.3 | 10.5;
// 2048 rows, 512 out of 512 x 2 (256) 43.0 | 38.9; 2048 rows, 1024 out of 1024 x 2 (512) 111.6 | 116.5; 8192 rows, 512 out of
// 1024 x 2 (1024) 190.7 | 211.2; 4096 rows over 128 experts, 512 out of 512 x 2 (512) 88.7 | 85.1; 256 over 128 82.1 | 64.0.
constexpr int kRowsFill = 512;
// The weight gradients, whose tiles each write 16 or 4 KB: 32 x 32 below 320 tiles of the larger kind.  Training, us, 64 x 64 | 32 x 32, 8 experts
// unless given: 8192 tokens top-2, 128 x 256 (192 tiles) 187.8 | 189.5; 4096 top-2, 192 x 192 (216)
// 137.4 | 125.0; 2048 top-2, 256 x 256, 5 experts (240) 118.7 | 108.4; 4096 top-1, 192 x 256 (288) 100.0 | 95.4; 3000 top-2, 320 x 320, 4 experts (300)
// 190.7 | 184.3; 4096 top-2, 256 x 256 (384) 161.3 | 166.2; 300 top-2, 512 x 320, 4 experts (480) 65.5 | 67.6.
constexpr int kWgradFill = 320;

// Split tiles.  SwiGLU, down projection and dXp: by the widths alone, so that a token's results are the same bits in a micro-batch and in
// the whole batch (dH stays on the f32 instruction: 16 k-tiles and two operands beside the result, 94 | 104 us).  From 512 x 512 on: training, us, f32
// instruction | split, 8 experts top-2 unless given, 128 tokens, 1024 and 4096:  256 x 256 44 | 47, 105 | 100 (2048), 264 | 261 (8192);  384 x 384 53 | 59,
// 107 | 104, 265 | 247;  512 x 512 62 | 68, 152 | 143, 378 | 349, of 4096 top-4 over 128 experts 877 | 781;  1024 x 1024 105 | 117 (64), 262 | 240 (512);
// 2048 top-4, 512 x 1024, 16 experts 663 | 565.  (Small tiles only where there were few of the large ones, as the f32 instruction has it, is 11 % faster at 128 tokens and
// up to 4 % at some thousand, and gives a token other bits there.)
constexpr int64_t kSplitRows = 1 << 18;
// Their size.  128 x 128 from 184 tiles on (dXp, beside the weight gradients: 128), with 64 rows per expert and a quarter of the columns dead at most;
// 64 x 64 from 512 (down 320, dXp 64).  us, 128 | 64 | 32, by the number of tiles of 128:  SwiGLU 64 34 | 25 | 24, 128 35 | 32 | 36, 176 67 | 55 | 71,
// 192 56 | 70 | 78, 376 51 | 64 | 73, 512 76 | 80 | 97, 32 rows per expert 107 | 92 | 93, 64 113 | 124 | 130;  down 64 32 | 22 | 21, 88 56 | 37 | 41,
// 128 33 | 29 | 33, 164 45 | 40 | 53, 188 33 | 38 | 42, 200 38 | 43 | 50, 256 47 | 44 | 56;  dXp and the gradients 32 57 | 34 | 40, 64 58 | 53 | 67, 88 136 | 118 | 163,
// 128 85 | 88 | 119, 256 252 | 291 | 415, 32 rows per expert 305 | 252 | 258.
int64_t split_columns(int n) { return ceil_div(n, Split128::BP) * Split128::BP; }
// The weight gradients: one tile per compute unit and more, with the same allowance, and 64 rows per expert.  3 x 8 experts: 4096 tokens top-2,
// 320 x 320 (150 tiles' worth) 97 | 116, 256 x 1024 (384) 230 | 185, 1024 top-2, 512 x 512 (384) 71 | 66; 64 rows per expert 165 | 150, 32
// 483 | 487, 16 16.1 | 20.9.
bool split_wgrads(int64_t S, int E, int d, int F) {
    const int64_t n = (int64_t)d * F;
    return S >= 64 * (int64_t)E && 3 * E * n >= 256ll * Split128::BP * Split128::BP && 4 * n >= 3 * split_columns(d) * split_columns(F);
}

template <class C, int MODE>
int rows_blocks(int S, const F32RowArgs &a) {
    const int NOUT = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) ? a.F : a.d, BF = MODE == PLAIN_FFN1 ? C::BP / 2 : C::BP;
    return (int)f32_rows_grid(S, a.E, C::BQ, ceil_div(NOUT, BF));
}
template <class C, int MODE>
void rows_launch(int S, const F32RowArgs &a, hipStream_t s) {
    f32_rows_kernel<C, MODE><<<rows_blocks<C, MODE>(S, a), C::NT, 0, s>>>(a);
}

bool few_row_tiles(int S, int E, int NOUT, int width) {
    return ceil_div(S, 64) * ceil_div(NOUT, width) < kRowsFill || S < 64 * (int64_t)E;
}
bool split_rows(int d, int F) { return (int64_t)d * F >= kSplitRows; }
template <class C>
bool split_fills(int S, int NOUT, int BF, int64_t tiles) {
    const int64_t columns = ceil_div(NOUT, BF);
    return ceil_div(S, C::BQ) * columns >= tiles && 4 * (int64_t)NOUT >= 3 * columns * BF;
}
// whether a contraction's tiles are 128 x 128, 64 x 64 or 32 x 32
template <int MODE>
int split_width(int S, int E, int NOUT) {
    constexpr int h = MODE == PLAIN_FFN1 ? 2 : 1;   // features of both weights
    if (S >= 64 * (int64_t)E && split_fills<Split128>(S, NOUT, Split128::BP / h, MODE == PLAIN_DXP ? 128 : 184)) return 128;
    return split_fills<Split64>(S, NOUT, Split64::BP / h, MODE == PLAIN_DXP ? 64 : MODE == PLAIN_DOWN ? 320 : 512) ? 64 : 32;
}
template <int MODE>
void rows_by_size(int S, const F32RowArgs &a, hipStream_t s) {
    const int NOUT = (MODE == PLAIN_FFN1 || MODE == PLAIN_DH) ? a.F : a.d;
    typedef typename std::conditional<MODE == PLAIN_FFN1, F32Short1, F32Short>::type Short;
    auto f = few_row_tiles(S, a.E, NOUT, MODE == PLAIN_FFN1 ? 32 : 64) ? rows_launch<Short, MODE> : rows_launch<F32Tile, MODE>;
    if constexpr (MODE != PLAIN_DH)
        if (split_rows(a.d, a.F)) {
            typedef typename std::conditional<MODE == PLAIN_FFN1, Split32x1, Split32>::type Small;
            const int w = split_width<MODE>(S, a.E, NOUT);
            f = w == 128 ? rows_launch<Split128, MODE> : w == 64 ? rows_launch<Split64, MODE> : rows_launch<Small, MODE>;
        }
    f(S, a, s);
}

bool few_wgrad_tiles(int E, int d, int F) { return 3 * (int64_t)E * ceil_div(d, 64) * ceil_div(F, 64) < kWgradFill; }
template <class C>
int wgrad_blocks(int E, F32Wgrad3 &all) {
    int per = 0;
    for (auto &g : all.g) per += g.tiles = (int)(ceil_div(g.NQ, C::BQ) * ceil_div(g.NP, C::BP));
    return (int)((int64_t)E * per);
}
template <class C>
void wgrad_launch(int E, int T, int K, const int32_t *offsets, F32Wgrad3 all, int accumulate, hipStream_t s) {
    const int n = wgrad_blocks<C>(E, all);
    f32_wgrad_kernel<C><<<n, C::NT, 0, s>>>(E, T, K, offsets, all, accumulate);
}
F32Wgrad3 wgrad_args(int d, int F, const float *H, const float *dYrows, const int32_t *dyperm, const float *xrows, const int32_t *xperm,
                     const float *dA, const float *dB, float *dWg, float *dWu, float *dWd) {
    return {{{H, dYrows, nullptr, dyperm, dWd, F, d, 0}, {xrows, dA, xperm, nullptr, dWg, d, F, 0}, {xrows, dB, xperm, nullptr, dWu, d, F, 0}}};
}

template <class C>
void dh_launch(int S, const F32RowArgs &a, const F32Gate &gate, const RouterFinish<float> &wrt, int nt, hipStream_t s) {
    const int ng = nt + (int)ceil_div(gate.T, 4), first = (ng + 7) / 8 * 8;
    f32_dh_kernel<C><<<first + rows_blocks<C, PLAIN_DH>(S, a), C::NT, 0, s>>>(a, gate, wrt, nt, ng, first);
}
template <class CR, class CW, typename IdxT>
void grads_launch(int S, const F32RowArgs &a, int T, int K, const int32_t *offsets, F32Wgrad3 all, int accumulate,
                  const PlainDwr<float, IdxT> &w, hipStream_t s) {
    const int nw = (int)plain_dwr_blocks(w.Tn, w.d, w.E), first = (nw + 7) / 8 * 8, second = first + rows_blocks<CR, PLAIN_DXP>(S, a);
    f32_grads_kernel<CR, CW, IdxT><<<second + wgrad_blocks<CW>(a.E, all), CR::NT, 0, s>>>(a, a.E, T, K, offsets, all, accumulate, w, nw, first,
                                                                                        second);
}

}  // namespace

hipError_t f32_rows(int mode, int S, int d, int E, int F, const int32_t *offsets, const float *in0, const float *in1, int T,
                    const int32_t *perm, int K, const float *gates, const float *W0, const float *W1, const float *FA,
                    const float *FB, float *o0, float *o1, float *o2, hipStream_t s) {
    auto f = mode == PLAIN_FFN1 ? rows_by_size<PLAIN_FFN1> : mode == PLAIN_DOWN ? rows_by_size<PLAIN_DOWN>
           : mode == PLAIN_DH ? rows_by_size<PLAIN_DH> : rows_by_size<PLAIN_DXP>;
    f(S, F32RowArgs{d, E, F, offsets, in0, in1, T, perm, K, gates, W0, W1, FA, FB, o0, o1, o2}, s);
    return hipGetLastError();
}

hipError_t f32_wgrads(int d, int E, int F, int T, int K, const int32_t *offsets, const float *H, const float *dYrows,
                      const int32_t *dyperm, const float *xrows, const int32_t *xperm, const float *dA, const float *dB,
                      float *dWg, float *dWu, float *dWd, int accumulate, hipStream_t s) {
    auto f = split_wgrads((int64_t)T * K, E, d, F) ? wgrad_launch<Split128> : few_wgrad_tiles(E, d, F) ? wgrad_launch<F32Short> : wgrad_launch<F32Tile>;
    f(E, T, K, offsets, wgrad_args(d, F, H, dYrows, dyperm, xrows, xperm, dA, dB, dWg, dWu, dWd), accumulate, s);
    return hipGetLastError();
}

bool f32_backward_supported(int act, int T, int d, int F) {
    return act == R3_F32 && d % 4 == 0 && F % 4 == 0 && (int64_t)T * d * 4 < (1ll << 31) - 16;
}

hipError_t f32_backward(const F32Backward &b, hipStream_t s) {
    {
        ProfScope ps(PROF_DH, s);
        const F32RowArgs a = {b.d, b.E, b.F, b.offsets, b.dy, nullptr, b.T, b.perm, b.K, b.gates, b.Wd, nullptr, b.FA, b.FB, b.dA, b.dB, nullptr};
        const F32Gate gate = {b.T, b.d, b.K, b.dy, b.Yp, b.gates, b.inv_perm, b.dz, b.dzrow};
        RouterFinish<float> wrt;
        const int nt = wrt.transpose_only(b.d, b.E, b.Wr, b.WrT);
        (few_row_tiles(b.S, b.E, b.F, 64) ? dh_launch<F32Short> : dh_launch<F32Tile>)(b.S, a, gate, wrt, nt, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    ProfScope ps(PROF_WGRAD, s);
    const F32RowArgs a = {b.d, b.E, b.F, b.offsets, b.dA, b.dB, 0, nullptr, 1, nullptr, b.Wg, b.Wu, nullptr, nullptr, b.dXp, nullptr, nullptr};
    const F32Wgrad3 all = wgrad_args(b.d, b.F, b.H, b.dy, b.perm, b.xrows, b.xperm, b.dA, b.dB, b.dWg, b.dWu, b.dWd);
    const bool fr = few_row_tiles(b.S, b.E, b.d, 64), fw = few_wgrad_tiles(b.E, b.d, b.F);
    auto go = [&](auto idx) {
        typedef typename std::remove_const<typename std::remove_pointer<decltype(idx)>::type>::type IdxT;
        const PlainDwr<float, IdxT> w = {b.T, b.d, b.E, b.K, plain_dwr_rows(b.T, b.d, b.E), b.x, b.dz, idx, b.stride, b.part};
        const bool sw = split_wgrads(b.S, b.E, b.d, b.F);
        auto split = [&](auto cr) { return sw ? grads_launch<decltype(cr), Split128, IdxT> : grads_launch<decltype(cr), F32Tile, IdxT>; };
        auto f32 = [&](auto cr) {
            typedef decltype(cr) CR;
            return sw ? grads_launch<CR, Split128, IdxT> : fw ? grads_launch<CR, F32Short, IdxT> : grads_launch<CR, F32Tile, IdxT>;
        };
        auto f = fr ? f32(F32Short{}) : f32(F32Tile{});
        if (split_rows(b.d, b.F)) {
            const int w = split_width<PLAIN_DXP>(b.S, b.E, b.d);
            f = w == 128 ? split(Split128{}) : w == 64 ? split(Split64{}) : split(Split32{});
        }
        f(b.S, a, b.T, b.K, b.offsets, all, b.accumulate, w, s);
    };
    if (b.idx_dtype == R3_IDX_U8) go((const uint8_t *)b.idx);
    else go((const uint16_t *)b.idx);
    return hipGetLastError();
}

}  // namespace r3
