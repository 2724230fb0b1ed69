// f32 contractions on the bf16 matrix instruction: D[p][q] = sum_k P[p][k] Q[q][k].
//
// An f32 value is exactly the sum of three bf16 (the rounding of it, the rounding of what is left, the rest), which are below 2^-8 and 2^-17 of
// it after the first, so a product of two is nine bf16 products, each exact in f32.  Six are formed; the three left out are at most 2^-24 of
// the whole, half a unit in its last place, and 6e-9 of the norm of a sum of random ones.  Small ones are added first.  A
// 16x16x32 MFMA adds 32 products and the accumulator and rounds once (terms more than 24 bits below the largest are lost), where the f32
// instruction rounds after every product, so from three products on the sums come out closer to 64 bits, not further: relative 2-norm of 32 products
// 1.03e-7 -> 3.8e-8, 512 4.05e-7 -> 3.34e-7 (32x32x16 MFMAs: 6.9e-8, 3.39e-7); sums of one and two are left to the f32 instruction.
//
// Where that argument ends the f32 instruction has the word (split_loop), for the results concerned and no others: an infinity or a NaN in an
// operand, or a value that rounds to an infinity, leaves NaN or infinities in every result that it
// meets; a value below 2^-110 has bits below the smallest bf16, which is looked for while splitting (split_loses), since a row or column of
// them shows in nothing else when the rest of the tile is ordinary.
//
// Tiles of every size add the same products in the same order, and which results are taken from the f32 instruction follows from their own row and
// column: a result does not depend on what shares its tile nor on the tile's size.
//
// What bounds it, tiles of 128 x 128: of the 2300 cycles that a wave's 64 x 64 x 32 takes, two waves to a SIMD, its 96 MFMAs need 1536, half of them
// with the issue to themselves; splitting its share of the tiles and looking for small values is 200 vector instructions, and the card runs at
// 1.9-2.1 GHz under all of it.  (On the f32 instruction 4096 at least, at 2.3 GHz.)  So a value is split once per work-group, on its way to LDS, where
// 48 KB of planes leave room for two work-groups, one of which splits while the other multiplies.  T=2048 d=512 E=16 K=4 F=1024, us, f32 instruction in
// 64 x 64 tiles -> this: SwiGLU 156 -> 121, down 87 -> 82, all gradients and dXp 405 -> 249.
// Small tiles, which layers of few rows take: the chain of one k-tile (fragments out of LDS, six MFMAs in a row, the next k-tile's splitting
// among them, the way back into LDS), 750 cycles for 32 x 32 and 580 on the f32 instruction.  128 tokens top-2, 512 x 512, 8 experts: SwiGLU
// 13.2 -> 16.0, down 9.8 -> 11.6.  No faster: four k-tiles on their way instead of two, fragments a k-tile ahead, two or four k-tiles
// between barriers, waves that only split beside waves that only multiply (128 x 128: 30 % faster with a compute unit to itself,
// 12-17 % slower where there is work for two).
#pragma once
#include "r3_mfma2.h"

namespace r3 {

typedef float f32x4_t __attribute__((ext_vector_type(4)));

// 4 waves as 2 (P) x 2 (Q), each TP x TQ tiles of 16 x 16.  STAGES: k-tiles in LDS; with one, two barriers a k-tile
template <int TP_, int TQ_, int STAGES_, int MINW_>
struct SplitCfg {
    static constexpr bool SPLIT = true;
    static constexpr int TP = TP_, TQ = TQ_, STAGES = STAGES_, MINW = MINW_, NT = 256;
    static constexpr int BP = 32 * TP, BQ = 32 * TQ, PPLANE = BP * 64, QPLANE = BQ * 64, STAGE = 3 * (PPLANE + QPLANE), LDS = STAGES * STAGE;
};
template <class C> using SplitAcc = f32x4_t[C::TP][C::TQ];

template <int N> struct SplitRaw { float f[N][8]; };   // [row][k]

template <int N>
__device__ __forceinline__ void buffer_load_floats(rsrc_t r, int voff, float (&f)[N]) {
    const auto b = __builtin_amdgcn_make_buffer_rsrc((void *)(((uint64_t)(uint32_t)r[1] << 32) | (uint32_t)r[0]), 0, r[2], r[3]);
    if constexpr (N == 4) {
        const float4 v = __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(b, voff, 0, 0));
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    } else if constexpr (N == 2) {
        const float2 v = __builtin_bit_cast(float2, __builtin_amdgcn_raw_buffer_load_b64(b, voff, 0, 0));
        f[0] = v.x; f[1] = v.y;
    } else {
        f[0] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, voff, 0, 0));
    }
}

// A tile's R rows x 32 k are brought in by 128 threads, eight k (a group) of N = R / 32 rows each.
// K-contiguous rows: thread u has k 8 (u % 4) .. + 7 of rows u / 4 + 32 i
template <int R>
struct SplitRows {
    static constexpr int N = R / 32;
    Src src;
    int voff[N], k0, KK;
    // whether a k-tile is whole, in any case; the one before the last that may not be, or -1
    static __device__ __forceinline__ bool inside(int kt, int nk) { return kt < nk - 1; }
    static __device__ __forceinline__ int middle() { return -1; }
    static __device__ __forceinline__ int row(int u, int i) { return (u >> 2) + 32 * i; }
    static __device__ __forceinline__ int group(int u) { return u & 3; }
    __device__ __forceinline__ void init(const float *base, uint64_t bytes, int KK_, int u) {
        src = Src{(const char *)base, bytes, 128};
        KK = KK_;
        k0 = 8 * group(u);
    }
    __device__ __forceinline__ void set_row(int i, int r) { voff[i] = (r * KK + k0) * 4; }
    __device__ __forceinline__ void load(int kt, SplitRaw<N> &v) const {
        const rsrc_t r = src_rsrc(src, kt);
        const int k = kt * 32 + k0;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            float a[4], b[4];
            buffer_load_floats(r, k < KK ? voff[i] : kOutsideWindow, a);
            buffer_load_floats(r, k + 4 < KK ? voff[i] + 16 : kOutsideWindow, b);
#pragma unroll
            for (int j = 0; j < 4; ++j) v.f[i][j] = a[j], v.f[i][4 + j] = b[j];
        }
    }
};

// feature-contiguous k-rows, the tile's rows being features: thread u has k 8 g .. + 7 of N neighbouring features.
// HALVES: the tile is R / 2 features of one matrix and the same R / 2 of another (a wave each).
template <int R, bool HALVES>
struct SplitCols {
    static constexpr int N = R / 32;
    Src src;
    int voff, ld4;
    // whether a k-tile is whole, in any case; the one before the last that may not be, or -1
    static __device__ __forceinline__ bool inside(int kt, int nk) { return kt < nk - 1; }
    static __device__ __forceinline__ int middle() { return -1; }
    static __device__ __forceinline__ int row(int u, int i) { return (HALVES ? (u >> 6) * (R / 2) + N * (u & 15) : N * (u & 31)) + i; }
    static __device__ __forceinline__ int group(int u) { return HALVES ? (u >> 4) & 3 : u >> 5; }
    // base: first k-row, first feature of the tile (HALVES: of this wave's matrix); ld: floats per k-row
    __device__ __forceinline__ void init(const float *base, uint64_t bytes, int ld, int u) {
        src = Src{(const char *)base, bytes, (uint32_t)(128 * ld)};
        ld4 = 4 * ld;
        voff = 8 * group(u) * ld4 + 4 * N * (HALVES ? u & 15 : u & 31);
    }
    static __device__ __forceinline__ void load_k(rsrc_t r, int off, SplitRaw<N> &v, int k) {
        float a[N];
        buffer_load_floats(r, off, a);
#pragma unroll
        for (int i = 0; i < N; ++i) v.f[i][k] = a[i];
    }
    __device__ __forceinline__ void load(int kt, SplitRaw<N> &v) const {
        const rsrc_t r = src_rsrc(src, kt);
#pragma unroll
        for (int k = 0; k < 8; ++k) load_k(r, voff + k * ld4, v, k);
    }
};

// the same with k-row r being row perm[r] / K of a matrix, of which there are n
template <int R>
struct SplitGather {
    typedef SplitCols<R, false> Cols;
    static constexpr int N = Cols::N;
    Cols op;
    const int32_t *perm;
    int n, K;
    // whether a k-tile is whole, in any case; the one before the last that may not be, or -1
    static __device__ __forceinline__ bool inside(int kt, int nk) { return kt < nk - 1; }
    static __device__ __forceinline__ int middle() { return -1; }
    static __device__ __forceinline__ int row(int u, int i) { return Cols::row(u, i); }
    static __device__ __forceinline__ int group(int u) { return Cols::group(u); }
    __device__ __forceinline__ void init(const float *m, uint64_t bytes, int ld, int u, const int32_t *perm_, int n_, int K_) {
        op.init(m, bytes, ld, u);
        op.src.step = 0;
        op.voff = 4 * N * (u & 31);
        perm = perm_;
        n = n_;
        K = K_;
    }
    // a lane works out the row of one k, the others fetch it from there
    __device__ __forceinline__ void load(int kt, SplitRaw<N> &v) const {
        const int lane = threadIdx.x & 63, mine = kt * 32 + (lane & 31);
        const int off = mine < n ? perm[mine] / K * op.ld4 : kOutsideWindow;
        const rsrc_t r = src_rsrc(op.src, 0);
        const int g = group(threadIdx.x & 127);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int at = __shfl(off, 8 * g + k, 64);
            Cols::load_k(r, at == kOutsideWindow ? at : at + op.voff, v, k);
        }
    }
};

// a reduction over two sources of the same shape, the second from k-tile `first` on
template <class Op>
struct SplitPair {
    static constexpr int N = Op::N;
    Op op;
    Src second;
    int first;
    __device__ __forceinline__ bool inside(int kt, int nk) const { return kt < nk - 1 && kt != middle(); }
    __device__ __forceinline__ int middle() const { return op.KK % 32 ? first - 1 : -1; }
    static __device__ __forceinline__ int row(int u, int i) { return Op::row(u, i); }
    static __device__ __forceinline__ int group(int u) { return Op::group(u); }
    __device__ __forceinline__ void load(int kt, SplitRaw<N> &v) const {
        Op o = op;
        const bool later = kt >= first;
        if (later) o.src = second;
        o.load(later ? kt - first : kt, v);
    }
};

// Where the 16 bytes of group g (8 k) of row r stand in a plane.  Rows are 64 bytes, four to the 256 of all banks.  Sixteen lanes meet in an access of 16
// bytes a lane: 0-3, 12-15 and 20-27 of 32, and the others.  A fragment read's are then rows 0-3 and 12-15 of one group and 4-11 of the next; those of a
// K-contiguous operand's store four rows of all groups; those of features that came four to a load run through the row's bits 2-5: the place is a one-to-one function
// of each.  (With g itself in place of its permutation a fragment's rows met two by two, conflicts in a tenth of the kernels' cycles; with rows
// in their order besides the third sort met four ways: training of 2048 tokens, 512 x 1024, 592 | 586 us.)
__device__ __forceinline__ int split_at(int r, int g) {
    const int turned = ((g ^ (g >> 1)) & 1) | ((g & 1) << 1);   // 0 3 1 2
    return (r ^ ((r >> 4) & 3)) * 64 + ((turned ^ ((r >> 2) & 3)) << 4);
}

// eight f32 as three planes of bf16
__device__ __forceinline__ void split_store(const float (&f)[8], char *at, int plane) {
    float r[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = f[i];
#pragma unroll
    for (int p = 0; p < 3; ++p) {
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            w[i] = pack_bf16x2(r[2 * i], r[2 * i + 1]);
            if (p < 2) {
                r[2 * i] -= __uint_as_float(w[i] << 16);
                r[2 * i + 1] -= __uint_as_float(w[i] & 0xffff0000u);
            }
        }
        *(uint4 *)(at + p * plane) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}
template <class Op>
__device__ __forceinline__ void split_store_tile(const SplitRaw<Op::N> &v, char *operand, int plane) {
    const int u = threadIdx.x & 127, g = Op::group(u);
#pragma unroll
    for (int i = 0; i < Op::N; ++i) split_store(v.f[i], operand + split_at(Op::row(u, i), g), plane);
}
// Which of a thread's rows (bit i: row i) have a value that is not the sum of its pieces because the last of them lies below the smallest
// bf16, 2^-133: a value of 2^-110 and more has no bits there, zero has none at all.
constexpr float kSplitLeast = 0x1p-110f;
template <int N>
__device__ __forceinline__ int split_loses(const SplitRaw<N> &v) {
    int rows = 0;
#pragma unroll
    for (int i = 0; i < N; ++i) {
        uint32_t least = ~0u;   // of twice the magnitude, less one: a zero counts as the largest
#pragma unroll
        for (int k = 0; k < 8; ++k) least = min(least, 2 * __float_as_uint(v.f[i][k]) - 1);
        rows |= least < 2 * 0x08800000u - 1 ? 1 << i : 0;
    }
    return rows;
}
// the smallest magnitudes that a thread has seen, one of two chains each, zeros among them: half an instruction a value
struct SplitLeast {
    float m[2] = {1.0f, 1.0f};
    template <int N> __device__ __forceinline__ void take(const SplitRaw<N> &v, bool counts) {
        float t[2] = {m[0], m[1]};
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int k = 0; k < 8; k += 2) asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(t[k / 2 & 1]) : "v"(v.f[i][k]), "v"(v.f[i][k + 1]));
#pragma unroll
        for (int k = 0; k < 2; ++k) m[k] = counts ? t[k] : m[k];
    }
    __device__ __forceinline__ bool ordinary() const { return fminf(m[0], m[1]) >= kSplitLeast; }
};
// the values as they are, rows of 128 bytes
template <class Op>
__device__ __forceinline__ void raw_store_tile(const SplitRaw<Op::N> &v, char *operand) {
    const int u = threadIdx.x & 127, g = Op::group(u);
#pragma unroll
    for (int i = 0; i < Op::N; ++i) {
        const int r = Op::row(u, i), s = (r >> 1) & 7;
        const float(&f)[8] = v.f[i];
        *(float4 *)(operand + r * 128 + (((2 * g) ^ s) << 4)) = make_float4(f[0], f[1], f[2], f[3]);
        *(float4 *)(operand + r * 128 + (((2 * g + 1) ^ s) << 4)) = make_float4(f[4], f[5], f[6], f[7]);
    }
}

__device__ __forceinline__ void split_meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// A wave's tiles: rows prow(i) .. + 15 of P and qrow(j) .. + 15 of Q; a lane's results are rows 4 (lane / 16) .. + 3 of P, column lane % 16 of Q.
// HALVES: half of its P tiles are features of one matrix, half the same features of the other.
template <class C, bool HALVES>
struct SplitWave {
    static __device__ __forceinline__ int wp() { return (threadIdx.x >> 6) & 1; }
    static __device__ __forceinline__ int wq() { return threadIdx.x >> 7; }
    static __device__ __forceinline__ int prow(int i) {
        if constexpr (HALVES) return i / (C::TP / 2) * (C::BP / 2) + 16 * (C::TP / 2 * wp() + i % (C::TP / 2));
        else return 16 * (C::TP * wp() + i);
    }
    static __device__ __forceinline__ int qrow(int j) { return 16 * (C::TQ * wq() + j); }
};

template <class C> struct SplitFrag { bf16x8_t p[C::TP][3], q[C::TQ][3]; };

// One k-tile from the planes.
template <class C, class W>
__device__ __forceinline__ void split_read(SplitFrag<C> &f, const char *lds) {
    const int lane = threadIdx.x & 63, at = split_at(lane & 15, lane >> 4);
    // a tile's first row is a multiple of 16, whose bits 4 and 5 move a row's place
    auto tile = [&](int row0) { return (at ^ ((row0 & 48) << 2)) + row0 * 64; };
#pragma unroll
    for (int s = 0; s < 3; ++s) {   // in the order in which they are wanted
#pragma unroll
        for (int i = 0; i < C::TP; ++i) f.p[i][2 - s] = *(const bf16x8_t *)(lds + (2 - s) * C::PPLANE + tile(W::prow(i)));
#pragma unroll
        for (int j = 0; j < C::TQ; ++j) f.q[j][s] = *(const bf16x8_t *)(lds + 3 * C::PPLANE + s * C::QPLANE + tile(W::qrow(j)));
    }
}
// Small products first.  Every size of tile adds the same products in the same order: a result does not depend on it.
template <class C>
__device__ __forceinline__ void split_multiply(SplitAcc<C> &acc, const SplitFrag<C> &f) {
    constexpr int A[6] = {2, 1, 0, 1, 0, 0}, B[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
    for (int x = 0; x < 6; ++x)
#pragma unroll
        for (int i = 0; i < C::TP; ++i)
#pragma unroll
            for (int j = 0; j < C::TQ; ++j)
                acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f.p[i][A[x]], f.q[j][B[x]], acc[i][j], 0, 0, 0);
}

template <class C>
__device__ __forceinline__ void split_zero(SplitAcc<C> &acc) {
#pragma unroll
    for (int i = 0; i < C::TP; ++i)
#pragma unroll
        for (int j = 0; j < C::TQ; ++j) acc[i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
}

// nk > 0 k-tiles, for a wave that stages `op`; which of this thread's rows had a value that was not its pieces' sum.
// One stage: the test costs what it takes of the issue, and a branch in the loop keeps the splitting from among the MFMAs.  So of the k-tiles that cannot be
// padded the smallest magnitudes are kept, and only where those are not ordinary (a zero or a small value) the operand is gone through
// once more; the last k-tile of each source, which may be, is tested by itself.  (A minimum and a branch every k-tile: SwiGLU and all of the training
// of 2048 tokens, 512 x 1024 132 and 571 us, this 122 and 569, no test 119 and 547; SwiGLU of 3000 rows, 1024 x 512 71, 57, 59.  With a
// gradient of zeros in two tokens of five the weight gradients, whose operands are then gone through twice, 253 -> 277 us.)  The small tiles, which
// wait for their MFMAs, test everything.
template <class C, class W, bool IS_P, class Op>
__device__ __forceinline__ int split_chain(SplitAcc<C> &acc, int nk, const Op &op, char *lds) {
    constexpr int plane = IS_P ? C::PPLANE : C::QPLANE, at = IS_P ? 0 : 3 * C::PPLANE;
    if constexpr (C::STAGES == 1) {
        SplitRaw<Op::N> v;
        SplitLeast least;
        op.load(0, v);
        int lost = split_loses(v);
        split_store_tile<Op>(v, lds + at, plane);
        op.load(min(1, nk - 1), v);
        split_meet();
        for (int kt = 0; kt < nk; ++kt) {
            SplitFrag<C> f;
            split_read<C, W>(f, lds);
            split_multiply<C>(acc, f);
            split_meet();
            least.take(v, op.inside(kt + 1, nk));
            split_store_tile<Op>(v, lds + at, plane);
            op.load(min(kt + 2, nk - 1), v);
            split_meet();
        }
        lost |= split_loses(v);
        const int middle = op.middle();
        if (middle >= 0) {
            op.load(middle, v);
            lost |= split_loses(v);
        }
        if (__ballot(!least.ordinary())) {   // (by whole waves: a gathered operand's lanes take its rows from each other)
            SplitRaw<Op::N> w[3];
#pragma unroll
            for (int j = 0; j < 3; ++j) op.load(min(1 + j, nk - 1), w[j]);
#pragma nounroll
            for (int kt = 1; kt < nk - 1; kt += 3)
#pragma unroll
                for (int j = 0; j < 3; ++j) {   // (some k-tiles twice)
                    lost |= split_loses(w[j]);
                    op.load(min(kt + j + 3, nk - 1), w[j]);
                }
        }
        return lost;
    } else {
        SplitRaw<Op::N> v[2];
        op.load(0, v[0]);
        op.load(1, v[1]);
        int lost = split_loses(v[0]);
        split_store_tile<Op>(v[0], lds + at, plane);
        op.load(2, v[0]);
        split_meet();
        for (int k0 = 0;; k0 += 2) {
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                SplitFrag<C> f;
                split_read<C, W>(f, lds + j * C::STAGE);
                split_multiply<C>(acc, f);
                lost |= split_loses(v[1 - j]);
                split_store_tile<Op>(v[1 - j], lds + (1 - j) * C::STAGE + at, plane);   // (past the last k-tile: zeros)
                op.load(k0 + j + 3, v[1 - j]);
                split_meet();
                if (k0 + j + 1 == nk) return lost;   // (not out of the inner loop alone: the loads would be waited for as on every way round)
            }
        }
    }
}
// the same on the f32 instruction, products and sums as the tiles of r3_f32.hip have them
template <class C, class W, bool IS_P, class Op>
__device__ __forceinline__ void plain_chain(SplitAcc<C> &acc, int nk, const Op &op, char *lds) {
    const int lane = threadIdx.x & 63;
    SplitRaw<Op::N> v;
#pragma nounroll
    for (int kt = 0; kt < nk; ++kt) {
        op.load(kt, v);
        raw_store_tile<Op>(v, lds + (IS_P ? 0 : C::BP * 128));
        split_meet();
#pragma nounroll
        for (int g = 0; g < 2; ++g) {
            auto read = [&](const char *operand, int row0, float(&f)[4]) {
                const int row = row0 + (lane & 15);
                const float4 x = *(const float4 *)(operand + row * 128 + (((4 * g + (lane >> 4)) ^ ((row >> 1) & 7)) << 4));
                f[0] = x.x; f[1] = x.y; f[2] = x.z; f[3] = x.w;
            };
            float a[C::TP][4], b[C::TQ][4];
#pragma unroll
            for (int i = 0; i < C::TP; ++i) read(lds, W::prow(i), a[i]);
#pragma unroll
            for (int j = 0; j < C::TQ; ++j) read(lds + C::BP * 128, W::qrow(j), b[j]);
#pragma unroll
            for (int s = 0; s < 4; ++s)
#pragma unroll
                for (int i = 0; i < C::TP; ++i)
#pragma unroll
                    for (int j = 0; j < C::TQ; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][s], b[j][s], acc[i][j], 0, 0, 0);
        }
        split_meet();
    }
}

// Whether any of the tile's results is one that the pieces do not give.
template <class C>
__device__ __forceinline__ bool split_failed(const SplitAcc<C> &acc, int lost, char *lds) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < C::TP; ++i)
#pragma unroll
        for (int j = 0; j < C::TQ; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) m = max(m, __float_as_uint(acc[i][j][k]) & 0x7fffffffu);
    int *codes = (int *)lds + C::NT;   // (the waves have met since the last read of the planes)
    const int code = __ballot(m >= 0x7f800000u || lost != 0) != 0;
    if ((threadIdx.x & 63) == 0) codes[threadIdx.x >> 6] = code;
    split_meet();
    const int4 all = *(const int4 *)codes;
    return __builtin_amdgcn_readfirstlane(all.x | all.y | all.z | all.w);
}
// Which ones: bit (i TQ + j) 4 + k, those that are not finite, and those of a row of P or Q with a value that is not its pieces' sum.  The others
// stand as they are, so that a row's results do not depend on the rows that share its tile.
template <class C, class W, class OpP, class OpQ>
__device__ __forceinline__ uint64_t split_failures(const SplitAcc<C> &acc, bool is_p, int lost, char *lds) {
    int *rows = (int *)lds;
    static_assert(C::BP + C::BQ <= C::NT, "");
    const int u = threadIdx.x & 127, lane = threadIdx.x & 63;
    if (threadIdx.x < C::BP + C::BQ) rows[threadIdx.x] = 0;
    split_meet();
    if (is_p) {
        for (int i = 0; i < OpP::N; ++i)
            if (lost >> i & 1) rows[OpP::row(u, i)] = 1;
    } else {
        for (int i = 0; i < OpQ::N; ++i)
            if (lost >> i & 1) rows[C::BP + OpQ::row(u, i)] = 1;
    }
    split_meet();
    uint64_t bits = 0;
#pragma unroll
    for (int i = 0; i < C::TP; ++i)
#pragma unroll
        for (int j = 0; j < C::TQ; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool bad = (__float_as_uint(acc[i][j][k]) & 0x7fffffffu) >= 0x7f800000u || rows[W::prow(i) + 4 * (lane >> 4) + k] ||
                                 rows[C::BP + W::qrow(j) + (lane & 15)];
                bits |= (uint64_t)bad << ((i * C::TQ + j) * 4 + k);
            }
    split_meet();
    return bits;
}

// P is staged by waves 0 and 1, Q by waves 2 and 3, each in a loop of its own (they pass the same barriers).  `products`: of a result.  One
// or two are left to the f32 instruction, which has no more than their own roundings (one: 2.5e-8 of the norm, six products' sum 3.5e-8; two
// 3.1e-8 and 3.4e-8; three 3.6e-8 and 3.3e-8, 32 1.0e-7 and 3.8e-8).
template <class C, class W, class OpP, class OpQ>
__device__ __forceinline__ void split_loop(SplitAcc<C> &acc, int nk, int products, const OpP &P, const OpQ &Q, char *lds) {
    split_zero<C>(acc);
    if (nk <= 0) return;
    const bool is_p = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 7)) == 0;
    uint64_t again = ~0ull;
    if (products > 2) {
        const int lost = is_p ? split_chain<C, W, true>(acc, nk, P, lds) : split_chain<C, W, false>(acc, nk, Q, lds);
        if (!split_failed<C>(acc, lost, lds)) return;
        again = split_failures<C, W, OpP, OpQ>(acc, is_p, lost, lds);
    }
    SplitAcc<C> f;
    split_zero<C>(f);
    if (is_p) plain_chain<C, W, true>(f, nk, P, lds);
    else plain_chain<C, W, false>(f, nk, Q, lds);
#pragma unroll
    for (int i = 0; i < C::TP; ++i)
#pragma unroll
        for (int j = 0; j < C::TQ; ++j)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc[i][j][k] = again >> ((i * C::TQ + j) * 4 + k) & 1 ? f[i][j][k] : acc[i][j][k];
}

}  // namespace r3
