// f32 contractions on the bf16 matrix instruction: D[p][q] = sum_k P[p][k] Q[q][k] for tiles of 128 x 128.
//
// An f32 value is exactly the sum of three bf16 (the rounding of it, the rounding of what is left, the rest), so a product of two
// is nine bf16 products, each exact in f32.  Six are formed; the three left out are less than 2^-25 of the whole (the pieces
// are at most 2^-9 and 2^-18 of the value).  Small ones are added first.  A 32x32x16 MFMA adds 16 products and
// the accumulator and rounds once, where the f32 instruction rounds after every product, so the sums come out
// closer to 64 bits, not further (2048 tokens top-4, 512 x 1024, 16 experts: relative 2-norm of y 8.4e-7 -> 7.3e-7,
// dx 9.9e-7 -> 8.6e-7, weight gradients 7.3e-7 -> 6.2e-7).
//
// Where that argument ends the tile is multiplied again on the f32 instruction (split_failed): an infinity or a NaN in an
// operand, or a value that rounds to an infinity, leaves NaN or infinities in every result that it
// meets; and a value below 2^-110 has bits below the smallest bf16, which is looked for while splitting (split_loses), since a row or column of
// them shows in nothing else when the rest of the tile is ordinary.
//
// What bounds it: of the 2300 cycles that a wave's 64 x 64 x 32 takes, two waves to a SIMD, its 48 MFMAs need 1536, half of them with the
// issue to themselves; splitting its share of the tiles is 180 vector instructions, and the card runs at 1.9-2.1 GHz under all of
// it.  (On the f32 instruction 4096 at least, at 2.3 GHz.)  So a value is split once per work-group, on its way to LDS, where
// 48 KB of planes leave room for two work-groups, one of which splits while the other multiplies.  Splitting raw tiles as they come out of LDS, a value
// by two waves, was no slower where a compute unit had one tile and no faster with two (T=2048 d=512 E=16 K=4 F=1024: SwiGLU 137 us
// and 136, gradients 297 and 280); the dot instructions, which would take the remainder in one step, wait for the matrix pipe.
// T=2048 d=512 E=16 K=4 F=1024, us, f32 instruction in 64 x 64 tiles -> this: SwiGLU 174 -> 128, down 89 -> 80, all gradients and dXp 405 -> 271.
#pragma once
#include "r3_mfma2.h"

namespace r3 {

constexpr int kSplitTile = 128, kSplitThreads = 256, kSplitMinWaves = 2;
constexpr int kSplitPlane = kSplitTile * 64;               // 128 rows of 32 bf16
constexpr int kSplitOperand = 3 * kSplitPlane;
constexpr int kSplitLds = 2 * kSplitOperand;               // 48 KB
typedef f32x16_t SplitAcc[2][2];                           // 4 waves of 64 x 64

typedef float SplitRaw[4][8];                              // [row][k]

__device__ __forceinline__ float4 buffer_load16(rsrc_t r, int voff) {
    return __builtin_bit_cast(float4, __builtin_amdgcn_raw_buffer_load_b128(__builtin_amdgcn_make_buffer_rsrc(
        (void *)(((uint64_t)(uint32_t)r[1] << 32) | (uint32_t)r[0]), 0, r[2], r[3]), voff, 0, 0));
}

// A tile's elements are brought in by 128 threads, eight k (a group) of four rows each.
// K-contiguous rows: thread u has k 8 (u % 4) .. + 7 of rows u / 4 + 32 i
struct SplitRows {
    Src src;
    int voff[4], k0, KK;
    static __device__ __forceinline__ int row(int u, int i) { return (u >> 2) + 32 * i; }
    static __device__ __forceinline__ int group(int u) { return u & 3; }
    __device__ __forceinline__ void init(const float *base, uint64_t bytes, int KK_, int u) {
        src = Src{(const char *)base, bytes, 128};
        KK = KK_;
        k0 = 8 * group(u);
    }
    __device__ __forceinline__ void set_row(int i, int r) { voff[i] = (r * KK + k0) * 4; }
    __device__ __forceinline__ void load(int kt, SplitRaw &v) const {
        const rsrc_t r = src_rsrc(src, kt);
        const int k = kt * 32 + k0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4 a = buffer_load16(r, k < KK ? voff[i] : kOutsideWindow);
            const float4 b = buffer_load16(r, k + 4 < KK ? voff[i] + 16 : kOutsideWindow);
            v[i][0] = a.x; v[i][1] = a.y; v[i][2] = a.z; v[i][3] = a.w;
            v[i][4] = b.x; v[i][5] = b.y; v[i][6] = b.z; v[i][7] = b.w;
        }
    }
};

// feature-contiguous k-rows, the tile's rows being features: thread u has k 8 g .. + 7 of four neighbouring features.
// HALVES: the tile is 64 features of one matrix and the same 64 of another (a wave each).
template <bool HALVES>
struct SplitCols {
    Src src;
    int voff, ld4;
    static __device__ __forceinline__ int row(int u, int i) { return (HALVES ? (u & 64) + 4 * (u & 15) : 4 * (u & 31)) + i; }
    static __device__ __forceinline__ int group(int u) { return HALVES ? (u >> 4) & 3 : u >> 5; }
    // base: first k-row, first feature of the tile (HALVES: of this wave's matrix); ld: floats per k-row
    __device__ __forceinline__ void init(const float *base, uint64_t bytes, int ld, int u) {
        src = Src{(const char *)base, bytes, (uint32_t)(128 * ld)};
        ld4 = 4 * ld;
        voff = 8 * group(u) * ld4 + 16 * (HALVES ? u & 15 : u & 31);
    }
    __device__ __forceinline__ void put(SplitRaw &v, int k, float4 a) const { v[0][k] = a.x; v[1][k] = a.y; v[2][k] = a.z; v[3][k] = a.w; }
    __device__ __forceinline__ void load(int kt, SplitRaw &v) const {
        const rsrc_t r = src_rsrc(src, kt);
#pragma unroll
        for (int k = 0; k < 8; ++k) put(v, k, buffer_load16(r, voff + k * ld4));
    }
};

// the same with k-row r being row perm[r] / K of a matrix, of which there are n
struct SplitGather {
    SplitCols<false> op;
    const int32_t *perm;
    int n, K;
    static __device__ __forceinline__ int row(int u, int i) { return SplitCols<false>::row(u, i); }
    static __device__ __forceinline__ int group(int u) { return SplitCols<false>::group(u); }
    __device__ __forceinline__ void init(const float *m, uint64_t bytes, int ld, int u, const int32_t *perm_, int n_, int K_) {
        op.init(m, bytes, ld, u);
        op.src.step = 0;
        op.voff = 16 * (u & 31);
        perm = perm_;
        n = n_;
        K = K_;
    }
    // a lane works out the row of one k, the others fetch it from there
    __device__ __forceinline__ void load(int kt, SplitRaw &v) const {
        const int lane = threadIdx.x & 63, mine = kt * 32 + (lane & 31);
        const int off = mine < n ? perm[mine] / K * op.ld4 : kOutsideWindow;
        const rsrc_t r = src_rsrc(op.src, 0);
        const int g = group(threadIdx.x & 127);
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int at = __shfl(off, 8 * g + k, 64);
            op.put(v, k, buffer_load16(r, at == kOutsideWindow ? at : at + op.voff));
        }
    }
};

// a reduction over two sources of the same shape, the second from k-tile `first` on
template <class Op>
struct SplitPair {
    Op op;
    Src second;
    int first;
    static __device__ __forceinline__ int row(int u, int i) { return Op::row(u, i); }
    static __device__ __forceinline__ int group(int u) { return Op::group(u); }
    __device__ __forceinline__ void load(int kt, SplitRaw &v) const {
        Op o = op;
        const bool later = kt >= first;
        if (later) o.src = second;
        o.load(later ? kt - first : kt, v);
    }
};

// Where the 16 bytes of group g (8 k) of row r stand in a plane.  Rows are 64 bytes, four to the 256 of all banks; the place in those is a
// one-to-one function of the row's bits 0-3, which sixteen lanes of a fragment read run through, of bits 2-5, which sixteen lanes storing
// features that came four to a load do, and of bits 0-1 and the group, which a K-contiguous operand's do.  (With rows in their order
// and g ^ ((r >> 1) ^ (r >> 3)) the second sort met four ways, conflicts in a fifth of the kernels' cycles: training of 2048 tokens, 512 x 1024, 592 | 586 us.)
__device__ __forceinline__ int split_at(int r, int g) { return (r ^ ((r >> 4) & 3)) * 64 + ((g ^ ((r >> 2) & 3)) << 4); }

// eight f32 as three planes of bf16
__device__ __forceinline__ void split_store(const float (&f)[8], char *at) {
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
        *(uint4 *)(at + p * kSplitPlane) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}
// Whether one of a thread's values is not the sum of its pieces because the last of them lies below the smallest bf16, 2^-133: a value
// of 2^-110 and more has no bits there, zero has none at all.  A minimum of two values takes one instruction, and where it is an ordinary
// number (a tile without padding) that was all.
__device__ __forceinline__ bool split_loses(const SplitRaw &v) {
    float m = 1.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 8; k += 2) asm("v_min3_f32 %0, |%1|, |%2|, %0" : "+v"(m) : "v"(v[i][k]), "v"(v[i][k + 1]));
    if (m >= 0x1p-110f) return false;
    uint32_t least = ~0u;   // of twice the magnitude, less one: a zero counts as the largest
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int k = 0; k < 8; ++k) least = min(least, 2 * __float_as_uint(v[i][k]) - 1);
    return least < 2 * 0x08800000u - 1;
}
template <class Op>
__device__ __forceinline__ void split_store_tile(const SplitRaw &v, char *operand) {
    const int u = threadIdx.x & 127, g = Op::group(u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = Op::row(u, i);
        split_store(v[i], operand + split_at(r, g));
    }
}
// the values as they are, rows of 128 bytes
template <class Op>
__device__ __forceinline__ void raw_store_tile(const SplitRaw &v, char *operand) {
    const int u = threadIdx.x & 127, g = Op::group(u);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int r = Op::row(u, i), s = (r >> 1) & 7;
        *(float4 *)(operand + r * 128 + (((2 * g) ^ s) << 4)) = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
        *(float4 *)(operand + r * 128 + (((2 * g + 1) ^ s) << 4)) = make_float4(v[i][4], v[i][5], v[i][6], v[i][7]);
    }
}

__device__ __forceinline__ void split_meet() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// One k-tile from the planes.  p0, p1: the wave's first rows of its two P tiles (Q: q0 and q0 + 32).
__device__ __forceinline__ void split_multiply(SplitAcc &acc, const char *lds, int p0, int p1, int q0) {
    constexpr int A[6] = {2, 1, 0, 1, 0, 0}, B[6] = {0, 1, 2, 0, 1, 0};
    const int lane = threadIdx.x & 63, r = lane & 31;
    const int at = split_at(r, lane >> 5);
    // a tile's first row is a multiple of 32, whose bit 5 moves a row's place by two rows
    auto tile = [&](int row0) { return (at ^ ((row0 & 32) << 2)) + row0 * 64; };
    const int ap0 = tile(p0), ap1 = tile(p1), aq0 = tile(q0), aq1 = tile(q0 + 32);
    bf16x8_t p[2][2][3], q[2][2][3];
    auto read = [&](int u) {
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const char *a = lds + s * kSplitPlane;
            p[u][0][s] = *(const bf16x8_t *)(a + (ap0 ^ (u << 5)));
            p[u][1][s] = *(const bf16x8_t *)(a + (ap1 ^ (u << 5)));
            q[u][0][s] = *(const bf16x8_t *)(a + kSplitOperand + (aq0 ^ (u << 5)));
            q[u][1][s] = *(const bf16x8_t *)(a + kSplitOperand + (aq1 ^ (u << 5)));
        }
    };
    read(0);
    read(1);
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int x = 0; x < 6; ++x)
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[u][i][A[x]], q[u][j][B[x]], acc[i][j], 0, 0, 0);
}

__device__ __forceinline__ void split_zero(SplitAcc &acc) {
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j) acc[i][j] = f32x16_t{};
}

__device__ __forceinline__ bool split_failed(const SplitAcc &acc, bool lost, char *lds) {
    uint32_t m = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int k = 0; k < 16; ++k) m = max(m, __float_as_uint(acc[i][j][k]) & 0x7fffffffu);
    int *codes = (int *)lds;   // (the waves have met since the last read of the planes)
    const int code = __ballot(m >= 0x7f800000u || lost) != 0;
    if ((threadIdx.x & 63) == 0) codes[threadIdx.x >> 6] = code;
    split_meet();
    const int all = codes[0] | codes[1] | codes[2] | codes[3];
    split_meet();
    return all;
}

// nk k-tiles, for a wave that stages `op` to `mine`
// nk > 0; whether a value of this thread's was not its pieces' sum
template <class Op>
__device__ __forceinline__ bool split_chain(SplitAcc &acc, int nk, const Op &op, char *lds, int operand, int p0, int p1, int q0) {
    SplitRaw v;
    op.load(0, v);
    bool lost = split_loses(v);
    split_store_tile<Op>(v, lds + operand * kSplitOperand);
    op.load(1, v);
    split_meet();
    for (int kt = 0; kt < nk; ++kt) {
        split_multiply(acc, lds, p0, p1, q0);
        split_meet();
        if (kt + 1 == nk) break;
        lost |= split_loses(v);
        split_store_tile<Op>(v, lds + operand * kSplitOperand);
        op.load(kt + 2, v);
        split_meet();
    }
    return lost;
}
// the same on the f32 instruction
template <class Op>
__device__ __forceinline__ void plain_chain(SplitAcc &acc, int nk, const Op &op, char *lds, int operand, int p0, int p1, int q0) {
    const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
    SplitRaw v;
#pragma nounroll
    for (int kt = 0; kt < nk; ++kt) {
        op.load(kt, v);
        raw_store_tile<Op>(v, lds + operand * (kSplitTile * 128));
        split_meet();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int at = r * 128 + (((4 * (c >> 1) + 2 * h + (c & 1)) ^ ((r >> 1) & 7)) << 4);
            const float4 a0 = *(const float4 *)(lds + at + p0 * 128), a1 = *(const float4 *)(lds + at + p1 * 128);
            const float4 b0 = *(const float4 *)(lds + kSplitTile * 128 + at + q0 * 128), b1 = *(const float4 *)(lds + kSplitTile * 128 + at + (q0 + 32) * 128);
            const float a[2][4] = {{a0.x, a0.y, a0.z, a0.w}, {a1.x, a1.y, a1.z, a1.w}}, b[2][4] = {{b0.x, b0.y, b0.z, b0.w}, {b1.x, b1.y, b1.z, b1.w}};
#pragma unroll
            for (int k = 0; k < 4; ++k)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i][k], b[j][k], acc[i][j], 0, 0, 0);
        }
        split_meet();
    }
}

// P is staged by waves 0 and 1, Q by waves 2 and 3, each in a loop of its own (they pass the same barriers).  `products`: of a result.  One
// or two are left to the f32 instruction, which has no more than their own roundings (one: 2.5e-8 of the norm, six products' sum 3.5e-8; two
// 3.1e-8 and 3.4e-8; three 3.6e-8 and 3.3e-8, 32 1.0e-7 and 6.9e-8).
template <class OpP, class OpQ>
__device__ __forceinline__ void split_loop(SplitAcc &acc, int nk, int products, const OpP &P, const OpQ &Q, char *lds, int p0, int p1, int q0) {
    if (nk <= 0) return;
    const bool is_p = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 7)) == 0;
    if (products > 2) {
        const bool lost = is_p ? split_chain(acc, nk, P, lds, 0, p0, p1, q0) : split_chain(acc, nk, Q, lds, 1, p0, p1, q0);
        if (!split_failed(acc, lost, lds)) return;
        split_zero(acc);
    }
    if (is_p) plain_chain(acc, nk, P, lds, 0, p0, p1, q0);
    else plain_chain(acc, nk, Q, lds, 1, p0, p1, q0);
}

}  // namespace r3
