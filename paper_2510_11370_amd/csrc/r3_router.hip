// Router logits, replay gate and agreement in one launch (Section 4.1: first equation and the replay-gate
// equation; Section 3.2, router level):
//   s = x W_r (+ bias),  g_j = exp(s[id_j] - m) / sum_i exp(s[id_i] - m) over the recorded ids (m their maximum).
// A work-group owns a few tokens and all experts, so a token's logits never leave it unless asked for.
//
// What bounds it: for few tokens latency, for many the read of x.  Every work-group streams the whole of W_r (L2), so
// a serial walk over k is a chain of round trips: 32 of them took 24 us at 64 tokens, d = 2048.  The kernels keep
// several stages of k in flight, but add up in the order of k, whatever the number of tokens: split over the waves, a
// token's logits were other bits in a micro-batch than in the whole batch.
#include <algorithm>

#include "r3_finish.h"
#include "r3_kernels.h"
#include "r3_mfma.h"
#include "r3_mfma2.h"
#include "r3_topk.h"

namespace r3 {

// The gate (and agreement) of a work-group's tokens from their logits in LDS: rows of PITCH floats, entries at and past
// E undefined.  8 lanes take a token.  A recorded id >= E is clamped and raises R3_DATA_IDX_RANGE; a non-finite
// logit among the recorded ones raises R3_DATA_NONFINITE.  agree (K <= 8): the token's own top-K mask (the record
// kernel's selection) against the mask of the recorded ids; the block adds its counts once (integer atomics).
// `part`: 2 * waves 64-bit words of LDS that hold nothing else.
template <int NV, int NT, typename IdxT>
__device__ __forceinline__ void gate_from_lds(const float *sl, int pitch, int t0, int nq, int T, int E, int K,
                                              const IdxT *__restrict__ idx, int64_t stride, float *__restrict__ gates,
                                              unsigned long long *agree, int32_t *status, unsigned long long *part) {
    const int sub = threadIdx.x & 7;
    int bad = 0;
    unsigned long long equal = 0, common = 0;
    for (int q = threadIdx.x >> 3; q < nq; q += NT / 8) {
        const int t = t0 + q;
        const bool live = t < T;
        const float *row = sl + q * pitch;
        const IdxT *id = idx + (int64_t)(live ? t : 0) * stride;
        // gate: slots sub, sub + 8, ... of the token
        float m = -INFINITY;
        for (int j = sub; j < K; j += 8) {
            int e = (int)id[j];
            if (e >= E) { bad |= R3_DATA_IDX_RANGE; e = E - 1; }
            const float z = row[e];
            if (live && !(fabsf(z) <= 3.4028235e38f)) bad |= R3_DATA_NONFINITE;
            m = fmaxf(m, z);
        }
        m = fmaxf(m, __shfl_xor(m, 1, 8));
        m = fmaxf(m, __shfl_xor(m, 2, 8));
        m = fmaxf(m, __shfl_xor(m, 4, 8));
        float den = 0.0f;
        for (int j = sub; j < K; j += 8) den += expf(row[min((int)id[j], E - 1)] - m);
        den += __shfl_xor(den, 1, 8);
        den += __shfl_xor(den, 2, 8);
        den += __shfl_xor(den, 4, 8);
        const float inv = 1.0f / den;
        if (live)
            for (int j = sub; j < K; j += 8) gates[(int64_t)t * K + j] = expf(row[min((int)id[j], E - 1)] - m) * inv;
        if (agree) {
            uint32_t key[NV][4];
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const float4 v = *(const float4 *)(row + 32 * i + 4 * sub);
                const int e = 32 * i + 4 * sub;
                bool nf;
                // (experts that do not exist rank with the NaNs, behind every real one of that rank)
                key[i][0] = e < E ? order_key(v.x, nf) : 0u;
                key[i][1] = e + 1 < E ? order_key(v.y, nf) : 0u;
                key[i][2] = e + 2 < E ? order_key(v.z, nf) : 0u;
                key[i][3] = e + 3 < E ? order_key(v.w, nf) : 0u;
            }
            uint32_t own[NV], rec[NV];
            topk_mask8<NV>(key, K, sub, own);
            const int e = sub < K ? min((int)id[sub], E - 1) : -1;
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                uint32_t w = (e >> 5) == i ? 1u << (e & 31) : 0u;   // e = -1 matches no word
                w |= group8_exchange<0>(w);
                w |= group8_exchange<1>(w);
                w |= group8_exchange<2>(w);
                rec[i] = w;
            }
            int shared = 0;
#pragma unroll
            for (int i = 0; i < NV; ++i) shared += __popc(own[i] & rec[i]);
            if (live && sub == 0) {
                common += (unsigned long long)shared;
                equal += shared == K;
            }
        }
    }
    if (bad && status) atomicOr(status, bad);
    if (agree) {
        equal = wave_sum(equal);
        common = wave_sum(common);
        const int w = threadIdx.x / kWave;
        if (lane_id() == 0) {
            part[2 * w] = equal;
            part[2 * w + 1] = common;
        }
        __syncthreads();
        if (threadIdx.x == 0) {
            unsigned long long a0 = 0, a1 = 0;
            for (int i = 0; i < NT / kWave; ++i) {
                a0 += part[2 * i];
                a1 += part[2 * i + 1];
            }
            if (a1) atomicAdd(agree + 1, a1);
            if (a0) atomicAdd(agree, a0);
        }
    }
}

// Partial logits of the k groups (red: [WK][BQ][pitch], EP columns each) added up in ascending order into group
// 0's rows, plus the bias; whole rows go to logits_out if it is given.
template <int WK, int BQ, int EP, int NT>
__device__ __forceinline__ void add_logits(float *red, int pitch, int t0, int T, int E, const float *__restrict__ bias,
                                           float *__restrict__ logits_out) {
    for (int i = threadIdx.x; i < BQ * (EP / 4); i += NT) {
        const int q = i / (EP / 4), e = i % (EP / 4) * 4;
        float *p = red + q * pitch + e;
        float4 v = *(const float4 *)p;
#pragma unroll
        for (int g = 1; g < WK; ++g) {
            const float4 w = *(const float4 *)(p + g * BQ * pitch);
            v.x += w.x; v.y += w.y; v.z += w.z; v.w += w.w;
        }
        float s[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int c = 0; c < 4; ++c)
            if (bias && e + c < E) s[c] += bias[e + c];
        *(float4 *)p = make_float4(s[0], s[1], s[2], s[3]);
        if (logits_out && t0 + q < T) {
            float *o = logits_out + (int64_t)(t0 + q) * E + e;
            if (E % 4 == 0) {
                if (e < E) *(float4 *)o = make_float4(s[0], s[1], s[2], s[3]);
            } else {
#pragma unroll
                for (int c = 0; c < 4; ++c)
                    if (e + c < E) o[c] = s[c];
            }
        }
    }
}

// ---------------------------------------------------------------------------
// bf16 (d and E multiples of 8, E <= 512).  A work-group takes 32 or 64 tokens and all experts.  Its eight waves bring
// stages of SK k into a ring of NBUF in LDS with direct loads, one barrier per stage; the 32 x 32 results are dealt to the
// waves and each is one chain of 32x32x16 instructions over ascending k.  So a token's logits are the same bits
// whatever the number of tokens, and those of a sum in the order of k.
// Few, large stages: with few work-groups a stage costs about 0.3 us however small it is (barrier, LDS round trip, the
// chain's end).  T=64 d=2048, us with half the k per stage: E=128 9.2 | 15.9, E=256 14.9 | 17.4, E=512 26.1 | 29.8.
// W_r stage: EP / 64 tiles [SK k][64 experts].  Their k-rows are 128 B: two to a bank line, so their 64-byte halves
// swap by bit 1 of k and the transposing reads (4 k-rows of 64 B at a time) touch every bank once.  x stage: SK / 32
// tiles [BQ tokens][32 k] (KcFrag<32>).
// ---------------------------------------------------------------------------
template <int EP_, int TQ_>
struct RouterCfg {
    static constexpr int EP = EP_, TQ = TQ_, BQ = 32 * TQ, NW = 8, NT = 64 * NW, PITCH = EP + 4;
    // k per stage: what lets two or three stages into LDS
    static constexpr int SK = EP == 64 ? 256 / TQ : EP == 128 ? 128 : EP == 256 ? 128 / TQ : 64;
    static constexpr int WT = SK * EP * 2, XT = SK * BQ * 2, STAGE = WT + XT;
    static constexpr int NBUF = (160 * 1024 - 256) / STAGE;
    static constexpr int WCH = WT / 1024, XCH = XT / 1024;                       // loads of 1 KB; of the whole work-group
    static constexpr int WPW = WCH / NW, XPW = (XCH + NW - 1) / NW;              // of a wave (the last one: the first XLAST waves)
    static constexpr int XLAST = XCH - (XPW - 1) * NW;
    static constexpr int NE = EP / 32, TILES = NE * TQ, TPW = (TILES + NW - 1) / NW;   // 32 x 32 results; of a wave
    static constexpr int RING = NBUF * STAGE, RED = BQ * PITCH * 4;
    static constexpr int LDS = (RING > RED ? RING : RED) + 2 * NW * 8;
    static_assert(WCH % NW == 0 && NBUF >= 2 && LDS <= 160 * 1024, "router stages");
};

// at most N of this wave's loads outstanding, and none of its LDS reads
template <int N>
__device__ __forceinline__ void router_wait() {
    __builtin_amdgcn_s_waitcnt((N & 15) | (7 << 4) | (0 << 8) | ((N >> 4) << 14));
}

template <class C, typename IdxT>
__global__ void __launch_bounds__(C::NT)
router_gate_kernel(int T, int d, int E, int K, const bf16_t *__restrict__ x, const bf16_t *__restrict__ Wr,
                   const float *__restrict__ bias, const IdxT *__restrict__ idx, int64_t stride,
                   float *__restrict__ gates, float *__restrict__ logits_out, unsigned long long *agree,
                   int32_t *status) {
    extern __shared__ __attribute__((aligned(1024))) char lds[];
    constexpr int SK = C::SK, XG = C::BQ / 16;
    const int lane = lane_id(), wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int t0 = blockIdx.x * C::BQ;
    const uint32_t base = lds_addr(lds);
    // W_r chunk c (1 KB): k-rows 8 (c % (SK / 8)) .. + 7 of expert tile c / (SK / 8), eight 16-byte pieces each.
    // (k-rows past d are past the end of W_r and read zero)
    const Src sw = Src{(const char *)Wr, (uint64_t)d * E * 2, (uint32_t)(SK * E * 2)};
    int woff[C::WPW];
#pragma unroll
    for (int i = 0; i < C::WPW; ++i) {
        const int ch = wave + C::NW * i, k = ch % (SK / 8) * 8 + (lane >> 3), p = lane & 7;
        const int e = ch / (SK / 8) * 64 + (((((p >> 2) ^ (k >> 1)) & 1) << 2) | (p & 3)) * 8;
        woff[i] = e < E ? (k * E + e) * 2 : kOutsideWindow;
    }
    // x chunk c: tokens 16 (c % XG) .. + 15 of k-tile c / XG, four pieces each, piece p of token r at p ^ ((r >> 2) & 3)
    const Src sx = Src{(const char *)(x + (int64_t)t0 * d), clamp_bytes((int64_t)(T - t0) * d * 2), (uint32_t)(SK * 2)};
    int xoff[C::XPW], xk[C::XPW];
#pragma unroll
    for (int i = 0; i < C::XPW; ++i) {
        const int ch = wave + C::NW * i;
        xk[i] = ch / XG * 32 + ((lane & 3) ^ ((lane >> 4) & 3)) * 8;   // (bits 2,3 of the token are bits 4,5 of the lane)
        xoff[i] = ((ch % XG * 16 + (lane >> 2)) * d + xk[i]) * 2;
    }
    auto issue = [&](int it, int buf) {
        const uint32_t dst = base + buf * C::STAGE + 1024 * wave;
        const rsrc_t rw = src_rsrc(sw, it), rx = src_rsrc(sx, it);
#pragma unroll
        for (int i = 0; i < C::WPW; ++i) lds_load16(rw, dst + 1024 * C::NW * i, woff[i]);
#pragma unroll
        for (int i = 0; i < C::XPW; ++i)
            if (i + 1 < C::XPW || wave < C::XLAST)   // (k past d: the next token's values in memory)
                lds_load16(rx, dst + C::WT + 1024 * C::NW * i, it * SK + xk[i] < d ? xoff[i] : kOutsideWindow);
    };
    // fragment addresses: W_r by the transposing read (see TrFrag), x rows as KcFrag<32>
    const int b = lane >> 4, i16 = lane & 15;
    const int wrow = (8 * (b >> 1) + (i16 >> 2)) * 128 + (i16 & 1) * 8;   // + 4 k-rows: the upper half of the 8 k
    const int wsub = (2 * (b & 1) + ((i16 & 3) >> 1)) * 16, wsw = (i16 >> 3) & 1;
    KcFrag<32> xf;
    xf.init(0, lane);
    f32x16_t acc[C::TPW];
#pragma unroll
    for (int i = 0; i < C::TPW; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.0f;

    const int nit = (d + SK - 1) / SK;
#pragma unroll
    for (int p = 0; p < C::NBUF - 1; ++p) issue(p, p);
    int buf = 0;
    for (int it = 0; it < nit; ++it) {
        asm volatile("" ::: "memory");
        // this stage is in when only the loads of the later ones are outstanding
        if (C::XLAST == C::NW || wave < C::XLAST) router_wait<(C::NBUF - 2) * (C::WPW + C::XPW)>();
        else router_wait<(C::NBUF - 2) * (C::WPW + C::XPW - 1)>();
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        // the buffer asked for now is the one read last time round: those reads are over
        issue(it + C::NBUF - 1, buf == 0 ? C::NBUF - 1 : buf - 1);
        const char *wt = lds + buf * C::STAGE, *xt = wt + C::WT;
        if (wave < C::TILES) {
#pragma unroll
            for (int s = 0; s < SK / 16; ++s)
#pragma unroll
                for (int i = 0; i < C::TPW; ++i) {
                    const int id = wave + C::NW * i, e = id % C::NE, q = id / C::NE;
                    if (C::TILES % C::NW != 0 && id >= C::TILES) continue;
                    // bit 1 of the k-row is that of i16 >> 2 (rows 8 (b >> 1), + 4 and 16 s do not change it)
                    const char *p = wt + (e >> 1) * (SK * 128) + s * 16 * 128 + wrow + ((e ^ wsw) & 1) * 64 + wsub;
                    const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p));
                    const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4_ptr)(p + 4 * 128));
                    const bf16x8_t a = __builtin_bit_cast(bf16x8_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                    acc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, xf.read(xt + (s >> 1) * (C::BQ * 64), q, s & 1), acc[i], 0, 0, 0);
                }
        }
        buf = buf == C::NBUF - 1 ? 0 : buf + 1;
    }
    router_wait<0>();   // no load may land in what follows
    __syncthreads();
    float *red = (float *)lds;
#pragma unroll
    for (int i = 0; i < C::TPW; ++i) {
        const int id = wave + C::NW * i, e = id % C::NE, q = id / C::NE;
        if (id >= C::TILES) continue;
#pragma unroll
        for (int g = 0; g < 4; ++g)
            *(float4 *)(red + (32 * q + (lane & 31)) * C::PITCH + 32 * e + 8 * g + 4 * (lane >> 5)) =
                make_float4(acc[i][4 * g], acc[i][4 * g + 1], acc[i][4 * g + 2], acc[i][4 * g + 3]);
    }
    __syncthreads();
    if (bias || logits_out) {
        add_logits<1, C::BQ, C::EP, C::NT>(red, C::PITCH, t0, T, E, bias, logits_out);
        __syncthreads();
    }
    gate_from_lds<C::NE, C::NT, IdxT>(red, C::PITCH, t0, C::BQ, T, E, K, idx, stride, gates, agree, status,
                                      (unsigned long long *)(lds + C::LDS - 2 * 8 * C::NW));
}

// ---------------------------------------------------------------------------
// The same for E = 128 and many tokens: 128 tokens per work-group, so that W_r is streamed a quarter as often, and two
// work-groups per compute unit, so that one's gates and prologue hide behind the other's loads.  k is walked in
// sequence, two k-tiles ahead.
// ---------------------------------------------------------------------------
typedef TileCfg<128, 128, 2, 2, 64> TLGate;   // 128 experts x 128 tokens
template <typename IdxT>
__global__ void __launch_bounds__(TLGate::NT, 2)
router_gate_many_kernel(int T, int d, int K, const bf16_t *__restrict__ x, const bf16_t *__restrict__ Wr,
                        const float *__restrict__ bias, const IdxT *__restrict__ idx, int64_t stride,
                        float *__restrict__ gates, float *__restrict__ logits_out, unsigned long long *agree,
                        int32_t *status) {
    typedef TLGate TL;
    constexpr int E = TL::BP, PITCH = E + 4;   // floats per LDS row (the pad spreads rows over the banks)
    extern __shared__ __attribute__((aligned(16))) char lds[];
    __shared__ unsigned long long part[2 * TL::NWAVES];
    const int t0 = blockIdx.x * TL::BQ;
    auto fp = [&](int kt, int k, int c) -> uint4 { return ld16(Wr + (int64_t)(kt * TL::BK + k) * E + c * 8); };
    auto fq = [&](int kt, int r, int c) -> uint4 {
        return ld16(x + (int64_t)min(t0 + r, T - 1) * d + kt * TL::BK + c * 8);
    };
    f32x16_t acc[TL::TP][TL::TQ];
    zero_acc<TL>(acc);
    mfma_mainloop_ahead2<TL, true, false>(acc, d / TL::BK, fp, fq, lds);   // ends with a barrier: the stages are free
    float *sl = (float *)lds;
    for_each_quad<TL>([&](int tp, int tq, int g, int p, int q) {
        float4 v = make_float4(acc[tp][tq][4 * g], acc[tp][tq][4 * g + 1], acc[tp][tq][4 * g + 2], acc[tp][tq][4 * g + 3]);
        if (bias) {
            const float4 b = *(const float4 *)(bias + p);
            v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
        }
        *(float4 *)(sl + q * PITCH + p) = v;
    });
    __syncthreads();
    if (logits_out)   // whole rows, 16 bytes per lane
        for (int i = threadIdx.x; i < TL::BQ * (E / 4); i += TL::NT) {
            const int q = i / (E / 4), c = i % (E / 4);
            if (t0 + q < T) *(float4 *)(logits_out + (int64_t)(t0 + q) * E + 4 * c) = *(const float4 *)(sl + q * PITCH + 4 * c);
        }
    gate_from_lds<E / 32, TL::NT, IdxT>(sl, PITCH, t0, TL::BQ, T, E, K, idx, stride, gates, agree, status, part);
}

// ---------------------------------------------------------------------------
// f32 arithmetic, any d, E <= 128, both activation types: 16 tokens per work-group, 8 waves that take every 8th step of
// 16 k.  Both operands go straight from global memory into fragments of the 16x16x4 instruction (a lane's four k
// of a step are neighbours in x; W_r rows are read 16 experts at a time, out of cache).
// ---------------------------------------------------------------------------
template <int NE, bool VEC, typename T, typename IdxT>
__global__ void __launch_bounds__(512)
plain_gate_kernel(int Tn, int d, int E, int K, const T *__restrict__ x, const T *__restrict__ Wr,
                  const float *__restrict__ bias, const IdxT *__restrict__ idx, int64_t stride, float *__restrict__ gates,
                  float *__restrict__ logits_out, unsigned long long *agree, int32_t *status) {
    constexpr int EP = NE < 2 ? 32 : 16 * NE, PITCH = EP + 4;   // (agreement reads rows in pieces of 32)
    __shared__ __attribute__((aligned(16))) float red[8 * 16 * PITCH];
    __shared__ unsigned long long part[16];
    typedef float f32x4_t __attribute__((ext_vector_type(4)));
    const int lane = lane_id(), wave = threadIdx.x >> 6, r16 = lane & 15, k4 = 4 * (lane >> 4);
    const int t0 = blockIdx.x * 16;
    const T *xr = x + (int64_t)min(t0 + r16, Tn - 1) * d;
    f32x4_t acc[NE];
#pragma unroll
    for (int e = 0; e < NE; ++e) acc[e] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
    const int nst = (d + 127) / 128;
    for (int it = 0; it < nst; ++it) {
        const int k = (it * 8 + wave) * 16 + k4;
        float xv[4] = {0.0f, 0.0f, 0.0f, 0.0f}, wv[NE][4];
        if constexpr (VEC) {   // d is a multiple of four
            if (k < d) {
                if constexpr (sizeof(T) == 4) {
                    const float4 v = *(const float4 *)(xr + k);
                    xv[0] = v.x; xv[1] = v.y; xv[2] = v.z; xv[3] = v.w;
                } else {
                    const uint2 u = *(const uint2 *)(xr + k);
                    xv[0] = __uint_as_float(u.x << 16); xv[1] = __uint_as_float(u.x & 0xffff0000u);
                    xv[2] = __uint_as_float(u.y << 16); xv[3] = __uint_as_float(u.y & 0xffff0000u);
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (k + i < d) xv[i] = Elem<T>::ld(xr + k + i);
        }
#pragma unroll
        for (int e = 0; e < NE; ++e)
#pragma unroll
            for (int i = 0; i < 4; ++i)
                wv[e][i] = k + i < d && 16 * e + r16 < E ? Elem<T>::ld(Wr + (int64_t)(k + i) * E + 16 * e + r16) : 0.0f;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < NE; ++e) acc[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(wv[e][i], xv[i], acc[e], 0, 0, 0);
    }
#pragma unroll
    for (int e = 0; e < NE; ++e)
        *(float4 *)(red + (wave * 16 + r16) * PITCH + 16 * e + k4) = make_float4(acc[e][0], acc[e][1], acc[e][2], acc[e][3]);
    __syncthreads();
    add_logits<8, 16, 16 * NE, 512>(red, PITCH, t0, Tn, E, bias, logits_out);
    __syncthreads();
    gate_from_lds<(NE + 1) / 2, 512, IdxT>(red, PITCH, t0, 16, Tn, E, K, idx, stride, gates, agree, status, part);
}

// ---------------------------------------------------------------------------
// Router weight gradient dW_r[c][e] = sum_t x[t][c] ds[t][e], in parts over the tokens.  ds has K entries in a row of E:
// it is never in memory.  A work-group (128 hidden columns x 128 experts, 64 tokens per k-tile) keeps its ds tile in
// LDS, takes the old tile's entries out and puts the new one's in, each as a hi and a lo bf16 (dz to about 16 bits) in
// columns that meet in one lane's accumulators.  A token's entries belong to one wave, whose clearing and setting are
// in order.  Two work-groups per compute unit; x comes in two k-tiles ahead.  Bound by the read of x and, for few
// tokens, the parts.  With ds in memory as [T][2E] and hi and lo parts written apart, us with the sum of the parts:
// T=65536 d=2048 E=128 K=8 142 -> 109, T=16384 52 -> 44, T=1001 26 -> 17, T=6000 d=1024 E=384 K=4 54 -> 28; half or twice
// the work-groups: 145 / 123 at 65536 tokens, 48 / 56 at 16384.  The kernel that made ds: 28 -> 14 us at T=65536.
// ---------------------------------------------------------------------------
constexpr int kDwrQ = 128, kDwrP = 128, kDwrK = 64;
constexpr int kDwrPBytes = kDwrK * 2 * kDwrP * 2, kDwrQBytes = kDwrK * kDwrQ * 2, kDwrLds = kDwrPBytes + 2 * kDwrQBytes;

// EPT = 8, K > 16: too many registers for two k-tiles ahead and for what to take out again.  x and the first 8 entries come
// one k-tile ahead (those past 8, K > 32, while the tile is made), and a wave clears its tokens' rows (8 KB) instead.
// T=16384 d=2048 E=128, us on the f32 tiles, which such layers took for a while | here: K=17 762 | 50, K=24 905 | 54, K=32 1088 | 59,
// K=64 1816 | 90.
template <int EPT, typename IdxT>   // EPT: entries per thread and k-tile, 4 EPT >= K (or 8)
__global__ void __launch_bounds__(256, 2)
router_dwr_kernel(int T, int d, int E, int K, int rows, const bf16_t *__restrict__ x, const float *__restrict__ dz,
                  const IdxT *__restrict__ idx, int64_t stride, float *__restrict__ part) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int npt = (E + kDwrP - 1) / kDwrP, nqt = (d + kDwrQ - 1) / kDwrQ;
    const int sp = blockIdx.x / (npt * nqt), rem = blockIdx.x - sp * npt * nqt;
    const int qt = rem / npt, q0 = qt * kDwrQ, p0 = (rem - qt * npt) * kDwrP;
    const int r0 = sp * rows, r1 = min(T, r0 + rows), nk = (r1 - r0 + kDwrK - 1) / kDwrK;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wp = wave & 1, wq = wave >> 1;
    char *const pt = lds, *const qs = lds + kDwrPBytes;
    constexpr bool kMany = EPT > 4;
    constexpr int kSets = kMany ? 1 : 2;   // k-tiles on their way
    uint4 rq[kSets][4];
    int eid[kSets][EPT];
    float ez[kSets][EPT];
    // entry n of the wave's 16 tokens: token n / K of them (by a multiplication: n < 1024, K <= 64), position n % K
    const int inv_k = (65536 + K - 1) / K;
    auto token = [&](int n) { return (n * inv_k) >> 16; };
    auto eload = [&](int kt, int first, auto &id, auto &z) {
        constexpr int N = sizeof(id) / sizeof(id[0]);
        const int t0 = r0 + kt * kDwrK + 16 * wave, live = max(0, min(16, r1 - t0)) * K;
        const float *zb = dz + (int64_t)t0 * K;
        const IdxT *ib = idx + (int64_t)t0 * stride;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int n = first + lane + 64 * i, t = token(n);
            id[i] = -1;
            z[i] = 0.0f;
            if (n < live) {
                id[i] = min((int)ib[t * stride + n - t * K], E - 1) - p0;
                z[i] = zb[n];
            }
        }
    };
    auto gload = [&](int kt, int set) {
        const int t0 = r0 + kt * kDwrK;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = tid + 256 * i, t = t0 + n / 16, c = q0 + n % 16 * 8;
            rq[set % kSets][i] = t < r1 && c < d ? ld16(x + (int64_t)t * d + c) : zero16();
        }
        if constexpr (!kMany) eload(kt, 0, eid[set % kSets], ez[set % kSets]);
    };
    int old[EPT];
#pragma unroll
    for (int i = 0; i < EPT; ++i) old[i] = -1;
    // expert e's hi half is column (e / 64) * 128 + e % 64, its lo half 64 columns on (128 bytes, a bit of the offset)
    auto eset = [&](int first, const auto &id, const auto &z) {
        constexpr int N = sizeof(id) / sizeof(id[0]);
#pragma unroll
        for (int i = 0; i < N; ++i) {
            if constexpr (!kMany) old[i] = -1;
            if (id[i] >= 0 && id[i] < kDwrP) {
                const int k = 16 * wave + token(first + lane + 64 * i);
                const int c = (id[i] >> 6) * 128 + (id[i] & 63);
                const int at = tr_off<2 * kDwrP>(k, c >> 3) + (c & 7) * 2;
                const bf16_t hi = f32_to_bf16(z[i]);
                *(bf16_t *)(pt + at) = hi;
                *(bf16_t *)(pt + (at ^ 128)) = f32_to_bf16(z[i] - bf16_to_f32(hi));
                if constexpr (!kMany) old[i] = at;
            }
        }
    };
    auto put = [&](int kt, int stage) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int n = tid + 256 * i;
            *(uint4 *)(qs + stage * kDwrQBytes + tr_off<kDwrQ>(n / 16, n % 16)) = rq[stage % kSets][i];
        }
        if constexpr (kMany) {
#pragma unroll
            for (int i = 0; i < 8; ++i) ((uint4 *)(pt + wave * (kDwrPBytes / 4)))[lane + 64 * i] = zero16();
            asm volatile("" ::: "memory");
            eset(0, eid[0], ez[0]);
#pragma unroll 1
            for (int n = EPT * 64; n < 16 * K; n += EPT * 64) {
                int id[EPT];
                float z[EPT];
                eload(kt, n, id, z);
                eset(n, id, z);
            }
        } else {
#pragma unroll
            for (int i = 0; i < EPT; ++i)
                if (old[i] >= 0) {
                    *(bf16_t *)(pt + old[i]) = 0;
                    *(bf16_t *)(pt + (old[i] ^ 128)) = 0;
                }
            asm volatile("" ::: "memory");
            eset(0, eid[stage % kSets], ez[stage % kSets]);
        }
    };
    TrFrag<2 * kDwrP> pf;
    TrFrag<kDwrQ> qf;
    pf.init(wp * 128);
    qf.init(wq * 64);
    f32x16_t acc[4][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.0f;
    auto multiply = [&](int stage) {
#pragma unroll
        for (int s = 0; s < kDwrK / 16; ++s) {
            bf16x8_t a[4], b[2];
#pragma unroll
            for (int i = 0; i < 4; ++i) a[i] = pf.read(pt, i, s);
#pragma unroll
            for (int j = 0; j < 2; ++j) b[j] = qf.read(qs + stage * kDwrQBytes, j, s);
#pragma unroll
            for (int i = 0; i < 4; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };
    for (int i = tid; i < kDwrPBytes / 16; i += 256) ((uint4 *)pt)[i] = zero16();
    if constexpr (kMany) {
        for (int kt = -1; kt < nk; ++kt) {
            eload(kt + 1, 0, eid[0], ez[0]);
            gload(kt + 1, 0);
            if (kt >= 0) multiply(kt & 1);
            __syncthreads();
            put(kt + 1, (kt + 1) & 1);
            __syncthreads();
        }
    } else {
        gload(0, 0);
        gload(1, 1);
        __syncthreads();
        put(0, 0);
        __syncthreads();
        for (int kt = 0; kt < nk; kt += 2) {
            gload(kt + 2, 0);
            multiply(0);
            __syncthreads();
            put(kt + 1, 1);
            __syncthreads();
            if (kt + 1 < nk) {
                gload(kt + 3, 1);
                multiply(1);
                __syncthreads();
                put(kt + 2, 0);
                __syncthreads();
            }
        }
    }
    float *o = part + (int64_t)sp * d * E;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const int e = p0 + wp * 64 + i * 32 + g * 8 + (lane >> 5) * 4, c = q0 + wq * 64 + j * 32 + (lane & 31);
                float v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = acc[i][j][4 * g + u] + acc[i + 2][j][4 * g + u];
                if (c >= d) continue;
                float *at = o + (int64_t)c * E + e;
                if (E % 4 == 0) {
                    if (e < E) *(float4 *)at = make_float4(v[0], v[1], v[2], v[3]);
                } else {
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        if (e + u < E) at[u] = v[u];
                }
            }
}

// The router's last step (r3_finish.h) where no other launch takes it in: step by step f32 layers and the plain kernels.
template <typename T>
__global__ void __launch_bounds__(1024) router_finish_kernel(RouterFinish<T> a) {
    __shared__ RouterFinishLds<T> lds;
    router_finish_block<1024>(a, blockIdx.x, lds);
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
namespace {

template <int EP, int TQ, typename IdxT>
void launch_router(int T, int d, int E, int K, const void *x, const void *Wr, const float *bias, const void *idx,
                   int64_t stride, float *gates, float *logits_out, int64_t *agree, int32_t *status, hipStream_t s) {
    typedef RouterCfg<EP, TQ> C;
    auto k = router_gate_kernel<C, IdxT>;
    (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, C::LDS);
    k<<<(T + C::BQ - 1) / C::BQ, C::NT, C::LDS, s>>>(T, d, E, K, (const bf16_t *)x, (const bf16_t *)Wr, bias, (const IdxT *)idx,
                                                   stride, gates, logits_out, (unsigned long long *)agree, status);
}

template <int NE, bool VEC, typename T, typename IdxT>
void launch_plain(int Tn, int d, int E, int K, const void *x, const void *Wr, const float *bias, const void *idx,
                  int64_t stride, float *gates, float *logits_out, int64_t *agree, int32_t *status, hipStream_t s) {
    plain_gate_kernel<NE, VEC, T, IdxT><<<(Tn + 15) / 16, 512, 0, s>>>(Tn, d, E, K, (const T *)x, (const T *)Wr, bias,
                                                                 (const IdxT *)idx, stride, gates, logits_out,
                                                                 (unsigned long long *)agree, status);
}

template <typename IdxT>
void router_by_size(int T, int d, int E, int K, const void *x, const void *Wr, const float *bias, const void *idx,
                    int64_t stride, float *gates, float *logits_out, int64_t *agree, int32_t *status, hipStream_t s) {
    // d = 2048, us at 32 tokens per work-group / 64 (/ E = 128: the kernel for many).  Both are at their best as long as
    // every work-group has a compute unit of its own:
    //   tokens    E=64         E=128                  E=256        E=384        E=512
    //     4096    8.8 / 10.2    9.9 /  13.0 /  29.1   18.2 / 21.4  23.9 / 30.7  30.5 / 38.3
    //     8192    9.0 / 10.8   10.9 /  14.8 /  29.6   20.1 / 21.7  26.0 / 33.3  35.5 / 40.4
    //    12000   16.4 / 11.5   19.2 /  15.9 /  29.6   36.5 / 22.3  47.5 / 33.9  65.8 / 40.5
    //    32768   35.5 / 25.2   39.0 /  33.7 /  35.6   74.6 / 47.3  96.7 / 71.3   136 / 87.5
    //    65536   67.5 / 53.3   86.1 /  66.5 /  48.2    158 / 96.2   194 /  146   267 /  175
    //   131072    161 /  126    207 /   150 /   137    384 /  214   402 /  308   610 /  370
    // (24576 tokens, E=128: 30.3 / 32.3 / 32.1)
    constexpr int kCus = 256;
    const bool wide = T > 32 * kCus;
    if (T > 128 * kCus && E == 128 && d % 64 == 0) {
        constexpr int LDS = std::max(TLGate::LDS_BYTES, TLGate::BQ * (TLGate::BP + 4) * 4);
        (void)hipFuncSetAttribute((const void *)router_gate_many_kernel<IdxT>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
        router_gate_many_kernel<IdxT><<<(T + TLGate::BQ - 1) / TLGate::BQ, TLGate::NT, LDS, s>>>(
            T, d, K, (const bf16_t *)x, (const bf16_t *)Wr, bias, (const IdxT *)idx, stride, gates, logits_out,
            (unsigned long long *)agree, status);
        return;
    }
#define R3_ROUTER(EP)                                                                                            \
    (wide ? launch_router<EP, 2, IdxT> : launch_router<EP, 1, IdxT>)(T, d, E, K, x, Wr, bias, idx, stride, gates, \
                                                                     logits_out, agree, status, s)
    if (E <= 64) R3_ROUTER(64);
    else if (E <= 128) R3_ROUTER(128);
    else if (E <= 256) R3_ROUTER(256);
    else if (E <= 384) R3_ROUTER(384);
    else R3_ROUTER(512);
#undef R3_ROUTER
}

template <typename T, typename IdxT>
void plain_by_size(int Tn, int d, int E, int K, const void *x, const void *Wr, const float *bias, const void *idx,
                   int64_t stride, float *gates, float *logits_out, int64_t *agree, int32_t *status, hipStream_t s) {
    const bool vec = d % 4 == 0;
    auto f = E <= 16   ? (vec ? launch_plain<1, true, T, IdxT> : launch_plain<1, false, T, IdxT>)
             : E <= 32 ? (vec ? launch_plain<2, true, T, IdxT> : launch_plain<2, false, T, IdxT>)
             : E <= 64 ? (vec ? launch_plain<4, true, T, IdxT> : launch_plain<4, false, T, IdxT>)
                       : (vec ? launch_plain<8, true, T, IdxT> : launch_plain<8, false, T, IdxT>);
    f(Tn, d, E, K, x, Wr, bias, idx, stride, gates, logits_out, agree, status, s);
}

}  // namespace

static bool bf16_dwr(int act, int d, bool plain_only) { return act == R3_BF16 && d % 8 == 0 && !plain_only; }
// tokens per part: whole k-tiles, and enough parts for two work-groups on every compute unit
static int dwr_rows(int T, int d, int E) {
    const int64_t tiles = (int64_t)((d + kDwrQ - 1) / kDwrQ) * ((E + kDwrP - 1) / kDwrP), kts = (T + kDwrK - 1) / kDwrK;
    const int64_t ns = std::max<int64_t>(1, std::min<int64_t>(kts, 512 / tiles));
    return (int)((kts + ns - 1) / ns * kDwrK);
}

size_t router_dwr_ws_bytes(int act, int T, int d, int E, bool plain_only) {
    return align_up((size_t)router_dwr_nparts(act, T, d, E, plain_only) * d * E * sizeof(float), 256);
}

template <typename IdxT>
static void launch_dwr(int T, int d, int E, int K, const void *x, const float *dz, const void *idx, int64_t stride,
                       float *part, hipStream_t s) {
    const int rows = dwr_rows(T, d, E);
    const int grid = (T + rows - 1) / rows * ((d + kDwrQ - 1) / kDwrQ) * ((E + kDwrP - 1) / kDwrP);
    auto k = K <= 4 ? router_dwr_kernel<1, IdxT> : K <= 8 ? router_dwr_kernel<2, IdxT> : K <= 16 ? router_dwr_kernel<4, IdxT>
                                                                                     : router_dwr_kernel<8, IdxT>;
    k<<<grid, 256, kDwrLds, s>>>(T, d, E, K, rows, (const bf16_t *)x, dz, (const IdxT *)idx, stride, part);
}

int router_dwr_nparts(int act, int T, int d, int E, bool plain_only) {
    const int rows = bf16_dwr(act, d, plain_only) ? dwr_rows(T, d, E) : plain_dwr_rows(T, d, E);
    return (T + rows - 1) / rows;
}
hipError_t router_dwr_parts(int T, int d, int E, int K, int act, const void *x, const float *dz, const void *idx, int idx_dtype, int64_t stride,
                            float *part, bool plain_only, hipStream_t s) {
    ProfScope ps(PROF_DWR, s);
    if (bf16_dwr(act, d, plain_only)) (idx_dtype == R3_IDX_U8 ? launch_dwr<uint8_t> : launch_dwr<uint16_t>)(T, d, E, K, x, dz, idx, stride, part, s);
    else plain_dwr_parts(T, d, E, K, act, x, dz, idx, idx_dtype, stride, part, s);
    return hipGetLastError();
}

hipError_t router_backward(int T, int d, int E, int K, int act, const void *x, const void *Wr, const float *dz, const void *idx,
                           int idx_dtype, int64_t stride, const int32_t *offsets, const float *dzrow, float *part, float *dWr,
                           float *dbias, void *WrT, int accumulate, bool plain_only, hipStream_t s) {
    const hipError_t rc = router_dwr_parts(T, d, E, K, act, x, dz, idx, idx_dtype, stride, part, plain_only, s);
    if (rc != hipSuccess) return rc;
    ProfScope ps(PROF_DWR, s);
    auto finish = [&](auto f) {
        const int blocks = f.template fill<1024>(d, E, router_dwr_nparts(act, T, d, E, plain_only), accumulate, dzrow, part, offsets, dbias, dWr,
                                                 Wr, WrT);
        router_finish_kernel<<<blocks, 1024, 0, s>>>(f);
        return hipGetLastError();
    };
    return act == R3_BF16 ? finish(RouterFinish<bf16_t>{}) : finish(RouterFinish<float>{});
}

bool router_gate_supported(int act, int d, int E, bool plain_only) {
    if (act == R3_BF16 && !plain_only && d % 8 == 0 && E % 8 == 0 && E <= 512) return true;
    return E <= 128;
}

hipError_t router_gate(int T, int d, int E, int K, int act, const void *x, const void *Wr, const float *bias, const void *idx,
                       int idx_dtype, int64_t stride, float *gates, float *logits_out, int64_t *agree, int32_t *status,
                       bool plain_only, hipStream_t s) {
    ProfScope ps(PROF_GATE, s);
    const bool u8 = idx_dtype == R3_IDX_U8;
    if (act == R3_BF16 && !plain_only && d % 8 == 0 && E % 8 == 0 && E <= 512) {
        auto f = u8 ? router_by_size<uint8_t> : router_by_size<uint16_t>;
        f(T, d, E, K, x, Wr, bias, idx, stride, gates, logits_out, agree, status, s);
    } else {
        auto f = act == R3_BF16 ? (u8 ? plain_by_size<bf16_t, uint8_t> : plain_by_size<bf16_t, uint16_t>)
                                : (u8 ? plain_by_size<float, uint8_t> : plain_by_size<float, uint16_t>);
        f(T, d, E, K, x, Wr, bias, idx, stride, gates, logits_out, agree, status, s);
    }
    return hipGetLastError();
}

}  // namespace r3
