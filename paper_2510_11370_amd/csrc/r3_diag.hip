// Discrepancy diagnostics of Section 3 of arxiv 2510.11370 as HBM-bound reductions:
//   routing differences between two records (Section 3.2: router, token and sequence level),
//   k3 estimate of KL(pi_train || pi_infer) and the extreme-token fraction F(tau) (Section 3.1).
// Counts are integers (atomics on integers commute, so every result is reproducible); the one
// floating-point sum is reduced in a fixed order through per-block partials.
#include <cmath>

#include "r3_kernels.h"

namespace r3 {
namespace {

constexpr int kMaxTau = 8;
constexpr int kDiagBlocks = 1024;    // policy partials; one thread each in the final sum
constexpr int kPolicyThreads = 512;
constexpr int kMaxDiffBlocks = 1024;

constexpr int kDiffTok = 128;      // tokens of one work-group's tile
constexpr int kDiffThreads = 512;

// number of ids of a[0..K) that do not occur in b[0..K) (sets of distinct ids, any order)
template <typename IdxT>
__device__ __forceinline__ int differing(const IdxT *a, const IdxT *b, int K) {
    int common = 0;
    for (int i = 0; i < K; ++i) {
        const IdxT v = a[i];
        bool hit = false;
        for (int j = 0; j < K; ++j) hit |= (b[j] == v);
        common += hit;
    }
    return K - common;
}

// One router's K ids in registers, fetched in loads of U bytes.
template <typename IdxT, int K, int U> struct IdSet {
    static constexpr int kBytes = K * (int)sizeof(IdxT), kWords = (kBytes + 3) / 4, kPer = 4 / (int)sizeof(IdxT);
    uint32_t w[kWords];
    __device__ __forceinline__ void load(const IdxT *p) {
        if constexpr (U == 16) {
            const uint4 v = *(const uint4 *)p;
            w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
        } else if constexpr (U == 8) {
            const uint2 v = *(const uint2 *)p;
            w[0] = v.x; w[1] = v.y;
        } else if constexpr (U == 4) {
#pragma unroll
            for (int i = 0; i < kWords; ++i) w[i] = ((const uint32_t *)p)[i];
        } else {
#pragma unroll
            for (int i = 0; i < kWords; ++i) {
                const uint32_t lo = ((const uint16_t *)p)[2 * i];
                w[i] = 2 * i + 1 < kBytes / 2 ? lo | ((uint32_t)((const uint16_t *)p)[2 * i + 1] << 16) : lo;
            }
        }
    }
    __device__ __forceinline__ bool operator!=(const IdSet &o) const {
        uint32_t x = 0;
#pragma unroll
        for (int i = 0; i < kWords; ++i) x |= w[i] ^ o.w[i];
        return x != 0;
    }
    __device__ __forceinline__ uint32_t rep(int i) const {   // id i in every field of a word
        constexpr uint32_t kMask = sizeof(IdxT) == 1 ? 0xffu : 0xffffu, kOne = sizeof(IdxT) == 1 ? 0x01010101u : 0x00010001u;
        return ((w[i / kPer] >> (i % kPer * (8 * (int)sizeof(IdxT)))) & kMask) * kOne;
    }
    // ids of *this that o does not hold: each is looked up with the zero-field test on o ^ (id in every field);
    // fields past K hold o's last id
    __device__ __forceinline__ int differing_from(IdSet o) const {
        constexpr uint32_t kOne = sizeof(IdxT) == 1 ? 0x01010101u : 0x00010001u, kTop = kOne << (8 * sizeof(IdxT) - 1);
        if constexpr (kBytes % 4 != 0) o.w[kWords - 1] |= o.rep(K - 1) << (8 * (kBytes % 4));
        int common = 0;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            const uint32_t r = rep(i);
            uint32_t hit = 0;
#pragma unroll
            for (int j = 0; j < kWords; ++j) {
                const uint32_t x = o.w[j] ^ r;
                hit |= (x - kOne) & ~x & kTop;
            }
            common += hit != 0;
        }
        return K - common;
    }
};

// A work-group takes tiles of kDiffTok tokens x all layers.  The set comparison proper costs about 100 vector
// instructions a router, and with one router in ten different nearly every wave met one and paid them all: 24 of the
// 35 us that two 48 x 131072 x 8 records took.  So a wave only tests for equal words, and moves the sets that differ
// into a queue of its own in LDS, 64 of which are compared at a time.  The routers of a tile are dealt to the lanes
// in the order of the record's addresses (tokens first, or layers first in a token-major record), six in flight.
// K = 0: sets of any size and alignment, compared element by element in place (the queue holds their positions).
// 48 x 131072 x 8 one-byte ids: 35.5 -> 24.5 us.
template <typename IdxT, int K, int U>
__global__ void __launch_bounds__(kDiffThreads)
routing_diff_kernel(int T, int Krt, int L, const IdxT *__restrict__ a, const IdxT *__restrict__ b,
                    int64_t token_stride, int64_t layer_stride, unsigned long long *__restrict__ router_hist,
                    int32_t *__restrict__ token_choices, int32_t *__restrict__ token_routers) {
    constexpr int kUnroll = 6, kWaves = kDiffThreads / kWave, kQueue = 2 * kWave;
    constexpr bool kRegs = K > 0;
    typedef IdSet<IdxT, kRegs ? K : 4, kRegs ? U : 2> Set;
    constexpr int kQWords = kRegs ? 2 * Set::kWords : 1;
    __shared__ int hist[kMaxK + 1], choices[kDiffTok], routers[kDiffTok];
    __shared__ uint32_t q_set[kWaves][kQWords][kQueue];
    __shared__ int q_tok[kWaves][kQueue];
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int Kn = kRegs ? K : Krt;
    for (int i = threadIdx.x; i <= Kn; i += kDiffThreads) hist[i] = 0;
    // a lane's next router is `dtok` tokens and `dl` layers on; in token-major records the layer wraps
    const bool wrap = layer_stride < token_stride;
    const int dtok = wrap ? kDiffThreads / L : 0, dl = wrap ? kDiffThreads % L : kDiffThreads / kDiffTok;
    for (int64_t tile = blockIdx.x; tile * kDiffTok < T; tile += gridDim.x) {
        const int t0 = (int)(tile * kDiffTok), nt = min(kDiffTok, T - t0);
        if (threadIdx.x < kDiffTok) choices[threadIdx.x] = routers[threadIdx.x] = 0;
        __syncthreads();
        int tok = wrap ? (int)threadIdx.x / L : (int)threadIdx.x % kDiffTok;
        int l = wrap ? (int)threadIdx.x % L : (int)threadIdx.x / kDiffTok;
        int queued = 0;                                  // the same in every lane
        auto compare = [&](int e) {                      // queue entry e of this wave
            int d, tk;
            if constexpr (kRegs) {
                Set x, y;
#pragma unroll
                for (int i = 0; i < Set::kWords; ++i) {
                    x.w[i] = q_set[w][i][e];
                    y.w[i] = q_set[w][Set::kWords + i][e];
                }
                d = x.differing_from(y);
                tk = q_tok[w][e];
            } else {
                tk = q_tok[w][e];
                const int64_t o = (int64_t)q_set[w][0][e] * layer_stride + (int64_t)(t0 + tk) * token_stride;
                d = differing(a + o, b + o, Kn);
            }
            if (d > 0) {
                atomicAdd(&hist[d], 1);
                atomicAdd(&choices[tk], d);
                atomicAdd(&routers[tk], 1);
            }
        };
        while (__any(tok < nt && l < L)) {
            Set x[kUnroll], y[kUnroll];
            int tk[kUnroll], ll[kUnroll];
            bool ne[kUnroll];
#pragma unroll
            for (int i = 0; i < kUnroll; ++i) {
                const bool in = tok < nt && l < L;
                const int64_t o = in ? (int64_t)l * layer_stride + (int64_t)(t0 + tok) * token_stride
                                     : (int64_t)t0 * token_stride;   // a router of the tile, read and not counted
                tk[i] = tok;
                ll[i] = l;
                ne[i] = in;
                if constexpr (kRegs) {
                    x[i].load(a + o);
                    y[i].load(b + o);
                } else {
                    bool diff = false;
                    for (int k = 0; k < Kn; ++k) diff |= a[o + k] != b[o + k];
                    ne[i] = in && diff;
                }
                tok += dtok;
                l += dl;
                if (wrap && l >= L) {
                    l -= L;
                    ++tok;
                }
            }
#pragma unroll
            for (int i = 0; i < kUnroll; ++i) {
                if constexpr (kRegs) ne[i] = ne[i] && x[i] != y[i];
                const unsigned long long m = __ballot(ne[i]);
                if (m == 0) continue;
                if (ne[i]) {
                    const int e = queued + __popcll(m & ((1ull << lane) - 1));
                    if constexpr (kRegs) {
#pragma unroll
                        for (int j = 0; j < Set::kWords; ++j) {
                            q_set[w][j][e] = x[i].w[j];
                            q_set[w][Set::kWords + j][e] = y[i].w[j];
                        }
                    } else {
                        q_set[w][0][e] = (uint32_t)ll[i];
                    }
                    q_tok[w][e] = tk[i];
                }
                queued += __popcll(m);
                if (queued >= kWave) {
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                    queued -= kWave;
                    compare(queued + lane);
                    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        if (lane < queued) compare(lane);
        __syncthreads();
        if ((int)threadIdx.x < nt) {
            token_choices[t0 + threadIdx.x] = choices[threadIdx.x];
            token_routers[t0 + threadIdx.x] = routers[threadIdx.x];
            if (routers[threadIdx.x] < L) atomicAdd(&hist[0], L - routers[threadIdx.x]);
        }
        __syncthreads();
    }
    for (int i = threadIdx.x; i <= Kn; i += kDiffThreads)
        if (hist[i]) atomicAdd(&router_hist[i], (unsigned long long)hist[i]);
}

// One thread per token, its layers in a loop: for records of few layers, which do not fill the other kernel's work-groups
// (and a quarter of the work-groups adds to the histogram).
template <typename IdxT, int K, int U>
__global__ void __launch_bounds__(256)
routing_diff_tokens_kernel(int T, int Krt, int L, const IdxT *__restrict__ a, const IdxT *__restrict__ b,
                           int64_t token_stride, int64_t layer_stride, unsigned long long *__restrict__ router_hist,
                           int32_t *__restrict__ token_choices, int32_t *__restrict__ token_routers) {
    constexpr bool kRegs = K > 0;
    typedef IdSet<IdxT, kRegs ? K : 4, kRegs ? U : 2> Set;
    __shared__ int hist[kMaxK + 1];
    const int Kn = kRegs ? K : Krt;
    for (int i = threadIdx.x; i <= Kn; i += 256) hist[i] = 0;
    __syncthreads();
    const int t = blockIdx.x * 256 + threadIdx.x;
    int choices = 0, routers = 0;
    if (t < T)
        for (int l = 0; l < L; ++l) {
            const int64_t o = (int64_t)l * layer_stride + (int64_t)t * token_stride;
            int d;
            if constexpr (kRegs) {
                Set x, y;
                x.load(a + o);
                y.load(b + o);
                d = x != y ? x.differing_from(y) : 0;
            } else {
                d = differing(a + o, b + o, Kn);
            }
            if (d > 0) {
                choices += d;
                ++routers;
                atomicAdd(&hist[d], 1);
            }
        }
    const int same = wave_sum(t < T ? L - routers : 0);
    if (lane_id() == 0 && same) atomicAdd(&hist[0], same);
    if (t < T) {
        token_choices[t] = choices;
        token_routers[t] = routers;
    }
    __syncthreads();
    for (int i = threadIdx.x; i <= Kn; i += 256)
        if (hist[i]) atomicAdd(&router_hist[i], (unsigned long long)hist[i]);
}

// W waves per sequence: exact integer sum of the tokens' differing routers, one division.  One wave walking a
// sequence of 2048 tokens is 32 round trips to memory in a row (11 us); sixteen waves make it two (4.2 us).
template <int W>
__global__ void __launch_bounds__(W == 1 ? 256 : W * kWave)
sequence_mean_kernel(int nseq, const int32_t *__restrict__ seq_offsets, const int32_t *__restrict__ token_routers,
                     double *__restrict__ seq_mean) {
    const int s = W == 1 ? blockIdx.x * (256 / kWave) + threadIdx.x / kWave : blockIdx.x;
    if (s >= nseq) return;
    const int lo = seq_offsets[s], hi = seq_offsets[s + 1];
    long long sum = 0;
    for (int64_t t = (int64_t)lo + (W == 1 ? lane_id() : (int)threadIdx.x); t < hi; t += W * kWave) sum += token_routers[t];
    sum = wave_sum(sum);
    if constexpr (W > 1) {
        __shared__ long long part[W];
        if (lane_id() == 0) part[threadIdx.x / kWave] = sum;
        __syncthreads();
        sum = 0;
        for (int i = 0; i < W; ++i) sum += part[i];
        if (threadIdx.x == 0) seq_mean[s] = hi > lo ? (double)sum / (double)(hi - lo) : 0.0;
    } else {
        if (lane_id() == 0) seq_mean[s] = hi > lo ? (double)sum / (double)(hi - lo) : 0.0;
    }
}

// e^d - 1 - d = d^2 (1/2! + d/3! + d^2/4! + ...): for |d| <= 0.5 the series through d^14/16! is
// exact to double rounding (next term < 3e-19 of the first) and free of the cancellation that
// e^d - 1 - d suffers for small d; beyond, expm1(d) - d.  Most tokens have |log r| << 0.5, and the
// library expm1 alone kept this reduction at 3 percent of the memory rate.
__device__ __forceinline__ double k3_term(double d) {
    if (fabs(d) > 0.5) return expm1(d) - d;
    constexpr double c[15] = {5.00000000000000000e-01, 1.66666666666666657e-01, 4.16666666666666644e-02, 8.33333333333333322e-03, 1.38888888888888894e-03, 1.98412698412698413e-04, 2.48015873015873016e-05, 2.75573192239858925e-06, 2.75573192239858883e-07, 2.50521083854417202e-08, 2.08767569878681002e-09, 1.60590438368216133e-10, 1.14707455977297245e-11, 7.64716373181981641e-13, 4.77947733238738525e-14};
    double p = c[14];
#pragma unroll
    for (int k = 13; k >= 0; --k) p = fma(p, d, c[k]);
    return d * d * p;
}

struct TauArgs {
    float log_tau[kMaxTau];   // float(log(double(tau))); +inf beyond ntau
};

struct PolicyPartial {
    double k3;
    unsigned long long over[kMaxTau];
};

// log r = logp_train - logp_infer.  k3 term e^d - 1 - d in double (for |d| ~ 1e-3 the term is
// d^2/2 and would lose most of its digits in float), see k3_term(); the threshold test
// |log r| > log tau is taken in float on the float difference.  The next four
// elements of each array are in flight while four are evaluated, eight waves on a SIMD, NT counters at most.  (Counting with population counts of the compare masks on the scalar unit was slower:
// 36 us.)  10 M tokens: 24.6 -> 22.3 us.
template <int NT>
__global__ void __launch_bounds__(kPolicyThreads)
policy_partial_kernel(int64_t n, const float *__restrict__ lt, const float *__restrict__ li, TauArgs taus,
                      PolicyPartial *__restrict__ part) {
    constexpr int kWaves = kPolicyThreads / kWave;
    double k3 = 0.0;
    int over[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) over[i] = 0;
    auto one = [&](float a, float b) {
        const double d = (double)a - (double)b;
        k3 += k3_term(d);
        const float ad = fabsf(a - b);
#pragma unroll
        for (int j = 0; j < NT; ++j) over[j] += ad > taus.log_tau[j];
    };
    // 16-byte loads when both arrays allow it (the order of a thread's terms is fixed either way)
    const bool vec = (((uintptr_t)lt | (uintptr_t)li) & 15) == 0;
    const int64_t n4 = vec ? n / 4 : 0;
    const int64_t stride = (int64_t)gridDim.x * kPolicyThreads;
    int64_t i = (int64_t)blockIdx.x * kPolicyThreads + threadIdx.x;
    if (i < n4) {
        float4 a = ((const float4 *)lt)[i], b = ((const float4 *)li)[i];
        for (;;) {
            i += stride;
            const int64_t next = i < n4 ? i : n4 - 1;      // the last round fetches a pair it does not use
            const float4 an = ((const float4 *)lt)[next], bn = ((const float4 *)li)[next];
            one(a.x, b.x);
            one(a.y, b.y);
            one(a.z, b.z);
            one(a.w, b.w);
            if (i >= n4) break;
            a = an;
            b = bn;
        }
    }
    for (i = 4 * n4 + (int64_t)blockIdx.x * kPolicyThreads + threadIdx.x; i < n; i += stride) one(lt[i], li[i]);
    __shared__ double sk[kWaves];
    __shared__ int so[kWaves][kMaxTau];
    const int w = threadIdx.x / kWave;
    k3 = wave_sum(k3);
#pragma unroll
    for (int j = 0; j < NT; ++j) over[j] = wave_sum(over[j]);
    if (lane_id() == 0) {
        sk[w] = k3;
#pragma unroll
        for (int j = 0; j < kMaxTau; ++j) so[w][j] = j < NT ? over[j < NT ? j : 0] : 0;
    }
    __syncthreads();
    if (threadIdx.x < 1 + kMaxTau) {
        double s = 0.0;
        unsigned long long c = 0;
        for (int i = 0; i < kWaves; ++i) {
            s += sk[i];
            if (threadIdx.x > 0) c += (unsigned long long)so[i][threadIdx.x - 1];
        }
        if (threadIdx.x == 0) part[blockIdx.x].k3 = s;
        else part[blockIdx.x].over[threadIdx.x - 1] = c;
    }
}

// fixed-order sum of the block partials, one thread each: lanes by wave_sum's tree, then the waves in order
__global__ void __launch_bounds__(kDiagBlocks)
policy_final_kernel(int64_t n, int nblocks, int ntau, const PolicyPartial *__restrict__ part, double *__restrict__ kl,
                    double *__restrict__ frac) {
    constexpr int kWaves = kDiagBlocks / kWave;
    __shared__ double sk[kWaves];
    __shared__ unsigned long long so[kWaves][kMaxTau];
    const int b = threadIdx.x, w = b / kWave;
    const double s = wave_sum(b < nblocks ? part[b].k3 : 0.0);
    unsigned long long c[kMaxTau];
#pragma unroll
    for (int j = 0; j < kMaxTau; ++j) c[j] = j < ntau ? wave_sum(b < nblocks ? part[b].over[j] : 0ull) : 0ull;
    if (lane_id() == 0) {
        sk[w] = s;
#pragma unroll
        for (int j = 0; j < kMaxTau; ++j) so[w][j] = c[j];
    }
    __syncthreads();
    if (b == 0) {
        double t = 0.0;
        for (int i = 0; i < kWaves; ++i) t += sk[i];
        *kl = n > 0 ? t / (double)n : 0.0;
    } else if (b <= ntau) {
        unsigned long long t = 0;
        for (int i = 0; i < kWaves; ++i) t += so[i][b - 1];
        frac[b - 1] = n > 0 ? (double)t / (double)n : 0.0;
    }
}

}  // namespace

size_t policy_ws_bytes() { return align_up((size_t)kDiagBlocks * sizeof(PolicyPartial), 256); }
int policy_max_tau() { return kMaxTau; }

hipError_t launch_routing_diff(int T, int K, int L, const void *a, const void *b, int idx_dtype, int64_t token_stride,
                               int64_t layer_stride, const int32_t *seq_offsets, int nseq, int64_t *router_hist,
                               int32_t *token_choices, int32_t *token_routers, double *seq_mean, hipStream_t s) {
    // sets whose size and addresses allow whole loads are kept in registers, others are compared in place
    const int ib = idx_dtype == R3_IDX_U8 ? 1 : 2;
    auto fits = [&](int U) {
        return (token_stride * ib) % U == 0 && (layer_stride * ib) % U == 0 && (uintptr_t)a % U == 0 && (uintptr_t)b % U == 0;
    };
    const int tiles = (T + kDiffTok - 1) / kDiffTok;
    const int grid = tiles < kMaxDiffBlocks ? tiles : kMaxDiffBlocks;
    // Where a thread per token is the faster one, us per token / by tiles, K=8 one-byte ids: T=131072 one layer 8.5 / 17.1, eight
    // 10.8 / 18.0, 24 layers 20.2 / 21.5 (two-byte ids 22.5 / 24.9), 48 layers 36 / 24.5; T=4096 eight 7.3 / 7.3, 24 layers
    // 12.8 / 7.3; token-major T=131072 eight 12.0 / 18.0, twelve 16.5 / 18.0 (two-byte ids 28.6 / 19.9).  Compared in place, K=12: T=131072 one
    // layer 13.1 / 30.6, four 27.7 / 31.1, six 38.5 / 31.3; T=64 two layers 11.1 / 11.2, three 16.0 / 12.4.
    const bool many = T >= 65536, token_major = layer_stride < token_stride && L > 1;
    auto few_layers = [&](bool regs) {
        if (regs) return L <= 8 || (many && (token_major ? L <= 12 && L * K * ib <= 96 : L <= 24));
        return K * L <= 24 || (many && !token_major && (K * L <= 48 || L == 1));
    };
#define R3_DIFF(TT, KK, UU)                                                                                            \
    (few_layers(KK > 0) ? routing_diff_tokens_kernel<TT, KK, UU> : routing_diff_kernel<TT, KK, UU>)                      \
        <<<few_layers(KK > 0) ? (T + 255) / 256 : grid, few_layers(KK > 0) ? 256 : kDiffThreads, 0, s>>>(               \
            T, K, L, (const TT *)a, (const TT *)b, token_stride, layer_stride, (unsigned long long *)router_hist,       \
            token_choices, token_routers)
    {
        ProfScope ps(PROF_ROUTING_DIFF, s);
        if (ib == 1) {
            if (K == 8 && fits(8)) R3_DIFF(uint8_t, 8, 8);
            else if (K == 6 && fits(2)) R3_DIFF(uint8_t, 6, 2);
            else if (K == 4 && fits(4)) R3_DIFF(uint8_t, 4, 4);
            else if (K == 2 && fits(2)) R3_DIFF(uint8_t, 2, 2);
            else R3_DIFF(uint8_t, 0, 0);
        } else {
            if (K == 8 && fits(16)) R3_DIFF(uint16_t, 8, 16);
            else if (K == 6 && fits(4)) R3_DIFF(uint16_t, 6, 4);
            else if (K == 4 && fits(8)) R3_DIFF(uint16_t, 4, 8);
            else if (K == 2 && fits(4)) R3_DIFF(uint16_t, 2, 4);
            else R3_DIFF(uint16_t, 0, 0);
        }
    }
#undef R3_DIFF
    if (seq_mean && nseq > 0) {
        // sequences of 512 tokens and more on average take a work-group each, shorter ones a wave
        if (T / nseq >= 512)
            sequence_mean_kernel<16><<<nseq, 16 * kWave, 0, s>>>(nseq, seq_offsets, token_routers, seq_mean);
        else
            sequence_mean_kernel<1><<<(nseq + 3) / 4, 256, 0, s>>>(nseq, seq_offsets, token_routers, seq_mean);
    }
    return hipGetLastError();
}

hipError_t launch_policy_discrepancy(int64_t n, const float *lt, const float *li, int ntau, const float *tau_host,
                                     double *kl, double *frac, void *ws, hipStream_t s) {
    PolicyPartial *part = (PolicyPartial *)ws;
    TauArgs taus;
    for (int i = 0; i < kMaxTau; ++i) taus.log_tau[i] = i < ntau ? (float)log((double)tau_host[i]) : INFINITY;
    int64_t want = (n + 4 * kPolicyThreads - 1) / (4 * kPolicyThreads);
    const int blocks = (int)(want < 1 ? 1 : (want > kDiagBlocks ? kDiagBlocks : want));
    ProfScope ps(PROF_POLICY, s);
    // two of the dozen or so vector instructions per element and threshold are spent on each counter
    switch ((ntau + 1) / 2) {
        case 0: case 1: policy_partial_kernel<2><<<blocks, kPolicyThreads, 0, s>>>(n, lt, li, taus, part); break;
        case 2: policy_partial_kernel<4><<<blocks, kPolicyThreads, 0, s>>>(n, lt, li, taus, part); break;
        case 3: policy_partial_kernel<6><<<blocks, kPolicyThreads, 0, s>>>(n, lt, li, taus, part); break;
        default: policy_partial_kernel<8><<<blocks, kPolicyThreads, 0, s>>>(n, lt, li, taus, part); break;
    }
    policy_final_kernel<<<1, kDiagBlocks, 0, s>>>(n, blocks, ntau, part, kl, frac);
    return hipGetLastError();
}

}  // namespace r3
