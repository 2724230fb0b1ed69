// Routing kernels of the replayed MoE layer (arxiv 2510.11370, Section 4.1):
// TopKMask record, replay gate, dispatch permutation, weighted combine, and the
// element-wise parts of the backward.  All of them are bound by HBM traffic, so
// they move 16-byte vectors per lane, read every input once and use wave-level
// reductions; none uses floating-point atomics (results are bit-reproducible).
#include <algorithm>

#include <type_traits>

#include "r3_finish.h"
#include "r3_kernels.h"
#include "r3_tiles.h"
#include "r3_topk.h"

namespace r3 {

// ---------------------------------------------------------------------------
// TopKMask
// ---------------------------------------------------------------------------
// General record: one wave per token, rank counting, E <= 4096, K <= 64.
// key of element e beats key of element f if larger, or equal with lower id.
template <typename IdxT>
__global__ void __launch_bounds__(256)
record_topk_wave_kernel(int T, int E, int K, const float *__restrict__ logits, int64_t ld,
                        IdxT *__restrict__ idx, int64_t stride, int32_t *status) {
    extern __shared__ uint32_t keys_all[];
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int t = blockIdx.x * 4 + w;
    uint32_t *keys = keys_all + w * E;
    bool bad = false;
    if (t < T)
        for (int e = lane; e < E; e += kWave) {
            bool nf;
            keys[e] = order_key(logits[(int64_t)t * ld + e], nf);
            bad |= nf;
        }
    __syncthreads();
    if (t >= T) return;
    int emitted = 0;  // wave-uniform
    for (int base = 0; base < E; base += kWave) {
        int e = base + lane;
        bool sel = false;
        if (e < E) {
            uint32_t mine = keys[e];
            int ahead = 0;
            for (int f = 0; f < E; ++f) {
                uint32_t kf = keys[f];
                ahead += (kf > mine || (kf == mine && f < e)) ? 1 : 0;
            }
            sel = ahead < K;
        }
        uint64_t m = __ballot(sel);
        if (sel) {
            int pos = emitted + __popcll(m & ((1ull << lane) - 1ull));
            idx[(int64_t)t * stride + pos] = (IdxT)e;
        }
        emitted += __popcll(m);
    }
    if (__ballot(bad) && lane == 0 && status) atomicOr(status, R3_DATA_NONFINITE);
}

// K <= 8, E <= 32 NV <= 512: 8 lanes per token (8 tokens per wave), one pass over the row.  Lane `sub` of a token holds the
// keys of ids 32 i + 4 sub + c (i < NV, c < 4: one 128-byte segment per token per load instruction), and after the
// merges the ids above the threshold and equal to it are E-bit masks, OR-ed over the 8 lanes (topk_mask8).
// Lane `sub` writes the sub-th set bit, so the K ids land ascending in one segment.  VEC: rows are whole 16-byte
// pieces; FULL: E = 32 NV as well (T=131072 E=256 K=8: 29.5 us without the guards, 32.3 with).  Bound by the read of the logits; with one id at a time per lane and three passes over the row
// E=384 took 37 us at 6000 tokens, 9.8 now.
template <typename IdxT, int NV, bool VEC, bool FULL>
__global__ void __launch_bounds__(256)
record_topk_vec_kernel(int T, int E, int K, const float *__restrict__ logits, int64_t ld, IdxT *__restrict__ idx,
                       int64_t stride, int32_t *status) {
    const int t = blockIdx.x * 32 + (int)(threadIdx.x >> 3);
    const int sub = threadIdx.x & 7;
    const bool live = t < T;
    const float *row = logits + (int64_t)(live ? t : 0) * ld;
    uint32_t key[NV][4];
    bool bad = false;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        const int e = 32 * i + 4 * sub;
        float v[4] = {0.0f, 0.0f, 0.0f, 0.0f};
        if constexpr (VEC) {
            if (FULL || e < E) {
                const float4 q = *(const float4 *)(row + e);
                v[0] = q.x; v[1] = q.y; v[2] = q.z; v[3] = q.w;
            }
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
                if (e + c < E) v[c] = row[e + c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            bool nf;
            const uint32_t k = order_key(v[c], nf);
            // (ids that do not exist rank with the NaNs, behind every real one of that rank)
            key[i][c] = FULL || e + c < E ? k : 0u;
            bad |= nf;
        }
    }
    uint32_t gt[NV];
    topk_mask8<NV>(key, K, sub, gt);
    // lane `sub` emits the sub-th selected id
    int want = sub, id = -1;
#pragma unroll
    for (int i = 0; i < NV; ++i) {
        uint32_t w = gt[i];
        const int c = __popc(w);
        if (id < 0) {
            if (want < c) {
                for (int j = 0; j < want; ++j) w &= w - 1u;
                id = 32 * i + __ffs((int)w) - 1;
            } else {
                want -= c;
            }
        }
    }
    if (live) {
        if (sub < K && id >= 0) idx[(int64_t)t * stride + sub] = (IdxT)id;
        if (bad && status) atomicOr(status, R3_DATA_NONFINITE);
    }
}

template <typename IdxT>
static bool launch_record_vec(int T, int E, int K, const float *logits, int64_t ld, IdxT *idx, int64_t stride,
                              int32_t *status, hipStream_t s) {
    if (K > 8 || E > 512) return false;
    const bool vec = E % 4 == 0 && ld % 4 == 0 && ((uintptr_t)logits & 15) == 0;
#define R3_RECORD(NV)                                                                            \
    (vec ? (E == 32 * NV ? record_topk_vec_kernel<IdxT, NV, true, true> : record_topk_vec_kernel<IdxT, NV, true, false>) \
         : record_topk_vec_kernel<IdxT, NV, false, false>)
    auto k = E <= 32 ? R3_RECORD(1) : E <= 64 ? R3_RECORD(2) : E <= 128 ? R3_RECORD(4) : E <= 256 ? R3_RECORD(8)
             : E <= 384 ? R3_RECORD(12) : R3_RECORD(16);
#undef R3_RECORD
    k<<<(T + 31) / 32, 256, 0, s>>>(T, E, K, logits, ld, idx, stride, status);
    return true;
}

hipError_t launch_record_topk(int T, int E, int K, const float *logits, int64_t ld, void *idx,
                              int idx_dtype, int64_t stride, int32_t *status, hipStream_t s) {
    ProfScope ps(PROF_RECORD, s);
    if (idx_dtype == R3_IDX_U8 ? launch_record_vec(T, E, K, logits, ld, (uint8_t *)idx, stride, status, s)
                               : launch_record_vec(T, E, K, logits, ld, (uint16_t *)idx, stride, status, s))
        return hipGetLastError();
    {
        size_t lds = (size_t)4 * E * sizeof(uint32_t);
        int grid = (T + 3) / 4;
        if (idx_dtype == R3_IDX_U8)
            record_topk_wave_kernel<uint8_t><<<grid, 256, lds, s>>>(T, E, K, logits, ld, (uint8_t *)idx,
                                                                   stride, status);
        else
            record_topk_wave_kernel<uint16_t><<<grid, 256, lds, s>>>(T, E, K, logits, ld,
                                                                    (uint16_t *)idx, stride, status);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Replay gate from logits in memory: one thread per token.
// g_j = exp(s[idx_j] - m) / sum_i exp(s[idx_i] - m), m = max over the set.
// ---------------------------------------------------------------------------
template <typename IdxT>
__global__ void __launch_bounds__(256)
gate_kernel(int T, int E, int K, const float *__restrict__ logits, const IdxT *__restrict__ idx,
            int64_t stride, float *__restrict__ gates, int32_t *status) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= T) return;
    const IdxT *id = idx + (int64_t)t * stride;
    const float *row = logits + (int64_t)t * E;
    float m = -INFINITY;
    int bad = 0;
    for (int j = 0; j < K; ++j) {
        int e = (int)id[j];
        if (e >= E) {
            bad |= R3_DATA_IDX_RANGE;
            e = E - 1;
        }
        const float z = row[e];
        if (!(fabsf(z) <= 3.4028235e38f)) bad |= R3_DATA_NONFINITE;
        m = fmaxf(m, z);
    }
    float den = 0.0f;
    for (int j = 0; j < K; ++j) {
        int e = min((int)id[j], E - 1);
        float p = expf(row[e] - m);
        gates[(int64_t)t * K + j] = p;
        den += p;
    }
    float inv = 1.0f / den;
    for (int j = 0; j < K; ++j) gates[(int64_t)t * K + j] *= inv;
    if (bad && status) atomicOr(status, bad);
}

hipError_t launch_gate(int T, int E, int K, const float *logits, const void *idx, int idx_dtype,
                       int64_t stride, float *gates, int32_t *status, hipStream_t s) {
    ProfScope ps(PROF_GATE, s);
    int grid = (T + 255) / 256;
    if (idx_dtype == R3_IDX_U8)
        gate_kernel<uint8_t><<<grid, 256, 0, s>>>(T, E, K, logits, (const uint8_t *)idx, stride, gates, status);
    else
        gate_kernel<uint16_t><<<grid, 256, 0, s>>>(T, E, K, logits, (const uint16_t *)idx, stride, gates, status);
    return hipGetLastError();
}

// Routing agreement (Section 3.2, router level): per token compare the top-K
// set of the training logits with the recorded set.  A wave takes a token at a
// time: its E order keys sit in the wave's LDS strip, and for each recorded
// expert all 64 lanes count the keys ahead of it (one ballot per 64 experts).
// A wave walks many tokens and a block adds its totals once: agree[0] += tokens
// with equal sets, agree[1] += shared experts.  Integer atomics only.
template <typename IdxT>
__global__ void __launch_bounds__(256)
agreement_kernel(int T, int E, int K, const float *__restrict__ logits, const IdxT *__restrict__ idx,
                 int64_t stride, unsigned long long *agree) {
    extern __shared__ uint32_t keys_all[];
    __shared__ unsigned long long part[4][2];
    const int w = threadIdx.x / kWave, lane = lane_id();
    uint32_t *keys = keys_all + w * E;
    unsigned long long equal = 0, common = 0;
    for (int t = blockIdx.x * 4 + w; t < T; t += gridDim.x * 4) {
        for (int e = lane; e < E; e += kWave) {
            bool nf;
            keys[e] = order_key(logits[(int64_t)t * E + e], nf);
        }
        // one wave's LDS writes are complete before its later LDS reads
        __builtin_amdgcn_s_waitcnt(0);
        __builtin_amdgcn_wave_barrier();
        int shared = 0;
        for (int j = 0; j < K; ++j) {
            const int e = min((int)idx[(int64_t)t * stride + j], E - 1);
            const uint32_t mine = keys[e];
            int ahead = 0;
            for (int f0 = 0; f0 < E; f0 += kWave) {
                const int f = f0 + lane;
                const uint32_t kf = f < E ? keys[f] : 0u;
                const bool before = f < E && (kf > mine || (kf == mine && f < e));
                ahead += __popcll(__ballot(before));
            }
            shared += ahead < K;
        }
        common += (unsigned long long)shared;
        equal += shared == K;
        __builtin_amdgcn_wave_barrier();   // the strip is rewritten for the next token
    }
    if (lane == 0) {
        part[w][0] = equal;
        part[w][1] = common;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        unsigned long long a0 = 0, a1 = 0;
        for (int i = 0; i < 4; ++i) {
            a0 += part[i][0];
            a1 += part[i][1];
        }
        if (a1) atomicAdd(agree + 1, a1);
        if (a0) atomicAdd(agree, a0);
    }
}

hipError_t launch_agreement(int T, int E, int K, const float *logits, const void *idx, int idx_dtype,
                            int64_t stride, int64_t *agree, hipStream_t s) {
    ProfScope ps(PROF_AGREEMENT, s);
    size_t lds = (size_t)4 * E * sizeof(uint32_t);
    int grid = (T + 3) / 4;
    if (grid > 2048) grid = 2048;
    if (idx_dtype == R3_IDX_U8)
        agreement_kernel<uint8_t><<<grid, 256, lds, s>>>(T, E, K, logits, (const uint8_t *)idx, stride,
                                                        (unsigned long long *)agree);
    else
        agreement_kernel<uint16_t><<<grid, 256, lds, s>>>(T, E, K, logits, (const uint16_t *)idx, stride,
                                                         (unsigned long long *)agree);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Dispatch permutation: stable counting sort of the T*K slots by expert.  The placement never depends on arrival
// order, so perm is unique.
//
// Up to 1024 experts (dispatch_kernel): a work-group owns a chunk of slots, 64 per wave and step, and needs for every
// expert the slots before its chunk and in all.  It finds them itself, without waiting for another work-group:
// it counts all ids (LDS atomics; they are one or two bytes each, read as 16-byte vectors out of L2), or, when
// that would be too many, adds up the chunk counts a first launch has left.  The expert GEMMs' tile table and
// the per-row gates come out of the same launch where the caller wants them.  Bound by
// latency: r3_permute, K=8 E=128, took 26.5 us at T=1001 and 55.6 at T=131072 in three dependent launches (count, scan,
// place), 9.3 in one and 28.1 in two; the tile table was a fourth.
// Beyond 1024 experts: three launches (count per chunk, scan over the chunks, place).
// ---------------------------------------------------------------------------
// A wave's chunk is walked 64 slots at a time, kPermBatch such steps per batch: the ids of a whole
// batch are fetched before any of them is used, so the wave pays one memory round trip per batch
// instead of one per step.
constexpr int kPermBatch = 16;
// slot -> (token, position) in 32-bit arithmetic (T*K < 2^31), a shift when K is a power of two:
// a 64-bit division by a run-time K is some hundred instructions, and these kernels did two per slot
struct SlotSplit {
    int K, shift;
    __device__ __forceinline__ explicit SlotSplit(int K_) : K(K_), shift((K_ & (K_ - 1)) == 0 ? __ffs(K_) - 1 : -1) {}
    __device__ __forceinline__ void operator()(int sl, int &t, int &j) const {
        if (shift >= 0) {
            t = sl >> shift;
            j = sl & (K - 1);
        } else {
            t = (int)((unsigned)sl / (unsigned)K);
            j = sl - t * K;
        }
    }
};
constexpr int kWaitLds = 15 | (7 << 4) | (0 << 8) | (3 << 14);   // s_waitcnt lgkmcnt(0): LDS only, not the stores

constexpr int kDispWaves = 16, kDispMaxE = 1024;
constexpr int kDispStep = 64 * kDispWaves;       // slots a work-group takes per step
struct DispatchArgs {
    int T, E, K, steps, nchunks;
    int64_t stride;
    const int32_t *chunk_hist;                   // [nchunks][E] slots per chunk and expert (HIST only)
    int32_t *counts, *offsets, *inv_perm, *perm, *status;
    DispatchExtra x;
};

// sum over the lanes up to and with this one
__device__ __forceinline__ int wave_scan(int v) {
    const int lane = lane_id();
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int u = __shfl_up(v, o, kWave);
        if (lane >= o) v += u;
    }
    return v;
}
// the same over a block of 1024 threads; `tmp`: 16 ints of LDS
__device__ __forceinline__ int block_scan(int v, int32_t *tmp) {
    const int w = threadIdx.x >> 6;
    v = wave_scan(v);
    __syncthreads();
    if (lane_id() == kWave - 1) tmp[w] = v;
    __syncthreads();
    for (int i = 0; i < w; ++i) v += tmp[i];
    return v;
}

// slots per expert of every chunk
template <typename IdxT>
__global__ void __launch_bounds__(1024)
dispatch_count_kernel(int T, int E, int K, const IdxT *__restrict__ idx, int64_t stride, int steps,
                      int32_t *__restrict__ chunk_hist) {
    extern __shared__ int32_t sm[];
    for (int e = threadIdx.x; e < E; e += 1024) sm[e] = 0;
    __syncthreads();
    const int S = T * K, s0 = blockIdx.x * steps * kDispStep;
    const SlotSplit split(K);
    for (int i = 0; i < steps; i += 4) {
        int ev[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int sl = s0 + (i + u) * kDispStep + threadIdx.x;
            int t, j;
            split(min(sl, S - 1), t, j);
            ev[u] = i + u < steps && sl < S ? min((int)idx[(int64_t)t * stride + j], E - 1) : -1;
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (ev[u] >= 0) atomicAdd(&sm[ev[u]], 1);
    }
    __syncthreads();
    for (int e = threadIdx.x; e < E; e += 1024) chunk_hist[(int64_t)blockIdx.x * E + e] = sm[e];
}

template <typename IdxT, bool HIST>
__global__ void __launch_bounds__(1024)
dispatch_kernel(const IdxT *__restrict__ idx, DispatchArgs a) {
    extern __shared__ int32_t sm[];
    const int E = a.E, K = a.K, S = a.T * K;
    int32_t *cnt = sm, *before = sm + kDispWaves * E, *after = before + E, *tmp = after + E;   // cnt: [wave][E]
    const int w = threadIdx.x >> 6, lane = lane_id(), c = blockIdx.x;
    const bool table = c == a.nchunks;            // the last work-group (if asked for) only makes the tile table
    const int chunk = a.steps * kDispStep;
    const int s0 = c * chunk + w * a.steps * 64;  // this wave's slots
    const SlotSplit split(K);
    for (int i = threadIdx.x; i < (kDispWaves + 2) * E; i += 1024) sm[i] = 0;
    __syncthreads();
    auto fetch = [&](int step) -> int {           // this lane's id of a step, -1 past the end
        const int sl = s0 + step * 64 + lane;
        if (step >= a.steps || sl >= S) return -1;
        int t, j;
        split(sl, t, j);
        return (int)idx[(int64_t)t * a.stride + j];
    };
    // this wave's counts, and the checks of its ids
    int first = -1;                               // the first step's id is kept for the placement
    if (!table) {
        // a token's K ids sit in K neighbouring lanes of one step when K divides 64: the duplicate check
        // compares lanes then, instead of loading ids again
        const bool lanes_hold_token = 64 % K == 0;
        int bad = 0;
        for (int i = 0; i < a.steps; i += 4) {
            int ev[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) ev[u] = fetch(i + u);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                int e = ev[u];
                const bool live = e >= 0;
                if (live && e >= E) {
                    bad |= R3_DATA_IDX_RANGE;
                    e = E - 1;
                }
                if (i == 0 && u == 0) first = e;
                if (lanes_hold_token) {
                    const int j = lane % K;       // (a wave's steps start at multiples of 64)
                    for (int back = 1; back < K; ++back) {
                        const int other = __shfl(e, lane - back);
                        if (live && back <= j && other == e) bad |= R3_DATA_IDX_DUP;
                    }
                } else if (live) {
                    int t, j;
                    split(s0 + (i + u) * 64 + lane, t, j);
                    for (int jj = 0; jj < j; ++jj)
                        if (min((int)idx[(int64_t)t * a.stride + jj], E - 1) == e) bad |= R3_DATA_IDX_DUP;
                }
                if (live) atomicAdd(&cnt[w * E + e], 1);
            }
        }
        if (bad && a.status) atomicOr(a.status, bad);
    }
    // slots before this chunk, and from it on, per expert
    if constexpr (HIST) {
        int Ep = 1;
        while (Ep < E) Ep <<= 1;
        const int e = threadIdx.x % Ep, g = threadIdx.x / Ep, G = 1024 / Ep;
        int b = 0, f = 0;
        if (e < E)
            for (int q = g; q < a.nchunks; q += 8 * G) {
                int h[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) h[u] = q + u * G < a.nchunks ? a.chunk_hist[(int64_t)(q + u * G) * E + e] : 0;
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    b += q + u * G < c ? h[u] : 0;
                    f += q + u * G < c ? 0 : h[u];
                }
            }
        if (b) atomicAdd(&before[e], b);
        if (f) atomicAdd(&after[e], f);
    } else if (a.stride == K && ((uintptr_t)idx & 15) == 0) {
        constexpr int PER = 16 / sizeof(IdxT);    // ids per vector (chunks start at multiples of it)
        const int nv = S / PER, cv = c * chunk / PER;
        for (int v0 = threadIdx.x; v0 < nv; v0 += 4 * 1024) {
            uint4 d[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) d[u] = v0 + u * 1024 < nv ? ((const uint4 *)idx)[v0 + u * 1024] : make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (v0 + u * 1024 >= nv) break;
                int32_t *to = v0 + u * 1024 < cv ? before : after;
                const uint32_t q[4] = {d[u].x, d[u].y, d[u].z, d[u].w};
#pragma unroll
                for (int i = 0; i < PER; ++i)
                    atomicAdd(&to[min((int)((q[i * sizeof(IdxT) / 4] >> (8 * sizeof(IdxT) * (i % (4 / sizeof(IdxT))))) &
                                            (sizeof(IdxT) == 1 ? 0xffu : 0xffffu)), E - 1)], 1);
            }
        }
        for (int sl = nv * PER + threadIdx.x; sl < S; sl += 1024)
            atomicAdd(&(sl < c * chunk ? before : after)[min((int)idx[sl], E - 1)], 1);
    } else {
        for (int i = threadIdx.x; i < S; i += 8 * 1024) {
            int ev[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                int t, j;
                split(min(i + u * 1024, S - 1), t, j);
                ev[u] = min((int)idx[(int64_t)t * a.stride + j], E - 1);
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (i + u * 1024 < S) atomicAdd(&(i + u * 1024 < c * chunk ? before : after)[ev[u]], 1);
        }
    }
    __syncthreads();
    // offsets, and where every wave's slots of an expert start
    const int e = threadIdx.x;
    const int bef = e < E ? before[e] : 0, n = e < E ? bef + after[e] : 0;
    const int off = block_scan(n, tmp) - n;
    if (e < E) {
        int run = off + bef;
#pragma unroll
        for (int i = 0; i < kDispWaves; ++i) {
            const int h = cnt[i * E + e];
            cnt[i * E + e] = run;
            run += h;
        }
        if (c == 0) {
            a.counts[e] = n;
            a.offsets[e] = off;
            if (e == E - 1) a.offsets[E] = off + n;
        }
    }
    if (table) {
        int32_t *tiles = a.x.tiles;
        const int nt = (n + kRowTile - 1) / kRowTile;
        const int end = block_scan(nt, tmp), start = end - nt;
        for (int i = 0; i < nt; ++i) {
            tiles[kTileHdr + 2 * (start + i)] = e;
            tiles[kTileHdr + 1 + 2 * (start + i)] = off + i * kRowTile;
        }
        if (threadIdx.x < 64) tiles[2 + threadIdx.x] = 0;
        if (threadIdx.x == 1023) {
            tiles[0] = end;
            for (int x = 0; x <= 8; ++x) tiles[kTileX + x] = (int)(((int64_t)end * x) >> 3);
        }
        return;
    }
    __syncthreads();
    int ebits = 1;
    while ((1 << ebits) < E) ++ebits;
    const uint64_t lt = (1ull << lane) - 1ull;
    int32_t *mine = cnt + w * E;
    for (int i = 0; i < a.steps; ++i) {
        const int sl = s0 + i * 64 + lane;
        const int ev = i == 0 ? first : fetch(i);
        const bool live = ev >= 0;
        const int ee = live ? min(ev, E - 1) : 0;
        // lanes holding the same expert
        uint64_t same = __ballot(live);
        for (int b = 0; b < ebits; ++b) {
            const uint64_t bal = __ballot((ee >> b) & 1);
            same &= ((ee >> b) & 1) ? bal : ~bal;
        }
        if (live) {
            const int row = mine[ee] + __popcll(same & lt);
            a.inv_perm[sl] = row;
            a.perm[row] = (int32_t)sl;
            if (a.x.grow) a.x.grow[row] = a.x.gates[sl];
        }
        if (i + 1 == a.steps) break;
        // (LDS traffic only: the stores above need not have landed)
        __builtin_amdgcn_s_waitcnt(kWaitLds);
        __builtin_amdgcn_wave_barrier();
        // the highest lane of each group advances the group's counter
        if (live && (same >> lane) == 1ull) mine[ee] += __popcll(same);
        __builtin_amdgcn_s_waitcnt(kWaitLds);
        __builtin_amdgcn_wave_barrier();
    }
}

__global__ void __launch_bounds__(256)
permute_hist_kernel(int T, int E, int K, const uint16_t *__restrict__ idx, int64_t stride, int chunk,
                    int nchunks, int32_t *__restrict__ chunk_hist, int32_t *status) {
    extern __shared__ int32_t hist_all[];
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int c = blockIdx.x * 4 + w;
    int32_t *hist = hist_all + w * E;
    for (int e = lane; e < E; e += kWave) hist[e] = 0;
    __syncthreads();
    if (c >= nchunks) return;
    const int S = T * K, s0 = c * chunk;
    const SlotSplit split(K);
    // a token's K ids sit in K neighbouring lanes of one step when K divides 64 (chunks start at
    // multiples of 64): then the duplicate check compares lanes instead of loading ids again
    const bool lanes_hold_token = 64 % K == 0;
    int bad = 0;
    for (int i0 = 0; i0 < chunk; i0 += kWave * kPermBatch) {
        int ev[kPermBatch];
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int sl = s0 + i0 + u * kWave + lane;
            ev[u] = -1;
            if (i0 + u * kWave < chunk && sl < S) {
                int t, j;
                split(sl, t, j);
                ev[u] = (int)idx[(int64_t)t * stride + j];
            }
        }
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int sl = s0 + i0 + u * kWave + lane;
            int e = ev[u];
            const bool live = e >= 0;
            if (live && e >= E) {
                bad |= R3_DATA_IDX_RANGE;
                e = E - 1;
            }
            if (lanes_hold_token) {
                const int j = lane % K;   // (sl % K: chunk starts and steps are multiples of 64)
                for (int back = 1; back < K; ++back) {
                    const int other = __shfl(e, lane - back);
                    if (live && back <= j && other == e) bad |= R3_DATA_IDX_DUP;
                }
            } else if (live) {
                int t, j;
                split(sl, t, j);
                for (int jj = 0; jj < j; ++jj)
                    if (min((int)idx[(int64_t)t * stride + jj], E - 1) == e) bad |= R3_DATA_IDX_DUP;
            }
            if (live) atomicAdd(&hist[e], 1);
        }
    }
    // LDS atomics of one wave are complete before its later LDS reads
    __builtin_amdgcn_s_waitcnt(0);
    __builtin_amdgcn_wave_barrier();
    for (int e = lane; e < E; e += kWave) chunk_hist[(int64_t)c * E + e] = hist[e];
    if (bad && status) atomicOr(status, bad);
}

// One block of 1024 threads (more than 1024 experts).  chunk_base [nchunks,E] receives the exclusive running count of
// chunk_hist over chunks; counts/offsets are written.
__global__ void __launch_bounds__(1024)
permute_scan_kernel(int E, int nchunks, const int32_t *__restrict__ chunk_hist, int32_t *__restrict__ chunk_base,
                    int32_t *__restrict__ counts, int32_t *__restrict__ offsets) {
    __shared__ int32_t tot[kMaxE];
    __shared__ int32_t tmp[16];
    for (int e = threadIdx.x; e < E; e += 1024) {
        int32_t run = 0;
        int c = 0;
        for (; c + 8 <= nchunks; c += 8) {   // (guards in here took 7 % of the whole call: E=2048 T=131072 K=8 173 us, 159 without)
            int32_t h[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) h[u] = chunk_hist[(int64_t)(c + u) * E + e];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                chunk_base[(int64_t)(c + u) * E + e] = run;
                run += h[u];
            }
        }
        for (; c < nchunks; ++c) {
            const int32_t h = chunk_hist[(int64_t)c * E + e];
            chunk_base[(int64_t)c * E + e] = run;
            run += h;
        }
        tot[e] = run;
        counts[e] = run;
    }
    __syncthreads();
    // exclusive scan of tot[0..E): each thread owns a contiguous span
    const int per = (E + 1023) / 1024, b = threadIdx.x * per;
    int32_t sum = 0;
    for (int i = 0; i < per; ++i)
        if (b + i < E) sum += tot[b + i];
    int32_t run = block_scan(sum, tmp) - sum;
    for (int i = 0; i < per; ++i)
        if (b + i < E) {
            offsets[b + i] = run;
            run += tot[b + i];
        }
    if (threadIdx.x == 1023) offsets[E] = run;
}

__global__ void __launch_bounds__(256)
permute_place_kernel(int T, int E, int K, const uint16_t *__restrict__ idx, int64_t stride, int chunk,
                     int nchunks, const int32_t *__restrict__ chunk_base,
                     const int32_t *__restrict__ offsets, int32_t *__restrict__ inv_perm,
                     int32_t *__restrict__ perm) {
    extern __shared__ int32_t cnt_all[];
    const int w = threadIdx.x / kWave, lane = lane_id();
    const int c = blockIdx.x * 4 + w;
    int32_t *cnt = cnt_all + w * E;
    if (c < nchunks)
        for (int e = lane; e < E; e += kWave) cnt[e] = offsets[e] + chunk_base[(int64_t)c * E + e];
    __syncthreads();
    if (c >= nchunks) return;
    const int S = T * K, s0 = c * chunk;
    const SlotSplit split(K);
    int ebits = 1;
    while ((1 << ebits) < E) ++ebits;
    const uint64_t lt = (1ull << lane) - 1ull;
    for (int i0 = 0; i0 < chunk; i0 += kWave * kPermBatch) {
        int ev[kPermBatch];
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int sl = s0 + i0 + u * kWave + lane;
            ev[u] = -1;
            if (i0 + u * kWave < chunk && sl < S) {
                int t, j;
                split(sl, t, j);
                ev[u] = min((int)idx[(int64_t)t * stride + j], E - 1);
            }
        }
#pragma unroll
        for (int u = 0; u < kPermBatch; ++u) {
            const int sl = s0 + i0 + u * kWave + lane;
            const bool live = ev[u] >= 0;
            const int e = live ? ev[u] : 0;
            // lanes holding the same expert
            uint64_t same = __ballot(live);
            for (int b = 0; b < ebits; ++b) {
                uint64_t bal = __ballot((e >> b) & 1);
                same &= ((e >> b) & 1) ? bal : ~bal;
            }
            if (live) {
                int row = cnt[e] + __popcll(same & lt);
                inv_perm[sl] = row;
                perm[row] = (int32_t)sl;
            }
            // (LDS traffic only: the stores above need not have landed)
            __builtin_amdgcn_s_waitcnt(kWaitLds);
            __builtin_amdgcn_wave_barrier();
            // the highest lane of each group advances the group's counter
            if (live && (same >> lane) == 1ull) cnt[e] += __popcll(same);
            __builtin_amdgcn_s_waitcnt(kWaitLds);
            __builtin_amdgcn_wave_barrier();
        }
    }
}

// 16-byte load of data that is read once per launch: marked non-temporal, so that the rows are not
// kept in L2 (measured: the gathered-row reads of combine run 20 % faster; the same hint on stores
// was slower)
template <typename V> __device__ __forceinline__ V ld_once(const V *p) {
    if constexpr (sizeof(V) == 16) {
        typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
        return __builtin_bit_cast(V, __builtin_nontemporal_load((const u32x4 *)p));
    } else {
        return *p;
    }
}

// Row gather by token: the block reads x[t] once and writes its K copies.
// V is the vector type moved per thread (uint4 when rows are 16-byte multiples).
template <typename V>
__global__ void __launch_bounds__(256)
gather_rows_kernel(int T, int K, int row_vecs, const V *__restrict__ x,
                   const int32_t *__restrict__ inv_perm, V *__restrict__ Xp) {
    const int t = blockIdx.x;
    __shared__ int32_t rows[kMaxK];
    if (threadIdx.x < (unsigned)K) rows[threadIdx.x] = inv_perm[(int64_t)t * K + threadIdx.x];
    __syncthreads();
    for (int c = threadIdx.x; c < row_vecs; c += blockDim.x) {
        V v = x[(int64_t)t * row_vecs + c];
        for (int j = 0; j < K; ++j) Xp[(int64_t)rows[j] * row_vecs + c] = v;
    }
}

static int pick_chunk(int64_t S) {
    // slots per wave-chunk: at least 1024, at most 512 chunks in total
    int64_t c = 1024;
    while ((S + c - 1) / c > 512) c *= 2;
    return (int)c;
}

size_t permute_ws_bytes(int T, int E, int K) {
    int64_t S = (int64_t)T * K;
    int chunk = pick_chunk(S);
    int64_t nchunks = (S + chunk - 1) / chunk;
    return 2 * align_up((size_t)nchunks * E * sizeof(int32_t), 256);  // histograms + running bases
}

// Where counting all ids in every work-group gives way to a launch that counts the chunks first, us of r3_permute, all / first:
//   slots          E=8 K=2      E=64 K=4     E=128 K=8    E=384 K=4    E=1024 K=8
//     8192        7.8 / 11.1   7.9 / 10.9   8.1 / 10.8   7.9 / 11.0    8.6 / 12.4
//    16384        9.4 / 11.1   8.0 / 11.0   8.9 / 11.3   8.0 / 11.1    9.3 / 13.0
//    32768       14.3 / 10.7   9.8 / 11.0  11.0 / 11.4   8.6 / 11.0   10.4 / 13.8
//    65536       23.7 / 10.9  13.8 / 10.9  15.0 / 11.3  11.3 / 11.9   12.9 / 15.6
// With the same experts in every token the LDS atomics collide (16384 slots 19 to 22 / 11, 32768 32 to 36 / 11), so the line
// is drawn where the first column still gains and the collisions cost 10 us.
constexpr int64_t kDispCountAll = 16384;

template <typename IdxT>
static void launch_dispatch(int T, int E, int K, const IdxT *idx, int64_t stride, int32_t *counts, int32_t *offsets,
                            int32_t *inv_perm, int32_t *perm, int32_t *status, void *ws, const DispatchExtra &x,
                            hipStream_t s) {
    const int64_t S = (int64_t)T * K;
    const bool hist = S > kDispCountAll;
    const int chunk = hist ? std::max(2 * kDispStep, pick_chunk(S)) : kDispStep;
    DispatchArgs a = {T, E, K, chunk / kDispStep, (int)((S + chunk - 1) / chunk), stride, (const int32_t *)ws, counts, offsets,
                      inv_perm, perm, status, x};
    if (hist) dispatch_count_kernel<IdxT><<<a.nchunks, 1024, E * sizeof(int32_t), s>>>(T, E, K, idx, stride, a.steps, (int32_t *)ws);
    const size_t lds = ((size_t)(kDispWaves + 2) * E + kDispWaves) * sizeof(int32_t);
    auto k = hist ? dispatch_kernel<IdxT, true> : dispatch_kernel<IdxT, false>;
    if (lds > 65536) (void)hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    k<<<a.nchunks + (x.tiles ? 1 : 0), 1024, lds, s>>>(idx, a);
}

bool dispatch_makes_tiles(int E) { return E <= kDispMaxE; }

hipError_t launch_permute(int T, int d, int E, int K, int elem_bytes, const void *x, const void *idx,
                          int idx_dtype, int64_t stride, int32_t *counts, int32_t *offsets,
                          int32_t *inv_perm, int32_t *perm, void *Xp, int32_t *status, void *ws, const DispatchExtra &extra,
                          hipStream_t s) {
    if (E <= kDispMaxE) {
        ProfScope ps(PROF_PERMUTE_INDEX, s);
        if (idx_dtype == R3_IDX_U8)
            launch_dispatch(T, E, K, (const uint8_t *)idx, stride, counts, offsets, inv_perm, perm, status, ws, extra, s);
        else
            launch_dispatch(T, E, K, (const uint16_t *)idx, stride, counts, offsets, inv_perm, perm, status, ws, extra, s);
    } else {
        const int64_t S = (int64_t)T * K;
        const int chunk = pick_chunk(S);
        const int nchunks = (int)((S + chunk - 1) / chunk);
        int32_t *chunk_hist = (int32_t *)ws;
        int32_t *chunk_base = (int32_t *)((char *)ws + align_up((size_t)nchunks * E * sizeof(int32_t), 256));
        const int grid = (nchunks + 3) / 4;
        const size_t lds = (size_t)4 * E * sizeof(int32_t);
        const uint16_t *id = (const uint16_t *)idx;   // (more than 256 experts)
        ProfScope ps(PROF_PERMUTE_INDEX, s);
        permute_hist_kernel<<<grid, 256, lds, s>>>(T, E, K, id, stride, chunk, nchunks, chunk_hist, status);
        permute_scan_kernel<<<1, 1024, 0, s>>>(E, nchunks, chunk_hist, chunk_base, counts, offsets);
        permute_place_kernel<<<grid, 256, lds, s>>>(T, E, K, id, stride, chunk, nchunks, chunk_base, offsets, inv_perm, perm);
    }
    if (Xp) {
        ProfScope ps(PROF_GATHER_ROWS, s);
        const int64_t row_bytes = (int64_t)d * elem_bytes;
        if (row_bytes % 16 == 0)
            gather_rows_kernel<uint4><<<T, 256, 0, s>>>(T, K, (int)(row_bytes / 16), (const uint4 *)x,
                                                       inv_perm, (uint4 *)Xp);
        else if (row_bytes % 4 == 0)
            gather_rows_kernel<uint32_t><<<T, 256, 0, s>>>(T, K, (int)(row_bytes / 4),
                                                          (const uint32_t *)x, inv_perm, (uint32_t *)Xp);
        else
            gather_rows_kernel<uint16_t><<<T, 256, 0, s>>>(T, K, (int)(row_bytes / 2),
                                                          (const uint16_t *)x, inv_perm, (uint16_t *)Xp);
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Combine: y[t] = sum_j g[t,j] * Yp[inv_perm[t*K+j]], j ascending, f32.
// A block takes 256 / LPT tokens, LPT lanes each; a lane owns VEC consecutive columns at a time.
// ---------------------------------------------------------------------------
// Lanes per token: a row shorter than 256 vectors leaves lanes of a block idle, so the block takes two, four or eight tokens; but a small
// batch stays spread over the compute units.  With K known (by_k) and the router's last step beside dx, us, before | now: 3001 tokens top-6, 1000
// columns, combine 10.4 | 9.7, router_finish and dx 20.4 | 13.8; 6000 top-4, 1024 columns 14.3 | 12.9, 22.7 | 20.3; 131072 top-2, 512 columns,
// the forward pass 418 | 400.
static int row_lanes(int T, int row_vecs) {
    int n = 256;
    while (n > 32 && n / 2 >= row_vecs && (int64_t)T * n / 2 >= 1024 * 256) n /= 2;
    return n;
}
template <typename T, int VEC> struct VecIO;
template <> struct VecIO<bf16_t, 8> {
    typedef bf16_t Elem;
    static constexpr int kVec = 8;
    typedef uint4 V;
    static __device__ __forceinline__ void unpack(const V &v, float *f) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            f[2 * i] = __uint_as_float(w[i] << 16);
            f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
        }
    }
    static __device__ __forceinline__ V pack(const float *f) {
        V v;
        v.x = pack_bf16x2(f[0], f[1]);
        v.y = pack_bf16x2(f[2], f[3]);
        v.z = pack_bf16x2(f[4], f[5]);
        v.w = pack_bf16x2(f[6], f[7]);
        return v;
    }
};
template <> struct VecIO<float, 4> {
    typedef float Elem;
    static constexpr int kVec = 4;
    typedef float4 V;
    static __device__ __forceinline__ void unpack(const V &v, float *f) {
        f[0] = v.x; f[1] = v.y; f[2] = v.z; f[3] = v.w;
    }
    static __device__ __forceinline__ V pack(const float *f) { return make_float4(f[0], f[1], f[2], f[3]); }
};
template <> struct VecIO<bf16_t, 1> {
    typedef bf16_t Elem;
    static constexpr int kVec = 1;
    typedef bf16_t V;
    static __device__ __forceinline__ void unpack(const V &v, float *f) { f[0] = bf16_to_f32(v); }
    static __device__ __forceinline__ V pack(const float *f) { return f32_to_bf16(f[0]); }
};
template <> struct VecIO<float, 1> {
    typedef float Elem;
    static constexpr int kVec = 1;
    typedef float V;
    static __device__ __forceinline__ void unpack(const V &v, float *f) { f[0] = v; }
    static __device__ __forceinline__ V pack(const float *f) { return f[0]; }
};

// KT > 0: K known at compile time, so that a thread's K row loads are all in flight together
template <class F> static void by_k(int K, F f) {
    switch (K) {
        case 1: f(std::integral_constant<int, 1>{}); break;
        case 2: f(std::integral_constant<int, 2>{}); break;
        case 4: f(std::integral_constant<int, 4>{}); break;
        case 6: f(std::integral_constant<int, 6>{}); break;
        case 8: f(std::integral_constant<int, 8>{}); break;
        default: f(std::integral_constant<int, 0>{});
    }
}
template <typename T, int VEC, int KT>
__global__ void __launch_bounds__(256)
combine_kernel(int Tn, int Krt, int lanes, int row_vecs, const typename VecIO<T, VEC>::V *__restrict__ Yp,
               const float *__restrict__ gates, const int32_t *__restrict__ inv_perm,
               typename VecIO<T, VEC>::V *__restrict__ y) {
    typedef VecIO<T, VEC> IO;
    const int K = KT > 0 ? KT : Krt;
    const int t0 = blockIdx.x * (256 / lanes), n = min(256 / lanes, Tn - t0) * K;
    __shared__ int32_t rows_s[8 * kMaxK];
    __shared__ float g_s[8 * kMaxK];
    for (int i = threadIdx.x; i < n; i += 256) {
        rows_s[i] = inv_perm[(int64_t)t0 * K + i];
        g_s[i] = gates ? gates[(int64_t)t0 * K + i] : 1.0f;   // no gates: rows arrive gated
    }
    __syncthreads();
    const int tok = (int)threadIdx.x / lanes, t = t0 + tok;
    if (t >= Tn) return;
    const int32_t *rows = rows_s + tok * K;
    const float *g = g_s + tok * K;
    for (int c = threadIdx.x & (lanes - 1); c < row_vecs; c += lanes) {
        float acc[VEC];
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = 0.0f;
        if constexpr (KT > 0) {
            typename IO::V v[KT];
#pragma unroll
            for (int j = 0; j < KT; ++j) v[j] = ld_once(&Yp[(int64_t)rows[j] * row_vecs + c]);
#pragma unroll
            for (int j = 0; j < KT; ++j) {   // fixed j order: the sum is the same for every launch shape
                float f[VEC];
                IO::unpack(v[j], f);
                const float gj = g[j];
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = fmaf(gj, f[i], acc[i]);
            }
        } else {
            for (int j = 0; j < K; ++j) {
                float f[VEC];
                IO::unpack(Yp[(int64_t)rows[j] * row_vecs + c], f);
                const float gj = g[j];
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = fmaf(gj, f[i], acc[i]);
            }
        }
        y[(int64_t)t * row_vecs + c] = IO::pack(acc);
    }
}

hipError_t launch_combine(int T, int d, int K, int act, const void *Yp, const float *gates,
                          const int32_t *inv_perm, void *y, hipStream_t s) {
    ProfScope ps(PROF_COMBINE, s);
    auto go = [&](auto io, auto kt) {
        typedef decltype(io) IO;
        const int vecs = d / IO::kVec, lanes = row_lanes(T, vecs), tpb = 256 / lanes;
        combine_kernel<typename IO::Elem, IO::kVec, decltype(kt)::value><<<(T + tpb - 1) / tpb, 256, 0, s>>>(
            T, K, lanes, vecs, (const typename IO::V *)Yp, gates, inv_perm, (typename IO::V *)y);
    };
    if (act == R3_BF16) {
        if (d % 8 == 0) by_k(K, [&](auto kt) { go(VecIO<bf16_t, 8>{}, kt); });
        else go(VecIO<bf16_t, 1>{}, std::integral_constant<int, 0>{});
    } else {
        if (d % 4 == 0) by_k(K, [&](auto kt) { go(VecIO<float, 4>{}, kt); });
        else go(VecIO<float, 1>{}, std::integral_constant<int, 0>{});
    }
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Backward through combine and masked softmax, one block per token:
//   dg_j = <dy_t, Yp[row_j]>,  dYp[row_j] = g_j * dy_t,
//   dz_j = g_j (dg_j - sum_i g_i dg_i).
// Writes dz [T,K] f32, and dzrow[row_j] = dz_j unless that is NULL.
// ---------------------------------------------------------------------------
template <typename T, int VEC, int KT>
__global__ void __launch_bounds__(256)
gate_backward_kernel(int Krt, int row_vecs, const typename VecIO<T, VEC>::V *__restrict__ dy,
                     const typename VecIO<T, VEC>::V *__restrict__ Yp, const float *__restrict__ gates,
                     const int32_t *__restrict__ inv_perm, typename VecIO<T, VEC>::V *__restrict__ dYp,
                     float *__restrict__ dz, float *__restrict__ dzrow, int gated) {
    typedef VecIO<T, VEC> IO;
    const int K = KT > 0 ? KT : Krt;
    const int t = blockIdx.x;
    const int nw = blockDim.x / kWave, w = threadIdx.x / kWave, lane = lane_id();
    __shared__ int32_t rows[kMaxK];
    __shared__ float g[kMaxK];
    __shared__ float part[4][kMaxK];
    __shared__ float dgs[kMaxK];
    if (threadIdx.x < (unsigned)K) {
        rows[threadIdx.x] = inv_perm[(int64_t)t * K + threadIdx.x];
        g[threadIdx.x] = gates[(int64_t)t * K + threadIdx.x];
    }
    __syncthreads();
    if constexpr (KT > 0) {
        // dy is read once per column chunk and the K rows of Yp are all in flight together; per
        // thread and per j the products are summed in the same order as in the loop below
        float dot[KT];
#pragma unroll
        for (int j = 0; j < KT; ++j) dot[j] = 0.0f;
        for (int c = threadIdx.x; c < row_vecs; c += blockDim.x) {
            float a[VEC];
            IO::unpack(dy[(int64_t)t * row_vecs + c], a);
            typename IO::V v[KT];
#pragma unroll
            for (int j = 0; j < KT; ++j) v[j] = ld_once(&Yp[(int64_t)rows[j] * row_vecs + c]);
#pragma unroll
            for (int j = 0; j < KT; ++j) {
                float b[VEC], o[VEC];
                IO::unpack(v[j], b);
                const float gj = g[j];
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    dot[j] = fmaf(a[i], b[i], dot[j]);
                    o[i] = gj * a[i];
                }
                dYp[(int64_t)rows[j] * row_vecs + c] = IO::pack(o);
            }
        }
#pragma unroll
        for (int j = 0; j < KT; ++j) {
            const float dsum = wave_sum(dot[j]);
            if (lane == 0) part[w][j] = dsum;
        }
    } else {
        for (int j = 0; j < K; ++j) {
            float dot = 0.0f;
            const float gj = g[j];
            for (int c = threadIdx.x; c < row_vecs; c += blockDim.x) {
                float a[VEC], b[VEC], o[VEC];
                IO::unpack(dy[(int64_t)t * row_vecs + c], a);
                IO::unpack(Yp[(int64_t)rows[j] * row_vecs + c], b);
#pragma unroll
                for (int i = 0; i < VEC; ++i) {
                    dot = fmaf(a[i], b[i], dot);
                    o[i] = gj * a[i];
                }
                dYp[(int64_t)rows[j] * row_vecs + c] = IO::pack(o);
            }
            dot = wave_sum(dot);
            if (lane == 0) part[w][j] = dot;
        }
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)K) {
        float v = 0.0f;
        for (int i = 0; i < nw; ++i) v += part[i][threadIdx.x];
        dgs[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x < (unsigned)K) {
        // gated: the rows of Yp are g o, so the dot products are already g_j dg_j
        float mix = 0.0f;
        for (int j = 0; j < K; ++j) mix = gated ? mix + dgs[j] : fmaf(g[j], dgs[j], mix);
        float v = gated ? dgs[threadIdx.x] - g[threadIdx.x] * mix : g[threadIdx.x] * (dgs[threadIdx.x] - mix);
        dz[(int64_t)t * K + threadIdx.x] = v;
        if (dzrow) dzrow[rows[threadIdx.x]] = v;
    }
}

template <typename T, int VEC>
static hipError_t gate_backward_dispatch(int Tn, int K, int row_vecs, const void *dy, const void *Yp, const float *gates,
                                         const int32_t *inv_perm, void *dYp, float *dz, float *dzrow, int gated,
                                         hipStream_t s) {
    typedef typename VecIO<T, VEC>::V V;
    // (K = 4 in registers: 8.4 -> 10.3 us at 2048 f32 tokens of 512)
    auto k = K == 8 && VEC > 1 ? gate_backward_kernel<T, VEC, 8> : gate_backward_kernel<T, VEC, 0>;
    k<<<Tn, 256, 0, s>>>(K, row_vecs, (const V *)dy, (const V *)Yp, gates, inv_perm, (V *)dYp, dz, dzrow, gated);
    return hipGetLastError();
}

hipError_t launch_gate_backward(int T, int d, int K, int act, const void *dy, const void *Yp, const float *gates,
                                const int32_t *inv_perm, void *dYp, float *dz, float *dzrow, int gated, hipStream_t s) {
    ProfScope ps(PROF_GATE_BWD, s);
    if (act == R3_BF16)
        return d % 8 == 0 ? gate_backward_dispatch<bf16_t, 8>(T, K, d / 8, dy, Yp, gates, inv_perm, dYp, dz, dzrow, gated, s)
                          : gate_backward_dispatch<bf16_t, 1>(T, K, d, dy, Yp, gates, inv_perm, dYp, dz, dzrow, gated, s);
    return d % 4 == 0 ? gate_backward_dispatch<float, 4>(T, K, d / 4, dy, Yp, gates, inv_perm, dYp, dz, dzrow, gated, s)
                      : gate_backward_dispatch<float, 1>(T, K, d, dy, Yp, gates, inv_perm, dYp, dz, dzrow, gated, s);
}

// ---------------------------------------------------------------------------
// Masked-softmax backward when the expert-gradient GEMM has already formed the dot products: its
// epilogue leaves, for every row r, `nparts` partial sums whose total is w = g <dy_t, o_r> = g dg.
//   w_j = sum_p wpart[row_j][p] (p ascending),   dz_j = g_j (dg_j - sum_i g_i dg_i) = w_j - g_j sum_i w_i
// One thread per slot, a token's K slots in neighbouring lanes (KP: K rounded up to a power of two).
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
gate_backward_parts_kernel(int T, int K, int KP, int nparts, const float *__restrict__ wpart,
                           const float *__restrict__ gates, const int32_t *__restrict__ inv_perm, float *__restrict__ dz,
                           float *__restrict__ dzrow, RouterFinish<bf16_t> wrt, int nwrt) {
    __shared__ RouterFinishLds<bf16_t> lds;
    if ((int)blockIdx.x < nwrt) {   // W_r^T, which dx will want, has nothing to wait for
        router_finish_block<256>(wrt, blockIdx.x, lds);
        return;
    }
    const int j = threadIdx.x % KP, t = ((int)blockIdx.x - nwrt) * (256 / KP) + threadIdx.x / KP;
    const bool live = t < T && j < K;
    float w = 0.0f, g = 0.0f;
    int row = 0;
    if (live) {
        row = inv_perm[(int64_t)t * K + j];
        const float *p = wpart + (int64_t)row * nparts;
        for (int i = 0; i < nparts; ++i) w += p[i];
        g = gates[(int64_t)t * K + j];
    }
    // sum of w over the token's slots, in a fixed order: KP neighbouring lanes (KP <= 64 divides 64)
    float mix = w;
    for (int o = 1; o < KP; o <<= 1) mix += __shfl_xor(mix, o, 64);
    if (live) {
        dz[(int64_t)t * K + j] = w - g * mix;
        if (dzrow) dzrow[row] = w - g * mix;
    }
}

hipError_t launch_gate_backward_parts(int T, int K, int nparts, const float *wpart, const float *gates,
                                      const int32_t *inv_perm, float *dz, float *dzrow, int d, int E, const void *Wr, void *WrT,
                                      hipStream_t s) {
    ProfScope ps(PROF_GATE_BWD, s);
    RouterFinish<bf16_t> wrt;
    const int nwrt = wrt.transpose_only(d, E, Wr, WrT);
    int KP = 1;
    while (KP < K) KP <<= 1;                        // K <= kMaxK = 64
    const int tpb = 256 / KP;
    gate_backward_parts_kernel<<<nwrt + (T + tpb - 1) / tpb, 256, 0, s>>>(T, K, KP, nparts, wpart, gates, inv_perm, dz, dzrow, wrt, nwrt);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Final input gradient, tokens and lanes as in combine_kernel:
//   dx[t] = sum_j dXp[row_j]  +  sum_j dz[t,j] * W_r[:, idx_j]
// WrT is W_r transposed ([E,d], act dtype) so that the router term reads rows.
// The first nfin blocks: the rest of the router's backward (the sum of dW_r's parts, dbias), which waits for the same launches.
// ---------------------------------------------------------------------------
template <typename T, int VEC, typename IdxT, int KT>
__global__ void __launch_bounds__(256)
dx_finish_kernel(int Tn, int E, int Krt, int lanes, int row_vecs, const typename VecIO<T, VEC>::V *__restrict__ dXp,
                 const typename VecIO<T, VEC>::V *__restrict__ WrT, const float *__restrict__ dz,
                 const int32_t *__restrict__ inv_perm, const IdxT *__restrict__ idx, int64_t stride,
                 typename VecIO<T, VEC>::V *__restrict__ dx, RouterFinish<T> fin, int nfin) {
    typedef VecIO<T, VEC> IO;
    const int K = KT > 0 ? KT : Krt;
    __shared__ union {
        RouterFinishLds<T> fin;
        struct {
            int32_t rows[8 * kMaxK], ids[8 * kMaxK];
            float z[8 * kMaxK];
        } tok;
    } lds;
    if ((int)blockIdx.x < nfin) {
        router_finish_block<256>(fin, blockIdx.x, lds.fin);
        return;
    }
    const int t0 = ((int)blockIdx.x - nfin) * (256 / lanes), n = min(256 / lanes, Tn - t0) * K;
    for (int i = threadIdx.x; i < n; i += 256) {
        const int q = i / K;
        lds.tok.rows[i] = inv_perm[(int64_t)t0 * K + i];
        lds.tok.ids[i] = min((int)idx[(int64_t)(t0 + q) * stride + i - q * K], E - 1);
        lds.tok.z[i] = dz[(int64_t)t0 * K + i];
    }
    __syncthreads();
    const int tok = (int)threadIdx.x / lanes, t = t0 + tok;
    if (t >= Tn) return;
    const int32_t *rows = lds.tok.rows + tok * K, *ids = lds.tok.ids + tok * K;
    const float *z = lds.tok.z + tok * K;
    for (int c = threadIdx.x & (lanes - 1); c < row_vecs; c += lanes) {
        float acc[VEC];
#pragma unroll
        for (int i = 0; i < VEC; ++i) acc[i] = 0.0f;
        if constexpr (KT > 0) {   // all 2K row loads in flight together; same summation order as below
            typename IO::V v[KT], w[KT];
#pragma unroll
            for (int j = 0; j < KT; ++j) v[j] = ld_once(&dXp[(int64_t)rows[j] * row_vecs + c]);
#pragma unroll
            for (int j = 0; j < KT; ++j) w[j] = WrT[(int64_t)ids[j] * row_vecs + c];
#pragma unroll
            for (int j = 0; j < KT; ++j) {
                float f[VEC];
                IO::unpack(v[j], f);
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] += f[i];
            }
#pragma unroll
            for (int j = 0; j < KT; ++j) {
                float f[VEC];
                IO::unpack(w[j], f);
                const float zj = z[j];
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = fmaf(zj, f[i], acc[i]);
            }
        } else {
            for (int j = 0; j < K; ++j) {
                float f[VEC];
                IO::unpack(dXp[(int64_t)rows[j] * row_vecs + c], f);
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] += f[i];
            }
            for (int j = 0; j < K; ++j) {
                float f[VEC];
                IO::unpack(WrT[(int64_t)ids[j] * row_vecs + c], f);
                const float zj = z[j];
#pragma unroll
                for (int i = 0; i < VEC; ++i) acc[i] = fmaf(zj, f[i], acc[i]);
            }
        }
        dx[(int64_t)t * row_vecs + c] = IO::pack(acc);
    }
}

hipError_t launch_dx_finish(int T, int d, int E, int K, int act, const void *dXp, const void *WrT, const float *dz, const int32_t *inv_perm,
                            const void *idx, int idx_dtype, int64_t stride, void *dx, const void *fin, int nfin,
                            hipStream_t s) {
    ProfScope ps(PROF_DX_FINISH, s);
    auto launch = [&](auto io, auto kt, auto id) {
        typedef decltype(io) IO;
        typedef typename IO::V V;
        const int vecs = d / IO::kVec, lanes = row_lanes(T, vecs), tpb = 256 / lanes;
        RouterFinish<typename IO::Elem> f = {};
        if (fin) f = *(const RouterFinish<typename IO::Elem> *)fin;
        dx_finish_kernel<typename IO::Elem, IO::kVec, typename std::remove_const<typename std::remove_pointer<decltype(id)>::type>::type,
                         decltype(kt)::value><<<nfin + (T + tpb - 1) / tpb, 256, 0, s>>>(
            T, E, K, lanes, vecs, (const V *)dXp, (const V *)WrT, dz, inv_perm, id, stride, (V *)dx, f, nfin);
    };
    auto go = [&](auto io) {
        auto kt = [&](auto k) {
            if (idx_dtype == R3_IDX_U8) launch(io, k, (const uint8_t *)idx);
            else launch(io, k, (const uint16_t *)idx);
        };
        if constexpr (decltype(io)::kVec > 1) by_k(K, kt);
        else kt(std::integral_constant<int, 0>{});
    };
    if (act == R3_BF16) {
        if (d % 8 == 0) go(VecIO<bf16_t, 8>{});
        else go(VecIO<bf16_t, 1>{});
    } else {
        if (d % 4 == 0) go(VecIO<float, 4>{});
        else go(VecIO<float, 1>{});
    }
    return hipGetLastError();
}

}  // namespace r3
