// The last step of the router's backward: three sorts of work that do not wait for each other, a work-group of NT threads each (in a launch of
// their own, or beside others: W_r^T with the gate's backward and the rest with dx, for bf16 tiles and for f32 after the one-call forward).
//   dbias[e] (+)= the sum of dz over the rows of expert e (fixed order; first in the grid, as a skewed load's hot expert takes
//     longest);
//   dW_r[i] (+)= sum_s part[s][i], s ascending, NT values;
//   W_r^T, which dx reads, a 32 x 32 tile.
#pragma once
#include "r3_common.h"

namespace r3 {

template <typename T> struct RouterFinish {
    int d, E, nsplit, accumulate, bias_blocks, sum_blocks;
    const float *dzrow, *part;
    const int32_t *offsets;
    float *dbias, *dWr;
    const T *Wr;
    T *WrT;
    // (dbias may be NULL) returns the number of work-groups
    template <int NT>
    int fill(int d_, int E_, int nsplit_, int accumulate_, const float *dzrow_, const float *part_, const int32_t *offsets_, float *dbias_,
             float *dWr_, const void *Wr_, void *WrT_) {
        d = d_; E = E_; nsplit = nsplit_; accumulate = accumulate_;
        bias_blocks = dbias_ ? E : 0;
        sum_blocks = (int)(((int64_t)d * E + NT - 1) / NT);
        dzrow = dzrow_; part = part_; offsets = offsets_;
        dbias = dbias_; dWr = dWr_;
        Wr = (const T *)Wr_; WrT = (T *)WrT_;
        return bias_blocks + sum_blocks + ((d + 31) / 32) * ((E + 31) / 32);
    }
    // W_r^T alone, and its work-groups
    int transpose_only(int d_, int E_, const void *Wr_, void *WrT_) {
        *this = {};
        d = d_; E = E_;
        Wr = (const T *)Wr_; WrT = (T *)WrT_;
        return ((d + 31) / 32) * ((E + 31) / 32);
    }
};
template <typename T> struct RouterFinishLds {
    float tmp[16];
    T tile[32][33];
};

template <int NT, typename T>
__device__ __forceinline__ void router_finish_block(const RouterFinish<T> &a, int blk, RouterFinishLds<T> &lds) {
    static_assert(1024 % NT == 0, "");
    const int tid = threadIdx.x, E = a.E;
    if (blk < a.bias_blocks) {
        // 1024 chains whatever NT is, V of them to a thread: the same bits in either launch, and rounding that grows with n / 1024 (a
        // chain to a thread of 256: on normal values 1.35 times this error at 65536 rows of an expert, 1.6 at 131072)
        constexpr int V = 1024 / NT;
        const int e = blk, r1 = a.offsets[e + 1];
        float chain[V] = {};
        for (int r = a.offsets[e] + tid; r < r1; r += 4 * 1024) {
            float v[V][4];
#pragma unroll
            for (int c = 0; c < V; ++c)
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int at = r + c * NT + u * 1024;
                    v[c][u] = at < r1 ? a.dzrow[at] : 0.0f;
                }
#pragma unroll
            for (int c = 0; c < V; ++c) chain[c] += (v[c][0] + v[c][1]) + (v[c][2] + v[c][3]);
        }
#pragma unroll
        for (int c = 0; c < V; ++c) {
            const float w = wave_sum(chain[c]);
            if (lane_id() == 0) lds.tmp[c * (NT / kWave) + (tid >> 6)] = w;
        }
        __syncthreads();
        if (tid == 0) {
            float acc = a.accumulate ? a.dbias[e] : 0.0f;
            for (int i = 0; i < 1024 / kWave; ++i) acc += lds.tmp[i];
            a.dbias[e] = acc;
        }
        return;
    }
    blk -= a.bias_blocks;
    if (blk < a.sum_blocks) {
        const int64_t n = (int64_t)a.d * E, i = (int64_t)blk * NT + tid;
        if (i >= n) return;
        float acc = a.accumulate ? a.dWr[i] : 0.0f;
        for (int s = 0; s < a.nsplit; s += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = s + u < a.nsplit ? a.part[(int64_t)(s + u) * n + i] : 0.0f;
#pragma unroll
            for (int u = 0; u < 8; ++u) acc += v[u];
        }
        a.dWr[i] = acc;
        return;
    }
    blk -= a.sum_blocks;
    const int ne = (E + 31) / 32, e0 = blk % ne * 32, c0 = blk / ne * 32, lo = tid & 31;
#pragma unroll
    for (int hi = tid >> 5; hi < 32; hi += NT / 32)
        if (c0 + hi < a.d && e0 + lo < E) lds.tile[hi][lo] = a.Wr[(int64_t)(c0 + hi) * E + e0 + lo];
    __syncthreads();
#pragma unroll
    for (int hi = tid >> 5; hi < 32; hi += NT / 32)
        if (e0 + hi < E && c0 + lo < a.d) a.WrT[(int64_t)(e0 + hi) * a.d + c0 + lo] = lds.tile[lo][hi];
}

}  // namespace r3
