// What the f32 tile kernels (r3_f32.hip) and those for any width (r3_plain.hip) share.
#pragma once
#include "r3_common.h"

namespace r3 {

// row-tiled contractions over the expert-sorted rows:
//   FFN1: A = rows Wg, B = rows Wu; H = (g) silu(A) B; FA = B silu'(A), FB = silu(A)
//   DOWN: Yp = H Wd        DH: dh = dYp Wd^T, dA = dh FA, dB = dh FB        DXP: dA Wg^T + dB Wu^T
enum { PLAIN_FFN1, PLAIN_DOWN, PLAIN_DH, PLAIN_DXP };

// A tile of BQ rows (tiles of BQ rows, experts ascending) and its column tile, e = -1 past the last one.  Every wave finds it
// by itself: a lane adds up the tiles of its share of the experts, the wave
// scans the sums and the lane that holds the tile walks its share.  (A table made by a launch of its own
// costs more than this: the layers that come here are small.)
struct RowTile {
    int e, row0, row1, col;
};
// XCD: block b takes tile (b % 8) n / 8 + b / 8 of the n that exist, so that the tiles of an expert meet in few L2s
// (launched with f32_rows_grid() blocks); else row tile b / npt, column tile b % npt.
template <bool XCD>
__device__ __forceinline__ RowTile find_row_tile(const int32_t *__restrict__ offsets, int E, int BQ, int block, int npt) {
    const int lane = lane_id(), per = (E + kWave - 1) / kWave;
    const int e0 = min(lane * per, E), e1 = min(e0 + per, E);
    int mine = 0, lo = offsets[e0];
    for (int e = e0; e < e1; ++e) {
        const int hi = offsets[e + 1];
        mine += (hi - lo + BQ - 1) / BQ;
        lo = hi;
    }
    int incl = mine;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
        const int v = __shfl_up(incl, o, kWave);
        if (lane >= o) incl += v;
    }
    RowTile t = {-1, 0, 0, 0};
    int id = block;
    if constexpr (XCD) {
        const int each = (__builtin_amdgcn_readlane(incl, kWave - 1) * npt + 7) >> 3;
        if ((block >> 3) >= each) return t;
        id = (block & 7) * each + (block >> 3);
    }
    const int want = id / npt;
    t.col = id - want * npt;
    const uint64_t past = __ballot(incl > want);
    if (past == 0) return t;
    const int owner = __builtin_amdgcn_readfirstlane(__ffsll((unsigned long long)past) - 1);
    int left = want - __builtin_amdgcn_readlane(incl - mine, owner);
    for (int e = owner * per; e < min((owner + 1) * per, E); ++e) {   // wave-uniform
        const int a = offsets[e], b = offsets[e + 1], n = (b - a + BQ - 1) / BQ;
        if (left < n) {
            t.e = e;
            t.row0 = a + left * BQ;
            t.row1 = min(b, t.row0 + BQ);
            return t;
        }
        left -= n;
    }
    return t;
}
// row tiles of BQ rows over E ragged segments of S rows: at most this many
inline int64_t max_row_tiles(int64_t S, int E, int BQ) { return S / BQ + (E < S ? E : S); }
// blocks of a launch that takes its tiles by XCD: whole rounds of 8
inline int64_t f32_rows_grid(int64_t S, int E, int BQ, int64_t npt) { return (max_row_tiles(S, E, BQ) * npt + 7) / 8 * 8; }

// r3_f32.hip; widths must be multiples of four.  T: rows of the un-permuted matrix (with perm), of less than 2 GB.
hipError_t f32_rows(int mode, int S, int d, int E, int F, const int32_t *offsets, const float *in0, const float *in1, int T,
                    const int32_t *perm, int K, const float *gates, const float *W0, const float *W1, const float *FA,
                    const float *FB, float *o0, float *o1, float *o2, hipStream_t s);
hipError_t f32_wgrads(int d, int E, int F, int T, int K, const int32_t *offsets, const float *H, const float *dYrows,
                      const int32_t *dyperm, const float *xrows, const int32_t *xperm, const float *dA, const float *dB,
                      float *dWg, float *dWu, float *dWd, int accumulate, hipStream_t s);

// The expert gradients and the gate's for a forward that left H and Yp gated, two launches: dz (and dzrow, unless NULL), W_r^T and dH; then
// dW_gate, dW_up, dW_down, dXp and the parts of dW_r, plain_dwr_rows() tokens each.
struct F32Backward {
    int S, T, d, E, F, K, accumulate;
    const int32_t *offsets, *perm, *inv_perm;
    const float *dy, *x, *xrows;      // xrows: x with xperm = perm, or the expert-sorted copy with xperm = NULL
    const int32_t *xperm;
    const void *idx;
    int idx_dtype;
    int64_t stride;
    const float *gates, *Yp, *H, *FA, *FB, *Wr, *Wg, *Wu, *Wd;
    float *dz, *dzrow, *dA, *dB, *dXp, *part, *dWg, *dWu, *dWd, *WrT;
};
bool f32_backward_supported(int act, int T, int d, int F);
hipError_t f32_backward(const F32Backward &b, hipStream_t s);

}  // namespace r3
