// Internal launch interface between the C ABI (r3_api.hip) and the kernel files.
#pragma once
#include "r3_common.h"

namespace r3 {

// Optional per-kernel timing with HIP events on the launch stream (off by default).
// A ProfScope brackets one kernel launch; r3_profile_read() sums what was recorded.
enum ProfTag {
    PROF_RECORD = 0, PROF_LOGITS, PROF_GATE, PROF_PERMUTE_INDEX, PROF_GATHER_ROWS, PROF_FFN1, PROF_FFN2,
    PROF_COMBINE, PROF_GATE_BWD, PROF_DWR, PROF_DH, PROF_WGRAD, PROF_DXP, PROF_DX_FINISH, PROF_WGRAD_PAIR,
    PROF_ROUTING_DIFF, PROF_POLICY, PROF_CACHE_APPEND, PROF_CACHE_GATHER, PROF_AGREEMENT, PROF_NTAGS
};
struct ProfScope {
    int tag, slot;
    hipStream_t s;
    ProfScope(int tag, hipStream_t s);
    ~ProfScope();
};

// r3_route.hip
hipError_t launch_record_topk(int T, int E, int K, const float *logits, int64_t ld, void *idx,
                              int idx_dtype, int64_t stride, int32_t *status, hipStream_t s);
hipError_t launch_gate(int T, int E, int K, const float *logits, const void *idx, int idx_dtype,
                       int64_t stride, float *gates, int32_t *status, hipStream_t s);
hipError_t launch_agreement(int T, int E, int K, const float *logits, const void *idx, int idx_dtype,
                            int64_t stride, int64_t *agree, hipStream_t s);
size_t permute_ws_bytes(int T, int E, int K);
// What the dispatch may make in the same launch (dispatch_makes_tiles(E)): the expert GEMMs' tile table without
// reduction segments, grow[row] = gates of the row's slot.  All or none.
struct DispatchExtra {
    int32_t *tiles;
    const float *gates;
    float *grow;
};
bool dispatch_makes_tiles(int E);
hipError_t launch_permute(int T, int d, int E, int K, int elem_bytes, const void *x, const void *idx,
                          int idx_dtype, int64_t stride, int32_t *counts, int32_t *offsets,
                          int32_t *inv_perm, int32_t *perm, void *Xp, int32_t *status, void *ws, const DispatchExtra &extra,
                          hipStream_t s);
hipError_t launch_combine(int T, int d, int K, int act, const void *Yp, const float *gates,
                          const int32_t *inv_perm, void *y, hipStream_t s);
// gated != 0: Yp holds gate-scaled rows (g o), so <dy, Yp_j> is already g_j dg_j.  dzrow (or NULL): dz in the order
// of the rows, dzrow[inv_perm[i]] = dz[i]
hipError_t launch_gate_backward(int T, int d, int K, int act, const void *dy, const void *Yp, const float *gates,
                                const int32_t *inv_perm, void *dYp, float *dz, float *dzrow, int gated, hipStream_t s);
// masked-softmax backward from the row parts written by the expert-gradient GEMM:
// w_j = sum_p wpart[row_j][p] (= g_j dg_j), dz_j = w_j - g_j sum_i w_i; writes dz [T,K], and dzrow as above
hipError_t launch_gate_backward_parts(int T, int K, int nparts, const float *wpart, const float *gates,
                                      const int32_t *inv_perm, float *dz, float *dzrow, int d, int E, const void *Wr, void *WrT,
                                      hipStream_t s);
// fin, nfin: work-groups of the router's last step to run beside it (a RouterFinish of the activations' type; NULL, 0: none)
hipError_t launch_dx_finish(int T, int d, int E, int K, int act, const void *dXp, const void *WrT, const float *dz, const int32_t *inv_perm,
                            const void *idx, int idx_dtype, int64_t stride, void *dx, const void *fin, int nfin,
                            hipStream_t s);

// r3_diag.hip
size_t policy_ws_bytes();
int policy_max_tau();
hipError_t launch_routing_diff(int T, int K, int L, const void *a, const void *b, int idx_dtype, int64_t token_stride,
                               int64_t layer_stride, const int32_t *seq_offsets, int nseq, int64_t *router_hist,
                               int32_t *token_choices, int32_t *token_routers, double *seq_mean, hipStream_t s);
hipError_t launch_policy_discrepancy(int64_t n, const float *lt, const float *li, int ntau, const float *tau_host,
                                     double *kl, double *frac, void *ws, hipStream_t s);

// r3_cache.hip
hipError_t launch_cache_append(int idx_bytes, int L, int K, int P, void *pages, int64_t num_pages,
                               const int32_t *block_table, int nseq, int max_blocks, int64_t n,
                               const int32_t *seq_id, const int32_t *position, const void *idx_new,
                               int64_t layer_stride, int64_t token_stride, int32_t *status, hipStream_t s);
hipError_t launch_cache_gather(int idx_bytes, int L, int K, int P, const void *pages, int64_t num_pages,
                               const int32_t *block_table, int nseq, int max_blocks, const int32_t *seq_start,
                               int T, void *out, int32_t *status, hipStream_t s);

// r3_plain.hip (f32 arithmetic, any widths, both activation types)
hipError_t plain_router_logits(int T, int d, int E, int act, const void *x, const void *Wr, const float *bias,
                               float *logits, hipStream_t s);
// perm != NULL: `rows` is x [T,d] and row r of the grouped operand is x[perm[r] / K] (no gathered copy);
// gates != NULL (with perm): H is stored scaled by the gate of the row's slot, gates[perm[r]]
hipError_t plain_ffn1(int S, int d, int E, int F, int act, const void *rows, int T, const int32_t *perm, int K,
                      const int32_t *offsets, const void *Wg, const void *Wu, void *H, void *FA, void *FB,
                      const float *gates, hipStream_t s);
hipError_t plain_ffn2(int S, int d, int E, int F, int act, const void *H, const int32_t *offsets, const void *Wd,
                      void *Yp, hipStream_t s);
hipError_t plain_dh(int S, int d, int E, int F, int act, const void *dYp, const int32_t *offsets, const void *Wd,
                    const void *FA, const void *FB, void *dA, void *dB, hipStream_t s);
hipError_t plain_dxp(int S, int d, int E, int F, int act, const void *dA, const void *dB, const int32_t *offsets,
                     const void *Wg, const void *Wu, void *dXp, hipStream_t s);
// dWd (+)= H^T dYrows, dWg (+)= xrows^T dA, dWu (+)= xrows^T dB per expert.  dyperm / xperm != NULL: that operand is
// an un-permuted matrix and row r of the reduction is its row perm[r] / K
hipError_t plain_wgrads(int d, int E, int F, int T, int K, int act, const int32_t *offsets, const void *H, const void *dYrows,
                        const int32_t *dyperm, const void *xrows, const int32_t *xperm, const void *dA, const void *dB,
                        float *dWg, float *dWu, float *dWd, int accumulate, hipStream_t s);
int plain_dwr_rows(int T, int d, int E);          // tokens per part
unsigned plain_dwr_blocks(int T, int d, int E);   // work-groups of 256
void plain_dwr_parts(int T, int d, int E, int K, int act, const void *x, const float *dz, const void *idx, int idx_dtype,
                     int64_t stride, float *part, hipStream_t s);

// r3_router.hip: logits + replay gate (+ agreement counts, K <= 8) in one launch.  plain_only: f32 arithmetic
bool router_gate_supported(int act, int d, int E, bool plain_only);
hipError_t router_gate(int T, int d, int E, int K, int act, const void *x, const void *Wr, const float *bias, const void *idx,
                       int idx_dtype, int64_t stride, float *gates, float *logits_out, int64_t *agree, int32_t *status,
                       bool plain_only, hipStream_t s);

// Router weight gradient dW_r (+)= x^T ds, ds[t][idx[t][j]] = dz[t][j]; part: router_dwr_ws_bytes() bytes.  dbias (+)=
// column sums of ds, unless NULL (dzrow: dz in the order of the rows).  WrT [E,d] = W_r^T
size_t router_dwr_ws_bytes(int act, int T, int d, int E, bool plain_only);
// its first step alone, parts of dW_r over the tokens, and their number
hipError_t router_dwr_parts(int T, int d, int E, int K, int act, const void *x, const float *dz, const void *idx, int idx_dtype, int64_t stride,
                            float *part, bool plain_only, hipStream_t s);
int router_dwr_nparts(int act, int T, int d, int E, bool plain_only);
hipError_t router_backward(int T, int d, int E, int K, int act, const void *x, const void *Wr, const float *dz, const void *idx,
                           int idx_dtype, int64_t stride, const int32_t *offsets, const float *dzrow, float *part, float *dWr,
                           float *dbias, void *WrT, int accumulate, bool plain_only, hipStream_t s);

// r3_gemm.hip (bf16 MFMA)
bool mfma_ffn_supported(int64_t S, int d, int F);
bool mfma_ffn_ragged(int d, int F);      // widths that are not whole tiles of 256
bool mfma_router_supported(int d, int E);
size_t mfma_tiles_bytes(int64_t S, int E);
// split_rows > 0: experts with more rows than that are cut into parts of at most that many rows for the
// weight gradients (mfma_wgrad_split_rows picks it); 0: never; < 0: the pass has no
// weight gradients and the table gets no reduction segments at all
hipError_t mfma_build_tiles(int E, const int32_t *offsets, int32_t *tiles, int split_rows, hipStream_t s);
// the same launch also makes the row -> token list, tok[inv_perm[i]] = i / K (mfma_row_tokens_bytes(): padded), and the
// gates in that order, grow[inv_perm[i]] = gates[i]
hipError_t mfma_build_tiles_and_row_tokens(int E, const int32_t *offsets, int32_t *tiles, int split_rows, int S, int K,
                                           const int32_t *inv_perm, const float *gates, int32_t *tok, float *grow,
                                           hipStream_t s);
// 0 unless `part_bytes_available` holds the partial products of every slot a split may use
int mfma_wgrad_split_rows(int64_t S, int tiles_per_seg, size_t part_bytes_available, size_t bytes_per_slot);
// perm != NULL: `Xp` is x [T,d] (T*d*2 bytes readable) and the first contraction gathers its rows
// through perm in the tile loads
hipError_t mfma_ffn_forward(int64_t S, int d, int E, int F, const void *Xp, const int32_t *perm, int K, int T,
                            const int32_t *offsets, const int32_t *tiles, const void *Wg, const void *Wu,
                            const void *Wd, void *Yp, void *H, void *FA, void *FB, const float *grow,
                            hipStream_t s);
// The expert gradients of a backward, with the gate's in between (r3_gemm.hip):
//   u = dy Wd^T with the rows of dy read through tok (row r is dy[tok[r]], dy is [T,d], T * d * 2 < 2^31); dA = g u FA, dB = g u FB,
//   Hg = g H and wpart [S, row_parts] f32, whose row sums are g <dy, o>.  Hg == NULL: H already holds g H (the one-call forward wrote it so);
//   dz (and, if not NULL, dzrow) from wpart; beside it W_r^T, which dx will want;
//   dWd (+)= Hg^T dy, dWg (+)= X^T dA, dWu (+)= X^T dB per expert, X the rows of x read through tok, or Xp if given;
//   dXp = dA Wg^T + dB Wu^T.
// `tiles` is the table of mfma_build_tiles_and_row_tokens(); if that was built with split_rows > 0, `part` is the place for the partial
// products of the weight gradients (dXp's own, which is written after they are added), else NULL.
struct FfnBackward {
    int64_t S;
    int T, d, E, F, K, accumulate, row_parts;
    const int32_t *offsets, *tiles, *tok, *inv_perm;
    const float *grow, *gates;
    const void *dy, *x, *Xp, *FA, *FB, *H, *Wg, *Wu, *Wd, *Wr;
    void *dA, *dB, *Hg, *dXp, *WrT;
    float *wpart, *dz, *dzrow, *part, *dWg, *dWu, *dWd;
};
hipError_t mfma_ffn_backward(const FfnBackward &b, hipStream_t s);
size_t mfma_row_tokens_bytes(int64_t S);
hipError_t mfma_router_logits(int T, int d, int E, const void *x, const void *Wr, const float *bias,
                              float *logits, hipStream_t s);

}  // namespace r3
