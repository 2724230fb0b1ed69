// Dense steps of the replayed MoE layer on bf16 MFMA (gfx950):
//   router logits  s = x W_r                       (Section 4.1, first equation)
//   grouped SwiGLU expert FFN, forward              (the E_i of the output equation)
//   its data gradients and weight gradients.
// Every kernel is one instance of the tile loop in r3_mfma.h with its own
// operand addressing and epilogue.  Expert segments are ragged: a small kernel
// turns `offsets` into a list of (expert, first row) row tiles on the device, so
// nothing returns to the host between the permutation and the contractions.
#include <type_traits>

#include "r3_kernels.h"
#include "r3_mfma.h"
#include "r3_mfma2.h"
#include "r3_tiles.h"

namespace r3 {

static_assert(kRowTile == kTile, "the tile table's row tiles are the GEMMs'");

// ---------------------------------------------------------------------------
// Tile table (layout in r3_tiles.h), built by one block per pass.
// The weight-gradient kernels' tiles last as long as their expert has rows: taken longest first from a
// shared counter, a heavily loaded expert no longer starts late and finishes alone.  A segment is an
// expert's whole row range, or, when `split_rows` > 0, one of ceil(n / split_rows) equal parts of it
// (a multiple of 32 rows each): under a skewed load one expert's reduction can be longer than a compute
// unit's fair share of the whole launch, and no order of whole experts balances that.  Part 0 of an
// expert has slot -1 (its product goes to the gradient itself), part p > 0 has its own slot >= 0 in a
// scratch array of partial products, which a second launch adds to the gradient in slot order, so the
// result does not depend on which work-group ran what.  Segments that only pad the list to a multiple of
// 8 have slot -2 and are skipped.  At most kMaxSplitSlots slots are handed out (the caller's split_rows
// >= S / kMaxSplitSlots guarantees that this is never the binding limit).
// ---------------------------------------------------------------------------
__device__ __forceinline__ int *tile_counters(const int32_t *tiles, int launch) {
    return const_cast<int *>(tiles) + 2 + 8 * launch;
}
// position of the item of rank `rank` among n (a multiple of 8) when the list is cut into 8 contiguous
// shares: dealt in serpentine order, so that every share holds an equal mix, heaviest first
__device__ __forceinline__ int dealt_position(int rank, int n) {
    const int j = rank >> 3, c = rank & 7;
    return ((j & 1) ? 7 - c : c) * (n >> 3) + j;
}
// rnk[i] = number of items that come before item i when the n items (a multiple of 8) are sorted by descending key, ties
// by index.  A block of 1024 threads; an item's comparisons are shared out among 1024 / n' threads (n' = n
// rounded up to a power of two) and added up in LDS.  (One thread per item walking all n keys is a
// chain of n dependent LDS reads: 6 us at n = 128.)  Bound by the comparisons: four keys a read, and as the items of a wave are neighbours,
// ties matter one way before them and the other way after, so that a comparison is two instructions but for their own.  With the index compared
// every time this kernel took 18.4 us at 384 experts, 11.0 at 256, 9.5 at 128; now 11.9, 8.6 and 8.8.
// keys: 16-byte aligned.
__device__ __forceinline__ int ranked_before(const int32_t *keys, int o0, int o1, int i) {
    const int k = keys[i], w0 = __builtin_amdgcn_readfirstlane(i & ~(kWave - 1));
    int r = 0;
    auto count = [&](int from, int to, auto below) {
        for (int o = from; o < to; o += 4) {
            const int4 m = *(const int4 *)(keys + o);
            r += (m.x > below(o)) + (m.y > below(o + 1)) + (m.z > below(o + 2)) + (m.w > below(o + 3));
        }
    };
    const int a = max(o0, min(o1, w0)), b = max(a, min(o1, w0 + kWave));
    count(o0, a, [&](int) { return k - 1; });
    count(a, b, [&](int o) { return o < i ? k - 1 : k; });
    count(b, o1, [&](int) { return k; });
    return r;
}
__device__ __forceinline__ void block_ranks(int n, const int32_t *keys, int32_t *rnk) {
    for (int i = threadIdx.x; i < n; i += 1024) rnk[i] = 0;
    __syncthreads();
    if (n <= 1024) {
        int np2 = kWave;   // (whole waves share a part)
        while (np2 < n) np2 <<= 1;
        const int sub = 1024 / np2, i = threadIdx.x % np2, part = threadIdx.x / np2;
        const int per = ((n + sub - 1) / sub + 3) & ~3, o0 = min(n, part * per), o1 = min(n, o0 + per);
        if (i < n) {
            const int r = ranked_before(keys, o0, o1, i);
            if (r) atomicAdd(&rnk[i], r);
        }
    } else {
        for (int i = threadIdx.x; i < n; i += 1024) rnk[i] = ranked_before(keys, 0, n, i);
    }
    __syncthreads();
}

__global__ void __launch_bounds__(1024)
build_row_tiles_kernel(int E, int BQ, const int32_t *__restrict__ offsets, int32_t *__restrict__ tiles,
                       int split_rows, int S, int K, const int32_t *__restrict__ inv_perm,
                       const float *__restrict__ gates, int32_t *__restrict__ tok, float *__restrict__ grow) {
    // Work-groups past the first make the row -> token list (and the per-row gates) of the same pass: the
    // two jobs wait for the same inputs and are both too short to be worth a launch of their own.
    if (blockIdx.x > 0) {
        const int slot = (blockIdx.x - 1) * 1024 + threadIdx.x;
        if (slot < S) {
            const int r = inv_perm[slot];
            tok[r] = slot / K;
            grow[r] = gates[slot];
        } else if (slot < S + kRowTokensPad) {
            tok[slot] = 0;
        }
        return;
    }
    __shared__ int32_t start[kMaxE + 1];
    __shared__ int32_t off[kMaxE + 1];
    __shared__ int32_t seg0[kMaxE + 1];     // first segment of expert e
    __shared__ __attribute__((aligned(16))) int32_t seglen[kMaxSegs];    // rows of every segment (-1: padding)
    __shared__ int32_t rnk[kMaxSegs];
    __shared__ int32_t nseg_s;
    // the offsets come in once, in parallel (read one by one by a single thread they cost a memory
    // round trip each, and this kernel sits between two others on every pass)
    for (int e = threadIdx.x; e <= E; e += blockDim.x) off[e] = offsets[e];
    __syncthreads();
    // Row tiles, parts and split experts per expert, then their running sums over the experts: every
    // thread takes kMaxE / 1024 neighbouring experts and the block scans the threads' totals.  (One
    // thread adding them up one after the other pays an LDS round trip per expert: 6 us for 128 experts,
    // in a kernel that sits between two others on every pass.)
    constexpr int PER = kMaxE / 1024;
    constexpr int NS = 3;                    // scanned: row tiles, parts, split experts
    __shared__ int32_t scan[NS][1024];
    int nt[PER], np[PER], tot[NS] = {0, 0, 0};
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int e = PER * threadIdx.x + i;
        const int n = e < E ? off[e + 1] - off[e] : 0;
        nt[i] = (n + BQ - 1) / BQ;
        np[i] = e < E ? (split_rows > 0 ? max(1, (n + split_rows - 1) / split_rows) : 1) : 0;
        tot[0] += nt[i];
        tot[1] += np[i];
        tot[2] += np[i] > 1;
    }
    for (int k = 0; k < NS; ++k) scan[k][threadIdx.x] = tot[k];
    __syncthreads();
    for (int dlt = 1; dlt < 1024; dlt <<= 1) {
        int v[NS];
        for (int k = 0; k < NS; ++k) v[k] = (int)threadIdx.x >= dlt ? scan[k][threadIdx.x - dlt] : 0;
        __syncthreads();
        for (int k = 0; k < NS; ++k) scan[k][threadIdx.x] += v[k];
        __syncthreads();
    }
    const int ntiles = scan[0][1023];
    // more parts than there are slots for (the caller's split_rows rules that out): no splitting at all
    const bool split = scan[1][1023] - E <= kMaxSplitSlots;
    {
        int run[NS];
        for (int k = 0; k < NS; ++k) run[k] = scan[k][threadIdx.x] - tot[k];   // exclusive
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int e = PER * threadIdx.x + i;
            if (e < E) {
                start[e] = run[0];
                seg0[e] = split ? run[1] : e;
                if (split && np[i] > 1) {   // slots are handed out in expert order: segments before e minus experts before e
                    tiles[kTileHot + 1 + 3 * run[2]] = e;
                    tiles[kTileHot + 2 + 3 * run[2]] = run[1] - e;
                    tiles[kTileHot + 3 + 3 * run[2]] = np[i] - 1;
                }
            }
            run[0] += nt[i];
            run[1] += np[i];
            run[2] += np[i] > 1;
        }
    }
    if (threadIdx.x == 1023) {
        const int segs = split ? scan[1][1023] : E;
        start[E] = ntiles;
        seg0[E] = segs;
        tiles[0] = ntiles;
        tiles[kTileHot] = split ? scan[2][1023] : 0;
        nseg_s = (segs + 7) & ~7;
        tiles[1] = nseg_s;
    }
    if (threadIdx.x < 64) tiles[2 + threadIdx.x] = 0;
    __syncthreads();
    if (threadIdx.x <= 8) tiles[kTileX + threadIdx.x] = (int)(((int64_t)ntiles * threadIdx.x) >> 3);
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        const int n = start[e + 1] - start[e];
        for (int i = 0; i < n; ++i) {
            tiles[kTileHdr + 2 * (start[e] + i)] = e;
            tiles[kTileHdr + 1 + 2 * (start[e] + i)] = off[e] + i * BQ;
        }
    }
    if (split_rows < 0) return;   // (a pass with no weight gradients needs no segments)
    const int nseg = nseg_s;
    // part lengths: equal parts, a multiple of 32 rows, the last one takes what is left
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        const int n = off[e + 1] - off[e], parts = seg0[e + 1] - seg0[e];
        const int len = parts > 1 ? ((n + parts - 1) / parts + 31) & ~31 : n;
        for (int p = 0; p < parts; ++p) seglen[seg0[e] + p] = max(0, min(len, n - p * len));
    }
    for (int i = seg0[E] + threadIdx.x; i < nseg; i += blockDim.x) seglen[i] = -1;
    __syncthreads();
    // rank every segment by length (ties by position) and write it where it is dealt to
    block_ranks(nseg, seglen, rnk);
    for (int e = threadIdx.x; e < E; e += blockDim.x) {
        const int n = off[e + 1] - off[e], parts = seg0[e + 1] - seg0[e];
        const int len = parts > 1 ? ((n + parts - 1) / parts + 31) & ~31 : n;
        const int slot = seg0[e] - e;   // slots were handed out in expert order (used if parts > 1)
        for (int p = 0; p < parts; ++p) {
            const int i = seg0[e] + p, m = seglen[i];
            int32_t *sg = tiles + kTileSeg + 4 * dealt_position(rnk[i], nseg);
            const int r0 = off[e] + min(p * len, n);
            sg[0] = e;
            sg[1] = r0;
            sg[2] = r0 + m;
            sg[3] = p == 0 ? -1 : slot + p - 1;
        }
    }
    for (int i = seg0[E] + threadIdx.x; i < nseg; i += blockDim.x) {
        int32_t *sg = tiles + kTileSeg + 4 * dealt_position(rnk[i], nseg);
        sg[0] = 0; sg[1] = 0; sg[2] = 0; sg[3] = -2;
    }
}

static inline int max_row_tiles(int64_t S, int E, int BQ) { return (int)(S / BQ) + E; }

// Grid of a persistent launch: one work-group per compute unit of the current device (a
// multiple of 8, so that every XCD gets the same number), fewer when there are fewer tiles.
static int device_cus() {
    static int cus[64] = {0};
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) dev = 0;
    if (cus[dev] == 0) {
        int n = 0;
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 8) n = 256;
        cus[dev] = n / 8 * 8;
    }
    return cus[dev];
}
static int persistent_grid(int64_t max_tiles) {
    const int cus = device_cus();
    const int64_t g = (max_tiles + 7) / 8 * 8;
    return (int)(g < cus ? g : cus);
}

__device__ __forceinline__ uint2 pack4(float a, float b, float c, float d) {
    return make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
}
__device__ __forceinline__ void unpack4(uint2 v, float *f) {
    f[0] = __uint_as_float(v.x << 16);
    f[1] = __uint_as_float(v.x & 0xffff0000u);
    f[2] = __uint_as_float(v.y << 16);
    f[3] = __uint_as_float(v.y & 0xffff0000u);
}

// ---------------------------------------------------------------------------
// FFN, first contraction + SwiGLU:  A = Xp Wg, B = Xp Wu, H = silu(A) * B.
// The P operand is two 128-feature sub-tiles, one of W_gate and one of W_up, at
// the same features, so a wave holds both pre-activations of a (row, feature)
// pair in the same lane: MFMA tiles 0..3 are gate, tiles 4..7 the matching up.
// What is saved for the backward are not A and B but the two factors its SwiGLU
// step multiplies dh with: FA = B silu'(A) (dA = dh FA) and FB = silu(A)
// (dB = dh FB); the sigmoid is in registers here anyway, and the backward's
// epilogue is left with two multiplications per element.
// ---------------------------------------------------------------------------
// RAGGED (this and the following expert GEMMs): widths that are multiples of 8 but not of the tile.  Loads past
// a matrix's end read zero by the buffer bounds, chunks past the end of a reduction are masked (OpKC64's TAIL),
// features past an output's width are computed on whatever their columns hold and not stored.  The flag is a
// template parameter because the whole-tile kernels have no registers to spare for the guards.
// T=3001 d=1000 E=64 K=6 F=704, forward + backward: 4.2 ms on f32 tiles, 0.72 ms on these.  Their sigmoid is expf and a
// division, as on the f32 tiles: the exponential of sigmoid_fast is off by tens of ulp at arguments below -50.
template <bool GATHER, bool RAGGED>
__global__ void __launch_bounds__(kThreads2, kMinWavesPerSimd)
ffn1_kernel(int S, int d, int F, const bf16_t *__restrict__ Xp, const int32_t *__restrict__ perm, int K, int T,
            const int32_t *__restrict__ offsets, const int32_t *__restrict__ tiles, const bf16_t *__restrict__ Wg,
            const bf16_t *__restrict__ Wu, bf16_t *__restrict__ H, bf16_t *__restrict__ FA, bf16_t *__restrict__ FB,
            const float *__restrict__ grow, int stream) {
    __shared__ __attribute__((aligned(1024))) char lds[kRowLds];   // one piece: a tail tile lays it out differently
    char *const bufA = lds, *const bufB = lds + kSuperBytes;
    char *const s0 = bufA, *const s1 = bufA + kStageBytes, *const s2 = bufB, *const s3 = bufB + kStageBytes;
    constexpr int BF = 128;  // features per tile
    const int npt = RAGGED ? (F + BF - 1) / BF : F / BF, nw = RAGGED ? (d + kBK3 - 1) / kBK3 : d / kBK3;
    OpTR128x2<!RAGGED> P;
    P.init(F * 2, 0, 64 * ((threadIdx.x >> 6) % kWP2));
    __shared__ int4 qstash[GATHER ? 2 * 256 : 1];   // the gathered rows' offsets (no registers to spare for them)
    OpKC64<GATHER, GATHER, false, RAGGED> Q;
    Q.init(d * 2, kWaveRowsQ * ((threadIdx.x >> 6) / kWP2), qstash);
    if constexpr (RAGGED) Q.set_tail(d);
    __shared__ int mailbox[2];
    __shared__ __attribute__((aligned(256))) char gates_lds[RAGGED ? 4 : 4 * kTile];
    RowTileLoop tl(tiles + kTileX, npt, tile_counters(tiles, 0));
    struct Tile {
        int e, row0, row_end, f0;
    };
    auto decode = [&](int slot_) {
        const int id = tl.id(slot_);
        const int tile = id / npt, pt = id - tile * npt;
        Tile t;
        t.e = tiles[kTileHdr + 2 * tile];
        t.row0 = tiles[kTileHdr + 1 + 2 * tile];
        t.row_end = offsets[t.e + 1];
        t.f0 = pt * BF;
        return t;
    };
    auto aim = [&](const Tile &t) {   // point the operands at a tile
        const int64_t wb = ((int64_t)d * F - t.f0) * 2;
        P.src[0] = Src{(const char *)(Wg + (int64_t)t.e * d * F + t.f0), clamp_bytes(wb), (uint32_t)(kBK2 * F * 2)};
        P.src[1] = Src{(const char *)(Wu + (int64_t)t.e * d * F + t.f0), clamp_bytes(wb), (uint32_t)(kBK2 * F * 2)};
        if constexpr (GATHER) {
            // dispatch folded into the tile load: `Xp` is x [T,d]; each lane's eight rows of the tile
            // are read from their tokens' rows (rows past the end of the permutation repeat the last
            // one; they are never stored)
            Q.set_source(0, Xp, clamp_bytes((int64_t)T * d * 2));
            const int chunk = Q.lane_chunk();
            int v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = (perm[min(t.row0 + Q.lane_row(i), S - 1)] / K) * (d * 2) + chunk;
            Q.set_rows(v);
        } else {
            Q.set_source(0, Xp + (int64_t)t.row0 * d, clamp_bytes((int64_t)(S - t.row0) * d * 2));
        }
    };
    if (!tl.valid(tl.first())) return;
    Tile cur = decode(tl.first());
    aim(cur);
    for (int slot = tl.first(), next = tl.second(); tl.valid(slot);) {
    // the next tile's coordinates are fetched now (scalar loads), a whole tile before their use
    const bool more = tl.valid(next);
    const Tile nxt = more ? decode(next) : cur;
    const int row0 = cur.row0, row_end = cur.row_end, f0 = cur.f0;
    {   // lane constants made anew for every tile (see rowgemm_kernel)
        const int t0 = opaque_tid();
        Q.set_lane(d * 2, kWaveRowsQ * ((t0 >> 6) / kWP2), t0, qstash);
    }

    if (!RAGGED && grow) issue_row_gates(grow, row0, S, gates_lds);
    Acc2 acc;
    zero_acc2(acc);
    if (row_end - row0 <= kTailRows) mfma_tail_loop3(acc, nw, P, Q, lds, row_end - row0);
    else mfma_mainloop3<!RAGGED>(acc, nw, P, Q, lds, row_end - row0);
    tl.prefetch();
    if (more) aim(nxt);   // here, so that the row-index loads of a gathered tile hide behind the epilogue

    // per wave: 64 rows x 64 features of H (and FA, FB), 32 rows at a time through LDS
    // (three patches, so that one tensor's stores and the next one's deposits overlap); a tail tile: 64 or 32 rows x 32
    const int tid = opaque_tid();
    const int lane = tid & 63;
    const WaveTile wt(row_end - row0, tid);
    char *patch = wave_patch(s0, s1, s2, s3, tid);
    const int r16 = lane & 15, f4 = (lane >> 4) * 4;   // a lane's row and four features of every 16 x 16 tile
    const bool save = FA != nullptr;
    // two copies: with the tail's conditions in it a full tile's came out 4 % slower; one at ragged widths, where two, with
    // expf and a division each, outgrow the instruction cache (8 % slower)
    auto epilogue = [&](auto is_tail) {
        const bool tail = is_tail;
        const int fw = f0 + (tail ? 32 * wt.quarter : 64 * ((tid >> 6) % kWP2));   // the wave's first feature
#pragma unroll
        for (int blk = 0; blk < kWaveRowsQ / 32; ++blk) {
            if (tail && blk >= wt.blocks) continue;
            const int brow = row0 + wt.row + blk * 32;             // first row of this block
            const int valid = min(32, row_end - brow);             // may be <= 0
            const int64_t o = ((int64_t)brow * F + fw) * 2;        // byte offset of the block
            RowStage<128> sh{patch, tid}, sa{patch + RowStage<128>::BYTES, tid}, sb{patch + 2 * RowStage<128>::BYTES, tid};
            // grow != NULL: H leaves as g H, g the gate of the row's slot (the down projection then yields
            // gated rows and the gradient of W_down finds its row operand ready); FA and FB are not scaled
            // (at ragged widths straight from memory: few windows hide the way through LDS, 2000 tokens top-4, 264 x 392, 16 experts 23.0 us, from
            // memory 22.1; 3001 top-6, 1000 x 704, 64 experts, forward 184.1 and 182.6)
            float2 gates = make_float2(1.0f, 1.0f);
            if (grow) {
                if constexpr (RAGGED) gates = make_float2(grow[min(brow + r16, S - 1)], grow[min(brow + 16 + r16, S - 1)]);
                else gates = row_gates(gates_lds, wt.row + blk * 32 + r16);
            }
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const int tq = 2 * blk + t, q = 16 * t + r16;
                const float gq = t ? gates.y : gates.x;
#pragma unroll
                for (int tp = 0; tp < kHalfP; ++tp) {
                    if (tp >= 2 && tail) continue;
                    float h[4], fa[4], fb[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float a = acc[tp][tq][i], b = acc[tp + kHalfP][tq][i];
                        const float sg = RAGGED ? sigmoidf_(a) : sigmoid_fast(a);
                        fb[i] = a * sg;                                  // silu(a)
                        h[i] = gq * (fb[i] * b);
                        fa[i] = b * fmaf(fb[i], 1.0f - sg, sg);          // b silu'(a), silu'(a) = sg (1 + a (1 - sg))
                    }
                    const int bo = (tp * 16 + f4) * 2;
                    sh.put8(q, bo, pack4(h[0], h[1], h[2], h[3]));
                    if (save) {
                        sa.put8(q, bo, pack4(fa[0], fa[1], fa[2], fa[3]));
                        sb.put8(q, bo, pack4(fb[0], fb[1], fb[2], fb[3]));
                    }
                }
            }
            const int whole = tail ? 64 : 128, width = RAGGED ? min(whole, (F - fw) * 2) : whole;
            sh.flush((char *)H + o, (int64_t)F * 2, valid, width, stream);
            if (save) {
                sa.flush((char *)FA + o, (int64_t)F * 2, valid, width, stream);
                sb.flush((char *)FB + o, (int64_t)F * 2, valid, width, stream);
            }
        }
    };
    if constexpr (RAGGED) epilogue(wt.quarter >= 0);
    else if (wt.quarter >= 0) epilogue(std::true_type{});
    else epilogue(std::false_type{});
    const int after = tl.finish(mailbox);
    slot = next;
    next = after;
    cur = nxt;
    }
}

// ---------------------------------------------------------------------------
// Row-ragged contraction with a plain or SwiGLU-backward epilogue:
//   out[row][p0+p] = sum_k Q[row][k] * Pmat[e](p, k)
// MODE 0: Yp = H Wd          P from Wd[e] [F,d]  (TR: k rows, features c), K = F
// MODE 1: u = dy Wd^T        P from Wd[e] [F,d]  (KC: feature rows f),      K = d
//         The Q rows are the upstream gradient's rows read through the row -> token list (row r is
//         dy[tok[r]]): the gated copy g*dy of every slot is never written.  Epilogue, with g the
//         row's gate, FA = B silu'(A) and FB = silu(A) saved by the forward:
//           dA = g u FA,  dB = g u FB,  Hg = g H  (the row operand of dW_down = Hg^T dy),
//           wpart[row][2 pt + wp] = g * sum over this wave's 128 features of u H
//         The parts of a row add up to g <dy, o> = g dg (o = H Wd: <dy, H Wd> = <dy Wd^T, H>), which is
//         all the masked-softmax backward needs, so the expert outputs are not read again either.
//         GATED: the forward already stored g H in place of H (one-call forward); the parts are then
//         sums of u (g H) and nothing is written for H.
// MODE 2: dXp = dA Wg^T + dB Wu^T   P from Wg[e], Wu[e] [d,F] (KC: rows c), K = 2F
//         (two-phase reduction: first F over (dA, Wg), then F over (dB, Wu))
// ---------------------------------------------------------------------------
template <int MODE, bool GATED, bool RAGGED>
__device__ __forceinline__ void
rowgemm_tiles(char *lds, int4 *qstash, char *gates_lds, int *mailbox, int S, int d, int F, const bf16_t *__restrict__ Q0, const bf16_t *__restrict__ Q1,
               const int32_t *__restrict__ offsets, const int32_t *__restrict__ tiles,
               const bf16_t *__restrict__ W0, const bf16_t *__restrict__ W1, const bf16_t *__restrict__ FA,
               const bf16_t *__restrict__ FB, bf16_t *__restrict__ out0, bf16_t *__restrict__ out1,
               const int32_t *__restrict__ tok, int T, const float *__restrict__ grow,
               const bf16_t *__restrict__ Hs, bf16_t *__restrict__ out2, float *__restrict__ wpart, int stream) {
    char *const bufA = lds, *const bufB = lds + kSuperBytes;
    char *const s0 = bufA, *const s1 = bufA + kStageBytes, *const s2 = bufB, *const s3 = bufB + kStageBytes;
    const int NOUT = (MODE == 1) ? F : d;  // width of the output
    const int KQ = (MODE == 1) ? d : F;    // width of the Q source rows
    const int npt = RAGGED ? (NOUT + kTile - 1) / kTile : NOUT / kTile;
    const int nwk = RAGGED ? (KQ + kBK3 - 1) / kBK3 : KQ / kBK3;   // windows of 64 k
    const int nw = (MODE == 2) ? 2 * nwk : nwk;
    const int wp0 = (threadIdx.x >> 6) % kWP2, wq0 = (threadIdx.x >> 6) / kWP2;
    // operand forms: the weights are feature-contiguous (TR) for MODE 0, K-contiguous otherwise
    typedef typename std::conditional<MODE == 0, OpTR256<!RAGGED>, OpKC64<false, false, !RAGGED, RAGGED>>::type POp;
    constexpr bool GATHER = MODE == 1;     // Q rows through the row -> token list (their offsets in qstash: no registers to spare for them)
    POp P;
    OpKC64<GATHER, GATHER, false, RAGGED> Q;
    if constexpr (MODE == 0) {
        P.init(d * 2, 0, 128 * wp0);
    } else {
        P.init((MODE == 1 ? d : F) * 2, 128 * wp0);
        if constexpr (MODE == 2) P.wswitch = nwk;
        if constexpr (RAGGED) P.set_tail(KQ);
    }
    Q.init(KQ * 2, kWaveRowsQ * wq0, qstash);
    if constexpr (MODE == 2) Q.wswitch = nwk;
    if constexpr (RAGGED) Q.set_tail(KQ);
    RowTileLoop tl(tiles + kTileX, npt, tile_counters(tiles, MODE == 1 ? 0 : 1));
    struct Tile {
        int e, row0, row_end, p0;
    };
    auto decode = [&](int slot_) {
        const int id = tl.id(slot_);
        const int tile = id / npt, pt = id - tile * npt;
        Tile t;
        t.e = tiles[kTileHdr + 2 * tile];
        t.row0 = tiles[kTileHdr + 1 + 2 * tile];
        t.row_end = offsets[t.e + 1];
        t.p0 = pt * kTile;
        return t;
    };
    auto aim = [&](const Tile &t) {   // point the operands at a tile
        const bf16_t *w0 = W0 + (int64_t)t.e * d * F;
        if constexpr (GATHER) {
            // each lane's eight rows of the tile come from their tokens' rows of Q0 [T, KQ] (rows past the
            // end of the list read token 0: the list is padded with zeros; they are never stored)
            Q.set_source(0, Q0, clamp_bytes((int64_t)T * KQ * 2));
            const int chunk = Q.lane_chunk();
            int v[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] = tok[min(t.row0 + Q.lane_row(i), S)] * (KQ * 2) + chunk;
            Q.set_rows(v);
        } else {
            Q.set_source(0, Q0 + (int64_t)t.row0 * KQ, clamp_bytes((int64_t)(S - t.row0) * KQ * 2));
        }
        if constexpr (MODE == 2) Q.set_source(1, Q1 + (int64_t)t.row0 * KQ, clamp_bytes((int64_t)(S - t.row0) * KQ * 2));
        if constexpr (MODE == 0) {
            P.src = Src{(const char *)(w0 + t.p0), clamp_bytes(((int64_t)d * F - t.p0) * 2), (uint32_t)(kBK2 * d * 2)};
        } else if constexpr (MODE == 1) {
            P.set_source(0, w0 + (int64_t)t.p0 * d, clamp_bytes((int64_t)(F - t.p0) * d * 2));
        } else {
            const bf16_t *w1 = W1 + (int64_t)t.e * d * F;
            P.set_source(0, w0 + (int64_t)t.p0 * F, clamp_bytes((int64_t)(d - t.p0) * F * 2));
            P.set_source(1, w1 + (int64_t)t.p0 * F, clamp_bytes((int64_t)(d - t.p0) * F * 2));
        }
    };
    if (!tl.valid(tl.first())) return;
    Tile cur = decode(tl.first());
    if constexpr (GATHER) aim(cur);
    for (int slot = tl.first(), next = tl.second(); tl.valid(slot);) {
    // the next tile's coordinates are fetched now (scalar loads), a whole tile before their use
    const bool more = tl.valid(next);
    const Tile nxt = more ? decode(next) : cur;
    const int row0 = cur.row0, row_end = cur.row_end, p0 = cur.p0;
    if constexpr (!GATHER) aim(cur);
    if constexpr (MODE == 1) {
        // the operands' lane constants are made anew for every tile, from a thread index the compiler
        // cannot trace: kept across tiles they are live through the epilogue, the fullest part of this
        // kernel, and are then spilled, with reloads in the tile loop that wait on the tile loads
        const int t0 = opaque_tid();
        P.set_lane(d * 2, 128 * ((t0 >> 6) % kWP2), t0);
        Q.set_lane(KQ * 2, kWaveRowsQ * ((t0 >> 6) / kWP2), t0, qstash);
    }
    if constexpr (MODE == 0 && RAGGED) {   // likewise: the guards of ragged widths need the registers
        const int t0 = opaque_tid();
        Q.set_lane(KQ * 2, kWaveRowsQ * ((t0 >> 6) / kWP2), t0);
    }

    if constexpr (MODE == 1) issue_row_gates(grow, row0, S, gates_lds);
    Acc2 acc;
    zero_acc2(acc);
    if (row_end - row0 <= kTailRows) mfma_tail_loop3(acc, nw, P, Q, lds, row_end - row0);
    else mfma_mainloop3<!RAGGED>(acc, nw, P, Q, lds, row_end - row0);
    tl.prefetch();
    if constexpr (GATHER)
        if (more) aim(nxt);   // here, so that the row-index loads of the next tile hide behind the epilogue

    // per wave: 64 rows x 128 features, 32 rows at a time through LDS; a tail tile: 64 or 32 rows x 64
    const int tid = opaque_tid();
    const int lane = tid & 63;
    const WaveTile wt(row_end - row0, tid);
    const bool tail = wt.quarter >= 0;
    const int wp = tail ? wt.quarter >> 1 : (tid >> 6) % kWP2;         // the wave's 128 features, of which a tail tile's wave
    const int pw = tail ? 64 * wt.quarter : 128 * wp;                  // has the first or the second half
    RowStage<256> st{wave_patch(s0, s1, s2, s3, tid), tid};
    const int r16 = lane & 15, f4 = (lane >> 4) * 4;   // a lane's row and four features of every 16 x 16 tile
    const int whole = tail ? 128 : 256, width = RAGGED ? min(whole, (NOUT - p0 - pw) * 2) : whole;   // bytes of the wave's features
    if constexpr (MODE == 1) {
        // Rounds of 32 rows x 64 features (four, a tail tile two or one), each in three phases: FA -> dA, FB -> dB, H -> g H and the
        // row's dot product.  A phase's rows come in row-contiguously into a patch, each lane replaces
        // exactly the quads it read, and the patch goes out row-contiguously.  The rows of the next phase
        // are asked for while this one is worked on (three phases ahead, straight into LDS: this kernel 0-2 % faster,
        // no step any faster, so it is not what the epilogue waits for; through registers that spills).  A lane's products u H of one
        // 32-row block belong to two rows (r16 and 16 + r16).
        typedef RowStage<128> Patch;
        const Patch sa{st.base, tid}, sb{st.base + Patch::BYTES, tid}, sh{st.base + 2 * Patch::BYTES, tid};
        // A row's dot product is summed per 64 features and those sums are added in pairs, in a full tile (whose waves have both) as in a
        // tail: a row's dz is the same bits whichever kind of tile its expert's other rows make it.
        float *const whalf = (float *)(st.base + 3 * Patch::BYTES);   // the wave's first sums
        constexpr int NR = 2 * (kWaveRowsQ / 32);   // (GATED: the H phases only read)
        auto where = [&](int r, int &valid) -> int64_t {
            const int brow = row0 + wt.row + (r >> 1) * 32;
            valid = min(32, row_end - brow);
            return ((int64_t)brow * NOUT + p0 + pw) * 2 + (r & 1) * 128;
        };
        auto ask = [&](int r, int which) -> Patch::Rows {
            int valid;
            const int64_t o = where(r, valid);
            const char *src = which == 0 ? (const char *)FA : which == 1 ? (const char *)FB : (const char *)Hs;
            return sa.fetch(src + o, (int64_t)NOUT * 2, valid, width - 128 * (r & 1));
        };
        Patch::Rows rr = ask(0, 0);
        float gq[2] = {0.0f, 0.0f}, wsum[2] = {0.0f, 0.0f};
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            const int blk = r >> 1, half = r & 1;
            if (blk >= wt.blocks || (half && tail)) continue;
            const int brow = row0 + wt.row + blk * 32;
#pragma unroll
            for (int which = 0; which < 3; ++which) {
                const Patch &sp = which == 0 ? sa : which == 1 ? sb : sh;
                int valid;
                const int64_t oh = where(r, valid);
                sp.deposit(rr);
                if (which < 2) rr = ask(r, which + 1);
                else if (r + 1 < NR) {
                    const int rn = tail ? r + 2 : r + 1;   // the wave's next round
                    if ((rn >> 1) < wt.blocks) rr = ask(rn, 0);
                }
                if (which == 0) {
                    if (half == 0) {
                        const float2 gates = row_gates(gates_lds, wt.row + blk * 32 + r16);
                        gq[0] = gates.x;
                        gq[1] = gates.y;
                    }
                    wsum[0] = wsum[1] = 0.0f;
                }
#pragma unroll
                for (int t = 0; t < 2; ++t)
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const int tp = half * 4 + g, tq = 2 * blk + t, q = 16 * t + r16;
                        const int bo = (g * 16 + f4) * 2;
                        float v[4], o[4];
                        unpack4(sp.get8(q, bo), v);
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const float u = acc[tp][tq][i];
                            if (which == 2) {
                                wsum[t] = fmaf(u, v[i], wsum[t]);
                                o[i] = gq[t] * v[i];
                            } else {
                                o[i] = gq[t] * u * v[i];
                            }
                        }
                        if (!(GATED && which == 2)) sp.put8(q, bo, pack4(o[0], o[1], o[2], o[3]));
                    }
                bf16_t *dst = which == 0 ? out0 : which == 1 ? out1 : out2;
                if (!(GATED && which == 2)) sp.flush((char *)dst + oh, (int64_t)NOUT * 2, valid, width - 128 * half, stream);
                if (which == 2) {
                    // the four lanes that hold a row add up; lanes 0..15 have the first 16 rows, 16..31 the others
                    float w[2];
#pragma unroll
                    for (int t = 0; t < 2; ++t) {
                        w[t] = wsum[t] + __shfl_xor(wsum[t], 16, 64);
                        w[t] = (GATED ? 1.0f : gq[t]) * (w[t] + __shfl_xor(w[t], 32, 64));
                    }
                    const int q = lane & 31;
                    const float wq = lane < 16 ? w[0] : w[1];
                    if (lane < 32 && half == 0) whalf[32 * blk + q] = wq;
                    else if (lane < 32 && brow + q < row_end) {
#pragma clang fp contract(off)   // (the product with the gate is rounded, as where it passes through LDS)
                        wpart[(int64_t)(brow + q) * (2 * npt) + 2 * (p0 / kTile) + wp] = whalf[32 * blk + q] + wq;
                    }
                }
            }
        }
        if (tail) {   // 128 features' products are two waves': the even one adds its neighbour's
            asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
            const float *other = (const float *)(wave_patch(s0, s1, s2, s3, tid ^ 64) + 3 * Patch::BYTES);
            const int row = row0 + wt.row + lane;
            if (!(wt.quarter & 1) && lane < 32 * wt.blocks && row < row_end)
                wpart[(int64_t)row * (2 * npt) + 2 * (p0 / kTile) + wp] = whalf[lane] + other[lane];
        }
    } else {
#pragma unroll
        for (int blk = 0; blk < kWaveRowsQ / 32; ++blk) {
            if (blk >= wt.blocks) continue;
            const int brow = row0 + wt.row + blk * 32;
            const int valid = min(32, row_end - brow);
            const int64_t o = ((int64_t)brow * NOUT + p0 + pw) * 2;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int tp = 0; tp < kTP2; ++tp) {
                    if (tp >= kTailP && tail) continue;
                    const f32x4_t v = acc[tp][2 * blk + t];
                    st.put8(16 * t + r16, (tp * 16 + f4) * 2, pack4(v[0], v[1], v[2], v[3]));
                }
            st.flush((char *)out0 + o, (int64_t)NOUT * 2, valid, width);
        }
    }
    const int after = tl.finish(mailbox);
    slot = next;
    next = after;
    cur = nxt;
    }
}

// ---------------------------------------------------------------------------
// Weight gradients:  out[e][q][p] (+)= sum_{r in expert e} Qs[r][q] * Ps[r][p]
// Both operands are [row][feature] matrices, so both tiles are TR; the k loop
// runs over the expert's rows and the buffer bound zero-fills the tail.
// ---------------------------------------------------------------------------
// GATHER: Ps is the un-permuted matrix [nrows, NPd] and row r of the reduction is its row tok[r]
// (dW_down = Hg^T dy straight from the upstream gradient: no per-slot copy of dy is read).
// LATE: its work-groups come from other tiles, at different times (TileLoop::join)
template <bool GATHER, bool RAGGED, bool LATE>
__device__ __forceinline__ void
wgrad_tiles(char *s0, char *s1, char *s2, char *s3, char *ring, int *mailbox, int NQd, int NPd, const bf16_t *__restrict__ Qs, const bf16_t *__restrict__ Ps,
             const int32_t *__restrict__ tok, int nrows, const int32_t *__restrict__ tiles,
             float *__restrict__ out, float *__restrict__ part, int accumulate, int *ctr) {
    const int nqt = RAGGED ? (NQd + kTile - 1) / kTile : NQd / kTile, npt = RAGGED ? (NPd + kTile - 1) / kTile : NPd / kTile;
    const int wp0 = (threadIdx.x >> 6) % kWP2, wq0 = (threadIdx.x >> 6) / kWP2;
    // operands are set up once; a tile only moves their source windows (column offset included)
    typename std::conditional<GATHER, OpTR256G, OpTR256<>>::type P;
    OpTR256<> Q;
    if constexpr (GATHER) {
        P.init(NPd * 2, 128 * wp0, ring);
    } else {
        P.init(NPd * 2, 0, 128 * wp0);
    }
    Q.init(NQd * 2, 0, kWaveRowsQ * wq0);
    // tiles of one reduction segment (an expert's rows, or one part of them) are neighbours in the list
    TileLoop tl(tiles[1] * nqt * npt, ctr);
    if constexpr (LATE) tl.join(mailbox + 2);
    for (int slot = tl.first(), next = tl.second(); tl.valid(slot);) {
    const int id = tl.id(slot);
    const int eo = id / (nqt * npt);
    const int rem = id - eo * nqt * npt;
    const int32_t *sg = tiles + kTileSeg + 4 * eo;
    const int e = sg[0], r0 = sg[1], r1 = sg[2], pslot = sg[3];
    const int qt = rem / npt, pt = rem - qt * npt;
    const int q0 = qt * kTile, p0 = pt * kTile;
    if (pslot != -2) {   // (a segment that only pads the list has no tile)
    if constexpr (GATHER) {
        P.aim(Ps, (uint64_t)nrows * NPd * 2, p0 * 2, tok + r0, r1 - r0);
    } else {
        P.src = Src{(const char *)(Ps + (int64_t)r0 * NPd + p0), clamp_bytes(((int64_t)(r1 - r0) * NPd - p0) * 2),
                    (uint32_t)(kBK2 * NPd * 2)};
    }
    Q.src = Src{(const char *)(Qs + (int64_t)r0 * NQd + q0), clamp_bytes(((int64_t)(r1 - r0) * NQd - q0) * 2),
                (uint32_t)(kBK2 * NQd * 2)};

    Acc2 acc;
    zero_acc2(acc);
    mfma_mainloop2(acc, (r1 - r0 + kBK2 - 1) / kBK2, P, Q, s0, s1, s2, s3);
    tl.prefetch();

    // per wave: 64 rows (q) x 128 features (p) of f32, as 32-row x 64-feature blocks through LDS
    const int tid = opaque_tid();
    const int lane = tid & 63, wq = (tid >> 6) / kWP2, wp = (tid >> 6) % kWP2;
    RowStage<256> st{wave_patch(s0, s1, s2, s3, tid), tid};
    const int r16 = lane & 15, f4 = (lane >> 4) * 4;   // a lane's row and four features of every 16 x 16 tile
    // part 0 of an expert's rows goes to the gradient, a later part to its own slot of partial products
    char *o = (char *)(pslot < 0 ? out + (int64_t)e * NQd * NPd : part + (int64_t)pslot * NQd * NPd);
    const int add = pslot < 0 ? accumulate : 0;
    const bool stream = pslot < 0 && (!RAGGED || NPd % 32 == 0);   // (partial products are read again at once)
#pragma unroll
    for (int blk = 0; blk < kWaveRowsQ / 32; ++blk)
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4_t v = acc[half * 4 + g][2 * blk + t];
                    st.put16(16 * t + r16, (g * 16 + f4) * 4, make_float4(v[0], v[1], v[2], v[3]));
                }
            const int64_t off = ((int64_t)(q0 + wq * kWaveRowsQ + blk * 32) * NPd + p0 + wp * 128 + half * 64) * 4;
            if constexpr (RAGGED)
                st.flush_f32(o + off, (int64_t)NPd * 4, NQd - (q0 + wq * kWaveRowsQ + blk * 32), add, stream,
                             (NPd - p0 - wp * 128 - half * 64) * 4);
            else st.flush_f32(o + off, (int64_t)NPd * 4, 32, add, stream);
        }
    } else {
        tl.prefetch();
    }
    const int after = tl.finish(mailbox);
    slot = LATE ? after : next;
    next = after;
    }
}

// ---------------------------------------------------------------------------
// Two weight gradients with a common row operand in one pass:
//   out0[e][q][p] (+)= sum_r Qs[r][q] * P0[r][p],   out1[e][q][p] (+)= sum_r Qs[r][q] * P1[r][p]
// (dW_gate and dW_up: Qs = Xp, P0 = dA, P1 = dB).  The P tile is two 128-feature sub-tiles, one
// of P0 and one of P1 at the same features, as in the forward SwiGLU kernel, so the Xp tile is
// fetched once for both products.
// ---------------------------------------------------------------------------
// GATHER: Qs is the un-permuted matrix [nrows, NQd] and row r of the reduction is its row tok[r]
// (dW_gate, dW_up straight from x: no gathered copy of the tokens is read).
template <bool GATHER, bool RAGGED, bool LATE>
__device__ __forceinline__ void
wgrad_pair_tiles(char *s0, char *s1, char *s2, char *s3, char *ring, int *mailbox, int NQd, int NPd, const bf16_t *__restrict__ Qs, const int32_t *__restrict__ tok, int nrows,
                  const bf16_t *__restrict__ P0, const bf16_t *__restrict__ P1, const int32_t *__restrict__ tiles,
                  float *__restrict__ out0, float *__restrict__ out1, float *__restrict__ part0,
                  float *__restrict__ part1, int accumulate, int *ctr) {
    constexpr int BF = 128;  // features of P0 (and of P1) per tile
    const int nqt = RAGGED ? (NQd + kTile - 1) / kTile : NQd / kTile, npt = RAGGED ? (NPd + BF - 1) / BF : NPd / BF;
    const int wp0 = (threadIdx.x >> 6) % kWP2, wq0 = (threadIdx.x >> 6) / kWP2;
    OpTR128x2<> P;
    P.init(NPd * 2, 0, 64 * wp0);
    typename std::conditional<GATHER, OpTR256G, OpTR256<>>::type Q;
    if constexpr (GATHER) {
        Q.init(NQd * 2, kWaveRowsQ * wq0, ring);
    } else {
        Q.init(NQd * 2, 0, kWaveRowsQ * wq0);
    }
    // reduction segments as in wgrad_kernel: an expert's rows or one part of them
    TileLoop tl(tiles[1] * nqt * npt, ctr);
    if constexpr (LATE) tl.join(mailbox + 2);
    for (int slot = tl.first(), next = tl.second(); tl.valid(slot);) {
    const int id = tl.id(slot);
    const int eo = id / (nqt * npt);
    const int rem = id - eo * nqt * npt;
    const int32_t *sg = tiles + kTileSeg + 4 * eo;
    const int e = sg[0], r0 = sg[1], r1 = sg[2], pslot = sg[3];
    const int qt = rem / npt, pt = rem - qt * npt;
    const int q0 = qt * kTile, p0 = pt * BF;
    if (pslot != -2) {
    const uint64_t pbytes = clamp_bytes(((int64_t)(r1 - r0) * NPd - p0) * 2);
    P.src[0] = Src{(const char *)(P0 + (int64_t)r0 * NPd + p0), pbytes, (uint32_t)(kBK2 * NPd * 2)};
    P.src[1] = Src{(const char *)(P1 + (int64_t)r0 * NPd + p0), pbytes, (uint32_t)(kBK2 * NPd * 2)};
    if constexpr (GATHER) {
        Q.aim(Qs, (uint64_t)nrows * NQd * 2, q0 * 2, tok + r0, r1 - r0);
    } else {
        Q.src = Src{(const char *)(Qs + (int64_t)r0 * NQd + q0), clamp_bytes(((int64_t)(r1 - r0) * NQd - q0) * 2),
                    (uint32_t)(kBK2 * NQd * 2)};
    }

    Acc2 acc;
    zero_acc2(acc);
    mfma_mainloop2(acc, (r1 - r0 + kBK2 - 1) / kBK2, P, Q, s0, s1, s2, s3);
    tl.prefetch();

    const bool stream = pslot < 0 && (!RAGGED || NPd % 32 == 0);   // (partial products are read again at once)
    // per wave: 64 rows (q) x 64 features (p) of each product, 32-row blocks through LDS
    const int tid = opaque_tid();
    const int lane = tid & 63, wq = (tid >> 6) / kWP2, wp = (tid >> 6) % kWP2;
    RowStage<256> st{wave_patch(s0, s1, s2, s3, tid), tid};
    const int r16 = lane & 15, f4 = (lane >> 4) * 4;   // a lane's row and four features of every 16 x 16 tile
#pragma unroll
    for (int blk = 0; blk < kWaveRowsQ / 32; ++blk)
#pragma unroll
        for (int half = 0; half < 2; ++half) {   // MFMA tiles 0..3: first product; 4..7: second
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    const f32x4_t v = acc[half * 4 + g][2 * blk + t];
                    st.put16(16 * t + r16, (g * 16 + f4) * 4, make_float4(v[0], v[1], v[2], v[3]));
                }
            char *o = (char *)(pslot < 0 ? (half ? out1 : out0) + (int64_t)e * NQd * NPd
                                         : (half ? part1 : part0) + (int64_t)pslot * NQd * NPd);
            const int64_t off = ((int64_t)(q0 + wq * kWaveRowsQ + blk * 32) * NPd + p0 + wp * 64) * 4;
            if constexpr (RAGGED)
                st.flush_f32(o + off, (int64_t)NPd * 4, NQd - (q0 + wq * kWaveRowsQ + blk * 32), pslot < 0 ? accumulate : 0, stream,
                             (NPd - p0 - wp * 64) * 4);
            else st.flush_f32(o + off, (int64_t)NPd * 4, 32, pslot < 0 ? accumulate : 0, stream);
        }
    } else {
        tl.prefetch();
    }
    const int after = tl.finish(mailbox);
    slot = LATE ? after : next;
    next = after;
    }
}

// ---------------------------------------------------------------------------
// Launches.  dH and dW_down, dXp and dW_gate/dW_up do not wait for each other: sharing one, a work-group that finds no tile of the first
// left goes on with the second, instead of idling through the first one's last round (the rule is at mfma_ffn_backward).
// ---------------------------------------------------------------------------
struct RowGemmArgs {
    int S, d, F;
    const bf16_t *Q0, *Q1;
    const int32_t *offsets, *tiles;
    const bf16_t *W0, *W1, *FA, *FB;
    bf16_t *out0, *out1;
    const int32_t *tok;
    int T;
    const float *grow;
    const bf16_t *H;
    bf16_t *Hg;
    float *wpart;
    int stream;
};
struct WgradArgs {
    int NQd, NPd;
    const bf16_t *Qs, *P0, *P1;     // (P1: dW_gate and dW_up)
    const int32_t *tok;
    int nrows;
    const int32_t *tiles;
    float *out0, *out1, *part0, *part1;
    int accumulate;
    int *ctr;
};
// Spelled out in the kernels' own parameters: __restrict__ means nothing on a struct's members, and without it tile
// coordinates come in through vector loads (down projection of 16384 tokens 436 -> 450 us).
#define R3_ROWGEMM_PARAMS                                                                                                         \
    int S, int d, int F, const bf16_t *__restrict__ Q0, const bf16_t *__restrict__ Q1, const int32_t *__restrict__ offsets,        \
        const int32_t *__restrict__ tiles, const bf16_t *__restrict__ W0, const bf16_t *__restrict__ W1,                           \
        const bf16_t *__restrict__ FA, const bf16_t *__restrict__ FB, bf16_t *__restrict__ out0, bf16_t *__restrict__ out1,        \
        const int32_t *__restrict__ tok, int T, const float *__restrict__ grow, const bf16_t *__restrict__ Hs,                     \
        bf16_t *__restrict__ Hg, float *__restrict__ wpart, int stream
#define R3_ROWGEMM_ARGS S, d, F, Q0, Q1, offsets, tiles, W0, W1, FA, FB, out0, out1, tok, T, grow, Hs, Hg, wpart, stream
#define R3_ROWGEMM_FIELDS(a)                                                                                                      \
    a.S, a.d, a.F, a.Q0, a.Q1, a.offsets, a.tiles, a.W0, a.W1, a.FA, a.FB, a.out0, a.out1, a.tok, a.T, a.grow, a.H, a.Hg, a.wpart, a.stream

template <bool PAIR, bool GATHER, bool RAGGED, bool LATE>
__device__ __forceinline__ void wgrad_run(char *lds, char *ring, int *mailbox, int NQd, int NPd, const bf16_t *__restrict__ Qs,
                                          const bf16_t *__restrict__ P0, const bf16_t *__restrict__ P1, const int32_t *__restrict__ tok, int nrows,
                                          const int32_t *__restrict__ tiles, float *__restrict__ out0, float *__restrict__ out1,
                                          float *__restrict__ part0, float *__restrict__ part1, int accumulate, int *ctr) {
    char *const s1 = lds + kStageBytes, *const s2 = lds + 2 * kStageBytes, *const s3 = lds + 3 * kStageBytes;
    if constexpr (PAIR)
        wgrad_pair_tiles<GATHER, RAGGED, LATE>(lds, s1, s2, s3, ring, mailbox, NQd, NPd, Qs, tok, nrows, P0, P1, tiles, out0, out1, part0,
                                               part1, accumulate, ctr);
    else
        wgrad_tiles<GATHER, RAGGED, LATE>(lds, s1, s2, s3, ring, mailbox, NQd, NPd, Qs, P0, tok, nrows, tiles, out0, part0, accumulate, ctr);
}
template <int MODE, bool GATED, bool RAGGED>
__global__ void __launch_bounds__(kThreads2, kMinWavesPerSimd) rowgemm_kernel(R3_ROWGEMM_PARAMS) {
    __shared__ __attribute__((aligned(1024))) char lds[kRowLds];   // one piece: a tail tile lays it out differently
    __shared__ int4 stash[MODE == 1 ? 2 * 256 : 1];
    __shared__ __attribute__((aligned(256))) char gates[MODE == 1 ? 4 * kTile : 4];
    __shared__ int mailbox[2];
    rowgemm_tiles<MODE, GATED, RAGGED>(lds, stash, gates, mailbox, R3_ROWGEMM_ARGS);
}
template <bool PAIR, bool GATHER, bool RAGGED>
__global__ void __launch_bounds__(kThreads2, kMinWavesPerSimd)
wgrad_kernel(int NQd, int NPd, const bf16_t *__restrict__ Qs, const bf16_t *__restrict__ P0, const bf16_t *__restrict__ P1,
             const int32_t *__restrict__ tok, int nrows, const int32_t *__restrict__ tiles, float *__restrict__ wout0,
             float *__restrict__ wout1, float *__restrict__ part0, float *__restrict__ part1, int accumulate, int *ctr) {
    __shared__ __attribute__((aligned(1024))) char lds[4 * kStageBytes];
    __shared__ __attribute__((aligned(256))) char ring[GATHER ? kIndexRingBytes : 16];
    __shared__ int mailbox[2];
    wgrad_run<PAIR, GATHER, RAGGED, false>(lds, ring, mailbox, NQd, NPd, Qs, P0, P1, tok, nrows, tiles, wout0, wout1, part0, part1, accumulate, ctr);
}
// MODE 1: dH (of a forward that left H gated), then dW_down; MODE 2: dXp, then dW_gate and dW_up
template <int MODE, bool GATHER, bool RAGGED>
__global__ void __launch_bounds__(kThreads2, kMinWavesPerSimd)
grads_kernel(R3_ROWGEMM_PARAMS, int NQd, int NPd, const bf16_t *__restrict__ Qs, const bf16_t *__restrict__ P0,
             const bf16_t *__restrict__ P1, const int32_t *__restrict__ wtok, int nrows, float *__restrict__ wout0,
             float *__restrict__ wout1, float *__restrict__ part0, float *__restrict__ part1, int accumulate, int *ctr) {
    __shared__ __attribute__((aligned(1024))) char lds[kRowLds];
    __shared__ int4 stash[MODE == 1 ? 2 * 256 : 1];
    __shared__ __attribute__((aligned(256))) char gates[MODE == 1 ? 4 * kTile : 4];
    __shared__ int mailbox[3];
    static_assert(4 * kStageBytes + kIndexRingBytes <= kRowLds, "");
    rowgemm_tiles<MODE, MODE == 1, RAGGED>(lds, stash, gates, mailbox, R3_ROWGEMM_ARGS);
    wgrad_run<MODE == 2, GATHER, RAGGED, true>(lds, lds + 4 * kStageBytes, mailbox, NQd, NPd, Qs, P0, P1, wtok, nrows, tiles, wout0, wout1,
                                               part0, part1, accumulate, ctr);
}

// ---------------------------------------------------------------------------
// Router logits  s[t][e] = sum_c x[t][c] Wr[c][e] (+ bias[e]), f32 out.
// ---------------------------------------------------------------------------
template <class TL>
__global__ void __launch_bounds__(TL::NT)
logits_kernel(int T, int d, int E, const bf16_t *__restrict__ x, const bf16_t *__restrict__ Wr,
              const float *__restrict__ bias, float *__restrict__ logits) {
    extern __shared__ __attribute__((aligned(16))) char lds[];
    const int npt = E / TL::BP;
    const int nqt = (T + TL::BQ - 1) / TL::BQ;
    const int id = blockIdx.x;
    if (id >= nqt * npt) return;
    const int qt = id / npt, pt = id - qt * npt;
    const int t0 = qt * TL::BQ, p0 = pt * TL::BP;
    auto fp = [&](int kt, int k, int c) -> uint4 {
        return ld16(Wr + (int64_t)(kt * TL::BK + k) * E + p0 + c * 8);
    };
    auto fq = [&](int kt, int r, int c) -> uint4 {
        return ld16(x + (int64_t)min(t0 + r, T - 1) * d + kt * TL::BK + c * 8);
    };
    f32x16_t acc[TL::TP][TL::TQ];
    zero_acc<TL>(acc);
    mfma_mainloop<TL, true, false>(acc, d / TL::BK, fp, fq, lds);
    for_each_quad<TL>([&](int tp, int tq, int g, int p, int q) {
        const int t = t0 + q;
        if (t >= T) return;
        float4 v = make_float4(acc[tp][tq][4 * g], acc[tp][tq][4 * g + 1], acc[tp][tq][4 * g + 2],
                               acc[tp][tq][4 * g + 3]);
        if (bias) {
            const float4 b = *(const float4 *)(bias + p0 + p);
            v.x += b.x; v.y += b.y; v.z += b.z; v.w += b.w;
        }
        *(float4 *)(logits + (int64_t)t * E + p0 + p) = v;
    });
}

// ---------------------------------------------------------------------------
// The partial products of split reductions into their gradients: for every split expert, in slot order
// (a fixed order: the sum does not depend on the launch shape).  n4 = float4s per expert matrix; a
// second gradient with slots of its own (out1, part1) is optional.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256)
wgrad_parts_kernel(int64_t n4, const int32_t *__restrict__ tiles, float *__restrict__ out0,
                   const float *__restrict__ part0, float *__restrict__ out1, const float *__restrict__ part1) {
    const int hot = tiles[kTileHot];
    for (int j = 0; j < hot; ++j) {
        const int e = tiles[kTileHot + 1 + 3 * j], s0 = tiles[kTileHot + 2 + 3 * j], ns = tiles[kTileHot + 3 + 3 * j];
        for (int which = 0; which < (out1 ? 2 : 1); ++which) {
            float4 *o = (float4 *)(which ? out1 : out0) + (int64_t)e * n4;
            const float4 *p = (const float4 *)(which ? part1 : part0) + (int64_t)s0 * n4;
            for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n4;
                 i += (int64_t)gridDim.x * blockDim.x) {
                float4 a = o[i];
                for (int q = 0; q < ns; ++q) {
                    const float4 b = p[(int64_t)q * n4 + i];
                    a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
                }
                o[i] = a;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------
typedef TileCfg<128, 64, 2, 2, 64> TLLogits;   // router: 128 experts x 64 tokens

// Rows come in 16-byte pieces (d, F multiples of 8).  Layers of very small matrices and few rows are left to the
// f32 tiles (r3_plain.hip): a 256 x 256 tile of 40 x 40 features is nearly all padding and both paths are a chain of
// launches then.  Where the line lies, forward + backward, bf16 tiles vs f32 tiles: 512 tokens top-4, 16 experts:
// 96 x 96 134 vs 115 us, 128 x 128 136 vs 123, 200 x 128 148 vs 145; 64 tokens: 256 x 64 125 vs 109, 192 x 192
// (64 experts) 140 vs 146; 4096 tokens: 64 x 64 188 vs 210, 320 x 320 (64 experts) 262 vs 762.
bool mfma_ffn_supported(int64_t S, int d, int F) {
    if (d % 8 != 0 || F % 8 != 0) return false;
    const int64_t w = (int64_t)d * F;
    return !(w <= (1 << 15) && S * w <= (1 << 25));
}
bool mfma_ffn_ragged(int d, int F) { return d % kTile != 0 || F % kTile != 0; }
bool mfma_router_supported(int d, int E) { return E % 128 == 0 && d % 128 == 0; }

size_t mfma_tiles_bytes(int64_t S, int E) {
    return align_up((size_t)(kTileHdr + 2 * (size_t)max_row_tiles(S, E, kTile)) * sizeof(int32_t), 256);
}

template <class K>
static void allow_lds(K kernel, int bytes) {
    (void)hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
}

hipError_t mfma_build_tiles(int E, const int32_t *offsets, int32_t *tiles, int split_rows, hipStream_t s) {
    build_row_tiles_kernel<<<1, 1024, 0, s>>>(E, kTile, offsets, tiles, split_rows, 0, 1, nullptr, nullptr, nullptr,
                                              nullptr);
    return hipGetLastError();
}

hipError_t mfma_build_tiles_and_row_tokens(int E, const int32_t *offsets, int32_t *tiles, int split_rows, int S, int K,
                                           const int32_t *inv_perm, const float *gates, int32_t *tok, float *grow,
                                           hipStream_t s) {
    build_row_tiles_kernel<<<1 + (S + kRowTokensPad + 1023) / 1024, 1024, 0, s>>>(E, kTile, offsets, tiles, split_rows,
                                                                                  S, K, inv_perm, gates, tok, grow);
    return hipGetLastError();
}

static int64_t tiles_of(int64_t n, int tile) { return (n + tile - 1) / tile; }

// Whether what the forward saves and what dH leaves go out with the non-temporal hint.  As a rule they do (see RowStage).  Where
// an expert has few rows, a backward is bound by writing the weight gradients, and reading its rows from memory through
// that queue is slow: they are left in the caches then, if they fit.  Kernels, us, streamed | left: 1001 tokens of the
// 2048 x 768 x 128-expert layer, 63 rows per expert, dW_gate/dW_up 318 | 304, 2000 tokens 328 | 308; 6000 tokens of 1024 x 512 x 384, Zipf, dW_down
// 217 | 156.  Training, balanced load, rows per expert and MB of a matrix of rows, us: 2048 x 768 x 128 top-8, 62 and 11 1051 | 1043, 125 and
// 23 1227 | 1218, 187 and 35 1348 | 1335, 250 and 46 1600 | 1602; 1000 x 704 x 64 top-6, 140 and 12 418 | 417, 187 and 16 443 | 445, 281 and 24
// 579 | 583; 1024 x 512 x 384 top-4, 125 and 46 1392 | 1390, 166 and 62 1553 | 1573, 187 and 70 1630 | 1645; 512 x 1280 x 256 top-8, 62 and 39
// 995 | 1010 (the one case found on the wrong side), 125 and 78 1171 | 1193, 187 and 117 1412 | 1443.
static int stream_rows(int64_t S, int E, int F) {
    return !(S < 192 * (int64_t)E && S * F * 2 <= (48ll << 20));
}

// The same for the H of a forward that saves nothing for a backward, which only the down projection reads.  At whole widths H leaves
// with the hint; at ragged ones, where its rows mostly end inside a line, only if it is too large to wait in the caches, or if the pass is
// mostly the stream of more weights than these hold.  Forward pass, us, streamed | left: 393 tokens top-6, d=392 F=592 E=16 57.1 | 53.8; 1000
// tokens top-4, 776 x 1416, 32 experts (211 MB of weights) 131.5 | 126.1; 1000 x 704, 64 experts (270 MB), top-6: 1000 tokens 103.7 | 106.1, 2000
// 134.3 | 133.9, 3001 (25 MB of H) 192.1 | 188.9, 8000 (68 MB) 334.0 | 331.9, 12000 (101 MB) 453.4 | 453.6, 16000 (135 MB) 575.5 | 578.1,
// 32000 (270 MB) 1055.6 | 1073.7.  Whole: 1024 x 768, 64 experts, top-6, 2000 tokens 122.0 | 125.2, 2048 x 768, 128 experts, top-8, 1000
// tokens 266.5 | 269.5.
template <bool RAGGED>
static int stream_unsaved_h(int64_t S, int d, int E, int F) {
    const bool weights = S < 128 * (int64_t)E && 6 * (int64_t)E * d * F > (256ll << 20);
    return !(RAGGED && !weights && S * F * 2 <= (96ll << 20));
}

template <bool GATHER, bool RAGGED>
static void launch_ffn1(int64_t S, int d, int E, int F, const void *Xp, const int32_t *perm, int K, int T,
                        const int32_t *offsets, const int32_t *tiles, const void *Wg, const void *Wu, void *H, void *FA,
                        void *FB, const float *grow, hipStream_t s) {
    const int64_t n = max_row_tiles(S, E, kTile) * tiles_of(F, 128);
    ffn1_kernel<GATHER, RAGGED><<<persistent_grid(n), kThreads2, 0, s>>>(
        (int)S, d, F, (const bf16_t *)Xp, perm, K, T, offsets, tiles, (const bf16_t *)Wg, (const bf16_t *)Wu, (bf16_t *)H,
        (bf16_t *)FA, (bf16_t *)FB, grow, FA ? stream_rows(S, E, F) : stream_unsaved_h<RAGGED>(S, d, E, F));
}

static int64_t rowgemm_grid_tiles(int mode, int64_t S, int d, int E, int F) {
    return max_row_tiles(S, E, kTile) * tiles_of(mode == 1 ? F : d, kTile);
}
static int64_t wgrad_grid_tiles(int E, int NQd, int NPd, bool pair) {
    return (int64_t)(E + kMaxSplitSlots + 8) * tiles_of(NQd, kTile) * tiles_of(NPd, pair ? 128 : kTile);
}
template <int MODE, bool GATED, bool RAGGED>
static void launch_rowgemm(int E, const RowGemmArgs &a, hipStream_t s) {
    rowgemm_kernel<MODE, GATED, RAGGED><<<persistent_grid(rowgemm_grid_tiles(MODE, a.S, a.d, E, a.F)), kThreads2, 0, s>>>(R3_ROWGEMM_FIELDS(a));
}
template <bool PAIR, bool GATHER, bool RAGGED>
static void launch_wgrad(int E, const WgradArgs &w, hipStream_t s) {
    wgrad_kernel<PAIR, GATHER, RAGGED><<<persistent_grid(wgrad_grid_tiles(E, w.NQd, w.NPd, PAIR)), kThreads2, 0, s>>>(
        w.NQd, w.NPd, w.Qs, w.P0, w.P1, w.tok, w.nrows, w.tiles, w.out0, w.out1, w.part0, w.part1, w.accumulate, w.ctr);
}
template <int MODE, bool GATHER, bool RAGGED>
static void launch_grads(int E, const RowGemmArgs &a, const WgradArgs &w, hipStream_t s) {
    const int64_t n = std::max(rowgemm_grid_tiles(MODE, a.S, a.d, E, a.F), wgrad_grid_tiles(E, w.NQd, w.NPd, MODE == 2));
    grads_kernel<MODE, GATHER, RAGGED><<<persistent_grid(n), kThreads2, 0, s>>>(R3_ROWGEMM_FIELDS(a), w.NQd, w.NPd, w.Qs, w.P0, w.P1, w.tok, w.nrows,
                                                                           w.out0, w.out1, w.part0, w.part1, w.accumulate, w.ctr);
}

hipError_t mfma_ffn_forward(int64_t S, int d, int E, int F, const void *Xp, const int32_t *perm, int K, int T,
                            const int32_t *offsets, const int32_t *tiles, const void *Wg, const void *Wu,
                            const void *Wd, void *Yp, void *H, void *FA, void *FB, const float *grow,
                            hipStream_t s) {
    const bool rag = mfma_ffn_ragged(d, F);
    {
        ProfScope ps(PROF_FFN1, s);
        auto f = perm ? (rag ? launch_ffn1<true, true> : launch_ffn1<true, false>)
                      : (rag ? launch_ffn1<false, true> : launch_ffn1<false, false>);
        f(S, d, E, F, Xp, perm, K, T, offsets, tiles, Wg, Wu, H, FA, FB, grow, s);
    }
    ProfScope ps(PROF_FFN2, s);
    RowGemmArgs a = {(int)S, d, F};
    a.Q0 = (const bf16_t *)H; a.offsets = offsets; a.tiles = tiles; a.W0 = (const bf16_t *)Wd; a.out0 = (bf16_t *)Yp; a.stream = stream_rows(S, E, F);
    (rag ? launch_rowgemm<0, false, true> : launch_rowgemm<0, false, false>)(E, a, s);
    return hipGetLastError();
}

// Rows per part of a split reduction for a launch whose segments have `tiles_per_seg` tiles each: a tile
// should not last longer than a third of a compute unit's fair share of the launch (0: never split).
// Never below S / kMaxSplitSlots, so that the slots always suffice.
int mfma_wgrad_split_rows(int64_t S, int tiles_per_seg, size_t part_bytes_available, size_t bytes_per_slot) {
    if (part_bytes_available < (size_t)kMaxSplitSlots * bytes_per_slot) return 0;
    const int cus = device_cus();
    int64_t r = S * tiles_per_seg / (3 * (int64_t)cus);
    r = std::max<int64_t>(r, (S + kMaxSplitSlots - 1) / kMaxSplitSlots);
    r = std::max<int64_t>(r, 2048);
    r = (r + 31) / 32 * 32;
    return r >= S ? 0 : (int)r;
}

// dH and dW_down share a launch where dH does not make dW_down's rows (gated), dXp and dW_gate/dW_up do, unless reductions may be cut into
// parts (whose place is dXp's).  us, each its own launch | shared: 3001 tokens top-6, 1000 x 704, 64 experts, whose launches are 1.4 to 6 rounds
// of tiles, 147 | 130 and 205 | 181, training 594 | 537; 1001 top-8, 2048 x 768, 128 experts 270 | 246 and 462 | 460, 1045 | 1029; training: 1099
// top-2, 176 x 96, 6 experts, Zipf 130 | 105, 20000 top-2, 512 x 1280, 64 experts, Zipf 1308 | 1184, 4096 top-8, 2048 x 768, 128 experts 1639 | 1562,
// 4000 top-8, 768 x 512, 256 experts 723 | 685.  dXp before dW_gate/dW_up: its long tiles end a launch raggedly (3001 tokens 567 instead of 538).  Past some
// 12000 tokens of the 2048 x 768 layer, where skewed reductions are cut, the last rounds are a few per cent of a launch: dH and dW_down of
// 16384 tokens in one, training the same, 65536 Zipf .3 % faster.
hipError_t mfma_ffn_backward(const FfnBackward &b, hipStream_t s) {
    const int E = b.E;
    const bool rag = mfma_ffn_ragged(b.d, b.F), gated = !b.Hg;
    const int64_t n = (int64_t)b.d * b.F;
    RowGemmArgs dh = {(int)b.S, b.d, b.F};
    dh.Q0 = (const bf16_t *)b.dy; dh.offsets = b.offsets; dh.tiles = b.tiles; dh.W0 = (const bf16_t *)b.Wd;
    dh.FA = (const bf16_t *)b.FA; dh.FB = (const bf16_t *)b.FB; dh.out0 = (bf16_t *)b.dA; dh.out1 = (bf16_t *)b.dB;
    dh.tok = b.tok; dh.T = b.T; dh.grow = b.grow; dh.H = (const bf16_t *)b.H; dh.Hg = (bf16_t *)b.Hg; dh.wpart = b.wpart;
    dh.stream = stream_rows(b.S, E, b.F);
    RowGemmArgs dxp = {(int)b.S, b.d, b.F};
    dxp.Q0 = (const bf16_t *)b.dA; dxp.Q1 = (const bf16_t *)b.dB; dxp.offsets = b.offsets; dxp.tiles = b.tiles;
    dxp.W0 = (const bf16_t *)b.Wg; dxp.W1 = (const bf16_t *)b.Wu; dxp.out0 = (bf16_t *)b.dXp; dxp.stream = dh.stream;
    int *ctr = const_cast<int *>(b.tiles) + 2;
    WgradArgs down = {b.F, b.d, (const bf16_t *)(gated ? b.H : b.Hg), (const bf16_t *)b.dy, nullptr, b.tok, b.T, b.tiles, b.dWd, nullptr,
                      b.part, nullptr, b.accumulate, ctr + 8 * 2};
    WgradArgs pair = {b.d, b.F, (const bf16_t *)(b.Xp ? b.Xp : b.x), (const bf16_t *)b.dA, (const bf16_t *)b.dB, b.Xp ? nullptr : b.tok, b.T,
                      b.tiles, b.dWg, b.dWu, b.part, b.part ? b.part + (int64_t)kMaxSplitSlots * n : nullptr, b.accumulate, ctr + 8 * 3};
    if (gated && !b.part) {
        ProfScope ps(PROF_DH, s);
        (rag ? launch_grads<1, true, true> : launch_grads<1, true, false>)(E, dh, down, s);
    } else {
        {
            ProfScope ps(PROF_DH, s);
            auto f = gated ? (rag ? launch_rowgemm<1, true, true> : launch_rowgemm<1, true, false>)
                           : (rag ? launch_rowgemm<1, false, true> : launch_rowgemm<1, false, false>);
            f(E, dh, s);
        }
        ProfScope ps(PROF_WGRAD, s);
        (rag ? launch_wgrad<false, true, true> : launch_wgrad<false, true, false>)(E, down, s);
        if (b.part) wgrad_parts_kernel<<<512, 256, 0, s>>>(n / 4, b.tiles, b.dWd, b.part, nullptr, nullptr);
    }
    hipError_t rc = launch_gate_backward_parts(b.T, b.K, b.row_parts, b.wpart, b.gates, b.inv_perm, b.dz, b.dzrow, b.d, E, b.Wr, b.WrT, s);
    if (rc != hipSuccess) return rc;
    if (!b.part) {
        ProfScope ps(PROF_WGRAD_PAIR, s);
        auto f = b.Xp ? (rag ? launch_grads<2, false, true> : launch_grads<2, false, false>)
                      : (rag ? launch_grads<2, true, true> : launch_grads<2, true, false>);
        f(E, dxp, pair, s);
        return hipGetLastError();
    }
    {
        ProfScope ps(PROF_WGRAD_PAIR, s);
        auto f = b.Xp ? (rag ? launch_wgrad<true, false, true> : launch_wgrad<true, false, false>)
                      : (rag ? launch_wgrad<true, true, true> : launch_wgrad<true, true, false>);
        f(E, pair, s);
        wgrad_parts_kernel<<<512, 256, 0, s>>>(n / 4, b.tiles, b.dWg, b.part, b.dWu, pair.part1);
    }
    ProfScope ps(PROF_DXP, s);
    (rag ? launch_rowgemm<2, false, true> : launch_rowgemm<2, false, false>)(E, dxp, s);
    return hipGetLastError();
}

size_t mfma_row_tokens_bytes(int64_t S) { return (size_t)(S + kRowTokensPad) * sizeof(int32_t); }

hipError_t mfma_router_logits(int T, int d, int E, const void *x, const void *Wr, const float *bias,
                              float *logits, hipStream_t s) {
    typedef TLLogits TL;
    allow_lds(logits_kernel<TL>, TL::LDS_BYTES);
    const int tiles = ((T + TL::BQ - 1) / TL::BQ) * (E / TL::BP);
    ProfScope ps(PROF_LOGITS, s);
    logits_kernel<TL><<<tiles, TL::NT, TL::LDS_BYTES, s>>>(T, d, E, (const bf16_t *)x, (const bf16_t *)Wr, bias,
                                                         logits);
    return hipGetLastError();
}

}  // namespace r3
