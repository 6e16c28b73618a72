// Sparse convolution engine: forward (a4), transposed forward (a5, the same
// kernel on the role-reversed map), input gradient (a6) and weight gradient
// (a7).
//
// Forward / input gradient: output-stationary.  A workgroup owns a tile of
// 128 consecutive output rows and up to 64 output columns, accumulated in
// LDS.  For each offset it finds the pairs whose output row lies in the tile
// through the kernel map's 64-row group index (pairs of one offset are sorted
// by output row, so they are contiguous), gathers the input rows 16 pairs at
// a time as the A operand of an MFMA tile, multiplies by the offset's weight
// and adds the 16 result rows into the LDS tile.  Each output row is written
// to HBM once, with no global atomics and no zero-fill pass.
//
// Weight gradient: split-K over the pairs of each offset.  A workgroup
// reduces a chunk of one offset's pairs into a 64 x 64 fp32 tile (MFMA with
// the pair index as the reduction dimension) and stores it as a partial; a
// second kernel adds the partials of each offset in a fixed order.
#include <climits>
#include <vector>

#include "conv_common.h"
#include "conv_bf16.h"
#include "conv_blk.h"

namespace gsc {

constexpr int kThreads = 256;
constexpr int kTileRows = 128;
constexpr int kTileGroups = kTileRows / GSC_GROUP_ROWS;
constexpr int kColSlice = 64;
constexpr int kAccStride = kColSlice + 1;
constexpr int kDwTile = 64;

// ---------------------------------------------------------------------------
// output-stationary gather -> MFMA -> LDS accumulate
//   Y[sca[p]] += X[gat[p]] * B_w  for every pair p of segment k, w = sel(k)
//   X: n_x x ca, Y: n_y x cb, B_w = W[w] (ca x cb) or W[w]^T.
// ---------------------------------------------------------------------------
template <typename TIn, typename TOut, bool WT, typename Sel>
__global__ void __launch_bounds__(kThreads)
k_conv_os(const TIn* __restrict__ X, int64_t n_x, const TIn* __restrict__ W, const int32_t* __restrict__ gat,
          const int32_t* __restrict__ sca, const int64_t* __restrict__ gidx, int K, int64_t G, int ca,
          int cb, int64_t n_y, TOut* __restrict__ Y, Sel sel) {
    __shared__ float acc[kTileRows * kAccStride];
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int r16 = lane & 15, q = lane >> 4;
    const int64_t tile = xcd_unit(blockIdx.x, gridDim.x);
    const int64_t row0 = tile * kTileRows;
    const int col0 = blockIdx.y * kColSlice;
    const int ncols = min(kColSlice, cb - col0);
    const int nnb = (ncols + 15) >> 4;

    for (int i = tid; i < kTileRows * kAccStride; i += kThreads) acc[i] = 0.f;
    __syncthreads();

    const int64_t g0 = tile * kTileGroups;
    const int64_t g1 = min(g0 + kTileGroups, G);
    int item = 0;
    for (int k = 0; k < K; ++k) {
        const int64_t lo = gidx[(int64_t)k * G + g0];
        const int64_t hi = gidx[(int64_t)k * G + g1];
        const int64_t np = hi - lo;
        for (int64_t pb = 0; pb < np; pb += 16, ++item) {
            if ((item & 3) != wave) continue;
            const int w = sel(k);
            const int64_t p = lo + pb + r16;
            const bool in_grp = pb + r16 < np;
            int32_t gr = in_grp ? gat[p] : 0;
            int32_t sr = in_grp ? sca[p] : 0;
            const bool pv = in_grp && gr >= 0 && gr < n_x && sr >= row0 && sr < row0 + kTileRows;
            floatx4 d[4];
#pragma unroll
            for (int nb = 0; nb < 4; ++nb) d[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
            if constexpr (sizeof(TIn) == 4) {
                // fp32: v_mfma_f32_16x16x4_f32, A[row][kk] = X[gat][kb + kk], lane = (row, kk)
                for (int kb = 0; kb < ca; kb += 4) {
                    const int ch = kb + q;
                    const float a = (pv && ch < ca) ? to_f32(X[(int64_t)gr * ca + ch]) : 0.f;
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb) {
                        if (nb < nnb) {
                            const int col = col0 + nb * 16 + r16;
                            const float b = (ch < ca && col < cb) ? to_f32(w_at<TIn, WT>(W, w, ch, col, ca, cb)) : 0.f;
                            d[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, d[nb], 0, 0, 0);
                        }
                    }
                }
            } else {
                // bf16: v_mfma_f32_16x16x16_bf16, lane = (row, 4 consecutive kk)
                for (int kb = 0; kb < ca; kb += 16) {
                    shortx4 a;
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int ch = kb + 4 * q + e;
                        a[e] = (pv && ch < ca) ? (short)X[(int64_t)gr * ca + ch] : (short)0;
                    }
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb) {
                        if (nb < nnb) {
                            const int col = col0 + nb * 16 + r16;
                            shortx4 b;
#pragma unroll
                            for (int e = 0; e < 4; ++e) {
                                const int brow = kb + 4 * q + e;
                                b[e] = (brow < ca && col < cb) ? (short)w_at<TIn, WT>(W, w, brow, col, ca, cb)
                                                               : (short)0;
                            }
                            d[nb] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(a, b, d[nb], 0, 0, 0);
                        }
                    }
                }
            }
            // D row 4q + j of block nb belongs to pair row 4q + j, column r16
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int prow = 4 * q + j;
                const int32_t srow = __shfl(sr, prow, 64);
                const int valid_row = __shfl((int)pv, prow, 64);
                if (valid_row) {
                    float* a_row = acc + (int)(srow - row0) * kAccStride;
#pragma unroll
                    for (int nb = 0; nb < 4; ++nb)
                        if (nb < nnb && nb * 16 + r16 < ncols) atomicAdd(a_row + nb * 16 + r16, d[nb][j]);
                }
            }
        }
    }
    __syncthreads();
    for (int i = tid; i < kTileRows * ncols; i += kThreads) {
        const int r = i / ncols, c = i - r * ncols;
        const int64_t row = row0 + r;
        if (row < n_y) store_out(Y + row * cb + col0 + c, acc[r * kAccStride + c]);
    }
}

// ---------------------------------------------------------------------------
// fp32 specialisation for reduction width CA and output width CB, one of them 16
// (the other 16, 32 or 64).  Differences from the generic kernel:
//   * the (offset, 16-pair group) items of a tile are split into four
//     contiguous ranges, one per wave, so a wave meets few distinct offsets and
//     keeps the offset's B fragments (CA/4 x CB/16 floats per lane) in
//     registers across its groups;
//   * lane (r16, q) gathers channels [q*CA/4, (q+1)*CA/4) of pair r16's row with
//     16-byte loads; MFMA step s then reduces over channels {q*CA/4 + s}, and B
//     uses the same channel permutation;
//   * the next group's row gather is issued before the current group's MFMAs.
// ---------------------------------------------------------------------------
template <int CA>
struct RowFrag {
    float v[CA / 4];
};

// Branch-free row fragment load: the address is always valid (row is
// clamped by the caller) and invalid pairs are zeroed with a select, so the
// loads of a batch are issued back to back with no wait between them.
template <int CA>
__device__ __forceinline__ void load_row_frag(const float* __restrict__ X, int64_t row, int q, bool ok,
                                              RowFrag<CA>& a) {
    constexpr int KS = CA / 4;
    const floatx4u* src = reinterpret_cast<const floatx4u*>(X + row * CA + q * KS);
#pragma unroll
    for (int i = 0; i < KS / 4; ++i) {
        const floatx4 t = src[i];
        a.v[4 * i + 0] = ok ? t.x : 0.f;
        a.v[4 * i + 1] = ok ? t.y : 0.f;
        a.v[4 * i + 2] = ok ? t.z : 0.f;
        a.v[4 * i + 3] = ok ? t.w : 0.f;
    }
}

constexpr int kMaxKLds = 256;   // offsets whose tile table fits in LDS (specialised kernels)
constexpr int kItemBatch = 4;   // items per wave in flight

// Per-tile offset table in LDS: pairs of offset k in this tile start at
// s_lo[k] (global pair index), there are s_np[k] of them, and its 16-pair
// items are numbered from s_ib[k]; s_ib[K] = items of the tile.
struct TileTable {
    int64_t lo[kMaxKLds];
    int32_t np[kMaxKLds];
    int32_t ib[kMaxKLds + 1];
};

__device__ __forceinline__ void build_tile_table(TileTable& t, const int64_t* __restrict__ gidx, int K, int64_t G,
                                                 int64_t g0, int64_t g1) {
    for (int k = threadIdx.x; k < K; k += kThreads) {
        const int64_t lo = gidx[(int64_t)k * G + g0];
        t.lo[k] = lo;
        t.np[k] = (int32_t)(gidx[(int64_t)k * G + g1] - lo);
    }
    __syncthreads();
    if (threadIdx.x < 64) {   // wave 0: exclusive scan of item counts
        int carry = 0;
        for (int k0 = 0; k0 < K; k0 += 64) {
            const int k = k0 + threadIdx.x;
            const int v = k < K ? (t.np[k] + 15) >> 4 : 0;
            int inc = v;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int u = __shfl_up(inc, d, 64);
                if ((int)threadIdx.x >= d) inc += u;
            }
            if (k < K) t.ib[k] = carry + inc - v;
            carry += __shfl(inc, 63, 64);
        }
        if (threadIdx.x == 0) t.ib[K] = carry;
    }
    __syncthreads();
}

// Wave-per-group fp32 kernel.  Each wave owns one 64-row group of output
// rows (the kernel map's group granularity) and accumulates it in a private
// LDS region with plain read-modify-write: no LDS atomics, no workgroup
// barriers, deterministic order.  The wave's per-offset table (first pair,
// pair count, first item) is held one offset per lane (K <= 64).
constexpr int kWaveKMax = 64;

template <int CA, int CB, bool WT, typename Sel>
__global__ void __launch_bounds__(kThreads)
k_conv_f32(const float* __restrict__ X, int64_t n_x, const float* __restrict__ W, const int32_t* __restrict__ gat,
           const int32_t* __restrict__ sca, const int64_t* __restrict__ gidx, int K, int64_t G, int64_t n_y,
           float* __restrict__ Y, Sel sel) {
    constexpr int KS = CA / 4;
    constexpr int NNB = CB / 16;
    constexpr int AS = CB + 1;
    constexpr int RG = GSC_GROUP_ROWS;
    constexpr int B = kItemBatch;
    static_assert(CA * CB <= 1024, "the registers of a batch");
    __shared__ float acc_all[kThreads / 64][RG * AS];
    const int tid = threadIdx.x;
    const int wave = tid >> 6, lane = tid & 63;
    const int r16 = lane & 15, q = lane >> 4;
    const int64_t g = xcd_unit(blockIdx.x, gridDim.x) * (kThreads / 64) + wave;
    if (g >= G) return;                        // no barrier below, so a wave may leave early
    float* acc = acc_all[wave];
    const int64_t row0 = g * RG;
    for (int i = lane; i < RG * AS; i += 64) acc[i] = 0.f;
    wave_lds_sync();

    // per-offset table, one offset per lane
    int64_t lo = 0;
    int np = 0;
    if (lane < K) {
        lo = gidx[(int64_t)lane * G + g];
        np = (int)(gidx[(int64_t)lane * G + g + 1] - lo);
    }
    const int nit = (np + 15) >> 4;
    int incl = nit;                            // inclusive scan of items over lanes
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const int u = __shfl_up(incl, d, 64);
        if (lane >= d) incl += u;
    }
    const int excl = incl - nit;
    const int total = __shfl(incl, 63, 64);

    // pair indices of the batch starting at item0; every address is valid
    // (lanes past the end of a group re-read its last pair, items past the
    // end repeat the last item) and the invalid ones are masked
    auto fetch_idx = [&](int item0, int (&kb)[B], int32_t (&gr)[B], int32_t (&sr)[B], bool (&ok)[B]) {
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int item = min(item0 + b, total - 1);
            const int k = __popcll(__ballot(incl <= item));     // offset of the item
            kb[b] = k;
            const int64_t klo = __shfl(lo, k, 64);
            const int knp = __shfl(np, k, 64);
            const int pb = (item - __shfl(excl, k, 64)) * 16 + r16;
            const int64_t p = klo + min(pb, knp - 1);
            gr[b] = gat[p];
            sr[b] = sca[p];
            ok[b] = item0 + b < total && pb < knp;
        }
    };
    int kb[B], kbn[B];
    int32_t gr[B], sr[B], grn[B], srn[B];
    bool ok[B], okn[B];
    if (total > 0) fetch_idx(0, kb, gr, sr, ok);
    for (int item0 = 0; item0 < total; item0 += B) {
        // 1. rows and weights of the batch
        RowFrag<CA> a[B];
        float bfr[B][KS][NNB];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            ok[b] = ok[b] && gr[b] >= 0 && gr[b] < n_x && sr[b] >= row0 && sr[b] < row0 + RG;
            load_row_frag<CA>(X, ok[b] ? gr[b] : 0, q, ok[b], a[b]);
            const int w = sel(kb[b]);
            if constexpr (WT) {
                // W[w]^T: lane (r16, q) needs W[w][col][q*KS .. q*KS + KS), contiguous
#pragma unroll
                for (int nb = 0; nb < NNB; ++nb) {
                    const floatx4u* src =
                        reinterpret_cast<const floatx4u*>(W + ((int64_t)w * CB + nb * 16 + r16) * CA + q * KS);
#pragma unroll
                    for (int i = 0; i < KS / 4; ++i) {
                        const floatx4 t = src[i];
                        bfr[b][4 * i + 0][nb] = t.x;
                        bfr[b][4 * i + 1][nb] = t.y;
                        bfr[b][4 * i + 2][nb] = t.z;
                        bfr[b][4 * i + 3][nb] = t.w;
                    }
                }
            } else {
#pragma unroll
                for (int s = 0; s < KS; ++s)
#pragma unroll
                    for (int nb = 0; nb < NNB; ++nb)
                        bfr[b][s][nb] = W[((int64_t)w * CA + q * KS + s) * CB + nb * 16 + r16];
            }
        }
        // 2. next batch's indices in flight during this batch's MFMAs
        if (item0 + B < total) fetch_idx(item0 + B, kbn, grn, srn, okn);
        // 3. group row of each MFMA output row (pair row 4q + j), -1 if none
        int lrow[B][4];
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int mine = ok[b] ? (int)(sr[b] - row0) : -1;
#pragma unroll
            for (int j = 0; j < 4; ++j) lrow[b][j] = __shfl(mine, 4 * q + j, 64);
        }
        // 4. MFMA, then add the 16 result rows into the wave's rows (distinct
        //    within an item; items of the wave are applied in order)
#pragma unroll
        for (int b = 0; b < B; ++b) {
            floatx4 d[NNB];
#pragma unroll
            for (int nb = 0; nb < NNB; ++nb) d[nb] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s)
#pragma unroll
                for (int nb = 0; nb < NNB; ++nb)
                    d[nb] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[b].v[s], bfr[b][s][nb], d[nb], 0, 0, 0);
            wave_lds_sync();   // rows updated by other lanes for earlier items
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if (lrow[b][j] >= 0) {
                    float* arow = acc + lrow[b][j] * AS;
#pragma unroll
                    for (int nb = 0; nb < NNB; ++nb) arow[nb * 16 + r16] += d[nb][j];
                }
            }
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            kb[b] = kbn[b];
            gr[b] = grn[b];
            sr[b] = srn[b];
            ok[b] = okn[b];
        }
    }
    wave_lds_sync();
    // 5. the group's rows, written once
    for (int i = lane; i < RG * CB; i += 64) {
        const int r = i / CB, cc = i - r * CB;
        const int64_t row = row0 + r;
        if (row < n_y) Y[row * CB + cc] = acc[r * AS + cc];
    }
}

// Rows of 32 or 64 channels on both sides.  The kernel above reads an offset's
// weights (16 KB at 64 x 64) for every 16 pairs, four times what it gathers.
// Here a workgroup of four waves owns kWideRows output rows and a wave 16 of
// their columns (with 32 columns, two waves share a column block and take a
// step's halves in turn): its part of an offset's weights stays in registers
// while the offset's pairs in the tile go by, kWidePairs a step, so the 16-pair
// MFMA steps are fuller too (a tile has twice a group's pairs).  The rows are
// gathered once for the four waves into LDS (double buffered, one barrier a
// step; the rows of the next three steps are on their way in registers).  A
// wave adds only to its own columns of the tile's sums in LDS, one offset after
// another, and the pairs of an offset have distinct rows: no atomics, and an
// output row's products are added in increasing offset order.
//
// 239,878 rows, 1.84 M pairs, 64 x 64 (138 us of MFMA time at the clock the
// run holds), each call repeated by itself: forward 346 -> 245 us, input
// gradient 447 -> 269 us, the matrix cores busy for 283 million SIMD cycles (47 %
// at 2.4 GHz); among a block's other kernels 278 and 282 us.  192 or 256 rows a
// tile leave two or one workgroups per CU (295 us).  32 x 32: 123 -> 92 and 161
// -> 104 us, and no shape from 60 to 300,082 rows was faster on the kernel above.
constexpr int kWideRows = 2 * GSC_GROUP_ROWS;   // three workgroups per CU (33 KB of sums and 16 KB of rows each)
constexpr int kWidePairs = 32;                  // pairs of a step

template <int CA, int CB, bool WT, typename Sel, bool EP>
__global__ void __launch_bounds__(kThreads, 2)
k_conv_f32_wide(const float* __restrict__ X, int64_t n_x, const float* __restrict__ W, const int32_t* __restrict__ gat,
                const int32_t* __restrict__ sca, const int64_t* __restrict__ gidx, int K, int64_t G, int64_t n_y,
                float* __restrict__ Y, Sel sel, Epilogue ep) {
    constexpr int CW = CB / 16;                      // the waves' column blocks
    constexpr int HW = 4 / CW;                       // waves of one column block, taking a step's 16-pair halves in turn
    constexpr int KS = CA / 4;
    constexpr int CH = CA / 4;                       // 16-byte chunks of a row
    constexpr int PER = kWidePairs * CH / kThreads;  // chunks a thread gathers per step
    __shared__ __attribute__((aligned(16))) float acc[(kWideRows + 1) * CB];   // and a row for pairs that are none
    __shared__ __attribute__((aligned(16))) floatx4 rows[2][kWidePairs * CH];
    __shared__ __attribute__((aligned(16))) int32_t lrow[2][kWidePairs];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int r16 = lane & 15, q = lane >> 4;
    const int wc = wave % CW, wh = wave / CW;
    const int64_t tile = xcd_unit(blockIdx.x, gridDim.x);
    constexpr int TG = kWideRows / GSC_GROUP_ROWS;
    const int64_t g0 = tile * TG, g1 = min(g0 + TG, G);
    const int64_t row0 = tile * kWideRows;
    for (int i = tid; i < kWideRows * CB / 4; i += kThreads) reinterpret_cast<float4*>(acc)[i] = float4{0.f, 0.f, 0.f, 0.f};

    // the tile's pairs of every offset, one offset per lane (K <= 64)
    int64_t lo = 0;
    int np = 0;
    if (lane < K) {
        lo = gidx[(int64_t)lane * G + g0];
        np = (int)(gidx[(int64_t)lane * G + g1] - lo);
    }
    // steps in offset order (uniform): offset k, pairs [pb, pb + kWidePairs) of it (k = -1 past the last)
    unsigned long long left = __ballot(np > 0);
    unsigned long long wleft = left;   // offsets whose weights have not been asked for
    if (left) {                        // uniform
    int fk = -1, fpb = 0, fnp = 0;     // the front of the walk
    int64_t flo = 0;
    const auto next_step = [&]() __attribute__((always_inline)) {
        fpb += kWidePairs;
        if (fpb >= fnp) {
            fk = left ? __ffsll((long long)left) - 1 : -1;
            left &= left - 1;
            fpb = 0;
            fnp = 0;
            flo = 0;
            if (fk >= 0) {
                fnp = __builtin_amdgcn_readlane(np, fk);
                const uint32_t l0 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)lo, fk);
                const uint32_t l1 = (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)((uint64_t)lo >> 32), fk);
                flo = (int64_t)(((uint64_t)l1 << 32) | l0);
            }
        }
    };
    // Thread t gathers chunk t % CH of every RPI-th row of a step.  Steps go through D slots of registers:
    // a step's rows are loaded D steps ahead, their indices 2 D (with the indices one step ahead of the
    // rows, every step waited for them: 360 us); every step issues the same loads at valid addresses (pairs past an offset's last repeat it, steps past the end read pair 0).
    constexpr int RPI = kThreads / CH;   // rows per round of the block
    constexpr int D = 3;
    const int mine = tid / CH;           // the thread's row of each round
    const floatx4u* Xc = reinterpret_cast<const floatx4u*>(X) + tid % CH;
    int sk[D], spb[D], snp[D];      // the steps whose rows are loaded
    int ik[D], ipb[D], inp[D];      // those whose indices are
    int32_t gr[D][PER], sr[D][PER];
    floatx4 rv[D][PER];
    int32_t lr[D][PER];
    const auto load_idx = [&](auto P) __attribute__((always_inline)) {
        constexpr int j = decltype(P)::value;
        next_step();
        ik[j] = fk;
        ipb[j] = fpb;
        inp[j] = fnp;
        const int32_t *gp = gat + flo, *sp = sca + flo;   // uniform
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const uint32_t p = (uint32_t)max(min(fpb + i * RPI + mine, fnp - 1), 0);
            gr[j][i] = gp[p];
            sr[j][i] = sp[p];
        }
        return false;
    };
    const auto load_rows = [&](auto P) __attribute__((always_inline)) {
        constexpr int j = decltype(P)::value;
        sk[j] = ik[j];
        spb[j] = ipb[j];
        snp[j] = inp[j];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int32_t g = gr[j][i], o = sr[j][i];
            const uint32_t at_row = (uint32_t)o - (uint32_t)row0;
            const bool ok = (spb[j] + i * RPI + mine < snp[j]) & ((uint32_t)g < (uint32_t)n_x) &
                            (at_row < (uint32_t)kWideRows);
            lr[j][i] = ok ? (int32_t)at_row * CB : kWideRows * CB;
            rv[j][i] = Xc[(uint64_t)(ok ? (uint32_t)g : 0u) * CH];
        }
    };
    // weights of offset k for the wave's columns: lane (c, q) holds B_k[q KS + s][16 wc + c]
    float w[KS], wn[KS];
    const auto load_w = [&](int k, float (&v)[KS]) __attribute__((always_inline)) {
        const int m = sel(k);
        if constexpr (WT) {
            const floatx4u* src =
                reinterpret_cast<const floatx4u*>(W + ((int64_t)m * CB + wc * 16 + r16) * CA + q * KS);
#pragma unroll
            for (int i = 0; i < KS / 4; ++i) {
                const floatx4 t = src[i];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * i + e] = t[e];
            }
        } else {
#pragma unroll
            for (int s = 0; s < KS; ++s) v[s] = W[((int64_t)m * CA + q * KS + s) * CB + wc * 16 + r16];
        }
    };
    // chunk c of row r of a step lies at r * CH + c with c's bits exchanged by the row's, so that the 16 rows of
    // an operand read lie in different banks
    const auto at = [](int r, int c) { return r * CH + (c ^ ((r / (16 / CH)) & (CH - 1))); };

    const auto next_w = [&]() __attribute__((always_inline)) {
        const int k = wleft ? __ffsll((long long)wleft) - 1 : 0;
        wleft &= wleft - 1;
        return k;
    };
    run_steps(load_idx, std::make_index_sequence<D>{});
    load_w(next_w(), w);
    load_w(next_w(), wn);
    const auto fill = [&](auto P) __attribute__((always_inline)) {
        load_rows(P);
        load_idx(P);
        return false;
    };
    run_steps(fill, std::make_index_sequence<D>{});
    int buf = 0;
    const auto step = [&](auto P) __attribute__((always_inline)) -> bool {
        constexpr int j = decltype(P)::value;
        const int ck = sk[j], cpb = spb[j], cnp = snp[j];
#pragma unroll
        for (int i = 0; i < PER; ++i) {
            const int r = i * RPI + mine;
            rows[buf][at(r, tid % CH)] = rv[j][i];
            lrow[buf][r] = lr[j][i];   // (the row's lanes write the same)
        }
        load_rows(P);
        load_idx(P);
        __syncthreads();
        const auto operand = [&](int h, float (&a)[KS]) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < KS / 4; ++i) {
                const floatx4 t = rows[buf][at(16 * h + r16, q * (KS / 4) + i)];
#pragma unroll
                for (int e = 0; e < 4; ++e) a[4 * i + e] = t[e];
            }
        };
        float* col = acc + wc * 16 + r16;
        const auto add = [&](const int4& l, const floatx4& d) __attribute__((always_inline)) {
            // the pairs of a step have distinct rows, but for those that are none
            const float s0 = col[l.x], s1 = col[l.y], s2 = col[l.z], s3 = col[l.w];
            col[l.x] = s0 + d[0];
            col[l.y] = s1 + d[1];
            col[l.z] = s2 + d[2];
            col[l.w] = s3 + d[3];
        };
        const int h0 = HW == 1 ? 0 : wh;   // the wave's first half
        if (HW == 1 ? cpb + 16 < cnp : cpb + 16 * h0 < cnp) {   // uniform: both halves hold pairs, or the wave's own
            const int4 l0 = *reinterpret_cast<const int4*>(&lrow[buf][16 * h0 + 4 * q]);
            float a0[KS];
            operand(h0, a0);
            floatx4 d0 = {0.f, 0.f, 0.f, 0.f};
            if constexpr (HW == 1) {
                const int4 l1 = *reinterpret_cast<const int4*>(&lrow[buf][16 + 4 * q]);
                float a1[KS];
                operand(1, a1);
                floatx4 d1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int s = 0; s < KS; ++s) {
                    d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[s], w[s], d0, 0, 0, 0);
                    d1 = __builtin_amdgcn_mfma_f32_16x16x4f32(a1[s], w[s], d1, 0, 0, 0);
                }
                add(l0, d0);
                add(l1, d1);
            } else {
#pragma unroll
                for (int s = 0; s < KS; ++s) d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[s], w[s], d0, 0, 0, 0);
                add(l0, d0);
            }
        } else if (HW == 1) {
            const int4 l0 = *reinterpret_cast<const int4*>(&lrow[buf][4 * q]);
            float a0[KS];
            operand(0, a0);
            floatx4 d0 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int s = 0; s < KS; ++s) d0 = __builtin_amdgcn_mfma_f32_16x16x4f32(a0[s], w[s], d0, 0, 0, 0);
            add(l0, d0);
        }
        buf ^= 1;
        const int k = sk[(j + 1) % D];
        if (k < 0) return true;
        if (k != ck) {   // uniform: on to the next offset's weights, and ask for the ones after them
#pragma unroll
            for (int s = 0; s < KS; ++s) w[s] = wn[s];
            load_w(next_w(), wn);
        }
        return false;
    };
    while (!run_steps(step, std::make_index_sequence<D>{})) {
    }
    }
    __syncthreads();
    for (int i = tid; i < kWideRows * CB / 4; i += kThreads) {
        const int64_t row = row0 + i / (CB / 4);
        if (row >= n_y) continue;
        floatx4 v = reinterpret_cast<const floatx4*>(acc)[i];
        if constexpr (EP) {
            const int c = 4 * (i % (CB / 4));
#pragma unroll
            for (int e = 0; e < 4; ++e)
                v[e] = epi_apply(v[e], ep.scale ? ep.scale[c + e] : 1.f, ep.shift ? ep.shift[c + e] : 0.f, ep.relu);
        }
        reinterpret_cast<floatx4u*>(Y)[row * (CB / 4) + i % (CB / 4)] = v;
    }
}

// ---------------------------------------------------------------------------
// weight gradient
// ---------------------------------------------------------------------------
// Work items of the weight gradient: offset k's pairs are split into chunks
// of `ch` pairs (the last one shorter); ibase[k] = first item of offset k,
// ibase[K] = total.  Equal chunks keep the work items balanced whatever the
// offsets' sizes (the centre offset of a submanifold map has one pair per
// row, the others far fewer).
//
// order[t] (nullable; holds cap items) = the item to run as the t-th: the
// offsets' chunks merged by their place c / n_k in their offset (pairs are
// sorted by output row, so chunks of equal places read about the same rows),
// so that the workgroups of an XCD, which take consecutive t, share the rows
// of one range in its L2 instead of each sweeping all rows for an offset of its
// own.  k_dw_lds_bf16<128, 128>, 3.7 million pairs over 480,288 rows: 296 us
// without, 190 with, 51 % of its requests then hit the L2; the kernels that are
// not bound by the gathers (k_dw_f32, k_dw_bf16, 256 channels) were no faster
// and run without.  The place of an item is counted, not sorted: for every
// offset k', the chunks c' with (2c' + 1) n_k < (2c + 1) n_k' (or equal, and
// k' < k).  Above kDwOrderMaxK offsets, whose counting would take longer than
// the launch (5 us), the items run in their own order.
//
// counter (nullable) is set to 0 on the way (the input gradient's tile
// counter, when that pass runs after this kernel).
constexpr int kDwOrderMaxK = 128;
// Items of up to kDwSplitMax pairs, and those of any size of the float32 kernel
// for any width, are halved while they give fewer than kDwSplitItems workgroups
// (about one per CU; an item has one for each 64 x 64 tile of dW), down to
// kDwSplitMin pairs: an item is a serial chain (3 to 16 channels over 2,000
// rows, 2,430 pairs: the call 80 -> 73 us; 96 x 96 over the same rows the weight
// gradient 94 -> 23 us).  With more items shorter ones cost more than they
// balance (896,000 pairs of 32 x 32 in items of 512: 312 -> 317 us), and bf16
// items of 2048 pairs (128 channels) gain nothing (480,288 pairs of 64 x 128:
// 468 -> 471 us).
constexpr int64_t kDwSplitMax = 1024, kDwSplitMin = 256, kDwSplitItems = 256;
constexpr int kDwItemThreads = 256;

__global__ void __launch_bounds__(kDwItemThreads) k_dw_items(const int64_t* __restrict__ seg, int K, int64_t ch, int64_t split,
                                                             int64_t* __restrict__ ibase, int64_t* __restrict__ chunk,
                                                             int32_t* __restrict__ order, int64_t cap,
                                                             unsigned* counter) {
    __shared__ int64_t base[kMaxKConv + 1];
    // split: items below which they are halved (uniform)
    for (const int64_t pairs = seg[K] - seg[0]; ch > kDwSplitMin && pairs < split * ch;) ch /= 2;
    if (threadIdx.x < 64) {   // 64 offsets per round, their item counts scanned with shuffles
        const int lane = threadIdx.x;
        if (counter && lane == 0 && blockIdx.x == 0) *counter = 0u;
        int64_t carry = 0;
        for (int k0 = 0; k0 < K; k0 += 64) {
            const int k = k0 + lane;
            const int64_t n = k < K ? seg[k + 1] - seg[k] : 0;
            const int64_t c = n > 0 ? (n + ch - 1) / ch : 0;
            int64_t inc = c;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int64_t u = __shfl_up(inc, d, 64);
                if (lane >= d) inc += u;
            }
            if (k < K) base[k] = carry + inc - c;
            carry += __shfl(inc, 63, 64);
        }
        if (lane == 0) base[K] = carry;
    }
    __syncthreads();
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k <= K; k += kDwItemThreads) {
            ibase[k] = base[k];
            if (k < K) chunk[k] = ch;
        }
    const int64_t item = (int64_t)blockIdx.x * kDwItemThreads + threadIdx.x;
    if (!order || item >= min(base[K], cap)) return;
    if (K > kDwOrderMaxK || base[K] > cap) {
        order[item] = (int32_t)item;
        return;
    }
    int k = 0, hi = K - 1;   // last k with base[k] <= item
    while (k < hi) {
        const int mid = (k + hi + 1) >> 1;
        if (base[mid] <= item) k = mid;
        else hi = mid - 1;
    }
    const int64_t nk = base[k + 1] - base[k];
    const double place = (double)(2 * (item - base[k]) + 1), inv = 1.0 / (double)(2 * nk);
    int64_t t = 0;
    for (int o = 0; o < K; ++o) {
        const int64_t no = base[o + 1] - base[o];
        // the quotient is at least 1 / (2 n_k) from an integer or is one; a quarter of that outweighs the rounding
        const double v = place * (double)no + (double)nk - (o < k ? 0.0 : 1.0);
        const int64_t m = (int64_t)floor((v + 0.25) * inv);
        t += m < no ? m : no;
    }
    order[t] = (int32_t)item;
}

// Per-wave partial tiles are summed in wave order (deterministic), then stored.
template <int R, int C>
__device__ __forceinline__ void dw_store_partial(float* sh, const floatx4 (&d)[4][4], int na, int nbk, int wave,
                                                 int q, int r16, int rows, int cols, float* __restrict__ out,
                                                 int64_t ld) {
    constexpr int S = C + 1;
    float* mine = sh + wave * R * S;
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b)
            if (a < na && b < nbk)
#pragma unroll
                for (int j = 0; j < 4; ++j) mine[(16 * a + 4 * q + j) * S + 16 * b + r16] = d[a][b][j];
    __syncthreads();
    for (int i = threadIdx.x; i < rows * cols; i += kThreads) {
        const int r = i / cols, c = i - r * cols;
        float v = sh[r * S + c];
        for (int w = 1; w < kThreads / 64; ++w) v += sh[w * R * S + r * S + c];
        out[r * ld + c] = v;
    }
}

// Generic weight-gradient partial (any dtype, any width): a 16 NA x 16 NB tile
// of X[in]^T dY[out] over one chunk of one offset's pairs, NA or NB 1 where
// that side has at most 16 channels and 4 otherwise.  Bound by the latency of
// its loads: 3 -> 16 channels over 2,000 rows took 38 us with one step of
// 4 pairs at a time (and a tile of 64 x 64 whatever the width), 13 us with
// eight.
template <typename TIn, int NA, int NB>
__global__ void __launch_bounds__(kThreads)
k_dw_partial(const TIn* __restrict__ X, int64_t n_in, const TIn* __restrict__ dY, int64_t n_out,
             const int32_t* __restrict__ in_idx, const int32_t* __restrict__ out_idx, const int64_t* __restrict__ seg,
             const int64_t* __restrict__ ibase, const int64_t* __restrict__ chunk, int K, int ci, int co,
             float* __restrict__ part) {
    constexpr int R = 16 * NA, C = 16 * NB;
    __shared__ float sh[4 * R * (C + 1)];
    int k;
    int64_t p_begin, p_end;
    // the grid covers an upper bound of the items; order the real ones XCD-wise
    if ((int64_t)blockIdx.x >= ibase[K]) return;
    const int64_t item = xcd_unit(blockIdx.x, ibase[K]);
    if (!dw_item(ibase, chunk, seg, K, item, &k, &p_begin, &p_end)) return;
    const int ntj = (co + kDwTile - 1) / kDwTile;
    const int ci0 = (blockIdx.y / ntj) * kDwTile, co0 = (blockIdx.y % ntj) * kDwTile;
    const int na = (min(kDwTile, ci - ci0) + 15) >> 4, nbk = (min(kDwTile, co - co0) + 15) >> 4;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, q = lane >> 4;

    floatx4 d[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) d[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

    if constexpr (sizeof(TIn) == 4) {
        // 4 pairs per MFMA step (reduction index kk = q); the waves interleave
        // groups of U steps, whose row numbers and then rows are loaded together
        // from clamped addresses: one step at a time is a chain of two loads
        // per 4 pairs
        constexpr int U = NA * NB == 1 ? 8 : 4;
        if (n_in < 1 || n_out < 1) p_begin = p_end;   // no row to clamp to
        for (int64_t p0 = p_begin + 4 * U * wave; p0 < p_end; p0 += 16 * U) {
            int32_t g[U], s[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int64_t p = min(p0 + 4 * u + q, p_end - 1);
                g[u] = in_idx[p];
                s[u] = out_idx[p];
            }
            float xa[U][NA], yb[U][NB];
            bool v[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                v[u] = p0 + 4 * u + q < p_end && g[u] >= 0 && g[u] < n_in && s[u] >= 0 && s[u] < n_out;
                const TIn* xr = X + (int64_t)(v[u] ? g[u] : 0) * ci;
                const TIn* yr = dY + (int64_t)(v[u] ? s[u] : 0) * co;
#pragma unroll
                for (int a = 0; a < NA; ++a)
                    if (NA == 1 || a < na) xa[u][a] = to_f32(xr[min(ci0 + 16 * a + r16, ci - 1)]);
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (NB == 1 || b < nbk) yb[u][b] = to_f32(yr[min(co0 + 16 * b + r16, co - 1)]);
            }
            // columns past the widths hold repeats, which are not stored
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int a = 0; a < NA; ++a)
#pragma unroll
                    for (int b = 0; b < NB; ++b)
                        if ((NA == 1 || a < na) && (NB == 1 || b < nbk))
                            d[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[u] ? xa[u][a] : 0.f, v[u] ? yb[u][b] : 0.f,
                                                                          d[a][b], 0, 0, 0);
        }
    } else {
        // 16 pairs per MFMA step: lane (r16, q) supplies pairs 4q .. 4q+3
        for (int64_t p0 = p_begin + 16 * wave; p0 < p_end; p0 += 64) {
            int32_t g[4], s[4];
            bool v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int64_t p = p0 + 4 * q + e;
                g[e] = p < p_end ? in_idx[p] : -1;
                s[e] = p < p_end ? out_idx[p] : -1;
                v[e] = g[e] >= 0 && g[e] < n_in && s[e] >= 0 && s[e] < n_out;
            }
            shortx4 xa[NA], yb[NB];
#pragma unroll
            for (int a = 0; a < NA; ++a) {
                const int c = ci0 + 16 * a + r16;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    xa[a][e] = (v[e] && a < na && c < ci) ? (short)X[(int64_t)g[e] * ci + c] : (short)0;
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const int c = co0 + 16 * b + r16;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    yb[b][e] = (v[e] && b < nbk && c < co) ? (short)dY[(int64_t)s[e] * co + c] : (short)0;
            }
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    if (a < na && b < nbk)
                        d[a][b] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(xa[a], yb[b], d[a][b], 0, 0, 0);
        }
    }
    // D[m][n]: m = 4q + j (input channel), n = r16 (output channel)
    const int rows = min(kDwTile, ci - ci0), cols = min(kDwTile, co - co0);
    dw_store_partial<R, C>(sh, d, na, nbk, wave, q, r16, rows, cols,
                                       part + (item * ci + ci0) * (int64_t)co + co0, co);
}

// fp32 weight gradient for CI x CO <= 64 x 64 (multiples of 16).  Each wave
// stages 32 pairs at a time in a private LDS buffer: lane l loads half a row
// of X[in_idx] and of dY[out_idx] for pair l % 32 with 16-byte loads (all
// addresses valid: pairs past the chunk are clamped and their dY half-rows
// zeroed by a select), then eight 16x16x4 MFMA steps reduce the 32 pairs,
// reading A = X rows and B = dY rows from LDS.
constexpr int kDwStage = 32;

// Row halves of the 32-pair sub-chunk at p0: lane (pr, half) loads half of
// X[in_idx[p0 + pr]] and of dY[out_idx[p0 + pr]].  Every address is valid
// (pairs past the chunk are clamped) and their dY half-rows are zeroed.
template <int CI, int CO>
struct DwRows {
    float4 x[CI / 8];
    float4 y[CO / 8];
};

template <int CI, int CO>
__device__ __forceinline__ DwRows<CI, CO> dw_fetch(const float* __restrict__ X, const float* __restrict__ dY,
                                                   const int32_t* __restrict__ in_idx,
                                                   const int32_t* __restrict__ out_idx, int64_t n_in, int64_t n_out,
                                                   int64_t p0, int64_t p_end, int pr, int half) {
    DwRows<CI, CO> r;
    const int64_t p = min(p0 + pr, p_end - 1);
    int32_t g = in_idx[p], sidx = out_idx[p];
    const bool v = p0 + pr < p_end && g >= 0 && g < n_in && sidx >= 0 && sidx < n_out;
    g = v ? g : 0;
    sidx = v ? sidx : 0;
    const float4* xr = reinterpret_cast<const float4*>(X + (int64_t)g * CI + half * (CI / 2));
    const float4* yr = reinterpret_cast<const float4*>(dY + (int64_t)sidx * CO + half * (CO / 2));
#pragma unroll
    for (int i = 0; i < CI / 8; ++i) r.x[i] = xr[i];
#pragma unroll
    for (int i = 0; i < CO / 8; ++i) {
        const float4 t = yr[i];
        r.y[i] = v ? t : float4{0.f, 0.f, 0.f, 0.f};
    }
    return r;
}

template <int CI, int CO>
__global__ void __launch_bounds__(kThreads)
k_dw_f32(const float* __restrict__ X, int64_t n_in, const float* __restrict__ dY, int64_t n_out,
         const int32_t* __restrict__ in_idx, const int32_t* __restrict__ out_idx, const int64_t* __restrict__ seg,
         const int64_t* __restrict__ ibase, const int64_t* __restrict__ chunk, int K, float* __restrict__ part) {
    constexpr int NA = CI / 16, NB = CO / 16;
    constexpr int XS = CI + 4, YS = CO + 4;            // row strides (16-byte aligned rows)
    constexpr int STAGE = kDwStage * (XS + YS);
    constexpr int RED = CI * (CO + 1);
    constexpr int SH = (STAGE > RED ? STAGE : RED) * (kThreads / 64);
    __shared__ __attribute__((aligned(16))) float sh[SH];
    int k;
    int64_t p_begin, p_end;
    // the grid covers an upper bound of the items; order the real ones XCD-wise
    if ((int64_t)blockIdx.x >= ibase[K]) return;
    const int64_t item = xcd_unit(blockIdx.x, ibase[K]);
    if (!dw_item(ibase, chunk, seg, K, item, &k, &p_begin, &p_end)) return;
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, q = lane >> 4;
    float* xs = sh + wave * STAGE;
    float* ys = xs + kDwStage * XS;
    floatx4 d[4][4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) d[a][b] = floatx4{0.f, 0.f, 0.f, 0.f};

    const int pr = lane % kDwStage, half = lane / kDwStage;
    constexpr int64_t kStep = kDwStage * (kThreads / 64);
    int64_t p0 = p_begin + kDwStage * wave;
    for (; p0 < p_end; p0 += kStep) {
        const DwRows<CI, CO> rows = dw_fetch<CI, CO>(X, dY, in_idx, out_idx, n_in, n_out, p0, p_end, pr, half);
        float4* xw = reinterpret_cast<float4*>(xs + pr * XS + half * (CI / 2));
        float4* yw = reinterpret_cast<float4*>(ys + pr * YS + half * (CO / 2));
#pragma unroll
        for (int i = 0; i < CI / 8; ++i) xw[i] = rows.x[i];
#pragma unroll
        for (int i = 0; i < CO / 8; ++i) yw[i] = rows.y[i];
        wave_lds_sync();   // lanes read rows other lanes of the wave staged
#pragma unroll
        for (int t = 0; t < kDwStage / 4; ++t) {
            const int row = 4 * t + q;
            float xa[NA], yb[NB];
#pragma unroll
            for (int a = 0; a < NA; ++a) xa[a] = xs[row * XS + 16 * a + r16];
#pragma unroll
            for (int b = 0; b < NB; ++b) yb[b] = ys[row * YS + 16 * b + r16];
#pragma unroll
            for (int a = 0; a < NA; ++a)
#pragma unroll
                for (int b = 0; b < NB; ++b)
                    d[a][b] = __builtin_amdgcn_mfma_f32_16x16x4f32(xa[a], yb[b], d[a][b], 0, 0, 0);
        }
        wave_lds_sync();   // the next stage overwrites rows other lanes just read
    }
    __syncthreads();   // staging buffers are reused for the partial sums
    dw_store_partial<CI, CO>(sh, d, NA, NB, wave, q, r16, CI, CO, part + item * CI * (int64_t)CO, CO);
}

// dW[k] = sum of offset k's partials in a fixed order.  A block covers 64 V
// elements of one offset (V = 4: a 16-byte load per lane, for wide layers
// with ci * co a multiple of 4 and dW 16-byte aligned); wave w adds partials
// w, w + 4, w + 8, ... with eight loads in flight, and the four wave sums are
// combined in wave order.
template <int V>
__global__ void __launch_bounds__(kThreads) k_dw_reduce(const float* __restrict__ part, const int64_t* __restrict__ ibase,
                                                        int ci, int co, float* __restrict__ dW) {
    typedef float vec __attribute__((ext_vector_type(V)));
    __shared__ vec sh[4][64];
    const int k = blockIdx.y;
    const int64_t cc = (int64_t)ci * co;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t e = ((int64_t)blockIdx.x * 64 + lane) * V;
    const int64_t ee = e < cc ? e : 0;
    const int64_t i0 = ibase[k], i1 = ibase[k + 1];
    vec acc8[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) acc8[u] = vec(0.f);
    for (int64_t it = i0 + wave; it < i1; it += 32) {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            const int64_t i = it + 4 * u;
            const vec v = *reinterpret_cast<const vec*>(part + (i < i1 ? i : i0) * cc + ee);
            acc8[u] += i < i1 ? v : vec(0.f);   // a select, not a branch: all eight loads stay in flight
        }
    }
    vec v = vec(0.f);
#pragma unroll
    for (int u = 0; u < 8; ++u) v += acc8[u];
    sh[wave][lane] = v;
    __syncthreads();
    if (wave == 0 && e < cc)
        *reinterpret_cast<vec*>(dW + (int64_t)k * cc + e) = ((sh[0][lane] + sh[1][lane]) + sh[2][lane]) + sh[3][lane];
}

static int dw_tiles(int ci, int co) { return ((ci + kDwTile - 1) / kDwTile) * ((co + kDwTile - 1) / kDwTile); }

// pairs per dW work item: 1024 for one output tile, more for wide layers so
// that the number of partial tiles stays moderate
static int64_t dw_chunk(int ci, int co) {
    const int t = dw_tiles(ci, co);
    return t <= 1 ? 1024 : (t <= 4 ? 2048 : (t <= 16 ? 4096 : 8192));
}

// items below which k_dw_items halves them (where it does)
static int64_t dw_split_items(int ci, int co) { return (kDwSplitItems + dw_tiles(ci, co) - 1) / dw_tiles(ci, co); }

// upper bound of the work items for at most n_pairs pairs (of either dtype: the
// workspace's size; or, with split false, of a kernel whose items are not
// halved: its grid, as workgroups without an item push the others together on
// the same CUs: bf16 96 x 96, 20 items in a grid for 129, 123 -> 156 us)
static int64_t dw_items_bound(int64_t n_pairs, int K, int ci, int co, bool split = true) {
    const int64_t ch = dw_chunk(ci, co), full = (n_pairs + ch - 1) / ch;
    if (!split) return full + K;
    // halved items: fewer than 2 dw_split_items, each but an offset's last full
    return std::max(full, std::min((n_pairs + kDwSplitMin - 1) / kDwSplitMin, 2 * dw_split_items(ci, co))) + K;
}

static size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

static bool dw_f32_specialised(int ci, int co) {
    return (ci == 16 || ci == 32 || ci == 64) && (co == 16 || co == 32 || co == 64);
}

template <int CA, int CB, bool WT, typename Sel>
static void launch_f32_wide(const void* X, int64_t n_x, const void* W, const int32_t* gat, const int32_t* sca,
                            const int64_t* gidx, int K, int64_t G, int64_t n_y, void* Y, Sel sel, const Epilogue& ep,
                            hipStream_t s) {
    const unsigned tiles = (unsigned)((n_y + kWideRows - 1) / kWideRows);
    auto* kern = k_conv_f32_wide<CA, CB, WT, Sel, false>;
    if constexpr (!WT) {   // the forward pass may carry an epilogue
        if (ep.on()) kern = k_conv_f32_wide<CA, CB, WT, Sel, true>;
    }
    hipLaunchKernelGGL(kern, dim3(tiles), dim3(kThreads), 0, s, reinterpret_cast<const float*>(X), n_x,
                       reinterpret_cast<const float*>(W), gat, sca, gidx, K, G, n_y, reinterpret_cast<float*>(Y), sel,
                       ep);
}

template <int CA, int CB, bool WT, typename Sel>
static void launch_f32(const void* X, int64_t n_x, const void* W, const int32_t* gat, const int32_t* sca,
                       const int64_t* gidx, int K, int64_t G, int64_t n_y, void* Y, Sel sel, hipStream_t s) {
    const int64_t blocks = (G + kThreads / 64 - 1) / (kThreads / 64);
    hipLaunchKernelGGL((k_conv_f32<CA, CB, WT, Sel>), dim3((unsigned)blocks), dim3(kThreads), 0, s,
                       reinterpret_cast<const float*>(X), n_x, reinterpret_cast<const float*>(W), gat, sca, gidx,
                       K, G, n_y, reinterpret_cast<float*>(Y), sel);
}

// fp32 shapes with a specialised kernel
template <bool WT, typename Sel>
static bool try_f32(int ca, int cb, const void* X, int64_t n_x, const void* W, const int32_t* gat,
                    const int32_t* sca, const int64_t* gidx, int K, int64_t G, int64_t n_y,
                    void* Y, Sel sel, hipStream_t s) {
#define GSC_F32_CASE(A, B)                                                                     \
    if (ca == A && cb == B) {                                                                  \
        launch_f32<A, B, WT, Sel>(X, n_x, W, gat, sca, gidx, K, G, n_y, Y, sel, s);            \
        return true;                                                                           \
    }
    GSC_F32_CASE(16, 16) GSC_F32_CASE(16, 32) GSC_F32_CASE(32, 16) GSC_F32_CASE(16, 64) GSC_F32_CASE(64, 16)
#undef GSC_F32_CASE
    return false;
}

// *fused (nullable): the kernel that ran has applied the epilogue.
template <typename TIn, typename TOut, bool WT, typename Sel>
static int launch_os(const void* X, int64_t n_x, const void* W, const int32_t* gat, const int32_t* sca,
                     const int64_t* gidx, int K, int ca, int cb, int64_t n_y, void* Y, Sel sel,
                     hipStream_t s, const Epilogue& ep = Epilogue{}, bool* fused = nullptr) {
    if (n_y == 0) return GSC_OK;
    const int64_t tiles = (n_y + kTileRows - 1) / kTileRows;
    const int64_t G = (n_y + GSC_GROUP_ROWS - 1) / GSC_GROUP_ROWS;
    if constexpr (sizeof(TIn) == 4) {
        if (K <= kWaveKMax && (ca == 32 || ca == 64) && (cb == 32 || cb == 64)) {
#define GSC_WIDE_CASE(A, B) \
    if (ca == A && cb == B) launch_f32_wide<A, B, WT, Sel>(X, n_x, W, gat, sca, gidx, K, G, n_y, Y, sel, ep, s);
            GSC_WIDE_CASE(32, 32) GSC_WIDE_CASE(32, 64) GSC_WIDE_CASE(64, 32) GSC_WIDE_CASE(64, 64)
#undef GSC_WIDE_CASE
            if (fused) *fused = true;
            GSC_LAUNCH_CHECK();
            return GSC_OK;
        }
        if (K <= kWaveKMax && try_f32<WT, Sel>(ca, cb, X, n_x, W, gat, sca, gidx, K, G, n_y, Y, sel, s)) {
            GSC_LAUNCH_CHECK();
            return GSC_OK;
        }
    }
    dim3 grid((unsigned)tiles, (unsigned)((cb + kColSlice - 1) / kColSlice));
    hipLaunchKernelGGL((k_conv_os<TIn, TOut, WT, Sel>), grid, dim3(kThreads), 0, s, reinterpret_cast<const TIn*>(X),
                       n_x, reinterpret_cast<const TIn*>(W), gat, sca, gidx, K, G, ca, cb, n_y,
                       reinterpret_cast<TOut*>(Y), sel);
    GSC_LAUNCH_CHECK();
    return GSC_OK;
}

// The epilogue as a pass of its own over complete rows (row-form forward).
template <typename T>
__global__ void k_affine_act(T* __restrict__ y, int64_t n, int c, Epilogue ep) {
    const int64_t total = n * c;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < total; i += (int64_t)gridDim.x * blockDim.x) {
        const int col = (int)(i % c);
        const float sc = ep.scale ? ep.scale[col] : 1.f;
        const float sh = ep.shift ? ep.shift[col] : 0.f;
        store_out(&y[i], epi_apply(to_f32(y[i]), sc, sh, ep.relu));
    }
}

int affine_act(int dtype, void* Y, int64_t n, int c, const Epilogue& ep, hipStream_t s) {
    const int64_t total = n * c;
    if (total == 0) return GSC_OK;
    const unsigned grid = (unsigned)((total + 255) / 256 < 8192 ? (total + 255) / 256 : 8192);
    if (dtype == GSC_BF16)
        hipLaunchKernelGGL(k_affine_act<uint16_t>, dim3(grid), dim3(256), 0, s, reinterpret_cast<uint16_t*>(Y), n, c,
                           ep);
    else
        hipLaunchKernelGGL(k_affine_act<float>, dim3(grid), dim3(256), 0, s, reinterpret_cast<float*>(Y), n, c, ep);
    GSC_LAUNCH_CHECK();
    return GSC_OK;
}

// Backward of the epilogue y = act(z * scale + shift) (Sec. 4.5, the
// non-spatial functions after a convolution; the chain rule per element):
// g = dy where the ReLU passed (y > 0; everywhere without it), dz = g * scale,
// and per channel dscale = sum over rows of g * z, dshift = sum of g, with z
// recovered from y as (y - shift) / scale on the rows where g counts.  The
// division is by one number per channel, so the sums hold g * ((y - shift) p),
// p the power of two of ab_factor, and their total is divided once.  Rows are
// split into kAbChunks chunks at most; a block sums its chunk per channel (lane
// l of a channel takes rows l, l + L, ...; the L lanes are added in lane
// order), the chunk sums go to part, and a second kernel adds them in a fixed
// order (so the sums are deterministic).
//
// Bound: HBM (two reads and a write of n x c).  A thread owns V adjacent
// channels (16 bytes) of a row, kAbRows rows in flight, where rows are whole
// 16-byte groups and all three arrays are 16-byte aligned; otherwise V = 1.
// 480,288 x 128 bf16 (369 MB): one element per thread and a division each took
// 252 us; 239,878 x 64 float32 (184 MB) 76 us.
constexpr int kAbThreads = 256;
constexpr int64_t kAbChunks = 1024;
constexpr int kAbRows = 4;

static int64_t ab_chunks(int64_t n) {
    const int64_t c = (n + 63) / 64;
    return c < 1 ? 1 : (c > kAbChunks ? kAbChunks : c);
}

// The factor p of a channel's (y - shift): the power of two that brings |scale|
// into [1/2, 1) (as near as float32's exponents allow), so (y - shift) p is
// exact and no larger than the quotient, nor less than half of it: what the
// sums hold neither overflows nor underflows where the quotients would not
// (without it a scale of 1e-30 lost gradients below 1e-8).  Scale 0 or NaN: 1
// / scale, and nothing is left to divide by; the sums are then the quotients'.
__device__ __forceinline__ bool ab_no_quotient(float scale) { return scale == 0.f || scale != scale; }
__device__ __forceinline__ float ab_factor(float scale) {
    if (ab_no_quotient(scale)) return 1.f / scale;
    const int e = (int)((__float_as_uint(scale) >> 23) & 255u);
    return __uint_as_float((uint32_t)min(max(253 - e, 1), 254) << 23);
}
__device__ __forceinline__ double ab_divisor(float scale) {
    return ab_no_quotient(scale) ? 1.0 : (double)scale * (double)ab_factor(scale);
}

// V elements of T as one load or store (16 bytes when V > 1)
template <typename T, int V>
struct alignas(sizeof(T) * V) AbVec {
    T v[V];
};

template <typename T, int V>
__global__ void __launch_bounds__(kAbThreads) k_affine_act_bwd(const T* __restrict__ y, const T* __restrict__ dy,
                                                               int64_t n, int c, Epilogue ep, T* __restrict__ dz,
                                                               float* __restrict__ part_s, float* __restrict__ part_t) {
    typedef AbVec<T, V> Vec;
    __shared__ float ss[V][kAbThreads], st[V][kAbThreads];
    const int64_t chunks = gridDim.x;
    const int64_t r0 = n * blockIdx.x / chunks, r1 = n * (blockIdx.x + 1) / chunks;
    const int cv = c / V;                                 // channel groups of a row
    const int span = cv < kAbThreads ? cv : kAbThreads;   // groups a block takes at a time
    const int L = kAbThreads / span;                      // lanes per group
    const int t = threadIdx.x;
    const int lane = t / span, gi = t % span;
    for (int gb = 0; gb < cv; gb += span) {
        const int grp = gb + gi;
        float gs[V], gt[V], sc[V], sh[V], pre[V];
#pragma unroll
        for (int e = 0; e < V; ++e) gs[e] = gt[e] = 0.f;
        if (lane < L && grp < cv) {
#pragma unroll
            for (int e = 0; e < V; ++e) {
                sc[e] = ep.scale ? ep.scale[grp * V + e] : 1.f;
                sh[e] = ep.shift ? ep.shift[grp * V + e] : 0.f;
                pre[e] = ab_factor(sc[e]);
            }
            for (int64_t rb = r0 + lane; rb < r1; rb += kAbRows * L) {
                Vec yv[kAbRows], gv[kAbRows];
#pragma unroll
                for (int i = 0; i < kAbRows; ++i) {   // rows past the chunk re-read its last one of this lane
                    const int64_t r = rb + i * L < r1 ? rb + i * L : rb;
                    yv[i] = reinterpret_cast<const Vec*>(y)[r * cv + grp];
                    gv[i] = reinterpret_cast<const Vec*>(dy)[r * cv + grp];
                }
#pragma unroll
                for (int i = 0; i < kAbRows; ++i) {
                    if (rb + i * L >= r1) break;
                    Vec o;
#pragma unroll
                    for (int e = 0; e < V; ++e) {
                        const float yf = to_f32(yv[i].v[e]);
                        const float g = ep.relu && !(yf > 0.f) ? 0.f : to_f32(gv[i].v[e]);
                        store_out(&o.v[e], g * sc[e]);
                        const float z = (yf - sh[e]) * pre[e];
                        gs[e] = fmaf(g, g != 0.f ? z : 0.f, gs[e]);
                        gt[e] += g;
                    }
                    reinterpret_cast<Vec*>(dz)[(rb + i * L) * cv + grp] = o;
                }
            }
        }
        if (part_s) {
            __syncthreads();   // the previous channel groups' sums are read
#pragma unroll
            for (int e = 0; e < V; ++e) {
                ss[e][t] = gs[e];
                st[e][t] = gt[e];
            }
            __syncthreads();
            for (int i = t; i < span * V; i += kAbThreads) {
                const int e = i % V, g2 = i / V;
                if (gb + g2 >= cv) continue;
                float a = 0.f, b = 0.f;
                for (int l = 0; l < L; ++l) {
                    a += ss[e][l * span + g2];
                    b += st[e][l * span + g2];
                }
                part_s[(int64_t)blockIdx.x * c + (gb + g2) * V + e] = a;
                part_t[(int64_t)blockIdx.x * c + (gb + g2) * V + e] = b;
            }
        }
    }
}

// The channel sums from the chunk sums: a block takes kAbSumCh channels, lane
// l of a channel adds chunks l, l + kAbSumLanes, ... in double, and the lanes'
// sums are added pairwise.  Bound: latency (1 MB of partials); a thread per
// channel adding its 1,024 chunks one after another took 260 us.
constexpr int kAbSumCh = 16, kAbSumLanes = 64;

__global__ void __launch_bounds__(kAbSumCh * kAbSumLanes)
k_affine_act_bwd_sum(const float* __restrict__ part_s, const float* __restrict__ part_t, int64_t chunks, int c,
                     const float* __restrict__ scale, float* __restrict__ dscale, float* __restrict__ dshift) {
    __shared__ double sa[kAbSumLanes][kAbSumCh], sb[kAbSumLanes][kAbSumCh];
    const int ci = threadIdx.x % kAbSumCh, l = threadIdx.x / kAbSumCh;
    const int ch = blockIdx.x * kAbSumCh + ci;
    double a = 0.0, b = 0.0;
    if (ch < c) {
#pragma unroll 4
        for (int64_t k = l; k < chunks; k += kAbSumLanes) {
            a += part_s[k * c + ch];
            b += part_t[k * c + ch];
        }
    }
    sa[l][ci] = a;
    sb[l][ci] = b;
    for (int d = kAbSumLanes / 2; d > 0; d >>= 1) {
        __syncthreads();
        if (l < d) {
            sa[l][ci] += sa[l + d][ci];
            sb[l][ci] += sb[l + d][ci];
        }
    }
    if (l == 0 && ch < c) {
        if (dscale) dscale[ch] = (float)(sa[0][ci] / ab_divisor(scale ? scale[ch] : 1.f));
        if (dshift) dshift[ch] = (float)sb[0][ci];
    }
}

template <typename T>
static void launch_affine_act_bwd(const void* Y, const void* dY, int64_t n, int c, const Epilogue& ep, void* dZ,
                                  float* part_s, float* part_t, hipStream_t s) {
    constexpr int V = 16 / sizeof(T);
    const bool wide = c % V == 0 && (((uintptr_t)Y | (uintptr_t)dY | (uintptr_t)dZ) & 15) == 0;
    auto* kern = wide ? k_affine_act_bwd<T, V> : k_affine_act_bwd<T, 1>;
    hipLaunchKernelGGL(kern, dim3((unsigned)ab_chunks(n)), dim3(kAbThreads), 0, s, reinterpret_cast<const T*>(Y),
                       reinterpret_cast<const T*>(dY), n, c, ep, reinterpret_cast<T*>(dZ), part_s, part_t);
}

}  // namespace gsc

using namespace gsc;

extern "C" {

static bool fwd_uses_bf16_engine(int32_t dtype, int32_t c_in, int32_t c_out, int32_t K) {
    return dtype == GSC_BF16 && conv_bf16_supported(c_in, c_out, K);
}

// Workspace of the forward pass: the bf16 engines' transposed weights, then
// (tile engine) the tile counter.
static size_t fwd_counter_offset(int32_t c_in, int32_t c_out, int32_t K) {
    return (transpose_ws_bytes(K, c_in, c_out) + 255) & ~(size_t)255;
}

size_t gsc_conv_fwd_ws_bytes(int32_t dtype, int32_t c_in, int32_t c_out, int32_t K) {
    if (c_in < 1 || c_out < 1 || K < 1) return 0;
    return fwd_uses_bf16_engine(dtype, c_in, c_out, K) ? fwd_counter_offset(c_in, c_out, K) + 256 : 0;
}

// The plan (perm, bmask, ibase, items) is all given or all null (checked
// when there are output rows; with none the plan is not read).
static int plan_args(const char* who, int64_t n, const int32_t* perm, const uint32_t* bmask, const int64_t* ibase,
                     const int32_t* items, bool* given) {
    *given = false;
    if (n == 0) return GSC_OK;
    const int nn = (perm != nullptr) + (bmask != nullptr) + (ibase != nullptr) + (items != nullptr);
    if (nn != 0 && nn != 4) return fail(GSC_EINVAL, "%s: the block plan needs perm, bmask, ibase and items", who);
    *given = nn == 4;
    return GSC_OK;
}

static bool aligned16(const void* p) { return ((uintptr_t)p & 15) == 0; }

// The fp32 engine over a plan of one or more ranges of offsets (see
// gsc_conv_plan): one launch per range, each adding its sums to the rows
// written by the ranges before it; the epilogue goes with the last.
static int blk_f32_ranges(int ca, int cb, const float* X, int64_t n_x, const float* W, bool wt, const WSel& sel,
                          int K, const BlockPlan& plan, int64_t n_y, float* Y, hipStream_t s, const Epilogue& ep) {
    const int R = plan_ranges(K), S = plan_range_size(K);
    if (R == 1) return conv_blk_f32(ca, cb, X, n_x, W, wt, sel, K, plan, n_y, Y, s, ep);
    const int64_t nb = gsc_plan_blocks(n_y);
    for (int r = 0; r < R; ++r) {
        const int k0 = r * S, kr = K - k0 < S ? K - k0 : S;
        const BlockPlan pr{plan.perm + (int64_t)r * n_y, plan.bmask + (int64_t)r * nb,
                           plan.ibase + (int64_t)r * (nb + 1), plan.items + (int64_t)k0 * nb * 16};
        WSel sr{};
        for (int k = 0; k < kr && wt; ++k) sr.w[k] = sel.w[k0 + k];
        const float* Wr = wt ? W : W + (int64_t)k0 * ca * cb;   // forward: the range's own matrices
        const int rc = conv_blk_f32(ca, cb, X, n_x, Wr, wt, sr, kr, pr, n_y, Y, s, r == R - 1 ? ep : Epilogue{},
                                    r > 0);
        if (rc) return rc;
    }
    return GSC_OK;
}

int32_t gsc_conv_block_engine(int32_t dtype, int32_t c_red, int32_t c_out, int32_t K) {
    if (dtype == GSC_F32)
        return K >= 1 && K <= kPlanMaxKAll && blk_f32_supported(c_red, c_out, plan_range_size(K)) ? 1 : 0;
    if (dtype == GSC_BF16) return blk_bf16_supported(c_red, c_out, K) ? 1 : 0;
    return 0;
}

static int conv_fwd(int32_t dtype, const void* X, int64_t n_in, int32_t c_in, const void* W, int32_t c_out,
                    int32_t K, const int32_t* in_idx, const int32_t* out_idx, const int64_t* gidx, int64_t n_pairs,
                    const int32_t* perm, const uint32_t* bmask, const int64_t* ibase, const int32_t* items,
                    const Epilogue& ep, void* Y, int64_t n_out, void* ws, size_t ws_bytes, hipStream_t s) {
    if (dtype != GSC_F32 && dtype != GSC_BF16) return fail(GSC_EINVAL, "conv_fwd: unknown dtype %d", dtype);
    if (n_in < 0 || n_out < 0 || n_in > INT32_MAX || n_out > INT32_MAX)
        return fail(GSC_EINVAL, "conv_fwd: bad row counts n_in=%lld n_out=%lld", (long long)n_in, (long long)n_out);
    if (c_in < 1 || c_out < 1) return fail(GSC_EINVAL, "conv_fwd: channels must be >= 1");
    if (K < 1 || K > kMaxKConv) return fail(GSC_EINVAL, "conv_fwd: K=%d outside [1,%d]", K, kMaxKConv);
    if (n_pairs < 0) return fail(GSC_EINVAL, "conv_fwd: n_pairs < 0");
    if (n_out > 0 && (!Y || !gidx || !W)) return fail(GSC_EINVAL, "conv_fwd: null Y/gidx/W");
    if (n_pairs > 0 && (!X || !in_idx || !out_idx)) return fail(GSC_EINVAL, "conv_fwd: null X/in_idx/out_idx");
    const size_t need = gsc_conv_fwd_ws_bytes(dtype, c_in, c_out, K);
    if (need > 0 && (!ws || ws_bytes < need))
        return fail(GSC_ESHORT, "conv_fwd: ws needs %zu bytes, got %zu", need, ws ? ws_bytes : (size_t)0);
    bool planned = false;
    int rc = plan_args("conv_fwd", n_out, perm, bmask, ibase, items, &planned);
    if (rc) return rc;
    if (planned && gsc_conv_block_engine(dtype, c_in, c_out, K) && aligned16(X) && aligned16(W) &&
        (dtype != GSC_BF16 || blk_bf16_fits(n_in, c_in))) {
        if (n_in > 0 && !X) return fail(GSC_EINVAL, "conv_fwd: X is null");
        const BlockPlan plan{perm, bmask, ibase, items};
        if (dtype == GSC_BF16) {   // B_k = W[k]: the engine reads its columns, so the transposed copy
            const bool tile = n_in > 0 && tile_bf16_supported(c_in, c_out, K);
            unsigned* counter = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(ws) +
                                                            fwd_counter_offset(c_in, c_out, K));
            rc = transpose_w_bf16(W, K, c_in, c_out, ws, s, tile ? counter : nullptr);   // also zeroes the counter
            if (rc) return rc;
            if (tile)
                return conv_tile_bf16<WIdentity>(c_in, c_out, X, n_in, ws, WIdentity{}, K, plan,
                                                 (n_out + kPlanBlockRows - 1) / kPlanBlockRows, n_out, Y, counter, s,
                                                 ep, /*counter_ready=*/true);
            return conv_blk_bf16<WIdentity>(c_in, c_out, X, n_in, ws, WIdentity{}, K, plan, n_out, Y, s, ep);
        }
        static const WSel kNoSel{};
        return blk_f32_ranges(c_in, c_out, reinterpret_cast<const float*>(X), n_in, reinterpret_cast<const float*>(W),
                              false, kNoSel, K, plan, n_out, reinterpret_cast<float*>(Y), s, ep);
    }
    // row form: except where a kernel writes complete sums once, the epilogue
    // is a pass of its own over Y
    bool fused = false;
    if (dtype == GSC_F32) {
        rc = launch_os<float, float, false>(X, n_in, W, in_idx, out_idx, gidx, K, c_in, c_out, n_out, Y,
                                            WIdentity{}, s, ep, &fused);
    } else if (fwd_uses_bf16_engine(dtype, c_in, c_out, K)) {
        if (n_out == 0) return GSC_OK;
        rc = transpose_w_bf16(W, K, c_in, c_out, ws, s);
        if (rc) return rc;
        rc = conv_bf16<WIdentity>(c_in, c_out, X, n_in, ws, in_idx, out_idx, gidx, nullptr, K, n_out, Y, WIdentity{},
                                  s);
    } else {
        rc = launch_os<uint16_t, uint16_t, false>(X, n_in, W, in_idx, out_idx, gidx, K, c_in, c_out, n_out,
                                                  Y, WIdentity{}, s);
    }
    if (rc || !ep.on() || fused) return rc;
    return affine_act(dtype, Y, n_out, c_out, ep, s);
}

int gsc_sparse_conv_fwd(int32_t dtype, const void* X, int64_t n_in, int32_t c_in, const void* W, int32_t c_out,
                        int32_t K, const int32_t* in_idx, const int32_t* out_idx, const int64_t* seg,
                        const int64_t* gidx, int64_t n_pairs, const int32_t* perm, const uint32_t* bmask,
                        const int64_t* ibase, const int32_t* items, void* Y, int64_t n_out, void* ws,
                        size_t ws_bytes, void* stream) {
    (void)seg;
    clear_error();
    return conv_fwd(dtype, X, n_in, c_in, W, c_out, K, in_idx, out_idx, gidx, n_pairs, perm, bmask, ibase, items,
                    Epilogue{}, Y, n_out, ws, ws_bytes, reinterpret_cast<hipStream_t>(stream));
}

int gsc_sparse_conv_fwd_affine(int32_t dtype, const void* X, int64_t n_in, int32_t c_in, const void* W,
                               int32_t c_out, int32_t K, const int32_t* in_idx, const int32_t* out_idx,
                               const int64_t* seg, const int64_t* gidx, int64_t n_pairs, const int32_t* perm,
                               const uint32_t* bmask, const int64_t* ibase, const int32_t* items, const float* scale,
                               const float* shift, int32_t act, void* Y, int64_t n_out, void* ws, size_t ws_bytes,
                               void* stream) {
    (void)seg;
    clear_error();
    if (act != GSC_ACT_NONE && act != GSC_ACT_RELU) return fail(GSC_EINVAL, "conv_fwd_affine: unknown act %d", act);
    Epilogue ep;
    ep.scale = scale;
    ep.shift = shift;
    ep.relu = act == GSC_ACT_RELU;
    return conv_fwd(dtype, X, n_in, c_in, W, c_out, K, in_idx, out_idx, gidx, n_pairs, perm, bmask, ibase, items, ep,
                    Y, n_out, ws, ws_bytes, reinterpret_cast<hipStream_t>(stream));
}

// Workspace of the backward pass: the weight gradient's chunk tables and
// partial sums, then the tile counter of the input gradient's tile engine.
static size_t bwd_counter_offset(int64_t n_pairs, int32_t c_in, int32_t c_out, int32_t K) {
    const int64_t items = dw_items_bound(n_pairs, K, c_in, c_out);
    return 2 * al256((size_t)(K + 1) * sizeof(int64_t)) + al256((size_t)items * sizeof(int32_t)) +
           al256((size_t)items * c_in * c_out * sizeof(float));
}

size_t gsc_conv_bwd_ws_bytes(int64_t n_pairs, int32_t c_in, int32_t c_out, int32_t K) {
    if (n_pairs < 0 || c_in < 1 || c_out < 1 || K < 1) return 0;
    return bwd_counter_offset(n_pairs, c_in, c_out, K) + 256;
}

int gsc_sparse_conv_bwd(int32_t dtype, const void* X, const void* W, const void* dY, int64_t n_in, int32_t c_in,
                        int32_t c_out, int32_t K, const int32_t* in_idx, const int32_t* out_idx, const int64_t* seg,
                        int64_t n_pairs, const int32_t* t_in_idx, const int32_t* t_out_idx, const int64_t* t_seg,
                        const int64_t* t_gidx, int64_t t_n_pairs, const int32_t* t_wsel, const int32_t* t_perm,
                        const uint32_t* t_bmask, const int64_t* t_ibase, const int32_t* t_items, void* dX, float* dW,
                        int64_t n_out, void* ws, size_t ws_bytes, void* stream) {
    (void)t_seg;
    clear_error();
    if (dtype != GSC_F32 && dtype != GSC_BF16) return fail(GSC_EINVAL, "conv_bwd: unknown dtype %d", dtype);
    if (n_in < 0 || n_out < 0 || n_in > INT32_MAX || n_out > INT32_MAX)
        return fail(GSC_EINVAL, "conv_bwd: bad row counts");
    if (c_in < 1 || c_out < 1) return fail(GSC_EINVAL, "conv_bwd: channels must be >= 1");
    if (K < 1 || K > kMaxKConv) return fail(GSC_EINVAL, "conv_bwd: K=%d outside [1,%d]", K, kMaxKConv);
    if (!W) return fail(GSC_EINVAL, "conv_bwd: W is null");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    if (dW) {
        if (n_pairs < 0) return fail(GSC_EINVAL, "conv_bwd: n_pairs < 0");
        if (!seg || !ws) return fail(GSC_EINVAL, "conv_bwd: null seg/ws");
        if (n_pairs > 0 && (!X || !dY || !in_idx || !out_idx)) return fail(GSC_EINVAL, "conv_bwd: null X/dY/idx");
        const size_t need = gsc_conv_bwd_ws_bytes(n_pairs, c_in, c_out, K);
        if (ws_bytes < need) return fail(GSC_ESHORT, "conv_bwd: ws needs %zu bytes, got %zu", need, ws_bytes);
    }
    // the weight gradient's work items (at the start of ws)
    const int64_t dw_ch = dw_chunk(c_in, c_out);
    int64_t* dw_ibase = ws ? reinterpret_cast<int64_t*>(ws) : nullptr;
    int64_t* dw_chunks =
        ws ? reinterpret_cast<int64_t*>(reinterpret_cast<char*>(ws) + al256((size_t)(K + 1) * sizeof(int64_t)))
           : nullptr;
    const int64_t dw_room = dw_items_bound(n_pairs < 0 ? 0 : n_pairs, K, c_in, c_out);   // what ws holds
    const int64_t dw_split =
        dw_ch <= kDwSplitMax || (dtype == GSC_F32 && !dw_f32_specialised(c_in, c_out)) ? dw_split_items(c_in, c_out) : 0;
    const int64_t dw_items = dw_items_bound(n_pairs < 0 ? 0 : n_pairs, K, c_in, c_out, dw_split > 0);
    int32_t* dw_order =
        ws ? reinterpret_cast<int32_t*>(reinterpret_cast<char*>(ws) + 2 * al256((size_t)(K + 1) * sizeof(int64_t)))
           : nullptr;
    // conv_tile.hip's kernels copy 16 bytes at a time and number the rows' bytes in 32 bits; rows that start anywhere
    // else take the kernels that load them into registers
    const bool dw_tile = dtype == GSC_BF16 && dw_tile_bf16_supported(c_in, c_out, dw_ch) && aligned16(X) &&
                         aligned16(dY) && blk_bf16_fits(n_in, c_in) && blk_bf16_fits(n_out, c_out);
    const bool ordered = dw_tile && c_in <= 128;
    if (!ordered) dw_order = nullptr;
    const dim3 dw_items_grid(ordered ? (unsigned)((dw_items + kDwItemThreads - 1) / kDwItemThreads) : 1u);
    bool dw_items_done = false;
    if (dX) {
        if (t_n_pairs < 0) return fail(GSC_EINVAL, "conv_bwd: t_n_pairs < 0");
        if (n_in > 0 && (!t_gidx || !t_wsel)) return fail(GSC_EINVAL, "conv_bwd: null t_gidx/t_wsel");
        if (t_n_pairs > 0 && (!dY || !t_in_idx || !t_out_idx))
            return fail(GSC_EINVAL, "conv_bwd: null dY/t_in_idx/t_out_idx");
        // the role-reversed map's offsets pair one to one with the forward map's
        WSel sel;
        std::vector<uint8_t> seen((size_t)K, 0);
        for (int k = 0; k < K; ++k) {
            if (t_wsel[k] < 0 || t_wsel[k] >= K)
                return fail(GSC_EINVAL, "conv_bwd: t_wsel[%d]=%d outside [0,%d)", k, t_wsel[k], K);
            if (seen[t_wsel[k]]++)
                return fail(GSC_EINVAL, "conv_bwd: t_wsel is not a permutation (%d appears twice)", t_wsel[k]);
            sel.w[k] = (int16_t)t_wsel[k];
        }
        bool planned = false;
        int rc = plan_args("conv_bwd", n_in, t_perm, t_bmask, t_ibase, t_items, &planned);
        if (rc) return rc;
        if (planned && gsc_conv_block_engine(dtype, c_out, c_in, K) && aligned16(dY) && aligned16(W) &&
            (dtype != GSC_BF16 || blk_bf16_fits(n_out, c_out))) {
            const BlockPlan plan{t_perm, t_bmask, t_ibase, t_items};
            if (dtype == GSC_BF16 && n_out > 0 && tile_bf16_supported(c_out, c_in, K)) {
                // B_k[ch][col] = W[sel(k)][col][ch]: W is already the engine's layout.  The tile
                // counter sits after the weight gradient's part of ws, when ws is given in full.
                unsigned* counter = nullptr;
                if (ws && n_pairs >= 0 && ws_bytes >= gsc_conv_bwd_ws_bytes(n_pairs, c_in, c_out, K))
                    counter = reinterpret_cast<unsigned*>(reinterpret_cast<char*>(ws) +
                                                          bwd_counter_offset(n_pairs, c_in, c_out, K));
                if (counter && dW) {   // one small launch: the weight gradient's items and the tile counter
                    hipLaunchKernelGGL(k_dw_items, dw_items_grid, dim3(kDwItemThreads), 0, s, seg, K, dw_ch, dw_split,
                                       dw_ibase, dw_chunks, dw_order, dw_items, counter);
                    GSC_LAUNCH_CHECK();
                    dw_items_done = true;
                }
                rc = conv_tile_bf16<WSel>(c_out, c_in, dY, n_out, W, sel, K, plan,
                                          (n_in + kPlanBlockRows - 1) / kPlanBlockRows, n_in, dX, counter, s,
                                          Epilogue{}, /*counter_ready=*/dw_items_done);
            } else if (dtype == GSC_BF16)   // B_k[ch][col] = W[sel(k)][col][ch]: W is already the engine's layout
                rc = conv_blk_bf16<WSel>(c_out, c_in, dY, n_out, W, sel, K, plan, n_in, dX, s);
            else
                rc = blk_f32_ranges(c_out, c_in, reinterpret_cast<const float*>(dY), n_out,
                                    reinterpret_cast<const float*>(W), true, sel, K, plan, n_in,
                                    reinterpret_cast<float*>(dX), s, Epilogue{});
        }
        else if (dtype == GSC_F32)
            rc = launch_os<float, float, true>(dY, n_out, W, t_in_idx, t_out_idx, t_gidx, K, c_out, c_in,
                                               n_in, dX, sel, s);
        else if (conv_bf16_supported(c_out, c_in, K))   // W[w] (c_in x c_out) is already the B layout of dY W^T
            rc = conv_bf16<WSel>(c_out, c_in, dY, n_out, W, t_in_idx, t_out_idx, t_gidx, nullptr, K, n_in, dX, sel,
                                 s);
        else
            rc = launch_os<uint16_t, uint16_t, true>(dY, n_out, W, t_in_idx, t_out_idx, t_gidx, K, c_out,
                                                     c_in, n_in, dX, sel, s);
        if (rc) return rc;
    }
    if (dW) {
        const int64_t items = dw_items;
        char* w = reinterpret_cast<char*>(ws);
        int64_t* ibase = dw_ibase;
        int64_t* chunk = dw_chunks;
        float* part = reinterpret_cast<float*>(w + 2 * al256((size_t)(K + 1) * sizeof(int64_t)) +
                                               al256((size_t)dw_room * sizeof(int32_t)));
        if (!dw_items_done) {
            hipLaunchKernelGGL(k_dw_items, dw_items_grid, dim3(kDwItemThreads), 0, s, seg, K, dw_ch, dw_split, ibase, chunk,
                               dw_order, dw_items, (unsigned*)nullptr);
            GSC_LAUNCH_CHECK();
        }
        if (dtype == GSC_F32 && dw_f32_specialised(c_in, c_out)) {
            auto X32 = reinterpret_cast<const float*>(X);
            auto dY32 = reinterpret_cast<const float*>(dY);
#define GSC_DW_CASE(A, B)                                                                              \
    if (c_in == A && c_out == B)                                                                       \
        hipLaunchKernelGGL((k_dw_f32<A, B>), dim3((unsigned)items), dim3(kThreads), 0, s, X32, n_in, dY32, \
                           n_out, in_idx, out_idx, seg, ibase, chunk, K, part);
            GSC_DW_CASE(16, 16) GSC_DW_CASE(16, 32) GSC_DW_CASE(16, 64) GSC_DW_CASE(32, 16) GSC_DW_CASE(32, 32)
            GSC_DW_CASE(32, 64) GSC_DW_CASE(64, 16) GSC_DW_CASE(64, 32) GSC_DW_CASE(64, 64)
#undef GSC_DW_CASE
        } else if (dw_tile) {
            int rc = dw_tile_bf16(c_in, c_out, X, n_in, dY, n_out, in_idx, out_idx, seg, ibase, chunk, dw_order, K,
                                  items, part, s);
            if (rc) return rc;
        } else if (dtype == GSC_BF16 && dw_bf16_supported(c_in, c_out)) {
            int rc = dw_bf16(c_in, c_out, X, n_in, dY, n_out, in_idx, out_idx, seg, ibase, chunk, K, items, part, s);
            if (rc) return rc;
        } else {
            const unsigned tiles = (unsigned)dw_tiles(c_in, c_out);
#define GSC_DWP_CASE(T, NA, NB)                                                                               \
    hipLaunchKernelGGL((k_dw_partial<T, NA, NB>), dim3((unsigned)items, tiles), dim3(kThreads), 0, s,          \
                       reinterpret_cast<const T*>(X), n_in, reinterpret_cast<const T*>(dY), n_out, in_idx, out_idx, \
                       seg, ibase, chunk, K, c_in, c_out, part)
#define GSC_DWP_WIDTHS(T)                             \
    if (c_in <= 16 && c_out <= 16) GSC_DWP_CASE(T, 1, 1); \
    else if (c_in <= 16) GSC_DWP_CASE(T, 1, 4);       \
    else if (c_out <= 16) GSC_DWP_CASE(T, 4, 1);      \
    else GSC_DWP_CASE(T, 4, 4)
            if (dtype == GSC_F32) {
                GSC_DWP_WIDTHS(float);
            } else {
                GSC_DWP_WIDTHS(uint16_t);
            }
#undef GSC_DWP_WIDTHS
#undef GSC_DWP_CASE
        }
        GSC_LAUNCH_CHECK();
        const int64_t cc = (int64_t)c_in * c_out;
        // 16-byte lanes where that still leaves thousands of blocks (wide layers)
        if (cc % 4 == 0 && cc >= 16384 && reinterpret_cast<uintptr_t>(dW) % 16 == 0)
            hipLaunchKernelGGL(k_dw_reduce<4>, dim3((unsigned)((cc + 255) / 256), (unsigned)K), dim3(kThreads), 0, s,
                               part, ibase, c_in, c_out, dW);
        else
            hipLaunchKernelGGL(k_dw_reduce<1>, dim3((unsigned)((cc + 63) / 64), (unsigned)K), dim3(kThreads), 0, s,
                               part, ibase, c_in, c_out, dW);
        GSC_LAUNCH_CHECK();
    }
    return GSC_OK;
}

// Workspace of gsc_sparse_conv_bwd_fwdmap: the weight gradient's part (as
// gsc_sparse_conv_bwd's, with its tile counter), the dX map (dense form,
// pairs, segments, group index) and the transposition's scratch, then, when a
// block engine takes the input gradient, the dX map's plan and its scratch.
struct FwdmapWs {
    size_t dw, dense, t_in, t_out, t_seg, t_gidx, tr, perm, bmask, ibase, items, plan, total;
};

static FwdmapWs fwdmap_layout(int32_t dtype, int64_t n_in, int64_t cap, int32_t c_in, int32_t c_out, int32_t K) {
    FwdmapWs L{};
    const int64_t G = gsc_kmap_groups(n_in);
    size_t o = 0;
    auto take = [&](size_t b) {
        const size_t at = o;
        o += al256(b);
        return at;
    };
    L.dw = take(gsc_conv_bwd_ws_bytes(cap, c_in, c_out, K));
    L.dense = take((size_t)K * n_in * sizeof(int32_t));
    L.t_in = take((size_t)cap * sizeof(int32_t));
    L.t_out = take((size_t)cap * sizeof(int32_t));
    L.t_seg = take((size_t)(K + 1) * sizeof(int64_t));
    L.t_gidx = take((size_t)(K * G + 1) * sizeof(int64_t));
    L.tr = take(gsc_kernel_map_transpose_ws_bytes(n_in, K));
    if (gsc_conv_block_engine(dtype, c_out, c_in, K)) {
        const int64_t R = gsc_plan_ranges(K), nb = gsc_plan_blocks(n_in);
        L.perm = take((size_t)R * n_in * sizeof(int32_t));
        L.bmask = take((size_t)R * nb * sizeof(uint32_t));
        L.ibase = take((size_t)R * (nb + 1) * sizeof(int64_t));
        L.items = take((size_t)K * nb * 16 * sizeof(int32_t));
        L.plan = take(gsc_conv_plan_ws_bytes(n_in, K));
    } else {
        L.perm = L.bmask = L.ibase = L.items = L.plan = SIZE_MAX;
    }
    L.total = o;
    return L;
}

size_t gsc_conv_bwd_fwdmap_ws_bytes(int32_t dtype, int64_t n_in, int64_t cap_pairs, int32_t c_in, int32_t c_out,
                                    int32_t K) {
    if ((dtype != GSC_F32 && dtype != GSC_BF16) || n_in < 0 || cap_pairs < 0 || c_in < 1 || c_out < 1 || K < 1 ||
        K > kMaxKConv)
        return 0;
    return fwdmap_layout(dtype, n_in, cap_pairs, c_in, c_out, K).total;
}

int gsc_sparse_conv_bwd_fwdmap(int32_t dtype, const void* X, const void* W, const void* dY, int64_t n_in,
                               int32_t c_in, int32_t c_out, int32_t K, const int32_t* in_idx, const int32_t* out_idx,
                               const int64_t* seg, int64_t cap_pairs, int32_t transpose, void* dX, float* dW,
                               int64_t n_out, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (dtype != GSC_F32 && dtype != GSC_BF16) return fail(GSC_EINVAL, "conv_bwd_fwdmap: unknown dtype %d", dtype);
    if (K < 1 || K > kMaxKConv) return fail(GSC_EINVAL, "conv_bwd_fwdmap: K=%d outside [1,%d]", K, kMaxKConv);
    if (n_in < 0 || n_out < 0 || n_in > INT32_MAX || n_out > INT32_MAX || cap_pairs < 0 || c_in < 1 || c_out < 1)
        return fail(GSC_EINVAL, "conv_bwd_fwdmap: bad sizes");
    if (!seg || !ws) return fail(GSC_EINVAL, "conv_bwd_fwdmap: null seg/ws");
    const size_t need = gsc_conv_bwd_fwdmap_ws_bytes(dtype, n_in, cap_pairs, c_in, c_out, K);
    if (ws_bytes < need) return fail(GSC_ESHORT, "conv_bwd_fwdmap: ws needs %zu bytes, got %zu", need, ws_bytes);
    // a: the pairs' rows of X, b: their rows of Y (the transposed convolution ran the map with roles exchanged)
    const int32_t* a = transpose ? out_idx : in_idx;
    const int32_t* b = transpose ? in_idx : out_idx;
    const FwdmapWs L = fwdmap_layout(dtype, n_in, cap_pairs, c_in, c_out, K);
    char* w = reinterpret_cast<char*>(ws);
    int32_t* t_in = reinterpret_cast<int32_t*>(w + L.t_in);
    int32_t* t_out = reinterpret_cast<int32_t*>(w + L.t_out);
    int64_t* t_seg = reinterpret_cast<int64_t*>(w + L.t_seg);
    int64_t* t_gidx = reinterpret_cast<int64_t*>(w + L.t_gidx);
    int32_t* dense = reinterpret_cast<int32_t*>(w + L.dense);
    const bool planned = L.plan != SIZE_MAX;
    int32_t* perm = planned ? reinterpret_cast<int32_t*>(w + L.perm) : nullptr;
    uint32_t* bmask = planned ? reinterpret_cast<uint32_t*>(w + L.bmask) : nullptr;
    int64_t* ibase = planned ? reinterpret_cast<int64_t*>(w + L.ibase) : nullptr;
    int32_t* items = planned ? reinterpret_cast<int32_t*>(w + L.items) : nullptr;
    int rc;
    if (dX) {
        // the dX map: the same pairs listed by their row of X (and its plan)
        rc = gsc_kernel_map_transpose(a, b, seg, K, cap_pairs, n_in, t_in, t_out, t_seg, t_gidx, dense, w + L.tr,
                                      gsc_kernel_map_transpose_ws_bytes(n_in, K), stream);
        if (rc) return rc;
        if (planned) {
            rc = gsc_conv_plan(dense, n_in, K, perm, bmask, ibase, items, (int64_t)K * gsc_plan_blocks(n_in),
                               w + L.plan, gsc_conv_plan_ws_bytes(n_in, K), stream);
            if (rc) return rc;
        }
    }
    std::vector<int32_t> ident((size_t)K);
    for (int k = 0; k < K; ++k) ident[k] = k;   // segment k of the dX map holds offset k's pairs
    return gsc_sparse_conv_bwd(dtype, X, W, dY, n_in, c_in, c_out, K, a, b, seg, cap_pairs, t_in, t_out, t_seg,
                               t_gidx, cap_pairs, ident.data(), perm, bmask, ibase, items, dX, dW, n_out, w + L.dw,
                               gsc_conv_bwd_ws_bytes(cap_pairs, c_in, c_out, K), stream);
}

size_t gsc_affine_act_bwd_ws_bytes(int64_t n, int32_t c) {
    if (n < 0 || c < 1) return 0;
    return 2 * al256((size_t)ab_chunks(n) * c * sizeof(float));
}

int gsc_affine_act_bwd(int32_t dtype, const void* Y, const void* dY, int64_t n, int32_t c, const float* scale,
                       const float* shift, int32_t act, void* dZ, float* dscale, float* dshift, void* ws,
                       size_t ws_bytes, void* stream) {
    clear_error();
    if (dtype != GSC_F32 && dtype != GSC_BF16) return fail(GSC_EINVAL, "affine_act_bwd: unknown dtype %d", dtype);
    if (act != GSC_ACT_NONE && act != GSC_ACT_RELU) return fail(GSC_EINVAL, "affine_act_bwd: unknown act %d", act);
    if (n < 0 || c < 1) return fail(GSC_EINVAL, "affine_act_bwd: bad sizes n=%lld c=%d", (long long)n, c);
    if (n > 0 && (!Y || !dY || !dZ)) return fail(GSC_EINVAL, "affine_act_bwd: null Y/dY/dZ");
    const bool sums = dscale || dshift;
    if (sums) {
        const size_t need = gsc_affine_act_bwd_ws_bytes(n, c);
        if (!ws || ws_bytes < need)
            return fail(GSC_ESHORT, "affine_act_bwd: ws needs %zu bytes, got %zu", need, ws ? ws_bytes : (size_t)0);
    }
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    Epilogue ep;
    ep.scale = scale;
    ep.shift = shift;
    ep.relu = act == GSC_ACT_RELU;
    const int64_t chunks = ab_chunks(n);
    float* part_s = sums ? reinterpret_cast<float*>(ws) : nullptr;
    float* part_t = sums ? reinterpret_cast<float*>(reinterpret_cast<char*>(ws) +
                                                    al256((size_t)chunks * c * sizeof(float)))
                         : nullptr;
    if (dtype == GSC_BF16)
        launch_affine_act_bwd<uint16_t>(Y, dY, n, c, ep, dZ, part_s, part_t, s);
    else
        launch_affine_act_bwd<float>(Y, dY, n, c, ep, dZ, part_s, part_t, s);
    GSC_LAUNCH_CHECK();
    if (sums) {
        hipLaunchKernelGGL(k_affine_act_bwd_sum, dim3((unsigned)((c + kAbSumCh - 1) / kAbSumCh)),
                           dim3(kAbSumCh * kAbSumLanes), 0, s, part_s, part_t, chunks, c, scale, dscale, dshift);
        GSC_LAUNCH_CHECK();
    }
    return GSC_OK;
}

}  // extern "C"
