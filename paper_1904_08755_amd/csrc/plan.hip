// Block plan of a kernel map for the convolution kernels.
//
// The block convolution engines compute 16 output rows at a time (one MFMA
// row block) and keep the block's sums in registers: for every offset that
// any of the 16 rows has, they gather the 16 input rows (a zero row where a
// row has no pair at that offset) and multiply by that offset's weights.  The
// cost of a block is therefore the number of distinct offsets among its rows.
// In the natural row order a block's rows point every way and almost all
// offsets occur; the plan orders the output rows by neighbour mask (bit k set
// when the row has a pair at offset k), so rows with the same neighbourhood
// shape share blocks, and the blocks' offset sets shrink to about those of
// single rows.  The sort key puts the mask's popcount, capped to the bits
// that the last 10-bit digit leaves free, above the mask: rows are grouped
// by neighbour count first, so a run of blocks (the tile engine's tile of
// 16) also has fewer distinct offsets, and the plan's positions come in
// rough order of cost (which the tile engine uses to hand out its largest
// tiles first).
//
// Output, for n_out rows, nb = ceil(n_out / 16) blocks:
//   perm[i]      output row at position i (i < n_out);
//   bmask[b]     union of the masks of block b's rows (positions 16b..16b+15);
//   ibase[b]     first item of block b (exclusive scan of popcount(bmask));
//                ibase[nb] = number of items;
//   items[16*t + r]  for item t = ibase[b] + j, the j-th offset k of bmask[b]
//                in increasing order: the input row paired with position
//                16b + r at offset k, or -1 if there is none.
// Input: the map's dense form nbr[k][j] (input row or -1), which the kernel
// map writes as it probes.  Steps:
//   masks:  every row's mask from its column of nbr, its sort key, and the
//           digit counts of every kMaskRows rows;
//   counts: the digit counts' totals, and their prefixes over the row groups
//           (where the first pass's tiles place their keys);
//   sort:   stable LSD radix sort of (key, row) by key = (min(popcount of
//           the mask, cap) << K) | mask, 10-bit digits, one kernel per digit
//           (cap: plan_key_cap);
//   count:  block unions and item counts, scanned within kBlkTile blocks;
//   fill:   the item bases, and one lane per position writes its entry of each
//           of its block's items.
// Everything is deterministic and runs without a host round trip.
#include <algorithm>
#include <climits>
#include <cstdlib>

#include "gsc_internal.h"

namespace gsc {

constexpr int kPlanThreads = 256;
constexpr int kRsBits = 10;                       // radix digit width
constexpr int kRsBins = 1 << kRsBits;
constexpr int kRsThreads = 1024;                  // radix sort block
// Keys per thread: 2 in the first pass, whose tiles do not wait for each other
// (300,000 keys: 7.4 us against 9.1 with 4), and in later passes 4 from
// kRsWideKeys keys on, where the look-back over half as many tiles outweighs a
// tile's longer work (300,000 keys: 16.7 us against 18.2; 40,000 keys: 11.6
// against 10.4).
constexpr int kRsPer = 2, kRsPerWide = 4;
constexpr int64_t kRsWideKeys = 100000;
constexpr int kRsTile = kRsThreads * kRsPer;      // keys per block of the first pass
constexpr int kRsMaxPasses = 4;                   // keys of up to 40 bits
constexpr int kMaskRows = 1024;                   // rows (and threads) of a block of the mask kernel
static_assert(kRsTile % kMaskRows == 0, "a sort tile is a whole number of counted row groups");

static size_t al256(size_t b) { return (b + 255) & ~(size_t)255; }

// The popcount field of the sort key: as many bits as the last 10-bit digit
// of the K-bit mask leaves free (at most 6, and within a 32-bit key); its
// largest value, 0 when there is no room.  K = 27: 3 bits, counts capped at 7.
__host__ __device__ inline int plan_key_pbits(int K) {
    const int spare = (K + kRsBits - 1) / kRsBits * kRsBits - K;
    const int a = spare < 32 - K ? spare : 32 - K;
    return a < 6 ? a : 6;
}
__host__ __device__ inline uint32_t plan_key_cap(int K) { return (1u << plan_key_pbits(K)) - 1u; }

// Offsets of plan range r of a K-offset map planned in ranges of S offsets
// (the last one may be shorter), and their mask bits.
__host__ __device__ inline int range_k0(int r, int S) { return r * S; }
__host__ __device__ inline int range_len(int r, int S, int K) { return K - r * S < S ? K - r * S : S; }
__host__ __device__ inline uint32_t range_kmask(int kr) { return kr >= 32 ? ~0u : (1u << kr) - 1u; }

// ---------------------------------------------------------------------------
// masks from the dense map
// ---------------------------------------------------------------------------
// Range r = blockIdx.y of the plan: keys[r * n + j] for its offsets, and how
// many of the block's keys have each digit of each pass: cnt[((r * passes + p)
// * nm + block) * kRsBins + digit].  (Also clears the sort's tickets and
// look-back entries, zero[0, nzero).)  Bound: nbr read once; B loads in flight
// per lane.
__global__ void __launch_bounds__(kMaskRows) k_plan_masks(const int32_t* __restrict__ nbr, int64_t n, int Kall, int S,
                                                          int passes, uint32_t* __restrict__ keys,
                                                          uint16_t* __restrict__ cnt, uint32_t* __restrict__ zero,
                                                          int64_t nzero, uint32_t* __restrict__ lb_status) {
    __shared__ uint32_t hist[kRsMaxPasses * kRsBins];
    const int t = threadIdx.x;
    const int64_t lin = (int64_t)blockIdx.y * gridDim.x + blockIdx.x;   // block number over all ranges
    if (lb_status && lin == 0 && t == 0) *lb_status = 0u;               // the plan call's first kernel
    for (int64_t i = lin * kMaskRows + t; i < nzero; i += (int64_t)gridDim.x * gridDim.y * kMaskRows) zero[i] = 0;
    for (int i = t; i < passes * kRsBins; i += kMaskRows) hist[i] = 0;
    const int rg = blockIdx.y;
    const int K = range_len(rg, S, Kall);
    const uint32_t cap = plan_key_cap(K);
    nbr += (int64_t)range_k0(rg, S) * n;
    keys += (int64_t)rg * n;
    const int64_t j = (int64_t)blockIdx.x * kMaskRows + t;
    const bool valid = j < n;
    const int64_t jj = valid ? j : n - 1;
    uint32_t m = 0;
    constexpr int B = 9;   // table entries loaded together (a divisor of 27)
    for (int k0 = 0; k0 < K; k0 += B) {
        int32_t r[B];
#pragma unroll
        for (int b = 0; b < B; ++b) r[b] = nbr[(int64_t)min(k0 + b, K - 1) * n + jj];
#pragma unroll
        for (int b = 0; b < B; ++b) m |= (uint32_t)(k0 + b < K && r[b] >= 0) << ((k0 + b) & 31);
    }
    const uint32_t c = min((uint32_t)__popc(m), cap);
    const uint32_t key = cap ? m | (c << K) : m;   // cap > 0 only where K + its bits <= 32
    if (valid) keys[j] = key;
    __syncthreads();   // hist is clear
    if (valid)
        for (int p = 0; p < passes; ++p) atomicAdd(&hist[p * kRsBins + ((key >> (p * kRsBits)) & (kRsBins - 1))], 1u);
    __syncthreads();
    const int64_t nm = gridDim.x;
    for (int i = t; i < passes * kRsBins; i += kMaskRows)
        cnt[(((int64_t)rg * passes + i / kRsBins) * nm + blockIdx.x) * kRsBins + i % kRsBins] = (uint16_t)hist[i];
}

// ---------------------------------------------------------------------------
// stable LSD radix sort of (key, value) by key, one kernel per pass
// ---------------------------------------------------------------------------
// Block (x, y) = (64 digits, range and pass): the digits' totals over the nm
// row groups into ghist, and for the first pass, whose keys lie in row order,
// the exclusive prefix over the groups before each sort tile into pre[(r * nrs
// + tile) * kRsBins + digit].  16 lanes per digit take a sixteenth of the
// tiles each.
constexpr int kCntLanes = 16;
constexpr int kSub = kRsTile / kMaskRows;   // row groups of a tile

__global__ void __launch_bounds__(64 * kCntLanes) k_rs_counts(const uint16_t* __restrict__ cnt, int64_t nm, int64_t nrs,
                                                              int passes, uint32_t* __restrict__ ghist,
                                                              uint32_t* __restrict__ pre) {
    __shared__ uint32_t part[kCntLanes][64];
    const int d = blockIdx.x * 64 + (threadIdx.x & 63), lane = threadIdx.x >> 6;
    const int rg = blockIdx.y / passes, p = blockIdx.y % passes;
    cnt += (int64_t)blockIdx.y * nm * kRsBins;
    const int64_t t0 = nrs * lane / kCntLanes, t1 = nrs * (lane + 1) / kCntLanes;
    uint32_t sum = 0;
    for (int64_t g = t0 * kSub; g < t1 * kSub; g += 8) {
        uint32_t v[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] = g + i < t1 * kSub && g + i < nm ? cnt[(g + i) * kRsBins + d] : 0u;
#pragma unroll
        for (int i = 0; i < 8; ++i) sum += v[i];
    }
    part[lane][threadIdx.x & 63] = sum;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int i = 0; i < kCntLanes; ++i) {
        const uint32_t v = part[i][threadIdx.x & 63];
        if (i < lane) before += v;
        all += v;
    }
    if (lane == 0) ghist[((int64_t)rg * kRsMaxPasses + p) * kRsBins + d] = all;
    if (p != 0) return;
    for (int64_t t = t0; t < t1; ++t) {
        pre[((int64_t)rg * nrs + t) * kRsBins + d] = before;
#pragma unroll
        for (int i = 0; i < kSub; ++i) before += t * kSub + i < nm ? cnt[(t * kSub + i) * kRsBins + d] : 0u;
    }
}

// A pass takes the keys in tiles of PER per thread.  A wave ranks its own contiguous
// keys of the tile with a counter per digit of its own (lanes with equal
// digits found with kRsBits ballots, rounds of 64 keys in index order), so
// ranking needs no barrier; then the waves' counts are scanned per digit, and
// a key's place is its digit's start in the pass's output + the keys of that
// digit in earlier tiles + in earlier waves + its rank.
//
// The keys of earlier tiles: known beforehand in the first pass (FIRST:
// k_rs_counts).  Later passes take tiles in ticket order (an atomic counter, so
// every tile a block waits for is already running), publish the tile's count
// of each digit and look back over the earlier tiles' published counts (the
// decoupled look-back of Merrill and Garland's single-pass prefix scan: a
// tile's entry holds either its own count or, once known, its inclusive
// prefix).
//
// Bound: latency.  With ranks from block-wide rounds (five barriers and up to
// 15 counters read per key and round) and the look-back in every pass, 300,000
// keys took 20.7 us a pass and 40,000 keys 13.3 us.
constexpr uint32_t kStAgg = 1u << 30;             // entry holds the tile's own count
constexpr uint32_t kStIncl = 1u << 31;            // entry holds the inclusive prefix
constexpr uint32_t kStCount = kStAgg - 1;
constexpr int64_t kRsMaxKeys = kStCount;          // counts must fit below the flag bits
constexpr int kSpinMax = 1 << 22;                 // bound on polls of one entry (not reached in practice)

// Tiles of all ranges share the ticket: ticket T is tile T % nrs of range
// T / nrs, which looks back over its own range's tiles only (all of them
// took smaller tickets).  Range r's keys and values are at r * n, its look-
// back entries (or prefixes) at r * nrs * kRsBins, its digit counts at r *
// kRsMaxPasses * kRsBins (ghist points at the pass's row of range 0).
template <bool FIRST, int PER>
__global__ void __launch_bounds__(kRsThreads) k_rs_pass(const uint32_t* __restrict__ kin,
                                                        const int32_t* __restrict__ vin, int64_t n, int64_t nrs,
                                                        int shift, const uint32_t* __restrict__ ghist,
                                                        uint32_t* __restrict__ status, uint32_t* __restrict__ ticket,
                                                        uint32_t* __restrict__ kout, int32_t* __restrict__ vout,
                                                        int spin_max, uint32_t* __restrict__ lb_status) {
    constexpr int W = kRsThreads / 64;
    static_assert(kRsThreads == kRsBins, "one thread per digit");
    __shared__ uint32_t start[kRsBins];
    __shared__ uint16_t wcnt[W][kRsBins];
    __shared__ uint32_t tile_sh;
    __shared__ uint32_t wsum[W];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    if (!FIRST && tid == 0) tile_sh = atomicAdd(ticket, 1u);
    for (int i = tid; i < W * kRsBins / 2; i += kRsThreads) reinterpret_cast<uint32_t*>(&wcnt[0][0])[i] = 0;
    __syncthreads();
    const int64_t T = FIRST ? (int64_t)blockIdx.x : (int64_t)tile_sh;
    const int64_t rg = T / nrs, t = T - rg * nrs;
    kin += rg * n;
    vout += rg * n;
    kout += rg * n;
    if (!FIRST) vin += rg * n;
    status += rg * nrs * kRsBins;
    const uint32_t dc = ghist[rg * kRsMaxPasses * kRsBins + tid];
    const int64_t base = t * (kRsThreads * PER) + wave * (64 * PER) + lane;
    uint32_t key[PER];
    int32_t val[PER];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const int64_t idx = base + r * 64;
        const int64_t ii = idx < n ? idx : 0;
        key[r] = kin[ii];
        val[r] = FIRST ? (int32_t)idx : vin[ii];
    }
    const uint32_t prefix = FIRST ? status[t * kRsBins + tid] : 0u;
    // ranks within the wave
    const unsigned long long below = lanemask_lt();
    uint32_t rank[PER];
    uint16_t* mine = wcnt[wave];
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        const bool valid = base + r * 64 < n;
        const int d = (int)((key[r] >> shift) & (kRsBins - 1));
        unsigned long long peers = __ballot(valid);
#pragma unroll
        for (int b = 0; b < kRsBits; ++b) {
            const bool bit = (d >> b) & 1;
            const unsigned long long m = __ballot(bit);
            peers &= bit ? m : ~m;
        }
        const uint32_t seen = mine[d];
        wave_lds_sync();   // every lane has read its digit's counter
        rank[r] = seen + (uint32_t)__popcll(peers & below);
        if (valid && (peers & below) == 0) mine[d] = (uint16_t)(seen + __popcll(peers));
        wave_lds_sync();
    }
    // where digit tid's keys start in this pass's output (the keys of smaller digits)
    uint32_t dinc = dc;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const uint32_t u = __shfl_up(dinc, o, 64);
        if (lane >= o) dinc += u;
    }
    if (lane == 63) wsum[wave] = dinc;
    __syncthreads();   // the waves' counts are complete
    uint32_t dbase = dinc - dc;
    for (int i = 0; i < wave; ++i) dbase += wsum[i];
    uint32_t c = 0;   // digit tid: the waves' counts become exclusive prefixes, the tile's count their sum
#pragma unroll
    for (int w = 0; w < W; ++w) {
        const uint32_t v = wcnt[w][tid];
        wcnt[w][tid] = (uint16_t)c;
        c += v;
    }
    uint32_t before = prefix;
    if (!FIRST) {   // publish the tile's count of digit tid, then look back for the keys before the tile
        // (the entries are the only data exchanged, so relaxed atomics at
        // agent scope suffice: they go to L2 and every poll sees the latest)
        uint32_t* entry = status + t * kRsBins + tid;
        __hip_atomic_store(entry, (t == 0 ? kStIncl : kStAgg) | c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (t > 0) {
            constexpr int LW = 4;   // predecessors' entries loaded together
            bool done = false;
            for (int64_t j0 = t - 1; !done && j0 >= 0; j0 -= LW) {
                uint32_t v[LW];
#pragma unroll
                for (int i = 0; i < LW; ++i)
                    v[i] = j0 - i >= 0 ? __hip_atomic_load(status + (j0 - i) * kRsBins + tid, __ATOMIC_RELAXED,
                                                           __HIP_MEMORY_SCOPE_AGENT)
                                       : kStIncl;
#pragma unroll
                for (int i = 0; i < LW; ++i) {
                    if (done) break;
                    uint32_t x = spin_max < 0 ? 0u : v[i];   // spin_max < 0: give up at once (tests only)
                    for (int spin = 0; x == 0 && spin < spin_max; ++spin) {   // not published yet: it will be
                        __builtin_amdgcn_s_sleep(1);
                        x = __hip_atomic_load(status + (j0 - i) * kRsBins + tid, __ATOMIC_RELAXED,
                                              __HIP_MEMORY_SCOPE_AGENT);
                    }
                    if (x == 0) {   // gave up: the prefix is wrong, and the plan call's status says so
                        __hip_atomic_fetch_or(lb_status, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        done = true;
                        break;
                    }
                    before += x & kStCount;
                    done = (x & kStIncl) != 0;
                }
            }
            __hip_atomic_store(entry, kStIncl | ((before + c) & kStCount), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    start[tid] = dbase + before;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < PER; ++r) {
        if (base + r * 64 >= n) continue;
        const int d = (int)((key[r] >> shift) & (kRsBins - 1));
        const uint32_t pos = start[d] + wcnt[wave][d] + rank[r];
        if (pos < n) {   // always true for consistent counts; keeps a bad input from writing outside
            kout[pos] = key[r];
            vout[pos] = val[r];
        }
    }
}

// ---------------------------------------------------------------------------
// blocks: union masks and item counts, then the items
// ---------------------------------------------------------------------------
// OR of a value over the 16 lanes of its block (lanes 16j..16j+15).
__device__ __forceinline__ uint32_t block_or16(uint32_t v) {
#pragma unroll
    for (int d = 1; d < 16; d <<= 1) v |= (uint32_t)__shfl_xor((int)v, d, 64);
    return v;
}

// A thread per block: its union mask and item count, and the exclusive scan of
// the counts within the kBlkTile blocks of a workgroup (lpre; the sum to
// part).  Range r = blockIdx.y (its keys at r * n, its blocks at r * nb, its
// sums at r * gridDim.x).  (The sorted keys are masked to the range's offsets
// and the rows clamped to [0, n): after a look-back that gave up they need not
// be what the sort meant, and the plan must still stay inside its arrays.)
constexpr int kBlkTile = 256;

__global__ void __launch_bounds__(kBlkTile) k_blk_count(const uint32_t* __restrict__ keys, int Kall, int S, int64_t n,
                                                        int64_t nb, uint32_t* __restrict__ bmask,
                                                        int32_t* __restrict__ lpre, int32_t* __restrict__ part) {
    __shared__ int32_t wsum[kBlkTile / 64];
    const int rg = blockIdx.y;
    const uint32_t kmask = range_kmask(range_len(rg, S, Kall));
    keys += (int64_t)rg * n;
    const int64_t b = (int64_t)blockIdx.x * kBlkTile + threadIdx.x;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t u = 0;
    if (b < nb) {
        uint32_t v[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) v[i] = keys[min(16 * b + i, n - 1)];   // (the last key again past the end)
#pragma unroll
        for (int i = 0; i < 16; ++i) u |= v[i];
        u &= kmask;
        bmask[(int64_t)rg * nb + b] = u;
    }
    const int32_t c = __popc(u);
    int32_t inc = c;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const int32_t x = __shfl_up(inc, o, 64);
        if (lane >= o) inc += x;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    int32_t before = inc - c, all = 0;
    for (int i = 0; i < kBlkTile / 64; ++i) {
        if (i < wave) before += wsum[i];
        all += wsum[i];
    }
    if (b < nb) lpre[(int64_t)rg * nb + b] = before;
    if (threadIdx.x == 0) part[(int64_t)rg * gridDim.x + blockIdx.x] = all;
}

// Range r = blockIdx.y: keys and perm at r * n, the range's offsets' dense
// rows from nbr + k0 * n, ibase at r * (nb + 1), items from items + 16 k0 nb.
// A workgroup's blocks lie in one tile of k_blk_count's, so it adds up the
// `parts` sums of the tiles before that one (a load per lane for 65,536
// blocks) instead of waiting for a scan of all counts (two launches, 10 us).
__global__ void __launch_bounds__(kPlanThreads) k_blk_fill(const uint32_t* __restrict__ keys, int Kall, int S,
                                                           const int32_t* __restrict__ perm,
                                                           const int32_t* __restrict__ nbr,
                                                           const int32_t* __restrict__ lpre,
                                                           const int32_t* __restrict__ part, int64_t parts,
                                                           int64_t* __restrict__ ibase, int64_t n, int64_t nb,
                                                           int32_t* __restrict__ items) {
    static_assert(kBlkTile * 16 % kPlanThreads == 0, "a workgroup's blocks lie in one counted tile");
    __shared__ int64_t wsum[kPlanThreads / 64];
    const int rg = blockIdx.y;
    const int k0 = range_k0(rg, S);
    const uint32_t kmask = range_kmask(range_len(rg, S, Kall));
    keys += (int64_t)rg * n;
    perm += (int64_t)rg * n;
    nbr += (int64_t)k0 * n;
    lpre += (int64_t)rg * nb;
    part += (int64_t)rg * parts;
    ibase += (int64_t)rg * (nb + 1);
    items += (int64_t)k0 * nb * 16;
    const int64_t i = (int64_t)blockIdx.x * kPlanThreads + threadIdx.x;
    const int64_t b = i >> 4;
    const int r = threadIdx.x & 15;
    const bool valid = i < n;
    const uint32_t key = valid ? keys[i] & kmask : 0u;
    const int32_t pr = valid ? perm[i] : 0;
    const int32_t lp = b < nb ? lpre[b] : 0;
    const int64_t tile = (int64_t)blockIdx.x * kPlanThreads / (16 * kBlkTile);
    int64_t sum = 0;
    for (int64_t x = threadIdx.x; x < tile; x += kPlanThreads) sum += part[x];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = sum;
    __syncthreads();
    int64_t base = lp;
    for (int w = 0; w < kPlanThreads / 64; ++w) base += wsum[w];
    const uint32_t u = block_or16(key);
    if (b >= nb) return;   // whole blocks of 16 lanes leave together
    if (r == 0) {
        ibase[b] = base;
        if (b == nb - 1) ibase[nb] = base + __popc(u);
    }
    const int64_t row = pr >= 0 && pr < n ? pr : 0;
    uint32_t m = u;
    // four of the block's offsets per round, their table entries loaded together
    for (int j = 0; m != 0; j += 4) {
        int kk[4];
        int32_t v[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            kk[t] = m ? __ffs(m) - 1 : -1;
            m &= m - 1;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) v[t] = kk[t] >= 0 && ((key >> kk[t]) & 1u) ? nbr[(int64_t)kk[t] * n + row] : -1;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            if (kk[t] >= 0) items[(base + j + t) * 16 + r] = v[t];
    }
}

// Sets each range's ibase[0] = 0 (ibase[r]: nb = 0) and clears the
// look-back status (a plan over no rows).
__global__ void k_plan_empty(int64_t* ibase, int R, uint32_t* lb_status) {
    if (blockIdx.x == 0 && (int)threadIdx.x < R) {
        ibase[threadIdx.x] = 0;
        if (lb_status && threadIdx.x == 0) *lb_status = 0u;
    }
}

static int plan_passes(int S) {
    // as many passes as for the widest range's mask alone (the popcount field fills spare bits)
    return (S + plan_key_pbits(S) + kRsBits - 1) / kRsBits;
}

// The workspace of a plan over n rows in R ranges of S offsets: keys and
// values twice, the digit counts of the row groups, their totals and the first
// pass's prefixes, the zeroed words (tickets, later passes' look-back entries),
// the blocks' item counts scanned within tiles and the tiles' sums.
struct PlanWs {
    uint32_t *ka, *kb;
    int32_t *va, *vb;
    uint16_t* mcnt;
    uint32_t *ghist, *pre, *ticket, *st;
    int64_t nzero, nm, nrs, nrs_later, parts;   // row groups, tiles of the first and the later passes, block tiles
    bool wide;                                  // later passes: kRsPerWide keys per thread
    int32_t *lpre, *part;
    size_t bytes;   // up to here
};

static PlanWs plan_ws_layout(void* ws, int64_t n, int R, int passes) {
    const int64_t nb = (n + 15) / 16;
    PlanWs L{};
    L.nm = (n + kMaskRows - 1) / kMaskRows;
    L.nrs = (n + kRsTile - 1) / kRsTile;
    L.wide = n >= kRsWideKeys;
    const int64_t later = L.wide ? kRsThreads * kRsPerWide : kRsTile;
    L.nrs_later = (n + later - 1) / later;
    L.parts = (nb + kBlkTile - 1) / kBlkTile;
    char* base = reinterpret_cast<char*>(ws);
    size_t o = 0;
    auto take = [&](size_t bytes) {
        char* p = base ? base + o : nullptr;
        o += al256(bytes);
        return p;
    };
    L.ka = reinterpret_cast<uint32_t*>(take((size_t)R * n * sizeof(uint32_t)));
    L.kb = reinterpret_cast<uint32_t*>(take((size_t)R * n * sizeof(uint32_t)));
    L.va = reinterpret_cast<int32_t*>(take((size_t)R * n * sizeof(int32_t)));
    L.vb = reinterpret_cast<int32_t*>(take((size_t)R * n * sizeof(int32_t)));
    L.mcnt = reinterpret_cast<uint16_t*>(take((size_t)R * passes * L.nm * kRsBins * sizeof(uint16_t)));
    L.ghist = reinterpret_cast<uint32_t*>(take((size_t)R * kRsMaxPasses * kRsBins * sizeof(uint32_t)));
    L.pre = reinterpret_cast<uint32_t*>(take((size_t)R * L.nrs * kRsBins * sizeof(uint32_t)));
    L.nzero = kRsMaxPasses + (int64_t)(passes - 1) * R * L.nrs_later * kRsBins;
    L.ticket = reinterpret_cast<uint32_t*>(take((size_t)L.nzero * sizeof(uint32_t)));
    L.st = L.ticket ? L.ticket + kRsMaxPasses : nullptr;
    L.lpre = reinterpret_cast<int32_t*>(take((size_t)R * nb * sizeof(int32_t)));
    L.part = reinterpret_cast<int32_t*>(take((size_t)R * L.parts * sizeof(int32_t)));
    L.bytes = o;
    return L;
}

// All ranges of a plan (R ranges of S offsets, the last one K - (R-1) S)
// go through one launch per step: the kernels take the range from the
// grid's second dimension (the radix passes from the tile's number), so a
// map with more than 32 offsets costs the launches of one plan.
// lb_status: the plan call's look-back status word, cleared by the first
// kernel and set by a pass that gave up.
static int plan_enqueue(const int32_t* nbr, int64_t n, int K, int R, int S, int32_t* perm, uint32_t* bmask,
                        int64_t* ibase, int32_t* items, void* ws, uint32_t* lb_status, int spin_max, hipStream_t s) {
    const int64_t nb = (n + 15) / 16;
    const int passes = plan_passes(S);
    const PlanWs L = plan_ws_layout(ws, n, R, passes);
    if (n == 0) {
        hipLaunchKernelGGL(k_plan_empty, dim3(1), dim3(64), 0, s, ibase, R, lb_status);
        GSC_LAUNCH_CHECK();
        return GSC_OK;
    }
    hipLaunchKernelGGL(k_plan_masks, dim3((unsigned)L.nm, (unsigned)R), dim3(kMaskRows), 0, s, nbr, n, K, S, passes,
                       L.ka, L.mcnt, L.ticket, L.nzero, lb_status);
    GSC_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_rs_counts, dim3(kRsBins / 64, (unsigned)(R * passes)), dim3(64 * kCntLanes), 0, s, L.mcnt, L.nm,
                       L.nrs, passes, L.ghist, L.pre);
    GSC_LAUNCH_CHECK();
    const uint32_t* kin = L.ka;
    const int32_t* vin = nullptr;
    for (int p = 0; p < passes; ++p) {
        uint32_t* kout = (p & 1) ? L.ka : L.kb;
        int32_t* vout = (p == passes - 1) ? perm : ((p & 1) ? L.va : L.vb);
        const uint32_t* gh = L.ghist + (int64_t)p * kRsBins;
        if (p == 0) {
            hipLaunchKernelGGL((k_rs_pass<true, kRsPer>), dim3((unsigned)(L.nrs * R)), dim3(kRsThreads), 0, s, kin, vin, n,
                               L.nrs, 0, gh, L.pre, (uint32_t*)nullptr, kout, vout, spin_max, lb_status);
        } else {
            auto* kern = L.wide ? k_rs_pass<false, kRsPerWide> : k_rs_pass<false, kRsPer>;
            hipLaunchKernelGGL(kern, dim3((unsigned)(L.nrs_later * R)), dim3(kRsThreads), 0, s, kin, vin, n, L.nrs_later,
                               p * kRsBits, gh, L.st + (int64_t)(p - 1) * R * L.nrs_later * kRsBins, L.ticket + p, kout,
                               vout, spin_max, lb_status);
        }
        GSC_LAUNCH_CHECK();
        kin = kout;
        vin = vout;
    }
    hipLaunchKernelGGL(k_blk_count, dim3((unsigned)L.parts, (unsigned)R), dim3(kBlkTile), 0, s, kin, K, S, n, nb, bmask,
                       L.lpre, L.part);
    GSC_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_blk_fill, dim3((unsigned)((n + kPlanThreads - 1) / kPlanThreads), (unsigned)R),
                       dim3(kPlanThreads), 0, s, kin, K, S, perm, nbr, L.lpre, L.part, L.parts, ibase, n, nb, items);
    GSC_LAUNCH_CHECK();
    return GSC_OK;
}

// The look-back status word sits in the last 256 bytes of the plan's ws.
static uint32_t* plan_status_word(void* ws, int64_t n_out, int K) {
    return reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(ws) + gsc_conv_plan_ws_bytes(n_out, K) - 256);
}

// Polls of one look-back entry before a pass gives up: kSpinMax, or the value
// of the environment variable GSC_PLAN_SPIN_LIMIT (a test hook: a negative
// value gives up at the first poll, so the failure path can be exercised
// while every kernel still ends normally).
static int lookback_spin_limit() {
    const char* e = getenv("GSC_PLAN_SPIN_LIMIT");
    if (!e || !*e) return kSpinMax;
    const long v = strtol(e, nullptr, 10);
    return v < -1 ? -1 : (v > kSpinMax ? kSpinMax : (int)v);
}

}  // namespace gsc

using namespace gsc;

extern "C" {

int64_t gsc_plan_blocks(int64_t n_out) { return n_out <= 0 ? 0 : (n_out + 15) / 16; }

int32_t gsc_plan_ranges(int32_t K) { return K < 1 || K > kPlanMaxKAll ? 0 : plan_ranges(K); }

size_t gsc_conv_plan_ws_bytes(int64_t n_out, int32_t K) {
    if (n_out < 0 || n_out > kRsMaxKeys || K < 1 || K > kPlanMaxKAll) return 0;
    return plan_ws_layout(nullptr, n_out, plan_ranges(K), plan_passes(plan_range_size(K))).bytes + 256;
}

int gsc_conv_plan(const int32_t* nbr, int64_t n_out, int32_t K, int32_t* perm, uint32_t* bmask, int64_t* ibase,
                  int32_t* items, int64_t cap_items, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (K < 1 || K > kPlanMaxKAll) return fail(GSC_EINVAL, "conv_plan: K=%d outside [1,%d]", K, kPlanMaxKAll);
    if (n_out < 0 || n_out > kRsMaxKeys)
        return fail(GSC_EINVAL, "conv_plan: n_out=%lld outside [0, %lld]", (long long)n_out, (long long)kRsMaxKeys);
    if (!ibase || !ws) return fail(GSC_EINVAL, "conv_plan: null ibase/ws");
    if (n_out > 0 && (!nbr || !perm || !bmask || !items))
        return fail(GSC_EINVAL, "conv_plan: null nbr/perm/bmask/items");
    const int64_t need_items = (int64_t)K * gsc_plan_blocks(n_out);
    if (cap_items < need_items)
        return fail(GSC_ESHORT, "conv_plan: cap_items=%lld, need K*ceil(n_out/16) = %lld", (long long)cap_items,
                    (long long)need_items);
    const size_t need = gsc_conv_plan_ws_bytes(n_out, K);
    if (ws_bytes < need) return fail(GSC_ESHORT, "conv_plan: ws needs %zu bytes, got %zu", need, ws_bytes);
    // every range of offsets in the same launches
    return plan_enqueue(nbr, n_out, K, plan_ranges(K), plan_range_size(K), perm, bmask, ibase, items, ws,
                        plan_status_word(ws, n_out, K), lookback_spin_limit(), reinterpret_cast<hipStream_t>(stream));
}

int gsc_conv_plan_status(const void* ws, size_t ws_bytes, int64_t n_out, int32_t K, void* stream) {
    clear_error();
    const size_t need = gsc_conv_plan_ws_bytes(n_out, K);
    if (!ws || need == 0) return fail(GSC_EINVAL, "conv_plan_status: null ws or bad n_out/K");
    if (ws_bytes < need) return fail(GSC_ESHORT, "conv_plan_status: ws needs %zu bytes, got %zu", need, ws_bytes);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    uint32_t word = 0;
    if (hipMemcpyAsync(&word, plan_status_word(const_cast<void*>(ws), n_out, K), sizeof(word), hipMemcpyDeviceToHost,
                       s) != hipSuccess ||
        hipStreamSynchronize(s) != hipSuccess)
        return fail(GSC_EHIP, "conv_plan_status: %s", hipGetErrorString(hipGetLastError()));
    if (word != 0)
        return fail(GSC_ETIMEOUT, "conv_plan: a radix pass gave up waiting for an earlier tile's count; the plan "
                                  "is not valid");
    return GSC_OK;
}

}  // extern "C"
