// Kernel map (a3): for every offset o_k and output row j, the input row of
// u_j + ts (.) o_k, if present.  Two passes over (output row, offset):
//   count: one lane per output row probes the table for every offset; the
//          input row found (or -1) goes to a dense offset-major neighbour
//          table nbr[k][j], and per offset a wave64 ballot of hits gives the
//          pair count of every 64-row group;
//   scan:  inclusive scan of each offset's group counts (one block per
//          offset; with many groups or offsets the device-wide scan);
//   fill:  each hit is placed at its group start plus its rank among the
//          wave's hits (popcount of the lower-lane mask), its input row read
//          from the neighbour table; the group starts (the group index gidx)
//          and the segment table come out on the way.
// Pairs of one offset therefore come out sorted by output row, and the
// result does not depend on scheduling.
//
// A grid table (see GridWord) answers a probe with an 8-byte word that stays in
// L2 and, for a hit, a row number; a hashed table with a slot, a random
// 128-byte line.
#include <algorithm>
#include <climits>
#include <mutex>
#include <vector>

#include "gsc_internal.h"

namespace gsc {

constexpr int kThreads = 256;
constexpr int kOffArgMax = 768;   // K * D offsets passed by value in the kernel arguments

// Offsets of the region, either by value in the kernel arguments (no host
// to device copy, so the map can be enqueued asynchronously) or in device
// memory (large regions, synchronous mode only).  Arguments are read where
// they lie, as the kernel's first one: indexed through the parameter itself,
// the compiler may copy all 3 KB of them to every lane's private memory first
// (count pass of 300,000 rows: 800 us instead of 20).
typedef const int32_t __attribute__((address_space(4))) KernargI32;
struct OffsArg {
    int32_t v[kOffArgMax];
    static __device__ __forceinline__ KernargI32* at(const OffsArg&, int64_t i) {
        return (KernargI32*)__builtin_amdgcn_kernarg_segment_ptr() + i;
    }
};
struct OffsPtr {
    const int32_t* p;
    static __device__ __forceinline__ const int32_t* at(const OffsPtr& o, int64_t i) { return o.p + i; }
};

__device__ __forceinline__ bool header_ok(const TableHeader* h, int ncol) {
    return (h->magic == kTableMagic || h->magic == kGridMagic) && h->ncol == ncol && h->status == 0;
}

// Offsets probed together per lane on a hashed table: 5 where a block has nine
// offsets (two rounds, as with 4 for up to eight; 27 offsets of 1 million rows
// 275 us, with 4 292 us), else 4 (7 and 8 offsets of 1 million rows 117 and
// 115 us, with 5 123 and 124 us).  Wide keys take one at a time, so that their
// path needs no more registers than the others.
template <typename KeyT, int NB>
constexpr int batch_of() { return sizeof(KeyT) > 8 ? 1 : NB; }

// Key arithmetic in KeyT (uint32_t when the table's keys fit in 32 bits, the
// usual case, uint64_t up to 62 bits, else the 128-bit wide key).  The packed
// key is linear in the coordinate: key(u + o) = base(u) + delta(o), exact (mod
// 2^bits) whenever every column of u + o lies in the table's box, so a probe
// is a range check per column and one add.
template <typename KeyT>
struct KeyOps;

template <>
struct KeyOps<uint32_t> {
    static __device__ __forceinline__ uint32_t hash(uint32_t k) { return fmix32(k); }
    static __device__ __forceinline__ bool eq(const Slot& e, uint32_t k) { return e.key == (unsigned long long)k; }
};
template <>
struct KeyOps<unsigned long long> {
    static __device__ __forceinline__ uint32_t hash(unsigned long long k) { return hash_key(k); }
    static __device__ __forceinline__ bool eq(const Slot& e, unsigned long long k) { return e.key == k; }
};
template <>
struct KeyOps<u128> {
    static __device__ __forceinline__ uint32_t hash(u128 k) { return hash_key_wide(k); }
    static __device__ __forceinline__ bool eq(const Slot& e, u128 k) { return e.key == wide_lo(k) && e.hi == wide_hi(k); }
};

// Count pass on a hashed table.  Each lane owns one output row.  Offsets are
// probed NB at a time; every load is issued unconditionally (a lane whose
// query is out of the box reads slot 0 and ignores it) so the NB loads are in
// flight together, and collision chains are followed in rounds.  A probe reads
// the whole 16-byte slot, so a hit also yields the input row, which goes to
// nbr[k * n_out + j] (-1 for a miss); hits are counted per 64-row group with
// a wave ballot.
template <typename KeyT, int NBT, typename Offs>
__device__ __forceinline__ void count_rows(const TableHeader* h, const Slot* __restrict__ slots,
                                           const int32_t* __restrict__ out_coords, int64_t n_out, int ncol,
                                           const Offs& offs, int k_begin, int k_end, int64_t G,
                                           int32_t* __restrict__ cnt, int32_t* __restrict__ nbr, bool ok, int64_t j) {
    const bool valid = ok && j < n_out;
    const int D = ncol - 1;
    const unsigned long long mask = ok ? (unsigned long long)h->capacity - 1 : 0;
    const int nblk = h->nblk;
    KeyT clear = ~(KeyT)0;
    int bsh[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        bsh[i] = h->blk_shift[i];
        if (i < nblk) clear &= ~((KeyT)1 << bsh[i]);
    }
    int32_t rel[kMaxCols], span[kMaxCols], shc[kMaxCols];
    KeyT base = 0;
    bool in_b = valid;
#pragma unroll
    for (int c = 0; c < kMaxCols; ++c) {
        if (c < ncol) {
            const int32_t lo = h->lo[c];
            shc[c] = h->shift[c];
            span[c] = h->hi[c] - lo;
            rel[c] = (valid ? out_coords[j * ncol + c] : lo) - lo;
            base += (KeyT)(uint32_t)rel[c] << shc[c];    // (KeyT)(int) sign-extends for 64-bit keys below
        }
    }
    if (sizeof(KeyT) >= 8) {   // redo with sign extension: rel may be negative when u is outside the box
        base = 0;
#pragma unroll
        for (int c = 0; c < kMaxCols; ++c)
            if (c < ncol) base += (KeyT)(long long)rel[c] << shc[c];
    }
    in_b = in_b && (uint32_t)rel[0] <= (uint32_t)span[0];
    const int64_t g = j >> 6;
    const bool writer = __lane_id() == 0 && g < G;
    constexpr int NB = batch_of<KeyT, NBT>();
    for (int k0 = k_begin; k0 < k_end; k0 += NB) {
        KeyT key[NB];
        unsigned long long pos[NB];
        bool pend[NB], hit[NB];
        int32_t row[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int k = min(k0 + b, k_end - 1);
            const auto* o = Offs::at(offs, (int64_t)k * D);
            bool in = in_b && k0 + b < k_end;
            KeyT delta = 0;
#pragma unroll
            for (int c = 1; c < kMaxCols; ++c) {
                if (c < ncol) {
                    in = in && (uint32_t)(rel[c] + o[c - 1]) <= (uint32_t)span[c];
                    delta += (KeyT)(long long)o[c - 1] << shc[c];
                }
            }
            const KeyT kk = base + delta;
            uint32_t local = 0;
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (i < nblk) local |= (uint32_t)((kk >> bsh[i]) & 1) << i;
            const uint32_t hash = KeyOps<KeyT>::hash(kk & clear);
            const unsigned long long hs = (((unsigned long long)hash << nblk) | local) & mask;
            key[b] = kk;
            pos[b] = in ? hs : 0;
            pend[b] = in;
            hit[b] = false;
            row[b] = -1;
        }
        for (unsigned long long round = 0; round <= mask; ++round) {
            Slot e[NB];
            if (round == 0) {
#pragma unroll
                for (int b = 0; b < NB; ++b) e[b] = slots[pos[b]];   // unconditional: all in flight
            } else {   // collision chains: few probes still pending
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    e[b].key = kEmptyKey;
                    e[b].val = -1;
                    e[b].hi = kHiUnset;
                    if (pend[b]) e[b] = slots[pos[b]];
                }
            }
            bool any = false;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                const bool h1 = pend[b] && KeyOps<KeyT>::eq(e[b], key[b]);
                const bool stop = h1 || e[b].key == kEmptyKey;
                hit[b] = hit[b] || h1;
                row[b] = h1 ? e[b].val : row[b];
                pend[b] = pend[b] && !stop;
                pos[b] = pend[b] ? ((pos[b] + 1) & mask) : pos[b];
                any = any || pend[b];
            }
            if (!__any(any)) break;
        }
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            const int k = k0 + b;
            if (k < k_end) {
                const unsigned long long m = __ballot(hit[b]);
                if (writer) cnt[(int64_t)k * G + g] = __popcll(m);
                if (j < n_out) nbr[(int64_t)k * n_out + j] = hit[b] ? row[b] : -1;
            }
        }
    }
}

// Count pass on a grid table: a lane per output row, kGridBatch offsets'
// words and then row numbers in flight together (a lane whose query lies
// outside the box, or on no cell of its step, reads word 0 and ignores it).
// Bound: the neighbour table written (4 K bytes per row) and the probes'
// address arithmetic.
//
// A block takes at most kGridBatch offsets (the grid's second dimension has
// the rest), so a lane's loads are one chain of header, row, word and row
// number, whatever K.
constexpr int kGridBatch = 9;

// The blocks of one row range and all its offsets run one after another on an
// XCD where the map is hashed and has more rows than this: they read the same
// lines of the table, which the XCD's L2 no longer holds once it has gone
// through all other rows (27 offsets: 300,000 rows 103 -> 88 us, 1 million
// 323 -> 275; 125 offsets of 1 million rows 1,633 -> 1,195).  With fewer rows,
// and on a grid's words, the other order was as fast or faster (29 offsets of
// 100,000 hashed rows 49 us against 52).
constexpr int64_t kNearRows = 200000;

template <int NC, typename Offs>
__device__ __forceinline__ void count_rows_grid(const void* table, const int32_t* __restrict__ out_coords, bool vec,
                                                int64_t n_out, int ncol, const Offs& offs, int k0, int k1, int64_t G,
                                                int32_t* __restrict__ cnt, int32_t* __restrict__ nbr, int64_t j) {
    const TableHeader* h = reinterpret_cast<const TableHeader*>(table);
    const GridWord* __restrict__ words = grid_words(table);
    const int32_t* __restrict__ rowof =
        reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(table) + h->rowof);
    const int D = ncol - 1;
    const bool valid = j < n_out;
    const int64_t jj = valid ? j : 0;
    int32_t x[NC], rel[NC];
    if (NC == 4 && vec) {
        const int4 q = reinterpret_cast<const int4*>(out_coords)[jj];
        x[0] = q.x;
        x[1 % NC] = q.y;
        x[2 % NC] = q.z;
        x[3 % NC] = q.w;
    } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) x[c] = c < ncol ? out_coords[jj * ncol + c] : 0;
    }
    uint32_t span[NC], low[NC], mul[NC];
    int step[NC];
    bool in_b = valid;
    uint32_t base = 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        rel[c] = 0;
        span[c] = low[c] = mul[c] = 0;
        step[c] = 0;
        if (c >= ncol) continue;
        span[c] = (uint32_t)(h->hi[c] - h->lo[c]);   // below 2^30
        step[c] = h->step[c];
        low[c] = (1u << step[c]) - 1u;
        mul[c] = h->cstride[c];
        // a row this far outside the box reaches it with no offset (|offset| <= 2^30); nearer ones plus an
        // offset stay within 32 bits, negative sums being above every span as unsigned numbers
        const int64_t d = (int64_t)x[c] - h->lo[c];
        const int64_t reach = c == 0 ? 0 : (int64_t)1 << 30;
        in_b = in_b && d >= -reach && d <= (int64_t)span[c] + reach;
        rel[c] = (int32_t)d;
        if (c == 0) {
            in_b = in_b && ((uint32_t)rel[c] & low[c]) == 0;
            base = ((uint32_t)rel[c] >> step[c]) * mul[c];
        }
    }
    bool stepped = false;   // uniform
    uint32_t all = base;
#pragma unroll
    for (int c = 1; c < NC; ++c) {
        stepped = stepped || step[c] != 0;
        all += (uint32_t)rel[c] * mul[c];
    }
    const int64_t g = j >> 6;
    const bool writer = (threadIdx.x & 63) == 0 && g < G;
    GridWord w[kGridBatch];
    uint32_t cell[kGridBatch];
    bool hit[kGridBatch];
    int32_t row[kGridBatch];
#pragma unroll
    for (int b = 0; b < kGridBatch; ++b) {
        const auto* o = Offs::at(offs, (int64_t)min(k0 + b, k1 - 1) * D);
        bool in = in_b && k0 + b < k1;
        uint32_t at;
        if (!stepped) {   // the cell is linear in the coordinate: the offset's part is a scalar
            uint32_t delta = 0;
#pragma unroll
            for (int c = 1; c < NC; ++c) {
                if (c >= ncol) continue;
                in = in && (uint32_t)rel[c] + (uint32_t)o[c - 1] <= span[c];
                delta += (uint32_t)o[c - 1] * mul[c];
            }
            at = all + delta;
        } else {
            at = base;
#pragma unroll
            for (int c = 1; c < NC; ++c) {
                if (c >= ncol) continue;
                const uint32_t v = (uint32_t)rel[c] + (uint32_t)o[c - 1];
                in = in && v <= span[c] && (v & low[c]) == 0;
                at += (v >> step[c]) * mul[c];
            }
        }
        cell[b] = in ? at : 0u;
        hit[b] = in;
        w[b] = words[cell[b] >> 5];
    }
#pragma unroll
    for (int b = 0; b < kGridBatch; ++b) {
        hit[b] = hit[b] && ((w[b].bits >> (cell[b] & 31)) & 1u);
        row[b] = rowof[hit[b] ? grid_place(w[b], cell[b]) : 0u];
    }
#pragma unroll
    for (int b = 0; b < kGridBatch; ++b) {
        if (k0 + b >= k1) break;
        const unsigned long long m = __ballot(hit[b]);
        if (writer) cnt[(int64_t)(k0 + b) * G + g] = __popcll(m);
        if (valid) nbr[(int64_t)(k0 + b) * n_out + j] = hit[b] ? row[b] : -1;
    }
}

template <typename Offs>
__global__ void __launch_bounds__(kThreads) k_kmap_count(Offs offs, const void* table,
                                                         const int32_t* __restrict__ out_coords, bool vec,
                                                         int64_t n_out, int ncol, int K, int64_t G,
                                                         int32_t* __restrict__ cnt, int32_t* __restrict__ nbr,
                                                         int64_t* err) {
    const TableHeader* h = reinterpret_cast<const TableHeader*>(table);
    const Slot* __restrict__ slots = table_slots(table);
    const bool ok = header_ok(h, ncol);
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) *err = ok ? 0 : 1;
    const int per = (K + gridDim.y - 1) / gridDim.y;
    unsigned rows = (unsigned)xcd_unit(blockIdx.x, gridDim.x), part = blockIdx.y;
    if (h->magic != kGridMagic && n_out > kNearRows) {   // uniform
        const unsigned unit = (unsigned)xcd_unit(blockIdx.y * gridDim.x + blockIdx.x, gridDim.x * gridDim.y);
        rows = unit / gridDim.y;
        part = unit - rows * gridDim.y;
    }
    const int64_t j = (int64_t)rows * kThreads + threadIdx.x;
    const int k0 = (int)part * per, k1 = min(K, k0 + per);
    // uniform: all lanes take the same path
    if (ok && h->magic == kGridMagic) {
        if (ncol == 4) count_rows_grid<4>(table, out_coords, vec, n_out, ncol, offs, k0, k1, G, cnt, nbr, j);
        else if (ncol == 5) count_rows_grid<5>(table, out_coords, vec, n_out, ncol, offs, k0, k1, G, cnt, nbr, j);
        else count_rows_grid<kMaxCols>(table, out_coords, vec, n_out, ncol, offs, k0, k1, G, cnt, nbr, j);
    } else if (h->total_bits <= 32) {
        if (per > 8) count_rows<uint32_t, 5>(h, slots, out_coords, n_out, ncol, offs, k0, k1, G, cnt, nbr, ok, j);
        else count_rows<uint32_t, 4>(h, slots, out_coords, n_out, ncol, offs, k0, k1, G, cnt, nbr, ok, j);
    } else if (h->total_bits <= kNarrowKeyBits) {
        if (per > 8)
            count_rows<unsigned long long, 5>(h, slots, out_coords, n_out, ncol, offs, k0, k1, G, cnt, nbr, ok, j);
        else
            count_rows<unsigned long long, 4>(h, slots, out_coords, n_out, ncol, offs, k0, k1, G, cnt, nbr, ok, j);
    } else {
        count_rows<u128, 1>(h, slots, out_coords, n_out, ncol, offs, k0, k1, G, cnt, nbr, ok, j);
    }
}

// Scan pass: the inclusive scan, in place, of the group counts of one offset
// per block (cnt[k * G + g], g < G).  The offsets' totals are the last entries,
// so the fill pass finds every group's start from them without a scan over
// all K * G counts: one launch instead of the two of the device-wide scan
// (which took 10 us for 27 x 4,689 counts).  A block walks G counts in rounds
// of kScanRound, so this is for at most two rounds (kScanMaxGroups): maps of
// 500,000 rows (7,812 groups) and 1, 8 and 27 offsets take 22.6, 33.1 and 73.0
// us against 25.1, 34.0 and 73.9 with the device-wide scan, of 1 million 37.9,
// 54.8 and 152.8 against 33.5, 51.7 and 149.9, of 4 million 124, 223 and 645
// against 92, 197 and 610.  The offsets' totals are scanned again by every fill
// block, so for at most kScanMaxK.
constexpr int kScanThreads = 1024;
constexpr int kScanPer = 4;
constexpr int64_t kScanRound = (int64_t)kScanThreads * kScanPer;
constexpr int64_t kScanMaxGroups = 2 * kScanRound;
constexpr int kScanMaxK = 1024;

__global__ void __launch_bounds__(kScanThreads) k_kmap_scan(int32_t* __restrict__ cnt, int64_t G) {
    __shared__ int32_t wsum[2][kScanThreads / 64];
    cnt += (int64_t)blockIdx.x * G;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    int32_t carry = 0;
    int buf = 0;
    for (int64_t g0 = 0; g0 < G; g0 += kScanRound, buf ^= 1) {
        const int64_t g = g0 + (int64_t)threadIdx.x * kScanPer;
        int32_t v[kScanPer];
#pragma unroll
        for (int i = 0; i < kScanPer; ++i) v[i] = g + i < G ? cnt[g + i] : 0;
#pragma unroll
        for (int i = 1; i < kScanPer; ++i) v[i] += v[i - 1];
        int32_t inc = v[kScanPer - 1];
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int32_t u = __shfl_up(inc, d, 64);
            if (lane >= d) inc += u;
        }
        if (lane == 63) wsum[buf][wave] = inc;
        __syncthreads();   // one barrier a round: the other round's sums are in the other buffer
        int32_t before = carry;
        for (int i = 0; i < kScanThreads / 64; ++i) {
            if (i < wave) before += wsum[buf][i];
            carry += wsum[buf][i];
        }
        before += inc - v[kScanPer - 1];
#pragma unroll
        for (int i = 0; i < kScanPer; ++i)
            if (g + i < G) cnt[g + i] = before + v[i];
    }
}

// Fill pass: lane j reads its row of the neighbour table offset by offset;
// each hit goes to its group start plus its rank among the wave's hits.
// SCAN: cnt holds the offsets' inclusive scans (k_kmap_scan); the block scans
// the offsets' totals, and the pass writes gidx, seg and *total itself, and no
// pair when the total exceeds cap.  Otherwise gidx is given.
template <bool SCAN>
__global__ void __launch_bounds__(kThreads) k_kmap_fill(int64_t n_out, int K, int64_t G,
                                                        const int32_t* __restrict__ nbr,
                                                        const int32_t* __restrict__ cnt, int64_t* __restrict__ gidx,
                                                        int64_t* __restrict__ seg, int64_t* __restrict__ total,
                                                        int32_t* __restrict__ in_idx, int32_t* __restrict__ out_idx,
                                                        int64_t cap) {
    __shared__ int64_t kbase[SCAN ? kScanMaxK + 1 : 1];
    const int64_t j = xcd_unit(blockIdx.x, gridDim.x) * kThreads + threadIdx.x;
    const bool valid = j < n_out;
    const int64_t g = j >> 6;
    const int lane = threadIdx.x & 63;
    if constexpr (SCAN) {
        if (threadIdx.x < 64) {   // exclusive scan of the offsets' totals
            int64_t carry = 0;
            for (int k0 = 0; k0 < K; k0 += 64) {
                const int k = k0 + lane;
                const int64_t c = k < K ? cnt[(int64_t)k * G + G - 1] : 0;
                int64_t inc = c;
#pragma unroll
                for (int d = 1; d < 64; d <<= 1) {
                    const int64_t u = __shfl_up(inc, d, 64);
                    if (lane >= d) inc += u;
                }
                if (k < K) kbase[k] = carry + inc - c;
                carry += __shfl(inc, 63, 64);
            }
            if (lane == 0) kbase[K] = carry;
        }
        __syncthreads();
        if (blockIdx.x == 0) {
            for (int k = threadIdx.x; k <= K; k += kThreads) seg[k] = kbase[k];
            if (threadIdx.x == 0) {
                gidx[(int64_t)K * G] = kbase[K];
                if (total) *total = kbase[K];
            }
        }
        if (kbase[K] > cap) cap = 0;   // (gidx is still written)
    }
    const unsigned long long below = lanemask_lt();
    constexpr int B = 9;   // offsets whose table entries are loaded together (a divisor of 27)
    for (int kc = 0; kc < K; kc += 63) {   // 63 offsets' group starts at a time, one per lane
        const int kl = kc + lane;
        int64_t start = 0;
        if (g < G && lane < 63 && kl < K) {
            if constexpr (SCAN) {
                start = kbase[kl] + (g > 0 ? cnt[(int64_t)kl * G + g - 1] : 0);
                gidx[(int64_t)kl * G + g] = start;
            } else {
                start = gidx[(int64_t)kl * G + g];
            }
        }
        const int kend = min(K, kc + 63);
        for (int k0 = kc; k0 < kend; k0 += B) {
            int32_t r[B];
#pragma unroll
            for (int b = 0; b < B; ++b) r[b] = valid && k0 + b < kend ? nbr[(int64_t)(k0 + b) * n_out + j] : -1;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                if (k0 + b >= kend) break;
                const int64_t gs = __shfl(start, k0 + b - kc, 64);
                const bool hit = r[b] >= 0;
                const unsigned long long m = __ballot(hit);
                if (hit) {
                    const int64_t pos = gs + __popcll(m & below);
                    if (pos < cap) {
                        in_idx[pos] = r[b];
                        out_idx[pos] = (int32_t)j;
                    }
                }
            }
        }
    }
}

// Group starts, segments and pairs from the dense form and the group counts.
// res (nullable, device): res[0] gets the number of pairs.  With n_pairs (host) the
// call waits and reads res[0..1], and sets it (ESHORT
// when it exceeds cap_pairs, EINVAL when the count pass found no valid table).
static int pairs_enqueue(int64_t n, int K, int64_t G, const int32_t* nbr, int32_t* cnt, int64_t* gidx, int64_t* seg,
                         int64_t* res, void* scan_ws, int32_t* in_idx, int32_t* out_idx, int64_t cap_pairs,
                         int64_t* n_pairs, int ncol, hipStream_t s) {
    const unsigned nblk = (unsigned)((n + kThreads - 1) / kThreads);
    const bool by_offset = G > 0 && G <= kScanMaxGroups && K <= kScanMaxK;
    if (by_offset) {
        hipLaunchKernelGGL(k_kmap_scan, dim3((unsigned)K), dim3(kScanThreads), 0, s, cnt, G);
        GSC_LAUNCH_CHECK();
        hipLaunchKernelGGL(k_kmap_fill<true>, dim3(nblk), dim3(kThreads), 0, s, n, K, G, nbr, cnt, gidx, seg, res,
                           in_idx, out_idx, cap_pairs);
        GSC_LAUNCH_CHECK();
    } else {
        // the scan also writes seg[k] = gidx[k * G] (a launch of its own without groups)
        int rc = G > 0 ? scan_counts(cnt, K * G, gidx, res, scan_ws, s, seg, G)
                       : scan_counts(cnt, 0, gidx, res, scan_ws, s);
        if (rc) return rc;
        if (G == 0) {
            rc = seg_from_gidx(gidx, K, G, seg, s);
            if (rc) return rc;
        }
    }
    int64_t bound = cap_pairs;
    if (n_pairs) {
        int64_t hres[2];
        GSC_HIP(hipMemcpyAsync(hres, res, sizeof(hres), hipMemcpyDeviceToHost, s));
        GSC_HIP(hipStreamSynchronize(s));
        // the count kernel (launched when n > 0) writes the header check
        if (nblk > 0 && hres[1])
            return fail(GSC_EINVAL, "kernel_map: in_table is not a valid table of %d-column rows", ncol);
        *n_pairs = hres[0];
        if (hres[0] > cap_pairs)
            return fail(GSC_ESHORT, "kernel_map: %lld pairs exceed cap_pairs=%lld", (long long)hres[0],
                        (long long)cap_pairs);
        bound = hres[0];
    }
    if (!by_offset && nblk > 0 && bound > 0) {
        hipLaunchKernelGGL(k_kmap_fill<false>, dim3(nblk), dim3(kThreads), 0, s, n, K, G, nbr, nullptr, gidx, nullptr,
                           nullptr, in_idx, out_idx, cap_pairs);
        GSC_LAUNCH_CHECK();
    }
    return GSC_OK;
}

static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

// ---------------------------------------------------------------------------
// Role reversal of a map without the coordinate table (Sec. 4.2: the pairs of
// the transposed convolution are those of the forward one with input and
// output exchanged).  A map lists each input row at most once per offset (its
// output coordinate is the input's minus the scaled offset), so the reversed
// map's dense form is a scatter of the pairs; the count, scan and fill passes
// of the kernel map then list the pairs by the former input row.
// ---------------------------------------------------------------------------
__global__ void k_fill_neg1(int32_t* __restrict__ p, int64_t n) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = -1;
}

// nbr[k * n_rev + in_idx[p]] = out_idx[p] for the pairs p < seg[K] (offset k
// of pair p found by a search of seg); a row outside [0, n_rev) is skipped
// (the caller's map is checked: err[0] is set).
__global__ void __launch_bounds__(kThreads) k_map_scatter(const int32_t* __restrict__ in_idx,
                                                          const int32_t* __restrict__ out_idx,
                                                          const int64_t* __restrict__ seg, int K, int64_t cap,
                                                          int64_t n_rev, int32_t* __restrict__ nbr,
                                                          int32_t* __restrict__ err) {
    const int64_t total = seg[K] < cap ? seg[K] : cap;
    for (int64_t p = (int64_t)blockIdx.x * kThreads + threadIdx.x; p < total; p += (int64_t)gridDim.x * kThreads) {
        int lo = 0, hi = K;   // the k with seg[k] <= p < seg[k + 1]
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (seg[mid] <= p) lo = mid;
            else hi = mid;
        }
        const int32_t r = in_idx[p];
        if (r >= 0 && r < n_rev) nbr[(int64_t)lo * n_rev + r] = out_idx[p];
        else atomicOr(err, 1);
    }
}

// cnt[k * G + g] = entries >= 0 of nbr[k * n][64 g .. 64 g + 63].
__global__ void __launch_bounds__(kThreads) k_nbr_count(const int32_t* __restrict__ nbr, int64_t n, int K, int64_t G,
                                                        int32_t* __restrict__ cnt) {
    const int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x;
    const int64_t g = j >> 6;
    const bool valid = j < n;
    for (int k = 0; k < K; ++k) {
        const unsigned long long m = __ballot(valid && nbr[(int64_t)k * n + j] >= 0);
        if ((threadIdx.x & 63) == 0 && g < G) cnt[(int64_t)k * G + g] = (int32_t)__popcll(m);
    }
}

template <typename Offs>
static int kmap_enqueue(const void* in_table, const int32_t* out_coords, int64_t n_out, int ncol, Offs offs, int K,
                        int64_t G, int32_t* in_idx, int32_t* out_idx, int64_t cap_pairs, int64_t* seg, int64_t* gidx,
                        int64_t* n_pairs, int64_t* res, int32_t* cnt, int32_t* nbr, void* scan_ws, hipStream_t s) {
    const unsigned nblk = (unsigned)((n_out + kThreads - 1) / kThreads);
    if (nblk > 0) {
        const bool vec = ncol == 4 && ((uintptr_t)out_coords & 15) == 0;   // rows as 16-byte words
        // a multiple of the XCDs, so that the blocks of one row range and all offsets share an L2
        const unsigned gx = (nblk + kNumXcd - 1) / kNumXcd * kNumXcd;
        const unsigned gy = (unsigned)((K + kGridBatch - 1) / kGridBatch);
        hipLaunchKernelGGL(k_kmap_count<Offs>, dim3(gx, gy), dim3(kThreads), 0, s, offs, in_table, out_coords, vec,
                           n_out, ncol, K, G, cnt, nbr, res + 1);
        GSC_LAUNCH_CHECK();
    }
    return pairs_enqueue(n_out, K, G, nbr, cnt, gidx, seg, res, scan_ws, in_idx, out_idx, cap_pairs, n_pairs, ncol, s);
}

// Host-side checks and the offsets scaled by the tensor stride (by value in
// `arg` when K * D <= kOffArgMax, always in `offs`).
static int kmap_prepare(const void* in_table, const int32_t* out_coords, int64_t n_out, int32_t D,
                        const int32_t* offsets, int32_t K, const int32_t* tensor_stride, int32_t* in_idx,
                        int32_t* out_idx, int64_t cap_pairs, int64_t* seg, int64_t* gidx, int64_t* n_pairs,
                        OffsArg& arg, std::vector<int32_t>& offs) {
    if (D < 1 || D + 1 > kMaxCols) return fail(GSC_EINVAL, "kernel_map: D=%d outside [1,%d]", D, kMaxCols - 1);
    if (K < 1) return fail(GSC_EINVAL, "kernel_map: K=%d must be >= 1", K);
    if (n_out < 0 || n_out > INT32_MAX) return fail(GSC_EINVAL, "kernel_map: n_out=%lld invalid", (long long)n_out);
    if (!in_table || !offsets || !seg || !gidx) return fail(GSC_EINVAL, "kernel_map: null in_table/offsets/seg/gidx");
    if (n_out > 0 && !out_coords) return fail(GSC_EINVAL, "kernel_map: out_coords is null");
    if (cap_pairs < 0) return fail(GSC_EINVAL, "kernel_map: cap_pairs < 0");
    if (cap_pairs > 0 && (!in_idx || !out_idx)) return fail(GSC_EINVAL, "kernel_map: null in_idx/out_idx");
    const bool by_value = (int64_t)K * D <= kOffArgMax;
    if (!n_pairs) {   // asynchronous mode
        if (cap_pairs < (int64_t)K * n_out)
            return fail(GSC_ESHORT, "kernel_map: asynchronous mode needs cap_pairs >= K*n_out = %lld",
                        (long long)K * n_out);
        if (!by_value)
            return fail(GSC_EINVAL, "kernel_map: asynchronous mode needs K*D <= %d (got %d)", kOffArgMax, K * D);
    }
    offs.assign((size_t)K * D, 0);
    for (int k = 0; k < K; ++k)
        for (int d = 0; d < D; ++d) {
            const int64_t ts = tensor_stride ? tensor_stride[d] : 1;
            if (ts < 1) return fail(GSC_EINVAL, "kernel_map: tensor_stride[%d]=%lld must be >= 1", d, (long long)ts);
            const int64_t v = ts * (int64_t)offsets[(size_t)k * D + d];
            if (v < -(1ll << 30) || v > (1ll << 30))
                return fail(GSC_ERANGE, "kernel_map: scaled offset %lld out of range", (long long)v);
            offs[(size_t)k * D + d] = (int32_t)v;
            if (by_value) arg.v[(size_t)k * D + d] = (int32_t)v;
        }
    return GSC_OK;
}

// Scratch of the allocation-free kernel map: a device array of fixed size in
// the library's code object.  Each GPU holds its own copy at its own address,
// taken once per device with hipGetSymbolAddress (the array's name is not a
// device address in host code).  Calls on one GPU share it, so calls that
// overlap on one GPU race.
constexpr size_t kNoAllocScratchBytes = (size_t)8 << 20;
__device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

static int noalloc_scratch(char** out) {
    int dev = -1;
    GSC_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(GSC_EINVAL, "kernel_map_noalloc: device %d unsupported", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        GSC_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) return fail(GSC_EHIP, "kernel_map_noalloc: no address for the scratch array on device %d", dev);
        g_scratch_ptr[dev] = p;
    }
    *out = reinterpret_cast<char*>(g_scratch_ptr[dev]);
    return GSC_OK;
}

}  // namespace gsc

using namespace gsc;

extern "C" {

int64_t gsc_kmap_groups(int64_t n_out) { return n_out <= 0 ? 0 : (n_out + 63) / 64; }

size_t gsc_kmap_ws_bytes(int64_t n_out, int32_t K, int32_t D) {
    if (n_out < 0 || K < 1 || D < 1) return 0;
    const int64_t G = gsc_kmap_groups(n_out);
    size_t b = align256((size_t)K * D * sizeof(int32_t));      // offsets (scaled)
    b += align256(3 * sizeof(int64_t));                         // total, error flag
    b += align256((size_t)K * G * sizeof(int32_t));             // counts
    b += align256((size_t)K * n_out * sizeof(int32_t));         // neighbour table
    b += scan_ws_bytes(K * G);
    return b + 256;
}

int gsc_kernel_map(const void* in_table, const int32_t* out_coords, int64_t n_out, int32_t D, const int32_t* offsets,
                   int32_t K, const int32_t* tensor_stride, int32_t* in_idx, int32_t* out_idx, int64_t cap_pairs,
                   int64_t* seg, int64_t* gidx, int32_t* nbr_out, int64_t* n_pairs, void* ws, size_t ws_bytes,
                   void* stream) {
    clear_error();
    if (!ws) return fail(GSC_EINVAL, "kernel_map: null ws");
    if (ws_bytes < gsc_kmap_ws_bytes(n_out, K, D))
        return fail(GSC_ESHORT, "kernel_map: ws needs %zu bytes, got %zu", gsc_kmap_ws_bytes(n_out, K, D), ws_bytes);
    OffsArg arg;
    std::vector<int32_t> offs;
    int rc = kmap_prepare(in_table, out_coords, n_out, D, offsets, K, tensor_stride, in_idx, out_idx, cap_pairs, seg,
                          gidx, n_pairs, arg, offs);
    if (rc) return rc;
    const bool by_value = (int64_t)K * D <= kOffArgMax;

    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int ncol = D + 1;
    const int64_t G = gsc_kmap_groups(n_out);
    char* w = reinterpret_cast<char*>(ws);
    int32_t* d_offs = reinterpret_cast<int32_t*>(w);
    w += align256((size_t)K * D * sizeof(int32_t));
    int64_t* res = reinterpret_cast<int64_t*>(w);   // res[0] = total, res[1] = header error
    w += align256(3 * sizeof(int64_t));
    int32_t* cnt = reinterpret_cast<int32_t*>(w);
    w += align256((size_t)K * G * sizeof(int32_t));
    int32_t* nbr = nbr_out ? nbr_out : reinterpret_cast<int32_t*>(w);   // the caller's dense map, if asked for
    w += align256((size_t)K * n_out * sizeof(int32_t));
    void* scan_ws = w;
    if (by_value)
        return kmap_enqueue(in_table, out_coords, n_out, ncol, arg, K, G, in_idx, out_idx, cap_pairs, seg, gidx,
                            n_pairs, res, cnt, nbr, scan_ws, s);
    // synchronous mode: the copy below completes before this call returns
    GSC_HIP(hipMemcpyAsync(d_offs, offs.data(), offs.size() * sizeof(int32_t), hipMemcpyHostToDevice, s));
    return kmap_enqueue(in_table, out_coords, n_out, ncol, OffsPtr{d_offs}, K, G, in_idx, out_idx, cap_pairs,
                        seg, gidx, n_pairs, res, cnt, nbr, scan_ws, s);
}

size_t gsc_kernel_map_noalloc_bytes(int64_t n_out, int32_t K) {
    if (n_out < 0 || K < 1) return 0;
    const int64_t G = gsc_kmap_groups(n_out);
    return align256(3 * sizeof(int64_t)) + align256((size_t)K * G * sizeof(int32_t)) + scan_ws_bytes(K * G);
}

int gsc_kernel_map_noalloc(const void* in_table, const int32_t* out_coords, int64_t n_out, int32_t D,
                           const int32_t* offsets, int32_t K, const int32_t* tensor_stride, int32_t* in_idx,
                           int32_t* out_idx, int64_t cap_pairs, int64_t* seg, int64_t* gidx, int32_t* nbr,
                           void* stream) {
    clear_error();
    if (!nbr) return fail(GSC_EINVAL, "kernel_map_noalloc: the dense form nbr is required");
    const size_t need = gsc_kernel_map_noalloc_bytes(n_out, K);
    if (n_out >= 0 && K >= 1 && need > kNoAllocScratchBytes)
        return fail(GSC_ERANGE, "kernel_map_noalloc: needs %zu bytes of scratch, the library holds %zu per GPU "
                    "(n_out=%lld, K=%d); use gsc_kernel_map with a workspace", need, kNoAllocScratchBytes,
                    (long long)n_out, K);
    OffsArg arg;
    std::vector<int32_t> offs;
    int rc = kmap_prepare(in_table, out_coords, n_out, D, offsets, K, tensor_stride, in_idx, out_idx, cap_pairs, seg,
                          gidx, nullptr, arg, offs);
    if (rc) return rc;
    char* w = nullptr;
    rc = noalloc_scratch(&w);
    if (rc) return rc;
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int64_t G = gsc_kmap_groups(n_out);
    int64_t* res = reinterpret_cast<int64_t*>(w);
    w += align256(3 * sizeof(int64_t));
    int32_t* cnt = reinterpret_cast<int32_t*>(w);
    w += align256((size_t)K * G * sizeof(int32_t));
    return kmap_enqueue(in_table, out_coords, n_out, D + 1, arg, K, G, in_idx, out_idx, cap_pairs, seg, gidx,
                        nullptr, res, cnt, nbr, w, s);
}

size_t gsc_kernel_map_transpose_ws_bytes(int64_t n_rev, int32_t K) {
    if (n_rev < 0 || K < 1) return 0;
    const int64_t G = gsc_kmap_groups(n_rev);
    return align256(sizeof(int64_t)) + align256((size_t)K * G * sizeof(int32_t)) + scan_ws_bytes(K * G) + 256;
}

int gsc_kernel_map_transpose(const int32_t* in_idx, const int32_t* out_idx, const int64_t* seg, int32_t K,
                             int64_t cap_pairs, int64_t n_rev, int32_t* t_in_idx, int32_t* t_out_idx, int64_t* t_seg,
                             int64_t* t_gidx, int32_t* t_nbr, void* ws, size_t ws_bytes, void* stream) {
    clear_error();
    if (K < 1 || cap_pairs < 0 || n_rev < 0 || n_rev > INT32_MAX)
        return fail(GSC_EINVAL, "kernel_map_transpose: bad K=%d, cap_pairs=%lld or n_rev=%lld", K,
                    (long long)cap_pairs, (long long)n_rev);
    if (!seg || !t_seg || !t_gidx || !t_nbr || !ws)
        return fail(GSC_EINVAL, "kernel_map_transpose: null seg/t_seg/t_gidx/t_nbr/ws");
    if (cap_pairs > 0 && (!in_idx || !out_idx || !t_in_idx || !t_out_idx))
        return fail(GSC_EINVAL, "kernel_map_transpose: null pair arrays");
    const size_t need = gsc_kernel_map_transpose_ws_bytes(n_rev, K);
    if (ws_bytes < need)
        return fail(GSC_ESHORT, "kernel_map_transpose: ws needs %zu bytes, got %zu", need, ws_bytes);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int64_t G = gsc_kmap_groups(n_rev);
    char* w = reinterpret_cast<char*>(ws);
    int32_t* err = reinterpret_cast<int32_t*>(w);
    w += align256(sizeof(int64_t));
    int32_t* cnt = reinterpret_cast<int32_t*>(w);
    w += align256((size_t)K * G * sizeof(int32_t));
    const int64_t n_dense = (int64_t)K * n_rev;
    hipLaunchKernelGGL(k_fill_neg1, dim3((unsigned)std::min<int64_t>((n_dense + kThreads - 1) / kThreads + 1, 4096)),
                       dim3(kThreads), 0, s, t_nbr, n_dense);
    GSC_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_zero_i64, dim3(1), dim3(64), 0, s, reinterpret_cast<int64_t*>(err), (int64_t)1);
    GSC_LAUNCH_CHECK();
    if (cap_pairs > 0) {
        hipLaunchKernelGGL(k_map_scatter, dim3((unsigned)std::min<int64_t>((cap_pairs + kThreads - 1) / kThreads, 8192)),
                           dim3(kThreads), 0, s, in_idx, out_idx, seg, K, cap_pairs, n_rev, t_nbr, err);
        GSC_LAUNCH_CHECK();
    }
    const unsigned nblk = (unsigned)((n_rev + kThreads - 1) / kThreads);
    if (nblk > 0) {
        hipLaunchKernelGGL(k_nbr_count, dim3(nblk), dim3(kThreads), 0, s, t_nbr, n_rev, K, G, cnt);
        GSC_LAUNCH_CHECK();
    }
    return pairs_enqueue(n_rev, K, G, t_nbr, cnt, t_gidx, t_seg, nullptr, w, t_in_idx, t_out_idx, cap_pairs, nullptr,
                         0, s);
}

int gsc_kernel_map_transpose_status(const void* ws, void* stream) {
    clear_error();
    if (!ws) return fail(GSC_EINVAL, "kernel_map_transpose_status: null ws");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int32_t e = 0;
    GSC_HIP(hipMemcpyAsync(&e, ws, sizeof(e), hipMemcpyDeviceToHost, s));
    GSC_HIP(hipStreamSynchronize(s));
    return e ? fail(GSC_EINVAL, "kernel_map_transpose: a pair's input row lies outside [0, n_rev)") : GSC_OK;
}

}  // extern "C"
