// Coordinate table (a1) and output coordinates of a strided convolution (a2).
//
// A table holds the rows (b, x_1..x_D) relative to their bounding box, which
// the device finds, so a build needs no host round trip.  It takes one of two
// forms, decided on the device from the box:
//   grid:  one bit per cell of the box and the row numbers of the occupied
//          cells (GridWord), when the box has at most as many cells as the
//          table's memory holds words for (see grid_layout);
//   hash:  open addressing with linear probing over 16-byte slots, the row
//          packed into a key relative to the box, batch column in the high
//          bits: any box of up to kMaxKeyBits key bits.
// At 300,082 rows of two rooms at 2 cm (120 cells per row) a grid takes 33 us
// to build and a map of 27 offsets 35 us, hashed slots 40 and 83 us.
#include <algorithm>
#include <climits>

#include <cstddef>
#include <cstring>

#include "gsc_internal.h"

namespace gsc {

constexpr int kThreads = 256;

struct StrideArg {
    int32_t s[kMaxCols];   // s[0] = 1 (batch), s[c] = stride of spatial column c (all 1: the rows as they are)
};

static StrideArg unit_stride() {
    StrideArg st;
    for (int c = 0; c < kMaxCols; ++c) st.s[c] = 1;
    return st;
}

template <int NC>
__device__ __forceinline__ void load_row(const int32_t* __restrict__ coords, bool vec, int64_t r, int ncol,
                                         const StrideArg& st, int32_t* v, bool* bad) {
    int32_t raw[NC];
    if (NC % 4 == 0 && vec) {   // uniform: rows of four or eight columns from a 16-byte aligned array
#pragma unroll
        for (int i = 0; i < NC / 4; ++i) {
            const int4 q = reinterpret_cast<const int4*>(coords)[r * (NC / 4) + i];
            raw[4 * i] = q.x;
            raw[(4 * i + 1) % NC] = q.y;
            raw[(4 * i + 2) % NC] = q.z;
            raw[(4 * i + 3) % NC] = q.w;
        }
    } else {
#pragma unroll
        for (int c = 0; c < NC; ++c) raw[c] = c < ncol ? coords[r * ncol + c] : 0;
    }
#pragma unroll
    for (int c = 0; c < NC; ++c) v[c] = c > 0 && c < ncol ? floor_mul(raw[c], st.s[c], bad) : raw[c];
}

constexpr int kBoxRows = 4;                     // rows in flight per thread (half as many points)

// Bounding box of a set of values per column.
struct Box {
    int32_t lo[kMaxCols], hi[kMaxCols], all_or[kMaxCols], all_and[kMaxCols];
    int32_t bad;
};

template <int NC>
__device__ __forceinline__ void box_wave(Box& x, int ncol) {
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c >= ncol) break;   // uniform
            x.lo[c] = min(x.lo[c], __shfl_xor(x.lo[c], d, 64));
            x.hi[c] = max(x.hi[c], __shfl_xor(x.hi[c], d, 64));
            x.all_or[c] |= __shfl_xor(x.all_or[c], d, 64);
            x.all_and[c] &= __shfl_xor(x.all_and[c], d, 64);
        }
        x.bad |= __shfl_xor(x.bad, d, 64);
    }
}

template <int NC>
__device__ __forceinline__ void box_empty(Box& x) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        x.lo[c] = INT_MAX;
        x.hi[c] = INT_MIN;
        x.all_or[c] = 0;
        x.all_and[c] = -1;
    }
    x.bad = 0;
}

// field f of box i of `count` boxes at p[f * count + i]
template <int NC>
__device__ __forceinline__ void box_store(const Box& x, int ncol, int32_t* p, int count, int i) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (c >= ncol) break;
        p[(4 * c) * count + i] = x.lo[c];
        p[(4 * c + 1) * count + i] = x.hi[c];
        p[(4 * c + 2) * count + i] = x.all_or[c];
        p[(4 * c + 3) * count + i] = x.all_and[c];
    }
    p[(kBoxInts - 1) * count + i] = x.bad;
}

template <int NC>
__device__ __forceinline__ void box_add(Box& x, int ncol, const int32_t* p, int count, int i) {
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        if (c >= ncol) break;
        x.lo[c] = min(x.lo[c], p[(4 * c) * count + i]);
        x.hi[c] = max(x.hi[c], p[(4 * c + 1) * count + i]);
        x.all_or[c] |= p[(4 * c + 2) * count + i];
        x.all_and[c] &= p[(4 * c + 3) * count + i];
    }
    x.bad |= p[(kBoxInts - 1) * count + i];
}

// Sparse tensor quantization (Sec. 4.1, Alg. 1): the rows are (b, floor(p/v))
// of points, which the box kernel works out and stores (qc) as it reads them.
struct VoxelArg {
    float v[kMaxCols - 1];   // voxel size per spatial axis
};
struct PointsArg {
    const float* points;     // null: no points, the rows are coords
    const int32_t* batch;
    int32_t* qc;
    VoxelArg voxel;
};

// (batch[r] or 0, floor(p_d / v_d)), the floor of the exact quotient of the
// stored float32 values; *bad: a coordinate outside +-2^30.
template <int NC>
__device__ __forceinline__ void quantize_row(const PointsArg& pa, int64_t r, int ncol, int32_t* v, bool* bad_out) {
    const int D = ncol - 1;
    bool bad = false;
    v[0] = pa.batch ? pa.batch[r] : 0;
#pragma unroll
    for (int c = 1; c < NC; ++c) {
        v[c] = 0;
        if (c >= ncol) continue;
        // The quotient rounded to double is at least floor(p / v) (every integer
        // below 2^53 is a double) and at most floor(p / v) + 1; the fma
        // residual p - f v is rounded once, so its sign is that of the exact
        // residual, and a negative one means f overshoots by one.
        const double p = (double)pa.points[r * D + c - 1], w = (double)pa.voxel.v[c - 1];
        double f = floor(p / w);
        if (fma(-f, w, p) < 0.0) f -= 1.0;
        bad = bad || !(f >= -1073741824.0 && f <= 1073741824.0);   // also NaN
        v[c] = bad ? 0 : (int32_t)f;
    }
    *bad_out = *bad_out || bad;
}

// First kernel of a build: the table's header, the words of a grid cleared,
// the row numbers set to row_init, and the box of every block's rows (also
// their common bits: the lowest bit that varies is the column's step).
// Blocks past the first `boxes` only clear.  Bound: the 16 bytes of a row read
// and about 50 cleared.  The blocks' boxes are combined by every block of the
// next kernel; atomics on one box in the header took most of the 11.7 us that
// this kernel's forerunner took at 300,000 rows (12-20 us up to 600,000),
// beside a kernel of 9 us that cleared slots.
template <int NC, bool POINTS>
__global__ void __launch_bounds__(kBoxThreads, NC <= 5 ? 6 : 4) k_box(const int32_t* __restrict__ coords, bool vec, int64_t n, int ncol,
                                                     StrideArg st, PointsArg pa, void* table, int64_t cap, GridLayout g,
                                                     int boxes, int64_t header_n, int32_t row_init) {
    constexpr int W = kBoxThreads / 64;
    __shared__ int32_t sh[kBoxInts * W];
    TableHeader* h = reinterpret_cast<TableHeader*>(table);
    if ((int)blockIdx.x >= boxes) {
        const int64_t i0 = (int64_t)(blockIdx.x - boxes) * kBoxThreads + threadIdx.x,
                      step = (int64_t)(gridDim.x - boxes) * kBoxThreads;
        int4* words = reinterpret_cast<int4*>(grid_words(table));
        for (int64_t i = i0; i < g.word_bytes / 16; i += step) words[i] = int4{0, 0, 0, 0};
        if (g.max_cells > 0 && row_init >= 0) {   // (a table without repeated rows writes every entry)
            int32_t* rowof = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(table) + g.rowof);
            for (int64_t i = i0; i < n; i += step) rowof[i] = row_init;
        }
        return;
    }
    const int64_t first = (int64_t)blockIdx.x * kBoxThreads + threadIdx.x, stride = (int64_t)boxes * kBoxThreads;
    Box x;
    box_empty<NC>(x);
    // a row past the end repeats the thread's first one
    constexpr int B = POINTS ? kBoxRows / 2 : kBoxRows;
    bool bad = false;
    for (int64_t r0 = first; r0 < n; r0 += B * stride) {
        int32_t v[B][NC];
#pragma unroll
        for (int i = 0; i < B; ++i) {
            const int64_t r = r0 + i * stride < n ? r0 + i * stride : r0;
            if constexpr (POINTS) {
                quantize_row<NC>(pa, r, ncol, v[i], &bad);
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (c < ncol) pa.qc[r * ncol + c] = v[i][c];
            } else {
                load_row<NC>(coords, vec, r, ncol, st, v[i], &bad);
            }
        }
#pragma unroll
        for (int i = 0; i < B; ++i) {
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                if (c >= ncol) break;
                x.lo[c] = min(x.lo[c], v[i][c]);
                x.hi[c] = max(x.hi[c], v[i][c]);
                x.all_or[c] |= v[i][c];
                x.all_and[c] &= v[i][c];
            }
        }
    }
    x.bad = bad;
    box_wave<NC>(x, ncol);
    if ((threadIdx.x & 63) == 0) box_store<NC>(x, ncol, sh, W, threadIdx.x >> 6);
    __syncthreads();
    if (threadIdx.x < 64) {
        box_empty<NC>(x);
        if (threadIdx.x < W) box_add<NC>(x, ncol, sh, W, threadIdx.x);
        box_wave<NC>(x, ncol);
        if (threadIdx.x == 0)
            box_store<NC>(x, ncol, reinterpret_cast<int32_t*>(reinterpret_cast<char*>(table) + g.part), boxes,
                          blockIdx.x);
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        h->ncol = ncol;
        h->capacity = cap;
        h->n = header_n;
        h->total = 0;
        h->rowof = (int64_t)g.rowof;
    }
}

__device__ __forceinline__ Slot empty_slot(int32_t val) {
    Slot e;
    e.key = kEmptyKey;
    e.val = val;
    e.hi = kHiUnset;
    return e;
}

// The slots whose memory the box kernel's results take.
struct SlotSpan {
    int64_t first, end;
};
__device__ __forceinline__ SlotSpan part_slots(const GridLayout& g, int parts) {
    const int64_t at = (int64_t)(g.part - kHeaderBytes);
    return SlotSpan{at / (int64_t)sizeof(Slot), (at + (int64_t)parts * kBoxInts * 4 + (int64_t)sizeof(Slot) - 1) / (int64_t)sizeof(Slot)};
}

// The header of a table over no rows (every query misses: lo > hi).
__global__ void __launch_bounds__(kThreads) k_table_empty(TableHeader* h, Slot* slots, int64_t cap, int ncol) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < cap; i += (int64_t)gridDim.x * blockDim.x)
        slots[i] = empty_slot(-1);
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    h->magic = kTableMagic;
    h->ncol = ncol;
    h->capacity = cap;
    h->n = 0;
    h->status = 0;
    h->total_bits = 0;
    for (int c = 0; c < kMaxCols; ++c) {
        h->lo[c] = INT_MAX;
        h->hi[c] = INT_MIN;
        h->shift[c] = h->bits[c] = 0;
    }
    h->nblk = 0;
    for (int i = 0; i < 3; ++i) h->blk_shift[i] = 0;
}

// The box of all rows, in LDS.
struct BoxPlan {
    int32_t lo[kMaxCols], hi[kMaxCols], vary[kMaxCols], step[kMaxCols];
    int32_t bad;
};

// Column c of the box of all rows from that of `count` parts (with column 0 the
// range flag), by one wave: four parts per lane, then the lanes.
__device__ __forceinline__ void box_column(BoxPlan& bp, const int32_t* part, int count, int c) {
    const int lane = threadIdx.x & 63;
    constexpr int B = kBoxBlocks / 64;
    int32_t f[4][B], bad = 0;
#pragma unroll
    for (int i = 0; i < B; ++i) {
        const int at = min(64 * i + lane, count - 1);   // (a repeated part changes nothing)
#pragma unroll
        for (int e = 0; e < 4; ++e) f[e][i] = part[(4 * c + e) * count + at];
        if (c == 0) bad |= part[(kBoxInts - 1) * count + at];   // uniform
    }
    int32_t lo = f[0][0], hi = f[1][0], all_or = f[2][0], all_and = f[3][0];
#pragma unroll
    for (int i = 1; i < B; ++i) {
        lo = min(lo, f[0][i]);
        hi = max(hi, f[1][i]);
        all_or |= f[2][i];
        all_and &= f[3][i];
    }
#pragma unroll
    for (int d = 32; d > 0; d >>= 1) {
        lo = min(lo, __shfl_xor(lo, d, 64));
        hi = max(hi, __shfl_xor(hi, d, 64));
        all_or |= __shfl_xor(all_or, d, 64);
        all_and &= __shfl_xor(all_and, d, 64);
    }
    const bool any = __any(bad != 0);
    if (lane == 0) {
        bp.lo[c] = lo;
        bp.hi[c] = hi;
        bp.vary[c] = all_or ^ all_and;
        bp.step[c] = all_or != all_and ? __ffs(all_or ^ all_and) - 1 : 0;
        if (c == 0) bp.bad = any;
    }
}

// The strides of a grid's cells (the product of the columns after each one),
// and whether the table takes that form.
template <int NC>
__device__ __forceinline__ bool grid_strides(const BoxPlan& bp, int ncol, const GridLayout& g, uint32_t* mul) {
    bool grid = g.max_cells > 0 && !bp.bad;
    int64_t cells = 1;
#pragma unroll
    for (int c = NC - 1; c >= 0; --c) {
        mul[c] = (uint32_t)cells;
        if (c >= ncol) continue;
        const int64_t span = (int64_t)bp.hi[c] - bp.lo[c];
        grid = grid && span < kGridMaxSpan;
        if (grid) cells *= (span >> bp.step[c]) + 1;   // both factors below 2^31
        grid = grid && cells <= g.max_cells;
    }
    return grid;
}

// The header's fields that follow from the box (one thread).
template <int NC>
__device__ __forceinline__ void write_layout(TableHeader* h, const BoxPlan& bp, int ncol, bool grid,
                                             const uint32_t* mul) {
    int total = 0;
    int32_t bits[NC], shift[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        bits[c] = 0;
        if (c >= ncol) continue;
        const int64_t range = (int64_t)bp.hi[c] - bp.lo[c];
        bits[c] = range > 0 ? 64 - __clzll((unsigned long long)range) : 0;
        total += bits[c];
    }
    int sh = 0;
#pragma unroll
    for (int c = NC - 1; c >= 0; --c) {
        shift[c] = sh;
        sh += bits[c];
    }
    int nb = 0;
    int32_t blk[3] = {0, 0, 0};
#pragma unroll
    for (int c = 0; c < kMaxCols; ++c) {
        const bool in = c < NC && c < ncol;
        const int cc = c < NC ? c : 0;
        h->lo[c] = in ? bp.lo[c] : INT_MAX;
        h->hi[c] = in ? bp.hi[c] : INT_MIN;
        h->shift[c] = in ? shift[cc] : 0;
        h->bits[c] = in ? bits[cc] : 0;
        h->step[c] = in ? (int8_t)bp.step[c] : 0;
        h->cstride[c] = in ? mul[cc] : 0;
        // the lowest varying key bit of the first three spatial columns that vary (see home_slot)
        if (c > 0 && in && bp.vary[c] && bp.step[c] < bits[cc]) {
#pragma unroll
            for (int i = 0; i < 3; ++i)
                if (nb == i) blk[i] = shift[cc] + bp.step[c];
            nb = nb < 3 ? nb + 1 : 3;
        }
    }
    for (int i = 0; i < 3; ++i) h->blk_shift[i] = blk[i];
    h->nblk = nb;
    h->total_bits = total;
    h->status = total > kMaxKeyBits || bp.bad ? ST_RANGE : 0;
    h->magic = grid ? kGridMagic : kTableMagic;
}

// Rows of which many may share a cell (points, coarse strides): what a block's
// rows do to one word or place is combined in LDS first, so that the block sends
// one atomic for it.  Atomics on one address take about 13 ns each, one after
// another, and a hot cell (a sensor's surroundings) has thousands of rows.  The
// larger the block the better (300,000 points around one spot, quantization in
// us: each row by itself 305, blocks of 256 242, of 512 218, of 1024 185), but
// few rows then leave CUs idle (14,490 points: 1024 106.9, 256 103.7).
constexpr int kMergeThreads = 1024, kMergeFew = 256;
constexpr int64_t kMergeMany = 65536;   // rows from which blocks of kMergeThreads take them
// A stride whose cells hold at most this many rows merges only the runs of
// equal words in a wave: 300,082 sorted 3D rows at stride 2 (8 a cell) 42 us
// against 52, at stride 4 (64) 40 against 45; at stride 16 52 us against 39, the
// same rows shuffled 150 against 99; 121,239 4D rows at stride 4 (256) 35.3
// against 34.4, 100,000 7D rows at stride 2 (128; hashed) 59.8 against 62.2.
constexpr int64_t kMergeCell = 128;

template <int TB>
struct MergeTable {
    static constexpr int kBits = TB == 1024 ? 11 : 9, kSlots = 1 << kBits;
    static_assert(kSlots == 2 * TB, "two slots per row");
    uint32_t key[kSlots], val[kSlots];
    __device__ __forceinline__ void clear(uint32_t v) {   // then a barrier
#pragma unroll
        for (int i = threadIdx.x; i < kSlots; i += TB) {
            key[i] = ~0u;
            val[i] = v;
        }
    }
    // the entry of k, null when another key has taken its place
    __device__ __forceinline__ uint32_t* entry(uint32_t k) {
        const uint32_t s = (k * 0x9e3779b1u) >> (32 - kBits);
        const uint32_t prev = atomicCAS(&key[s], ~0u, k);
        return prev == ~0u || prev == k ? &val[s] : nullptr;
    }
};

// Second kernel of a build: every block combines the boxes of the first one's
// blocks and decides the table's form; block 0 writes the header.  A grid:
// each row sets the bit of its cell, rows of a wave that share a word
// (neighbours of a sorted row list) in one atomic.
template <int NC, int MERGE>
__global__ void __launch_bounds__(MERGE > 0 ? MERGE : kThreads)
k_mark(const int32_t* __restrict__ coords, bool vec, int64_t n, int ncol, StrideArg st, void* table, int64_t cap,
       GridLayout g, int parts, int32_t init_val) {
    constexpr int TB = MERGE > 0 ? MERGE : kThreads;
    __shared__ BoxPlan bp;
    TableHeader* h = reinterpret_cast<TableHeader*>(table);
    const int64_t r = xcd_unit(blockIdx.x, gridDim.x) * TB + threadIdx.x;
    MergeTable<TB>* merge = nullptr;
    if constexpr (MERGE > 0) {
        __shared__ MergeTable<TB> sh;
        merge = &sh;
        merge->clear(0u);
    }
    int32_t v[NC];
    bool unused = false;   // the box kernel has found values outside int32
    load_row<NC>(coords, vec, r < n ? r : 0, ncol, st, v, &unused);   // in flight during the box
    const int32_t* part = reinterpret_cast<const int32_t*>(reinterpret_cast<const char*>(table) + g.part);
    for (int c = threadIdx.x >> 6; c < ncol; c += TB / 64) box_column(bp, part, parts, c);   // a wave per column
    __syncthreads();
    uint32_t mul[NC];
    const bool grid = grid_strides<NC>(bp, ncol, g, mul);
    if (blockIdx.x == 0 && threadIdx.x == 0) write_layout<NC>(h, bp, ncol, grid, mul);
    if (!grid) {   // empty slots, but for those that hold the boxes, which other blocks may still read
        const SlotSpan p = part_slots(g, parts);
        Slot* slots = table_slots(table);
        for (int64_t i = (int64_t)blockIdx.x * TB + threadIdx.x; i < cap; i += (int64_t)gridDim.x * TB)
            if (i < p.first || i >= p.end) slots[i] = empty_slot(init_val);
        return;
    }
    uint32_t word = ~0u, bits = 0;
    if (r < n) {
        uint32_t cell = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (c < ncol) cell += ((uint32_t)(v[c] - bp.lo[c]) >> bp.step[c]) * mul[c];
        word = cell >> 5;
        bits = 1u << (cell & 31);
    }
    // the bits of a run of lanes with the same word, collected in its first lane
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t ow = __shfl_down(word, d, 64), ob = __shfl_down(bits, d, 64);
        if ((int)(threadIdx.x & 63) + d < 64 && ow == word) bits |= ob;
    }
    const uint32_t pw = __shfl_up(word, 1, 64);
    const bool first = r < n && ((threadIdx.x & 63) == 0 || pw != word);
    if constexpr (MERGE > 0) {
        if (first) {
            uint32_t* e = merge->entry(word);
            atomicOr(e ? e : &grid_words(table)[word].bits, bits);
        }
        __syncthreads();
#pragma unroll
        for (int i = threadIdx.x; i < merge->kSlots; i += TB)
            if (merge->key[i] != ~0u) atomicOr(&grid_words(table)[merge->key[i]].bits, merge->val[i]);
    } else {
        if (first) atomicOr(&grid_words(table)[word].bits, bits);
    }
}

// Third kernel.  A grid: the row numbers' places.  A block takes a share of
// the words, adds up their occupied cells and claims that many places with
// one atomic; a word's `before` is its block's start plus the cells of the
// block's words before it (the order of the blocks is arbitrary and seen by
// nobody: a place only has to be the word's own).  A hash: the empty slots
// that the second kernel left out.
constexpr int kIndexThreads = 1024;
constexpr int kIndexWords = 6;
static_assert(kIndexWords * 32 >= kGridCells, "a thread per row takes all words of more than kSmallRows rows");

__global__ void __launch_bounds__(kIndexThreads) k_index(void* table, GridLayout g, int parts,
                                                         int32_t init_val) {
    TableHeader* h = reinterpret_cast<TableHeader*>(table);
    const int64_t first = (int64_t)blockIdx.x * kIndexThreads + threadIdx.x,
                  stride = (int64_t)gridDim.x * kIndexThreads;
    if (h->magic != kGridMagic) {   // uniform
        const SlotSpan p = part_slots(g, parts);
        for (int64_t i = p.first + first; i < p.end; i += stride) table_slots(table)[i] = empty_slot(init_val);
        return;
    }
    __shared__ uint32_t wsum[kIndexThreads / 64];
    __shared__ uint32_t base_sh;
    GridWord* words = grid_words(table);
    const int64_t range0 = (int64_t)h->hi[0] - h->lo[0];
    const int64_t cells = ((range0 >> h->step[0]) + 1) * (int64_t)h->cstride[0];
    const int64_t nw = (cells + 31) / 32;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    // kIndexWords words per thread, in registers
    const int64_t i0 = (int64_t)blockIdx.x * kIndexThreads;
    if (i0 >= nw) return;   // uniform
    uint32_t bits[kIndexWords];
    uint32_t sum = 0;
#pragma unroll
    for (int u = 0; u < kIndexWords; ++u) {
        const int64_t i = i0 + u * stride + threadIdx.x;
        bits[u] = i < nw ? words[i].bits : 0u;
    }
#pragma unroll
    for (int u = 0; u < kIndexWords; ++u) sum += (uint32_t)__popc(bits[u]);
    uint32_t inc = sum;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t u = __shfl_up(inc, d, 64);
        if (lane >= d) inc += u;
    }
    if (lane == 63) wsum[wave] = inc;
    __syncthreads();
    uint32_t before = 0, all = 0;
    for (int i = 0; i < kIndexThreads / 64; ++i) {
        if (i < wave) before += wsum[i];
        all += wsum[i];
    }
    if (threadIdx.x == 0) base_sh = all ? atomicAdd(&h->total, all) : 0u;
    __syncthreads();
    uint32_t run = base_sh + before + inc - sum;
#pragma unroll
    for (int u = 0; u < kIndexWords; ++u) {
        if (bits[u]) words[i0 + u * stride + threadIdx.x].before = run;   // (an empty word's is never read)
        run += (uint32_t)__popc(bits[u]);
    }
}

// Wide keys: the CAS claims a slot by the key's low 62 bits and the claiming
// thread then writes the high bits into Slot::hi.  A thread that meets the
// same low bits reads Slot::hi, and while it is still unset it polls the same
// slot again: the writer has claimed it and stores right after.  The claim's
// store comes before any comparison in every round, so a writer in the same
// wave has stored before its neighbours look.  The probing ends when the key
// is placed or found or the table has been walked through; a slot whose high
// bits stay unset past kWidePolls polls ends it with ST_FULL.
constexpr int kWidePolls = 1 << 22;

// One round of a wide find-or-insert at slot s: returns 1 placed (this thread
// claimed the slot), 2 found (the slot holds the key), 3 retry the same slot,
// 0 move on.
__device__ __forceinline__ int wide_round(Slot* slots, unsigned long long s, unsigned long long lo, int32_t hi) {
    const unsigned long long prev = atomicCAS(&slots[s].key, kEmptyKey, lo);
    const bool won = prev == kEmptyKey;
    if (won) __hip_atomic_store(&slots[s].hi, hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
    if (won) return 1;
    if (prev != lo) return 0;
    const int32_t h2 = __hip_atomic_load(&slots[s].hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return h2 == kHiUnset ? 3 : (h2 == hi ? 2 : 0);
}

// Hash: the slot that holds the row's key, claimed if none did: 1 claimed,
// 2 found, 0 none free (or a key outside the box, which cannot happen).
template <int NC>
__device__ __forceinline__ int find_or_insert(const TableView& tv, const int32_t* v, int total_bits, TableHeader* h,
                                              Slot* slots, unsigned long long* slot) {
    const unsigned long long mask = tv.sh.mask;
    if (total_bits > kNarrowKeyBits) {   // uniform
        u128 key;
        if (!pack_key_wide<NC>(tv, v, &key)) {
            atomicOr(&h->status, ST_RANGE);
            return 0;
        }
        const unsigned long long lo = wide_lo(key);
        const int32_t hi = wide_hi(key);
        unsigned long long s = home_slot_wide(tv.sh, key);
        int polls = 0;
        for (unsigned long long i = 0; i <= mask;) {
            const int res = wide_round(slots, s, lo, hi);
            if (res == 1 || res == 2) {
                *slot = s;
                return res;
            }
            if (res == 3) {
                if (++polls > kWidePolls) break;
                continue;
            }
            s = (s + 1) & mask;
            ++i;
        }
        atomicOr(&h->status, ST_FULL);
        return 0;
    }
    unsigned long long key;
    if (!pack_key<NC>(tv, v, &key)) {
        atomicOr(&h->status, ST_RANGE);
        return 0;
    }
    unsigned long long s = home_slot(tv.sh, key);
    for (unsigned long long i = 0; i <= mask; ++i) {
        const unsigned long long prev = atomicCAS(&slots[s].key, kEmptyKey, key);
        if (prev == kEmptyKey || prev == key) {
            *slot = s;
            return prev == key ? 2 : 1;
        }
        s = (s + 1) & mask;
    }
    atomicOr(&h->status, ST_FULL);
    return 0;
}

// The row number that a table keeps at place s: a slot of a hash, an entry of
// a grid's row numbers.
__device__ __forceinline__ int32_t* row_number(void* table, bool grid, const TableHeader* h, unsigned long long s) {
    return grid ? reinterpret_cast<int32_t*>(reinterpret_cast<char*>(table) + h->rowof) + s
                : &table_slots(table)[s].val;
}

// Fourth kernel: every row's number into the table.  MIN (strided and
// quantized rows, which repeat): the smallest row of each key stays, and the
// place of every row is kept in slot_of.  Rows of a wave are consecutive, so
// rows with the same key are often neighbouring lanes: only the first lane of
// each run of equal keys updates the place (its row is the run's smallest)
// and, in a hash, inserts; the others take its place by a shuffle.
template <int NC, bool MIN, int MERGE>
__global__ void __launch_bounds__(MERGE > 0 ? MERGE : kThreads)
k_place(const int32_t* __restrict__ coords, bool vec, int64_t n, int ncol, StrideArg st, void* table,
        int64_t* __restrict__ slot_of) {
    constexpr int TB = MERGE > 0 ? MERGE : kThreads;
    TableHeader* h = reinterpret_cast<TableHeader*>(table);
    const int64_t r = xcd_unit(blockIdx.x, gridDim.x) * TB + threadIdx.x;
    const bool valid = r < n;
    const bool grid = h->magic == kGridMagic;   // uniform
    if (h->status & ST_RANGE) {                 // uniform (set before this kernel)
        if (MIN && valid) slot_of[r] = 0;
        return;
    }
    int32_t v[NC];
    bool unused = false;
    load_row<NC>(coords, vec, valid ? r : 0, ncol, st, v, &unused);
    const int lane = threadIdx.x & 63;
    if (grid) {
        uint32_t cell = 0;
#pragma unroll
        for (int c = 0; c < NC; ++c)
            if (c < ncol) cell += ((uint32_t)(v[c] - h->lo[c]) >> h->step[c]) * h->cstride[c];
        const uint32_t place = grid_place(grid_words(table)[cell >> 5], cell);
        int32_t* rowof = row_number(table, true, h, 0);
        if (!MIN) {
            if (valid) rowof[place] = (int32_t)r;
            // fewer cells than rows: a row occurs twice
            if (blockIdx.x == 0 && threadIdx.x == 0 && h->total != (uint32_t)n) atomicOr(&h->status, ST_DUP);
            return;
        }
        const uint32_t prev = __shfl_up(place, 1, 64);
        if constexpr (MERGE > 0) {   // (all of the block's rows come here)
            __shared__ MergeTable<TB> merge;
            merge.clear(INT_MAX);
            __syncthreads();
            if (valid && (lane == 0 || prev != place)) {
                uint32_t* e = merge.entry(place);
                if (e) atomicMin(e, (uint32_t)r);
                else atomicMin(&rowof[place], (int32_t)r);
            }
            if (valid) slot_of[r] = (int64_t)place;
            __syncthreads();
#pragma unroll
            for (int i = threadIdx.x; i < merge.kSlots; i += TB)
                if (merge.key[i] != ~0u) atomicMin(&rowof[merge.key[i]], (int32_t)merge.val[i]);
        } else {
            if (valid && (lane == 0 || prev != place)) atomicMin(&rowof[place], (int32_t)r);
            if (valid) slot_of[r] = (int64_t)place;
        }
        return;
    }
    const TableView tv = table_view(h, ncol);
    Slot* slots = table_slots(table);
    const int total_bits = h->total_bits;
    unsigned long long s = 0;
    if (!MIN) {
        if (!valid) return;
        const int res = find_or_insert<NC>(tv, v, total_bits, h, slots, &s);
        if (res == 1) slots[s].val = (int32_t)r;
        if (res == 2) atomicOr(&h->status, ST_DUP);
        return;
    }
    bool follower = valid && lane > 0;
#pragma unroll
    for (int c = 0; c < NC; ++c) follower = (__shfl_up(v[c], 1, 64) == v[c]) && follower;
    const unsigned long long leaders = __ballot(valid && !follower);
    if (valid && !follower && find_or_insert<NC>(tv, v, total_bits, h, slots, &s)) atomicMin(&slots[s].val, (int32_t)r);
    // a follower's run starts at the highest leader lane at or below it
    const unsigned long long upto = lane == 63 ? ~0ull : ((2ull << lane) - 1ull);
    const unsigned long long lm = leaders & upto;
    const int ld = lm ? 63 - __clzll(lm) : lane;
    const unsigned long long ls = __shfl(s, ld, 64);
    if (valid) slot_of[r] = (int64_t)ls;
}

// mark representatives (the place holds this row) and count them per 64-row group
__global__ void __launch_bounds__(kThreads) k_rep_count(int64_t n, void* table, int64_t* slot_of, int32_t* cnt) {
    const TableHeader* h = reinterpret_cast<const TableHeader*>(table);
    const int64_t r = xcd_unit(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    bool rep = false;
    if (r < n && h->status == 0) {
        const int64_t s = slot_of[r];
        rep = *row_number(table, h->magic == kGridMagic, h, (unsigned long long)s) == (int32_t)r;
        if (rep) slot_of[r] = ~s;   // negative: representative
    }
    const unsigned long long m = __ballot(rep);
    const int64_t g = r >> 6;
    if (__lane_id() == 0 && g * 64 < n) cnt[g] = __popcll(m);
}

// The representatives become the output rows, in row order: their coordinates,
// their numbers in the table, and (quantization) their input rows and labels.
template <int NC>
__global__ void __launch_bounds__(kThreads) k_rep_write(const int32_t* __restrict__ coords, bool vec, int64_t n,
                                                        int ncol, StrideArg st, void* table, const int64_t* slot_of,
                                                        const int64_t* off, int32_t* __restrict__ out_coords,
                                                        int32_t* __restrict__ rep_row,
                                                        const int32_t* __restrict__ labels,
                                                        int32_t* __restrict__ out_labels) {
    const TableHeader* h = reinterpret_cast<const TableHeader*>(table);
    const int64_t r = xcd_unit(blockIdx.x, gridDim.x) * blockDim.x + threadIdx.x;
    bool rep = false;
    int64_t s = 0;
    if (r < n && h->status == 0) {
        s = slot_of[r];
        rep = s < 0;
        s = ~s;
    }
    const unsigned long long m = __ballot(rep);
    if (!rep) return;
    const int64_t row = off[r >> 6] + __popcll(m & lanemask_lt());
    int32_t v[NC];
    bool unused = false;
    load_row<NC>(coords, vec, r, ncol, st, v, &unused);
#pragma unroll
    for (int c = 0; c < NC; ++c)
        if (c < ncol) out_coords[row * ncol + c] = v[c];
    *row_number(table, h->magic == kGridMagic, h, (unsigned long long)s) = (int32_t)row;
    if (rep_row) rep_row[row] = (int32_t)r;
    if (out_labels) out_labels[row] = labels[r];
}

// Quantization: the voxel of every point (inverse), and ignore_label for a
// voxel of which a point has another label than its first one (f of Alg. 1;
// every writer of a voxel's label here stores the same value).
__global__ void __launch_bounds__(kThreads) k_quant_labels(int64_t n, void* table,
                                                           const int64_t* __restrict__ slot_of,
                                                           const int32_t* __restrict__ rep,
                                                           const int32_t* __restrict__ labels,
                                                           int32_t ignore_label, int32_t* __restrict__ inverse,
                                                           int32_t* __restrict__ out_labels) {
    const TableHeader* h = reinterpret_cast<const TableHeader*>(table);
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n || h->status != 0) return;
    int64_t sl = slot_of[r];
    if (sl < 0) sl = ~sl;   // a representative
    const int32_t o = *row_number(table, h->magic == kGridMagic, h, (unsigned long long)sl);
    if (o < 0 || o >= n) return;
    if (inverse) inverse[r] = o;
    if (out_labels && labels[r] != labels[rep[o]]) out_labels[o] = ignore_label;
}

// out[i] = labels[i] for the table's rows.
__global__ void __launch_bounds__(kThreads) k_copy_labels(const void* table, int64_t n,
                                                          const int32_t* __restrict__ labels,
                                                          int32_t* __restrict__ out) {
    const TableHeader* h = reinterpret_cast<const TableHeader*>(table);
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n && i < h->n && h->status == 0) out[i] = labels[i];
}

// ---------------------------------------------------------------------------
// Few rows: the whole build in one block
// ---------------------------------------------------------------------------
// Up to kSmallRows rows, the steps above by one block whose grid words, row
// numbers and output numbers lie in LDS; MIN also numbers the distinct keys
// and writes the output rows (as k_rep_count to k_quant_labels do).  A hash is
// claimed in LDS too: a slot's claim is the row that took it, compared by the
// rows' keys, and the slots are written once at the end (inserted in global
// memory, one block's chain of compare-and-swaps made a build of 2,000 rows 25
// us with narrow keys and 62 with wide ones; here 15 and 28).
// Bound: latency.  At 2,000 rows the launches of the separate kernels take 4 to
// 7 us each, one after another: a build four of them, a strided one seven, a
// quantization eight.
struct SmallOut {   // MIN
    int32_t *out_coords, *rep_row, *inverse, *out_labels;
    const int32_t* labels;
    int32_t ignore_label;
};

template <int NC, bool MIN, bool POINTS>
__global__ void __launch_bounds__(kSmallThreads) k_small(const int32_t* __restrict__ coords, bool vec, int n, int ncol,
                                                         StrideArg st, PointsArg pa, void* table, int64_t cap,
                                                         GridLayout g, int64_t header_n, SmallOut out) {
    constexpr int W = kSmallThreads / 64;
    __shared__ BoxPlan bp;
    __shared__ TableHeader hs;
    __shared__ int32_t sh[kBoxInts * W];
    // a grid: its words; a hash: the slots' claims (kNoClaim or a row), the rows' keys
    constexpr int kWordMem = kSmallWords * (int)(sizeof(uint32_t) + sizeof(uint16_t));
    constexpr int kClaimMem = kSmallSlots * (int)sizeof(uint32_t);
    constexpr int kKeyMem = kSmallRows * (int)(sizeof(unsigned long long) + sizeof(int32_t));
    __shared__ __attribute__((aligned(16))) unsigned char mem[kWordMem > kClaimMem + kKeyMem ? kWordMem : kClaimMem + kKeyMem];
    uint32_t* const bits = reinterpret_cast<uint32_t*>(mem);
    uint16_t* const before = reinterpret_cast<uint16_t*>(mem + kSmallWords * sizeof(uint32_t));
    uint32_t* const claim = reinterpret_cast<uint32_t*>(mem);
    unsigned long long* const klo = reinterpret_cast<unsigned long long*>(mem + kClaimMem);
    int32_t* const khi = reinterpret_cast<int32_t*>(mem + kClaimMem + kSmallRows * sizeof(unsigned long long));
    constexpr uint32_t kNoClaim = ~0u;
    __shared__ int32_t first[kSmallRows];    // a grid's row numbers; a hash: the smallest row of a claim's key
    __shared__ int32_t number[kSmallRows];   // output row of a representative, by its input row
    __shared__ uint8_t differs[MIN ? kSmallRows : 1];
    __shared__ int32_t wsum[W * kSmallPer];
    __shared__ int32_t failed;               // ST_DUP, ST_FULL
    TableHeader* h = reinterpret_cast<TableHeader*>(table);
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    int32_t v[kSmallPer][NC];
    Box x;
    box_empty<NC>(x);
    bool bad = false;
#pragma unroll
    for (int i = 0; i < kSmallPer; ++i) {
        const int r = min(i * kSmallThreads + t, n - 1);   // a row past the end repeats the last one
        if constexpr (POINTS) quantize_row<NC>(pa, r, ncol, v[i], &bad);
        else load_row<NC>(coords, vec, r, ncol, st, v[i], &bad);
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            if (c >= ncol) break;
            x.lo[c] = min(x.lo[c], v[i][c]);
            x.hi[c] = max(x.hi[c], v[i][c]);
            x.all_or[c] |= v[i][c];
            x.all_and[c] &= v[i][c];
        }
    }
    x.bad = bad;
    box_wave<NC>(x, ncol);
    if (lane == 0) box_store<NC>(x, ncol, sh, W, wave);
    __syncthreads();
    for (int c = wave; c < ncol; c += W) box_column(bp, sh, W, c);
    __syncthreads();
    uint32_t mul[NC];
    const bool grid = grid_strides<NC>(bp, ncol, g, mul);   // (max_cells fits the words in LDS)
    if (t == 0) {   // the header; the table's copy is written when total and status are known
        hs.ncol = ncol;
        hs.capacity = cap;
        hs.n = header_n;
        hs.total = 0;
        hs.rowof = (int64_t)g.rowof;
        write_layout<NC>(&hs, bp, ncol, grid, mul);
        if (bp.bad) *h = hs;
    }
    if (bp.bad) return;
    int32_t place[kSmallPer], fst[kSmallPer];
    Slot* slots = table_slots(table);
    int32_t* rowof = reinterpret_cast<int32_t*>(reinterpret_cast<char*>(table) + g.rowof);
    if (grid) {
        const int64_t span0 = (int64_t)bp.hi[0] - bp.lo[0];
        const int nw = (int)((((span0 >> bp.step[0]) + 1) * (int64_t)mul[0] + 31) / 32);
        for (int i = t; i < nw; i += kSmallThreads) bits[i] = 0;
        for (int i = t; i < n; i += kSmallThreads) first[i] = INT_MAX;
        __syncthreads();
        uint32_t cell[kSmallPer];
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            cell[i] = 0;
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (c < ncol) cell[i] += ((uint32_t)(v[i][c] - bp.lo[c]) >> bp.step[c]) * mul[c];
            if (i * kSmallThreads + t < n) atomicOr(&bits[cell[i] >> 5], 1u << (cell[i] & 31));
        }
        __syncthreads();
        // a thread's share of the words is contiguous here: an odd number of words, so that the lanes' reads
        // spread over the banks
        const int per = ((nw + kSmallThreads - 1) / kSmallThreads) | 1;
        const int w0 = min(t * per, nw), w1 = min(w0 + per, nw);
        uint32_t sum = 0;
        for (int i = w0; i < w1; ++i) sum += (uint32_t)__popc(bits[i]);
        uint32_t inc = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t u = __shfl_up(inc, d, 64);
            if (lane >= d) inc += u;
        }
        if (lane == 63) wsum[wave] = (int32_t)inc;
        __syncthreads();
        uint32_t run = inc - sum, total = 0;
        for (int i = 0; i < W; ++i) {
            if (i < wave) run += (uint32_t)wsum[i];
            total += (uint32_t)wsum[i];
        }
        for (int i = w0; i < w1; ++i) {
            before[i] = (uint16_t)run;
            run += (uint32_t)__popc(bits[i]);
        }
        if (t == 0) {
            hs.total = total;
            if (!MIN && total != (uint32_t)n) hs.status |= ST_DUP;   // fewer cells than rows: a row occurs twice
            *h = hs;
        }
        __syncthreads();
        GridWord* words = grid_words(table);
        for (int i = t; i < nw; i += kSmallThreads) words[i] = GridWord{bits[i], before[i]};
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int r = i * kSmallThreads + t;
            const uint32_t w = cell[i] >> 5;
            place[i] = (int32_t)grid_place(GridWord{bits[w], before[w]}, cell[i]);
            if (r < n) atomicMin(&first[place[i]], r);
        }
        __syncthreads();
        if (!MIN) {
            for (int i = t; i < (int)total; i += kSmallThreads) rowof[i] = first[i];
            return;
        }
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) fst[i] = first[place[i]];
    } else {
        for (int i = t; i < (int)cap; i += kSmallThreads) claim[i] = kNoClaim;
        for (int i = t; i < n; i += kSmallThreads) first[i] = INT_MAX;
        if (t == 0) failed = 0;
        __syncthreads();
        if (hs.status & ST_RANGE) {   // uniform: set by write_layout only
            if (t == 0) *h = hs;
            return;
        }
        const TableView tv = table_view(&hs, ncol);
        const bool wide = hs.total_bits > kNarrowKeyBits;   // uniform
        uint32_t home[kSmallPer];
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int r = i * kSmallThreads + t;
            if (r >= n) continue;
            if (wide) {   // (a key outside the box cannot happen)
                u128 key;
                pack_key_wide<NC>(tv, v[i], &key);
                klo[r] = wide_lo(key);
                khi[r] = wide_hi(key);
                home[i] = (uint32_t)home_slot_wide(tv.sh, key);
            } else {
                unsigned long long key;
                pack_key<NC>(tv, v[i], &key);
                klo[r] = key;
                khi[r] = kHiUnset;
                home[i] = (uint32_t)home_slot(tv.sh, key);
            }
        }
        __syncthreads();
        const uint32_t mask = (uint32_t)cap - 1u;
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int r = i * kSmallThreads + t;
            place[i] = 0;
            if (r >= n) continue;
            const unsigned long long lo = klo[r];
            const int32_t hi = khi[r];
            uint32_t s = home[i], owner = kNoClaim;
            for (uint32_t step = 0; step <= mask; ++step, s = (s + 1) & mask) {
                const uint32_t prev = atomicCAS(&claim[s], kNoClaim, (uint32_t)r);
                if (prev == kNoClaim || (klo[prev] == lo && khi[prev] == hi)) {
                    owner = prev == kNoClaim ? (uint32_t)r : prev;
                    break;
                }
            }
            if (owner == kNoClaim) atomicOr(&failed, ST_FULL);
            else if (MIN) atomicMin(&first[owner], r);
            else if (owner != (uint32_t)r) atomicOr(&failed, ST_DUP);
            if (owner != kNoClaim) place[i] = (int32_t)owner;
        }
        __syncthreads();
        if (t == 0) {
            hs.status |= failed;
            *h = hs;
        }
        if (!MIN) {
            for (int i = t; i < (int)cap; i += kSmallThreads) {
                const uint32_t c = claim[i];
                slots[i] = c == kNoClaim ? empty_slot(-1) : Slot{klo[c], (int32_t)c, khi[c]};
            }
            return;
        }
        if (failed) return;   // full
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) fst[i] = first[place[i]];
    }
    if constexpr (MIN) {
        // number the representatives (the first row of each key) in row order
        unsigned long long rep[kSmallPer];
        int32_t label[kSmallPer];   // read before any is written: out_labels may be the labels' array
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int r = i * kSmallThreads + t;
            rep[i] = __ballot(r < n && fst[i] == r);
            if (lane == 0) wsum[i * W + wave] = (int32_t)__popcll(rep[i]);
            if (r < n) differs[r] = 0;
        }
        __syncthreads();
        int32_t base[kSmallPer], n_out = 0;
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i)
            for (int w = 0; w < W; ++w) {
                if (w == wave) base[i] = n_out;
                n_out += wsum[i * W + w];
            }
        if (t == 0) h->n = n_out;
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int r = i * kSmallThreads + t;
            if (r >= n) continue;
            if (out.out_labels) label[i] = out.labels[r];
            if (fst[i] == r) number[r] = base[i] + (int32_t)__popcll(rep[i] & lanemask_lt());
            // a point with another label than the voxel's first one (every writer stores the same)
            else if (out.out_labels && label[i] != out.labels[fst[i]]) differs[fst[i]] = 1;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kSmallPer; ++i) {
            const int r = i * kSmallThreads + t;
            if (r >= n) continue;
            const int32_t o = number[fst[i]];
            if (out.inverse) out.inverse[r] = o;
            if (fst[i] != r) continue;
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (c < ncol) out.out_coords[(int64_t)o * ncol + c] = v[i][c];
            if (grid) rowof[place[i]] = o;
            if (out.rep_row) out.rep_row[o] = r;
            if (out.out_labels) out.out_labels[o] = differs[r] ? out.ignore_label : label[i];
        }
        if (grid) return;
        for (int i = t; i < (int)cap; i += kSmallThreads) {
            const uint32_t c = claim[i];
            slots[i] = c == kNoClaim ? empty_slot(INT_MAX) : Slot{klo[c], number[first[c]], khi[c]};
        }
    }
}

static unsigned grid_for(int64_t n, int per = kThreads) {
    int64_t g = (n + per - 1) / per;
    if (g < 1) g = 1;
    return (unsigned)g;
}

// rows that load as whole 16-byte words
static bool rows_vec(const int32_t* coords, int ncol) {
    return (ncol == 4 || ncol == 8) && ((uintptr_t)coords & 15) == 0;
}

static int read_status(const void* table, hipStream_t s, TableHeader* out) {
    GSC_HIP(hipMemcpyAsync(out, table, sizeof(TableHeader), hipMemcpyDeviceToHost, s));
    GSC_HIP(hipStreamSynchronize(s));
    return GSC_OK;
}

static int status_to_code(const TableHeader& h, const char* what) {
    if (h.status & ST_RANGE)
        return fail(GSC_ERANGE, "%s: coordinates need more than %d key bits (box needs %d)", what, kMaxKeyBits,
                    h.total_bits);
    if (h.status & ST_DUP) return fail(GSC_EDUP, "%s: a coordinate row occurs more than once", what);
    if (h.status & ST_FULL) return fail(GSC_EFULL, "%s: hash table full", what);
    return GSC_OK;
}

// The table of no rows.
static int empty_enqueue(int ncol, void* table, hipStream_t s) {
    const int64_t cap = table_capacity(0);
    hipLaunchKernelGGL(k_table_empty, dim3(1), dim3(kThreads), 0, s, reinterpret_cast<TableHeader*>(table),
                       table_slots(table), cap, ncol);
    GSC_LAUNCH_CHECK();
    return GSC_OK;
}

// The kernels that build a table over n > 0 rows: one for few rows (with MIN,
// rows that may repeat, it writes the results in `out` too), else four (with
// MIN, the places of all rows in slot_of, and reps_enqueue follows); with pa.points the rows are
// the quantized points, stored in pa.qc (= coords) on the way.
template <int NC, bool MIN>
static int table_enqueue_nc(const int32_t* coords, int64_t n, int ncol, const StrideArg& st, const PointsArg& pa,
                            void* table, int64_t header_n, int64_t* slot_of, const SmallOut& out, hipStream_t s) {
    const int64_t cap = table_capacity(n);
    const GridLayout g = grid_layout(n, cap);
    const bool vec = rows_vec(coords, ncol);
    if (n <= kSmallRows) {
        auto* small = MIN && pa.points ? k_small<NC, MIN, MIN> : k_small<NC, MIN, false>;
        hipLaunchKernelGGL(small, dim3(1), dim3(kSmallThreads), 0, s, coords, vec, (int)n, ncol, st, pa, table, cap, g,
                           header_n, out);
        GSC_LAUNCH_CHECK();
        return GSC_OK;
    }
    const int32_t init = MIN ? (int32_t)INT_MAX : -1;
    const int boxes = box_blocks(n, cap);
    // the words are cleared by blocks of their own (64 bytes a thread)
    const int64_t clear = std::min<int64_t>(g.word_bytes / (64 * kBoxThreads) + 1, 2048);
    auto* box = MIN && pa.points ? k_box<NC, MIN> : k_box<NC, false>;   // points only come with MIN
    hipLaunchKernelGGL(box, dim3((unsigned)(boxes + clear)), dim3(kBoxThreads), 0, s, coords, vec, n, ncol, st,
                       pa, table, cap, g, boxes, header_n, init);
    GSC_LAUNCH_CHECK();
    bool merge = MIN && pa.points;
    for (int64_t c = 1, cell = 1; MIN && c < ncol && !merge; ++c) merge = (cell *= st.s[c]) > kMergeCell;
    const bool large = n >= kMergeMany;
    const int tb = !merge ? kThreads : (large ? kMergeThreads : kMergeFew);
    auto* mark = k_mark<NC, 0>;
    auto* place = k_place<NC, MIN, 0>;
    if constexpr (MIN) {
        if (merge) mark = large ? k_mark<NC, kMergeThreads> : k_mark<NC, kMergeFew>;
        if (merge) place = large ? k_place<NC, MIN, kMergeThreads> : k_place<NC, MIN, kMergeFew>;
    }
    hipLaunchKernelGGL(mark, dim3(grid_for(n, tb)), dim3(tb), 0, s, coords, vec, n, ncol, st, table, cap, g, boxes, init);
    GSC_LAUNCH_CHECK();
    hipLaunchKernelGGL(k_index, dim3(grid_for(n, kIndexThreads)), dim3(kIndexThreads), 0, s, table, g, boxes, init);
    GSC_LAUNCH_CHECK();
    hipLaunchKernelGGL(place, dim3(grid_for(n, tb)), dim3(tb), 0, s, coords, vec, n, ncol, st, table, slot_of);
    GSC_LAUNCH_CHECK();
    return GSC_OK;
}

template <bool MIN>
static int table_enqueue(const int32_t* coords, int64_t n, int ncol, const StrideArg& st, const PointsArg& pa,
                         void* table, int64_t header_n, int64_t* slot_of, const SmallOut& out, hipStream_t s) {
    switch (ncol) {   // 3D and 4D rows with the columns unrolled
        case 4: return table_enqueue_nc<4, MIN>(coords, n, ncol, st, pa, table, header_n, slot_of, out, s);
        case 5: return table_enqueue_nc<5, MIN>(coords, n, ncol, st, pa, table, header_n, slot_of, out, s);
        default: return table_enqueue_nc<kMaxCols, MIN>(coords, n, ncol, st, pa, table, header_n, slot_of, out, s);
    }
}

// Number the distinct keys of a MIN table in the order of their first rows and
// write them out; their number ends in the header (n).
static int reps_enqueue(const int32_t* coords, int64_t n, int ncol, const StrideArg& st, void* table,
                        int64_t* slot_of, int32_t* cnt, int64_t* off, void* scan_ws, int32_t* out_coords,
                        int32_t* rep_row, const int32_t* labels, int32_t* out_labels, hipStream_t s) {
    TableHeader* h = reinterpret_cast<TableHeader*>(table);
    const int64_t groups = (n + 63) / 64;
    hipLaunchKernelGGL(k_rep_count, dim3(grid_for(n)), dim3(kThreads), 0, s, n, table, slot_of, cnt);
    GSC_LAUNCH_CHECK();
    int rc = scan_counts(cnt, groups, off, &h->n, scan_ws, s);
    if (rc) return rc;
    const bool vec = rows_vec(coords, ncol);
    auto* kern = ncol == 4 ? k_rep_write<4> : (ncol == 5 ? k_rep_write<5> : k_rep_write<kMaxCols>);
    hipLaunchKernelGGL(kern, dim3(grid_for(n)), dim3(kThreads), 0, s, coords, vec, n, ncol, st, table, slot_of, off,
                       out_coords, rep_row, labels, out_labels);
    GSC_LAUNCH_CHECK();
    return GSC_OK;
}

}  // namespace gsc

using namespace gsc;

extern "C" {

size_t gsc_table_bytes(int64_t n) {
    if (n < 0) return 0;
    return kHeaderBytes + (size_t)table_capacity(n) * sizeof(Slot);
}

static int build_enqueue(const int32_t* coords, int64_t n, int32_t D, void* table, size_t table_bytes,
                         hipStream_t s, const char* what) {
    if (D < 1 || D + 1 > kMaxCols) return fail(GSC_EINVAL, "%s: D=%d outside [1,%d]", what, D, kMaxCols - 1);
    if (n < 0 || n > INT32_MAX) return fail(GSC_EINVAL, "%s: n=%lld outside [0, 2^31)", what, (long long)n);
    if (!table) return fail(GSC_EINVAL, "%s: table is null", what);
    if (n > 0 && !coords) return fail(GSC_EINVAL, "%s: coords is null", what);
    if (table_bytes < gsc_table_bytes(n))
        return fail(GSC_ESHORT, "%s: table needs %zu bytes, got %zu", what, gsc_table_bytes(n), table_bytes);
    if (n == 0) return empty_enqueue(D + 1, table, s);
    return table_enqueue<false>(coords, n, D + 1, unit_stride(), PointsArg{}, table, n, nullptr, SmallOut{}, s);
}

int gsc_coords_build(const int32_t* coords, int64_t n, int32_t D, void* table, size_t table_bytes, void* stream) {
    clear_error();
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int rc = build_enqueue(coords, n, D, table, table_bytes, s, "coords_build");
    if (rc) return rc;
    TableHeader hh;
    rc = read_status(table, s, &hh);
    if (rc) return rc;
    return status_to_code(hh, "coords_build");
}

int gsc_coords_build_async(const int32_t* coords, int64_t n, int32_t D, void* table, size_t table_bytes,
                           void* stream) {
    clear_error();
    return build_enqueue(coords, n, D, table, table_bytes, reinterpret_cast<hipStream_t>(stream),
                         "coords_build_async");
}

int gsc_table_status(const void* table, void* stream) {
    clear_error();
    if (!table) return fail(GSC_EINVAL, "table_status: table is null");
    TableHeader hh;
    int rc = read_status(table, reinterpret_cast<hipStream_t>(stream), &hh);
    if (rc) return rc;
    if (hh.magic != kTableMagic && hh.magic != kGridMagic) return fail(GSC_EINVAL, "table_status: not a table built by gsc_coords_build");
    return status_to_code(hh, "table");
}

size_t gsc_stride_ws_bytes(int64_t n_in) {
    if (n_in < 0) return 0;
    const int64_t groups = (n_in + 63) / 64;
    size_t b = (size_t)n_in * sizeof(int64_t);            // slot of each row
    b = (b + 255) & ~(size_t)255;
    b += (size_t)groups * sizeof(int32_t);                // counts
    b = (b + 255) & ~(size_t)255;
    b += (size_t)(groups + 1) * sizeof(int64_t);          // offsets
    b = (b + 255) & ~(size_t)255;
    b += scan_ws_bytes(groups);
    return b + 256;
}

// The kernels of gsc_coords_stride; the output count ends in the header (n).
static int stride_enqueue(const int32_t* in_coords, int64_t n_in, int32_t D, const int32_t* stride,
                          int32_t* out_coords, void* out_table, size_t out_table_bytes, void* ws, size_t ws_bytes,
                          hipStream_t s, const char* what) {
    if (D < 1 || D + 1 > kMaxCols) return fail(GSC_EINVAL, "%s: D=%d outside [1,%d]", what, D, kMaxCols - 1);
    if (n_in < 0 || n_in > INT32_MAX) return fail(GSC_EINVAL, "%s: n_in=%lld invalid", what, (long long)n_in);
    if (!stride || !out_table) return fail(GSC_EINVAL, "%s: null stride/out_table", what);
    if (n_in > 0 && (!in_coords || !out_coords || !ws)) return fail(GSC_EINVAL, "%s: null in_coords/out_coords/ws", what);
    StrideArg st = unit_stride();
    for (int d = 0; d < D; ++d) {
        if (stride[d] < 1) return fail(GSC_EINVAL, "%s: stride[%d]=%d must be >= 1", what, d, stride[d]);
        st.s[d + 1] = stride[d];
    }
    if (out_table_bytes < gsc_table_bytes(n_in))
        return fail(GSC_ESHORT, "%s: out_table needs %zu bytes, got %zu", what, gsc_table_bytes(n_in), out_table_bytes);
    if (n_in > 0 && ws_bytes < gsc_stride_ws_bytes(n_in))
        return fail(GSC_ESHORT, "%s: ws needs %zu bytes, got %zu", what, gsc_stride_ws_bytes(n_in), ws_bytes);
    const int ncol = D + 1;
    if (n_in == 0) return empty_enqueue(ncol, out_table, s);
    const int64_t groups = (n_in + 63) / 64;
    char* w = reinterpret_cast<char*>(ws);
    int64_t* slot_of = reinterpret_cast<int64_t*>(w);
    w += ((size_t)n_in * sizeof(int64_t) + 255) & ~(size_t)255;
    int32_t* cnt = reinterpret_cast<int32_t*>(w);
    w += ((size_t)groups * sizeof(int32_t) + 255) & ~(size_t)255;
    int64_t* off = reinterpret_cast<int64_t*>(w);
    w += ((size_t)(groups + 1) * sizeof(int64_t) + 255) & ~(size_t)255;
    int rc = table_enqueue<true>(in_coords, n_in, ncol, st, PointsArg{}, out_table, 0, slot_of,
                                 SmallOut{out_coords, nullptr, nullptr, nullptr, nullptr, 0}, s);
    if (rc || n_in <= kSmallRows) return rc;
    return reps_enqueue(in_coords, n_in, ncol, st, out_table, slot_of, cnt, off, w, out_coords, nullptr, nullptr,
                        nullptr, s);
}

int gsc_coords_stride(const int32_t* in_coords, int64_t n_in, int32_t D, const int32_t* stride,
                      int32_t* out_coords, int64_t* n_out, void* out_table, size_t out_table_bytes, void* ws,
                      size_t ws_bytes, void* stream) {
    clear_error();
    if (!n_out) return fail(GSC_EINVAL, "coords_stride: null n_out");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int rc = stride_enqueue(in_coords, n_in, D, stride, out_coords, out_table, out_table_bytes, ws, ws_bytes, s,
                            "coords_stride");
    if (rc) return rc;
    TableHeader hh;
    rc = read_status(out_table, s, &hh);
    if (rc) return rc;
    rc = status_to_code(hh, "coords_stride");
    if (rc) return rc;
    *n_out = hh.n;
    return GSC_OK;
}

// The header's n, status and total_bits, contiguous: what the asynchronous
// form copies to the host.
static_assert(offsetof(TableHeader, status) == offsetof(TableHeader, n) + 8 &&
                  offsetof(TableHeader, total_bits) == offsetof(TableHeader, n) + 12,
              "header layout of the stride result");

int gsc_coords_stride_async(const int32_t* in_coords, int64_t n_in, int32_t D, const int32_t* stride,
                            int32_t* out_coords, int64_t* result, void* out_table, size_t out_table_bytes, void* ws,
                            size_t ws_bytes, void* stream) {
    clear_error();
    if (!result) return fail(GSC_EINVAL, "coords_stride_async: null result");
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    int rc = stride_enqueue(in_coords, n_in, D, stride, out_coords, out_table, out_table_bytes, ws, ws_bytes, s,
                            "coords_stride_async");
    if (rc) return rc;
    GSC_HIP(hipMemcpyAsync(result, &reinterpret_cast<TableHeader*>(out_table)->n, 16, hipMemcpyDeviceToHost, s));
    return GSC_OK;
}

int gsc_coords_stride_result(const int64_t* result, int64_t* n_out) {
    clear_error();
    if (!result || !n_out) return fail(GSC_EINVAL, "coords_stride_result: null result/n_out");
    TableHeader hh{};
    hh.n = result[0];
    std::memcpy(&hh.status, reinterpret_cast<const char*>(result) + 8, 4);
    std::memcpy(&hh.total_bits, reinterpret_cast<const char*>(result) + 12, 4);
    const int rc = status_to_code(hh, "coords_stride");
    if (rc) return rc;
    *n_out = hh.n;
    return GSC_OK;
}

size_t gsc_quantize_ws_bytes(int64_t n, int32_t D) {
    if (n < 0 || D < 1 || D + 1 > kMaxCols) return 0;
    const int64_t groups = (n + 63) / 64;
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    size_t b = al((size_t)n * (D + 1) * sizeof(int32_t));   // integer rows
    b += al((size_t)n * sizeof(int64_t));                    // slot of each row
    b += al((size_t)groups * sizeof(int32_t));               // counts
    b += al((size_t)(groups + 1) * sizeof(int64_t));         // offsets
    b += al((size_t)n * sizeof(int32_t));                    // labels, while out_labels is still being read
    b += scan_ws_bytes(groups);
    return b + 256;
}

int gsc_quantize(const float* points, const int32_t* batch, int64_t n, int32_t D, const float* voxel,
                 const int32_t* labels, int32_t ignore_label, int32_t* out_coords, int64_t* n_out, int32_t* rep,
                 int32_t* out_labels, int32_t* inverse, void* out_table, size_t out_table_bytes, void* ws,
                 size_t ws_bytes, void* stream) {
    clear_error();
    if (D < 1 || D + 1 > kMaxCols) return fail(GSC_EINVAL, "quantize: D=%d outside [1,%d]", D, kMaxCols - 1);
    if (n < 0 || n > INT32_MAX) return fail(GSC_EINVAL, "quantize: n=%lld invalid", (long long)n);
    if (!voxel || !n_out || !out_table) return fail(GSC_EINVAL, "quantize: null voxel/n_out/out_table");
    if (n > 0 && (!points || !out_coords || !rep || !ws))
        return fail(GSC_EINVAL, "quantize: null points/out_coords/rep/ws");
    if (n > 0 && out_labels && !labels) return fail(GSC_EINVAL, "quantize: out_labels without labels");
    VoxelArg va{};
    for (int d = 0; d < D; ++d) {
        if (!(voxel[d] > 0.f) || voxel[d] == INFINITY)
            return fail(GSC_EINVAL, "quantize: voxel[%d]=%g must be positive and finite", d, (double)voxel[d]);
        va.v[d] = voxel[d];
    }
    if (out_table_bytes < gsc_table_bytes(n))
        return fail(GSC_ESHORT, "quantize: out_table needs %zu bytes, got %zu", gsc_table_bytes(n), out_table_bytes);
    if (n > 0 && ws_bytes < gsc_quantize_ws_bytes(n, D))
        return fail(GSC_ESHORT, "quantize: ws needs %zu bytes, got %zu", gsc_quantize_ws_bytes(n, D), ws_bytes);
    hipStream_t s = reinterpret_cast<hipStream_t>(stream);
    const int ncol = D + 1;
    if (n == 0) {
        const int rc0 = empty_enqueue(ncol, out_table, s);
        if (rc0) return rc0;
        GSC_HIP(hipStreamSynchronize(s));
        *n_out = 0;
        return GSC_OK;
    }
    const int64_t groups = (n + 63) / 64;
    auto al = [](size_t b) { return (b + 255) & ~(size_t)255; };
    char* w = reinterpret_cast<char*>(ws);
    int32_t* qc = reinterpret_cast<int32_t*>(w);
    w += al((size_t)n * ncol * sizeof(int32_t));
    int64_t* slot_of = reinterpret_cast<int64_t*>(w);
    w += al((size_t)n * sizeof(int64_t));
    int32_t* cnt = reinterpret_cast<int32_t*>(w);
    w += al((size_t)groups * sizeof(int32_t));
    int64_t* off = reinterpret_cast<int64_t*>(w);
    w += al((size_t)(groups + 1) * sizeof(int64_t));
    int32_t* own_labels = reinterpret_cast<int32_t*>(w);
    w += al((size_t)n * sizeof(int32_t));
    // the voxels' labels are written while the points' are read
    const uintptr_t l0 = (uintptr_t)labels, o0 = (uintptr_t)out_labels, span = (uintptr_t)n * sizeof(int32_t);
    const bool overlap = out_labels && l0 < o0 + span && o0 < l0 + span;
    int32_t* lab = overlap ? own_labels : out_labels;
    const PointsArg pa{points, batch, qc, va};
    int rc = table_enqueue<true>(qc, n, ncol, unit_stride(), pa, out_table, 0, slot_of,
                                 SmallOut{out_coords, rep, inverse, out_labels, labels, ignore_label}, s);
    if (rc) return rc;
    const bool small = n <= kSmallRows;
    if (!small) {
        rc = reps_enqueue(qc, n, ncol, unit_stride(), out_table, slot_of, cnt, off, w, out_coords, rep, labels,
                          lab, s);
        if (rc) return rc;
    }
    if (!small && (out_labels || inverse)) {
        hipLaunchKernelGGL(k_quant_labels, dim3(grid_for(n)), dim3(kThreads), 0, s, n, out_table, slot_of, rep, labels,
                           ignore_label, inverse, lab);
        GSC_LAUNCH_CHECK();
    }
    if (!small && overlap) {
        hipLaunchKernelGGL(k_copy_labels, dim3(grid_for(n)), dim3(kThreads), 0, s, out_table, n, lab, out_labels);
        GSC_LAUNCH_CHECK();
    }
    TableHeader hh;
    rc = read_status(out_table, s, &hh);
    if (rc) return rc;
    rc = status_to_code(hh, "quantize");
    if (rc) return rc;
    *n_out = hh.n;
    return GSC_OK;
}

}  // extern "C"
