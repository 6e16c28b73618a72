// Memory of a coordinate table: its header, the two forms of what follows it,
// and the sizes of a grid.  Plain C++, so that the sizes can be checked without
// a GPU at row counts whose tables no test can hold.
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>
#include <cstdlib>

namespace gsc {

constexpr int kMaxCols = 8;                       // 1 batch column + up to 7 spatial
constexpr unsigned long long kEmptyKey = ~0ull;    // Slot::key holds <= 62 key bits
constexpr uint32_t kTableMagic = 0x54435347u;      // "GSCT": hashed slots
constexpr uint32_t kGridMagic = 0x47435347u;       // "GSCG": occupancy grid of the bounding box
constexpr size_t kHeaderBytes = 256;
// A packed key of up to kNarrowKeyBits bits lives in Slot::key alone; a wider
// one (up to kMaxKeyBits) keeps its low 62 bits there and the rest in
// Slot::hi, which the inserting thread writes right after claiming the slot
// (kHiUnset until then).
constexpr int kNarrowKeyBits = 62;
constexpr int kMaxKeyBits = 92;
constexpr int32_t kHiUnset = -1;

enum : int { ST_DUP = 1, ST_FULL = 2, ST_RANGE = 4 };

struct TableHeader {
    uint32_t magic;
    int32_t ncol;          // 1 + D
    int64_t capacity;      // slots, power of two
    int64_t n;             // number of keys
    int32_t status;        // ST_* bits set on the device
    int32_t total_bits;
    int32_t lo[kMaxCols];  // bounding box, inclusive
    int32_t hi[kMaxCols];
    int32_t shift[kMaxCols];
    int32_t bits[kMaxCols];
    int32_t nblk;            // spatial columns whose lowest varying key bit selects the slot in a line
    int32_t blk_shift[3];    // that key bit, per blocked column
    // a grid table (kGridMagic): cell of a row = sum over columns of
    // ((x_c - lo_c) >> step_c) * cstride_c
    int8_t step[kMaxCols];       // lowest varying bit of the column (coordinates of a coarser tensor stride)
    uint32_t cstride[kMaxCols];
    uint32_t total;              // occupied cells
    int64_t rowof;               // byte offset of the row numbers from the table's start (133 GB at 2^30 rows)
};
static_assert(sizeof(TableHeader) <= kHeaderBytes, "header too large");

// A grid table keeps, instead of slots, one bit per cell of the rows' bounding
// box in words of 32 cells, each with the number of occupied cells that come
// before it in the (arbitrary, but fixed) order of the row numbers:
// the row at an occupied cell is rowof[before + occupied cells of the word
// below it].  A query of an empty cell costs one 8-byte read, a neighbourhood
// shares words, and a scene's words stay in the XCDs' L2, where the hashed
// slots of the same rows (64 bytes or more per row) do not.
struct alignas(8) GridWord {
    uint32_t bits, before;
};
// The box of a grid table spans less than this per column, so that a query's
// distance from the box plus an offset stays within 32 bits.
constexpr int64_t kGridMaxSpan = (int64_t)1 << 30;

struct alignas(16) Slot {
    unsigned long long key;
    int32_t val;
    int32_t hi;   // key bits 62 and up of a wide key
};
static_assert(sizeof(Slot) == 16, "slot must be 16 bytes");

// capacity: a power of two >= 4n (load factor <= 1/4) and >= 64.  The
// environment variable GSC_TABLE_CAP_LIMIT (a test hook) caps it at the
// largest power of two >= 64 not above its value, so that a table too small
// for its rows, and the EFULL it reports, can be exercised; every insert and
// query still stops after one pass over the slots.
inline int64_t table_capacity(int64_t n) {
    int64_t cap = 64;
    while (cap < 4 * n) cap <<= 1;
    if (const char* e = getenv("GSC_TABLE_CAP_LIMIT")) {
        const long long lim = strtoll(e, nullptr, 10);
        while (cap > 64 && cap > lim) cap >>= 1;
    }
    return cap;
}

// The memory of a table for n rows of cap slots: the words of a grid, the box
// kernel's per-block results, then one row number per row.
struct GridLayout {
    int64_t word_bytes;   // words that the build clears, and so the most a grid may use
    size_t part;          // byte offsets from the table's start
    size_t rowof;
    int64_t max_cells;    // 0: hashed slots only
};

constexpr int kBoxThreads = 512;
constexpr int kBoxBlocks = 256;                 // at most; four per lane of the wave that combines them
constexpr int kBoxInts = 4 * kMaxCols + 1;      // lo, hi, or, and per column; out of range

// blocks of the box kernel; their results fit the slots' memory
inline int box_blocks(int64_t n, int64_t cap) {
    const int64_t per = kBoxThreads * 2;
    const int64_t b = std::min((n + per - 1) / per, cap * (int64_t)sizeof(Slot) / (kBoxInts * 4));
    return (int)std::clamp<int64_t>(b, 1, kBoxBlocks);
}

// A grid may have kGridCells cells per row (48 bytes of words each: three
// quarters of the table's memory at its smallest), or, with few rows, as many
// cells as kSmallRows rows where the table has room for their words.  The build
// of more rows clears that much before it knows the box, which at 300,000 rows
// (14 MB) costs about 3 us.  Rooms voxelised at 2 cm have 112 to
// 120 cells per row, at 4 to 5 cm 20 to 30; boxes past the limit are hashed.
// Cells are numbered in 32 bits, so no grid has more than kGridMaxCells (from
// 11 million rows on that is the nearer limit).
// The environment variable GSC_TABLE_CAP_LIMIT (a test hook for the hashed
// slots) turns grids off.
constexpr int64_t kGridCells = 192;
constexpr int64_t kGridMaxCells = (int64_t)1 << 31;
constexpr int kSmallPer = 3, kSmallThreads = 1024;               // see k_small
constexpr int kSmallRows = kSmallThreads * kSmallPer;
constexpr int kSmallWords = kSmallRows * (int)kGridCells / 32;
constexpr int kSmallSlots = 16384;                               // table_capacity(kSmallRows)
static_assert(kSmallSlots >= 4 * kSmallRows && kSmallSlots / 2 < 4 * kSmallRows, "slots of kSmallRows rows");

inline GridLayout grid_layout(int64_t n, int64_t cap) {
    GridLayout g{};
    const int64_t region = cap * (int64_t)sizeof(Slot);
    const int64_t rows = (4 * n + 15) / 16 * 16, part = ((int64_t)box_blocks(n, cap) * kBoxInts * 4 + 15) / 16 * 16;
    const int64_t want = n <= kSmallRows ? kSmallWords * (int64_t)sizeof(GridWord) : n * (kGridCells / 4);
    const int64_t room = region - rows - part;
    const bool on = n > 0 && room >= 16 && cap >= 4 * n && !getenv("GSC_TABLE_CAP_LIMIT");
    constexpr int64_t most = kGridMaxCells / 32 * (int64_t)sizeof(GridWord);
    g.word_bytes = on ? std::min(std::min(want, room), most) / 16 * 16 : 0;
    g.max_cells = g.word_bytes / (int64_t)sizeof(GridWord) * 32;
    // the boxes lie behind the words (without a grid anywhere: the slots are set after they have been read)
    g.part = kHeaderBytes + (on ? (size_t)(region - rows - part) : 0);
    g.rowof = kHeaderBytes + (on ? (size_t)(region - rows) : 0);
    return g;
}

}  // namespace gsc
