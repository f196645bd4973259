// Internal layout of a built VBR matrix: the index arrays of the format, the packed values in
// the order the MFMA kernel reads them, and the workgroup schedule.  Host and device code of the
// library share this header; nothing outside the library includes it.
#pragma once

#include <cstdint>
#include <memory>
#include <vector>

#include "vbr_spmm.h"

namespace vbrk {

constexpr int kSlabRows = 16;       // rows of one MFMA slab
constexpr int kStepK = 32;          // B rows consumed per K-step (one 16x16x32 MFMA deep)
constexpr int kMaxSlabs = 8;        // slabs per workgroup tile (128 rows)
constexpr int kFragElems = kSlabRows * kStepK;   // 512 16-bit values = 1 KiB per (slab, K-step)
constexpr int kMaxGatherSlabs = 4;  // slabs per column-gathered tile (64 rows) ...
constexpr int kMaxDeepSlabs = 2;    // ... and per deep one (32 rows)
constexpr int kSplitSteps = 12;     // K-steps from which on a tile is split over K in launches of few workgroups, while those that result may be more than two on
                                    // a CU (gathered, two slabs, 240 workgroups, not split and split: 10 K-steps 9.0 and 9.0 us, 8: 7.9 and 8.3, 6: 6.9 and 8.1) ...
constexpr int kSplitShort = 4;      // ... and where two on a CU hold them all: see plan_launches
// slabs of the tallest tile that can be split in a launch of the mixed kernel, with deeper rings (two workgroups on a CU) and without
constexpr int split_slabs(bool few) { return few ? 4 : 2; }
constexpr int kDeepN = 64;          // C columns per workgroup of a deep tile, and of a split launch
constexpr int kTileN = 256;         // C columns per workgroup of the tile kernel
constexpr int kWideN = 512;         // C columns per workgroup of the wide kernel
constexpr int kWideAhead = 5;       // K-steps behind a tile's last whose B rows it looks up, and does not use
constexpr int kPanelN = 128;        // C columns per workgroup of the panel kernel
constexpr int kZeroN = 1024;        // C columns per workgroup of the kernel that stores zeros
constexpr int kXcd = 8;             // L2 domains; workgroup i runs on domain i % 8

#ifdef __HIPCC__
#define VBRK_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define VBRK_HOST_DEVICE inline
#endif

// Bytes from B's first element to the end of its last row, and the most that offsets of 32 bits reach, less a page for the offset that stands for "none".
constexpr int64_t kNearBytes = 0xFFFFF000ll;
inline int64_t b_bytes_of(int64_t n_cols, int64_t ldb, int64_t N) { return n_cols > 0 ? ((n_cols - 1) * ldb + N) * 2 : 0; }

// What map_workgroup needs to know of a launch beside T and Q: the way column tiles are dealt, and for fewer than 8 of them, whole, four bits a
// domain each: its column tile, its number among the domains of that, and how many these are.  (Every wave divided for them: entry rows of 16384 x
// 16384, 8 entries a row, N = 8 4.2 and now 4.0 us, N = 256 9.5 and 9.3; 1024 rows in groups of 32, N = 256 4.6 and 4.4.)
struct ColumnMap { uint32_t even, ntile, member, members; };
inline ColumnMap column_map(uint32_t Q, bool even)
{
    ColumnMap m{even, 0, 0, 0};
    for (uint32_t x = 0; x < kXcd && Q < kXcd; ++x) {
        const uint32_t ntile = x % Q;
        m.ntile |= ntile << (4 * x);
        m.member |= x / Q << (4 * x);
        m.members |= (kXcd - ntile + Q - 1) / Q << (4 * x);
    }
    return m;
}

// Workgroup -> (one of T tiles, one of Q column tiles); false: nothing to do.  Workgroups are dealt to the 8 L2 domains round-robin; a
// domain keeps to few column tiles, every eighth, so that the B columns it gathers stay in its L2, and takes one after the other.  (Column tiles
// side by side on a domain: 16 x 16 blocks, 4096 x 16384, N = 4096 160 and 175 us among other calls, 64 x 64 blocks at 40 %, N = 8192 396 and 487;
// only in launches of the mixed kernel, graph of 16384 nodes, N = 4096 173.2 and 170.5, 40 other graphs the same.)
// The column tiles left over when every domain has as many: a domain takes one or none, with fewer than 8 column tiles in all several domains
// share one as long as there are domains.  Five or nine column tiles leave most domains half idle that way; `even` cuts each that is left over in
// shares, 8 or 4 of its tiles' workgroups in turn, so that all domains have the same number, of two column tiles at most (what it gains and
// where: even_columns).  A domain with parts of two takes the workgroups in the order of the tiles, the longest first, or (IN_TURN) one column
// tile after the other, which is better for rows of entries, many short workgroups that live on what is in the L2 (16384 x 16384, 8 entries a
// row, N = 640 22.9 and 21.2 us, N = 712 32.3 and 30.5) and worse for tiles (graph of 16384 nodes, N = 1200 65.5 and 78).
template <bool IN_TURN = false>
VBRK_HOST_DEVICE bool map_workgroup(uint32_t block, uint32_t T, uint32_t Q, const ColumnMap &m, int &tile, int &ntile)
{
    const uint32_t x = block % kXcd, own = Q / kXcd, rest = Q % kXcd;
    uint32_t j = block / kXcd;
    if (Q >= kXcd) {
        const uint32_t round = j / T;
        tile = (int)(j - round * T);
        ntile = (int)(x + kXcd * round);
        if (!m.even || round < own) return (uint32_t)ntile < Q;
        j -= own * T;
    } else if (!m.even) {
        ntile = (int)(m.ntile >> (4 * x) & 15);
        tile = (int)((m.member >> (4 * x) & 15) + (m.members >> (4 * x) & 15) * j);
        return (uint32_t)tile < T;
    }
    const uint32_t lg = rest & 1 ? 0 : rest & 2 ? 1 : 2, shares = kXcd >> lg, n = rest >> lg;      // of a column tile, and how many of them a domain has
    const uint32_t begin = x * n;
    uint32_t k = 0, period = j;
    if (n > 1) {
        if (IN_TURN) {
            const uint32_t periods = (T + shares - 1) >> (3 - lg), here = shares - (begin & (shares - 1)), first = n < here ? n : here;
            const bool second = j >= first * periods;
            if (second) j -= first * periods;
            const uint32_t width = second ? n - first : first;
            if (width == 0) return false;
            period = j / width;
            k = j - period * width + (second ? first : 0);
        } else {
            period = j / n;
            k = j - period * n;
        }
    }
    const uint32_t u = begin + k;
    ntile = (int)(kXcd * own + (u >> (3 - lg)));
    // (the share of the i-th of eight tiles is i with its bits turned round: the last tiles, less than eight, do not fall on one domain)
    tile = (int)(shares * period + ((0x73516240u >> (4 * (u & (shares - 1))) & 15) >> lg));
    return (uint32_t)tile < T;
}

// Workgroups of a launch over T row tiles and Q column tiles, by either way of map_workgroup.
inline int64_t grid_size(int64_t T, int64_t Q, bool even = false)
{
    if (even) {
        const int64_t rest = Q % kXcd, each = rest & -rest, shares = kXcd / each;
        return kXcd * (Q / kXcd * T + rest / each * ((T + shares - 1) / shares));
    }
    if (Q >= kXcd) return (int64_t)kXcd * ((Q + kXcd - 1) / kXcd) * T;
    return (int64_t)kXcd * ((T + (kXcd / Q) - 1) / (kXcd / Q));
}

// Number of a workgroup among those of a column tile -> the tile, and the quarter of the column tile if the tile has four workgroups (true): of the
// tiles of a mixed launch the first `whole` have one, `rest` have four, those of the first quarter before those of the second, and the others,
// tiles without a K-step, have one.  (Without tiles that have four, `whole` is all of them.)
VBRK_HOST_DEVICE bool split_tile(int &tile, int whole, int rest, int &quarter)
{
    quarter = 0;
    if (tile < whole) return false;
    const int q = (tile - whole) / rest;
    tile -= rest * (q < 3 ? q : 3);
    if (q > 3) return false;
    quarter = q;
    return true;
}

// One workgroup tile: up to kMaxSlabs slabs of ONE row group, walked over the group's K-steps (a block tile), or up to
// kMaxGatherSlabs slabs of the row list, walked over the columns its rows touch (a column-gathered tile).
struct TileDesc {
    int32_t ks_begin;    // first K-step of the tile's group (global K-step number); gathered: of the tile, in gcol
    int32_t n_ks;        // K-steps of the group; gathered: of the tile
    int64_t a_off;       // first value of the tile, in units of 8 values (16 bytes)
    int32_t row_begin;   // position in perm of the tile's first row; gathered: in prow
    int32_t n_rows;      // rows of the tile, 1 .. 16 * n_slabs
    int32_t n_slabs;     // ceil(n_rows / 16)
    int32_t group;       // row group the tile belongs to; column-gathered tiles: kTileGathered, or kTileDeep less the quarter
                         // of a 256-column tile (0 .. 3) a workgroup takes
};
constexpr int32_t kTileGathered = -1, kTileDeep = -2;
// Classes of tiles: block tiles of 1, 2, 3-4, 5-8 slabs, deep tiles, gathered tiles of 1, 2, 3-4 slabs.
constexpr int kClassDeep = 4, kClassGather = 5, kClasses = 8;
static_assert(sizeof(TileDesc) == 32, "TileDesc is read by the kernel as 2 x 16 bytes");

// Position inside a (slab, K-step) fragment of the value at slab row m and K-step-local column
// kk (0..31 = row of the staged B panel), for a slab that stores `rows` rows (16, or fewer for the
// last slab of a tile: padding rows are not stored).  Lane l = m + 16 q of the wave holds 8 values
// (slots 0..7) of slab row m; a fragment is laid out [q][m][slot], so it takes rows * 32 values.
// The K order inside the step is permuted so that the four B rows a 16-lane group reads with one
// transposed LDS read, together with those of its neighbour group, fall into distinct LDS banks:
//   kk = 8 u + 4 v + e  ->  q = 2 (u / 2) + v,  slot = 4 (u % 2) + e.
inline int frag_index(int m, int kk, int rows)
{
    int u = kk >> 3, v = (kk >> 2) & 1, e = kk & 3;
    int q = 2 * (u >> 1) + v;
    int slot = 4 * (u & 1) + e;
    return ((q * rows + m) << 3) + slot;
}

// Values per K-step of a tile: full slabs take 512, the last slab rows_last * 32.
inline int64_t tile_kstep_stride(int32_t n_rows, int32_t n_slabs)
{
    int rows_last = n_rows - (n_slabs - 1) * kSlabRows;
    return (int64_t)(n_slabs - 1) * kFragElems + (int64_t)rows_last * kStepK;
}

// One workgroup panel: a few slabs (8) cut from the rows of SHORT row groups (height < 16) in
// permuted order, whatever group they belong to, walked over the union of the column blocks of
// those groups.  A B row panel is loaded once per K-step for all slabs; a slab only multiplies
// where its own groups store a block (mask bit), its fragment then follows in the value stream.
struct PanelDesc {
    int32_t ks_begin;    // first physical K-step of the panel (index into the host's pk_mask / pk_row)
    int32_t n_ks;        // physical K-steps
    int64_t a_off;       // first value of the panel, in units of 8 values (16 bytes)
    int32_t row_begin;   // first row of the panel in the panel-row list
    int32_t n_rows;      // rows of the panel, 1 .. 16 * slabs per panel
    int32_t meta_begin;  // first record of the panel in the device's K-step stream (pk_meta)
    int32_t pad;
};
static_assert(sizeof(PanelDesc) == 32, "PanelDesc is read by the kernel as 2 x 16 bytes");

constexpr int kPanelMaxFrags = 8;    // fragments per physical K-step (one load per wave); more -> the step is split
constexpr int kPanelMetaPad = 12;    // records appended to a panel's K-step stream, so that the kernel's look-ahead needs no bound checks

// The stream kernel: a workgroup owns up to kStreamWaves * kStreamGroups row groups of one slab and kStreamN columns of C, and multiplies by a schedule
// (stream_schedule.h) of steps.  In a step every wave multiplies up to 4 .. kStreamMostOps K-steps of its groups, and brings up to two units of 16 B rows.
constexpr int kStreamN = 64, kStreamWaves = 8, kStreamGroups = 8;
constexpr int kStreamLeastOps = 4, kStreamMostOps = 8;
constexpr int kStreamUnits = 2;
constexpr int kStreamAhead = 2;        // units are in LDS that many steps after they were asked for
constexpr int kStreamSlots = 79;       // places for units in LDS, and one more that holds zeros
constexpr int kStreamUnitBytes = kSlabRows * kStreamN * 2;
constexpr int kStreamShare = 4;        // row tiles that share the first requests of B
constexpr int kStreamEarly = 48;       // units before its own that a workgroup asks for its share of them
constexpr int kStreamMinTiles = 64;    // tiles from which on a matrix may get a schedule
constexpr int kStreamLeastN = 512;     // columns of B from which on a call may take it
constexpr int kStreamMostCols = 1 << 24;      // B rows: what the kernel multiplies row numbers with has 24 bits
// Of every step a wave has two of these records, one for each half of its lanes: of the two units of a K-step, and of those it brings.
struct StreamRecord {
    // the lanes of a row of 16 hold two words each, which the others of the row get by a broadcast
    int32_t word[16][2];
    int32_t &slot(int i) { return word[i][0]; }                        // where the unit of the K-step behind this one is in LDS, in bytes
    int32_t &frag(int i) { return word[kStreamMostOps + i][0]; }       // fragments of the next step's K-steps, in bytes from the first value (in both records the same)
    int32_t &row() { return word[0][1]; }                              // first B row of the unit to ask for, ...
    int32_t &none() { return word[1][1]; }                             // ... kStreamNone if there is none, else 0, ...
    int32_t &to() { return word[2][1]; }                               // ... and where it goes
    int32_t &groups() { return word[3][1]; }                           // groups of this step's K-steps, four bits each, kStreamGroups: none (in both records the same)
    int32_t &early(int i) { return word[5 + i][1]; }                   // first B rows of two units to bring into the L2, -1: none
    int32_t slot(int i) const { return word[i][0]; }
    int32_t frag(int i) const { return word[kStreamMostOps + i][0]; }
    int32_t row() const { return word[0][1]; }
    int32_t none() const { return word[1][1]; }
    int32_t to() const { return word[2][1]; }
    int32_t early(int i) const { return word[5 + i][1]; }
    int32_t group(int i) const { return word[3][1] >> (4 * i) & 15; }
};
static_assert(sizeof(StreamRecord) == 128 && kStreamMostOps == 8, "read by the kernel as 16 x 8 bytes");
constexpr int32_t kStreamNone = (int32_t)(uint32_t)kNearBytes;
// what a workgroup's groups are: first positions in perm of wave w's at row_begin[w * kStreamGroups], -1: none
struct StreamTile {
    int32_t first_step, n_steps;
    int32_t row_begin[kStreamWaves * kStreamGroups];
};

// Byte offsets of the sections inside the device buffer (each 256-byte aligned).
struct DeviceLayout {
    int64_t zeros_off = 0, tiles_off = 0, krow_off = 0, perm_off = 0, vals_off = 0, total = 0;
    int64_t stream_tiles_off = 0, stream_steps_off = 0;
    int64_t panels_off = 0, pk_meta_off = 0, prow_off = 0;
    int64_t gcol_off = 0;      // by_entries: the entries; prow their rows
};

// The packed values on the host: not cleared when allocated, every tile writes its own part.
class HostValues {
public:
    void allocate(size_t n) { p_.reset(new uint16_t[n]); n_ = n; }
    uint16_t *data() { return p_.get(); }
    const uint16_t *data() const { return p_.get(); }
    size_t size() const { return n_; }
    const uint16_t &operator[](size_t i) const { return p_[i]; }

private:
    std::unique_ptr<uint16_t[]> p_;
    size_t n_ = 0;
};

// An entry: its column and the 16 bits of its value, together so that one load brings both: the low and the high half of a word where all columns
// are below kEntryNear, else a word each.
constexpr int64_t kEntryNear = 1 << 16;
struct Entry {
    int32_t col;
    uint32_t val;
};
constexpr int kEntryPad = 1;         // entries of zeros behind the last one: rows without entries, which stand last, read the one at their start, without effect

// A row of entries: the first of them, how many, and its row of C; 16 bytes, which one load brings.
struct EntryRow {
    int64_t start;
    int32_t len, row;
};
static_assert(sizeof(Entry) == 8 && sizeof(EntryRow) == 16, "read by the kernels as 4 or 8 and 16 bytes");

// Rows of a matrix as lists of entries, the longest row first (csr_spmm.hip multiplies them): positions 0 .. rows-1,
// the entries of a position at start[pos] .. start[pos + 1].
struct EntryRows {
    std::vector<int64_t> start;      // [rows + 1]
    std::vector<EntryRow> row;       // what the device knows of every position
    bool near = false;               // an entry is one word
    std::unique_ptr<uint32_t[]> entry;      // of one or two words, and kEntryPad behind them
    int64_t count = 0;               // of them, without these
    void allocate(int64_t n, int64_t n_cols)
    {
        near = n_cols <= kEntryNear;
        count = n;
        entry.reset(new uint32_t[(size_t)(n + kEntryPad) * (near ? 1 : 2)]);
        for (int64_t i = n; i < n + kEntryPad; ++i) put(i, 0, 0);
    }
    void put(int64_t i, int32_t col, uint16_t val)
    {
        if (near) {
            entry[(size_t)i] = (uint32_t)col | (uint32_t)val << 16;
        } else {
            entry[(size_t)i * 2] = (uint32_t)col;
            entry[(size_t)i * 2 + 1] = val;
        }
    }
    Entry get(int64_t i) const
    {
        if (near) return Entry{(int32_t)(entry[(size_t)i] & 0xFFFFu), entry[(size_t)i] >> 16};
        return Entry{(int32_t)entry[(size_t)i * 2], entry[(size_t)i * 2 + 1]};
    }
    size_t bytes() const { return entry ? (size_t)(count + kEntryPad) * (near ? 4 : sizeof(Entry)) : 0; }
};

}  // namespace vbrk

struct vbr {
    int64_t n_rows = 0, n_cols = 0, nnz = 0;
    int32_t col_block = 0, dtype = 0;
    int32_t n_groups = 0;
    // the VBR index (bit-exact part of the format)
    std::vector<int32_t> perm, row_groups;
    std::vector<int64_t> blk_ptr, blk_off;
    std::vector<int32_t> blk_col;
    // kernel-side data
    int32_t lg_gran = 0;                 // log2 of the B-row gather granularity (rows per krow entry)
    std::vector<int64_t> ks_ptr;         // [n_groups+1] first global K-step of each group
    std::vector<int32_t> krow;           // first B row of each granule of each K-step (granules of 8 rows or more), the last one repeated to the end
    std::vector<vbrk::TileDesc> tiles;    // block tiles, group by group
    std::vector<int64_t> group_first_tile;      // [n_groups+1] tiles of a group in `tiles`
    std::vector<vbrk::TileDesc> dev_tiles;      // `tiles` and `gtiles` as the device holds them: longest first, deep ones four times,
                                                // those without a K-step last
    int32_t n_work = 0;                         // of them with a K-step
    int32_t class_count[vbrk::kClasses] = {0};  // of these, per class ...
    int32_t long_count[vbrk::kClasses] = {0};   // ... and with at least kSplitSteps K-steps
    int64_t work_steps = 0;                     // the K-steps of these, a deep tile once, ...
    int32_t work_lists = 0, longest_list = 0;   // ... in how many lists, and of the longest one
    vbrk::HostValues vals;               // packed fragments: block tiles, panels, gathered tiles, then 1 KiB of zeros
    // Rows that are not multiplied in block tiles stand in a row list (prow): first those of groups of height < 16
    // ("low rows"), in an order of the packing's own, then those of taller groups whose blocks are mostly fill-in.
    // The list is cut into slabs of 16 positions.  A chunk of 8 slabs of low rows may be packed as ONE PANEL (its
    // slabs share the B rows of the union of their column blocks); all other slabs form COLUMN-GATHERED TILES of 1
    // to 4 slabs, which gather exactly the B rows of the columns their own rows touch.
    int32_t panel_slabs = 0;             // slabs per chunk (8); 0 = the matrix has no low rows
    int32_t deep_steps = 0;              // K-steps from which on a gathered tile is split over K (a "deep" tile)
    std::vector<int32_t> prow;           // original row of every position of the row list, -1 = padding
    std::vector<int32_t> row_pos;        // [n_rows] position in the row list of every position in perm, -1 = block tile
    std::vector<int32_t> chunk_panel;    // [n_chunks] index of its panel in `panels`, -1 = gathered tiles
    std::vector<int32_t> slab_tile;      // [n_slabs] index in `gtiles` of the slab's tile, -1 = in a panel
    std::vector<vbrk::TileDesc> gtiles;   // column-gathered tiles in creation order: row_begin = position in prow
    std::vector<int32_t> gcol;           // per K-step of a gathered tile 32 columns of A (= rows of B), rising, the last column repeated to the end
    std::vector<vbrk::PanelDesc> panels;
    std::vector<int32_t> pk_row;         // host only: first B row of each granule of each physical K-step, -1 = padding
    std::vector<uint32_t> pk_mask;       // host only: slabs present in each physical K-step
    std::vector<int32_t> pk_meta;        // device: per physical K-step one record {mask, granule rows...}; each panel's
                                         // records are followed by kPanelMetaPad records {0, rows of its last step}
    std::vector<int32_t> pk_logical;     // host only: K-step number inside the panel's union (a split step repeats it)
    std::vector<int64_t> pk_frag;        // host only: ordinal of the step's first fragment inside its panel
    std::vector<int64_t> p_union_ptr;    // host only: [n_panels+1] into p_union
    std::vector<int32_t> p_union;        // host only: ascending union of the column blocks of each panel
    // Block tiles of one slab, if all tiles are and some call takes the stream kernel, for that, too.
    std::vector<vbrk::StreamTile> stream_tiles;
    std::vector<vbrk::StreamRecord> stream_steps;
    int32_t stream_ops = 0;              // K-steps of a wave in a step of theirs
    int32_t stream_longest = 0;          // steps of the longest
    // A matrix whose blocking found next to nothing to share is kept as entries only: no tiles, no panels, no values above.
    bool by_entries = false;
    vbrk::EntryRows entries;
    vbrk::DeviceLayout lay;
    void *dev = nullptr;                 // uploaded buffer (caller-owned)
};
