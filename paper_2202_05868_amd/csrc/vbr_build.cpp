// VBR construction on the host: index arrays of the format (section 2 and the last paragraph of
// section 3.1 of the paper), values packed as MFMA fragments, and the workgroup schedule.
#include <algorithm>
#include <atomic>
#include <cstdint>
#include <memory>
#include <new>
#include <utility>
#include <vector>

#include "host_threads.h"
#include "stream_schedule.h"
#include "vbr_host.h"

namespace vbrk {

static int64_t stream_most_steps(const vbr *v, int64_t tiles, int ops);

namespace {

inline int64_t align_up(int64_t x, int64_t a) { return (x + a - 1) / a * a; }
inline int64_t steps_of(int64_t rows_of_b) { return (rows_of_b + kStepK - 1) / kStepK; }

inline int slab_class(int n_slabs)   // kernels exist for 1, 2, 4 and 8 slabs
{
    return n_slabs <= 1 ? 0 : n_slabs <= 2 ? 1 : n_slabs <= 4 ? 2 : 3;
}

inline int tile_class(const TileDesc &td)
{
    return td.group >= 0 ? slab_class(td.n_slabs) : td.group == kTileGathered ? kClassGather + slab_class(td.n_slabs) : kClassDeep;
}

// Rows of groups shorter than a slab go into panels when the block width allows the scalar
// gather path and there are enough of them to give every CU a panel or two (a panel is one long
// running workgroup per 128 columns; a handful of them would leave most of the chip idle).
// 8 slabs per panel: measured against 16, twice the workgroups (two resident per CU) gain more
// than the B rows shared by fewer slabs cost (noisy planted matrix 271 -> 185 us, others within 2 %).
constexpr int kPanelSlabs = 8;
constexpr int64_t kPanelMinRows = 4096;
inline bool use_panels(int lg_gran, int64_t short_rows) { return lg_gran >= 3 && short_rows >= kPanelMinRows; }
// Panels are a launch of their own, which the others wait for: a few of them, one workgroup each for up to 64 K-steps, are not worth it
// (7680 x 1856, 64-column blocks, N = 120, one panel among 250 tiles 41 us, all tiles 12.6; 6272 x 1984, N = 160, 17 panels 43 and 23; 6912 x
// 1920, N = 72, 17 panels 42 and 15).  (Against gathered tiles of up to 64 rows many of them are not the faster ones either: 6000 rows of 12
// 8-column blocks, N = 512, 47 panels 12.3 us, as tiles 6.2.)
constexpr int64_t kPanelMinCount = 20;
// Load instructions per K-step and 256 columns of C: a panel brings 32 B rows x 128 columns (8 loads)
// and up to 8 fragments (8 loads) per 128 columns; a one-slab tile 32 B rows x 256 columns (16 loads)
// and one fragment.  The direct-to-LDS load instruction is the unit of cost of both kernels.
constexpr int64_t kPanelStepCost = 32, kTileStepCost = 17;
constexpr int64_t kPanelMaxSteps = 64;       // a panel is not split over K: longer ones would outlast the launch
constexpr int64_t kSlabMaxCols = 1024;       // columns a slab of low rows gathers before the next group starts a new slab

// What a tile takes, in nanoseconds per workgroup of 256 columns: per K-step by its height (rates measured on full
// launches), and as much as four K-steps to start and to store.  Block tiles: 1, 2, 4, 8 slabs.  Gathered tiles: 1 to 4
// slabs; in the deep form (the four waves split the K-steps, 64 columns each) 1 or 2 slabs.
constexpr int64_t kBlockStepNs[4] = {190, 215, 300, 370};
constexpr int64_t kGatherStepNs[kMaxGatherSlabs] = {240, 255, 280, 300};
constexpr int64_t kDeepStepNs[kMaxDeepSlabs] = {290, 350};
constexpr int64_t kEntryPs = 7000, kEntryRowPs = 15000;      // the same for entry rows, in picoseconds per entry and per row
constexpr int64_t kEntriesMinRows = 8192;    // not where the two cross: see entries_cost_less
constexpr int64_t kTileStartSteps = 4;
constexpr int64_t kDeepSteps = 32;           // no tile of fewer K-steps is deep
constexpr int64_t kMergeMinSlabs = 64;       // fewer low slabs stay single: height costs workgroups, and there are few
constexpr int64_t kShortSteps = 8, kShortMinSlabs = 512;     // these three lines: see cut_into_tiles
constexpr int64_t kSmallSteps = 1152, kFewTiles = 96;
constexpr int64_t kEmptyApart = 512;         // workgroups: see plan_launches
constexpr int64_t kTwoOnACu = 512, kThreeOnACu = 768, kFourOnACu = 1024, kEightOnACu = 2048;      // workgroups that are resident with two, three, four and eight on a CU
constexpr int64_t kSegmentSlabs = 64;        // the cutting of the slab list into tiles is optimised over stretches of this length

inline int64_t gather_cost(int64_t cols, int n_slabs, int64_t deep_steps)
{
    const int64_t ks = steps_of(cols);
    if (ks < deep_steps) return (ks + kTileStartSteps) * kGatherStepNs[n_slabs - 1];
    if (n_slabs <= kMaxDeepSlabs) return (ks + kTileStartSteps) * kDeepStepNs[n_slabs - 1];
    return INT64_MAX / 4;
}

// K-steps from which on a tile is deep, for a matrix of `total` K-steps: the share of one of 768 resident workgroups at
// N = 2048.  N is not known here; the line holds for the others too.  Graph of 16384 nodes, 64 edges a node, half of it, this and
// twice as much: N = 256 36.8, 34.0, 59.3 us; N = 1024 67, 52, 67; N = 2048 106, 94, 109; N = 4096 225, 202, 216; of 8192 nodes and 64
// edges, N = 256 20.0, 19.9, 28.1; with fewer edges the three are within 4 %.
inline int64_t deep_from(int64_t total) { return std::max<int64_t>(kDeepSteps, total * 8 / 768); }

// What a thread needs to count and look up the columns and column blocks of a few rows.
struct Scratch {
    std::vector<int32_t> stamp, pos;   // per column
    std::vector<int32_t> block_pos;    // per column block
    int32_t now = 0;
    void fit(int64_t n_cols, int64_t n_blocks)
    {
        if (!stamp.empty()) return;
        stamp.assign((size_t)std::max<int64_t>(n_cols, 1), 0);
        pos.resize(stamp.size());
        block_pos.assign((size_t)std::max<int64_t>(n_blocks, 1), -1);
    }
    // columns of the row that none of the rows since the last begin() had
    void begin()
    {
        if (now == INT32_MAX) { std::fill(stamp.begin(), stamp.end(), 0); now = 0; }
        ++now;
    }
    int64_t add(const vbr_csr_t *csr, int64_t row)
    {
        int64_t fresh = 0;
        for (int64_t p = csr->row_ptr[row]; p < csr->row_ptr[row + 1]; ++p) {
            int32_t &s = stamp[csr->col_idx[p]];
            fresh += s != now;
            s = now;
        }
        return fresh;
    }
};

class Builder {
public:
    Builder(const vbr_csr_t *csr, const int32_t *perm, const int32_t *row_groups, int32_t G, int32_t col_block, vbr *v, bool schedules)
        : csr(csr), perm(perm), rg(row_groups), G(G), cb(col_block), M(csr->n_rows), KB(csr->n_cols / col_block), v(v), schedules(schedules),
          team(threads_for(csr->nnz + csr->n_rows, 1 << 15)), scratch((size_t)team.size())
    {
    }
    int build();

private:
    enum Kind : uint8_t { kLow, kBlocks, kGathered };
    struct Piece {                     // a stretch of groups, worked on by one thread
        int32_t g0, g1;
        std::vector<int32_t> blocks;   // column blocks of its groups, one group after the other
        int64_t first_block;
    };

    int64_t nnz_of(int64_t q0, int64_t q1) const
    {
        int64_t n = 0;
        for (int64_t q = q0; q < q1; ++q) n += csr->row_ptr[perm[q] + 1] - csr->row_ptr[perm[q]];
        return n;
    }
    // f(scratch, i) for i in [0, n), dealt in runs of `run` to whoever is free
    template <class F>
    void each(int64_t n, int64_t run, F f)
    {
        std::atomic<int64_t> next(0);
        auto work = [&](int member) {
            Scratch &s = scratch[(size_t)member];
            s.fit(csr->n_cols, KB);
            for (;;) {
                const int64_t b = next.fetch_add(run);
                if (b >= n) break;
                for (int64_t i = b; i < std::min(n, b + run); ++i) f(s, i);
            }
        };
        if (n <= run) work(0);
        else team.run(work);
    }

    void index_blocks();
    Kind kind_of(Scratch &s, int64_t r0, int64_t r1, int64_t n_blocks);
    bool entries_cost_less();
    void keep_entries();
    int block_tiles();
    void order_low_rows();
    bool hubs_first();
    void cluster_low_groups();
    void choose_panels();
    int emit_panel(int64_t chunk);
    void append_gathered_groups();
    void cut_into_tiles();
    int emit_gather_tiles();
    void fill_values();
    void schedule();
    void stream();
    void lay_out();

    const vbr_csr_t *csr;
    const int32_t *perm, *rg;
    const int32_t G, cb;
    const int64_t M, KB;
    vbr *v;
    const bool schedules;
    Team team;
    std::vector<Scratch> scratch;
    std::vector<Kind> kind;
    std::vector<Piece> pieces;
    std::vector<int32_t> low_groups, gathered_groups;
    int64_t a_units = 0;               // running size of the packed values, in units of 8 values
    int gran = 1, per_step = kStepK;
    bool panels_on = false;
    int64_t low_slabs = 0;             // slabs of low rows; those of the gathered groups follow in the row list
    std::vector<int32_t> prow_group;   // group of every position of the row list, -1 = padding
    std::vector<int64_t> panel_dst, panel_src;   // values of the panels: position in vals <- position in csr->vals
    std::vector<std::pair<int64_t, int64_t>> panel_range;   // [begin, end) of the panels' values, in units of 8
};

int Builder::build()
{
    v->n_rows = M;
    v->n_cols = csr->n_cols;
    v->nnz = csr->nnz;
    v->col_block = cb;
    v->dtype = csr->dtype;
    v->n_groups = G;
    v->perm.assign(perm, perm + M);
    v->row_groups.assign(rg, rg + G + 1);

    // B rows are gathered in granules of 2^lg_gran consecutive rows: the largest power of two
    // that divides the block width, at most one K-step.
    int lg = 0;
    while (lg < 5 && cb % (2 << lg) == 0) ++lg;
    v->lg_gran = lg;
    gran = 1 << lg;
    per_step = kStepK >> lg;             // krow entries per K-step
    int64_t short_rows = 0;
    for (int32_t g = 0; g < G; ++g)
        if (rg[g + 1] - rg[g] < kSlabRows) short_rows += rg[g + 1] - rg[g];
    panels_on = use_panels(lg, short_rows);

    index_blocks();
    if (entries_cost_less()) {
        keep_entries();
        lay_out();
        return VBR_OK;
    }
    int rc = block_tiles();
    if (rc != VBR_OK) return rc;
    v->row_pos.assign((size_t)M, -1);
    order_low_rows();
    choose_panels();
    for (int64_t c = 0; c < (int64_t)v->chunk_panel.size(); ++c)
        if (v->chunk_panel[(size_t)c] >= 0) {
            rc = emit_panel(c);
            if (rc != VBR_OK) return rc;
        }
    append_gathered_groups();
    cut_into_tiles();
    rc = emit_gather_tiles();
    if (rc != VBR_OK) return rc;
    fill_values();
    schedule();
    stream();
    lay_out();
    return VBR_OK;
}

// The VBR index arrays, and what becomes of every group.
void Builder::index_blocks()
{
    // stretches of groups of about the same number of entries
    const int64_t want = std::max<int64_t>(1, (csr->nnz + M) / (8 * team.size()));
    pieces.clear();
    int64_t load = 0;
    for (int32_t g = 0; g < G; ++g) {
        if (pieces.empty() || load >= want) {
            if (!pieces.empty()) pieces.back().g1 = g;
            pieces.push_back(Piece{g, G, {}, 0});
            load = 0;
        }
        load += nnz_of(rg[g], rg[g + 1]) + (rg[g + 1] - rg[g]);
    }
    kind.assign((size_t)G, kLow);
    v->blk_ptr.assign((size_t)G + 1, 0);
    each((int64_t)pieces.size(), 1, [&](Scratch &s, int64_t i) {
        Piece &pc = pieces[(size_t)i];
        for (int32_t g = pc.g0; g < pc.g1; ++g) {
            const size_t at = pc.blocks.size();
            for (int64_t q = rg[g]; q < rg[g + 1]; ++q) {
                const int64_t r = perm[q];
                int64_t last = -1, end = 0;             // the columns rise: one division per block, not per entry
                for (int64_t p = csr->row_ptr[r]; p < csr->row_ptr[r + 1]; ++p) {
                    const int64_t c = csr->col_idx[p];
                    if (c < end) continue;
                    last = c / cb;
                    end = (last + 1) * cb;
                    if (s.block_pos[last] < 0) { s.block_pos[last] = 0; pc.blocks.push_back((int32_t)last); }
                }
            }
            std::sort(pc.blocks.begin() + (std::ptrdiff_t)at, pc.blocks.end());
            for (size_t k = at; k < pc.blocks.size(); ++k) s.block_pos[pc.blocks[k]] = -1;
            const int64_t nb = (int64_t)(pc.blocks.size() - at);
            v->blk_ptr[(size_t)g + 1] = nb;
            kind[g] = kind_of(s, rg[g], rg[g + 1], nb);
        }
    });
    for (int32_t g = 0; g < G; ++g) v->blk_ptr[(size_t)g + 1] += v->blk_ptr[g];
    std::vector<int64_t> first_off((size_t)pieces.size() + 1, 0);
    for (size_t i = 0; i < pieces.size(); ++i) {
        pieces[i].first_block = v->blk_ptr[pieces[i].g0];
        int64_t area = 0;
        for (int32_t g = pieces[i].g0; g < pieces[i].g1; ++g) area += (v->blk_ptr[g + 1] - v->blk_ptr[g]) * (int64_t)(rg[g + 1] - rg[g]) * cb;
        first_off[i + 1] = first_off[i] + area;
    }
    v->blk_col.resize((size_t)v->blk_ptr[G]);
    v->blk_off.resize((size_t)v->blk_ptr[G] + 1);
    v->blk_off[0] = 0;
    each((int64_t)pieces.size(), 1, [&](Scratch &, int64_t i) {
        Piece &pc = pieces[(size_t)i];
        std::copy(pc.blocks.begin(), pc.blocks.end(), v->blk_col.begin() + pc.first_block);
        int64_t off = first_off[(size_t)i];
        for (int32_t g = pc.g0; g < pc.g1; ++g)
            for (int64_t b = v->blk_ptr[g]; b < v->blk_ptr[g + 1]; ++b) v->blk_off[(size_t)b + 1] = off += (int64_t)(rg[g + 1] - rg[g]) * cb;
        std::vector<int32_t>().swap(pc.blocks);
    });
    // A few groups with far more K-steps than the others set the time of a small matrix: gathered, their tiles can be deep.
    int64_t total = csr->nnz / (2 * kStepK);
    for (int32_t g = 0; g < G; ++g)
        if (kind[g] == kBlocks) total += steps_of((v->blk_ptr[g + 1] - v->blk_ptr[g]) * cb);
    for (int32_t g = 0; g < G; ++g) {
        if (kind[g] == kBlocks && steps_of((v->blk_ptr[g + 1] - v->blk_ptr[g]) * cb) >= deep_from(total)) kind[g] = kGathered;
        if (kind[g] == kLow) low_groups.push_back(g);
        if (kind[g] == kGathered) gathered_groups.push_back(g);
    }
}

// Groups lower than a slab join the low rows.  The blocks of a taller group may hold many columns without a single
// entry; when tiles that gather only the columns their rows touch take clearly less time, the group is packed that way.
Builder::Kind Builder::kind_of(Scratch &s, int64_t r0, int64_t r1, int64_t n_blocks)
{
    const int64_t h = r1 - r0, n_ks = steps_of(n_blocks * cb), slabs = (h + kSlabRows - 1) / kSlabRows;
    if (h < kSlabRows) return kLow;
    if (cb % 8 != 0) return kGathered;         // a wave loads 8 B rows of one granule
    const int64_t nt = (slabs + kMaxSlabs - 1) / kMaxSlabs;
    int64_t by_blocks = 0, by_columns = 0;
    for (int64_t t = 0; t < nt; ++t) by_blocks += n_ks * kBlockStepNs[slab_class((int)(slabs / nt + (t < slabs % nt ? 1 : 0)))];
    const int64_t step = kMaxGatherSlabs * kSlabRows;
    for (int64_t q = r0; q < r1; q += step) {
        const int64_t e = std::min(r1, q + step);
        int64_t cols = 0;
        s.begin();
        for (int64_t i = q; i < e; ++i) cols += s.add(csr, perm[i]);
        by_columns += steps_of(cols) * kGatherStepNs[(e - q + kSlabRows - 1) / kSlabRows - 1];
        if (5 * by_columns > 4 * by_blocks) return kBlocks;
    }
    return kGathered;
}

// Entries that share no B rows gain nothing from the matrix unit: a tile loads as many B rows as it has entries, and 16 values
// of fragment for every one of them.  Then the whole matrix is kept as rows of entries (one kernel, one launch).  The tiles
// are priced at tiles of 1 or of 4 slabs in the order of the blocking, or of falling length.  Unstructured matrices of 16
// entries a row, as entries and as tiles, N = 64, 256, 1024: 32768 rows, N = 256 25 and 33 us; 12288 rows 6.0 and 8.2, 9.4 and 11.3,
// 28.9 and 36.2; 8192: 5.9 and 7.8, 7.0 and 9.1, 18.9 and 23.6; 4096: 5.8 and 7.6, 5.9 and 8.1, 10.7 and 12.5; 2048: 5.8 and 6.0, 5.9
// and 7.4, 6.9 and 7.4; of 4 a row: 8192 5.8 and 8.1, 5.9 and 8.6, 13.2 and 13.6; 2048 5.9 and 5.7, 5.8 and 6.0, 5.9 and 6.2.  So
// kEntriesMinRows is not where the two cross, which they do between 1024 and 2048 rows: below it a matrix keeps its tiles all the same.
bool Builder::entries_cost_less()
{
    if (M < kEntriesMinRows) return false;
    const int64_t cost = kEntryPs * csr->nnz + kEntryRowPs * M;
    int64_t blocks = 0, rows = 0, nnz = 0, longest = 0;           // cost of the block tiles; rows and entries of all the others
    std::vector<int32_t> given;
    for (int32_t g = 0; g < G; ++g) {
        if (kind[g] == kBlocks) {
            const int64_t slabs = (rg[g + 1] - rg[g] + kSlabRows - 1) / kSlabRows;
            blocks += (steps_of((v->blk_ptr[g + 1] - v->blk_ptr[g]) * cb) + kTileStartSteps) * ((slabs + kMaxSlabs - 1) / kMaxSlabs) *
                      kBlockStepNs[slab_class((int)std::min<int64_t>(slabs, kMaxSlabs))] * 1000;
            if (blocks > cost) return false;
            continue;
        }
        for (int32_t q = rg[g]; q < rg[g + 1]; ++q) {
            const int64_t n = csr->row_ptr[perm[q] + 1] - csr->row_ptr[perm[q]];
            longest = std::max(longest, n);
            nnz += n;
            given.push_back(perm[q]);
        }
    }
    rows = (int64_t)given.size();
    const int64_t step = kMaxGatherSlabs * kSlabRows, n_tiles = (rows + step - 1) / step;
    // what sharing would have to bring: columns at which tiles of 4 slabs cost as much
    const int64_t most = ((cost - blocks) / (1000 * kGatherStepNs[kMaxGatherSlabs - 1]) - kTileStartSteps * n_tiles) * kStepK;
    std::vector<int32_t> sorted((size_t)rows), at((size_t)longest + 2, 0);
    auto key = [&](int32_t r) { return (size_t)(longest - (csr->row_ptr[r + 1] - csr->row_ptr[r])); };
    for (const int32_t r : given) ++at[key(r) + 1];
    for (size_t k = 0; k <= (size_t)longest; ++k) at[k + 1] += at[k];
    for (const int32_t r : given) sorted[(size_t)at[key(r)]++] = r;
    for (const std::vector<int32_t> *list : {&given, &sorted}) {
        std::atomic<int64_t> cols(0);
        each(n_tiles, 4, [&](Scratch &s, int64_t t) {
            int64_t n = 0;
            s.begin();
            for (int64_t k = t * step; k < std::min(rows, (t + 1) * step); ++k) n += s.add(csr, (*list)[(size_t)k]);
            cols += n;
        });
        if (cols <= most) return false;
    }
    // tiles of one slab, at best without a B row less than there are entries
    return cost < blocks + 1000 * (steps_of(nnz) + kTileStartSteps * (rows / kSlabRows)) * kGatherStepNs[0];
}

void Builder::keep_entries()
{
    v->by_entries = true;
    make_entry_rows(csr, team, v->entries);
    v->ks_ptr.assign((size_t)G + 1, 0);
    v->group_first_tile.assign((size_t)G + 1, 0);
    std::vector<int32_t> pos((size_t)M);
    for (int64_t i = 0; i < M; ++i) pos[(size_t)v->entries.row[(size_t)i].row] = (int32_t)i;
    v->row_pos.resize((size_t)M);
    for (int64_t q = 0; q < M; ++q) v->row_pos[(size_t)q] = pos[(size_t)perm[q]];
}

// K-step gather lists and tiles of the groups that are multiplied block by block.
int Builder::block_tiles()
{
    v->ks_ptr.assign((size_t)G + 1, 0);
    v->group_first_tile.assign((size_t)G + 1, 0);
    for (int32_t g = 0; g < G; ++g) {
        v->ks_ptr[(size_t)g + 1] = v->ks_ptr[g];
        v->group_first_tile[(size_t)g + 1] = v->group_first_tile[g];
        if (kind[g] != kBlocks) continue;
        const int64_t h = rg[g + 1] - rg[g], n_ks = steps_of((v->blk_ptr[g + 1] - v->blk_ptr[g]) * cb);
        const int64_t slabs = (h + kSlabRows - 1) / kSlabRows, nt = (slabs + kMaxSlabs - 1) / kMaxSlabs;
        if (v->ks_ptr[g] + n_ks > INT32_MAX / 64) return VBR_EINVAL;
        v->ks_ptr[(size_t)g + 1] += n_ks;
        v->group_first_tile[(size_t)g + 1] += nt;
        int64_t row = 0;
        for (int64_t t = 0; t < nt; ++t) {
            const int64_t s = slabs / nt + (t < slabs % nt ? 1 : 0);
            TileDesc td;
            td.ks_begin = (int32_t)v->ks_ptr[g];
            td.n_ks = (int32_t)n_ks;
            td.a_off = a_units;
            td.row_begin = (int32_t)(rg[g] + row);
            td.n_rows = (int32_t)std::min<int64_t>(s * kSlabRows, h - row);
            td.n_slabs = (int32_t)s;
            td.group = g;
            a_units += n_ks * tile_kstep_stride(td.n_rows, td.n_slabs) / 8;
            row += td.n_rows;
            v->tiles.push_back(td);
        }
    }
    v->krow.resize((size_t)(v->ks_ptr[G] * per_step));
    each((int64_t)pieces.size(), 1, [&](Scratch &, int64_t i) {
        for (int32_t g = pieces[(size_t)i].g0; g < pieces[(size_t)i].g1; ++g) {
            const int64_t n = (v->ks_ptr[g + 1] - v->ks_ptr[g]) * per_step, Kg = (v->blk_ptr[g + 1] - v->blk_ptr[g]) * cb;
            int32_t *out = v->krow.data() + v->ks_ptr[g] * per_step;
            for (int64_t e = 0; e < n; ++e) {
                const int64_t k = std::min(e * gran, Kg - gran);      // the last K-step is filled up with the last granule (times zeros)
                out[e] = (int32_t)((int64_t)v->blk_col[(size_t)(v->blk_ptr[g] + k / cb)] * cb + k % cb);
            }
        }
    });
    return VBR_OK;
}

// The order of the low rows in the row list is free (C is written through the list).  Tiles cut from a list in
// which rows with similar columns follow each other gather far fewer B rows.
void Builder::order_low_rows()
{
    if (!hubs_first()) cluster_low_groups();
    low_slabs = ((int64_t)v->prow.size() + kSlabRows - 1) / kSlabRows;
    v->panel_slabs = low_slabs > 0 ? kPanelSlabs : 0;
}

// Graphs with hubs: the longer a row, the more of its columns are those of the next longer one.  Where tiles of 64
// rows share at least a fifth more in the order of falling length than in the order of the blocking, that order
// is taken (graph of 16384 nodes: 0.37 gathered B rows per entry, against 0.49).
bool Builder::hubs_first()
{
    std::vector<int32_t> given, sorted;        // positions in perm
    int64_t longest = 0;
    int64_t low_rows = 0, other_rows = 0;
    for (const int32_t g : low_groups) low_rows += rg[g + 1] - rg[g];
    for (const int32_t g : gathered_groups)
        if (v->blk_ptr[g + 1] > v->blk_ptr[g]) other_rows += rg[g + 1] - rg[g];
    // the rows of gathered groups join the order if they are more than a few
    const bool all = 16 * other_rows > low_rows;
    for (int32_t g = 0; g < G; ++g) {
        if (kind[g] == kBlocks || (kind[g] == kGathered && !all)) continue;
        for (int32_t q = rg[g]; q < rg[g + 1]; ++q) {
            given.push_back(q);
            longest = std::max(longest, csr->row_ptr[perm[q] + 1] - csr->row_ptr[perm[q]]);
        }
    }
    const int64_t n = (int64_t)given.size(), step = kMaxGatherSlabs * kSlabRows;
    if (n < kMergeMinSlabs * kSlabRows) return false;
    std::vector<int32_t> at((size_t)longest + 2, 0);
    auto key = [&](int32_t q) { return (size_t)(longest - (csr->row_ptr[perm[q] + 1] - csr->row_ptr[perm[q]])); };
    for (const int32_t q : given) ++at[key(q) + 1];
    for (size_t k = 0; k <= (size_t)longest; ++k) at[k + 1] += at[k];
    sorted.resize((size_t)n);
    for (const int32_t q : given) sorted[(size_t)at[key(q)]++] = q;
    std::atomic<int64_t> shared[2] = {{0}, {0}};
    const int64_t n_tiles = (n + step - 1) / step;
    each(2 * n_tiles, 4, [&](Scratch &s, int64_t i) {
        const std::vector<int32_t> &list = i < n_tiles ? given : sorted;
        const int64_t b = (i % n_tiles) * step;
        int64_t cols = 0;
        s.begin();
        for (int64_t k = b; k < std::min(n, b + step); ++k) cols += s.add(csr, perm[list[(size_t)k]]);
        shared[i / n_tiles] += cols;
    });
    if (5 * shared[1] > 4 * shared[0]) return false;
    v->prow.resize((size_t)n);
    for (int64_t i = 0; i < n; ++i) {
        v->prow[(size_t)i] = perm[sorted[(size_t)i]];
        v->row_pos[(size_t)sorted[(size_t)i]] = (int32_t)i;
    }
    if (all) {
        low_groups.insert(low_groups.end(), gathered_groups.begin(), gathered_groups.end());
        gathered_groups.clear();
    }
    return true;
}

// Otherwise the list is built cluster by cluster: the first group not yet placed
// leads a cluster and takes with it every later group that shares at least half of the smaller
// of the two block sets with the LEADER (overlap coefficient >= 1/2, which unlike the Jaccard
// similarity does not fade when both sets carry noise blocks of their own), and then every later group with
// three quarters of the blocks that most of these have (noisy planted matrix: 187 -> 128 tiles).  This only orders the packing, the
// blocking is the caller's.  Candidates come from an index column block -> low groups.  When
// the first 512 leaders find next to nothing (unstructured matrices), the rest keeps its order.
void Builder::cluster_low_groups()
{
    const int64_t n_low = (int64_t)low_groups.size();
    std::vector<int32_t> order, cluster_first;      // cluster_first: index in `order` of every cluster's leader
    order.reserve((size_t)n_low);
    std::vector<int64_t> inv_ptr((size_t)KB + 1, 0);
    for (const int32_t g : low_groups)
        for (int64_t b = v->blk_ptr[g]; b < v->blk_ptr[g + 1]; ++b) inv_ptr[v->blk_col[b] + 1]++;
    for (int64_t b = 0; b < KB; ++b) inv_ptr[b + 1] += inv_ptr[b];
    std::vector<int32_t> inv((size_t)inv_ptr[KB]);
    {
        std::vector<int64_t> fill(inv_ptr.begin(), inv_ptr.end() - 1);
        for (int64_t i = 0; i < n_low; ++i) {
            const int32_t g = low_groups[i];
            for (int64_t b = v->blk_ptr[g]; b < v->blk_ptr[g + 1]; ++b) inv[fill[v->blk_col[b]]++] = (int32_t)i;
        }
    }
    std::vector<int64_t> first(inv_ptr.begin(), inv_ptr.end() - 1);
    std::vector<uint8_t> placed((size_t)n_low, 0);
    std::vector<int32_t> cnt((size_t)n_low, 0), hit, core, in_cluster((size_t)KB, 0);
    // the groups behind the leader i that share enough of the n given blocks, in rising order
    auto join = [&](int64_t i, const int32_t *blks, int64_t n, auto enough) {
        hit.clear();
        for (int64_t k = 0; k < n; ++k) {
            int64_t &f = first[blks[k]];
            while (f < inv_ptr[blks[k] + 1] && inv[f] <= i) ++f;
            for (int64_t e = f; e < inv_ptr[blks[k] + 1]; ++e) {
                const int32_t j = inv[e];
                if (!placed[j] && cnt[j]++ == 0) hit.push_back(j);
            }
        }
        size_t n_pass = 0;
        for (const int32_t j : hit) {
            const int64_t I = cnt[j];
            cnt[j] = 0;
            if (enough(I, v->blk_ptr[low_groups[j] + 1] - v->blk_ptr[low_groups[j]])) hit[n_pass++] = j;
        }
        std::sort(hit.begin(), hit.begin() + (std::ptrdiff_t)n_pass);
        for (size_t k = 0; k < n_pass; ++k) { placed[hit[k]] = 1; order.push_back(hit[k]); }
    };
    int64_t leaders = 0, followers = 0;
    bool clustering = true;
    for (int64_t i = 0; i < n_low; ++i) {
        if (placed[i]) continue;
        placed[i] = 1;
        cluster_first.push_back((int32_t)order.size());
        order.push_back((int32_t)i);
        if (!clustering) continue;
        const int32_t g = low_groups[i];
        const int64_t li = v->blk_ptr[g + 1] - v->blk_ptr[g];
        const size_t begin = order.size() - 1;
        // (only the groups that join are sorted: the candidates are thousands per leader on an unstructured matrix)
        join(i, v->blk_col.data() + v->blk_ptr[g], li, [&](int64_t I, int64_t lj) { return 2 * I >= std::min(li, lj); });
        if (order.size() - begin >= 4) {
            // what most members have in common is a better leader than the first of them, whose own noise blocks kept others out
            core.clear();
            for (size_t o = begin; o < order.size(); ++o)
                for (int64_t b = v->blk_ptr[low_groups[order[o]]]; b < v->blk_ptr[low_groups[order[o]] + 1]; ++b)
                    if (in_cluster[v->blk_col[b]]++ == 0) core.push_back(v->blk_col[b]);
            size_t n = 0;
            for (const int32_t blk : core) {
                if (2 * (size_t)in_cluster[blk] >= order.size() - begin) core[n++] = blk;
                in_cluster[blk] = 0;
            }
            core.resize(n);
            // ... nor do those stay that came for noise in common (one row too many costs its tile a slab)
            for (const int32_t blk : core) in_cluster[blk] = 1;
            size_t keep = begin + 1;
            for (size_t o = begin + 1; o < order.size(); ++o) {
                size_t I = 0;
                for (int64_t b = v->blk_ptr[low_groups[order[o]]]; b < v->blk_ptr[low_groups[order[o]] + 1]; ++b) I += (size_t)in_cluster[v->blk_col[b]];
                if (4 * I >= 3 * n) order[keep++] = order[o];
                else placed[order[o]] = 0;
            }
            order.resize(keep);
            for (const int32_t blk : core) in_cluster[blk] = 0;
            if (n > 0) join(i, core.data(), (int64_t)n, [&](int64_t I, int64_t) { return 4 * I >= 3 * (int64_t)n; });
        }
        followers += (int64_t)(order.size() - begin) - 1;
        if (++leaders == 512 && followers < 64) clustering = false;
    }
    // A cluster of two slabs' worth of rows or more begins and ends on a slab boundary (the list is
    // padded with -1: positions without a row), so that no slab mixes it with its neighbours.  And no
    // slab gathers more than kSlabMaxCols columns if it can be helped: a group whose columns would
    // take the slab beyond that starts a new slab (unrelated rows add up their columns, and the
    // longest slab of a launch, one workgroup per column tile, is what the launch waits for).
    cluster_first.push_back((int32_t)order.size());
    Scratch &s = scratch[0];
    s.fit(csr->n_cols, KB);
    s.begin();
    int64_t slab_cols = 0;
    auto new_slab = [&]() { s.begin(); slab_cols = 0; };
    auto pad_to_slab = [&]() {
        while (v->prow.size() % kSlabRows != 0) v->prow.push_back(-1);
        new_slab();
    };
    for (size_t c = 0; c + 1 < cluster_first.size(); ++c) {
        int64_t rows = 0;
        for (int32_t o = cluster_first[c]; o < cluster_first[c + 1]; ++o)
            rows += rg[low_groups[order[o]] + 1] - rg[low_groups[order[o]]];
        const bool align = rows >= 2 * kSlabRows;
        if (align) pad_to_slab();
        for (int32_t o = cluster_first[c]; o < cluster_first[c + 1]; ++o) {
            const int32_t g = low_groups[order[o]];
            int64_t fresh = 0;                      // columns of the group the current slab does not hold yet
            for (int64_t q = rg[g]; q < rg[g + 1]; ++q)
                for (int64_t p = csr->row_ptr[perm[q]]; p < csr->row_ptr[perm[q] + 1]; ++p)
                    fresh += s.stamp[csr->col_idx[p]] != s.now;
            if (v->prow.size() % kSlabRows != 0 && slab_cols + fresh > kSlabMaxCols) pad_to_slab();
            for (int64_t q = rg[g]; q < rg[g + 1]; ++q) {
                if (v->prow.size() % kSlabRows == 0) new_slab();      // a new slab begins here
                slab_cols += s.add(csr, perm[q]);
                v->row_pos[(size_t)q] = (int32_t)v->prow.size();
                v->prow.push_back(perm[q]);
            }
        }
        if (align) pad_to_slab();
    }
}

// Which chunks of 8 slabs of low rows are packed as panels.
void Builder::choose_panels()
{
    const int64_t n_prows = (int64_t)v->prow.size(), panel_rows = (int64_t)kPanelSlabs * kSlabRows;
    const int64_t n_chunks = (n_prows + panel_rows - 1) / panel_rows;
    v->chunk_panel.assign((size_t)n_chunks, -1);
    if (!panels_on) return;
    prow_group.assign((size_t)n_prows, -1);
    for (const int32_t g : low_groups)
        for (int64_t q = rg[g]; q < rg[g + 1]; ++q) prow_group[(size_t)v->row_pos[(size_t)q]] = g;
    // loads of the two packings for the chunk (per 256 columns of C)
    std::vector<uint8_t> panel((size_t)n_chunks, 0);
    each(n_chunks, 4, [&](Scratch &s, int64_t c) {
        const int64_t i0 = c * panel_rows, i1 = std::min(n_prows, i0 + panel_rows);
        std::vector<int32_t> blocks;
        int64_t cost_gather = INT64_MAX;                  // the cheaper of tiles of 1 and of 4 slabs
        for (const int64_t slabs : {(int64_t)1, (int64_t)kMaxGatherSlabs}) {
            int64_t cost = 0;
            for (int64_t s0 = i0; s0 < i1; s0 += slabs * kSlabRows) {
                int64_t cols = 0;
                s.begin();
                for (int64_t i = s0; i < std::min(i1, s0 + slabs * kSlabRows); ++i)
                    if (v->prow[(size_t)i] >= 0) cols += s.add(csr, v->prow[(size_t)i]);
                cost += steps_of(cols) * (kTileStepCost + slabs - 1);
            }
            cost_gather = std::min(cost_gather, cost);
        }
        for (int64_t i = i0; i < i1; ++i) {
            if (v->prow[(size_t)i] < 0) continue;
            for (int64_t p = csr->row_ptr[v->prow[(size_t)i]]; p < csr->row_ptr[v->prow[(size_t)i] + 1]; ++p) {
                const int32_t j = csr->col_idx[p] / cb;
                if (s.block_pos[j] < 0) { s.block_pos[j] = 0; blocks.push_back(j); }
            }
        }
        for (const int32_t j : blocks) s.block_pos[j] = -1;
        const int64_t steps = steps_of((int64_t)blocks.size() * cb);
        panel[(size_t)c] = steps > 0 && steps <= kPanelMaxSteps && cost_gather >= steps * kPanelStepCost;
    });
    if (std::count(panel.begin(), panel.end(), (uint8_t)1) < kPanelMinCount) return;
    int32_t n = 0;
    for (int64_t c = 0; c < n_chunks; ++c)
        if (panel[(size_t)c]) v->chunk_panel[(size_t)c] = n++;
}

int Builder::emit_panel(int64_t pn)
{
    const int R = kPanelSlabs;
    const int64_t panel_rows = (int64_t)R * kSlabRows, n_prows = (int64_t)v->prow.size();
    const int64_t i0 = pn * panel_rows, i1 = std::min(n_prows, i0 + panel_rows);
    Scratch &s = scratch[0];
    s.fit(csr->n_cols, KB);
    if (v->p_union_ptr.empty()) v->p_union_ptr.assign(1, 0);
    // union of blocks, and per block the slabs that hold it
    std::vector<int32_t> blocks;
    auto groups_of_chunk = [&](auto f) {
        for (int64_t i = i0; i < i1; ++i)
            if (prow_group[(size_t)i] >= 0) f(i, prow_group[(size_t)i]);
    };
    groups_of_chunk([&](int64_t i, int32_t g) {
        if (i > i0 && prow_group[(size_t)i - 1] == g) return;
        for (int64_t b = v->blk_ptr[g]; b < v->blk_ptr[g + 1]; ++b)
            if (s.block_pos[v->blk_col[b]] < 0) { s.block_pos[v->blk_col[b]] = 0; blocks.push_back(v->blk_col[b]); }
    });
    std::sort(blocks.begin(), blocks.end());
    const int64_t nu = (int64_t)blocks.size();
    for (int64_t u = 0; u < nu; ++u) s.block_pos[blocks[u]] = (int32_t)u;
    std::vector<uint32_t> blk_mask((size_t)nu, 0u);
    groups_of_chunk([&](int64_t i, int32_t g) {
        if (i > i0 && prow_group[(size_t)i - 1] == g && i % kSlabRows != 0) return;
        for (int64_t b = v->blk_ptr[g]; b < v->blk_ptr[g + 1]; ++b) blk_mask[s.block_pos[v->blk_col[b]]] |= 1u << ((i - i0) / kSlabRows);
    });
    v->p_union.insert(v->p_union.end(), blocks.begin(), blocks.end());
    v->p_union_ptr.push_back((int64_t)v->p_union.size());

    PanelDesc pd;
    pd.ks_begin = (int32_t)v->pk_mask.size();
    pd.a_off = a_units;
    pd.row_begin = (int32_t)i0;
    pd.n_rows = (int32_t)(i1 - i0);
    pd.pad = 0;
    pd.meta_begin = (int32_t)(v->pk_meta.size() / (size_t)(1 + per_step));
    const int64_t Ku = nu * cb, T = steps_of(Ku);
    std::vector<int64_t> frag_of((size_t)(T * R), -1);      // [logical step][slab] -> fragment ordinal in the panel, -1
    int64_t n_frags = 0;
    for (int64_t t = 0; t < T; ++t) {
        uint32_t m = 0;
        for (int64_t u = (t * kStepK) / cb; u <= std::min(nu - 1, (t * kStepK + kStepK - 1) / cb); ++u) m |= blk_mask[u];
        // a physical K-step carries at most kPanelMaxFrags fragments: split the rest into repeats
        while (m != 0) {
            uint32_t part = 0;
            int cnt = 0;
            for (int sl = 0; sl < R && cnt < kPanelMaxFrags; ++sl)
                if (m >> sl & 1) { part |= 1u << sl; frag_of[(size_t)(t * R + sl)] = n_frags + cnt; ++cnt; }
            m &= ~part;
            v->pk_mask.push_back(part);
            v->pk_logical.push_back((int32_t)t);
            v->pk_frag.push_back(n_frags);
            n_frags += cnt;
            for (int e = 0; e < per_step; ++e) {
                const int64_t k = t * kStepK + (int64_t)e * gran;
                v->pk_row.push_back(k < Ku ? (int32_t)((int64_t)blocks[k / cb] * cb + k % cb) : -1);
            }
        }
    }
    pd.n_ks = (int32_t)v->pk_mask.size() - pd.ks_begin;
    if ((int64_t)v->pk_mask.size() > INT32_MAX / 64) return VBR_EINVAL;
    // the device's K-step stream: one record per physical step, then the look-ahead padding
    for (int64_t ph = pd.ks_begin; ph < pd.ks_begin + pd.n_ks + (pd.n_ks > 0 ? kPanelMetaPad : 0); ++ph) {
        const int64_t src_ph = std::min<int64_t>(ph, pd.ks_begin + pd.n_ks - 1);
        v->pk_meta.push_back(ph < pd.ks_begin + pd.n_ks ? (int32_t)v->pk_mask[ph] : 0);
        for (int e = 0; e < per_step; ++e) v->pk_meta.push_back(v->pk_row[(size_t)src_ph * per_step + e]);
    }
    // values: one full 16 x 32 fragment per (physical step, present slab).  Only the target
    // position of every entry is noted here; the values are packed once the size of all of them is known.
    for (int64_t i = i0; i < i1; ++i) {
        const int64_t r = v->prow[(size_t)i];
        if (r < 0) continue;
        const int sl = (int)((i - i0) / kSlabRows), mrow = (int)((i - i0) % kSlabRows);
        for (int64_t p = csr->row_ptr[r]; p < csr->row_ptr[r + 1]; ++p) {
            const int64_t c = csr->col_idx[p];
            const int64_t k = (int64_t)s.block_pos[c / cb] * cb + c % cb;
            panel_dst.push_back(a_units * 8 + frag_of[(size_t)((k / kStepK) * R + sl)] * kFragElems +
                                frag_index(mrow, (int)(k % kStepK), kSlabRows));
            panel_src.push_back(p);
        }
    }
    panel_range.emplace_back(a_units, a_units + n_frags * (kFragElems / 8));
    a_units += n_frags * (kFragElems / 8);
    for (int64_t u = 0; u < nu; ++u) s.block_pos[blocks[u]] = -1;
    v->panels.push_back(pd);
    return VBR_OK;
}

// The rows of the taller groups that gather single columns follow the low rows in the row list, every group from a
// slab boundary on and, inside it, the longest rows first.
void Builder::append_gathered_groups()
{
    std::vector<int32_t> pos;
    for (const int32_t g : gathered_groups) {
        while (v->prow.size() % kSlabRows != 0) v->prow.push_back(-1);
        pos.clear();
        for (int32_t q = rg[g]; q < rg[g + 1]; ++q) pos.push_back(q);
        std::stable_sort(pos.begin(), pos.end(), [&](int32_t a, int32_t b) {
            return csr->row_ptr[perm[a] + 1] - csr->row_ptr[perm[a]] > csr->row_ptr[perm[b] + 1] - csr->row_ptr[perm[b]];
        });
        for (const int32_t q : pos) {
            v->row_pos[(size_t)q] = (int32_t)v->prow.size();
            v->prow.push_back(perm[q]);
        }
    }
}

// Cuts the slabs of the row list (those in no panel) into gathered tiles of 1 to 4 consecutive slabs.  A taller tile
// loads a B row once for all its slabs and multiplies it for all of them: what it gains is the columns they share.
// The cut of least estimated time is found stretch by stretch.
//   - Slabs of low rows are joined only where that saves at least a seventh of the gathered rows (joining slabs that
//     share nothing would make fewer, longer workgroups) and there are kMergeMinSlabs of them; or where the tile stays
//     short, so that starting and storing are most of its time, and there are enough of them to fill the chip still: graph
//     of 16384 nodes, 32 edges a node, N = 1024 49.6 -> 39.0 us, 8 edges 30.9 -> 25.5, N = 512 and 2048 within 3 %.  Lists of up to 16
//     K-steps instead of 8: within 2 %, but 8 edges, N = 2048 51 -> 46; from 64 slabs on instead of 512: within 4 %, but 98 edges,
//     N = 1024 70 -> 63.
//   - A tile of more K-steps than a resident workgroup's share of the whole (at N = 2048) would still be at it when the
//     rest is done.  It is "deep": the waves of a workgroup split its K-steps, and four workgroups its 256 columns.
//     In a matrix too small to fill the chip every longer tile is (kSmallSteps: the matrix's K-steps), and not higher than two slabs
//     either (kFewTiles: its tiles before that; 1024 x 1024 with 286 groups, N = 256: 8.2 -> 6.4 us).  Without and with kSmallSteps: 1536
//     x 1536, 32-column blocks, N = 1024 8.6 and 7.4; 4000 rows in groups of 1 to 100, N = 1024 9.2 and 7.8; 3072 x 3072, N = 512 9.8 and
//     12.1.  Without and with kFewTiles, 64-column blocks at 10 %, N = 256, 512, 1024: 2048 x 2048 8.3 and 7.7, 9.1 and 7.9, 15.4 and 8.6;
//     3072 9.8 and 7.9, 15.4 and 10.1, 16.7 and 16.3; 4096 9.8 and 10.0, 14.0 and 13.7, 15.9 and 20.0 (blocks at 5 %: 9.0 and 8.5, 12.3 and
//     9.0, 13.8 and 10.0); 6144 11.7 and 12.7, 14.5 and 20.2, 18.0 and 29.9.  The line at 96 tiles is right where B is narrow or the lists
//     are short; long lists against a wide B would have it at 48: the number of workgroups, and with it N, is what counts, and N is
//     not known here.
void Builder::cut_into_tiles()
{
    const int64_t n_slabs = ((int64_t)v->prow.size() + kSlabRows - 1) / kSlabRows;
    v->slab_tile.assign((size_t)n_slabs, -1);
    // group of slabs of the row list that a tile may not leave: low rows 0, gathered groups 1, 2, ...
    std::vector<int32_t> part((size_t)n_slabs, 0);
    for (size_t i = 0; i < gathered_groups.size(); ++i)
        for (int64_t q = rg[gathered_groups[i]]; q < rg[gathered_groups[i] + 1]; ++q)
            part[(size_t)(v->row_pos[(size_t)q] / kSlabRows)] = (int32_t)i + 1;
    auto in_panel = [&](int64_t sl) { return part[(size_t)sl] == 0 && v->chunk_panel[(size_t)(sl / kPanelSlabs)] >= 0; };
    // columns of the tile of len slabs from slab i on, -1 = not possible
    std::vector<int32_t> cols((size_t)n_slabs * kMaxGatherSlabs, -1);
    // (two at a time, not sixteen: the slabs of a graph's hubs have most of the entries; 4096 nodes, a build 1.02 and 0.88 ms, 16384 the same)
    each(n_slabs, 2, [&](Scratch &s, int64_t i) {
        if (in_panel(i)) return;
        int64_t n = 0;
        s.begin();
        for (int len = 1; len <= kMaxGatherSlabs; ++len) {
            const int64_t sl = i + len - 1;
            if (sl >= n_slabs || part[(size_t)sl] != part[(size_t)i] || in_panel(sl)) break;
            for (int64_t k = sl * kSlabRows; k < std::min((sl + 1) * kSlabRows, (int64_t)v->prow.size()); ++k)
                if (v->prow[(size_t)k] >= 0) n += s.add(csr, v->prow[(size_t)k]);
            cols[(size_t)(i * kMaxGatherSlabs + len - 1)] = (int32_t)n;
        }
    });
    // stretches
    std::vector<std::pair<int64_t, int64_t>> runs;
    for (int64_t i = 0; i < n_slabs;) {
        if (in_panel(i)) { ++i; continue; }
        int64_t e = i + 1;
        while (e < n_slabs && e - i < kSegmentSlabs && part[(size_t)e] == part[(size_t)i] && !in_panel(e)) ++e;
        runs.emplace_back(i, e);
        i = e;
    }
    std::vector<std::vector<uint8_t>> cut(runs.size());     // lengths of the tiles of every stretch, in order
    std::atomic<int64_t> total(0), working(0);              // K-steps, tiles that have any
    auto best_cuts = [&](int64_t deep_steps) {
        total = working = 0;
        each((int64_t)runs.size(), 2, [&](Scratch &, int64_t r) {
            const int64_t b = runs[(size_t)r].first, n = runs[(size_t)r].second - b;
            const bool low = part[(size_t)b] == 0, single = low && low_slabs < kMergeMinSlabs;
            std::vector<int64_t> best((size_t)n + 1, INT64_MAX / 2);
            std::vector<uint8_t> len_of((size_t)n + 1, 0);
            best[0] = 0;
            for (int64_t i = 0; i < n; ++i) {
                int64_t alone = 0;
                for (int len = 1; len <= kMaxGatherSlabs && i + len <= n; ++len) {
                    const int64_t c = cols[(size_t)((b + i) * kMaxGatherSlabs + len - 1)];
                    alone += cols[(size_t)((b + i + len - 1) * kMaxGatherSlabs)];
                    if (len > 1 && (single || (low && 7 * c > 6 * alone && !(steps_of(c) <= kShortSteps && low_slabs >= kShortMinSlabs)))) continue;
                    const int64_t cost = best[(size_t)i] + gather_cost(c, len, deep_steps);
                    if (cost < best[(size_t)(i + len)]) { best[(size_t)(i + len)] = cost; len_of[(size_t)(i + len)] = (uint8_t)len; }
                }
            }
            cut[(size_t)r].clear();
            int64_t steps = 0;
            for (int64_t e = n; e > 0; e -= len_of[(size_t)e]) {
                cut[(size_t)r].push_back(len_of[(size_t)e]);
                const int64_t ks = steps_of(cols[(size_t)((b + e - len_of[(size_t)e]) * kMaxGatherSlabs + len_of[(size_t)e] - 1)]);
                steps += ks;
                working += ks > 0;
            }
            std::reverse(cut[(size_t)r].begin(), cut[(size_t)r].end());
            total += steps;
        });
    };
    best_cuts(INT32_MAX);
    for (const TileDesc &td : v->tiles) total += td.n_ks;
    working += (int64_t)v->tiles.size();
    v->deep_steps = (int32_t)std::min<int64_t>(INT32_MAX, working <= kFewTiles ? (int64_t)kSplitSteps : deep_from(total));
    const int32_t mark = total < kSmallSteps ? (int32_t)std::min<int64_t>(v->deep_steps, kSplitSteps) : v->deep_steps;
    best_cuts(v->deep_steps);
    for (size_t r = 0; r < runs.size(); ++r) {
        int64_t sl = runs[r].first;
        for (const uint8_t len : cut[r]) {
            TileDesc td;
            td.ks_begin = 0;
            td.n_ks = (int32_t)steps_of(cols[(size_t)(sl * kMaxGatherSlabs + len - 1)]);
            td.a_off = 0;
            td.row_begin = (int32_t)(sl * kSlabRows);
            int64_t end = std::min<int64_t>((sl + len) * kSlabRows, (int64_t)v->prow.size());
            while (v->prow[(size_t)end - 1] < 0) --end;                    // padding behind the last row
            td.n_rows = (int32_t)(end - sl * kSlabRows);
            td.n_slabs = (td.n_rows + kSlabRows - 1) / kSlabRows;
            td.group = td.n_slabs <= kMaxDeepSlabs && td.n_ks >= mark ? kTileDeep : kTileGathered;
            for (int k = 0; k < len; ++k) v->slab_tile[(size_t)(sl + k)] = (int32_t)v->gtiles.size();
            v->gtiles.push_back(td);
            sl += len;
        }
    }
}

// Column lists of the gathered tiles: the ascending list of the columns its rows touch, cut into K-steps of 32.  The
// last K-step is filled up with the last column again: its place in the fragments is the first, the others hold zeros.
int Builder::emit_gather_tiles()
{
    int64_t g_ks = 0;
    for (TileDesc &td : v->gtiles) {
        if (g_ks + td.n_ks > INT32_MAX / 64) return VBR_EINVAL;
        td.ks_begin = (int32_t)g_ks;
        td.a_off = a_units;
        g_ks += td.n_ks;
        a_units += td.n_ks * tile_kstep_stride(td.n_rows, td.n_slabs) / 8;
    }
    v->gcol.resize((size_t)(g_ks * kStepK));
    each((int64_t)v->gtiles.size(), 1, [&](Scratch &s, int64_t i) {
        const TileDesc &td = v->gtiles[(size_t)i];
        int32_t *out = v->gcol.data() + (int64_t)td.ks_begin * kStepK, *at = out;
        // of many columns the marks are gone through, of few the columns are sorted: a mark takes about 1 ns, a column 13 to 18 (a build of a graph of 16384 nodes,
        // with all sorted and four tiles at a time, 3.0 and 2.4 ms, of 4096 nodes 1.25 and 0.88)
        const bool marks = 16 * (int64_t)td.n_ks * kStepK > csr->n_cols;
        int64_t n = 0;
        s.begin();
        for (int64_t k = td.row_begin; k < (int64_t)td.row_begin + td.n_rows; ++k) {
            const int64_t r = v->prow[(size_t)k];
            if (r < 0) continue;
            if (marks) {
                n += s.add(csr, r);
                continue;
            }
            for (int64_t p = csr->row_ptr[r]; p < csr->row_ptr[r + 1]; ++p)
                if (s.stamp[csr->col_idx[p]] != s.now) { s.stamp[csr->col_idx[p]] = s.now; *at++ = csr->col_idx[p]; }
        }
        if (marks) {
            for (int32_t c = 0; at < out + n; ++c) {
                *at = c;
                at += s.stamp[c] == s.now;
            }
        } else {
            std::sort(out, at);
        }
        if (at > out) std::fill(at, out + (int64_t)td.n_ks * kStepK, at[-1]);
    });
    return VBR_OK;
}

// The values: one allocation, block tiles' fragments, panels' fragments, gathered tiles' fragments, and one fragment
// of zeros behind the last value (loads that run past a panel's data stay inside, and the
// panel kernel's filler loads read it).  Every tile clears and fills its own part.
void Builder::fill_values()
{
    v->vals.allocate((size_t)a_units * 8 + kFragElems);
    std::fill(v->vals.data() + a_units * 8, v->vals.data() + v->vals.size(), (uint16_t)0);
    const uint16_t *src = static_cast<const uint16_t *>(csr->vals);
    uint16_t *vals = v->vals.data();
    for (const auto &r : panel_range) std::fill(vals + r.first * 8, vals + r.second * 8, (uint16_t)0);
    for (size_t e = 0; e < panel_dst.size(); ++e) vals[panel_dst[e]] = src[panel_src[e]];
    // a row of a tile: entry at place k of the tile's K dimension
    auto place = [&](const TileDesc &td, uint16_t *dst, int64_t stride, int32_t rr, int64_t k) -> uint16_t & {
        const int slab = rr / kSlabRows, m = rr % kSlabRows;
        const int rows = slab == td.n_slabs - 1 ? td.n_rows - slab * kSlabRows : kSlabRows;
        return dst[(k / kStepK) * stride + (int64_t)slab * kFragElems + frag_index(m, (int)(k % kStepK), rows)];
    };
    const int64_t n_block = (int64_t)v->tiles.size();
    each(n_block + (int64_t)v->gtiles.size(), 1, [&](Scratch &s, int64_t i) {
        const TileDesc &td = i < n_block ? v->tiles[(size_t)i] : v->gtiles[(size_t)(i - n_block)];
        const int64_t stride = tile_kstep_stride(td.n_rows, td.n_slabs);
        uint16_t *dst = vals + td.a_off * 8;
        std::fill(dst, dst + td.n_ks * stride, (uint16_t)0);
        if (i < n_block) {
            const int64_t b0 = v->blk_ptr[td.group], b1 = v->blk_ptr[td.group + 1];
            for (int64_t b = b0; b < b1; ++b) s.block_pos[v->blk_col[b]] = (int32_t)(b - b0);
            for (int32_t rr = 0; rr < td.n_rows; ++rr) {
                const int64_t r = perm[td.row_begin + rr];
                int64_t end = 0, shift = 0;
                for (int64_t p = csr->row_ptr[r]; p < csr->row_ptr[r + 1]; ++p) {
                    const int64_t c = csr->col_idx[p];
                    if (c >= end) {
                        const int64_t j = c / cb;
                        end = (j + 1) * cb;
                        shift = ((int64_t)s.block_pos[j] - j) * cb;
                    }
                    place(td, dst, stride, rr, c + shift) = src[p];
                }
            }
            for (int64_t b = b0; b < b1; ++b) s.block_pos[v->blk_col[b]] = -1;
        } else {
            const int32_t *list = v->gcol.data() + (int64_t)td.ks_begin * kStepK;
            for (int64_t k = (int64_t)td.n_ks * kStepK; k-- > 0;) s.pos[list[k]] = (int32_t)k;      // of equal ones the first
            for (int32_t rr = 0; rr < td.n_rows; ++rr) {
                const int64_t r = v->prow[(size_t)td.row_begin + rr];
                if (r < 0) continue;
                for (int64_t p = csr->row_ptr[r]; p < csr->row_ptr[r + 1]; ++p) place(td, dst, stride, rr, s.pos[csr->col_idx[p]]) = src[p];
            }
        }
    });
}

// The tiles as the device holds them, whatever their kind: the longest first, those without a K-step (rows without
// entries) last; a deep tile four times, once for every quarter of a column tile.
void Builder::schedule()
{
    struct Item { int64_t ns; TileDesc td; };
    std::vector<Item> items;
    auto put = [&](TileDesc td) {
        const int c = tile_class(td);
        const int64_t ns = c < kClassDeep ? kBlockStepNs[c] : c == kClassDeep ? kDeepStepNs[td.n_slabs - 1] / 4 : kGatherStepNs[td.n_slabs - 1];
        items.push_back(Item{td.n_ks == 0 ? -1 : (td.n_ks + kTileStartSteps) * ns, td});
    };
    for (const TileDesc &td : v->tiles) put(td);
    for (TileDesc td : v->gtiles)
        for (int quarter = td.group == kTileDeep ? 3 : 0; quarter >= 0; --quarter, --td.group) put(td);
    std::stable_sort(items.begin(), items.end(), [](const Item &a, const Item &b) { return a.ns > b.ns; });
    for (const Item &it : items) {
        v->dev_tiles.push_back(it.td);
        if (it.td.n_ks == 0) continue;
        v->n_work = (int32_t)v->dev_tiles.size();
        v->class_count[tile_class(it.td)]++;
        if (it.td.n_ks >= kSplitSteps) v->long_count[tile_class(it.td)]++;
        if (it.td.group >= kTileDeep) {                              // (of the four of a deep tile the first)
            v->work_steps += it.td.n_ks;
            ++v->work_lists;
            v->longest_list = std::max(v->longest_list, it.td.n_ks);
        }
    }
}

// The schedules of the stream kernel, where all tiles with a K-step are block tiles of one slab and some call takes the kernel (or `schedules` wants them).  The
// groups are dealt to the waves of as few workgroups as hold them, the longest first, each to the wave with the fewest K-steps.  A schedule takes a thread
// some 0.1 us and the device 40 to 300 bytes a K-step, beside 1 KiB of values, so it is made only where what is known before leaves the kernel a chance (65536 rows,
// 8 blocks of 16 a group of 1048576 columns, build on 8 threads 5.3 ms and 17.3 MB, with schedules that no call takes 7.0 and 22.3; 262144 x 16384 25.7 and 69.2, 29.1 and 85.1).
void Builder::stream()
{
    constexpr int kAll = kStreamWaves * kStreamGroups;
    const int64_t T = v->n_work, n_tiles = (T + kAll - 1) / kAll;
    if (T < kStreamMinTiles || v->class_count[0] != T || v->lg_gran < 4 || !v->panels.empty()) return;
    if ((int64_t)v->vals.size() * 2 > kNearBytes || v->n_cols > kStreamMostCols) return;
    // K-steps of a wave in a step: as many as the units of a step have on average (one row tile may have a single unit)
    const int64_t all_units = std::max<int64_t>(n_tiles * kStreamWaves * v->n_cols / (kSlabRows * kStreamWaves * kStreamUnits), 1);
    const int ops = (int)std::min<int64_t>(std::max<int64_t>((v->work_steps + all_units - 1) / all_units, kStreamLeastOps), kStreamMostOps);
    // the last of a row tile's units and the last K-step of a wave come at the earliest
    auto least = [&](int64_t units, int64_t load) { return std::max((units + kStreamWaves * kStreamUnits - 1) / (kStreamWaves * kStreamUnits), (load + ops - 1) / ops) + kStreamAhead + 1; };
    const int64_t most = schedules ? INT64_MAX : stream_most_steps(v, n_tiles, ops);
    if (least(0, (v->work_steps + n_tiles * kStreamWaves - 1) / (n_tiles * kStreamWaves)) > most) return;
    struct Wave { int64_t load; int32_t tiles; int32_t wave; };
    auto heavier = [](const Wave &a, const Wave &b) { return a.load != b.load ? a.load > b.load : a.wave > b.wave; };
    std::vector<Wave> waves;
    for (int32_t w = 0; w < n_tiles * kStreamWaves; ++w) waves.push_back(Wave{0, 0, w});
    std::vector<int32_t> tile_of((size_t)(n_tiles * kAll), -1);
    for (int32_t i = 0; i < T; ++i) {
        std::pop_heap(waves.begin(), waves.end(), heavier);
        Wave w = waves.back();
        waves.pop_back();
        tile_of[(size_t)(w.wave * kStreamGroups + w.tiles)] = i;
        w.load += v->dev_tiles[(size_t)i].n_ks;
        if (++w.tiles == kStreamGroups) continue;
        waves.push_back(w);
        std::push_heap(waves.begin(), waves.end(), heavier);
    }
    const int per = kStepK >> v->lg_gran;
    std::vector<std::vector<StreamRecord>> records((size_t)n_tiles);
    std::vector<std::vector<int32_t>> units((size_t)n_tiles);
    std::vector<int64_t> n_steps((size_t)n_tiles, 0);
    std::atomic<bool> pays(true);
    auto unit_of = [&](int32_t g, int32_t k, int h) {
        return v->krow[(size_t)(v->dev_tiles[(size_t)g].ks_begin + k) * per + (per == 2 ? h : 0)] / kSlabRows + (per == 2 ? 0 : h);
    };
    each(n_tiles, 1, [&](Scratch &s, int64_t t) {
        if (!pays.load(std::memory_order_relaxed)) return;
        std::vector<int32_t> &list = units[(size_t)t];
        int64_t load = 0;
        s.begin();
        for (int l = 0; l < kAll; ++l) {
            if (l % kStreamGroups == 0) load = 0;
            const int32_t g = tile_of[(size_t)(t * kAll + l)], n_ks = g < 0 ? 0 : v->dev_tiles[(size_t)g].n_ks;
            for (int32_t k = 0; k < n_ks; ++k)
                for (int h = 0; h < 2; ++h) {
                    const int32_t u = unit_of(g, k, h);
                    if (s.stamp[(size_t)u] != s.now) { s.stamp[(size_t)u] = s.now; list.push_back(u); }
                }
            load += n_ks;
            if (least((int64_t)list.size(), load) > most) {
                pays.store(false, std::memory_order_relaxed);
                return;
            }
        }
        std::sort(list.begin(), list.end());
    });
    if (!pays.load()) return;
    each(n_tiles, 1, [&](Scratch &s, int64_t t) {
        if (!pays.load(std::memory_order_relaxed)) return;
        const int32_t *group_of = tile_of.data() + t * kAll;
        const std::vector<int32_t> &list = units[(size_t)t];
        for (size_t i = 0; i < list.size(); ++i) s.pos[(size_t)list[i]] = (int32_t)i;
        int32_t n_ks[kAll];
        int64_t frag[kAll];
        for (int l = 0; l < kAll; ++l) {
            if (group_of[l] < 0) continue;
            const TileDesc &td = v->dev_tiles[(size_t)group_of[l]];
            n_ks[l] = td.n_ks;
            frag[l] = td.a_off * 16 >> 10;
        }
        auto unit = [&](int l, int32_t k, int h) { return s.pos[(size_t)unit_of(group_of[l], k, h)]; };
        const int sharers = (int)std::min<int64_t>(n_tiles, kStreamShare);
        n_steps[(size_t)t] = stream_schedule(ops, group_of, n_ks, frag, list, unit, (int)(t % sharers), sharers, records[(size_t)t]);
        if (n_steps[(size_t)t] == 0 || n_steps[(size_t)t] > most) pays.store(false, std::memory_order_relaxed);
    });
    if (!pays.load()) return;
    v->stream_ops = ops;
    int64_t total = 0;
    for (const int64_t n : n_steps) total += n;
    v->stream_steps.reserve((size_t)((total + 2) * 2 * kStreamWaves));
    for (int64_t t = 0; t < n_tiles; ++t) {
        StreamTile st;
        st.first_step = (int32_t)(v->stream_steps.size() / (2 * kStreamWaves));
        st.n_steps = (int32_t)n_steps[(size_t)t];
        for (int l = 0; l < kAll; ++l) {
            const int32_t i = tile_of[(size_t)(t * kAll + l)];
            st.row_begin[l] = i < 0 ? -1 : v->dev_tiles[(size_t)i].row_begin;
        }
        v->stream_tiles.push_back(st);
        v->stream_longest = std::max(v->stream_longest, st.n_steps);
        v->stream_steps.insert(v->stream_steps.end(), records[(size_t)t].begin(), records[(size_t)t].end());
    }
    v->stream_steps.resize(v->stream_steps.size() + 2 * 2 * kStreamWaves, StreamRecord());      // looked up behind the last step, and not used
}

void Builder::lay_out()
{
    DeviceLayout &L = v->lay;
    L.zeros_off = 0;                   // 256 zero bytes the panel kernel reads for padding
    L.tiles_off = 256;
    L.krow_off = align_up(L.tiles_off + (int64_t)v->dev_tiles.size() * (int64_t)sizeof(TileDesc), 256);
    L.perm_off = align_up(L.krow_off + (int64_t)v->krow.size() * 4, 256);
    L.panels_off = align_up(L.perm_off + M * 4, 256);
    L.pk_meta_off = align_up(L.panels_off + (int64_t)v->panels.size() * (int64_t)sizeof(PanelDesc), 256);
    L.prow_off = align_up(L.pk_meta_off + (int64_t)v->pk_meta.size() * 4, 256);
    L.gcol_off = align_up(L.prow_off + (int64_t)(v->by_entries ? v->entries.row.size() * sizeof(EntryRow) : v->prow.size() * 4), 256);
    L.stream_tiles_off = align_up(L.gcol_off + (int64_t)(v->by_entries ? v->entries.bytes() : v->gcol.size() * 4), 256);
    L.stream_steps_off = align_up(L.stream_tiles_off + (int64_t)v->stream_tiles.size() * (int64_t)sizeof(StreamTile), 256);
    L.vals_off = align_up(L.stream_steps_off + (int64_t)v->stream_steps.size() * (int64_t)sizeof(StreamRecord), 256);
    L.total = std::max<int64_t>(256, align_up(L.vals_off + (int64_t)v->vals.size() * 2, 256));
}

}  // namespace
}  // namespace vbrk

int vbrk::build_impl(const vbr_csr_t *csr, const int32_t *perm, const int32_t *row_groups, int32_t n_groups, int32_t col_block, vbr_t **out, bool schedules)
{
    int rc = validate_csr(csr, true);
    if (rc != VBR_OK) return rc;
    if (csr->n_cols % col_block != 0) return VBR_EINVAL;
    const int64_t M = csr->n_rows;
    if ((M > 0 && (!perm || !row_groups)) || !row_groups) return VBR_EINVAL;
    if (n_groups > M || (M > 0 && n_groups == 0)) return VBR_EINVAL;
    if (row_groups[0] != 0 || row_groups[n_groups] != M) return VBR_EINVAL;
    for (int32_t g = 0; g < n_groups; ++g)
        if (row_groups[g + 1] <= row_groups[g]) return VBR_EINVAL;
    std::vector<uint8_t> seen((size_t)M, 0);
    for (int64_t i = 0; i < M; ++i) {
        if (perm[i] < 0 || perm[i] >= M || seen[perm[i]]) return VBR_EINVAL;   // not a bijection
        seen[perm[i]] = 1;
    }
    std::unique_ptr<vbr> v(new vbr());
    rc = Builder(csr, perm, row_groups, n_groups, col_block, v.get(), schedules).build();
    if (rc != VBR_OK) return rc;
    *out = v.release();
    return VBR_OK;
}

extern "C" int vbr_build(const vbr_csr_t *csr, const int32_t *perm, const int32_t *row_groups,
                         int32_t n_groups, int32_t col_block, vbr_t **out)
{
    if (!csr || !out || n_groups < 0 || col_block <= 0) return VBR_EINVAL;
    *out = nullptr;
    try {
        return vbrk::build_impl(csr, perm, row_groups, n_groups, col_block, out, false);
    } catch (const std::bad_alloc &) {
        return VBR_ENOMEM;
    } catch (...) {
        return VBR_EINVAL;
    }
}

extern "C" int vbr_get_index(const vbr_t *v, const int32_t **row_groups, const int32_t **perm,
                             const int64_t **blk_ptr, const int32_t **blk_col, const int64_t **blk_off,
                             int64_t *n_groups, int64_t *n_blocks, int64_t *stored_elems)
{
    if (!v) return VBR_EINVAL;
    if (row_groups) *row_groups = v->row_groups.data();
    if (perm) *perm = v->perm.data();
    if (blk_ptr) *blk_ptr = v->blk_ptr.data();
    if (blk_col) *blk_col = v->blk_col.data();
    if (blk_off) *blk_off = v->blk_off.data();
    if (n_groups) *n_groups = v->n_groups;
    if (n_blocks) *n_blocks = (int64_t)v->blk_col.size();
    if (stored_elems) *stored_elems = v->blk_off.back();
    return VBR_OK;
}

extern "C" int vbr_unpack_block(const vbr_t *v, int64_t blk, void *dst_)
{
    using namespace vbrk;
    if (!v || !dst_ || blk < 0 || blk >= (int64_t)v->blk_col.size()) return VBR_EINVAL;
    const int32_t g = (int32_t)(std::upper_bound(v->blk_ptr.begin(), v->blk_ptr.end(), blk) - v->blk_ptr.begin() - 1);
    const int64_t pos = blk - v->blk_ptr[g];
    const int64_t cb = v->col_block;
    uint16_t *dst = static_cast<uint16_t *>(dst_);
    if (v->by_entries) {
        for (int64_t i = 0; i < v->row_groups[g + 1] - v->row_groups[g]; ++i) {
            const int64_t e = v->row_pos[(size_t)(v->row_groups[g] + i)];
            const int64_t end = v->entries.start[(size_t)e + 1], first = (int64_t)v->blk_col[blk] * cb;
            int64_t at = v->entries.start[(size_t)e], n = end - at;      // the row's first entry in the block
            while (n > 0) {
                const int64_t half = n / 2;
                const bool before = v->entries.get(at + half).col < first;
                at = before ? at + half + 1 : at;
                n = before ? n - half - 1 : half;
            }
            std::fill(dst + i * cb, dst + (i + 1) * cb, (uint16_t)0);
            for (Entry x; at < end && (x = v->entries.get(at)).col < first + cb; ++at) dst[i * cb + x.col - first] = (uint16_t)x.val;
        }
        return VBR_OK;
    }
    if (v->group_first_tile[g] == v->group_first_tile[g + 1]) {
        // the rows of the group sit in the row list, each in a slab of a panel or of a column-gathered tile
        const int64_t h = v->row_groups[g + 1] - v->row_groups[g];
        for (int64_t i = 0; i < h; ++i) {
            const int64_t pi = v->row_pos[(size_t)(v->row_groups[g] + i)], t = v->slab_tile[(size_t)(pi / kSlabRows)];
            if (t >= 0) {
                // the tile's column list rises, its last column may repeat: look every column of the block up
                const TileDesc &td = v->gtiles[(size_t)t];
                const int slab = (int)((pi - td.row_begin) / kSlabRows), m = (int)((pi - td.row_begin) % kSlabRows);
                const int rows = slab == td.n_slabs - 1 ? td.n_rows - slab * kSlabRows : kSlabRows;
                const int32_t *cb0 = v->gcol.data() + (int64_t)td.ks_begin * kStepK, *ce = cb0 + (int64_t)td.n_ks * kStepK;
                const int64_t stride = tile_kstep_stride(td.n_rows, td.n_slabs);
                for (int64_t c = 0; c < cb; ++c) {
                    const int32_t col = (int32_t)((int64_t)v->blk_col[blk] * cb + c);
                    const int32_t *it = std::lower_bound(cb0, ce, col);
                    if (it == ce || *it != col) { dst[i * cb + c] = 0; continue; }      // fill-in: not stored
                    const int64_t k = it - cb0;
                    dst[i * cb + c] = v->vals[(size_t)td.a_off * 8 + (size_t)((k / kStepK) * stride) + (size_t)slab * kFragElems + frag_index(m, (int)(k % kStepK), rows)];
                }
                continue;
            }
            const int64_t pidx = v->chunk_panel[(size_t)(pi / ((int64_t)v->panel_slabs * kSlabRows))];
            const PanelDesc &pd = v->panels[pidx];
            const int s = (int)((pi - pd.row_begin) / kSlabRows), m = (int)((pi - pd.row_begin) % kSlabRows);
            const int32_t *ub = &v->p_union[v->p_union_ptr[pidx]], *ue = &v->p_union[0] + v->p_union_ptr[pidx + 1];
            const int64_t u = std::lower_bound(ub, ue, v->blk_col[blk]) - ub;
            for (int64_t c = 0; c < cb; ++c) {
                const int64_t k = u * cb + c;
                const int32_t t32 = (int32_t)(k / kStepK);
                // physical steps of a logical step are consecutive; take the one that carries slab s
                const int32_t *lb = &v->pk_logical[pd.ks_begin], *le = lb + pd.n_ks;
                int64_t ph = pd.ks_begin + (std::lower_bound(lb, le, t32) - lb);
                while (!(v->pk_mask[ph] >> s & 1)) ++ph;
                const int rank = __builtin_popcount(v->pk_mask[ph] & ((1u << s) - 1u));
                dst[i * cb + c] = v->vals[(size_t)pd.a_off * 8 + (size_t)(v->pk_frag[ph] + rank) * kFragElems +
                                          frag_index(m, (int)(k % kStepK), kSlabRows)];
            }
        }
        return VBR_OK;
    }
    int64_t row = 0;
    for (int64_t t = v->group_first_tile[g]; t < v->group_first_tile[g + 1]; ++t) {
        const TileDesc &td = v->tiles[(size_t)t];
        const int64_t stride = tile_kstep_stride(td.n_rows, td.n_slabs);
        const int rows_last = td.n_rows - (td.n_slabs - 1) * kSlabRows;
        const uint16_t *src = &v->vals[(size_t)td.a_off * 8];
        for (int32_t rr = 0; rr < td.n_rows; ++rr, ++row) {
            const int slab = rr / kSlabRows, m = rr % kSlabRows;
            const int rows = slab == td.n_slabs - 1 ? rows_last : kSlabRows;
            for (int64_t c = 0; c < cb; ++c) {
                const int64_t k = pos * cb + c;
                dst[row * cb + c] = src[(k / kStepK) * stride + (int64_t)slab * kFragElems + frag_index(m, (int)(k % kStepK), rows)];
            }
        }
    }
    return VBR_OK;
}

namespace vbrk {

// Goes through the steps of the stream kernel as it does: every index inside what it indexes; every K-step of every tile once and in order, with the units
// of B in its slots that it takes, written in the step before its operands are read or earlier.  A slot counts as its next unit's from the step on that asks for
// it, so one written while a K-step still reads it shows as a K-step that finds another unit, or one not yet written.
static bool stream_holds(const vbr *v)
{
    constexpr int kStep = 2 * kStreamWaves, kAll = kStreamWaves * kStreamGroups, kZeros = kStreamSlots * kStreamUnitBytes;
    if (v->stream_tiles.empty()) return v->stream_steps.empty();
    if (v->stream_ops < kStreamLeastOps || v->stream_ops > kStreamMostOps || v->stream_steps.size() % kStep != 0) return false;
    if ((int64_t)v->vals.size() * 2 > kNearBytes || v->n_cols > kStreamMostCols || v->lg_gran < 4) return false;
    const int64_t n_steps = (int64_t)v->stream_steps.size() / kStep - 2;      // two more are looked up behind the last
    std::vector<int32_t> tile_at((size_t)v->n_rows, -1);
    for (int32_t i = 0; i < v->n_work; ++i) {
        const TileDesc &td = v->dev_tiles[(size_t)i];
        if (td.group < 0 || td.n_rows != kSlabRows || td.a_off % 64 != 0) return false;
        tile_at[(size_t)td.row_begin] = i;
    }
    int64_t tiles = 0;
    for (const StreamTile &st : v->stream_tiles) {
        if (st.first_step < 0 || st.n_steps < 0 || st.n_steps % kStreamAhead != 0 || st.first_step + (int64_t)st.n_steps > n_steps) return false;
        int32_t done[kAll] = {0}, tile[kAll];
        for (int l = 0; l < kAll; ++l) {
            tile[l] = -1;
            if (st.row_begin[l] < 0) continue;
            if ((int64_t)st.row_begin[l] + kSlabRows > v->n_rows) return false;
            std::swap(tile[l], tile_at[(size_t)st.row_begin[l]]);
            if (tile[l] < 0) return false;
            ++tiles;
        }
        struct Slot { int32_t row = -1, written = -1; } slots[kStreamSlots];
        for (int32_t t = 0; t < st.n_steps; ++t) {
            const StreamRecord *now = v->stream_steps.data() + (int64_t)(st.first_step + t) * kStep, *before = t > 0 ? now - kStep : nullptr;
            for (int e = 0; e < kStreamWaves * v->stream_ops; ++e) {
                const int w = e / v->stream_ops, i = e % v->stream_ops, g = now[2 * w].group(i);
                int32_t at[2], frag[2];
                for (int h = 0; h < 2; ++h) {
                    // (the kernel begins with zeros)
                    at[h] = i > 0 ? now[2 * w + h].slot(i - 1) : before ? before[2 * w + h].slot(v->stream_ops - 1) : kZeros;
                    frag[h] = before ? before[2 * w + h].frag(i) : kStreamNone;
                    if (at[h] < 0 || at[h] > kZeros || at[h] % kStreamUnitBytes != 0) return false;
                }
                if (frag[0] != frag[1] || g > kStreamGroups || g != now[2 * w + 1].group(i) || (frag[0] == kStreamNone) != (g == kStreamGroups)) return false;
                if (g == kStreamGroups) continue;
                const int l = w * kStreamGroups + g;
                if (tile[l] < 0) return false;
                const TileDesc &td = v->dev_tiles[(size_t)tile[l]];
                const int32_t k = done[l]++;
                if (k >= td.n_ks || (uint32_t)frag[0] != (uint32_t)(td.a_off * 16 + (int64_t)k * kFragElems * 2)) return false;
                for (int h = 0; h < 2; ++h) {
                    const int64_t b = (int64_t)(td.ks_begin + k) * kStepK + kSlabRows * h;
                    const int32_t row = v->krow[(size_t)(b >> v->lg_gran)] + (int32_t)(b & ((1 << v->lg_gran) - 1));
                    if (at[h] == kZeros) return false;
                    const Slot &s = slots[at[h] / kStreamUnitBytes];
                    if (s.row != row || s.written > t - (i == 0 ? 2 : 1)) return false;
                }
            }
            for (int i = 0; i < kStep; ++i) {
                // what this step asks for is written kStreamAhead steps later
                const StreamRecord &r = now[i];
                for (int e = 0; e < 2; ++e)
                    if (r.early(e) < -1 || (int64_t)r.early(e) + kSlabRows > v->n_cols) return false;
                if (r.none() == kStreamNone) {
                    if (r.to() != kZeros || r.row() != 0) return false;           // zeros to where the zeros are
                    continue;
                }
                if (r.none() != 0 || r.row() < 0 || r.row() % kSlabRows != 0 || (int64_t)r.row() + kSlabRows > v->n_cols) return false;
                if (r.to() < 0 || r.to() >= kZeros || r.to() % kStreamUnitBytes != 0) return false;
                Slot &s = slots[r.to() / kStreamUnitBytes];
                if (s.written >= t + kStreamAhead) return false;                          // two units at once
                s = Slot{r.row(), t + kStreamAhead};
            }
        }
        for (int l = 0; l < kAll; ++l)
            if (tile[l] >= 0 && done[l] != v->dev_tiles[(size_t)tile[l]].n_ks) return false;
    }
    return tiles == v->n_work;
}

}  // namespace vbrk

// Everything the kernels index with, checked against the sizes of what they index into: a wrong
// entry here would be a device access out of bounds, so the check is plain and complete.
extern "C" int vbr_audit(const vbr_t *v)
{
    using namespace vbrk;
    if (!v) return VBR_EINVAL;
    const int64_t M = v->n_rows, K = v->n_cols;
    const int gran = 1 << v->lg_gran, per_step = kStepK >> v->lg_gran;
    const HostValues &values = v->vals;
    const int64_t n_vals = (int64_t)values.size();
    if ((!v->by_entries && n_vals < kFragElems) || (int64_t)v->perm.size() != M) return VBR_EINVAL;
    for (int64_t i = 0; i < M; ++i)
        if (v->perm[i] < 0 || v->perm[i] >= M) return VBR_EINVAL;
    for (const int32_t e : v->krow)
        if (e < 0 || (int64_t)e + gran > K) return VBR_EINVAL;
    if (v->lg_gran < 3 && !v->krow.empty()) return VBR_EINVAL;      // the kernel takes whole groups of 8 rows
    if ((int64_t)v->krow.size() % per_step != 0) return VBR_EINVAL;
    const int64_t total_ks = (int64_t)v->krow.size() / per_step;
    if (v->lay.krow_off + ((int64_t)v->krow.size() + kWideAhead * per_step) * 4 > v->lay.total) return VBR_EINVAL;
    if (v->n_work < 0 || v->n_work > (int32_t)v->dev_tiles.size()) return VBR_EINVAL;
    int32_t count[kClasses] = {0};
    for (size_t i = 0; i < v->dev_tiles.size(); ++i) {
        const TileDesc &td = v->dev_tiles[i];
        if (td.n_rows < 1 || td.n_slabs != (td.n_rows + kSlabRows - 1) / kSlabRows || td.n_slabs > kMaxSlabs) return VBR_EINVAL;
        if (td.n_ks < 0 || td.ks_begin < 0 || (td.n_ks > 0) != ((int32_t)i < v->n_work)) return VBR_EINVAL;
        if (td.group >= 0) {
            if (td.row_begin < 0 || (int64_t)td.row_begin + td.n_rows > M || (int64_t)td.ks_begin + td.n_ks > total_ks) return VBR_EINVAL;
        } else {
            if (td.group <= kTileDeep - 4 || td.n_slabs > (td.group == kTileGathered ? kMaxGatherSlabs : kMaxDeepSlabs)) return VBR_EINVAL;
            if (td.row_begin < 0 || (int64_t)td.row_begin + td.n_rows > (int64_t)v->prow.size()) return VBR_EINVAL;
            if (((int64_t)td.ks_begin + td.n_ks) * kStepK > (int64_t)v->gcol.size()) return VBR_EINVAL;
        }
        // the fragments of all its K-steps lie inside the values (the zero fragment at the end excluded)
        if (td.a_off < 0 || td.a_off * 8 + (int64_t)td.n_ks * tile_kstep_stride(td.n_rows, td.n_slabs) > n_vals - kFragElems) return VBR_EINVAL;
        if (td.n_ks > 0) ++count[tile_class(td)];
    }
    for (int c = 0; c < kClasses; ++c)
        if (count[c] != v->class_count[c]) return VBR_EINVAL;                                // the plan picks its kernel by these
    const int rec = 1 + per_step;
    if ((int64_t)v->pk_meta.size() % rec != 0) return VBR_EINVAL;
    const int64_t n_rec = (int64_t)v->pk_meta.size() / rec;
    for (int64_t r = 0; r < n_rec; ++r) {
        if ((uint32_t)v->pk_meta[r * rec] >> kPanelSlabs) return VBR_EINVAL;                 // mask of at most 8 slabs
        for (int e = 0; e < per_step; ++e) {
            const int32_t row = v->pk_meta[r * rec + 1 + e];
            if (row < -1 || (row >= 0 && (int64_t)row + gran > K)) return VBR_EINVAL;
        }
    }
    for (const int32_t r : v->prow)
        if (r < -1 || r >= M) return VBR_EINVAL;          // -1: a padding position, never stored
    for (const PanelDesc &pd : v->panels) {
        if (pd.n_rows < 1 || pd.n_rows > kPanelSlabs * kSlabRows) return VBR_EINVAL;
        if (pd.row_begin < 0 || (int64_t)pd.row_begin + pd.n_rows > (int64_t)v->prow.size()) return VBR_EINVAL;
        if (pd.n_ks < 0 || pd.meta_begin < 0) return VBR_EINVAL;
        if (pd.n_ks > 0 && (int64_t)pd.meta_begin + pd.n_ks + kPanelMetaPad > n_rec) return VBR_EINVAL;
        int64_t frags = 0;
        for (int32_t k = 0; k < pd.n_ks; ++k) {
            const uint32_t m = (uint32_t)v->pk_meta[((int64_t)pd.meta_begin + k) * rec];
            const int cnt = __builtin_popcount(m);
            if (cnt < 1 || cnt > kPanelMaxFrags) return VBR_EINVAL;
            frags += cnt;
        }
        for (int32_t k = pd.n_ks; k < pd.n_ks + (pd.n_ks > 0 ? kPanelMetaPad : 0); ++k)
            if (v->pk_meta[((int64_t)pd.meta_begin + k) * rec] != 0) return VBR_EINVAL;      // look-ahead records carry no slab
        if (pd.a_off < 0 || pd.a_off * 8 + frags * kFragElems > n_vals - kFragElems) return VBR_EINVAL;
    }
    if ((int64_t)v->gcol.size() % kStepK != 0) return VBR_EINVAL;
    for (const int32_t c : v->gcol)
        if (c < 0 || c >= K) return VBR_EINVAL;
    if (v->by_entries) {
        const EntryRows &e = v->entries;
        if (!v->dev_tiles.empty() || !v->panels.empty() || (int64_t)e.start.size() != M + 1 || (int64_t)e.row.size() != M) return VBR_EINVAL;
        if (n_vals != 0 || !e.entry || e.start[0] != 0 || e.start[(size_t)M] != e.count) return VBR_EINVAL;
        for (int64_t i = 0; i < M; ++i) {
            const EntryRow &r = e.row[(size_t)i];
            if (r.row < 0 || r.row >= M || r.len < 0 || r.start != e.start[(size_t)i] || r.start + r.len != e.start[(size_t)i + 1]) return VBR_EINVAL;
            if (i > 0 && e.start[(size_t)i + 1] - e.start[(size_t)i] > e.start[(size_t)i] - e.start[(size_t)i - 1]) return VBR_EINVAL;
        }
        if ((e.count + 1) * (e.near ? 4 : (int64_t)sizeof(Entry)) > (int64_t)e.bytes()) return VBR_EINVAL;      // the one behind the last is read, too
        for (int64_t i = 0; i < e.count; ++i)
            if (e.get(i).col < 0 || e.get(i).col >= K) return VBR_EINVAL;
    }
    for (size_t i = v->by_entries ? 0 : (size_t)n_vals - kFragElems; i < (size_t)n_vals; ++i)
        if (values[i] != 0) return VBR_EINVAL;                                               // the zero fragment
    try {
        if (!stream_holds(v)) return VBR_EINVAL;
    } catch (const std::bad_alloc &) {
        return VBR_ENOMEM;
    }
    const DeviceLayout &L = v->lay;
    const int64_t ends[11] = {L.zeros_off + 256, L.tiles_off + (int64_t)v->dev_tiles.size() * (int64_t)sizeof(TileDesc),
                              L.krow_off + (int64_t)v->krow.size() * 4, L.perm_off + M * 4,
                              L.panels_off + (int64_t)v->panels.size() * (int64_t)sizeof(PanelDesc),
                              L.pk_meta_off + (int64_t)v->pk_meta.size() * 4, L.prow_off + (int64_t)(v->by_entries ? v->entries.row.size() * sizeof(EntryRow) : v->prow.size() * 4),
                              L.gcol_off + (int64_t)(v->by_entries ? v->entries.bytes() : v->gcol.size() * 4),
                              L.stream_tiles_off + (int64_t)v->stream_tiles.size() * (int64_t)sizeof(StreamTile),
                              L.stream_steps_off + (int64_t)(v->stream_steps.size() * sizeof(StreamRecord)), L.vals_off + n_vals * 2};
    const int64_t begins[11] = {L.zeros_off, L.tiles_off, L.krow_off, L.perm_off, L.panels_off, L.pk_meta_off, L.prow_off,
                                L.gcol_off, L.stream_tiles_off, L.stream_steps_off, L.vals_off};
    for (int i = 0; i < 11; ++i) {
        if (begins[i] % 256 != 0 || ends[i] > L.total) return VBR_EINVAL;
        if (i + 1 < 11 && ends[i] > begins[i + 1]) return VBR_EINVAL;                         // sections in this order, disjoint
    }
    return VBR_OK;
}

namespace vbrk {

void make_entry_rows(const vbr_csr_t *csr, Team &team, EntryRows &out)
{
    const int64_t M = csr->n_rows;
    // by falling length, by counting (a row has at most n_cols entries)
    int64_t longest = 0;
    for (int64_t i = 0; i < M; ++i) longest = std::max(longest, csr->row_ptr[i + 1] - csr->row_ptr[i]);
    std::vector<int32_t> at((size_t)longest + 2, 0);
    for (int64_t i = 0; i < M; ++i) ++at[(size_t)(longest - (csr->row_ptr[i + 1] - csr->row_ptr[i])) + 1];
    for (int64_t k = 0; k <= longest; ++k) at[(size_t)k + 1] += at[(size_t)k];
    out.row.resize((size_t)M);
    for (int64_t i = 0; i < M; ++i) out.row[(size_t)at[(size_t)(longest - (csr->row_ptr[i + 1] - csr->row_ptr[i]))]++].row = (int32_t)i;
    out.start.resize((size_t)M + 1);
    out.start[0] = 0;
    for (int64_t k = 0; k < M; ++k) {
        EntryRow &r = out.row[(size_t)k];
        r.start = out.start[(size_t)k];
        r.len = (int32_t)(csr->row_ptr[r.row + 1] - csr->row_ptr[r.row]);
        out.start[(size_t)k + 1] = r.start + r.len;
    }
    out.allocate(csr->nnz, csr->n_cols);
    const uint16_t *v = static_cast<const uint16_t *>(csr->vals);
    team.each(M, 256, [&](int64_t b, int64_t e) {
        for (int64_t k = b; k < e; ++k) {
            const int64_t p0 = csr->row_ptr[out.row[(size_t)k].row], to = out.start[(size_t)k], n = out.start[(size_t)k + 1] - to;
            if (out.near) {
                for (int64_t i = 0; i < n; ++i) out.entry[(size_t)(to + i)] = (uint32_t)csr->col_idx[p0 + i] | (uint32_t)v[p0 + i] << 16;
            } else {
                for (int64_t i = 0; i < n; ++i) out.put(to + i, csr->col_idx[p0 + i], v[p0 + i]);
            }
        }
    });
}

// Are the column tiles cut in even shares?  Then a domain meets up to two of those left over and brings parts of B that others bring too, so the
// busiest domain has to get clearly shorter, and a CU of it a workgroup less.  Whole tiles and shares: 16 x 16 blocks, 4096 x 8192, five column
// tiles 40.7 and 38.4 us, nine 81.9 and 62.1, 19: 113.7 and 100.1; 64 x 64 blocks at 30 %, 8192 x 8192, five 58.9 and 53.0, nine 108.6 and 87.7, 11:
// 113 and 100; graph of 16384 nodes, five 67.3 and 65.1, ten 125.8 and 116.4, of 8192 nodes 26.7 and 19.7, 43.9 and 42.6; groups of 50 rows, 5003
// x 4104, five 23.6 and 15.8; panels of 6000 rows, nine 19.9 and 15.0; entry rows, 16384 x 16384, 8 entries a row, five 23.6 and 18.8, nine 43.5 and
// 30.9.  Where the busiest has little more than the others: 14 column tiles 82.4 and 81.5, 120.1 and 118.8, seven 62.4 and 64.7, 65.9 and 67.1, 22:
// 121.5 and 120.4, 181.9 and 183.2; three, where whole tiles have two or three domains each, 34.5 and 37.0, entry rows 15.4 and 16.8.  One round of
// workgroups, 60 tiles, five: 15.1 and 17.1, six: 16.5 and 16.8; 40 tiles, six, 40 and 30 on a domain of 32 CUs: 16.3 and 13.1.
static bool even_columns(int64_t T, int64_t Q)
{
    if (Q <= 4 || Q == 7 || Q % kXcd == 0) return false;
    const int64_t whole = grid_size(T, Q), shares = grid_size(T, Q, true), cus = kTwoOnACu / 2;
    return 8 * whole >= 9 * shares && (whole + cus - 1) / cus > (shares + cus - 1) / cus;
}

// Are T tiles of 3 to 4 slabs for the wide kernel?  Two of its workgroups are resident on a CU, as of the tile kernel's, 64 on an L2 domain; 64 of them take
// 100 where 64 of the tile kernel, with half the columns, take 62, so it is ahead where both come in full rounds; but up to 32, one on a CU, take 77 and
// 50, and a launch of a single round gains less.  So the rounds of the busiest domain are counted.  8192 x 8192, blocks of 64 x 64, 132 K-steps, tile and
// wide kernel: N = 512 51.8 and 64.6 us, 1024 68 and 79, 1536 109 and 99, 2048 128 and 115, 3072 189 and 184, 4096 247 and 201, 6144 378 and 307, 8192 487
// and 396; 42 K-steps: 1024 24.3 and 28.0, 2048 42.0 and 40.5, 4096 86 and 81, 8192 184 and 153; 6144 rows (96 tiles), 98 K-steps: 2048 81 and 77, 3072
// 118 and 133, 4096 150 and 135, 8192 286 and 235; 64 tiles, 68: 4096 65.8 and 66.0, 8192 146 and 113.  Short lists mostly store: 132 tiles, N = 8192,
// 21 K-steps 186 and 163, 11: 136 and 126, 5: 91.3 and 88.9, 3: 71.5 and 71.4; 96 tiles, 1: 42.4 and 43.0.  Tiles have to be of like length: a
// workgroup of the wide kernel takes half as long again for a K-step, which a few long tiles would make the whole launch wait for, all the more
// where they are few and a domain has two column tiles and more at a time (K-steps of the longest and half of all, 40 tiles of 48 rows, 64 and 36, N = 5168: 54.8 and
// 66.1; 37, 124 and 69, 5952: 78.7 and 84.5; 32, 26 and 16, 7456: 26.8 and 28.3; 11 such products 3 % more; 38, 41 of all, 6200: 71.3 and 70.1; 48 tiles, 46 and
// 28, 4608: 40.1 and 37.5).  Against up to 1024
// columns it has nothing to save, A and B stay in the L2 (512 tiles of 33 rows, 5 K-steps, N = 1024: 26.8 and 30.0; 256 of 64, N = 648: 20.5 and 18.5,
// N = 1024: 21.4 and 21.7).  512 columns of more than 12288 rows of B are three times the L2: where tiles ask for them often, half as wide ones stay there better
// (195 tiles of 47 rows, 24 K-steps, 12544 rows, N = 2272: 73.4 and 92.0; 134, 27, 13504, 3072: 69.5 and 80.4; 230, 15, 16272, 3840: 124 and 138; 29 products
// 1.5 % more; 42 that use them up to four times 4 % less).
static bool wide_pays(const vbr *v, int64_t T, int64_t N)
{
    constexpr int64_t kHere = kTwoOnACu / kXcd;
    auto cost = [&](int64_t columns, int64_t full, int64_t half) {
        const int64_t Q = (N + columns - 1) / columns, n = grid_size(T, Q, even_columns(T, Q)) / kXcd, over = n % kHere;
        return n / kHere * full + (over > kHere / 2 ? full : over > 0 ? half : 0);
    };
    const int32_t longest = v->dev_tiles[0].n_ks, median = v->dev_tiles[(size_t)v->n_work / 2].n_ks;
    if (v->n_cols > 12288 && v->work_steps * kStepK > 4 * v->n_cols) return false;
    return N > 1024 && longest >= 4 && 10 * longest <= (T < 44 ? 14 : 20) * median && 10 * (10 + cost(kWideN, 100, 77)) <= 9 * cost(kTileN, 62, 50);
}

// Parts of stream_pays.
static int64_t stream_rounds(int64_t tiles, int64_t N) { return (grid_size(tiles, (N + kStreamN - 1) / kStreamN) / kXcd + 31) / 32; }
static int64_t stream_step_ns(int ops) { return 500 + 117 * ops; }
static int64_t stream_margin(int64_t tiles) { return tiles >= 24 ? 92 : 95; }
static int64_t tile_kernel_ns(const vbr *v, int64_t workgroups) { return 12000 + v->work_steps * workgroups / std::max<int32_t>(v->n_work, 1) * 7 / 10; }

// Is the stream kernel faster than `workgroups` of the kernel of one-slab tiles with a K-step, 256 columns each?  It has one workgroup on a CU, 32 on an L2 domain, which
// all take their steps, whether the round is full or not: that and what goes before and behind, 10 us a round, is its time, 0.5 us a step and 0.117 for
// each K-step of a wave in it.  The other takes 0.7 ns for a K-step of a workgroup, and somewhat longer where rows of B begin inside cache lines, as this one does.
// Tile and stream kernel, 16 x 16 blocks, other operands in every call: 4096 x 16384 at 10 %, N = 4096 163 and 109 us, 3072 126 and 104, 2560 123 and
// 105, unaligned 3504 176 and 121; at 6 % 114 and 87, 89 and 85, 85 and 84, 122 and 100; at 15 % 227 and 136, 174 and 130, 168 and 131, 243 and 148;
// 3072 rows, N = 4096, 10 % 135 and 105; 2048: 91 and 107, at 15 % 121 and 133; 1024: 56 and 124; 8192 x 8192, N = 4096 165 and 113, 2048: 83 and 57;
// 16384 x 8192, N = 1024 82 and 59; 4096 x 8192, N = 4096, 3 % 42.0 and 41.4, 10 %: 86 and 58, 30 %: 215 and 123, 50 %: 343 and 189; two rounds: N = 4160
// 103 and 103, 6144: 135 and 110, 8192: 175 and 121; 5120 rows, N = 4096: 110 and 106; 4096 x 4096, 10 % 49 and 39, 6 %: 37 and 32.  32-column blocks,
// 11200 x 1280 at 62 %, N = 1024 56 and 47, 4104: 222 and 196; short lists, 32768 x 512 at half, N = 512 38.3 and 38.4, 520: 58 and 66.
// The line lies where the estimate wins by 5 %, on the tile kernel's side of some that would gain: of these 2560 at 10 %, 3072 at 6 %, 4096 x 4096 at 6 % and 5120
// rows.  (5500 products drawn over what it takes, 64 to 3000 groups, 256 to 32768 columns, N up to 8192: 36 % less on average, 0.5 % of them more than 2 % slower.)
// Tiles without a K-step cost either kernel the same (64 groups, 10 % of 16384 columns, and 10000 rows without entries, N = 4096 76.7 and 140; 200 groups
// and as many: 164 and 115).
// With 24 row tiles and more the estimate is the least sure (2011 groups at 10 % of 2784 columns, N = 512 33.8 and 37.8; 2354, 15 % of 3904, 2752: 344 and 382; of
// 39 drawn ones between 92 and 95 % nine were slower, on average 3 % faster; of 2725 others six, up to 6 %).
static bool stream_pays(const vbr *v, int64_t N, int64_t ldb, bool aligned, int64_t workgroups)
{
    const int64_t tiles = (int64_t)v->stream_tiles.size();
    if (tiles == 0 || N < kStreamLeastN || b_bytes_of(v->n_cols, ldb, N) > kNearBytes || ldb * 2 >= 1 << 24) return false;
    const int64_t stream_ns = 4000 + stream_rounds(tiles, N) * (10000 + v->stream_longest * stream_step_ns(v->stream_ops)), tile_ns = tile_kernel_ns(v, workgroups);
    return 100 * (aligned ? stream_ns : stream_ns * 9 / 8) < stream_margin(tiles) * (aligned ? tile_ns : tile_ns * 7 / 6);
}

// The most steps that the longest of `tiles` row tiles may take for stream_pays to hold for any N and ldb: of the columns that make as many workgroups of the tile kernel
// the fewest, rows of B not aligned.  Beyond 64 column tiles by the rounds that the workgroups fill; fewer steps with every further one.
static int64_t stream_most_steps(const vbr *v, int64_t tiles, int ops)
{
    int64_t most = 0;
    for (int64_t Qt = 2; Qt <= 64; ++Qt) {
        const int64_t N = std::max<int64_t>(kStreamLeastN, (Qt - 1) * kTileN + 8);
        if (b_bytes_of(v->n_cols, N, N) > kNearBytes) break;
        const bool last = Qt == 64;
        const double rounds = last ? (double)tiles * (double)(4 * Qt - 3) / (32 * kXcd) : (double)stream_rounds(tiles, N);
        const double tile_ns = (double)tile_kernel_ns(v, last ? v->n_work * (Qt + kXcd - 1) : grid_size(v->n_work, Qt)) * 7 / 6;
        const double stream_ns = tile_ns * (double)stream_margin(tiles) / 100 * 8 / 9 + 2;
        most = std::max(most, (int64_t)(((stream_ns - 4000) / rounds - 10000) / (double)stream_step_ns(ops)));
    }
    return most;
}

EntryLaunch plan_entry_rows(const std::vector<int64_t> &start, int64_t n_cols, int64_t N, bool aligned)
{
    const int64_t M = (int64_t)start.size() - 1, nnz = start[(size_t)M];
    EntryLaunch L;
    // Columns a wave.  What counts is whether a part of B that wide stays in the 4 MB of a domain's L2 and how often its rows are used, how the column
    // tiles fall on the domains, and where rows of B begin inside cache lines the pieces that lie in one line more: 2 lines for 64 columns, 3 for 128, 5
    // for 256; wider ones also ask for the rows and entries of A less often.  Found on 12300 products, uniform matrices, graphs and blocks, 1000 to 33000
    // rows of A and of B, 2 to 2000 entries a row, N = 72 to 8192; what is taken is 1.3 % slower than the best of the three on average, more than 14 %
    // for one in fifty, and the same on 4100 others.  Times for 64, 128 and 256 columns in us; rows of A x of B, entries a row:
    //  - unaligned, up to 256: one column tile (20368 x 2496, 309, N = 80: 97, 70, 108; 23728 x 23712, 15, N = 136: 17.6, 18.4, 14.9; 24112 x 24096,
    //    134, N = 144: 94, 99, 73), but two for short rows where the second is three quarters full (15328 x 15328, 6, N = 240: 128 columns 9.8, 256
    //    10.6; 26016 x 26016, 21, N = 216: 35.0 and 32.7);
    //  - 128 columns of B do not stay, and each of its rows is used five times and more: 64 (aligned 22968 x 22944, 19, N = 512: 32.7, 37.3, 53.4;
    //    24272 x 24256, 98, N = 696: 165, 221, 313; unaligned 23720 x 23712, 26, N = 1760: 187, 225, 311), but not where the two take the same or 64
    //    take more: aligned beyond 1024 columns (24240 x 24224, 5, N = 2048: 124, 100, 98), unaligned up to 512, or used less (24104 x 24096, 3, N =
    //    2080: 98.8, 86.7, 86.6);
    //  - aligned, up to 256: 64 (on average 5 % less than 128 for short rows, 4 to 40 % for long ones), but for long rows from 2^27 products on, where
    //    128 take up to 10 % less.  Long rows, N = 264 to 448: 64, of which the domains have even shares (20064 x 8320, 352, N = 312: 200, 242, 268;
    //    6832 x 11584, 648, N = 480: 255, 192, 191);
    //  - long rows, as many column tiles of 256 for every domain (unaligned, one fewer, too), and entries enough for their waves: 256 (graph of 8192 nodes,
    //    33, N = 1936: 79, 66, 56; 16384, 20, N = 4016: 239, 191, 181; 4096, 45, N = 1832: 54, 49, 36; 8192, 31, N = 1640: 67, 63, 52; two fewer 4096, 23, N =
    //    3432: 52, 48, 56; one more 16384, 28, N = 2272: 166, 133, 136; 120000 entries, aligned, 16384, 7, N = 4096: 128 columns 103, 256 116);
    //  - long rows, unaligned, none much longer than the others, of a B of which 128 columns stay: 256 take 5 to 10 % less beyond 384 columns (8560 x 6304,
    //    210, N = 648: 168, 142, 118; 2072 x 2048, 278, N = 2552: 179, 143, 123), but as much or up to 15 % more for 5, 9 and, nearly full, 6 column tiles of
    //    128 (N = 520 to 640, 1032 to 1152 and 712 to 768); with one much longer than the others they take 10 % more;
    //  - else 128 (27456 x 4864, 6, aligned, N = 304: 15.5, 13.1, 17.1; 23656 x 4576, 7, unaligned, N = 744: 32.0, 27.7, 35.3).
    const int64_t longest = M > 0 ? start[1] : 0, work = nnz * N, tiles64 = (N + 63) / 64, tiles128 = (N + 127) / 128, tiles256 = (N + 255) / 256;
    const bool all_short = longest <= kEntryLongRow && nnz <= 32 * M, stays = n_cols * 256 <= 4 << 20, often = nnz >= 5 * n_cols;
    const bool alike = longest * M <= 4 * nnz, many = work >= (int64_t)1 << 27;
    if (N <= 64) L.lanes = 8;
    else if (!aligned && N <= 256) L.lanes = N <= 128 || (all_short && N >= 224) ? 16 : 32;
    else if (!stays && often && (aligned ? N <= 1024 : N > 512)) L.lanes = 8;
    else if (aligned && (tiles64 <= 4 ? all_short || !many : tiles64 < 8 && !all_short)) L.lanes = 8;
    else if (!all_short && (tiles256 % kXcd == 0 || (!aligned && tiles256 % kXcd == kXcd - 1)) && nnz >= (aligned ? 3 << 16 : 1 << 17)) L.lanes = 32;
    else if (!all_short && !aligned && alike && stays && many && N > 384 && tiles128 != 5 && tiles64 != 12 && tiles128 != 9) L.lanes = 32;
    else L.lanes = 16;
    // The loads of a row follow each other, the more of them the more lanes it has: fewer lanes where the longest row has too many of the loads of a SIMD
    // (1024 SIMDs, 512 columns of one entry a load; graph of 16384 nodes, 7 entries a row and 1610 in the longest, aligned, N = 480: 15, 23, 33 us; of
    // 4096 nodes, 12 and 1000, N = 200: 11, 17, 35; 2816 x 2816, 210 and 261, N = 80: 10.7, 14.3, 16.8).  128 and 64 columns take the same, aligned, where
    // it has 0.4 of them; unaligned, where 64 columns bring more lines, where it has half of them, or 1.2 if the others are hardly shorter.
    const int64_t tenths = aligned ? 4 : alike ? 12 : 5;
    while (L.lanes > 8 && !all_short) {
        const int64_t tiles = (N + 8 * L.lanes - 1) / (8 * L.lanes);
        const int64_t loads = longest <= kEntryLongRow ? longest : longest * L.lanes / (longest > std::max<int64_t>(kEntryHugeRow, nnz * tiles / 4096) ? 256 : 64);
        if (10 * loads * 1024 * 512 <= tenths * work) break;
        L.lanes /= 2;
    }
    const int64_t width = 8 * L.lanes, Q = (N + width - 1) / width;
    // A workgroup for a row costs its barrier and the fourfold sum; it pays where one wave would still be at the row when
    // the rest is done, i.e. beyond the share of all entries that one of 4096 waves takes (graph, N = 256: 66 -> 26 us;
    // a matrix whose rows all have 1638 entries is 20 % slower with it and stays without).
    auto longer_than = [&](int64_t len) {
        int64_t lo = 0, hi = M;
        while (lo < hi) {
            const int64_t mid = (lo + hi) / 2;
            if (start[(size_t)mid + 1] - start[(size_t)mid] > len) lo = mid + 1;
            else hi = mid;
        }
        return lo;
    };
    L.n_huge = (int32_t)longer_than(std::max<int64_t>(kEntryHugeRow, nnz * Q / 4096));
    L.n_long = (int32_t)longer_than(kEntryLongRow) - L.n_huge;
    const int64_t groups = 64 / std::max(L.lanes, 16), sets = (M - L.n_huge - L.n_long + groups - 1) / groups;
    L.waves = 4 * (int64_t)L.n_huge + L.n_long + sets;
    const int64_t T = (L.waves + 3) / 4;
    L.even = even_columns(T, Q);
    L.grid = grid_size(T, Q, L.even);
    // Rows of very different length, many of them long: the waves of the long ones load without a break and need no others beside them, and fewer at a time
    // ask for fewer rows of B in the L2 and leave the load path to those that take longest.  Eight, six and five workgroups on a CU: graph of 4096 nodes,
    // 39 edges a node, N = 2720 44.9, 40.8, 38.3 us; 94, 3408: 81.8, 77.1, 74.4; of 8192, 96, 256: 16.8, 16.4, 15.6; of 16384, 84, 256: 29.5, 28.1, 28.9; 34
    // graphs of 24 edges and more 2.7 % less with six (worst 3 % more) and 2 with five, of fewer edges 0 and 5 % more; like rows 1 % less and the
    // same; short rows 3 and 11 % more.  Waves of 128 and 256 columns ask for two and four times as much of B; with a row for a workgroup, six pay from 12
    // entries on (16384 nodes, eight and six: 14 edges, N = 736 36.1 and 28.3, 760 42.9 and 32.9; 18, 736: 36.7 and 30.7; 8192, 18, 2792: 65.7 and 62.4;
    // 4096, 17, 2152: 28.3 and 24.3; 70 graphs of 12 to 24 edges 4 % less, worst 3 % more).
    L.six = !alike && ((longest > kEntryLongRow && nnz >= 24 * M) || (L.lanes > 8 && longest > kEntryHugeRow && nnz >= 12 * M));
    // Rows of like length that are all resident begin at the low columns of A together.  Where a part of B as wide as a wave does not stay in the L2 and each of its
    // rows is used only now and then, they find rows of B there that others asked for just before as long as they keep step, which waves do that wait for
    // all of their loads now and then, and not those that never stop (8192 x 32768, 128 a row, N = 200: 1.72 and 2.25 million misses, 34.3 and 40.3 us;
    // 4096 x 32768, 256, 200: 33.4 and 39.5; 2520 x 30622, 55, 656: 24.5 and 27.8; 8192 x 65536, 128, 128: 18.3 and 22.4; 5700 x 112012, 182, 128: 23.2 and 27.2;
    // 109 products of uniform matrices 6 % less, worst 8 % more; 400 of block structure, which share more, the same).  Of fewer entries, with rows beyond
    // kEntryLongRow and 64 columns a wave, and with more rows than are resident the two take the same; of a B that stays, or whose rows are used more often, waves
    // that wait take 1 to 6 % more.
    L.together = longest * M <= 2 * nnz && (L.lanes > 8 || longest <= kEntryLongRow) && nnz >= 32 * M && nnz <= 40 * n_cols && n_cols * std::min(width, N) * 2 > 4 << 20 && 4 * L.grid >= kEightOnACu && L.grid <= kEightOnACu;
    return L;
}

}  // namespace vbrk

extern "C" int64_t vbr_device_bytes(const vbr_t *v) { return v ? v->lay.total : 0; }

namespace vbrk {

// The panels, then the tiles: one launch of the kernel of their class, or of the mixed kernel if there are several.
// One launch for all of them, not one per class: the classes' tails fill each other's gaps, and no launch waits for
// another.  Measured against launches side by side on streams of their own, and one behind the other: row groups of 16 to 128
// rows, N = 4096: 169 and 155 -> 137 us; graph of 16384 nodes, N = 4096: 192 and 195 -> 181; of 4096 nodes, N = 2048: 41 and
// 24 -> 20.
// Tiles without a K-step run behind the others, where their stores fill what those leave free.  The kernels of one and two slabs, of which more
// workgroups fit on a CU than of the mixed one, take them themselves (mixed, apart and so: 512 tiles of 16 rows, 40 K-steps, N = 4096, a quarter of the rows
// empty 241, 223 and 217 us, half 249, 239 and 229; 16 K-steps, N = 1024, a quarter 32.1, 31.4 and 29.0, 70 % 41.2, 45.2 and 42.7; 400 of 32 rows, 16
// K-steps, N = 4096, half 143, 149 and 134; on average 10 % less than mixed and 20 % less than apart).  Launches that are split over K stay mixed (two
// slabs, 40 K-steps, N = 256, 128 tiles mixed 9.7 and own kernel 11.2; 16: 7.6 and 5.9), and so do tall tiles, for which the mixed kernel is as good
// as their own (64 and 128 rows, 2 to 70 % empty: 0.3 and 1.3 % slower on average; 40 tiles of 64 rows, 40 K-steps, N = 4096 34.8 and 45.7), and tiles of a
// single K-step, which mostly store (70 tiles, N = 8200, 16 without a K-step: mixed 23.2, apart 23.5, own kernel 21.9).  Only where those without a K-step
// are many, but less than a quarter of the others, the two ways take nearly the same and they have a launch of the kernel that just stores zeros (in the
// launch of the others and apart: graphs of 16384 nodes, 32 edges a node, N = 4096 176 and 177, N = 3000 147 and 148, 64 edges 217 and 221, 198 and
// 196, of 8192 nodes, 16 edges, N = 4096 48 and 53; more than a quarter: 16384 nodes, 8 edges, N = 4096 94 and 101, N = 2048 44 and 49.  With few of them
// a launch of its own takes 3 us more).
int plan_launches(const vbr *v, int64_t N, bool aligned, Launch out[VBR_MAX_LAUNCHES], int64_t ldb)
{
    int n = 0;
    if (v->by_entries) {
        const EntryLaunch L = plan_entry_rows(v->entries.start, v->n_cols, N, aligned);
        out[n++] = Launch{VBR_LAUNCH_ENTRIES, 0, (int32_t)v->n_rows, L.grid};
        return n;
    }
    const int64_t Qt = (N + kTileN - 1) / kTileN, Qp = (N + kPanelN - 1) / kPanelN;
    if (!v->panels.empty()) {
        const int64_t P = (int64_t)v->panels.size();
        const bool even = even_columns(P, Qp);
        out[n++] = Launch{VBR_LAUNCH_PANEL, 0, (int32_t)P, grid_size(P, Qp, even), 0, false, 0, 0, even};
    }
    static const int32_t kind_of_class[kClasses] = {VBR_LAUNCH_TILE_1, VBR_LAUNCH_TILE_2, VBR_LAUNCH_TILE_4, VBR_LAUNCH_TILE_8, VBR_LAUNCH_TILE_MIXED,
                                                    VBR_LAUNCH_GATHER_1, VBR_LAUNCH_GATHER_2, VBR_LAUNCH_GATHER_4};
    int classes = 0, last = 0;
    for (int c = 0; c < kClasses; ++c)
        if (v->class_count[c] > 0) { ++classes; last = c; }
    const int32_t T_all = (int32_t)v->dev_tiles.size(), T_empty = T_all - v->n_work;
    const bool low_class = classes == 1 && (last < 2 || last == kClassGather || last == kClassGather + 1);
    const bool keeps_kernel = low_class && v->dev_tiles[0].n_ks > 1;
    const bool apart = !keeps_kernel && T_empty * Qt >= kEmptyApart && 4 * T_empty < v->n_work;
    const int32_t T = apart || v->n_work == 0 ? v->n_work : T_all;
    // (tiles without a K-step are gathered ones of up to 4 slabs: the kernel of these is the kernel of their class, and the mixed one takes them, too)
    if (T > 0) {
        const bool one_kind = classes == 1 && (T == v->n_work || last == kClasses - 1);
        // Tiles of up to four slabs with long lists whose workgroups leave CUs idle: four workgroups of 64 columns each instead, whose waves split
        // the K-steps.  Two of these fit on a CU, 64 on an L2 domain, and per K-step they take 4 B loads and a fragment per slab for 64 columns
        // where the others take 16 and one per slab for 256, so the gain ends the sooner the taller the tiles are.  With one of a tile's eight
        // workgroups on every domain (N = 512; not split and split, 60 K-steps of 32-column blocks): one slab, 128 tiles 22.9 and 20.8 us, 150:
        // 26.9 and 25.6 (13 K-steps: 10.0 and 9.5; 26, 160: 14.4 and 14.9); two slabs, 104: 24.8 and 25.2 (23: 14.2 and 13.4; 40: 17.9 and 19.1),
        // 128: 25.0 and 27.0; four, 64: 25.7 and 22.8, 68: 25.9 and 33.5, the 64 that are resident being the end.  Where rows of B begin inside a
        // line, 64 columns lie in two (26 K-steps, N = 504): one slab, 84: 12.5 and 11.5, 96: 12.6 and 12.7; two, 64: 13.4 and 10.4, 96: 13.7 and
        // 15.7; four, 56: 14.6 and 13.5, 96: 15.2 and 23.1.  With nine to twelve workgroups a tile the first domains have two and the others one:
        // what is resident counts on those (four slabs, 23 K-steps, N = 640, 30 tiles 12.7 and 9.5, 36: 12.9 and 14.7), but lower tiles gain as
        // long as the domains have less on the whole (two slabs, 64: 14.5 and 11.8, with 40 K-steps 17.8 and 17.9, 80: 14.4 and 15.6; one, 75: 13.5
        // and 11.8, 100: 14.1 and 15.5). With few columns a tile has fewer workgroups (6368 x 5792, 32-column blocks, N = 80, 150 tiles: not split
        // 15.3 us, split, two a tile, 9.5; tiles of 64 rows, 31 K-steps, N = 72: 160 tiles 15.6 and 11.8, 225 15.8 and 13.3, 300 18.0 and 20.7).
        // Tiles of more slabs are not split; where one of them takes longest, splitting the others brings nothing (heights 1 to 100, N = 1000, 80
        // workgroups: 13.9 and 14.9).  A deep tile is split already.
        // Shares of what may be split: per tile, in 4800ths, for one of its workgroups on every domain.
        static constexpr int64_t share_of_class[2][kClasses] = {{48, 64, 75, 100, 12, 48, 64, 75}, {32, 46, 75, 100, 12, 32, 46, 75}};
        // workgroups of a tile on the busiest domain and on all of them, in eighths (one of the mixed kernel beyond the last column ends at once)
        const int64_t Qd = (N + kDeepN - 1) / kDeepN;
        auto busiest = [](int64_t n, int64_t Q) { return Q >= kXcd ? 8 * n * ((Q + kXcd - 1) / kXcd) : 8 * n / (kXcd / Q); };
        const int64_t most = one_kind ? busiest(1, Qd) : Qt == 1 ? Qd : busiest(4, Qt);
        int64_t load = 0, resident = 0, splittable = 0;
        for (int c = 0; c < kClasses; ++c) {
            // Tiles of short lists take a quarter: their workgroups are soon over, and the mixed kernel leaves them whole, one of the four (30 tiles of
            // 64 rows and 30 K-steps among 250 of 32 rows and 5 K-steps, N = 72: not split, all counted, 15.2 us and 9.3; one kernel, N = 256: 10
            // tiles of 30 K-steps among 250 of 3 or 9, two slabs, 14.5 and 8.1, 14.7 and 9.7; 40 among 400, one slab, 13.5 and 9.3, 13.5 and 11.3;
            // 40 among 160, four slabs, 15.1 and 10.4, 15.1 and 13.2).
            const int64_t share = share_of_class[aligned][c] * v->long_count[c] + share_of_class[aligned][c] * (v->class_count[c] - v->long_count[c]) / 4;
            const bool low = c < 2 || c == kClassGather || c == kClassGather + 1;
            load += share * (most + (low ? Qd : most));
            resident += (c == kClassDeep ? v->class_count[c] / 4 : v->class_count[c]) * most;
            if (c != 3 && c != kClassDeep) splittable += v->class_count[c];
        }
        // Lists of four K-steps and more gain whatever the height of the tiles, as long as two workgroups on a CU hold all that result, 64 on a
        // domain.  Not split and split, column blocks of 32 at N = 512 (kernel time; a call from the host takes longer than most of these): one slab, 64
        // tiles of 4 K-steps 5.1 and 3.4 us, 6: 6.0 and 3.7, 10: 7.8 and 4.3; 16 tiles of 10: 7.8 and 3.4; two slabs, 64 tiles, 4: 5.5 and 4.5, 10: 8.2 and
        // 5.2; four, 4: 5.9 and 5.6, 10: 7.8 and 6.9.  Beyond, 96 tiles, 10 K-steps: 7.5 and 6.0, 8.0 and 7.1, 8.0 and 12.2; 4: 5.1 and 5.2, 5.5 and 6.3,
        // 6.0 and 8.1; 128: 7.2 and 6.7, 7.7 and 8.1, 8.5 and 14.1.
        const int32_t longest = v->dev_tiles[0].n_slabs <= 4 && splittable > 0 ? v->dev_tiles[0].n_ks : 0;
        const int32_t split = longest >= kSplitSteps && load <= 16 * 4800 ? kSplitSteps : longest >= kSplitShort && resident <= 8 * 64 ? kSplitShort : 0;
        const int32_t kind = one_kind || (keeps_kernel && !split) ? kind_of_class[last] : VBR_LAUNCH_TILE_MIXED;
        // Deeper rings allow only two workgroups on a CU and shorten the chain of K-steps of each: worth it where all workgroups are resident then
        // and their lists are long.  An L2 domain holds 64, and the busiest has an eighth of the grid: column tiles whose number does not divide by
        // eight do not fall evenly (82 tiles of 41 K-steps, N = 1352, 492 workgroups, 82 of them on one domain: 31.5 us, with two slots 26.8).  Two
        // slots and four, one slab, 512 workgroups: 6 K-steps 7.7 and 8.1 us, 13: 10.7 and 10.5, 19: 12.9 and 12.2, 26: 15.8 and 14.7, 60: 29.7 and
        // 27.4; 576 workgroups, 26: 17.1 and 23.9.  Where the grid leaves a workgroup a CU of its own nothing hides its chain, and short lists gain
        // too.  Groups of 16 to 32 rows, 240 workgroups, N = 512: 4 K-steps 5.7 and 5.7, 5: 6.6 and 6.3, 7: 7.6 and 7.1, 11: 9.1 and 8.5; N = 2048:
        // 5: 6.6 and 6.3, 11: 10.9 and 8.6, 16: 14.6 and 11.1; 320 workgroups, N = 512: 11: 9.7 and 9.6, 16: 11.8 and 11.3, 18: 12.8 and 12.0; groups
        // of 32 to 48 rows: 16: 12.8 and 13.0, 18: 13.7 and 13.5, 23: 15.4 and 14.9.  With deep tiles, whose chain is the longest, up to three
        // rounds, and all workgroups count, since the short ones fill up what is free beside the long (graphs of 4096 to 16384 nodes, 360 to 1448
        // workgroups: 13.1 and 9.7, 42.4 and 32.2, 63 and 52; N = 592, 1416 of them, 236 on the busiest domain: 33.2 and 24.5; 1744: 22.1 and 24.8,
        // 1776: 27.8 and 26.8, 2272: 43.1 and 47.2).
        const int64_t grid = grid_size(T, Qt);             // as if of whole column tiles
        // Beyond, only where the longest list is far longer than the others, five times the average and more, as in graphs with hubs: then its chain is
        // what counts while others fill the chip (nine to twelve column tiles, up to ten rounds, graphs of 4096 nodes, 2144 columns 35.1 and 32.1; 8192, 2592:
        // 48.8 and 44.3; 16384, 2552: 96.9 and 88.9; 86 products 8 % less, none more; up to six, where in addition it takes 3.5 times as long as all
        // lists shared out among the 512 places: 16384 nodes, 816 columns 49.1 and 36.3, 1048 59.8 and 49.7, 1352 58.0 and 54.5, 13 products 18 % less, none
        // more; below that 12 take from 7 % less to 6 % more).  Lists of like length, deep because the matrix is small, lose the places (64 x 64 blocks with
        // noise, two slots and four: 2816 x 4224, 1424 columns 19.6 and 21.5; 3776 x 2880, 824: 23.6 and 25.6; 1728 x 5248, 2432: 18.5 and 20.6; groups of
        // 1 to 100 rows, 1703 x 7440, 2624: 26.8 and 29.1; 65 products 3 % more).  Seven and eight column tiles take the same on average (1664 columns
        // 56.4 and 60.2, 1672: 60.5 and 57.8; 1952: 21.5 and 23.3), as do 13; 14 to 16 take more (3400: 46.0 and 49.3, 3720: 40.6 and 44.4).
        const bool hub = (int64_t)v->longest_list * v->work_lists >= 5 * v->work_steps;
        const bool outlasts = 2 * (int64_t)v->longest_list * kTwoOnACu >= 7 * v->work_steps * Qt;
        const int64_t deep_most = hub && Qt <= 6 && outlasts ? 6 : hub && Qt >= 9 && Qt <= 12 ? 10 : 3;
        const bool few = split || (v->class_count[kClassDeep] > 0 ? T * Qt <= deep_most * kTwoOnACu : grid <= kTwoOnACu && v->dev_tiles[0].n_ks >= (grid <= kTwoOnACu / 2 ? 5 : 18));
        // workgroups an L2 domain holds at once
        const int64_t at_once = (few || v->class_count[3] > 0 || kind == VBR_LAUNCH_TILE_4 ? kTwoOnACu : kind == VBR_LAUNCH_TILE_MIXED || kind == VBR_LAUNCH_GATHER_4 ? kThreeOnACu
                                                                                                                                                                  : kFourOnACu) / kXcd;
        // Six column tiles, the last of them narrow: the domains that would get most of it have little to do, and the others parts of two column tiles for
        // little less than a whole one, which they only take for a round of workgroups less (a sixteenth of a round more is none).  Whole and shares, 72
        // columns in the last, one-slab tiles of 16 x 16 blocks, 128 at once: 235 of them on a domain whole, 177 in shares 62.1 and 66.1 us; 256, 192: 45.1
        // and 47.5; 200, 150: 42.4 and 42.8; a round less: 170, 129: 40.2 and 31.8; graph of 4096 nodes, 229, 174 (64): 26.1 and 21.7; of 16384 nodes, 64
        // edges a node, 361, 273 (96): 98.5 and 90.6, 16 edges, 356, 267: 57.3 and 60.0; all 256 columns: 55.1 and 57.2, 41.4 and 41.4, 35.9 and 29.2,
        // 23.9 and 19.4, 88.1 and 78.3, 51.5 and 49.4.  Tiles of 5 to 8 slabs, which are fewer and of many lengths, gain all the same (row groups of 16 to
        // 128 rows 75.2 and 68.5, of 1 to 100 rows 23.3 and 20.1), and so do five and nine column tiles (80 columns in the last of five: 61.4 and 55.8, 37.7
        // and 36.8, 58.6 and 45.3; 72 of nine: 106 and 81, 102.8 and 102.7, 50.3 and 41.4).
        auto rounds = [&](bool even) { return std::max<int64_t>((grid_size(T, Qt, even) / kXcd - at_once / 16 + at_once - 1) / at_once, 1); };
        const bool narrow_sixth = Qt == 6 && N - 5 * kTileN <= kTileN / 2 && v->class_count[3] == 0 && rounds(false) == rounds(true);
        Launch L{kind, 0, T, 0, split, few, 0, 0, !split && !narrow_sixth && even_columns(T, Qt)};
        if (kind == VBR_LAUNCH_TILE_1 && !split && stream_pays(v, N, ldb ? ldb : N, aligned, grid_size(v->n_work, Qt, L.even))) {
            L.stream = true;
            L.even = false;
            L.grid = grid_size((int64_t)v->stream_tiles.size(), (N + kStreamN - 1) / kStreamN) + (T - v->n_work) * Qt;
        } else if (kind == VBR_LAUNCH_TILE_MIXED) {
            L.whole = split ? 0 : T;
            L.rest = split ? v->n_work : 0;
            // A last round of few workgroups takes as long as a full one.  Where an L2 domain has up to a quarter more than it holds at once (or
            // than it holds in two, three .. rounds), the last tiles, the shortest, are split: their workgroups are over in a third of the time.  Not
            // split and split, groups of 16 to 128 rows (64 workgroups at once), N = 512: 66 on a domain, 10 K-steps 17.8 and 15.2 us, 20: 25.4 and
            // 19.7; 70: 18.7 and 16.2, 25.8 and 22.1; 76: 19.8 and 19.1, 28.2 and 25.5; 84: 20.8 and 21.0, 29.6 and 28.6; 94: 23.4 and 24.2; 132: 32.1
            // and 30.1; 140: 32.7 and 31.2; 152: 33.8 and 34.4; 198: 43.3 and 41.4; groups of up to 64 rows (96 at once): 98: 18.7 and 16.0, 28.1 and
            // 22.5; 108: 20.4 and 17.9; 116: 21.4 and 19.4; 126: 21.9 and 22.0; 216: 34.2 and 33.2; N = 256, 1024, 2048 alike.  With more than eight
            // column tiles a domain has several of them, one behind the other, and the rounds are many: these stay whole.  Tiles without a K-step do not
            // count: they run behind the others and are over at once (66 tiles of 16 to 128 rows and 20 of them, N = 2048, counted and not, 10 K-steps
            // 18.1 and 15.7, 20: 26.7 and 20.8; 76 and 7: 26.9 and 23.6; 114 of up to 64 rows and 22, 10: 20.5 and 18.1).
            if (!split && Qt <= kXcd) {
                const int64_t work = v->n_work, members = kXcd / Qt;
                const int64_t here = L.even ? grid_size(work, Qt, true) / kXcd : (work + members - 1) / members, over = here > at_once ? here % at_once : 0;
                const int64_t last = L.even ? (kXcd * over + Qt - 1) / Qt : over * members;
                const TileDesc &first = v->dev_tiles[(size_t)std::max<int64_t>(work - last, 0)];
                if (over > 0 && 4 * over <= at_once && work > last && first.group > kTileDeep && first.n_slabs <= split_slabs(few) && first.n_ks >= kSplitShort) {
                    L.whole = (int32_t)(work - last);
                    L.rest = (int32_t)last;
                    L.split = kSplitShort;
                }
            }
            L.grid = grid_size(T + 3 * (int64_t)L.rest, Qt, L.even);
        } else if (kind == VBR_LAUNCH_TILE_4 && !split && wide_pays(v, T, N) && b_bytes_of(v->n_cols, ldb ? ldb : N, N) <= kNearBytes) {
            const int64_t Qw = (N + kWideN - 1) / kWideN;
            L.wide = true;
            L.even = even_columns(T, Qw);
            L.grid = grid_size(T, Qw, L.even);
        } else {
            L.grid = grid_size(T, split ? Qd : Qt, L.even);
        }
        out[n++] = L;
    }
    if (T < T_all) out[n++] = Launch{VBR_LAUNCH_ZERO_ROWS, T, T_all - T, (int64_t)(T_all - T) * kMaxGatherSlabs * ((N + kZeroN - 1) / kZeroN)};
    return n;
}

}  // namespace vbrk

extern "C" int vbr_get_launches(const vbr_t *v, int64_t N, int32_t *n_launches, int32_t *kinds, int64_t *tiles, int64_t *workgroups)
{
    if (!v || !n_launches || N < 0) return VBR_EINVAL;
    vbrk::Launch plan[VBR_MAX_LAUNCHES];
    const int n = (N == 0 || v->n_rows == 0) ? 0 : vbrk::plan_launches(v, N, N % 64 == 0, plan);
    *n_launches = n;
    for (int i = 0; i < n; ++i) {
        if (kinds) kinds[i] = plan[i].kind;
        if (tiles) tiles[i] = plan[i].n_tiles;
        if (workgroups) workgroups[i] = plan[i].grid;
    }
    return VBR_OK;
}

extern "C" int vbr_get_launch_functions(const vbr_t *v, int64_t N, const char **names)
{
    if (!v || !names || N < 0) return VBR_EINVAL;
    vbrk::Launch plan[VBR_MAX_LAUNCHES];
    const int n = (N == 0 || v->n_rows == 0) ? 0 : vbrk::plan_launches(v, N, N % 64 == 0, plan);
    for (int i = 0; i < n; ++i) {
        switch (plan[i].kind) {
        case VBR_LAUNCH_PANEL: names[i] = "vbr_spmm_panel_kernel"; break;
        case VBR_LAUNCH_TILE_MIXED: names[i] = "vbr_spmm_mixed_kernel"; break;
        case VBR_LAUNCH_ENTRIES: names[i] = "entry_rows_kernel"; break;
        case VBR_LAUNCH_ZERO_ROWS: names[i] = "vbr_spmm_zero_rows_kernel"; break;
        default: names[i] = plan[i].split ? "vbr_spmm_split_kernel" : plan[i].stream ? "vbr_spmm_stream_kernel" : plan[i].wide ? "vbr_spmm_wide_kernel" : "vbr_spmm_kernel"; break;
        }
    }
    return VBR_OK;
}

extern "C" int vbr_get_schedule(const vbr_t *v, int64_t *n_tiles, int64_t *n_ksteps, int64_t *packed_elems)
{
    if (!v) return VBR_EINVAL;
    if (n_tiles) *n_tiles = v->by_entries ? v->n_rows : (int64_t)v->tiles.size() + (int64_t)v->panels.size() + (int64_t)v->gtiles.size();
    if (n_ksteps) *n_ksteps = v->ks_ptr.back() + (int64_t)v->pk_mask.size() + (int64_t)v->gcol.size() / vbrk::kStepK;
    if (packed_elems) *packed_elems = v->by_entries ? v->entries.count : (int64_t)v->vals.size();
    return VBR_OK;
}

extern "C" int64_t vbr_get_tile_ksteps(const vbr_t *v, int64_t *out, int64_t cap)
{
    if (!v) return VBR_EINVAL;
    const int64_t n = (int64_t)(v->tiles.size() + v->gtiles.size() + v->panels.size());
    if (!out) return n;
    int64_t w = 0;
    for (const vbrk::TileDesc &t : v->tiles) { if (w < cap) out[w] = t.n_ks; ++w; }
    for (const vbrk::TileDesc &t : v->gtiles) { if (w < cap) out[w] = t.n_ks; ++w; }
    for (const vbrk::PanelDesc &t : v->panels) { if (w < cap) out[w] = t.n_ks; ++w; }
    return n;
}

extern "C" void vbr_free(vbr_t *v)
{
    delete v;
}

extern "C" const char *vbr_strerror(int code)
{
    switch (code) {
    case VBR_OK: return "ok";
    case VBR_EINVAL: return "invalid argument";
    case VBR_ENOMEM: return "out of host memory";
    case VBR_EHIP: return "HIP runtime error";
    case VBR_ESTATE: return "call out of order";
    case VBR_EUNSUPPORTED: return "unsupported input";
    default: return "unknown error";
    }
}
