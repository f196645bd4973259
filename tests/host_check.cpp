// Host-side check program for the sanitizer build: the library's host units (1-SA, VBR build, block
// unpacking, blocking curve, bounds audit) linked with the C oracle into one executable compiled with
// -fsanitize=address,undefined, and driven over seeded random matrices.  Every case compares the
// library with the oracle bit for bit and runs the audit of everything the kernels would index, so
// that an out-of-bounds access, an overflow or a leak in 500 lines of hand index arithmetic shows up
// on the CPU.  Test infrastructure: built and run by tests/test_host_sanitizers.py.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <vector>

#include "vbr_host.h"

// Allocations of the thread that sets it: as many succeed as it says, then they fail (negative: all succeed).
static thread_local long g_allocations_left = -1;
static void *allocate(std::size_t n)
{
    if (g_allocations_left == 0) return nullptr;
    if (g_allocations_left > 0) --g_allocations_left;
    return std::malloc(n ? n : 1);
}
void *operator new(std::size_t n)
{
    if (void *p = allocate(n)) return p;
    throw std::bad_alloc();
}
void *operator new(std::size_t n, const std::nothrow_t &) noexcept { return allocate(n); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }
void operator delete(void *p, const std::nothrow_t &) noexcept { std::free(p); }

extern "C" {
int oracle_sa1(int64_t n_rows, int64_t n_cols, const int64_t *row_ptr, const int32_t *col_idx, int32_t col_block,
               double tau, int32_t similarity_only, int32_t *perm, int32_t *row_groups, int32_t *n_groups);
int oracle_vbr_index(int64_t n_rows, int64_t n_cols, const int64_t *row_ptr, const int32_t *col_idx, int32_t col_block,
                     const int32_t *perm, const int32_t *row_groups, int32_t n_groups, int64_t *blk_ptr,
                     int32_t *blk_col, int64_t *blk_off, int64_t *n_blocks);
}

namespace {

struct Rng {
    uint64_t s;
    explicit Rng(uint64_t seed) : s(seed * 0x9E3779B97F4A7C15ull + 1) {}
    uint64_t next() { s ^= s << 13; s ^= s >> 7; s ^= s << 17; return s; }
    double uni() { return (double)(next() >> 11) * (1.0 / 9007199254740992.0); }
    int64_t below(int64_t n) { return (int64_t)(uni() * (double)n); }
};

struct Csr {
    int64_t m = 0, k = 0;
    std::vector<int64_t> row_ptr;
    std::vector<int32_t> col;
    std::vector<uint16_t> val;
    vbr_csr_t view() const
    {
        vbr_csr_t c;
        c.n_rows = m; c.n_cols = k; c.nnz = (int64_t)col.size();
        c.row_ptr = row_ptr.data(); c.col_idx = col.data(); c.vals = val.data(); c.dtype = VBR_F16;
        return c;
    }
};

// rows drawn from `n_base` base patterns over the column blocks, each with a little noise, so that
// identical rows, merges, refusals and the size limit all occur
Csr make(Rng &rng, int64_t m, int64_t kb, int col_block, double density, int n_base)
{
    Csr a;
    a.m = m; a.k = kb * col_block;
    std::vector<std::vector<uint8_t>> base((size_t)n_base, std::vector<uint8_t>((size_t)kb, 0));
    for (auto &b : base)
        for (auto &x : b) x = rng.uni() < density;
    a.row_ptr.push_back(0);
    for (int64_t i = 0; i < m; ++i) {
        const auto &b = base[(size_t)rng.below(n_base)];
        for (int64_t j = 0; j < kb; ++j) {
            const bool on = b[(size_t)j] != (rng.uni() < density * 0.1);
            if (!on) continue;
            for (int c = 0; c < col_block; ++c)
                if (c == 0 || rng.uni() < 0.4) {
                    a.col.push_back((int32_t)(j * col_block + c));
                    a.val.push_back((uint16_t)(1 + rng.below(0x7bff)));
                }
        }
        a.row_ptr.push_back((int64_t)a.col.size());
    }
    return a;
}

int g_cases = 0;
#define REQUIRE(cond) do { if (!(cond)) { std::fprintf(stderr, "host_check: %s failed at line %d (case %d)\n", #cond, __LINE__, g_cases); std::exit(1); } } while (0)

void check_matrix(const Csr &a, int col_block, double tau, bool all_blocks)
{
    ++g_cases;
    const vbr_csr_t c = a.view();
    std::vector<int32_t> perm((size_t)a.m), rg((size_t)a.m + 1), perm0((size_t)a.m), rg0((size_t)a.m + 1);
    int32_t G = 0, G0 = 0;
    REQUIRE(sa1_reorder(&c, col_block, tau, perm.data(), rg.data(), &G) == VBR_OK);
    REQUIRE(oracle_sa1(a.m, a.k, c.row_ptr, c.col_idx, col_block, tau, 0, perm0.data(), rg0.data(), &G0) == 0);
    REQUIRE(G == G0);
    REQUIRE(std::memcmp(perm.data(), perm0.data(), (size_t)a.m * 4) == 0);
    REQUIRE(std::memcmp(rg.data(), rg0.data(), ((size_t)G + 1) * 4) == 0);

    vbr_t *v = nullptr;
    REQUIRE(vbr_build(&c, perm.data(), rg.data(), G, col_block, &v) == VBR_OK);
    REQUIRE(vbr_audit(v) == VBR_OK);
    REQUIRE(vbr_device_bytes(v) >= 256 && vbr_device_bytes(v) % 256 == 0);
    const int32_t *vrg, *vperm, *bcol;
    const int64_t *bptr, *boff;
    int64_t ng, nb, stored;
    REQUIRE(vbr_get_index(v, &vrg, &vperm, &bptr, &bcol, &boff, &ng, &nb, &stored) == VBR_OK);
    const int64_t cap = c.nnz + 1;
    std::vector<int64_t> bptr0((size_t)G + 1), boff0((size_t)cap + 1);
    std::vector<int32_t> bcol0((size_t)cap);
    int64_t nb0 = 0;
    REQUIRE(oracle_vbr_index(a.m, a.k, c.row_ptr, c.col_idx, col_block, perm.data(), rg.data(), G, bptr0.data(),
                             bcol0.data(), boff0.data(), &nb0) == 0);
    REQUIRE(nb == nb0 && ng == G);
    REQUIRE(std::memcmp(bptr, bptr0.data(), ((size_t)G + 1) * 8) == 0);
    REQUIRE(std::memcmp(bcol, bcol0.data(), (size_t)nb * 4) == 0);
    REQUIRE(std::memcmp(boff, boff0.data(), ((size_t)nb + 1) * 8) == 0);
    REQUIRE(stored == boff0[(size_t)nb]);
    // stored blocks read back out of the packed layout = the zero-filled windows of the matrix
    std::vector<uint16_t> got, want;
    for (int32_t g = 0; g < G; ++g) {
        const int64_t h = rg[(size_t)g + 1] - rg[(size_t)g];
        for (int64_t b = bptr[g]; b < bptr[g + 1]; ++b) {
            if (!all_blocks && (b % 7) != 0) continue;
            got.assign((size_t)(h * col_block), 0xffff);
            want.assign((size_t)(h * col_block), 0);
            REQUIRE(vbr_unpack_block(v, b, got.data()) == VBR_OK);
            for (int64_t t = 0; t < h; ++t) {
                const int64_t r = perm[(size_t)(rg[(size_t)g] + t)];
                for (int64_t p = c.row_ptr[r]; p < c.row_ptr[r + 1]; ++p)
                    if (c.col_idx[p] / col_block == bcol[b]) want[(size_t)(t * col_block + c.col_idx[p] % col_block)] = a.val[(size_t)p];
            }
            REQUIRE(got == want);
        }
    }
    int32_t n_launch = 0, kinds[VBR_MAX_LAUNCHES];
    int64_t tiles[VBR_MAX_LAUNCHES], wgs[VBR_MAX_LAUNCHES];
    REQUIRE(vbr_get_launches(v, 264, &n_launch, kinds, tiles, wgs) == VBR_OK && n_launch <= VBR_MAX_LAUNCHES);
    vbr_free(v);
}

// `groups` groups of `rows` rows that all hold the first n_ks * 32 columns, in blocks of 32
vbr_t *stack(int groups, int rows, int n_ks)
{
    Csr a;
    a.m = (int64_t)groups * rows;
    a.k = 32 * n_ks;
    for (int64_t i = 0; i <= a.m; ++i) a.row_ptr.push_back(i * a.k);
    for (int64_t i = 0; i < a.m * a.k; ++i) a.col.push_back((int32_t)(i % a.k));
    a.val.assign(a.col.size(), 0x3c00);
    std::vector<int32_t> perm, rg;
    for (int64_t i = 0; i < a.m; ++i) perm.push_back((int32_t)i);
    for (int g = 0; g <= groups; ++g) rg.push_back(g * rows);
    const vbr_csr_t c = a.view();
    vbr_t *v = nullptr;
    REQUIRE(vbr_build(&c, perm.data(), rg.data(), groups, 32, &v) == VBR_OK);
    return v;
}

// Launches that are planned with two workgroups on a CU: 64 on each of the eight L2 domains, and the busiest counts.
void check_plan()
{
    ++g_cases;
    struct { int groups; int64_t N; bool few; } const cases[] = {{82, 1024, true},  {82, 1280, false}, {82, 1352, false}, {64, 1352, true},
                                                                 {65, 1352, false}, {64, 2048, true},  {65, 2048, false}, {64, 2056, false}};
    for (const auto &x : cases) {
        vbr_t *v = stack(x.groups, 16, 41);
        vbrk::Launch plan[VBR_MAX_LAUNCHES];
        REQUIRE(vbrk::plan_launches(v, x.N, x.N % 64 == 0, plan) == 1 && !plan[0].split);
        REQUIRE(plan[0].few == x.few);
        vbr_free(v);
    }
    // shorter lists: from 5 K-steps on where every workgroup has a CU, from 18 where two share one; not split, more than 64 on a domain
    struct { int groups, n_ks; int64_t N; bool few; } const lists[] = {{32, 5, 2048, true}, {32, 4, 2048, false}, {33, 17, 2048, false}, {33, 18, 2048, true},
                                                                       {64, 18, 2048, true}, {65, 18, 2048, false}, {65, 5, 2048, false}};
    for (const auto &x : lists) {
        vbr_t *v = stack(x.groups, 64, x.n_ks);
        vbrk::Launch plan[VBR_MAX_LAUNCHES];
        REQUIRE(vbrk::plan_launches(v, x.N, true, plan) == 1 && !plan[0].split);
        REQUIRE(plan[0].few == x.few);
        vbr_free(v);
    }
}

// `clusters` stretches of 16 rows, each a group of its own, that hold the same `len` of 4096 columns; before them 16 rows of `hub` columns.
vbr_t *clusters(int n, int len, int hub)
{
    Csr a;
    a.k = 4096;
    a.row_ptr.push_back(0);
    Rng rng(n + len);
    std::vector<int32_t> all(4096);
    for (int i = 0; i < 4096; ++i) all[(size_t)i] = i;
    for (int s = hub ? -1 : 0; s < n; ++s) {
        const int count = s < 0 ? hub : len;
        for (int i = 0; i < count; ++i) std::swap(all[(size_t)i], all[(size_t)(i + rng.below(4096 - i))]);
        std::sort(all.begin(), all.begin() + count);
        for (int r = 0; r < 16; ++r) {
            a.col.insert(a.col.end(), all.begin(), all.begin() + count);
            a.row_ptr.push_back((int64_t)a.col.size());
        }
    }
    a.m = (int64_t)a.row_ptr.size() - 1;
    a.val.assign(a.col.size(), 0x3c00);
    std::vector<int32_t> perm, rg;
    for (int64_t i = 0; i < a.m; ++i) perm.push_back((int32_t)i);
    for (int64_t i = 0; i <= a.m; ++i) rg.push_back((int32_t)i);
    const vbr_csr_t c = a.view();
    vbr_t *v = nullptr;
    REQUIRE(vbr_build(&c, perm.data(), rg.data(), (int32_t)a.m, 32, &v) == VBR_OK);
    return v;
}

// `groups` groups of 64 rows that hold n_ks blocks of 32 columns each, others for every group; the first `first` blocks
vbr_t *blocks_of(int groups, int n_ks, int64_t n_cols, int first)
{
    Csr a;
    a.m = (int64_t)groups * 64;
    a.k = n_cols;
    a.row_ptr.push_back(0);
    std::vector<int32_t> perm, rg = {0};
    for (int g = 0; g < groups; ++g) {
        std::vector<int32_t> cols;
        const int n = g == 0 ? first : n_ks;
        for (int i = 0; i < n; ++i)
            for (int c = 0; c < 32; ++c) cols.push_back((int32_t)((g * 5 + i * (n_cols / 32 / n)) % (n_cols / 32)) * 32 + c);
        std::sort(cols.begin(), cols.end());
        for (int r = 0; r < 64; ++r) {
            a.col.insert(a.col.end(), cols.begin(), cols.end());
            a.row_ptr.push_back((int64_t)a.col.size());
            perm.push_back((int32_t)perm.size());
        }
        rg.push_back((int32_t)perm.size());
    }
    a.val.assign(a.col.size(), 0x3c00);
    const vbr_csr_t c = a.view();
    vbr_t *v = nullptr;
    REQUIRE(vbr_build(&c, perm.data(), rg.data(), groups, 32, &v) == VBR_OK);
    return v;
}

// The wide kernel: not where 512 columns of B are far beyond the L2 and used often, nor where one list is longer than the others, the less of few tiles.
void check_wide()
{
    ++g_cases;
    struct { int groups, n_ks; int64_t n_cols, N; int first; bool wide; } const cases[] = {
        {128, 12, 12288, 4096, 12, true}, {128, 12, 12320, 4096, 12, true}, {128, 13, 12288, 4096, 13, true}, {128, 13, 12320, 4096, 13, false}, {128, 13, 12320, 1024, 13, false},
        {43, 10, 8192, 5632, 14, true}, {43, 10, 8192, 5632, 15, false}, {44, 10, 8192, 5632, 20, true}, {44, 10, 8192, 5632, 21, false}};
    for (const auto &x : cases) {
        vbr_t *v = blocks_of(x.groups, x.n_ks, x.n_cols, x.first);
        vbrk::Launch plan[VBR_MAX_LAUNCHES];
        REQUIRE(vbrk::plan_launches(v, x.N, true, plan) == 1 && plan[0].kind == VBR_LAUNCH_TILE_4 && !plan[0].split);
        if (plan[0].wide != x.wide) std::fprintf(stderr, "%d tiles, %d K-steps, %lld rows of B, N = %lld: wide %d\n", x.groups, x.n_ks, (long long)x.n_cols, (long long)x.N, plan[0].wide);
        REQUIRE(plan[0].wide == x.wide);
        // its offsets reach 4 GiB less a page
        const int64_t most = (0xFFFFF000ll / 2 - x.N) / (x.n_cols - 1) / 8 * 8;
        REQUIRE(vbrk::plan_launches(v, x.N, true, plan, most) == 1 && plan[0].wide == x.wide);
        REQUIRE(vbrk::plan_launches(v, x.N, true, plan, most + 8) == 1 && !plan[0].wide && plan[0].grid == vbrk::grid_size(x.groups, (x.N + 255) / 256, plan[0].even));
        vbr_free(v);
    }
}

// Groups of 16 rows, each with `least` to `most` of the column blocks, all columns of which some row of the group has, and `empty` rows without entries.
struct OneSlabGroups {
    Csr a;
    std::vector<int32_t> perm, rg;
    OneSlabGroups(Rng &rng, int groups, int col_block, int blocks, int least, int most, int empty)
    {
        a.m = 16 * groups + empty;
        a.k = (int64_t)blocks * col_block;
        a.row_ptr.push_back(0);
        rg.push_back(0);
        for (int g = 0; g < groups; ++g) {
            std::vector<uint8_t> on((size_t)blocks, 0);
            for (int64_t n = least + rng.below(most - least + 1); n > 0;) {
                uint8_t &b = on[(size_t)rng.below(blocks)];
                n -= !b;
                b = 1;
            }
            for (int r = 0; r < 16; ++r) {
                for (int b = 0; b < blocks; ++b)
                    for (int c = r % 4; on[(size_t)b] && c < col_block; c += 4) a.col.push_back(b * col_block + c);
                a.row_ptr.push_back((int64_t)a.col.size());
            }
            rg.push_back(16 * (g + 1));
        }
        for (int i = 0; i < empty; ++i) a.row_ptr.push_back((int64_t)a.col.size());
        if (empty) rg.push_back((int32_t)a.m);
        a.val.assign(a.col.size(), 0x3c00);
        for (int64_t i = 0; i < a.m; ++i) perm.push_back((int32_t)i);
    }
    vbr_t *build(int col_block, bool schedules) const
    {
        const vbr_csr_t c = a.view();
        vbr_t *v = nullptr;
        REQUIRE(vbrk::build_impl(&c, perm.data(), rg.data(), (int32_t)rg.size() - 1, col_block, &v, schedules) == VBR_OK && vbr_audit(v) == VBR_OK);
        return v;
    }
};

// The schedules of the stream kernel hold, whether a call takes them or not; vbr_build makes them exactly where some call may, and the plans are the same with
// and without those that none takes.
void check_stream()
{
    struct { int groups, col_block, blocks, least, most, empty; } const fixed[] = {
        {64, 16, 1, 1, 1, 0}, {64, 32, 1, 1, 1, 0}, {65, 16, 40, 1, 40, 0}, {127, 32, 30, 1, 2, 0}, {129, 48, 33, 1, 33, 5}, {200, 80, 1, 1, 1, 70}, {64, 16, 2000, 1, 1, 0}, {64, 16, 6, 1, 6, 0}, {513, 16, 300, 2, 4, 0},
        {70, 16, 300, 250, 300, 0}, {256, 16, 120, 90, 120, 0}, {256, 16, 120, 10, 120, 200}, {300, 64, 16, 16, 16, 0}, {1000, 16, 64, 20, 24, 0}, {1600, 16, 40, 20, 30, 0}, {520, 32, 16, 1, 16, 0}};
    Rng rng(77);
    int chosen = 0, refused = 0;
    for (int i = 0; i < 70; ++i) {
        ++g_cases;
        const int n_fixed = (int)(sizeof(fixed) / sizeof(fixed[0]));
        const int cbs[] = {16, 32, 48, 64, 80};
        int groups = 64 + (int)rng.below(150), cb = cbs[rng.below(5)], blocks = 1 + (int)rng.below(rng.below(2) ? 30 : 200), most = 1 + (int)rng.below(blocks), least = 1 + (int)rng.below(most);
        int empty = (int)rng.below(3) * 33;
        if (i < n_fixed) { groups = fixed[i].groups; cb = fixed[i].col_block; blocks = fixed[i].blocks; least = fixed[i].least; most = fixed[i].most; empty = fixed[i].empty; }
        const OneSlabGroups m(rng, groups, cb, blocks, least, most, empty);
        vbr_t *all = m.build(cb, true), *v = m.build(cb, false);
        REQUIRE(all->n_work == groups && (int)all->stream_tiles.size() == (groups + 63) / 64);
        REQUIRE(v->stream_tiles.empty() ? v->stream_steps.empty() && v->lay.vals_off == v->lay.stream_tiles_off : v->stream_steps.size() == all->stream_steps.size());
        bool taken = false;
        for (int64_t N = 64; N <= 40000; N += N < 9000 ? 8 : 1000)
            for (int64_t pad : {0, 8, 64}) {
                vbrk::Launch p[VBR_MAX_LAUNCHES], q[VBR_MAX_LAUNCHES];
                const bool aligned = (N + pad) % 64 == 0;
                const int n = vbrk::plan_launches(all, N, aligned, p, N + pad);
                REQUIRE(n == vbrk::plan_launches(v, N, aligned, q, N + pad));
                for (int l = 0; l < n; ++l) {
                    taken |= p[l].stream;
                    REQUIRE(p[l].stream == q[l].stream && p[l].kind == q[l].kind && p[l].grid == q[l].grid && p[l].split == q[l].split && p[l].even == q[l].even);
                }
            }
        (taken ? chosen : refused) += 1;
        vbr_free(all);
        vbr_free(v);
    }
    if (chosen < 10 || refused < 10) std::fprintf(stderr, "schedules of %d matrices taken, of %d not\n", chosen, refused);
    REQUIRE(chosen >= 10 && refused >= 10);
    // far from it: few K-steps against many rows of B, many groups
    struct { int groups, blocks, used; } const far[] = {{1024, 16384, 8}, {2048, 1024, 8}, {1024, 4096, 4}, {64, 1 << 18, 6}};
    for (const auto &x : far) {
        ++g_cases;
        vbr_t *v = OneSlabGroups(rng, x.groups, 16, x.blocks, x.used, x.used, 0).build(16, false);
        REQUIRE(v->n_work == x.groups && v->stream_tiles.empty() && v->stream_steps.empty() && v->lay.vals_off == v->lay.stream_tiles_off);
        vbr_free(v);
    }
}

// The audit finds a schedule that is wrong in one place: another slot for a unit or an operand, another unit, fragment or group, steps that are not there.
void check_stream_audit()
{
    using namespace vbrk;
    Rng rng(78);
    vbr_t *v = OneSlabGroups(rng, 100, 16, 200, 60, 90, 0).build(16, true);
    REQUIRE(v->stream_tiles.size() == 2);
    auto wrong = [&](int32_t &x, int32_t y) {
        ++g_cases;
        REQUIRE(x != y);
        std::swap(x, y);
        REQUIRE(vbr_audit(v) == VBR_EINVAL);
        std::swap(x, y);
    };
    for (int trial = 0; trial < 200; ++trial) {
        const StreamTile &st = v->stream_tiles[(size_t)rng.below(2)];
        const int64_t t = st.first_step + 1 + rng.below(st.n_steps - 1);
        StreamRecord *now = v->stream_steps.data() + t * 2 * kStreamWaves, &r = now[rng.below(2 * kStreamWaves)], &before = *(&r - 2 * kStreamWaves);
        const int i = (int)rng.below(v->stream_ops), other = kStreamUnitBytes * (1 + (int)rng.below(kStreamSlots - 1)), all = kStreamSlots * kStreamUnitBytes;
        if (r.none() == 0) {
            wrong(r.to(), (r.to() + other) % all);
            wrong(r.to(), all);
            wrong(r.row(), r.row() < kSlabRows ? r.row() + kSlabRows : r.row() - kSlabRows);
            wrong(r.row(), (int32_t)v->n_cols);
            wrong(r.none(), kStreamNone);
        }
        if (r.group(i) != kStreamGroups) {
            int32_t &at = i > 0 ? r.slot(i - 1) : before.slot(v->stream_ops - 1);
            wrong(at, (at + other) % all);
            wrong(at, all);
            wrong(before.frag(i), before.frag(i) + 1024);
            wrong(r.groups(), r.groups() ^ 1 << 4 * i);
            wrong(r.groups(), (r.groups() & ~(15 << 4 * i)) | kStreamGroups << 4 * i);
        }
        wrong(r.early(trial & 1), (int32_t)v->n_cols - kSlabRows + 1);
    }
    for (StreamTile &st : v->stream_tiles) {
        wrong(st.n_steps, st.n_steps + 1);
        wrong(st.n_steps, st.n_steps / 4 * kStreamAhead);
        wrong(st.n_steps, (int32_t)(v->stream_steps.size() / (2 * kStreamWaves)) / kStreamAhead * kStreamAhead);
        wrong(st.first_step, -1);
        wrong(st.first_step, st.first_step + 1);
        wrong(st.row_begin[0], -1);
    }
    REQUIRE(vbr_audit(v) == VBR_OK);
    vbr_free(v);
}

// Deep tiles beyond 1536 workgroups: deep rings only where one list is far longer than the others, and up to six column tiles longer than all shared out.
void check_deep_rings()
{
    ++g_cases;
    struct { int n, len, hub; int64_t N; bool few; } const cases[] = {
        {88, 544, 0, 1024, true},  {88, 544, 0, 1280, false}, {88, 544, 0, 1536, false}, {88, 544, 0, 2304, false}, {88, 544, 0, 3072, false},
        {400, 64, 4096, 1280, true}, {400, 64, 4096, 1536, true}, {400, 64, 4096, 1792, false}, {400, 64, 4096, 2304, true}, {400, 64, 4096, 3328, false},
        {300, 192, 1600, 1536, false}, {300, 192, 1600, 2304, true}};
    for (const auto &x : cases) {
        vbr_t *v = clusters(x.n, x.len, x.hub);
        vbrk::Launch plan[VBR_MAX_LAUNCHES];
        REQUIRE(vbrk::plan_launches(v, x.N, true, plan) == 1 && plan[0].kind == VBR_LAUNCH_TILE_MIXED && !plan[0].split);
        REQUIRE(v->class_count[vbrk::kClassDeep] > 0 && (int64_t)plan[0].n_tiles * ((x.N + 255) / 256) > (x.N == 1024 ? 0 : 1536));
        if (plan[0].few != x.few) std::fprintf(stderr, "%d clusters of %d, hub %d, N = %lld: few %d\n", x.n, x.len, x.hub, (long long)x.N, plan[0].few);
        REQUIRE(plan[0].few == x.few);
        vbr_free(v);
    }
}

// Short lists are split, whatever the grid is rounded up to: the plans of a few tiles of one height and of two.
void check_short_lists()
{
    ++g_cases;
    for (int rows : {16, 32, 64})
        for (int n_ks : {3, 4, 5, 7, 11, 12})
            for (int64_t N : {8, 64, 72, 256, 520}) {
                vbr_t *v = stack(3, rows, n_ks);
                vbrk::Launch plan[VBR_MAX_LAUNCHES];
                REQUIRE(vbrk::plan_launches(v, N, N % 64 == 0, plan) == 1);
                REQUIRE(plan[0].split == (n_ks < 4 ? 0 : n_ks < 12 ? vbrk::kSplitShort : vbrk::kSplitSteps));
                REQUIRE(plan[0].grid == vbrk::grid_size(3, plan[0].split ? (N + 63) / 64 : (N + 255) / 256));
                vbr_free(v);
            }
    const std::vector<int32_t> rg = {0, 64, 80, 85, 115, 118};
    Csr a;
    a.m = 118;
    a.k = 160;
    for (int64_t i = 0; i <= a.m; ++i) a.row_ptr.push_back(i * a.k);
    for (int64_t i = 0; i < a.m * a.k; ++i) a.col.push_back((int32_t)(i % a.k));
    a.val.assign(a.col.size(), 0x3c00);
    std::vector<int32_t> perm;
    for (int32_t i = 0; i < 118; ++i) perm.push_back(i);
    const vbr_csr_t c = a.view();
    vbr_t *v = nullptr;
    REQUIRE(vbr_build(&c, perm.data(), rg.data(), 5, 32, &v) == VBR_OK);
    for (int64_t N : {8, 64, 72, 256, 520}) {
        vbrk::Launch plan[VBR_MAX_LAUNCHES];
        REQUIRE(vbrk::plan_launches(v, N, N % 64 == 0, plan) == 1 && plan[0].kind == VBR_LAUNCH_TILE_MIXED);
        REQUIRE(plan[0].split == vbrk::kSplitShort && plan[0].whole == 0 && plan[0].rest == plan[0].n_tiles);
        REQUIRE(plan[0].grid == vbrk::grid_size(4 * (int64_t)plan[0].n_tiles, (N + 255) / 256));
    }
    vbr_free(v);
}

// Every tile meets every column tile once, whatever the way the workgroups are dealt, and cut in shares no domain has many more than an eighth.
template <bool IN_TURN>
void check_map()
{
    ++g_cases;
    for (int Q = 1; Q <= 34; ++Q)
        for (int T : {1, 2, 3, 5, 7, 8, 9, 12, 16, 31, 40, 77, 130})
            for (bool even : {false, true}) {
                const int rest = Q % 8, each = rest & -rest;
                if (even && rest == 0) continue;
                const int domain = even ? Q / 8 * T + rest / each * ((T * each + 7) / 8) : Q >= 8 ? (Q + 7) / 8 * T : (T + 8 / Q - 1) / (8 / Q);
                REQUIRE(vbrk::grid_size(T, Q, even) == 8 * domain);
                std::vector<int> seen((size_t)T * Q), load(8);
                int tile = 0, ntile = 0;
                const vbrk::ColumnMap map = vbrk::column_map(Q, even);
                for (int b = 0; b < 8 * domain; ++b)
                    if (vbrk::map_workgroup<IN_TURN>(b, T, Q, map, tile, ntile)) {
                        REQUIRE(tile >= 0 && tile < T && ntile >= 0 && ntile < Q);
                        ++seen[(size_t)tile * Q + ntile];
                        ++load[b % 8];
                    }
                REQUIRE(std::count(seen.begin(), seen.end(), 1) == (long)seen.size());
                if (even) REQUIRE(8 * *std::max_element(load.begin(), load.end()) <= T * Q + 8 * 7);
            }
}

// The workgroups of a column tile of a mixed launch: one for a tile, or one for each of its four quarters.
void check_split_tile()
{
    ++g_cases;
    for (int whole : {0, 1, 5, 40})
        for (int rest : {0, 1, 3, 17})
            for (int behind : {0, 1, 9}) {
                if (whole + rest + behind == 0 || (rest == 0 && behind > 0)) continue;
                std::vector<int> one((size_t)(whole + rest + behind)), quarters(one.size());
                for (int w = 0; w < whole + 4 * rest + behind; ++w) {
                    int tile = w, quarter = -1;
                    const bool four = vbrk::split_tile(tile, whole, rest, quarter);
                    REQUIRE(tile >= 0 && tile < (int)one.size() && four == (tile >= whole && tile < whole + rest) && quarter >= 0 && quarter < (four ? 4 : 1));
                    if (four) quarters[(size_t)tile] |= 1 << quarter;
                    ++one[(size_t)tile];
                }
                for (int t = 0; t < (int)one.size(); ++t) {
                    const bool four = t >= whole && t < whole + rest;
                    REQUIRE(one[(size_t)t] == (four ? 4 : 1) && quarters[(size_t)t] == (four ? 15 : 0));
                }
            }
}

// Lanes of a row of entries, 8 to a column tile of 64: by whether the part of B that a column tile takes stays in an L2 and how often its rows are
// used, and by how the column tiles fall on the domains.
void check_entry_plan()
{
    ++g_cases;
    struct { int64_t len, n_cols, N; int lanes; } const cases[] = {
        {5, 16384, 64, 8},    {5, 16384, 256, 8},   {5, 16384, 512, 16},   {5, 16384, 72, 16},   {5, 16384, 136, 32}, {5, 16384, 240, 16}, {5, 32768, 240, 16},
        {5, 16384, 264, 16},  {5, 32768, 296, 16},  {5, 16384, 632, 16},  {5, 32768, 680, 16},  {5, 16384, 1000, 16}, {5, 16384, 2056, 16},
        {500, 5936, 3032, 32}, {500, 16048, 3752, 32}, {500, 16384, 240, 32}, {500, 5184, 696, 32}, {500, 5184, 136, 32}};
    for (const auto &x : cases) {
        std::vector<int64_t> start;
        for (int64_t i = 0; i <= 9000; ++i) start.push_back(i * x.len);
        const vbrk::EntryLaunch L = vbrk::plan_entry_rows(start, x.n_cols, x.N, x.N % 64 == 0);
        if (L.lanes != x.lanes) std::fprintf(stderr, "%lld entries a row, %lld rows of B, N = %lld: %d lanes\n", (long long)x.len, (long long)x.n_cols, (long long)x.N, L.lanes);
        REQUIRE(L.lanes == x.lanes && L.grid >= 8 && L.waves >= 9000 * x.lanes / 64);
    }
    // by how often the rows of B are used, and one row (the first) longer than the others: fewer where its loads are too many of all
    struct { int64_t rows, len, longest, n_cols, N; int lanes; } const more[] = {
        {12300, 10, 10, 16000, 520, 16},   {12300, 9, 9, 16000, 520, 16},    {9000, 20, 20, 16000, 520, 16},  {12300, 10, 10, 16000, 1000, 16}, {12300, 10, 10, 16000, 320, 16},
        {30000, 5, 5, 16000, 1288, 16},   {9000, 5, 5, 16384, 632, 16},     {9000, 300, 300, 16000, 384, 8},  {9000, 300, 300, 16000, 600, 16},  {9000, 300, 300, 4096, 600, 16},
        {4096, 12, 1000, 4096, 200, 8},   {4096, 12, 1000, 4096, 1016, 8},  {4096, 12, 1000, 4096, 3752, 8}, {4096, 12, 256, 4096, 1016, 16},  {16384, 25, 3700, 16384, 1016, 16}};
    for (const auto &x : more) {
        std::vector<int64_t> start = {0, x.longest};
        for (int64_t i = 1; i < x.rows; ++i) start.push_back(start.back() + x.len);
        const vbrk::EntryLaunch L = vbrk::plan_entry_rows(start, x.n_cols, x.N, x.N % 64 == 0);
        if (L.lanes != x.lanes) std::fprintf(stderr, "%lld rows of %lld entries, %lld, %lld of B, N = %lld: %d lanes\n", (long long)x.rows, (long long)x.len, (long long)x.longest, (long long)x.n_cols, (long long)x.N, L.lanes);
        REQUIRE(L.lanes == x.lanes);
    }
    // six workgroups on a CU: for rows of unlike length, long ones among them, with 24 entries and more on average
    struct { int64_t rows, len, longest; bool six; } const unlike[] = {
        {16384, 25, 3700, true}, {16384, 24, 257, true}, {16384, 23, 300, false}, {16384, 25, 256, false}, {16384, 65, 257, false}, {4096, 600, 600, false}, {4096, 300, 1300, true}, {9000, 5, 5, false}};
    for (const auto &x : unlike) {
        std::vector<int64_t> start = {0, x.longest};
        for (int64_t i = 1; i < x.rows; ++i) start.push_back(start.back() + x.len);
        REQUIRE(vbrk::plan_entry_rows(start, 16384, 1024, true).six == x.six);
    }
    // ... with 12 where a wave takes 128 columns or more and a row has a workgroup
    struct { int64_t len, longest, N; int lanes; bool six; } const wider[] = {{12, 1900, 736, 16, true}, {11, 1700, 736, 16, false}, {20, 1024, 1400, 16, false}, {20, 1030, 1400, 16, true}, {14, 2000, 256, 8, false}};
    for (const auto &x : wider) {
        std::vector<int64_t> start = {0, x.longest};
        for (int64_t i = 1; i < 16384; ++i) start.push_back(start.back() + x.len);
        const vbrk::EntryLaunch L = vbrk::plan_entry_rows(start, 16384, x.N, x.N % 64 == 0);
        if (L.six != x.six || L.lanes != x.lanes) std::fprintf(stderr, "%lld entries, %lld, N = %lld: %d lanes, six %d\n", (long long)x.len, (long long)x.longest, (long long)x.N, L.lanes, L.six);
        REQUIRE(L.six == x.six && L.lanes == x.lanes);
    }
    // waves that keep step: 128 and 256 columns of a B that does not stay, all resident, rows of like length that use rows of B now and then
    struct { int64_t rows, len, longest, n_cols, N; bool together; } const steps[] = {
        {2048, 48, 64, 20000, 1024, true},  {2048, 48, 64, 70000, 1024, true},  {4096, 48, 64, 20000, 200, true},   {4096, 48, 64, 70000, 200, true}, {8192, 128, 150, 32768, 200, true}, {4096, 256, 300, 32768, 200, true},
        {8192, 128, 257, 32768, 200, false}, {8192, 31, 50, 32768, 200, false}, {8192, 128, 150, 26000, 200, false}, {8192, 128, 150, 32768, 64, false}, {4096, 60, 64, 10400, 200, false},
        {4096, 48, 64, 10600, 200, true},   {8192, 128, 150, 65536, 128, true}, {4096, 48, 64, 40000, 128, true}, {4096, 48, 64, 32768, 128, false}, {4507, 486, 560, 132664, 64, false}, {4000, 48, 64, 20000, 200, false},  {16384, 64, 90, 32768, 200, true},   {16392, 64, 90, 32768, 200, false}};
    for (const auto &x : steps) {
        std::vector<int64_t> start = {0, x.longest};
        for (int64_t i = 1; i < x.rows; ++i) start.push_back(start.back() + x.len);
        const vbrk::EntryLaunch L = vbrk::plan_entry_rows(start, x.n_cols, x.N, x.N % 64 == 0);
        if (L.together != x.together) std::fprintf(stderr, "%lld x %lld, %lld entries, N = %lld: %d lanes, grid %lld, together %d\n", (long long)x.rows, (long long)x.n_cols, (long long)x.len, (long long)x.N, L.lanes, (long long)L.grid, L.together);
        REQUIRE(L.together == x.together);
    }
    // the widths the tests of every length of a row's end stand for: four rows of every length up to 45, long rows among many others, and both
    for (int which : {0, 1, 2}) {
        std::vector<int64_t> start = {0};
        auto add = [&](int64_t first, int64_t last, int64_t step, int times) {
            for (int64_t len = last; len >= first; len -= step)
                for (int i = 0; i < times; ++i) start.push_back(start.back() + len);
        };
        if (which == 1) { add(1025, 1289, 8, 1); add(600, 600, 1, 500); add(257, 329, 1, 1); }
        if (which == 2) { add(1025, 1169, 16, 1); add(257, 329, 8, 4); }
        if (which != 1) add(0, 45, 1, 4);
        for (int64_t N : {64, 120, 128, 200, 208, 256}) {
            const bool aligned = N == 64 || N == (which == 2 ? 128 : 256);
            REQUIRE(vbrk::plan_entry_rows(start, 1500, N, aligned).lanes == (aligned || which == 2 ? 8 : N <= 128 ? 16 : 32));
        }
        // B beyond 4 GiB: with rows that begin inside cache lines
        if (which == 0) REQUIRE(vbrk::plan_entry_rows(start, 70000, 64, false).lanes == 8 && vbrk::plan_entry_rows(start, 65536, 128, false).lanes == 16 && vbrk::plan_entry_rows(start, 70000, 200, false).lanes == 32);
    }
    // widths of as many column tiles have as many lanes, rows of B padded to a cache line or not; long rows, in waves and workgroups of their own
    struct { int64_t rows, len, longest, n_cols, first_N, last_N; bool aligned; int lanes; } const widths[] = {
        {16384, 5, 5, 16384, 72, 256, true, 8},     {20000, 5, 5, 20000, 264, 320, true, 8},   {20000, 5, 5, 20000, 456, 512, true, 8},  {20000, 4, 4, 20000, 264, 1024, true, 16},
        {16384, 5, 5, 16384, 264, 320, true, 16},   {16384, 5, 5, 16384, 456, 512, true, 16},  {5003, 336, 336, 5000, 264, 448, true, 8}, {5003, 336, 336, 5000, 456, 512, true, 16},
        {20000, 5, 5, 20000, 264, 512, false, 16},  {20000, 5, 5, 20000, 520, 1024, false, 8}, {16384, 5, 5, 16384, 520, 1024, false, 16}, {16384, 30, 30, 16384, 136, 216, false, 32}, {16384, 30, 30, 16384, 224, 256, false, 16},
        {1250, 600, 1100, 2600, 200, 256, false, 32}, {1250, 600, 1100, 2600, 520, 584, false, 16}, {1250, 600, 1100, 2600, 392, 512, false, 32}, {1250, 600, 1100, 2600, 1032, 1152, false, 16}, {1250, 600, 1100, 2600, 1160, 1280, false, 32}, {1250, 600, 1100, 2600, 1800, 2048, true, 32},
        {4096, 45, 1800, 4096, 1288, 1528, false, 16}, {4096, 45, 1800, 4096, 1544, 2040, false, 32}, {4096, 45, 1800, 4096, 2056, 2304, false, 16}};
    for (const auto &x : widths)
        for (int64_t N = x.first_N; N <= x.last_N; N += 8) {
            std::vector<int64_t> start = {0, x.longest};
            for (int64_t i = 1; i < x.rows; ++i) start.push_back(start.back() + x.len);
            const vbrk::EntryLaunch L = vbrk::plan_entry_rows(start, x.n_cols, N, x.aligned);
            if (L.lanes != x.lanes) std::fprintf(stderr, "%lld rows of %lld entries, %lld of B, N = %lld: %d lanes\n", (long long)x.rows, (long long)x.len, (long long)x.n_cols, (long long)N, L.lanes);
            REQUIRE(L.lanes == x.lanes);
        }
}

// A matrix kept as entries whose last rows have none: the entry behind the last one, which these read, lies in the buffer, and is zero.
void check_last_entry()
{
    for (int64_t k : {65536, 65537}) {
        ++g_cases;
        Csr a;
        a.m = 9000;
        a.k = k;
        a.row_ptr.push_back(0);
        for (int64_t i = 0; i < a.m; ++i) {
            for (int64_t j = 0; i < 8990 && j < 6; ++j) a.col.push_back((int32_t)(j * (k / 6) + i * 7 % (k / 6)));
            a.row_ptr.push_back((int64_t)a.col.size());
        }
        a.val.assign(a.col.size(), 0x3c00);
        std::vector<int32_t> perm, rg;
        for (int64_t i = 0; i <= a.m; ++i) rg.push_back((int32_t)i);
        perm.assign(rg.begin(), rg.end() - 1);
        const vbr_csr_t c = a.view();
        vbr_t *v = nullptr;
        REQUIRE(vbr_build(&c, perm.data(), rg.data(), (int32_t)a.m, 1, &v) == VBR_OK && v->by_entries && vbr_audit(v) == VBR_OK);
        const vbrk::EntryRows &e = v->entries;
        REQUIRE(e.near == (k <= 65536) && e.row.back().len == 0 && e.row.back().start == e.count && e.count == (int64_t)a.col.size());
        REQUIRE(e.get(e.count).col == 0 && e.get(e.count).val == 0);
        REQUIRE(v->lay.gcol_off + (e.count + 1) * (e.near ? 4 : 8) <= vbr_device_bytes(v));
        vbr_free(v);
    }
}

// Every call with the first 0, 1, 2 ... of its allocations succeeding, up to `most` or until it gets all it asks for: it
// reports the failure, and nothing is thrown through the C interface.
template <class F>
void check_out_of_memory(F call, long most)
{
    ++g_cases;
    for (long n = 0; n < most; ++n) {
        int rc = 1;
        bool thrown = false;
        g_allocations_left = n;
        try {
            rc = call();
        } catch (...) {
            thrown = true;
        }
        g_allocations_left = -1;
        REQUIRE(!thrown);
        if (rc == VBR_OK) return;
        REQUIRE(rc == VBR_ENOMEM);
    }
    REQUIRE(most < 100);
}

void check_out_of_memory(const Csr &a, int col_block, long most)
{
    const vbr_csr_t c = a.view();
    std::vector<int32_t> perm((size_t)a.m), rg((size_t)a.m + 1);
    int32_t G = 0;
    REQUIRE(sa1_reorder(&c, col_block, 0.5, perm.data(), rg.data(), &G) == VBR_OK);
    std::vector<int32_t> perm1((size_t)a.m), rg1((size_t)a.m + 1);
    int32_t G1 = 0, sel = 0;
    const double ts[] = {0.2, 0.6};
    check_out_of_memory([&] { return sa1_reorder(&c, col_block, 0.5, perm1.data(), rg1.data(), &G1); }, most);
    check_out_of_memory([&] { return sa1_blocking_curve(&c, col_block, ts, 2, 8, nullptr, nullptr, nullptr, nullptr, &sel); }, most);
    check_out_of_memory([&] {
        vbr_t *v = nullptr;
        const int rc = vbr_build(&c, perm.data(), rg.data(), G, col_block, &v);
        if (rc != VBR_OK && v != nullptr) return 1;
        vbr_free(v);
        return rc;
    }, most);
}

}  // namespace

int main()
{
    Rng rng(12345);
    const double taus[] = {0.0, 0.3, 0.6, 1.0};
    // small matrices, every block width class (narrow gather path, granules of 8, 16, 32)
    for (int col_block : {1, 3, 8, 16, 32, 64})
        for (int trial = 0; trial < 4; ++trial) {
            const Csr a = make(rng, 1 + rng.below(400), 1 + rng.below(40), col_block, 0.05 + 0.3 * rng.uni(), 1 + (int)rng.below(30));
            for (double tau : taus) check_matrix(a, col_block, tau, true);
        }
    // thresholds next to zero, where the blocks of a row over the threshold exceed every integer
    for (int trial = 0; trial < 3; ++trial) {
        const Csr a = make(rng, 60 + rng.below(100), 20, 2, 0.15, 90);
        for (double tau : {5e-324, 1e-300, 1e-20, 1e-18}) check_matrix(a, 2, tau, true);
    }
    // thousands of short groups: the panel packing; tall groups beside them
    {
        const Csr a = make(rng, 6000, 40, 8, 0.08, 3000);
        check_matrix(a, 8, 0.9, false);
        const Csr b = make(rng, 5000, 24, 16, 0.15, 40);
        check_matrix(b, 16, 0.5, false);
        check_matrix(b, 16, 1.0, false);
    }
    // the candidate search on several threads against the same oracle
    {
        setenv("VBR_SA1_THREADS", "3", 1);
        const Csr a = make(rng, 5000, 300, 2, 0.02, 400);
        for (double tau : {0.2, 0.5, 0.9}) check_matrix(a, 2, tau, false);
        unsetenv("VBR_SA1_THREADS");
    }
    // blocking curve and error paths
    {
        const Csr a = make(rng, 300, 20, 4, 0.2, 12);
        const vbr_csr_t c = a.view();
        const double ts[] = {0.1, 0.5, 1.0};
        int64_t g[3], nb[3], st[3], sh[3];
        int32_t sel = -1;
        REQUIRE(sa1_blocking_curve(&c, 4, ts, 3, 8, g, nb, st, sh, &sel) == VBR_OK && sel >= 0 && sel < 3);
        REQUIRE(sa1_blocking_curve(&c, 4, ts, 3, 0, g, nb, st, sh, &sel) == VBR_EINVAL);
        std::vector<int32_t> perm((size_t)a.m, 0), rg = {0, (int32_t)a.m};
        vbr_t *v = nullptr;
        REQUIRE(vbr_build(&c, perm.data(), rg.data(), 1, 4, &v) == VBR_EINVAL && v == nullptr);   // not a bijection
        REQUIRE(sa1_reorder(&c, 3, 0.5, perm.data(), rg.data(), &sel) == VBR_EINVAL);            // 80 % 3 != 0
        REQUIRE(vbr_audit(nullptr) == VBR_EINVAL);
        ++g_cases;
    }
    check_plan();
    check_deep_rings();
    check_wide();
    check_stream();
    check_stream_audit();
    check_short_lists();
    check_map<false>();
    check_map<true>();
    check_split_tile();
    check_entry_plan();
    check_last_entry();
    // memory that runs out: at every allocation of a small matrix, and at the first ones of a matrix whose check takes threads
    {
        check_out_of_memory(make(rng, 90, 20, 8, 0.2, 40), 8, 100000);
        Csr a;
        a.m = 512;
        a.k = 4096;
        for (int64_t i = 0; i <= a.m; ++i) a.row_ptr.push_back(i * a.k);
        for (int64_t i = 0; i < a.m * a.k; ++i) a.col.push_back((int32_t)(i % a.k));
        a.val.assign(a.col.size(), 0x3c00);
        check_out_of_memory(a, 64, 4);
        // the audit of a matrix with schedules
        vbr_t *v = OneSlabGroups(rng, 70, 16, 40, 1, 40, 3).build(16, true);
        check_out_of_memory([&] { return vbr_audit(v); }, 100000);
        vbr_free(v);
    }
    std::printf("host_check ok: %d cases\n", g_cases);
    return 0;
}
