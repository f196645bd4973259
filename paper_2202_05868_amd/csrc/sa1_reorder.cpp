// 1-SA row reordering on the host: quotient rows, grouping of identical quotient rows by hash + exact
// compare, greedy merge with pattern update under the two-step merge condition.
// Sections 3.1 and 3.2 of the paper (Eq. 4, Eq. 5, Algorithms 1 and 2, Theorem 1's condition).
// Integer work throughout; the only floating-point operations are one binary64 division per
// candidate (Jaccard >= tau) and one floor per seed (the merge limit).
#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstdint>
#include <cstdlib>
#include <cstring>
#include <memory>
#include <new>
#include <numeric>
#include <vector>

#include <immintrin.h>

#include "host_threads.h"
#include "vbr_host.h"

namespace vbrk {

int validate_csr(const vbr_csr_t *csr, bool need_vals)
{
    if (!csr) return VBR_EINVAL;
    if (csr->n_rows < 0 || csr->n_cols < 0 || csr->nnz < 0) return VBR_EINVAL;
    if (csr->n_rows > INT32_MAX - 1 || csr->n_cols > INT32_MAX - 1) return VBR_EINVAL;
    if (!csr->row_ptr) return VBR_EINVAL;
    if (csr->nnz > 0 && !csr->col_idx) return VBR_EINVAL;
    if (need_vals && csr->nnz > 0 && !csr->vals) return VBR_EINVAL;
    if (csr->dtype != VBR_F16 && csr->dtype != VBR_BF16) return VBR_EINVAL;
    const int64_t *rp = csr->row_ptr;
    const int64_t M = csr->n_rows, K = csr->n_cols;
    if (rp[0] != 0 || rp[M] != csr->nnz) return VBR_EINVAL;
    for (int64_t i = 0; i < M; ++i)
        if (rp[i + 1] < rp[i] || rp[i + 1] > csr->nnz) return VBR_EINVAL;
    // rising columns: compared without a branch per entry, so that the loop over a row vectorises
    std::atomic<bool> bad(false);
    Team team(threads_for(csr->nnz, 1 << 20));
    team.each(M, std::max<int64_t>(64, M / (8 * team.size()) + 1), [&](int64_t b, int64_t e) {
        bool wrong = false;
        for (int64_t i = b; i < e; ++i) {
            const int32_t *c = csr->col_idx + rp[i];
            const int64_t n = rp[i + 1] - rp[i];
            if (n == 0) continue;
            unsigned down = 0;
            for (int64_t k = 1; k < n; ++k) down |= c[k] <= c[k - 1];          // unsorted or duplicate
            wrong |= down != 0 || c[0] < 0 || c[n - 1] >= K;
        }
        if (wrong) bad = true;
    });
    return bad ? VBR_EINVAL : VBR_OK;
}

namespace {

int64_t popcount_and_generic(const uint64_t *a, const uint64_t *b, int64_t w)
{
    int64_t s = 0;
    for (int64_t i = 0; i < w; ++i) s += __builtin_popcountll(a[i] & b[i]);
    return s;
}

// Same count with 512-bit AND + per-lane population count, where the host CPU has them
// (checked once at run time: the library is built on one machine and run on another).
__attribute__((target("avx512f,avx512vpopcntdq")))
int64_t popcount_and_avx512(const uint64_t *a, const uint64_t *b, int64_t w)
{
    __m512i acc = _mm512_setzero_si512();
    int64_t i = 0;
    for (; i + 8 <= w; i += 8)
        acc = _mm512_add_epi64(acc, _mm512_popcnt_epi64(_mm512_and_si512(_mm512_loadu_si512(a + i), _mm512_loadu_si512(b + i))));
    int64_t s = _mm512_reduce_add_epi64(acc);
    for (; i < w; ++i) s += __builtin_popcountll(a[i] & b[i]);
    return s;
}

// Scan of patterns laid out in blocks of 8 (word w of all eight side by side; len8: their sizes): mask[b] gets the
// members of block b that have at most `limit` bits outside x and a size from min_len to max_len.
struct ScanArgs {
    const uint64_t *y8, *not_x;
    const int32_t *len8;
    int64_t w, limit;
    int32_t min_len, max_len;
};
void scan_generic(const ScanArgs &s, int64_t b0, int64_t b1, uint8_t *mask)
{
    for (int64_t b = b0; b < b1; ++b) {
        unsigned m = 0;
        for (int k = 0; k < 8; ++k) {
            const int32_t len = s.len8[8 * b + k];
            if (len < s.min_len || len > s.max_len) continue;
            int64_t n = 0;
            for (int64_t i = 0; i < s.w; ++i) n += __builtin_popcountll(s.y8[(b * s.w + i) * 8 + k] & s.not_x[i]);
            m |= (unsigned)(n <= s.limit) << k;
        }
        mask[b] = (uint8_t)m;
    }
}

// W: words per pattern known when compiled (their complement stays in registers), 0: any number
template <int W>
__attribute__((target("avx512f,avx512vl,avx512vpopcntdq")))
void scan_avx512(const ScanArgs &s, int64_t b0, int64_t b1, uint8_t *mask)
{
    const int64_t words = W ? W : s.w;
    __m512i nx[W ? W : 1];
    for (int i = 0; i < W; ++i) nx[i] = _mm512_set1_epi64((long long)s.not_x[i]);
    const __m512i limit = _mm512_set1_epi64((long long)s.limit);
    const __m256i lo = _mm256_set1_epi32(s.min_len), hi = _mm256_set1_epi32(s.max_len);
    for (int64_t b = b0; b < b1; ++b) {
        const __m256i len = _mm256_loadu_si256((const __m256i *)(s.len8 + 8 * b));
        const __mmask8 fits = _mm256_mask_cmple_epi32_mask(_mm256_cmpge_epi32_mask(len, lo), len, hi);
        const uint64_t *y = s.y8 + b * words * 8;
        __m512i n = _mm512_setzero_si512();
        for (int64_t i = 0; i < words; ++i)
            n = _mm512_add_epi64(n, _mm512_popcnt_epi64(_mm512_and_si512(_mm512_loadu_si512(y + 8 * i),
                                                                         W ? nx[W ? i : 0] : _mm512_set1_epi64((long long)s.not_x[i]))));
        mask[b] = (uint8_t)_mm512_mask_cmple_epi64_mask(fits, n, limit);
    }
}

typedef int64_t (*popcount_and_fn)(const uint64_t *, const uint64_t *, int64_t);
typedef void (*scan_fn)(const ScanArgs &, int64_t, int64_t, uint8_t *);

bool has_vpopcnt()
{
    __builtin_cpu_init();
    return __builtin_cpu_supports("avx512f") && __builtin_cpu_supports("avx512vl") && __builtin_cpu_supports("avx512vpopcntdq");
}

// Threads of a call on a matrix of n_rows rows and nnz entries; the environment variable VBR_SA1_THREADS
// overrides the count.  One for every 2^16 of them, on 16 CPUs half as many and these (ms): a reordering of a graph of 16384 nodes 7.7 and 6.5, of 4096 nodes 0.93 and
// 0.65, no structure, 8704 rows 4.1 and 2.8, 12224 rows 3.5 and 2.6; a curve of ten thresholds of the 4096 nodes 7.1 and 5.7, of the 8704 rows 22.0 and 13.3, of
// the 12224 13.5 and 10.2, of 8192 rows of 64 x 64 blocks 1.53 and 1.39; other blocks, which mostly take less than a millisecond, the same.
int sa1_threads(int64_t n_rows, int64_t nnz)
{
    if (const char *e = std::getenv("VBR_SA1_THREADS")) {
        const long v = std::strtol(e, nullptr, 10);
        if (v >= 1) return (int)std::min<long>(v, 256);
    }
    return threads_for(64 * n_rows + nnz, 1 << 16);
}

// The quotient matrix after Algorithm 1: what the greedy pass works on, whatever the threshold.
struct Quotient {
    int64_t M = 0, KB = 0, W = 1;
    int32_t NC = 0;                     // classes of identical quotient rows, in order of their smallest row
    std::vector<int32_t> class_of;      // [M]
    std::vector<int32_t> size;          // [NC] rows of the class
    std::vector<int64_t> ptr;           // [NC + 1] into blk
    std::vector<int32_t> blk;           // column blocks of the class, the rarest (in the fewest classes) first
    std::vector<uint64_t> bits;         // [NC][W] the same as bit sets
    std::vector<uint64_t> bits8;        // the bit sets in blocks of 8 classes: word w of the eight side by side
    std::vector<int32_t> len8;          // and their sizes (-1 beyond the last class)
    // Inverted index.  Entries of a column block: the classes that hold it, split by the position the block
    // has in the class's rarest-first list into kBands bands (0, 1, 2-3, 4-7, ...), rising inside a band.
    static constexpr int kBands = 8;
    std::vector<int64_t> inv_ptr;       // [KB * kBands + 1]
    std::vector<int32_t> inv_class, inv_pos;

    int32_t len(int32_t c) const { return (int32_t)(ptr[c + 1] - ptr[c]); }
    const uint64_t *pattern(int32_t c) const { return &bits[(size_t)c * W]; }
    static int band(int64_t pos) { return pos == 0 ? 0 : std::min(kBands - 1, 64 - __builtin_clzll((unsigned long long)pos)); }
    static int64_t band_begin(int b) { return b == 0 ? 0 : (int64_t)1 << (b - 1); }
};

void make_quotient(const vbr_csr_t *csr, int32_t col_block, Team &team, Quotient &q)
{
    const int64_t M = csr->n_rows, KB = csr->n_cols / col_block, W = KB > 128 && KB <= 256 ? 4 : std::max<int64_t>(1, (KB + 63) / 64);   // 3 words as 4
    q.M = M;
    q.KB = KB;
    q.W = W;
    // Quotient rows (Eq. 4) as lists, written where the row's entries are; their hash is the sum over the
    // nonzero blocks (Eq. 5) of the block index scattered over 64 bits, with the row length added, which the
    // paper suggests to thin out collisions.
    const std::unique_ptr<int32_t[]> list_(new int32_t[(size_t)csr->nnz]), len(new int32_t[(size_t)M]);      // not cleared: written first
    const std::unique_ptr<uint64_t[]> hash(new uint64_t[(size_t)M]);
    int32_t *const list = list_.get();
    const int shift = (col_block & (col_block - 1)) == 0 ? __builtin_ctz((unsigned)col_block) : -1;
    team.each(M, 256, [&](int64_t r0, int64_t r1) {
        for (int64_t i = r0; i < r1; ++i) {
            int32_t *out = list + csr->row_ptr[i];
            int32_t n = 0;
            int64_t limit = 0;                       // first column beyond the last block listed
            uint64_t h = 0;
            for (int64_t p = csr->row_ptr[i]; p < csr->row_ptr[i + 1]; ++p) {
                const int32_t c = csr->col_idx[p];
                if (c < limit) continue;
                const int32_t j = shift >= 0 ? c >> shift : c / col_block;
                limit = ((int64_t)j + 1) * col_block;
                uint64_t x = ((uint64_t)(uint32_t)j + 1) * 0x9E3779B97F4A7C15ull;
                x ^= x >> 29;
                x *= 0xBF58476D1CE4E5B9ull;
                h += x ^ (x >> 32);
                out[n++] = j;
            }
            len[i] = n;
            hash[i] = h + (uint64_t)(uint32_t)n;
        }
    });

    // Algorithm 1 on the quotient rows: rows of equal hash are compared exactly.  Rows come in rising order,
    // so classes are numbered in order of their smallest row, the order in which Algorithm 2 visits them.
    int64_t cap = 16;
    while (cap < 2 * M) cap *= 2;
    std::vector<int32_t> table((size_t)cap, -1), rep;
    q.class_of.resize((size_t)M);
    rep.reserve((size_t)M);
    for (int64_t i = 0; i < M; ++i) {
        const int32_t *mine = list + csr->row_ptr[i];
        uint64_t at = hash[i] & (uint64_t)(cap - 1);
        for (;; at = (at + 1) & (uint64_t)(cap - 1)) {
            const int32_t c = table[at];
            if (c < 0) {
                table[at] = (int32_t)rep.size();
                q.class_of[i] = (int32_t)rep.size();
                rep.push_back((int32_t)i);
                q.size.push_back(1);
                break;
            }
            const int32_t r = rep[c];
            if (hash[r] == hash[i] && len[r] == len[i] &&
                std::memcmp(list + csr->row_ptr[r], mine, (size_t)len[i] * sizeof(int32_t)) == 0) {
                q.class_of[i] = c;
                ++q.size[c];
                break;
            }
        }
    }
    const int32_t NC = (int32_t)rep.size();
    q.NC = NC;
    q.ptr.assign((size_t)NC + 1, 0);
    for (int32_t c = 0; c < NC; ++c) q.ptr[c + 1] = q.ptr[c] + len[rep[c]];
    std::vector<int32_t> count((size_t)KB, 0);
    for (int32_t c = 0; c < NC; ++c)
        for (int32_t k = 0; k < len[rep[c]]; ++k) ++count[list[csr->row_ptr[rep[c]] + k]];
    q.blk.resize((size_t)q.ptr[NC]);
    q.bits.assign((size_t)NC * W, 0);
    q.bits8.assign((size_t)((NC + 7) / 8) * 8 * W, 0);
    q.len8.assign((size_t)((NC + 7) / 8) * 8, -1);
    std::vector<int32_t> by_count((size_t)KB), rank((size_t)KB);
    std::iota(by_count.begin(), by_count.end(), 0);
    std::stable_sort(by_count.begin(), by_count.end(), [&](int32_t a, int32_t b) { return count[a] < count[b]; });
    for (int64_t k = 0; k < KB; ++k) rank[by_count[k]] = (int32_t)k;
    team.each(NC, 256, [&](int64_t c0, int64_t c1) {
        for (int64_t c = c0; c < c1; ++c) {
            int32_t *b = q.blk.data() + q.ptr[c];
            const int32_t n = q.len((int32_t)c);
            const int32_t *src = list + csr->row_ptr[rep[c]];
            uint64_t *bits = q.bits.data() + c * W, *bits8 = q.bits8.data() + (c / 8) * 8 * W + c % 8;
            for (int32_t k = 0; k < n; ++k) {
                bits[src[k] >> 6] |= 1ull << (src[k] & 63);
                b[k] = rank[src[k]];
            }
            for (int64_t w = 0; w < W; ++w) bits8[8 * w] = bits[w];
            q.len8[(size_t)c] = n;
            std::sort(b, b + n);
            for (int32_t k = 0; k < n; ++k) b[k] = by_count[b[k]];
        }
    });
    // The inverted index by counting, over ranges of classes (one a thread, fewer where the lists outnumber
    // their entries): counts per range and list, their running sums list by list, then the entries.
    const int64_t lists = KB * Quotient::kBands;
    const int64_t parts = std::max<int64_t>(1, std::min<int64_t>(team.size(), q.ptr[NC] / (2 * lists + 1)));
    std::vector<int64_t> fill((size_t)(parts * lists), 0);
    auto each_entry = [&](int64_t part, auto f) {
        for (int32_t c = (int32_t)(NC * part / parts); c < (int32_t)(NC * (part + 1) / parts); ++c)
            for (int64_t k = q.ptr[c]; k < q.ptr[c + 1]; ++k) {
                const int64_t pos = k - q.ptr[c];
                f(fill[(size_t)(part * lists + (int64_t)q.blk[k] * Quotient::kBands + Quotient::band(pos))], c, pos);
            }
    };
    team.each(parts, 1, [&](int64_t p0, int64_t p1) {
        for (int64_t part = p0; part < p1; ++part) each_entry(part, [](int64_t &n, int32_t, int64_t) { ++n; });
    });
    q.inv_ptr.assign((size_t)lists + 1, 0);
    int64_t sum = 0;
    for (int64_t l = 0; l < lists; ++l) {
        for (int64_t part = 0; part < parts; ++part) {
            const int64_t n = fill[(size_t)(part * lists + l)];
            fill[(size_t)(part * lists + l)] = sum;
            sum += n;
        }
        q.inv_ptr[(size_t)l + 1] = sum;
    }
    q.inv_class.resize(q.blk.size());
    q.inv_pos.resize(q.blk.size());
    team.each(parts, 1, [&](int64_t p0, int64_t p1) {
        for (int64_t part = p0; part < p1; ++part)
            each_entry(part, [&](int64_t &at, int32_t c, int64_t pos) {
                q.inv_class[at] = c;
                q.inv_pos[at++] = (int32_t)pos;
            });
    });
}

// What Algorithm 2 makes of the classes at one threshold.
struct Grouping {
    std::vector<int32_t> group_of;      // [NC]
    std::vector<int64_t> blocks, rows;  // per group: column blocks of its pattern, rows
};

// Algorithm 2: one pass per seed over the later ungrouped classes in rising order, merging where the
// condition of section 3.2 holds and OR-ing the merged pattern into the group's.
//
// For a seed x the merge limit lam is fixed, and a class y with |x | y| > lam can never join: the pattern P
// only grows, and |P | y| >= |x | y|.  So every class the pass can merge is among the classes with at most
// d = lam - |x| blocks outside x, which depends on x alone.  `search` finds those (less the ones that tau
// rules out whatever P becomes: P has at most d blocks more than x, so at the end |P & y| <= |x & y| + d and
// |P | y| >= |x | y|), in rising order; the pass then applies the exact test to the ungrouped ones of them,
// one after the other.  It meets every class that could pass, in the order and with the pattern of the
// full scan.  Before that, the classes that pass the test against x itself are looked for: the first merge
// has to be one of them, they have at most |x| / tau - |x| blocks outside x (few when tau is high), and
// where there is none the seed stays alone.  The searches are independent of the pass, so several threads
// run ahead of it.
//
// Search by lists: at most d blocks of y lie outside x, so of y's d + 2 rarest blocks at least two lie in x
// (of all its blocks, all but d, where y has fewer).  Only list entries of those positions are walked; the
// classes met often enough are compared exactly.  Search by bit sets: y & ~x is counted for every later
// class, eight at a time.  A seed takes what it expects to cost less.
class Greedy {
public:
    Greedy(const Quotient &q, double tau) : q_(q), tau_(tau), need_((size_t)q.KB + 1, 0)
    {
        const bool wide = has_vpopcnt();
        popcount_and_ = wide ? popcount_and_avx512 : popcount_and_generic;
        scan_ = !wide ? scan_generic : q.W == 1 ? scan_avx512<1> : q.W == 2 ? scan_avx512<2> : q.W <= 4 ? scan_avx512<4> : scan_avx512<0>;
        scan_cost_ = wide ? 1 : 8;
        // The similarity test (double)I / (double)U >= tau is monotone in I for a fixed U, so it is
        // tabulated once: need[U] = smallest I that passes (found with the very same division, so
        // the decisions are bit-identical), need[0] = 0 (two empty patterns are similar).
        for (int64_t U = 1; U <= q.KB; ++U) {
            int64_t I = (int64_t)std::ceil(tau * (double)U);
            I = std::max<int64_t>(0, std::min<int64_t>(I, U));
            while (I > 0 && (double)(I - 1) / (double)U >= tau) --I;
            while (I <= U && !((double)I / (double)U >= tau)) ++I;      // I = U + 1: nothing passes
            need_[U] = (int32_t)I;
        }
    }

    Grouping run(Team *team)
    {
        Grouping g;
        g.group_of.assign((size_t)q_.NC, -1);
        P_.assign((size_t)q_.W, 0);
        if (need_[std::min<int64_t>(1, q_.KB)] == 0) run_all_pairs(g);
        else if (team && team->size() > 1) run_ahead(g, *team);
        else {
            Scratch s(q_);
            std::vector<int32_t> cand;
            for (int32_t seed = 0; seed < q_.NC; ++seed)
                if (g.group_of[seed] < 0) {
                    search(seed, s, cand);
                    take(g, seed, cand);
                }
        }
        return g;
    }

private:
    struct Scratch {
        explicit Scratch(const Quotient &q) : first(q.inv_ptr), cnt((size_t)q.NC, 0), mask((size_t)q.NC / 8 + 1, 0), not_x((size_t)q.W, 0) {}
        std::vector<int64_t> first;       // per list: its first entry above the seeds this scratch has seen (they rise)
        std::vector<uint8_t> cnt;         // bytes: the counters of 32 768 classes stay in the first-level cache
        std::vector<uint8_t> mask;
        std::vector<int32_t> hit;
        std::vector<uint64_t> not_x;
    };

    int64_t limit_of(int64_t lx) const { return (int64_t)std::floor((double)lx / (1.0 - 0.5 * tau_)); }

    // the later classes that the seed's pass may merge, rising; empty if none can be the first to merge
    void search(int32_t seed, Scratch &s, std::vector<int32_t> &out) const
    {
        out.clear();
        const int64_t lx = q_.len(seed), lam = std::min(limit_of(lx), q_.KB), d = lam - lx;
        if (lx == 0 || tau_ >= 1.0) return;               // identical patterns share a class already
        // U <= I / tau <= lx / tau for a class that passes against x; one more, the quotient being rounded
        // (compared before it becomes an integer: next to tau = 0 it is beyond them all)
        const double most = (double)lx / tau_;
        const int64_t d_first = most < (double)(lx + d) ? (int64_t)most + 1 - lx : d;
        if (d_first < d) {
            bool any = false;
            outside_at_most(seed, d_first, s, [&](int32_t, int64_t I, int64_t U) { any |= I >= need_[U]; });
            if (!any) return;
        }
        bool any = false;
        outside_at_most(seed, d, s, [&](int32_t c, int64_t I, int64_t U) {
            any |= I >= need_[U];
            if (I + d >= need_[U]) out.push_back(c);
        });
        if (!any) out.clear();
        std::sort(out.begin(), out.end());
    }

    // f(class, |x & y|, |x | y|) for every later class y that has at most d blocks outside the seed's pattern x, and enough blocks to pass at all
    template <class F>
    void outside_at_most(int32_t seed, int64_t d, Scratch &s, F f) const
    {
        const int64_t lx = q_.len(seed), min_len = std::max<int64_t>(need_[lx], 1);
        const uint64_t *x = q_.pattern(seed);
        auto keep = [&](int32_t c) {
            const int64_t ly = q_.len(c);
            if (ly < min_len || ly > lx + d) return;
            const int64_t I = popcount_and_(x, q_.pattern(c), q_.W), U = lx + ly - I;
            if (U <= lx + d) f(c, I, U);
        };
        constexpr int64_t kHits = 2;
        const int64_t prefix = d + kHits;
        const int last_band = Quotient::band(prefix - 1);
        const int32_t *xb = q_.blk.data() + q_.ptr[seed];
        int64_t list_work = 0;
        for (int64_t k = 0; k < lx; ++k) {
            const size_t l0 = (size_t)xb[k] * Quotient::kBands;
            list_work += q_.inv_ptr[l0 + last_band + 1] - q_.inv_ptr[l0];
        }
        // in steps of about a nanosecond: list entries (the later classes' share of them) and list heads, against blocks of 8 bit sets
        list_work = 3 * list_work * (q_.NC - seed) / q_.NC + 2 * lx * (last_band + 1) + q_.NC / 64;
        const int64_t bits_work = (scan_cost_ * q_.W + 3) * (int64_t)(q_.NC - seed) / 8;
        // min_len > d holds for every tau < 1 (tau lx > lx tau / (2 - tau)); if it ever did not, a class without a block in x could pass
        if (min_len <= d || prefix > 255 || list_work > bits_work) {
            for (int64_t w = 0; w < q_.W; ++w) s.not_x[w] = ~x[w];
            const int64_t b0 = (seed + 1) / 8, b1 = (q_.NC + 7) / 8;
            scan_(ScanArgs{q_.bits8.data(), s.not_x.data(), q_.len8.data(), q_.W, d, (int32_t)min_len, (int32_t)(lx + d)}, b0, b1, s.mask.data());
            for (int64_t b = b0; b < b1; ++b)
                for (unsigned m = s.mask[b]; m; m &= m - 1) {
                    const int64_t c = b * 8 + __builtin_ctz(m);
                    if (c > seed) keep((int32_t)c);
                }
            return;
        }
        s.hit.clear();
        std::memset(s.cnt.data() + seed, 0, (size_t)(q_.NC - seed));
        const bool all_long = min_len >= prefix;          // no class worth a look is shorter than the prefix
        for (int64_t k = 0; k < lx; ++k)
            for (int b = 0; b <= last_band; ++b) {
                const size_t l = (size_t)xb[k] * Quotient::kBands + b;
                int64_t e = s.first[l];
                const int64_t end = q_.inv_ptr[l + 1];
                while (e < end && q_.inv_class[e] <= seed) ++e;
                s.first[l] = e;
                const bool whole = b < Quotient::kBands - 1 && Quotient::band_begin(b + 1) <= prefix;
                for (; e < end; ++e) {
                    if (!whole && q_.inv_pos[e] >= prefix) continue;           // the band the prefix ends in
                    const int32_t c = q_.inv_class[e];
                    const int64_t hits = ++s.cnt[c];
                    const int64_t enough = all_long ? kHits : std::min<int64_t>(prefix, q_.len(c)) - d;
                    if (hits == enough) s.hit.push_back(c);
                }
            }
        for (const int32_t c : s.hit) keep(c);
    }

    // the exact merge test for class j against the current pattern; updates the pattern on success
    bool try_merge(int32_t j)
    {
        const int64_t lv = q_.len(j);
        if (sizeP_ == 0 && lv == 0) return true;           // both empty: similar, union 0 within any limit
        // |P & v| <= min and |P | v| >= max: if even min/max misses tau the exact ratio does too
        const int64_t lo = std::min(sizeP_, lv), hi = std::max(sizeP_, lv);
        if (lo < need_[hi] || hi > lam_max_) return false;
        const uint64_t *v = q_.pattern(j);
        const int64_t I = popcount_and_(P_.data(), v, q_.W);
        const int64_t U = sizeP_ + lv - I;
        if (I < need_[U] || U > lam_max_) return false;
        for (int64_t w = 0; w < q_.W; ++w) P_[w] |= v[w];
        sizeP_ = U;
        return true;
    }

    void start_group(Grouping &g, int32_t seed)
    {
        g.group_of[seed] = (int32_t)g.rows.size();
        g.rows.push_back(q_.size[seed]);
        std::memcpy(P_.data(), q_.pattern(seed), (size_t)q_.W * 8);
        sizeP_ = q_.len(seed);
        lam_max_ = limit_of(sizeP_);
    }

    void take(Grouping &g, int32_t seed, const std::vector<int32_t> &cand)
    {
        start_group(g, seed);
        const int32_t G = g.group_of[seed];
        for (const int32_t j : cand)
            if (g.group_of[j] < 0 && try_merge(j)) {
                g.group_of[j] = G;
                g.rows[G] += q_.size[j];
            }
        g.blocks.push_back(sizeP_);
    }

    // tau so small that a class sharing nothing with the pattern passes the similarity test: every later class is looked at
    void run_all_pairs(Grouping &g)
    {
        std::vector<int32_t> active((size_t)q_.NC), keep;
        std::iota(active.begin(), active.end(), 0);
        keep.reserve(active.size());
        while (!active.empty()) {
            const int32_t seed = active[0];
            start_group(g, seed);
            const int32_t G = g.group_of[seed];
            keep.clear();
            for (size_t t = 1; t < active.size(); ++t) {
                if (try_merge(active[t])) {
                    g.group_of[active[t]] = G;
                    g.rows[G] += q_.size[active[t]];
                } else keep.push_back(active[t]);
            }
            active.swap(keep);
            g.blocks.push_back(sizeP_);
        }
    }

    // The searches of the next ungrouped classes on all threads, then the pass over them; the batch grows
    // while most of what was searched turns out to be seeds, and shrinks when merges made the searches idle.
    void run_ahead(Grouping &g, Team &team)
    {
        std::vector<Scratch> scratch((size_t)team.size(), Scratch(q_));
        std::vector<std::vector<int32_t>> cand;
        std::vector<int32_t> batch;
        int64_t want = 4 * team.size();
        for (int32_t at = 0; at < q_.NC;) {
            batch.clear();
            for (; at < q_.NC && (int64_t)batch.size() < want; ++at)
                if (g.group_of[at] < 0) batch.push_back(at);
            if (cand.size() < batch.size()) cand.resize(batch.size());
            std::atomic<int64_t> next(0);
            const int64_t n = (int64_t)batch.size(), piece = std::max<int64_t>(1, std::min<int64_t>(16, n / (4 * team.size())));
            team.run([&](int member) {
                for (;;) {
                    const int64_t b = next.fetch_add(piece);
                    if (b >= n) break;
                    for (int64_t k = b; k < std::min(n, b + piece); ++k) search(batch[k], scratch[(size_t)member], cand[(size_t)k]);
                }
            });
            int64_t used = 0;
            for (int64_t k = 0; k < n; ++k)
                if (g.group_of[batch[k]] < 0) {
                    take(g, batch[k], cand[(size_t)k]);
                    ++used;
                }
            want = used * 2 > n ? std::min<int64_t>(want * 2, 512 * team.size()) : std::max<int64_t>(want / 2, 2 * team.size());
        }
    }

    const Quotient &q_;
    const double tau_;
    std::vector<int32_t> need_;
    popcount_and_fn popcount_and_;
    scan_fn scan_;
    int64_t scan_cost_;
    std::vector<uint64_t> P_;
    int64_t sizeP_ = 0, lam_max_ = 0;
};

}  // namespace

int sa1_reorder_impl(const vbr_csr_t *csr, int32_t col_block, double tau, int32_t *perm,
                     int32_t *row_groups, int32_t *n_groups)
{
    const int64_t M = csr->n_rows;
    Team team(sa1_threads(M, csr->nnz));
    Quotient q;
    make_quotient(csr, col_block, team, q);
    const Grouping g = Greedy(q, tau).run(&team);
    // Rows sorted by group, stable in the row index; groups are already numbered in seed order.
    const int32_t G = (int32_t)g.rows.size();
    std::vector<int32_t> start((size_t)G + 1, 0);
    for (int32_t i = 0; i < G; ++i) start[i + 1] = start[i] + (int32_t)g.rows[i];
    std::copy(start.begin(), start.end(), row_groups);
    for (int64_t i = 0; i < M; ++i) perm[start[g.group_of[q.class_of[i]]]++] = (int32_t)i;
    *n_groups = G;
    return VBR_OK;
}

}  // namespace vbrk

extern "C" int sa1_reorder(const vbr_csr_t *csr, int32_t col_block, double tau, int32_t *perm,
                           int32_t *row_groups, int32_t *n_groups)
{
    if (!csr || !perm || !row_groups || !n_groups) return VBR_EINVAL;
    if (col_block <= 0 || !(tau >= 0.0 && tau <= 1.0)) return VBR_EINVAL;
    try {
        const int rc = vbrk::validate_csr(csr, false);
        if (rc != VBR_OK) return rc;
        if (csr->n_cols % col_block != 0) return VBR_EINVAL;
        return vbrk::sa1_reorder_impl(csr, col_block, tau, perm, row_groups, n_groups);
    } catch (const std::bad_alloc &) {
        return VBR_ENOMEM;
    } catch (...) {
        return VBR_EINVAL;
    }
}

extern "C" int sa1_blocking_curve(const vbr_csr_t *csr, int32_t col_block, const double *taus, int32_t n_taus,
                                  int64_t target_height, int64_t *n_groups, int64_t *n_blocks,
                                  int64_t *stored_elems, int64_t *sum_heights, int32_t *selected)
{
    if (!csr || !taus || n_taus <= 0 || col_block <= 0 || target_height <= 0) return VBR_EINVAL;
    for (int32_t i = 0; i < n_taus; ++i)
        if (!(taus[i] >= 0.0 && taus[i] <= 1.0)) return VBR_EINVAL;
    try {
        const int rc = vbrk::validate_csr(csr, false);
        if (rc != VBR_OK) return rc;
        if (csr->n_cols % col_block != 0) return VBR_EINVAL;
        // The quotient matrix is the same for every threshold; the thresholds are independent of each other
        // and are dealt to the threads.  A stored block of group g has the group's height, and the group's
        // pattern lists its blocks, so the counts follow from the grouping of the classes alone.
        vbrk::Team team(vbrk::sa1_threads(csr->n_rows, csr->nnz));
        vbrk::Quotient q;
        vbrk::make_quotient(csr, col_block, team, q);
        std::vector<vbrk::Grouping> all((size_t)n_taus);
        team.each(n_taus, 1, [&](int64_t b, int64_t e) {
            for (int64_t i = b; i < e; ++i) all[(size_t)i] = vbrk::Greedy(q, taus[i]).run(nullptr);
        });
        int32_t best = 0;
        bool have = false;
        unsigned __int128 best_num = 0;    // |sum_heights - target * n_blocks| of the best so far
        int64_t best_den = 1;              // its n_blocks
        for (int32_t i = 0; i < n_taus; ++i) {
            const vbrk::Grouping &g = all[(size_t)i];
            int64_t nb = 0, sumh = 0;
            for (size_t k = 0; k < g.rows.size(); ++k) {
                nb += g.blocks[k];
                sumh += g.blocks[k] * g.rows[k];
            }
            if (n_groups) n_groups[i] = (int64_t)g.rows.size();
            if (n_blocks) n_blocks[i] = nb;
            if (stored_elems) stored_elems[i] = sumh * col_block;
            if (sum_heights) sum_heights[i] = sumh;
            if (nb > 0) {
                // distance of the average block height from the target: |sumh / nb - target|
                const __int128 diff = (__int128)sumh - (__int128)target_height * nb;
                const unsigned __int128 num = (unsigned __int128)(diff < 0 ? -diff : diff);
                if (!have || num * (unsigned __int128)best_den < best_num * (unsigned __int128)nb) {
                    have = true;
                    best = i;
                    best_num = num;
                    best_den = nb;
                }
            }
        }
        if (selected) *selected = best;
        return VBR_OK;
    } catch (const std::bad_alloc &) {
        return VBR_ENOMEM;
    } catch (...) {
        return VBR_EINVAL;
    }
}
