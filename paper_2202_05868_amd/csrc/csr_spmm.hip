// C = A.B row by row from lists of entries, one fp32 accumulator per output element, no matrix units: the comparator (the
// role the sparse-library routine plays in section 4.4.2 of the paper), and the form vbr_spmm multiplies a matrix in
// whose blocking found nothing to share.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <memory>
#include <new>
#include <vector>

#include "host_threads.h"
#include "vbr_device.h"
#include "vbr_host.h"

struct csr_dev {
    int64_t n_rows = 0, n_cols = 0, nnz = 0;
    int32_t dtype = 0;
    vbrk::EntryRows rows;
    int64_t entry_off = 0, total = 256;
    void *dev = nullptr;
};

namespace vbrk {
namespace {

constexpr int kCsrThreads = 256;     // 4 waves

typedef float float2v __attribute__((ext_vector_type(2)));

struct EntryParams {
    EntryRowsDev rows;
    const uint16_t *B;
    float *C;
    int64_t ldb, ldc;
    uint32_t b_bytes;                // bytes from B's first element to the end of its last row (WIDE: not used)
    int32_t n_rows, n_huge, n_long, N, n_waves, n_ntiles;
    ColumnMap map;
};

template <int DT>
__device__ __forceinline__ float half_to_f32(uint32_t pair, int hi)      // the low or the high 16 bits of a word
{
    if constexpr (DT == VBR_F16) return (float)__builtin_bit_cast(_Float16, (uint16_t)(hi ? pair >> 16 : pair));
    else return __builtin_bit_cast(float, hi ? pair & 0xFFFF0000u : pair << 16);
}

// LDS of a workgroup: partial sums of three waves, results on their way to C
template <int LANES>
constexpr int kPartialBytes = 3 * 8 * LANES * 4;
template <int LANES>
constexpr int kTurnedBytes = LANES == 8 ? 0 : 4 * 64 * 8 * 4;
constexpr int kSixBytes = 26 * 1024;       // so much of it is there six times on a CU, and not seven times
static_assert(6 * kSixBytes <= 160 * 1024 && 7 * kSixBytes > 160 * 1024 && kPartialBytes<32> + kTurnedBytes<32> <= kSixBytes, "six workgroups on a CU");

template <int U>
__device__ __forceinline__ uint32_t row_pair(uint32_t x)     // lane 2U of every row of 16 lanes to its first eight, lane 2U + 1 to the others
{
    const int lo = __builtin_amdgcn_mov_dpp((int)x, 0x150 + 2 * U, 0xf, 0xf, true);
    return (uint32_t)__builtin_amdgcn_update_dpp(lo, (int)x, 0x150 + 2 * U + 1, 0xf, 0xc, false);
}

__device__ __forceinline__ uint32_t half_turn(uint32_t x)    // the halves of every row of 16 lanes change places
{
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x128, 0xf, 0xf, true);
}

// What bounds it: the B rows gathered through the caches, nnz N 2 bytes, at 64 bytes per cycle and compute unit.  So
// everything is arranged for B to come from the L2 of the XCD and for enough loads to be in flight:
//   - a wave owns 8 LANES columns; an XCD keeps to few column tiles at a time (map below), whose B it holds in its L2;
//   - LANES lanes own a row of A: each 16 of them fetch 16 entries with one load, and every one of the entries is then
//     handed to all of them by a row broadcast of the vector unit.  Rows are taken longest first, so the rows
//     of a wave have nearly the same length and the long ones start early;
//   - rows beyond kEntryLongRow entries get a whole wave, rows beyond kEntryHugeRow a workgroup: its 64 / LANES (256 / LANES)
//     groups of lanes take the entries in turn, and the partial sums are added at the end.
// Entries past the end of a row are loads out of the buffer's range: they return zeros and cost no traffic.
// LANES: 8, 16 or 32 (64, 128 or 256 columns a wave), chosen by plan_entry_rows.  With 8, the 16 lanes of a row take two entries
// at a time and add their halves at the end.
// Eight loads of B are in flight from a row's first entry to its last: an addition is followed by the load of the entry eight further on, whose column
// was fetched a batch earlier, and no load stands in a branch, so that every wait is for one load and not for all.  A load of B takes the load path 17
// cycles, a word a lane 7, two words 17: so an entry whose column fits 16 bits is one word (NEAR), any other and a row's description are one load each.
// (Two words and one, and from six or seven waves a SIMD to eight for fp16: 3648 x 4864, 253 entries a row, N = 88 14.9 and 13.9 us, 32768 x 32768, 16 a row,
// N = 256 22.5 and 21.3, the graph below 199 and 196; 120 products of the cases' ranges 3 % less by the word alone.)  A row leaves through LDS: see there.
// TOGETHER: every eight loads a wave waits for all of them, which keeps the waves in step (plan_entry_rows says where that pays).
// Up to 64 registers, eight waves a SIMD; where the compiler keeps values across a branch at a row's end it takes more.
// WIDE, a B of 4 GiB and more, has 64-bit addresses: there an entry that is not there is a branch around its load, waits are for what the branch may have
// left open, and 62 to 74 registers leave six to eight waves a SIMD.  Against columns and values apart and waits for a batch (32768 x 65536, 16 a row, rows of B
// 66 kB apart, N = 64 33.7 and 33.6, 256: 54.3 and 52.8, 4096: 828 and 801; rows of 6 to 4000, 16384 x 65536: 30.1 and 28.6, 44.5 and 42.4, 467 and 436;
// two words, 32768 x 100000: 11.5 and 11.9, 50.0 and 49.9, 589 and 592).
// Measured on a graph of 16384 nodes with 426 000 entries (rows of 0 to 3600), with B and C beyond the caches, N = 4096: 215 us with the waits of a
// batch for all of its loads, columns and values apart and 16 bytes of every 32 a store, 199 with entries of two words, now 196 (17.8 TB/s of gathered B,
// texture-address unit 83 % busy).
template <int DT, bool WIDE, int LANES, bool NEAR, bool TOGETHER = false>
__global__ void __launch_bounds__(kCsrThreads) entry_rows_kernel(const EntryParams p)
{
    constexpr bool kPair = LANES == 8;                               // 16 lanes own a row, two entries at a time
    constexpr int kGroups = kPair ? 4 : 64 / LANES, kLgGroups = kGroups == 4 ? 2 : 1, kTileN = 8 * LANES;
    __shared__ float partial[kPartialBytes<LANES> / (kTileN * 4)][kTileN];
    const int lane = threadIdx.x & 63, g = lane / (64 / kGroups), s16 = lane & 15, chunk0 = lane % LANES;
    // workgroup -> (column tile, four waves' rows): workgroups are dealt to the 8 L2 domains round-robin
    const int T = (p.n_waves + 3) / 4, Q = p.n_ntiles;
    int ntile, tile;
    if (!map_workgroup<true>(blockIdx.x, T, Q, p.map, tile, ntile)) return;
    const int in_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = tile * 4 + in_wg;
    if (wave >= p.n_waves) return;
    // parts: the groups of lanes that share a row; part: this group's number among them
    const bool huge = tile < p.n_huge, whole = !huge && wave < 4 * p.n_huge + p.n_long;
    const int parts = huge ? 4 * kGroups : whole ? kGroups : 1, part = huge ? in_wg * kGroups + g : whole ? g : 0;
    const int first = p.n_huge + p.n_long, pos = huge ? tile : whole ? wave - 3 * p.n_huge : first + (wave - 3 * p.n_huge - first) * kGroups + g;
    const EntryRow mine = p.rows.row[pos < p.n_rows ? pos : p.n_rows - 1];
    const int32_t row = pos < p.n_rows ? mine.row : -1, len = pos < p.n_rows ? mine.len : 0;
    const int32_t max_len = __builtin_amdgcn_readfirstlane(len);     // the first row of a wave is its longest
    const int lg_parts = huge ? 2 + kLgGroups : whole ? kLgGroups : 0;
    const int step = 16 * parts;
    // this lane's entry of the first batch, and how far behind it the row's last one is; of a row without entries the place of its start counts as behind
    const int e0 = parts * s16 + part, to_last = len - 1 - e0;
    using Stored = std::conditional_t<NEAR, uint32_t, Entry>;
    const Stored *first_entry = static_cast<const Stored *>(p.rows.entry) + (mine.start + (len == 0) + e0);

    const int n0 = ntile * kTileN;
    const int last_chunk = (p.N - n0 < kTileN ? p.N - n0 : kTileN) / 8 - 1;
    const uint32_t coff = (uint32_t)(chunk0 <= last_chunk ? chunk0 : last_chunk) * 16;   // past column N: the last chunk again, never stored
    const uint32_t ldb_bytes = (uint32_t)(p.ldb * 2);
    const char *Bs = reinterpret_cast<const char *>(p.B + n0);
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(Bs), 0, WIDE ? 0 : (int)(p.b_bytes - (uint32_t)n0 * 2), 0x00020000);

    float acc[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) acc[i] = 0.f;
    auto load = [&](uint32_t off) -> uint4v {
        if constexpr (WIDE) {
            if ((int32_t)off < 0) return uint4v{0, 0, 0, 0};
            return *reinterpret_cast<const uint4v *>(Bs + (int64_t)off * (p.ldb * 2) + coff);
        } else {
            return __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(rsrc, (int)(off + coff), 0, 0));
        }
    };
    // (the empty statements keep additions and loads in the order written: moved past each other they take registers that cost waves)
    auto add = [&](uint32_t a_bits, uint4v &b) {
        if constexpr (DT == VBR_F16) asm volatile("" ::"v"(b));
        else asm volatile("" : "+v"(b));
        const float a = __builtin_bit_cast(float, a_bits);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = __builtin_fmaf(a, half_to_f32<DT>(b[i >> 1], i & 1), acc[i]);
        asm volatile("" : "+v"(acc[0]), "+v"(acc[1]), "+v"(acc[2]), "+v"(acc[3]), "+v"(acc[4]), "+v"(acc[5]), "+v"(acc[6]), "+v"(acc[7]));
        __builtin_amdgcn_sched_barrier(0);
    };
    // The entries of batch i, this lane's one of 16.  Behind the end of the row the last entry again, without effect: a load that every lane
    // makes is one the waits for the loads of B can count on.
    int32_t col;                                                     // where it does not stand in the word
    uint32_t word;
    bool there;
    auto fetch = [&](int batch) {
        const int32_t at = batch * step;
        const Stored e = first_entry[at < to_last ? at : to_last];
        if constexpr (NEAR) {
            word = e;
        } else {
            col = e.col;
            word = e.val;
        }
        there = at <= to_last;
    };
    uint32_t off = 0, a = 0;
    auto take = [&]() {                                              // the fetched entries become those to load and to add
        const uint32_t c = NEAR ? word & 0xFFFFu : (uint32_t)col;
        off = !there ? 0xFFFFF000u : WIDE ? c : c * ldb_bytes;
        a = there ? __builtin_bit_cast(uint32_t, half_to_f32<DT>(word, NEAR)) : 0;
    };
    uint4v b[8];
    auto hand = [](auto u, uint32_t x) {
        if constexpr (kPair) return row_pair<u.value>(x);
        else return row_lane<u.value>(x);
    };
    // loads of entries AT .. AT + N - 1 of `off`; additions of 8 from AT on, each followed by a load of one of `off` in its place
    auto issue = [&](auto n, auto at) { static_for<n.value>([&](auto u) { b[u.value] = load(hand(constant<at.value + u.value>(), off)); }); };
    auto finish = [&](auto n, auto at, uint32_t a) {
        static_for<n.value>([&](auto u) { add(hand(constant<at.value + u.value>(), a), b[u.value]); });
    };
    auto go_on = [&](auto at, uint32_t a, auto n, auto next) {
        static_for<8>([&](auto u) {
            add(hand(constant<at.value + u.value>(), a), b[u.value]);
            if constexpr (u.value < n.value) b[u.value] = load(hand(constant<next.value + u.value>(), off));
            __builtin_amdgcn_sched_barrier(0);
        });
    };
    auto keep_step = [&]() {
        if constexpr (TOGETHER) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    };
    constexpr constant<0> c0;
    constexpr constant<4> c4;
    constexpr constant<8> c8;
    int left = (max_len + parts - 1) >> lg_parts;                    // entries of this group of lanes, of the longest row of the wave
    if (left > 0) {
        fetch(0);
        take();
        int batch = 1;
        if constexpr (kPair) {
            if (left <= 8) {
                issue(c4, c0);
                finish(c4, c0, a);
            } else {
                if (left > 16) fetch(batch);
                issue(c8, c0);
                for (; left > 24; left -= 16) {
                    const uint32_t now = a;
                    take();
                    keep_step();
                    fetch(++batch);
                    go_on(c0, now, c8, c0);
                }
                if (left > 16) {
                    const uint32_t now = a;
                    take();
                    go_on(c0, now, c4, c0);
                    finish(c4, c0, a);
                } else {
                    finish(c8, c0, a);
                }
            }
        } else if (left <= 4) {
            issue(c4, c0);
            finish(c4, c0, a);
        } else {
            issue(c8, c0);
            for (; left > 20; left -= 16) {
                keep_step();
                fetch(batch++);
                go_on(c0, a, c8, c8);
                const uint32_t now = a;
                take();
                keep_step();
                go_on(c8, now, c8, c0);
            }
            // 5 to 20 are left, eight of them on their way: those beyond 12, and the last four of more than eight
            uint32_t now = a;
            if (left > 12) {
                if (left > 16) fetch(batch);
                go_on(c0, now, c8, c8);
                now = half_turn(a);
                if (left > 16) take();
                left -= 8;
            } else {
                off = half_turn(off);
                a = half_turn(a);
            }
            // (the first addition stands before the branch, or the compiler converts its eight values there and holds them in registers)
            add(hand(c0, now), b[0]);
            if (left > 8) {
                b[0] = load(hand(c0, off));
                __builtin_amdgcn_sched_barrier(0);
                static_for<7>([&](auto u) {
                    add(hand(constant<u.value + 1>(), now), b[u.value + 1]);
                    if constexpr (u.value < 3) b[u.value + 1] = load(hand(constant<u.value + 1>(), off));
                    __builtin_amdgcn_sched_barrier(0);
                });
                finish(c4, c0, a);
            } else {
                static_for<7>([&](auto u) { add(hand(constant<u.value + 1>(), now), b[u.value + 1]); });
            }
        }
    }
    if constexpr (kPair) {
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += __builtin_bit_cast(float, half_turn(__builtin_bit_cast(uint32_t, acc[i])));
    }
    if (parts > 1) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            if constexpr (LANES <= 16) acc[i] += __shfl_xor(acc[i], 16);
            acc[i] += __shfl_xor(acc[i], 32);
        }
    }
    if (huge) {                                                      // the same for every wave of the workgroup
        if (g == 0 && in_wg > 0) {
#pragma unroll
            for (int i = 0; i < 8; ++i) partial[in_wg - 1][chunk0 * 8 + i] = acc[i];
        }
        __syncthreads();
        if (in_wg > 0) return;
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += partial[0][chunk0 * 8 + i] + partial[1][chunk0 * 8 + i] + partial[2][chunk0 * 8 + i];
    }
    if constexpr (kPair) {                                           // each half of the 16 lanes stores four of the eight columns
        const int hi = lane >> 3 & 1, n = n0 + chunk0 * 8 + 4 * hi;
        const float4v out = hi ? float4v{acc[4], acc[5], acc[6], acc[7]} : float4v{acc[0], acc[1], acc[2], acc[3]};
        if (row >= 0 && n < p.N && (parts == 1 || g == 0)) __builtin_nontemporal_store(out, reinterpret_cast<float4v *>(p.C + row * p.ldc + n));
    } else {
        // A lane holds eight columns, 32 bytes of C: stored as they are, a store takes every other 16 bytes of its lines.  Through LDS, it is 1 KiB of whole
        // lines (16384 rows, N = 4096, only the rows' descriptions and stores: 116 and 52 us; that graph without its loads of B: 141 and 110).
        __shared__ __attribute__((aligned(16))) float turned[kTurnedBytes<LANES> / (64 * 8 * 4)][64 * 8];
        float *out_lds = turned[in_wg];
        *reinterpret_cast<float4v *>(out_lds + 8 * lane) = float4v{acc[0], acc[1], acc[2], acc[3]};
        *reinterpret_cast<float4v *>(out_lds + 8 * lane + 4) = float4v{acc[4], acc[5], acc[6], acc[7]};
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int from_lane = 32 * i + (lane >> 1), n = n0 + 4 * (lane + 64 * i) % kTileN;
            const float4v out = *reinterpret_cast<const float4v *>(out_lds + 4 * (lane + 64 * i));
            const int32_t r = __shfl(row, from_lane);
            if (r >= 0 && n < p.N && (parts == 1 || from_lane < LANES)) __builtin_nontemporal_store(out, reinterpret_cast<float4v *>(p.C + r * p.ldc + n));
        }
    }
}

using EntryKernel = void (*)(EntryParams);
template <int DT, bool NEAR>
constexpr EntryKernel entry_kernels[9] = {entry_rows_kernel<DT, false, 8, NEAR>, entry_rows_kernel<DT, false, 16, NEAR>, entry_rows_kernel<DT, false, 32, NEAR>,
                                          entry_rows_kernel<DT, true, 8, NEAR>, entry_rows_kernel<DT, true, 16, NEAR>, entry_rows_kernel<DT, true, 32, NEAR>,
                                          entry_rows_kernel<DT, false, 8, NEAR, true>, entry_rows_kernel<DT, false, 16, NEAR, true>, entry_rows_kernel<DT, false, 32, NEAR, true>};

inline int64_t align_up256(int64_t x) { return (x + 255) / 256 * 256; }

}  // namespace

int launch_entry_rows(const EntryLaunch &L, int32_t dtype, const EntryRowsDev &rows, int64_t n_rows, int64_t n_cols,
                      const void *B_dev, int64_t ldb, float *C_dev, int64_t ldc, int64_t N, void *hip_stream)
{
    EntryParams p;
    p.rows = rows;
    p.B = static_cast<const uint16_t *>(B_dev);
    p.C = C_dev;
    p.ldb = ldb;
    p.ldc = ldc;
    const int64_t b_bytes = b_bytes_of(n_cols, ldb, N);              // 32-bit offsets from its first element, if they reach
    const bool wide = b_bytes > kNearBytes;
    p.b_bytes = wide ? 0 : (uint32_t)b_bytes;
    p.n_rows = (int32_t)n_rows;
    p.N = (int32_t)N;
    const int width = 8 * L.lanes;
    p.n_ntiles = (int32_t)((N + width - 1) / width);
    p.map = column_map((uint32_t)p.n_ntiles, L.even);
    p.n_huge = L.n_huge;
    p.n_long = L.n_long;
    p.n_waves = (int32_t)L.waves;
    if (L.waves > INT32_MAX || L.grid > INT32_MAX) return VBR_EUNSUPPORTED;
    const int variant = (wide ? 3 : L.together ? 6 : 0) + (L.lanes == 32 ? 2 : L.lanes == 16 ? 1 : 0);
    const EntryKernel kernel = dtype == VBR_F16 ? (rows.near ? entry_kernels<VBR_F16, true>[variant] : entry_kernels<VBR_F16, false>[variant])
                                                : (rows.near ? entry_kernels<VBR_BF16, true>[variant] : entry_kernels<VBR_BF16, false>[variant]);
    const int lds = L.lanes == 32 ? kPartialBytes<32> + kTurnedBytes<32> : L.lanes == 16 ? kPartialBytes<16> + kTurnedBytes<16> : kPartialBytes<8> + kTurnedBytes<8>;
    hipLaunchKernelGGL(kernel, dim3((unsigned)L.grid), dim3(kCsrThreads), L.six ? (unsigned)(kSixBytes - lds) : 0u, static_cast<hipStream_t>(hip_stream), p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_last_hip_error((int)e); return VBR_EHIP; }
    return VBR_OK;
}

}  // namespace vbrk

extern "C" int csr_spmm_create(const vbr_csr_t *csr, csr_dev_t **out)
{
    if (!csr || !out) return VBR_EINVAL;
    *out = nullptr;
    try {
        const int rc = vbrk::validate_csr(csr, true);
        if (rc != VBR_OK) return rc;
        std::unique_ptr<csr_dev> h(new csr_dev());
        h->n_rows = csr->n_rows;
        h->n_cols = csr->n_cols;
        h->nnz = csr->nnz;
        h->dtype = csr->dtype;
        vbrk::Team team(vbrk::threads_for(csr->nnz, 1 << 18));
        vbrk::make_entry_rows(csr, team, h->rows);
        h->entry_off = vbrk::align_up256(csr->n_rows * (int64_t)sizeof(vbrk::EntryRow));
        h->total = vbrk::align_up256(h->entry_off + (int64_t)h->rows.bytes());
        *out = h.release();
        return VBR_OK;
    } catch (const std::bad_alloc &) {
        return VBR_ENOMEM;
    } catch (...) {
        return VBR_EINVAL;
    }
}

extern "C" int64_t csr_device_bytes(const csr_dev_t *h) { return h ? h->total : 0; }

extern "C" int csr_upload(csr_dev_t *h, void *buf_dev, void *hip_stream)
{
    if (!h || !buf_dev || (reinterpret_cast<uintptr_t>(buf_dev) & 255) != 0) return VBR_EINVAL;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char *d = static_cast<char *>(buf_dev);
    struct Part { int64_t off; const void *src; size_t bytes; };
    const Part parts[2] = {
        {0, h->rows.row.data(), h->rows.row.size() * sizeof(vbrk::EntryRow)},
        {h->entry_off, h->rows.entry.get(), h->rows.bytes()},
    };
    for (const Part &pt : parts) {
        if (pt.bytes == 0) continue;
        hipError_t e = hipMemcpyAsync(d + pt.off, pt.src, pt.bytes, hipMemcpyHostToDevice, stream);
        if (e != hipSuccess) { vbrk::set_last_hip_error((int)e); return VBR_EHIP; }
    }
    hipError_t e = hipStreamSynchronize(stream);
    if (e != hipSuccess) { vbrk::set_last_hip_error((int)e); return VBR_EHIP; }
    h->dev = buf_dev;
    return VBR_OK;
}

extern "C" int csr_spmm(const csr_dev_t *h, const void *B_dev, int64_t ldb, float *C_dev, int64_t ldc,
                        int64_t N, void *hip_stream)
{
    if (!h) return VBR_EINVAL;
    if (!h->dev) return VBR_ESTATE;
    if (N < 0 || N % 8 != 0 || N > (int64_t)INT32_MAX - 1024) return VBR_EINVAL;
    if (N == 0 || h->n_rows == 0) return VBR_OK;
    if (!B_dev || !C_dev || ldb < N || ldc < N || ldb % 8 != 0 || ldc % 4 != 0) return VBR_EINVAL;
    if ((reinterpret_cast<uintptr_t>(B_dev) & 15) != 0 || (reinterpret_cast<uintptr_t>(C_dev) & 15) != 0) return VBR_EINVAL;
    const char *d = static_cast<const char *>(h->dev);
    const vbrk::EntryRowsDev rows{reinterpret_cast<const vbrk::EntryRow *>(d), d + h->entry_off, h->rows.near};
    const vbrk::EntryLaunch L = vbrk::plan_entry_rows(h->rows.start, h->n_cols, N, ldb % 64 == 0 && (reinterpret_cast<uintptr_t>(B_dev) & 127) == 0);
    return vbrk::launch_entry_rows(L, h->dtype, rows, h->n_rows, h->n_cols, B_dev, ldb, C_dev, ldc, N, hip_stream);
}

extern "C" void csr_free(csr_dev_t *h) { delete h; }
