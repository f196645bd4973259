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
#include "vbr_host.h"

struct csr_dev {
    int64_t n_rows = 0, n_cols = 0, nnz = 0;
    int32_t dtype = 0;
    vbrk::EntryRows rows;
    int64_t row_off = 0, col_off = 0, val_off = 0, total = 256;
    void *dev = nullptr;
};

namespace vbrk {
namespace {

constexpr int kCsrThreads = 256;     // 4 waves

typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));

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

template <int I>
__device__ __forceinline__ uint32_t row_lane(uint32_t x)     // lane I of every row of 16 lanes, to the whole row
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + I, 0xf, 0xf, false);
}

template <int U>
__device__ __forceinline__ uint32_t row_pair(uint32_t x)     // lane 2U of every row of 16 lanes to its first eight, lane 2U + 1 to the others
{
    const int lo = __builtin_amdgcn_update_dpp(0, (int)x, 0x150 + 2 * U, 0xf, 0x3, false);
    return (uint32_t)__builtin_amdgcn_update_dpp(lo, (int)x, 0x150 + 2 * U + 1, 0xf, 0xc, false);
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
// Measured on a graph of 16384 nodes with 426 000 entries (rows of 0 to 3600), with B and C beyond the caches, N = 4096: 680 -> 208 us
// (17 TB/s of gathered B); N = 256: 329 -> 22 us.  4096 x 16384 with 1638 entries a row, N = 4096: 3.56 -> 1.90 ms (29 TB/s).
template <int DT, bool WIDE, int LANES>
__global__ void __launch_bounds__(kCsrThreads) entry_rows_kernel(const EntryParams p)
{
    constexpr bool kPair = LANES == 8;                               // 16 lanes own a row, two entries at a time
    constexpr int kGroups = kPair ? 4 : 64 / LANES, kTileN = 8 * LANES;
    __shared__ float partial[3][kTileN];
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
    const int32_t row = pos < p.n_rows ? p.rows.row[pos] : -1;
    const int64_t from = p.rows.start[pos < p.n_rows ? pos : p.n_rows];
    const int32_t len = (int32_t)(p.rows.start[pos < p.n_rows ? pos + 1 : p.n_rows] - from);
    const int32_t max_len = __builtin_amdgcn_readfirstlane(len);     // the first row of a wave is its longest
    const int step = 16 * parts;
    const int e0 = parts * s16 + part;                               // this lane's entry of a batch

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
    auto add = [&](uint32_t a_bits, const uint4v b) {
        const float a = __builtin_bit_cast(float, a_bits);
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] = __builtin_fmaf(a, half_to_f32<DT>(b[i >> 1], i & 1), acc[i]);
    };
    auto fetch = [&](int base, int32_t &col, uint32_t &a) {
        col = -1;
        a = 0;
        if (base + e0 < len) {
            col = p.rows.col[from + base + e0];
            a = p.rows.val[from + base + e0];
        }
    };
    int32_t col;
    uint32_t abits;
    fetch(0, col, abits);
    for (int base = 0; base < max_len; base += step) {
        const uint32_t off = WIDE ? (uint32_t)col : col >= 0 ? (uint32_t)col * ldb_bytes : 0xFFFFF000u;
        const uint32_t a = __builtin_bit_cast(uint32_t, half_to_f32<DT>(abits, 0));
        if (base + step < max_len) fetch(base + step, col, abits);
        const int left = max_len - base;                             // entries of the longest row of the wave
        const int rounds = (left + parts - 1) / parts;
        uint4v b[8];
        if constexpr (kPair) {
#define ENTRY_LOAD(U) b[U] = load(row_pair<U>(off))
#define ENTRY_ADD(U) add(row_pair<U>(a), b[U])
            ENTRY_LOAD(0); ENTRY_LOAD(1); ENTRY_LOAD(2); ENTRY_LOAD(3);
            if (rounds > 8) { ENTRY_LOAD(4); ENTRY_LOAD(5); ENTRY_LOAD(6); ENTRY_LOAD(7); }
            ENTRY_ADD(0); ENTRY_ADD(1); ENTRY_ADD(2); ENTRY_ADD(3);
            if (rounds > 8) { ENTRY_ADD(4); ENTRY_ADD(5); ENTRY_ADD(6); ENTRY_ADD(7); }
#undef ENTRY_LOAD
#undef ENTRY_ADD
        } else {
#define ENTRY_LOAD(U, S) b[U] = load(row_lane<U + S>(off))
#define ENTRY_ADD(U, S) add(row_lane<U + S>(a), b[U])
            ENTRY_LOAD(0, 0); ENTRY_LOAD(1, 0); ENTRY_LOAD(2, 0); ENTRY_LOAD(3, 0);
            if (rounds > 4) { ENTRY_LOAD(4, 0); ENTRY_LOAD(5, 0); ENTRY_LOAD(6, 0); ENTRY_LOAD(7, 0); }
            ENTRY_ADD(0, 0); ENTRY_ADD(1, 0); ENTRY_ADD(2, 0); ENTRY_ADD(3, 0);
            if (rounds > 8) { ENTRY_LOAD(0, 8); ENTRY_LOAD(1, 8); ENTRY_LOAD(2, 8); ENTRY_LOAD(3, 8); }
            if (rounds > 4) { ENTRY_ADD(4, 0); ENTRY_ADD(5, 0); ENTRY_ADD(6, 0); ENTRY_ADD(7, 0); }
            if (rounds > 12) { ENTRY_LOAD(4, 8); ENTRY_LOAD(5, 8); ENTRY_LOAD(6, 8); ENTRY_LOAD(7, 8); }
            if (rounds > 8) { ENTRY_ADD(0, 8); ENTRY_ADD(1, 8); ENTRY_ADD(2, 8); ENTRY_ADD(3, 8); }
            if (rounds > 12) { ENTRY_ADD(4, 8); ENTRY_ADD(5, 8); ENTRY_ADD(6, 8); ENTRY_ADD(7, 8); }
#undef ENTRY_LOAD
#undef ENTRY_ADD
        }
    }
    if constexpr (kPair) {
#pragma unroll
        for (int i = 0; i < 8; ++i) acc[i] += __shfl_xor(acc[i], 8);
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
    const int n = n0 + chunk0 * 8;
    if (row >= 0 && n < p.N && (parts == 1 || g == 0)) {
        float *c = p.C + row * p.ldc + n;
        if constexpr (kPair) {                                       // each half of the 16 lanes stores four of the eight columns
            const int hi = lane >> 3 & 1;
            const float4v out = hi ? float4v{acc[4], acc[5], acc[6], acc[7]} : float4v{acc[0], acc[1], acc[2], acc[3]};
            __builtin_nontemporal_store(out, reinterpret_cast<float4v *>(c + 4 * hi));
        } else {
            __builtin_nontemporal_store(float4v{acc[0], acc[1], acc[2], acc[3]}, reinterpret_cast<float4v *>(c));
            __builtin_nontemporal_store(float4v{acc[4], acc[5], acc[6], acc[7]}, reinterpret_cast<float4v *>(c + 4));
        }
    }
}

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
    // B within 4 GiB (less a page for the offset that stands for "no entry"): 32-bit offsets from its first element
    const int64_t b_bytes = n_cols > 0 ? ((n_cols - 1) * ldb + N) * 2 : 0;
    const bool wide = b_bytes > 0xFFFFF000ll;
    p.b_bytes = wide ? 0 : (uint32_t)b_bytes;
    p.n_rows = (int32_t)n_rows;
    p.N = (int32_t)N;
    p.n_ntiles = (int32_t)((N + 8 * L.lanes - 1) / (8 * L.lanes));
    p.map = column_map((uint32_t)p.n_ntiles, L.even);
    p.n_huge = L.n_huge;
    p.n_long = L.n_long;
    p.n_waves = (int32_t)L.waves;
    if (L.waves > INT32_MAX || L.grid > INT32_MAX) return VBR_EUNSUPPORTED;
    const int variant = (dtype == VBR_F16 ? 0 : 6) + (wide ? 3 : 0) + (L.lanes == 32 ? 2 : L.lanes == 16 ? 1 : 0);
    void (*const kernels[12])(EntryParams) = {
        entry_rows_kernel<VBR_F16, false, 8>, entry_rows_kernel<VBR_F16, false, 16>, entry_rows_kernel<VBR_F16, false, 32>,
        entry_rows_kernel<VBR_F16, true, 8>, entry_rows_kernel<VBR_F16, true, 16>, entry_rows_kernel<VBR_F16, true, 32>,
        entry_rows_kernel<VBR_BF16, false, 8>, entry_rows_kernel<VBR_BF16, false, 16>, entry_rows_kernel<VBR_BF16, false, 32>,
        entry_rows_kernel<VBR_BF16, true, 8>, entry_rows_kernel<VBR_BF16, true, 16>, entry_rows_kernel<VBR_BF16, true, 32>};
    hipLaunchKernelGGL(kernels[variant], dim3((unsigned)L.grid), dim3(kCsrThreads), 0, static_cast<hipStream_t>(hip_stream), p);
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
        vbrk::make_entry_rows(csr, team, 0, h->rows);
        h->row_off = vbrk::align_up256((csr->n_rows + 1) * 8);
        h->col_off = vbrk::align_up256(h->row_off + csr->n_rows * 4);
        h->val_off = vbrk::align_up256(h->col_off + csr->nnz * 4);
        h->total = vbrk::align_up256(h->val_off + csr->nnz * 2 + 256);
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
    const Part parts[4] = {
        {0, h->rows.start.data(), h->rows.start.size() * 8},
        {h->row_off, h->rows.row.data(), h->rows.row.size() * 4},
        {h->col_off, h->rows.col.data(), h->rows.col.size() * 4},
        {h->val_off, h->rows.val.data(), h->rows.val.size() * 2},
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
    const vbrk::EntryRowsDev rows{reinterpret_cast<const int64_t *>(d), reinterpret_cast<const int32_t *>(d + h->row_off),
                                  reinterpret_cast<const int32_t *>(d + h->col_off), reinterpret_cast<const uint16_t *>(d + h->val_off)};
    const vbrk::EntryLaunch L = vbrk::plan_entry_rows(h->rows.start, h->n_cols, N, ldb % 64 == 0 && (reinterpret_cast<uintptr_t>(B_dev) & 127) == 0);
    return vbrk::launch_entry_rows(L, h->dtype, rows, h->n_rows, h->n_cols, B_dev, ldb, C_dev, ldc, N, hip_stream);
}

extern "C" void csr_free(csr_dev_t *h) { delete h; }
