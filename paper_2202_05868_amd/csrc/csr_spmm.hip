// Comparator kernel: C = A.B straight from CSR (the role the sparse-library routine plays in
// section 4.4.2 of the paper), one fp32 accumulator per output element, no matrix units.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <new>
#include <vector>

#include "vbr_host.h"

struct csr_dev {
    int64_t n_rows = 0, n_cols = 0, nnz = 0;
    int32_t dtype = 0;
    std::vector<int64_t> row_ptr;
    std::vector<int32_t> col_idx;
    std::vector<uint16_t> vals;
    std::vector<int32_t> order;      // rows, longest first
    int64_t col_off = 0, val_off = 0, order_off = 0, total = 256;
    void *dev = nullptr;
};

namespace vbrk {
namespace {

constexpr int kCsrThreads = 256;     // 4 waves
constexpr int kCsrLongRow = 256;     // entries beyond which a row gets a wave of its own ...
constexpr int kCsrHugeRow = 1024;    // ... and a workgroup of its own

typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
typedef float float2v __attribute__((ext_vector_type(2)));
typedef float float4v __attribute__((ext_vector_type(4)));

struct CsrParams {
    const int64_t *row_ptr;
    const int32_t *col_idx;
    const uint16_t *vals;
    const int32_t *order;
    const uint16_t *B;
    float *C;
    int64_t ldb, ldc;
    uint32_t b_bytes;                // bytes from B's first element to the end of its last row (WIDE: not used)
    int32_t n_rows, n_huge, n_long, N, n_waves, n_ntiles;
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
//   - rows beyond kCsrLongRow entries get a whole wave, rows beyond kCsrHugeRow a workgroup: its 64 / LANES (256 / LANES)
//     groups of lanes take the entries in turn, and the partial sums are added at the end.
// Entries past the end of a row are loads out of the buffer's range: they return zeros and cost no traffic.
// LANES: 8, 16 or 32 (64, 128 or 256 columns a wave), chosen by csr_spmm.  With 8, the 16 lanes of a row take two entries
// at a time and add their halves at the end.
// Measured on a graph of 16384 nodes with 426 000 entries (rows of 0 to 3600), with B and C beyond the caches, N = 4096: 680 -> 208 us
// (17 TB/s of gathered B); N = 256: 329 -> 22 us.  4096 x 16384 with 1638 entries a row, N = 4096: 3.56 -> 1.90 ms (29 TB/s).
template <int DT, bool WIDE, int LANES>
__global__ void __launch_bounds__(kCsrThreads) csr_spmm_kernel(const CsrParams p)
{
    constexpr bool kPair = LANES == 8;                               // 16 lanes own a row, two entries at a time
    constexpr int kGroups = kPair ? 4 : 64 / LANES, kTileN = 8 * LANES;
    __shared__ float partial[3][kTileN];
    const int lane = threadIdx.x & 63, g = lane / (64 / kGroups), s16 = lane & 15, chunk0 = lane % LANES;
    // workgroup -> (column tile, four waves' rows): workgroups are dealt to the 8 L2 domains round-robin
    const int T = (p.n_waves + 3) / 4, Q = p.n_ntiles;
    const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
    int ntile, tile;
    if (Q >= 8) {
        ntile = x + 8 * (j / T);
        tile = j % T;
    } else {
        ntile = x % Q;
        tile = x / Q + ((8 - ntile + Q - 1) / Q) * j;
    }
    const int in_wg = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), wave = tile * 4 + in_wg;
    if (ntile >= Q || tile >= T || wave >= p.n_waves) return;
    // parts: the groups of lanes that share a row; part: this group's number among them
    const bool huge = tile < p.n_huge, whole = !huge && wave < 4 * p.n_huge + p.n_long;
    const int parts = huge ? 4 * kGroups : whole ? kGroups : 1, part = huge ? in_wg * kGroups + g : whole ? g : 0;
    const int first = p.n_huge + p.n_long, pos = huge ? tile : whole ? wave - 3 * p.n_huge : first + (wave - 3 * p.n_huge - first) * kGroups + g;
    const int32_t row = pos < p.n_rows ? p.order[pos] : -1;
    const int64_t p0 = row >= 0 ? p.row_ptr[row] : 0;
    const int32_t len = row >= 0 ? (int32_t)(p.row_ptr[row + 1] - p0) : 0;
    const int32_t max_len = __builtin_amdgcn_readfirstlane(len);    // the first row of a wave is its longest
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
        const bool ok = base + e0 < len;
        const int64_t at = ok ? p0 + base + e0 : 0;
        col = -1;
        a = 0;
        if (ok) {
            col = p.col_idx[at];
            a = p.vals[at];
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
#define CSR_LOAD(U, S) b[U] = load(row_lane<U + S>(off))
#define CSR_ADD(U, S) add(row_lane<U + S>(a), b[U])
        if constexpr (kPair) {
#define CSR_LOAD2(U) b[U] = load(row_pair<U>(off))
#define CSR_ADD2(U) add(row_pair<U>(a), b[U])
            CSR_LOAD2(0); CSR_LOAD2(1); CSR_LOAD2(2); CSR_LOAD2(3);
            if (rounds > 8) { CSR_LOAD2(4); CSR_LOAD2(5); CSR_LOAD2(6); CSR_LOAD2(7); }
            CSR_ADD2(0); CSR_ADD2(1); CSR_ADD2(2); CSR_ADD2(3);
            if (rounds > 8) { CSR_ADD2(4); CSR_ADD2(5); CSR_ADD2(6); CSR_ADD2(7); }
#undef CSR_LOAD2
#undef CSR_ADD2
        } else {
            CSR_LOAD(0, 0); CSR_LOAD(1, 0); CSR_LOAD(2, 0); CSR_LOAD(3, 0);
            if (rounds > 4) { CSR_LOAD(4, 0); CSR_LOAD(5, 0); CSR_LOAD(6, 0); CSR_LOAD(7, 0); }
            CSR_ADD(0, 0); CSR_ADD(1, 0); CSR_ADD(2, 0); CSR_ADD(3, 0);
            if (rounds > 8) { CSR_LOAD(0, 8); CSR_LOAD(1, 8); CSR_LOAD(2, 8); CSR_LOAD(3, 8); }
            if (rounds > 4) { CSR_ADD(4, 0); CSR_ADD(5, 0); CSR_ADD(6, 0); CSR_ADD(7, 0); }
            if (rounds > 12) { CSR_LOAD(4, 8); CSR_LOAD(5, 8); CSR_LOAD(6, 8); CSR_LOAD(7, 8); }
            if (rounds > 8) { CSR_ADD(0, 8); CSR_ADD(1, 8); CSR_ADD(2, 8); CSR_ADD(3, 8); }
            if (rounds > 12) { CSR_ADD(4, 8); CSR_ADD(5, 8); CSR_ADD(6, 8); CSR_ADD(7, 8); }
        }
#undef CSR_LOAD
#undef CSR_ADD
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
    if (parts > 1 && g != 0) return;
    const int n = n0 + chunk0 * 8;
    if (row < 0 || n >= p.N) return;
    if constexpr (kPair) {                                           // each half of the 16 lanes stores four of the eight columns
        const int hi = lane >> 3 & 1;
        const float4v out = hi ? float4v{acc[4], acc[5], acc[6], acc[7]} : float4v{acc[0], acc[1], acc[2], acc[3]};
        __builtin_nontemporal_store(out, reinterpret_cast<float4v *>(p.C + row * p.ldc + n + 4 * hi));
        return;
    }
    float *c = p.C + row * p.ldc + n;
    __builtin_nontemporal_store(float4v{acc[0], acc[1], acc[2], acc[3]}, reinterpret_cast<float4v *>(c));
    __builtin_nontemporal_store(float4v{acc[4], acc[5], acc[6], acc[7]}, reinterpret_cast<float4v *>(c + 4));
}

inline int64_t align_up256(int64_t x) { return (x + 255) / 256 * 256; }

}  // namespace
}  // namespace vbrk

extern "C" int csr_spmm_create(const vbr_csr_t *csr, csr_dev_t **out)
{
    if (!csr || !out) return VBR_EINVAL;
    *out = nullptr;
    const int rc = vbrk::validate_csr(csr, true);
    if (rc != VBR_OK) return rc;
    try {
        csr_dev *h = new csr_dev();
        h->n_rows = csr->n_rows;
        h->n_cols = csr->n_cols;
        h->nnz = csr->nnz;
        h->dtype = csr->dtype;
        h->row_ptr.assign(csr->row_ptr, csr->row_ptr + csr->n_rows + 1);
        h->col_idx.assign(csr->col_idx, csr->col_idx + csr->nnz);
        const uint16_t *v = static_cast<const uint16_t *>(csr->vals);
        h->vals.assign(v, v + csr->nnz);
        // rows by falling length, by counting (a row has at most n_cols entries)
        int64_t longest = 0;
        for (int64_t i = 0; i < csr->n_rows; ++i) longest = std::max(longest, csr->row_ptr[i + 1] - csr->row_ptr[i]);
        std::vector<int32_t> at((size_t)longest + 2, 0);
        for (int64_t i = 0; i < csr->n_rows; ++i) ++at[(size_t)(longest - (csr->row_ptr[i + 1] - csr->row_ptr[i])) + 1];
        for (int64_t k = 0; k <= longest; ++k) at[(size_t)k + 1] += at[(size_t)k];
        h->order.resize((size_t)csr->n_rows);
        for (int64_t i = 0; i < csr->n_rows; ++i) h->order[(size_t)at[(size_t)(longest - (csr->row_ptr[i + 1] - csr->row_ptr[i]))]++] = (int32_t)i;
        h->col_off = vbrk::align_up256((csr->n_rows + 1) * 8);
        h->val_off = vbrk::align_up256(h->col_off + csr->nnz * 4);
        h->order_off = vbrk::align_up256(h->val_off + csr->nnz * 2);
        h->total = vbrk::align_up256(h->order_off + csr->n_rows * 4 + 256);
        *out = h;
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
        {0, h->row_ptr.data(), h->row_ptr.size() * 8},
        {h->col_off, h->col_idx.data(), h->col_idx.size() * 4},
        {h->val_off, h->vals.data(), h->vals.size() * 2},
        {h->order_off, h->order.data(), h->order.size() * 4},
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
    vbrk::CsrParams p;
    p.row_ptr = reinterpret_cast<const int64_t *>(d);
    p.col_idx = reinterpret_cast<const int32_t *>(d + h->col_off);
    p.vals = reinterpret_cast<const uint16_t *>(d + h->val_off);
    p.order = reinterpret_cast<const int32_t *>(d + h->order_off);
    p.B = static_cast<const uint16_t *>(B_dev);
    p.C = C_dev;
    p.ldb = ldb;
    p.ldc = ldc;
    // B within 4 GiB (less a page for the offset that stands for "no entry"): 32-bit offsets from its first element
    const int64_t b_bytes = h->n_cols > 0 ? ((h->n_cols - 1) * ldb + N) * 2 : 0;
    const bool wide = b_bytes > 0xFFFFF000ll;
    p.b_bytes = wide ? 0 : (uint32_t)b_bytes;
    p.n_rows = (int32_t)h->n_rows;
    p.N = (int32_t)N;
    // Lanes a row, i.e. columns a wave (8 per lane): narrow tiles keep the B that a tile touches smallest and give many waves,
    // wide ones fetch and store B and C in longer pieces, which is what counts once they come from memory.  Measured with 64 / 128
    // / 256 columns: 32768 x 32768, 16 entries a row, N = 256: 28.8 / 32 / 38 us; graph of 16384 nodes, N = 256: 22 / 26 / 37,
    // N = 4096: 358 / 253 / 208, of 4096 nodes, N = 2048: 33 / 29 / 34; 224 entries a row, N = 512: 213 / 185 / 213, 388, N = 1024:
    // 365 / 270 / 241.  Rows of B that start inside a cache line lie in one line more, which 64 columns pay twice.
    const bool aligned = ldb % 64 == 0 && (reinterpret_cast<uintptr_t>(B_dev) & 127) == 0;
    const int lanes = N <= 64 || (N <= 256 && aligned) ? 8 : N > 128 && (!aligned || (N >= 1024 && h->nnz * N >= ((int64_t)1 << 29))) ? 32 : 16;
    p.n_ntiles = (int32_t)((N + 8 * lanes - 1) / (8 * lanes));
    // A workgroup for a row costs its barrier and the fourfold sum; it pays where one wave would still be at the row when
    // the rest is done, i.e. beyond the share of all entries that one of 4096 waves takes (graph, N = 256: 66 -> 26 us;
    // a matrix whose rows all have 1638 entries is 20 % slower with it and stays without).
    const int64_t huge_len = std::max<int64_t>(vbrk::kCsrHugeRow, h->nnz * p.n_ntiles / 4096);
    auto longer_than = [&](int64_t len) {
        return std::partition_point(h->order.begin(), h->order.end(), [&](int32_t r) { return h->row_ptr[r + 1] - h->row_ptr[r] > len; }) - h->order.begin();
    };
    const int64_t n_huge = longer_than(huge_len), n_long = longer_than(vbrk::kCsrLongRow) - n_huge;
    p.n_huge = (int32_t)n_huge;
    p.n_long = (int32_t)n_long;
    const int64_t rest = h->n_rows - n_huge - n_long, waves = 4 * n_huge + n_long + (rest * std::max(lanes, 16) + 63) / 64;
    p.n_waves = (int32_t)waves;
    const int64_t T = (waves + 3) / 4, Q = p.n_ntiles;
    const int64_t grid = Q >= 8 ? 8 * ((Q + 7) / 8) * T : 8 * ((T + 8 / Q - 1) / (8 / Q));
    if (waves > INT32_MAX || grid > INT32_MAX) return VBR_EUNSUPPORTED;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    const int variant = (h->dtype == VBR_F16 ? 0 : 6) + (wide ? 3 : 0) + (lanes == 32 ? 2 : lanes == 16 ? 1 : 0);
    void (*const kernels[12])(vbrk::CsrParams) = {
        vbrk::csr_spmm_kernel<VBR_F16, false, 8>, vbrk::csr_spmm_kernel<VBR_F16, false, 16>, vbrk::csr_spmm_kernel<VBR_F16, false, 32>,
        vbrk::csr_spmm_kernel<VBR_F16, true, 8>, vbrk::csr_spmm_kernel<VBR_F16, true, 16>, vbrk::csr_spmm_kernel<VBR_F16, true, 32>,
        vbrk::csr_spmm_kernel<VBR_BF16, false, 8>, vbrk::csr_spmm_kernel<VBR_BF16, false, 16>, vbrk::csr_spmm_kernel<VBR_BF16, false, 32>,
        vbrk::csr_spmm_kernel<VBR_BF16, true, 8>, vbrk::csr_spmm_kernel<VBR_BF16, true, 16>, vbrk::csr_spmm_kernel<VBR_BF16, true, 32>};
    hipLaunchKernelGGL(kernels[variant], dim3((unsigned)grid), dim3(vbrk::kCsrThreads), 0, stream, p);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) { vbrk::set_last_hip_error((int)e); return VBR_EHIP; }
    return VBR_OK;
}

extern "C" void csr_free(csr_dev_t *h) { delete h; }
