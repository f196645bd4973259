// C = A.B for many row groups of one slab (16 rows) against a wide B: the groups of a workgroup share the B rows they have in common.
#include <hip/hip_runtime.h>

#include <cstdint>

#include "vbr_device.h"
#include "vbr_host.h"

namespace vbrk {
namespace {

typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) short8v *lds_short8_ptr;
typedef __attribute__((address_space(3))) uint2v *lds_uint2_ptr;
typedef __attribute__((address_space(3))) uint4v *lds_uint4_ptr;
typedef __attribute__((address_space(3))) float4v *lds_float4_ptr;
typedef __attribute__((address_space(3))) unsigned char *lds_u8_ptr;

struct StreamParams {
    const StreamTile *tiles;
    const StreamRecord *steps;
    const int32_t *perm;
    const uint16_t *vals;
    const uint16_t *B;
    float *C;
    int64_t ldb, ldc;
    uint32_t b_bytes, a_bytes;
    const TileDesc *empty;    // tiles without a K-step, whose workgroups follow those of the others
    const int32_t *prow;
    uint32_t first_empty;     // the first of these
    int32_t N, n_tiles, n_ntiles;
    ColumnMap map;
};

constexpr int kStreamThreads = 64 * kStreamWaves;

// acc[g][f] += b[f] . a for the four f, g being bits 4 i .. 4 i + 3 of `groups`; nothing where that is kStreamGroups.  Written as a jump to one of eight pieces of
// 64 bytes, since as a switch every case got registers of its own and copies from and to those of the others (270 registers spilled).
#define STREAM_MULTIPLY(T) \
    "s_getpc_b64 s[90:91]\n"\
    ".Lstream_here%=:\n\t"\
    "s_bfe_u32 s92, %37, %38\n\t"\
    "s_lshl_b32 s92, s92, 6\n\t"\
    "s_add_u32 s92, s92, .Lstream_table%=-.Lstream_here%=\n\t"\
    "s_add_u32 s90, s90, s92\n\t"\
    "s_addc_u32 s91, s91, 0\n\t"\
    "s_setpc_b64 s[90:91]\n\t"\
    ".p2align 6\n"\
    ".Lstream_table%=:\n\t"\
    "v_mfma_f32_16x16x32_" T " %0, %32, %36, %0\n\tv_mfma_f32_16x16x32_" T " %1, %33, %36, %1\n\t"\
    "v_mfma_f32_16x16x32_" T " %2, %34, %36, %2\n\tv_mfma_f32_16x16x32_" T " %3, %35, %36, %3\n\t"\
    "s_branch .Lstream_end%=\n\t.p2align 6\n\t"\
    "v_mfma_f32_16x16x32_" T " %4, %32, %36, %4\n\tv_mfma_f32_16x16x32_" T " %5, %33, %36, %5\n\t"\
    "v_mfma_f32_16x16x32_" T " %6, %34, %36, %6\n\tv_mfma_f32_16x16x32_" T " %7, %35, %36, %7\n\t"\
    "s_branch .Lstream_end%=\n\t.p2align 6\n\t"\
    "v_mfma_f32_16x16x32_" T " %8, %32, %36, %8\n\tv_mfma_f32_16x16x32_" T " %9, %33, %36, %9\n\t"\
    "v_mfma_f32_16x16x32_" T " %10, %34, %36, %10\n\tv_mfma_f32_16x16x32_" T " %11, %35, %36, %11\n\t"\
    "s_branch .Lstream_end%=\n\t.p2align 6\n\t"\
    "v_mfma_f32_16x16x32_" T " %12, %32, %36, %12\n\tv_mfma_f32_16x16x32_" T " %13, %33, %36, %13\n\t"\
    "v_mfma_f32_16x16x32_" T " %14, %34, %36, %14\n\tv_mfma_f32_16x16x32_" T " %15, %35, %36, %15\n\t"\
    "s_branch .Lstream_end%=\n\t.p2align 6\n\t"\
    "v_mfma_f32_16x16x32_" T " %16, %32, %36, %16\n\tv_mfma_f32_16x16x32_" T " %17, %33, %36, %17\n\t"\
    "v_mfma_f32_16x16x32_" T " %18, %34, %36, %18\n\tv_mfma_f32_16x16x32_" T " %19, %35, %36, %19\n\t"\
    "s_branch .Lstream_end%=\n\t.p2align 6\n\t"\
    "v_mfma_f32_16x16x32_" T " %20, %32, %36, %20\n\tv_mfma_f32_16x16x32_" T " %21, %33, %36, %21\n\t"\
    "v_mfma_f32_16x16x32_" T " %22, %34, %36, %22\n\tv_mfma_f32_16x16x32_" T " %23, %35, %36, %23\n\t"\
    "s_branch .Lstream_end%=\n\t.p2align 6\n\t"\
    "v_mfma_f32_16x16x32_" T " %24, %32, %36, %24\n\tv_mfma_f32_16x16x32_" T " %25, %33, %36, %25\n\t"\
    "v_mfma_f32_16x16x32_" T " %26, %34, %36, %26\n\tv_mfma_f32_16x16x32_" T " %27, %35, %36, %27\n\t"\
    "s_branch .Lstream_end%=\n\t.p2align 6\n\t"\
    "v_mfma_f32_16x16x32_" T " %28, %32, %36, %28\n\tv_mfma_f32_16x16x32_" T " %29, %33, %36, %29\n\t"\
    "v_mfma_f32_16x16x32_" T " %30, %34, %36, %30\n\tv_mfma_f32_16x16x32_" T " %31, %35, %36, %31\n\t"\
    "s_branch .Lstream_end%=\n\t.p2align 6\n\t"\
    "\n.Lstream_end%=:\n"
#define STREAM_ACC(g) "+a"(acc[g][0]), "+a"(acc[g][1]), "+a"(acc[g][2]), "+a"(acc[g][3])
#define STREAM_OPERANDS \
    : STREAM_ACC(0), STREAM_ACC(1), STREAM_ACC(2), STREAM_ACC(3), STREAM_ACC(4), STREAM_ACC(5), STREAM_ACC(6), STREAM_ACC(7) \
    : "v"(b[0]), "v"(b[1]), "v"(b[2]), "v"(b[3]), "v"(a), "s"(groups), "n"(4 * I | 4 << 16) : "s90", "s91", "s92", "scc"
template <int DT, int I>
__device__ __forceinline__ void multiply(float4v (&acc)[kStreamGroups][kStreamN / 16], const short8v (&b)[kStreamN / 16], short8v a, int32_t groups)
{
    static_assert(kStreamGroups == 8 && kStreamN == 64, "as written");
    if constexpr (DT == VBR_F16) asm volatile(STREAM_MULTIPLY("f16") STREAM_OPERANDS);
    else asm volatile(STREAM_MULTIPLY("bf16") STREAM_OPERANDS);
}

// Rows of A without entries: zeros, a row of 256 columns a wave.
__device__ __forceinline__ void zero_rows(const StreamParams &p)
{
    const int chunks = (p.N + kTileN - 1) / kTileN, i = (int)(blockIdx.x - p.first_empty), lane = threadIdx.x & 63, n = i % chunks * kTileN + 4 * lane;
    const TileDesc td = p.empty[i / chunks];
    const int32_t rows = lane < td.n_rows ? p.prow[td.row_begin + lane] : -1;
#pragma unroll
    for (int r = 0; r < kMaxGatherSlabs * kSlabRows; r += kStreamWaves) {
        const int64_t row = __shfl(rows, r + (int)(threadIdx.x >> 6));          // a position of the row list may be padding (-1)
        if (row >= 0 && n < p.N) __builtin_nontemporal_store(float4v{0.f, 0.f, 0.f, 0.f}, reinterpret_cast<float4v *>(p.C + row * p.ldc + n));
    }
}

// 16 bytes of a row of C, at byte `at` of the `bytes` that a workgroup has of it.  Nothing reads them soon, so they go past the caches; but a cache line of which
// this is not all, where rows of C begin inside lines, is finished by another workgroup, and its parts are collected in the caches (with the hint for all, for
// these only not, for none; kernel times: 127 groups and 1000 rows without entries, N = 8184 55, 42 and 42 us, 229 groups, N = 3992 44, 37 and 37; 2452 groups, C
// of 277 MB, 240, 221 and 250; by halves of lines instead of lines 51, 41 and 238).  Rows that begin at half a line have the hint for all (127
// groups, N = 8176 40.6 and 38.3, but 4096 x 16384 at 10 %, N = 3504 103 and 105, 3056 99 and 101), as those that begin with one (4096: 100 and 107).
template <bool WHOLE>
__device__ __forceinline__ void store(float *to, float4v x, int at, int bytes)
{
    float4v *const to4 = reinterpret_cast<float4v *>(to);
    const int off = (int)(reinterpret_cast<uintptr_t>(to) & 127);
    if constexpr (WHOLE) {
        __builtin_nontemporal_store(x, to4);
    } else if (off <= at && at - off + 128 <= bytes) {
        asm volatile("" ::: "memory");                   // or the compiler makes one store of the two, without the hint
        __builtin_nontemporal_store(x, to4);
        asm volatile("" ::: "memory");
    } else {
        *to4 = x;
    }
}

// The tile kernel gathers the B rows of every group for itself, at 16 rows a group one load of 1 KiB for every four matrix instructions, and the load path
// bounds it.  Here a workgroup owns up to 64 groups and 64 columns of C and brings every unit of 16 B rows into LDS once for all of them: at 10 % of
// the blocks 6.4 groups use it.  A unit is used when a group comes to it, so what is brought and multiplied when is a schedule that the host
// makes once (stream_schedule.h); a step of it, between two barriers:
//   - a wave multiplies up to OPS K-steps of its eight groups, any group in any place: the 128 accumulators stay in place and a jump picks the four instructions;
//   - the operands of a K-step are its two units out of LDS, wherever these lie: half of the lanes read the one and half the other, 16 bytes a lane of
//     columns that were turned round on their way in, and no transposed read;
//   - its fragment of A, which no other wave needs, comes straight into registers, asked for a step before;
//   - the units: a lane loads eight columns of four rows, turns them by byte permutes and writes 8 bytes of each column, two steps later.  A row of 16
//     lanes writes 128 bytes in one piece (8 clocks a write where it did not, else 4), and operand f of the LDS image holds columns f and 4 + f of eight;
//   - where units and fragments are goes into addresses by the DPP of an addition, from a record of the step that each row of 16 lanes holds.
// No load that the products wait for stands in a branch, so that every wait is for one of them and not for all.  (Those that only bring lines into the L2 do.)
// A CU has some 80 lines on the way whatever it asks for, and returns them in order, so a line that comes from HBM holds up what follows it.  The row tiles
// on a domain ask for the same units at about the same time; each brings a quarter of them into the L2 three steps ahead, four bytes of a line a
// lane (other operands in every call: 16 x 16 blocks at 10 %, 4096 x 16384, N = 4096 116 and 108 us, 2048: 108 and 92).
// That matrix: 163 us in the tile kernel, 109 here, with the same operands in every call 145 and 93.  Its loads alone take 73, all but the loads 50, all but the
// matrix instructions 78.  By its profile (same operands) a CU makes 6900 loads, 29 clocks each, for 20 of which the texture-address unit is busy, 68 % of
// the time; the matrix unit is 26 % busy, waves wait 38 % of their time.  LDS counts 16.4 million cycles of bank conflicts, 32 % of the CUs' cycles, about four for each
// of the 4.0 million reads of operands, which the contiguous reads of a probe do without.  No unit is full: steps are short, and a CU has one workgroup.
// Deeper rings for A or B, loads of no value left out by the execution mask, other ways to deal column tiles to domains, row tiles that begin at different
// places of K: within 4 %.
template <int DT, int OPS, bool WHOLE>
__global__ void __launch_bounds__(kStreamThreads, 2) vbr_spmm_stream_kernel(const StreamParams p)
{
    constexpr int F = kStreamN / 16;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[(kStreamSlots + 1) * kStreamUnitBytes];
    if (blockIdx.x >= p.first_empty) return zero_rows(p);
    int tile, ntile;
    if (!map_workgroup(blockIdx.x, p.n_tiles, p.n_ntiles, p.map, tile, ntile)) return;
    const StreamTile &td = p.tiles[tile];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4, s16 = lane & 15;
    const int n0 = ntile * kStreamN;
    const lds_u8_ptr sm = (lds_u8_ptr)smem;
    const int n_steps = __builtin_amdgcn_readfirstlane(td.n_steps);

    float4v acc[kStreamGroups][F];
#pragma unroll
    for (int g = 0; g < kStreamGroups; ++g)
#pragma unroll
        for (int f = 0; f < F; ++f) acc[g][f] = float4v{0.f, 0.f, 0.f, 0.f};

    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.vals), 0, (int)p.a_bytes, 0x00020000);
    const uint32_t a_lane = lane * 16;
    auto load_a = [&](uint32_t at) -> uint4v { return __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, (int)(at + a_lane), 0, 0)); };

    // B: lane l brings columns 8 (l % 8) .. + 7 of four consecutive rows of one of the wave's two units
    const int cl = lane & 7, hf = lane >> 3 & 1, o = lane >> 4 & 1;
    const int columns = p.N - n0 < kStreamN ? p.N - n0 : kStreamN, last_chunk = columns / 8 - 1;
    const uint32_t ldb_bytes = (uint32_t)(p.ldb * 2);
    const __amdgpu_buffer_rsrc_t b_rsrc =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(p.B + n0), 0, (int)(p.b_bytes - (uint32_t)n0 * 2), 0x00020000);
    const uint32_t b_lane = (uint32_t)(cl <= last_chunk ? cl : last_chunk) * 16 + (uint32_t)(8 * hf + 4 * o) * ldb_bytes;
    uint4v bs[kStreamAhead][4];
    auto load_unit_rows = [&](auto set, auto i, uint32_t at) {
        bs[set.value][i.value] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(b_rsrc, (int)at, (int)(i.value * ldb_bytes), 0));
        __builtin_amdgcn_sched_barrier(0);
    };
    // turned round into LDS: 8 columns of 4 rows, 8 bytes each
    const uint32_t w_lane = o * 1024 + ((cl ^ (8 * o)) << 4) + hf * 8;      // of the first four columns; the others: the other half of the 256 bytes
    auto write_units = [&](auto set, auto w, uint32_t to) {        // a quarter of them
        const uint4v(&r)[4] = bs[set.value];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const uint32_t sel = h ? 0x07060302u : 0x05040100u;
            const uint2v x = {__builtin_amdgcn_perm(r[1][w.value], r[0][w.value], sel), __builtin_amdgcn_perm(r[3][w.value], r[2][w.value], sel)};
            *(lds_uint2_ptr)(sm + ((to + w_lane) ^ (w.value >> 1 << 7)) + (2 * (w.value & 1) + h) * 256) = x;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    const uint32_t r_lane = (q & 1) * 1024 + ((s16 ^ (8 * (q & 1))) << 4);
    short8v b[2][F];

    // lanes 16 i .. 16 i + 15 hold the 16 pairs of words of one of the two records
    const __amdgpu_buffer_rsrc_t rec_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<StreamRecord *>(p.steps + (int64_t)td.first_step * (2 * kStreamWaves)), 0,
                                                                              (n_steps + 2) * 2 * kStreamWaves * (int)sizeof(StreamRecord), 0x00020000);
    const uint32_t rec_lane = (2 * wave + (lane >> 5)) * (uint32_t)sizeof(StreamRecord) + s16 * 8;
    auto record = [&](int t) -> uint2v {
        return __builtin_bit_cast(uint2v, __builtin_amdgcn_raw_buffer_load_b64(rec_rsrc, (int)rec_lane, t * 2 * kStreamWaves * (int)sizeof(StreamRecord), 0));
    };
    uint2v cur = record(0), nxt = record(1);
    uint4v a[OPS];
#pragma unroll
    for (int i = 0; i < OPS; ++i) a[i] = uint4v{0, 0, 0, 0};
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int set = 0; set < kStreamAhead; ++set) bs[set][i] = uint4v{0, 0, 0, 0};
    constexpr uint32_t kZeros = kStreamSlots * kStreamUnitBytes;
    if (threadIdx.x < kStreamUnitBytes / 16) *(lds_uint4_ptr)(sm + kZeros + threadIdx.x * 16) = uint4v{0, 0, 0, 0};
    asm volatile("" ::"v"(cur), "v"(nxt));                               // waited for here, or every step waits for all loads
    __syncthreads();
#pragma unroll
    for (int f = 0; f < F; ++f) b[0][f] = *(lds_short8_ptr)(sm + kZeros + r_lane + f * 256);
    uint32_t to[kStreamAhead];
#pragma unroll
    for (int set = 0; set < kStreamAhead; ++set) to[set] = kZeros;
    uint32_t early[kStreamAhead] = {0, 0};
    int t = 0;
    auto step = [&](auto set) {
        const uint2v then = record(++t + 1);                   // (there are two more behind the last)
        // lines of B that are to be in the L2: four bytes of each
        asm volatile("" ::"v"(early[set.value]));
        if (__builtin_amdgcn_readlane((int)cur[1], 5) >= 0) {
            const int32_t row = (int32_t)(lane & 16 ? row_lane<6>(cur[1]) : row_lane<5>(cur[1]));
            early[set.value] = __builtin_amdgcn_raw_buffer_load_b32(b_rsrc, (int)(row < 0 ? (uint32_t)kNearBytes : __umul24(row + s16, ldb_bytes)), 0, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        uint32_t row_at = 0;
        const int32_t groups = __builtin_amdgcn_readlane((int)cur[1], 3);
        static_for<OPS>([&](auto i) {
            constexpr int kBuf = (set.value * OPS + i.value) & 1;
            __builtin_amdgcn_sched_barrier(0);
            const uint32_t at = row_lane<i.value>(cur[0]) + r_lane;
#pragma unroll
            for (int f = 0; f < F; ++f) b[kBuf ^ 1][f] = *(lds_short8_ptr)(sm + at + f * 256);
            __builtin_amdgcn_sched_barrier(0);
            multiply<DT, i.value>(acc, b[kBuf], __builtin_bit_cast(short8v, a[i.value]), groups);
            a[i.value] = load_a(row_lane<kStreamMostOps + i.value>(cur[0]));
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (i.value < 2) {
                write_units(set, constant<2 * i.value>(), to[set.value]);
                write_units(set, constant<2 * i.value + 1>(), to[set.value]);
            }
            if constexpr (i.value == 1) {
                to[set.value] = row_lane<2>(cur[1]);
                row_at = (__umul24(row_lane<0>(cur[1]), ldb_bytes) + b_lane) | row_lane<1>(cur[1]);      // none: out of range, which brings zeros
            }
            constexpr int kTurns = OPS - 2, kFirst = i.value < 2 ? 0 : (i.value - 2) * 4 / kTurns, kLast = i.value < 2 ? 0 : (i.value - 1) * 4 / kTurns;
            static_for<kLast - kFirst>([&](auto k) { load_unit_rows(set, constant<kFirst + k.value>(), row_at); });
        });
        __builtin_amdgcn_sched_barrier(0);
        cur = nxt;
        nxt = then;
        // The compiler does not know the matrix instructions, and may read or move the accumulators as soon as the loop ends: eight wait states, inside it
        if constexpr (set.value == kStreamAhead - 1) asm volatile("s_nop 7\n\ts_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    };
    while (t < n_steps) static_for<kStreamAhead>(step);        // (their number is a multiple)

    // lane (q, s16) holds, of row s16 of a group, columns 32 (q % 2) + 4 (q / 2) + 8 r + f: turned round in LDS, whole lines
    constexpr int kOutRow = kStreamN * 4 + 16;
    const lds_u8_ptr out = sm + wave * kSlabRows * kOutRow;
#pragma unroll
    for (int g = 0; g < kStreamGroups; ++g) {
        const int32_t first = td.row_begin[wave * kStreamGroups + g];
        if (first < 0) continue;
        const int32_t c_row = p.perm[first + s16];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            *(lds_float4_ptr)(out + s16 * kOutRow + (q & 1) * 128 + (q >> 1) * 16 + r * 32) = float4v{acc[g][0][r], acc[g][1][r], acc[g][2][r], acc[g][3][r]};
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4v x = *(lds_float4_ptr)(out + (4 * i + q) * kOutRow + s16 * 16);
            const int32_t row = __shfl(c_row, 4 * i + q);
            const int n = n0 + 4 * s16;
            if (n < p.N) store<WHOLE>(p.C + row * p.ldc + n, x, (n - n0) * 4, columns * 4);
        }
    }
}

using StreamKernel = void (*)(StreamParams);
template <int DT, bool WHOLE>
constexpr StreamKernel stream_kernels[kStreamMostOps - kStreamLeastOps + 1] = {
    vbr_spmm_stream_kernel<DT, 4, WHOLE>, vbr_spmm_stream_kernel<DT, 5, WHOLE>, vbr_spmm_stream_kernel<DT, 6, WHOLE>, vbr_spmm_stream_kernel<DT, 7, WHOLE>,
    vbr_spmm_stream_kernel<DT, 8, WHOLE>};

}  // namespace

int launch_stream(const vbr *v, const Launch &L, const void *B_dev, int64_t ldb, float *C_dev, int64_t ldc, int64_t N, void *hip_stream)
{
    const char *d = static_cast<const char *>(v->dev);
    StreamParams p;
    p.tiles = reinterpret_cast<const StreamTile *>(d + v->lay.stream_tiles_off);
    p.steps = reinterpret_cast<const StreamRecord *>(d + v->lay.stream_steps_off);
    p.perm = reinterpret_cast<const int32_t *>(d + v->lay.perm_off);
    p.vals = reinterpret_cast<const uint16_t *>(d + v->lay.vals_off);
    p.B = static_cast<const uint16_t *>(B_dev);
    p.C = C_dev;
    p.ldb = ldb;
    p.ldc = ldc;
    p.b_bytes = (uint32_t)b_bytes_of(v->n_cols, ldb, N);
    p.a_bytes = (uint32_t)(v->vals.size() * 2);
    p.N = (int32_t)N;
    p.n_tiles = (int32_t)v->stream_tiles.size();
    p.n_ntiles = (int32_t)((N + kStreamN - 1) / kStreamN);
    p.map = column_map((uint32_t)p.n_ntiles, L.even);
    p.empty = reinterpret_cast<const TileDesc *>(d + v->lay.tiles_off) + v->n_work;
    p.prow = reinterpret_cast<const int32_t *>(d + v->lay.prow_off);
    p.first_empty = (uint32_t)grid_size(p.n_tiles, p.n_ntiles);
    const bool whole = ldc % 16 == 0 && (reinterpret_cast<uintptr_t>(C_dev) & 63) == 0;
    const StreamKernel *kernels = v->dtype == VBR_F16 ? (whole ? stream_kernels<VBR_F16, true> : stream_kernels<VBR_F16, false>)
                                                      : (whole ? stream_kernels<VBR_BF16, true> : stream_kernels<VBR_BF16, false>);
    const StreamKernel kernel = kernels[v->stream_ops - kStreamLeastOps];
    hipLaunchKernelGGL(kernel, dim3((unsigned)L.grid), dim3(kStreamThreads), 0,
                       static_cast<hipStream_t>(hip_stream), p);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) { set_last_hip_error((int)e); return VBR_EHIP; }
    return VBR_OK;
}

}  // namespace vbrk
