// vbr_spmm on gfx950: C = A.B with A in packed VBR form (section 4.4.1 of the paper: every stored
// block is multiplied as a dense product on the matrix units).  The kernels share one scheme: a
// workgroup owns some slabs of 16 rows and a column tile of C, walks a list of K-steps of 32 B rows,
// brings the gathered B rows and the A fragments into rings of LDS slots with 128-bit direct-to-LDS
// loads, and issues v_mfma_f32_16x16x32 on them.
//   tile kernel    up to 8 slabs of ONE row group x 256 columns; K-steps = the group's column blocks
//   gathered tiles the same kernel with K-steps = the single columns its rows touch: up to 4 slabs of the
//                  rows of low groups, and of tall groups whose blocks are mostly fill-in
//   deep tiles     gathered tiles with very many columns: the waves of a workgroup split the K-steps
//   wide kernel    3 to 4 slabs of one row group x 512 columns, for long lists against a wide B: B goes to registers, A through LDS
//   stream kernel  up to 64 row groups of one slab x 64 columns, which share B rows (stream_spmm.hip)
//   panel kernel   8 slabs of low groups x 128 columns walking the union of their column blocks
//   mixed kernel   tiles of several of these classes in one launch
// Matrices whose rows share nothing are multiplied by the kernel in csr_spmm.hip.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>

#include "vbr_device.h"
#include "vbr_host.h"

namespace vbrk {

static thread_local int g_last_hip_error = 0;
void set_last_hip_error(int code) { g_last_hip_error = code; }

namespace {

constexpr int kThreads = 256;          // 4 waves
constexpr int kWaveN = 64;             // C columns per wave: 4 MFMA tiles of 16
constexpr int kRowBytes = kTileN * 2;  // one staged B row in LDS: 512 bytes, no padding
constexpr int kPanelBytes = kStepK * kRowBytes;   // 16 KiB of B per K-step
constexpr int kFragBytes = kFragElems * 2;        // 1 KiB per A fragment

typedef short short4v __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) short4v *lds_short4_ptr;
typedef __attribute__((address_space(3))) short8v *lds_short8_ptr;
typedef __attribute__((address_space(3))) float4v *lds_float4_ptr;
typedef __attribute__((address_space(3))) uint4v *lds_uint4_ptr;
typedef __attribute__((address_space(3))) int32_t *lds_i32_ptr;
typedef __attribute__((address_space(3))) unsigned char *lds_u8_ptr;
typedef __attribute__((address_space(4))) const int32_t *const_i32_ptr;

struct Params {
    const TileDesc *tiles;    // tiles of this launch
    const int32_t *krow;
    const int32_t *perm;
    const int32_t *gcol;      // column-gathered tiles: their column lists ...
    const int32_t *prow;      // ... and the list of the low rows their row positions refer to
    int32_t b_fits24;         // the rows of B the matrix can touch span less than 4 GiB, their number and length in bytes less than 2^24
    uint32_t b_bytes;         // wide kernel: bytes from B's first element to the end of its last row
    const uint16_t *vals;
    const uint16_t *B;
    float *C;
    int64_t ldb, ldc;
    int32_t N;
    int32_t lg_gran;
    int32_t n_tiles;          // T
    int32_t n_ntiles;         // Q = ceil(N / 256), of the split kernel ceil(N / 64)
    ColumnMap map;
    int32_t whole, rest;      // mixed kernel: tiles with one workgroup a column tile, and behind them some with four, see there ...
    int32_t split;            // ... and from how many K-steps on these are split
};

// 16 bytes per active lane from global memory straight into LDS, no register staging: lane l's
// data lands at lds_base + 16 l (lds_base wave-uniform, passed in M0).  The load is counted in
// vmcnt like any vector load; the compiler does not see it, so the waits are placed by hand.
// Every wave must issue the same, fixed number of these per K-step (never with an empty lane mask).
__device__ __forceinline__ void dma16(const void *gptr, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, off" ::"v"(gptr),
                 "s"((uint32_t)__builtin_amdgcn_readfirstlane(lds_base)) : "memory");
}
// same, address = wave-uniform base + zero-extended 32-bit lane offset
__device__ __forceinline__ void dma16_base(uint32_t voff, const void *base, uint32_t lds_base)
{
    // the base has to sit in scalar registers: say so explicitly (a no-op when it already does)
    const uint64_t b = reinterpret_cast<uint64_t>(base);
    const uint64_t sbase = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(b >> 32)) << 32) |
                           (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)b);
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %0, %1" ::"v"(voff), "s"(sbase),
                 "s"((uint32_t)__builtin_amdgcn_readfirstlane(lds_base)) : "memory");
}

// 4 bytes per active lane into LDS: lane l's at lds_base + 4 l
__device__ __forceinline__ void dma4(const void *gptr, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %0, off" ::"v"(gptr),
                 "s"((uint32_t)__builtin_amdgcn_readfirstlane(lds_base)) : "memory");
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}

// S  = slabs the instantiation computes (tiles of the class have S/2 < n_slabs <= S; 1 for S = 1).
// NS = slots of the LDS ring of B panels: NS-1 K-steps of B loads are in flight per workgroup.
// DA = prefetch distance of the A fragments in K-steps (ring of DA+1 slots): A is streamed from
//      beyond L2 while B mostly hits in L2, and the loads of a wave retire in order.
// The loop is bound by the instructions a wave needs per K-step, so the common case (block width a
// multiple of 8, full column tile, no padding rows in the K-step) is kept to a handful of scalar
// instructions per 1 KiB load; everything else takes the general path.
// B rows of the next K-steps, in LDS: one load of a wave brings those of 8 K-steps of a gathered tile (8 columns each) or of
// 64 of a block tile (one granule each); two such lists for each of the 4 waves.
constexpr int kListBytes = 2 * 4 * 64 * 4;
// With 5 to 8 slabs there is no room for them beside two workgroups on a CU.
template <int S, bool GATHER>
constexpr bool has_lists() { return GATHER || S < 8; }
template <int S, int NS, int DA, bool GATHER>
constexpr int tile_lds_bytes() { return NS * kPanelBytes + (DA + 1) * S * kFragBytes + (has_lists<S, GATHER>() ? kListBytes : 0); }

// GATHER: the tile is up to four slabs of the row list (prow: rows of low groups, and of taller ones whose blocks are mostly
// fill-in), and its K dimension the list of the single COLUMNS its rows touch (gcol, one entry per B row) instead of
// whole column blocks: the fill-in columns of the blocks, which hold nothing but zeros, are never loaded.
// NARROW: narrow column tiles have a way of their own to C (at the end).
template <int DT, int S, int NS, int DA, bool GATHER = false, bool NARROW = (S > 4)>
__device__ __forceinline__ void tile_body(const Params &p, const TileDesc td, const int ntile, unsigned char *smem)
{
    static_assert(NS >= 2 && DA >= NS, "A must be requested before the B panel of its K-step");
    constexpr bool kLists = has_lists<S, GATHER>();
    constexpr int NA = S >= 4 ? S / 4 : 1;      // A loads per wave per K-step
    constexpr int NAS = DA + 1;
    constexpr int kAStage = S * kFragBytes;
    constexpr int kBRing = NS * kPanelBytes;
    // loads younger than the last B load of K-step ks when the workgroup waits for it
    constexpr int kWait = (NS - 2) * 4 + (NS - 1) * NA;
    static_assert(kWait < 64, "vmcnt is a 6-bit counter");

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n0 = ntile * kTileN;
    const lds_u8_ptr sm = (lds_u8_ptr)smem;
    const uint32_t smem_base = (uint32_t)(uintptr_t)sm;      // LDS byte address, for M0
    const int n_ks = td.n_ks;
    const int q = lane >> 4, s16 = lane & 15;

    // C rows of the tile, lane l of register i that of row 64 i + l: requested first and used last.  A narrow column tile (see its stores) asks for
    // them when it stores: handed round from here they took longer (row groups of 1 to 100 rows, in a graph of calls, N = 72 5.7 and 5.4 us, N = 8
    // 9.3 and 9.0, N = 40 7.5 and 7.2), and the kernels that have both are faster at other N, too (N = 264 7.2 and 6.9, N = 672 8.5 and 8.1).
    const bool narrow = NARROW && p.N - n0 <= kTileN / 2;
    int32_t c_rows[(S + 3) / 4];
#pragma unroll
    for (int i = 0; i < (S + 3) / 4; ++i) {
        const int rr = 64 * i + lane;
        c_rows[i] = !narrow && rr < td.n_rows ? (GATHER ? p.prow : p.perm)[td.row_begin + rr] : -1;
    }

    float4v acc[S][4];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int f = 0; f < 4; ++f) acc[s][f] = float4v{0.f, 0.f, 0.f, 0.f};

    if (n_ks > 0) {
        // ---- B staging.  Per K-step a wave issues 4 loads; load i brings rows 8 wave + 2 i (lanes
        // 0-31) and 8 wave + 2 i + 1 (lanes 32-63) of the K-step, 512 bytes each, into 1 KiB of LDS.
        // LDS chunk c' (16 bytes) of row r holds global chunk c' ^ 2 (r % 8): the XOR spreads the
        // four rows one transposed read touches over distinct banks (rows are 512 bytes apart).
        const int half = lane >> 5;
        const int lg = p.lg_gran;
        const int gmask = (1 << lg) - 1;
        const uint32_t ldb_bytes = (uint32_t)(p.ldb * 2);          // host checked: 32 rows of B span less than 2^32 bytes
        const char *Btile = reinterpret_cast<const char *>(p.B) + (int64_t)n0 * 2;
        // In the last column tile the chunks at or beyond column N do not exist: their lanes fetch
        // the tile's last existing chunk again (the C columns it would feed are never stored, and
        // columns do not mix).
        const int last_chunk = (p.N - n0 < kTileN ? p.N - n0 : kTileN) / 8 - 1;
        uint32_t b_lane[4];      // offset of this lane's 16 bytes from the first row of the wave's granule; gathered tiles: from the row
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int chunk = (lane & 31) ^ (2 * (2 * i + half));
            b_lane[i] = (uint32_t)(chunk <= last_chunk ? chunk : last_chunk) * 16;
            if constexpr (!GATHER) b_lane[i] += (uint32_t)((8 * wave + 2 * i + half) & gmask) * ldb_bytes;
        }

        // ---- A staging.  A direct-to-LDS load costs the CU the same whatever its lane mask, so a
        // fragment is always one load: with 1 or 2 slabs the waves take turns (K-step a: wave a % 4,
        // resp. waves 2 (a % 2) + slab), with 4 or 8 slabs every wave loads S/4 fragments per K-step.
        // Lanes of rows a partial last slab does not store are masked off (their LDS bytes keep
        // whatever they held: those fragment rows only feed C rows that are never stored); a wave
        // whose slab does not exist in this tile reloads the tile's last slab instead, so that the
        // loads per wave follow a fixed pattern and no load has an empty lane mask.
        const int rows_last = td.n_rows - (td.n_slabs - 1) * kSlabRows;
        const uint32_t a_stride_bytes = (uint32_t)(((td.n_slabs - 1) * kFragElems + rows_last * kStepK) * 2);
        const char *Abase = reinterpret_cast<const char *>(p.vals) + td.a_off * 16;
        int a_slab[NA];
        uint32_t a_lane[NA];     // byte offset of this lane's 16 bytes inside a K-step of the tile
        bool a_on[NA];
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            if constexpr (S == 1) a_slab[i] = 0;
            else if constexpr (S == 2) a_slab[i] = wave & 1;
            else a_slab[i] = wave + 4 * i;
            if (a_slab[i] > td.n_slabs - 1) a_slab[i] = td.n_slabs - 1;
            const int rows = (a_slab[i] == td.n_slabs - 1) ? rows_last : kSlabRows;
            a_on[i] = s16 < rows;
            a_lane[i] = (uint32_t)((a_slab[i] * kFragElems + (q * rows + s16) * 8) * 2);
        }
        // does this wave load (part of) the A fragments of K-step a?
        auto a_turn = [&](int a) -> bool {
            if constexpr (S == 1) return (a & 3) == wave;
            else if constexpr (S == 2) return (a & 1) == (wave >> 1);
            else return true;
        };

        // The B rows of a K-step: of a block tile the first row of the granule that holds this wave's 8 rows, of a gathered one
        // its 8 columns.  The wave fetches them into LDS for many K-steps with one load and reads them a K-step before their
        // loads are issued.  (As scalar loads, one per K-step, they were waited for in every K-step; those of gathered tiles
        // missed the scalar cache every time: noisy planted matrix 36 -> 29 us.)
        constexpr int kSteps = GATHER ? 8 : 64;
        int32_t ent[4] = {0, 0, 0, 0};
        const lds_u8_ptr lists = sm + kBRing + NAS * kAStage + wave * (kListBytes / 4);
        auto issue_list = [&](int batch) {
            int k = batch * kSteps + (GATHER ? lane >> 3 : lane);
            if (k > n_ks - 1) k = n_ks - 1;
            const int32_t *src = GATHER ? p.gcol + ((int64_t)td.ks_begin + k) * kStepK + 8 * wave + (lane & 7)
                                        : p.krow + ((((int64_t)td.ks_begin + k) * kStepK + 8 * wave) >> lg);
            dma4(src, smem_base + kBRing + NAS * kAStage + wave * (kListBytes / 4) + (batch & 1) * (kListBytes / 8));
        };
        auto read_list = [&](int ks) {
            if constexpr (GATHER) {
                const lds_u8_ptr at = lists + (ks & (2 * kSteps - 1)) * 32 + half * 4;
#pragma unroll
                for (int i = 0; i < 4; ++i) ent[i] = *(lds_i32_ptr)(at + i * 8);
            } else {
                ent[0] = *(lds_i32_ptr)(lists + (ks & (2 * kSteps - 1)) * 4);
            }
        };
        // Without lists: scalar loads, two K-steps ahead of their use.
        int32_t rb0 = 0, rb1 = 0;
        auto load_row = [&](int ks) -> int32_t {
            // past the end: reload the last K-step (never computed); wave-uniform, and said so, or the
            // lookups below become vector loads, which cost the load path as much as a load of B
            const int kc = __builtin_amdgcn_readfirstlane(ks < n_ks ? ks : n_ks - 1);
            return ((const_i32_ptr)p.krow)[(((int64_t)td.ks_begin + kc) * kStepK + 8 * wave) >> lg];
        };
        auto issue_b = [&](int slot) {
            const uint32_t sb = smem_base + slot * kPanelBytes + 8 * wave * kRowBytes;
            if constexpr (GATHER) {
                // (behind the last column of the tile the list repeats it: the fragments hold zeros there)
                if (p.b_fits24) {        // scalar base + 32-bit lane offsets, the cheaper form of the load
#pragma unroll
                    for (int i = 0; i < 4; ++i) dma16_base(__umul24((uint32_t)ent[i], ldb_bytes) + b_lane[i], Btile, sb + 2 * i * kRowBytes);
                } else {
#pragma unroll
                    for (int i = 0; i < 4; ++i) dma16(Btile + (uint64_t)(uint32_t)ent[i] * ldb_bytes + b_lane[i], sb + 2 * i * kRowBytes);
                }
            } else {
                const int32_t row = kLists ? __builtin_amdgcn_readfirstlane(ent[0]) : rb0;
                const char *rowptr = Btile + (uint64_t)(uint32_t)row * ldb_bytes;          // scalar, 64-bit
#pragma unroll
                for (int i = 0; i < 4; ++i) dma16_base(b_lane[i], rowptr, sb + 2 * i * kRowBytes);
            }
        };
        auto issue_a = [&](int ks, int slot) {
            if (!a_turn(ks)) return;
            const int kc = ks < n_ks ? ks : n_ks - 1;
            const char *kptr = Abase + (int64_t)kc * a_stride_bytes;             // scalar
            const uint32_t sa = smem_base + kBRing + slot * kAStage;
#pragma unroll
            for (int i = 0; i < NA; ++i)
                if (a_on[i]) dma16_base(a_lane[i], kptr, sa + a_slab[i] * kFragBytes);
        };
        // wait until this wave's loads of K-step ks have landed: everything but the loads it issued
        // after the B panel of ks, i.e. in the iterations ks-NS+1 (its A part) .. ks-1
        auto wait_stage = [&](int ks) {
            if constexpr (S >= 4) {
                wait_vmcnt<kWait>();
            } else {
                int later_a = 0;
#pragma unroll
                for (int d = 1; d <= NS - 1; ++d) later_a += a_turn(ks - d + DA) ? 1 : 0;
                if (later_a == 0) wait_vmcnt<(NS - 2) * 4>();
                else if (later_a == 1) wait_vmcnt<(NS - 2) * 4 + 1>();
                else if (later_a == 2) wait_vmcnt<(NS - 2) * 4 + 2>();
                else if (later_a == 3) wait_vmcnt<(NS - 2) * 4 + 3>();
                else wait_vmcnt<(NS - 2) * 4 + 4>();
                static_assert(NS <= 5, "at most four later A loads are told apart");
            }
        };

        // B fragment of MFMA tile f, half r: lane (q, s16) reads 8 bytes of B row
        // R = 16 (q/2) + 8 r + 4 (q%2) + s16/4 at columns 64 wave + 16 f + 4 (s16%4) ..+3; the
        // transposed read hands every lane the 4 rows of ITS column (column s16 of the tile).
        uint32_t b_off[4];
        {
            const int R0 = 16 * (q >> 1) + 4 * (q & 1) + (s16 >> 2);       // r adds 8 rows: R % 8 unchanged
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                const int chunk = 8 * wave + 2 * f + ((s16 & 3) >> 1);
                b_off[f] = R0 * kRowBytes + ((chunk ^ (2 * (R0 & 7))) << 4) + (s16 & 1) * 8;
            }
        }
        // the LDS reads of a K-step are issued before the next loads (the inline asm keeps that
        // order), so that their latency overlaps with the address work of the loads
        short8v bfrag[4], afrag[S];
        auto read_frags = [&](int bslot, int aslot) {
            const lds_u8_ptr sb = sm + bslot * kPanelBytes;
            const lds_u8_ptr sa = sm + kBRing + aslot * kAStage;
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(sb + b_off[f]));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(sb + b_off[f] + 8 * kRowBytes));
                bfrag[f] = short8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            }
#pragma unroll
            for (int s = 0; s < S; ++s) afrag[s] = *(lds_short8_ptr)(sa + s * kFragBytes + lane * 16);
        };
        auto multiply = [&]() {
            // operands swapped: the result tile comes out transposed, so a lane holds 4 consecutive
            // columns of one C row and stores them as one 16-byte word
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int f = 0; f < 4; ++f) acc[s][f] = mfma16x16x32<DT>(bfrag[f], afrag[s], acc[s][f]);
        };

        // ---- software pipeline over the K-steps.  Issue order, as if the loop had started NS-1
        // iterations early: A(0 .. DA-NS), then B(t), A(DA-NS+1+t) for t = 0 .. NS-2; iteration ks
        // then issues B(ks+NS-1), A(ks+DA).  The prologue re-loads the last K-step for K-steps past the
        // end of a very short tile, so that the loop always starts with the same loads in flight.
        if constexpr (kLists) {
            issue_list(0);
            if (n_ks > kSteps) issue_list(1);
        } else {
            rb0 = load_row(0);
            rb1 = load_row(1);
        }
#pragma unroll
        for (int k = 0; k <= DA - NS; ++k) issue_a(k, k);
        if constexpr (kLists) {
            wait_vmcnt<0>();
            read_list(0);
        }
#pragma unroll
        for (int t = 0; t < NS - 1; ++t) {
            issue_b(t);
            if constexpr (kLists) {
                read_list(t + 1);
            } else {
                rb0 = rb1;
                rb1 = load_row(t + 2);
            }
            issue_a(DA - NS + 1 + t, DA - NS + 1 + t);
        }
        int bslot = 0, aslot = 0;
        for (int ks = 0; ks < n_ks; ++ks) {
            // The last iterations issue nothing for K-steps past the end (a short tile would spend a
            // tenth of its loads there); from the first iteration whose predecessors left loads out,
            // the counted wait no longer holds and the wave waits for everything it has in flight.
            if (ks + DA > n_ks) wait_vmcnt<0>();
            else wait_stage(ks);                   // this wave's loads of K-step ks have landed
            __builtin_amdgcn_s_barrier();          // ... and everybody else's; the slots of K-step ks-1 are free
            if constexpr (!kLists) asm volatile("" ::"s"(rb0));      // the scalar row lookup is waited for here, not behind the LDS reads
            read_frags(bslot, aslot);
            // the load path is what bounds the kernel: a wave that is about to issue its loads goes
            // ahead of the waves that are multiplying (measured: 3-4 % on the 16-row workload)
            __builtin_amdgcn_s_setprio(3);
            if (ks + NS - 1 < n_ks) issue_b(bslot == 0 ? NS - 1 : bslot - 1);
            if (ks + DA < n_ks) issue_a(ks + DA, aslot == 0 ? NAS - 1 : aslot - 1);
            if constexpr (kLists) {
                // the next list but one, into the place of the one whose last K-step has been read (an extra load in
                // flight only makes the counted waits stricter)
                const int next = ks + NS;
                if ((next & (kSteps - 1)) == 1 && (next / kSteps + 1) * kSteps < n_ks && next > kSteps) issue_list(next / kSteps + 1);
                read_list(next);
            }
            __builtin_amdgcn_s_setprio(0);
            multiply();
            if constexpr (!kLists) {
                rb0 = rb1;
                rb1 = load_row(ks + NS + 1);
            }
            bslot = bslot == NS - 1 ? 0 : bslot + 1;
            aslot = aslot == NAS - 1 ? 0 : aslot + 1;
        }
        wait_vmcnt<0>();                           // no load may still be writing LDS when the workgroup ends
    }

    // C rows go back to their original positions through perm; beta = 0.  A lane holds 4 columns of ONE row, so a
    // store straight from the accumulators touches 16 rows, 64 bytes each: half lines, which leave L2 as partial
    // writes (graph of 16384 nodes, N = 4096: 330 MB written for 268).  The wave turns every slab round in LDS (its own
    // 16 rows x 272 bytes: no bank conflicts) and stores 4 rows x 256 bytes at a time, around the caches' write
    // allocation.  That graph: 260 -> 222 us; 8192 x 8192 with 700 000 stored entries, N = 2048: 23.1 -> 18.7 us;
    // 16384 x 16384 with row groups of 16 to 128 rows, N = 512: 26.4 -> 23.5 us.
    // In a column tile of up to 128 columns there is little to write, and the way through LDS, slab after slab, is what counts
    // with 5 to 8 slabs: stored straight (24 tiles, 4 K-steps, N = 8: 7.5 and 5.9 us, N = 72: 7.7 and 6.0, N = 128: 7.7 and 6.6; 200
    // tiles, 8 K-steps, N = 64: 9.9 and 8.2, N = 128: 10.0 and 9.5, N = 160: 10.2 and 10.4; up to 4 slabs both take the same;
    // in the mixed kernel with tiles of up to 8 those of 4 have it too, without which its code runs 1 % slower at any N).
    if (n_ks > 0) __syncthreads();                  // the rings are read no more
    if constexpr (NARROW) {
        if (__builtin_expect(narrow, 0)) {
            int32_t row[S];
#pragma unroll
            for (int s = 0; s < S; ++s) {
                const int rr = s * kSlabRows + s16;
                row[s] = rr < td.n_rows ? (GATHER ? p.prow : p.perm)[td.row_begin + rr] : -1;
            }
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int f = 0; f < 4; ++f) {
                    const int n = n0 + wave * kWaveN + 16 * f + 4 * q;
                    if (row[s] >= 0 && n < p.N) __builtin_nontemporal_store(acc[s][f], reinterpret_cast<float4v *>(p.C + row[s] * p.ldc + n));
                }
            return;
        }
    }
    constexpr int kOutRow = kWaveN * 4 + 16;
    static_assert(4 * kSlabRows * kOutRow <= tile_lds_bytes<S, NS, DA, GATHER>(), "the turned slabs of the four waves fit the rings");
    const lds_u8_ptr out = sm + wave * kSlabRows * kOutRow;
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int f = 0; f < 4; ++f) *(lds_float4_ptr)(out + s16 * kOutRow + f * 64 + q * 16) = acc[s][f];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float4v x = *(lds_float4_ptr)(out + (4 * i + q) * kOutRow + s16 * 16);
            const int32_t row = __shfl(c_rows[s / 4], (s & 3) * kSlabRows + 4 * i + q);
            const int n = n0 + wave * kWaveN + 4 * s16;
            // a position of the low-row list may be padding (-1)
            if (row >= 0 && n < p.N) __builtin_nontemporal_store(x, reinterpret_cast<float4v *>(p.C + row * p.ldc + n));
        }
    }
}

constexpr int kDeepRow = kDeepN * 2;              // one staged B row: 128 bytes
constexpr int kDeepList = kStepK * 4;             // the list entries of a K-step
template <int S, int SLOTS>
constexpr int deep_wave_bytes() { return SLOTS * (kStepK * kDeepRow + S * kFragBytes + kDeepList); }

// A deep tile: a gathered tile of one or two slabs whose column list is so long that a workgroup of the tile kernel, which
// takes the K-steps one after the other, would still be at it when the rest of the launch is done (a hub of a graph:
// thousands of columns, 0.3 us per K-step).  Here a workgroup owns 64 columns of C and its four waves take the
// K-steps in turn, each with an LDS ring of its own and without a barrier; the four partial sums are added in LDS, in
// a fixed order.  The price is S fragments per 64 columns instead of per 256: 24 loads per K-step for two slabs
// instead of 18.
template <int DT, int S, int SLOTS, bool GATHER = true>
__device__ __forceinline__ void deep_body(const Params &p, const TileDesc td, const int n0, unsigned char *smem)
{
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (n0 >= p.N) return;
    const lds_u8_ptr sm = (lds_u8_ptr)smem;
    const int q = lane >> 4, s16 = lane & 15;
    constexpr int kB = kStepK * kDeepRow, kA = S * kFragBytes;
    const lds_u8_ptr mine = sm + wave * deep_wave_bytes<S, SLOTS>();
    const uint32_t base = (uint32_t)(uintptr_t)mine;             // [B slots][A slots][list slots]
    const lds_u8_ptr lists = mine + SLOTS * (kB + kA);
    const int n_ks = td.n_ks;
    // C row of row `lane` of the tile: requested first and used last
    const int32_t c_row = lane < td.n_rows ? (GATHER ? p.prow : p.perm)[td.row_begin + lane] : -1;

    float4v acc[S][4];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int f = 0; f < 4; ++f) acc[s][f] = float4v{0.f, 0.f, 0.f, 0.f};

    // B: load i brings rows 8 i + lane / 8 of the K-step, 128 bytes each.  LDS chunk c' of row r holds global chunk
    // c' ^ 2 ((r / 2) % 4): the eight rows half a wave reads with one transposed read fall into distinct banks.
    const int last_chunk = (p.N - n0 < kDeepN ? p.N - n0 : kDeepN) / 8 - 1;
    const int chunk = (lane & 7) ^ (2 * (lane >> 4 & 3));
    const char *Bcol = reinterpret_cast<const char *>(p.B) + (int64_t)n0 * 2 + (chunk <= last_chunk ? chunk : last_chunk) * 16;
    const uint64_t ldb_bytes = (uint64_t)p.ldb * 2;
    const int rows_last = td.n_rows - (td.n_slabs - 1) * kSlabRows;
    const uint32_t a_stride_bytes = (uint32_t)(((td.n_slabs - 1) * kFragElems + rows_last * kStepK) * 2);
    const char *Abase = reinterpret_cast<const char *>(p.vals) + td.a_off * 16;
    // the B rows of a K-step: one by one, or the first row of the granule of every eight
    const int lg = p.lg_gran, gmask = (1 << lg) - 1;
    auto issue_list = [&](int ks, int slot) {
        const int64_t k = (int64_t)td.ks_begin + ks;
        const uint32_t to = base + SLOTS * (kB + kA) + slot * kDeepList;
        if constexpr (GATHER) {
            if (lane < kStepK) dma4(p.gcol + k * kStepK + lane, to);
        } else {
            if (lane < kStepK / 8) dma4(p.krow + ((k * kStepK + 8 * lane) >> lg), to);
        }
    };
    auto issue = [&](int ks, int slot) {
        int32_t e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            if constexpr (GATHER) e[i] = *(lds_i32_ptr)(lists + slot * kDeepList + (8 * i + (lane >> 3)) * 4);
            else e[i] = *(lds_i32_ptr)(lists + slot * kDeepList + i * 4) + ((8 * i + (lane >> 3)) & gmask);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
            dma16(Bcol + (uint64_t)(uint32_t)e[i] * ldb_bytes, base + slot * kB + i * 1024);
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const int sl = s < td.n_slabs ? s : td.n_slabs - 1;               // no second slab: the first again, never stored
            const int rows = sl == td.n_slabs - 1 ? rows_last : kSlabRows;
            if (s16 < rows) dma16_base((uint32_t)((sl * kFragElems + (q * rows + s16) * 8) * 2), Abase + (int64_t)ks * a_stride_bytes,
                                       base + SLOTS * kB + slot * kA + s * kFragBytes);
        }
    };
    uint32_t b_off[4];
    {
        const int R0 = 16 * (q >> 1) + 4 * (q & 1) + (s16 >> 2);               // the other four rows: R0 + 8, the same swizzle
#pragma unroll
        for (int f = 0; f < 4; ++f) {
            const int c = 2 * f + ((s16 & 3) >> 1);
            b_off[f] = R0 * kDeepRow + ((c ^ (2 * (R0 >> 1 & 3))) << 4) + (s16 & 1) * 8;
        }
    }
    // The wave's own K-steps, 0 .. steps-1, are wave, wave + 4, ...  Iteration j issues the rows and fragments of step
    // j + P and the list of step j + 2 P (clamped to the last): P steps are in flight while one is multiplied, and a
    // list is there when its rows are requested.
    constexpr int P = SLOTS - 1, kPerStep = 4 + S + 1;
    static_assert((P - 1) * kPerStep < 64, "vmcnt is a 6-bit counter");
    const int steps = wave < n_ks ? (n_ks - wave + 3) / 4 : 0;
    auto list_at = [&](int j) { issue_list(wave + 4 * (j < steps ? j : steps - 1), j % SLOTS); };
    if (steps > 0) {
#pragma unroll
        for (int t = 0; t < P; ++t) list_at(t);
        wait_vmcnt<0>();
#pragma unroll
        for (int t = 0; t < P; ++t) {
            issue(wave + 4 * (t < steps ? t : steps - 1), t);
            list_at(t + P);
        }
        int slot = 0;
        for (int j = 0; j < steps; ++j) {
            if (j + P <= steps) wait_vmcnt<(P - 1) * kPerStep>();     // everything up to the rows and fragments of step j
            else wait_vmcnt<0>();
            short8v bfrag[4], afrag[S];
            const lds_u8_ptr sb = mine + slot * kB, sa = mine + SLOTS * kB + slot * kA;
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(sb + b_off[f]));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(sb + b_off[f] + 8 * kDeepRow));
                bfrag[f] = short8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            }
#pragma unroll
            for (int s = 0; s < S; ++s) afrag[s] = *(lds_short8_ptr)(sa + s * kFragBytes + lane * 16);
            if (j + P < steps) {
                issue(wave + 4 * (j + P), slot == 0 ? P : slot - 1);
                list_at(j + 2 * P);
            }
#pragma unroll
            for (int s = 0; s < S; ++s)
#pragma unroll
                for (int f = 0; f < 4; ++f) acc[s][f] = mfma16x16x32<DT>(bfrag[f], afrag[s], acc[s][f]);
            slot = slot == P ? 0 : slot + 1;
        }
        wait_vmcnt<0>();
    }

    constexpr int kOutRow = kDeepN * 4 + 16, kOutSlab = kSlabRows * kOutRow;
    __syncthreads();                                                           // nobody reads the rings any more
    const lds_u8_ptr out = sm + wave * S * kOutSlab;
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int f = 0; f < 4; ++f) *(lds_float4_ptr)(out + s * kOutSlab + s16 * kOutRow + f * 64 + q * 16) = acc[s][f];
    __syncthreads();
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const lds_u8_ptr at = sm + s * kOutSlab + (4 * wave + q) * kOutRow + s16 * 16;
        float4v x = *(lds_float4_ptr)at;
#pragma unroll
        for (int w = 1; w < 4; ++w) x += *(lds_float4_ptr)(at + w * S * kOutSlab);
        const int n = n0 + 4 * s16;
        const int32_t row = __shfl(c_row, s * kSlabRows + 4 * wave + q);
        if (row >= 0 && n < p.N) __builtin_nontemporal_store(x, reinterpret_cast<float4v *>(p.C + row * p.ldc + n));
    }
}

template <int S, int SLOTS>
constexpr int deep_lds_bytes()
{
    const int ring = 4 * deep_wave_bytes<S, SLOTS>(), out = 4 * S * kSlabRows * (kDeepN * 4 + 16);
    return ring > out ? ring : out;
}

constexpr int kStages = 2;      // LDS ring of B panels
constexpr int kStagesTall = 3;  // the same for block tiles of 5 to 8 slabs (80 KiB of LDS, two workgroups per CU): measured 3 % (K = 16 384)
                                // to 14 % (K = 8 192) faster than 2 on dense matrices; and of 3 to 4 slabs (64 KiB, two per CU): blocks of
                                // 64 x 64 at 40 %, N = 2048: 144 -> 126 us, at 5 %: 17.4 -> 16.0, N = 8192 the same; slower
                                // than 2 for the lower classes, and for gathered tiles, which want the third workgroup
constexpr int kStagesFew = 4;   // for tiles of 1 and 2 slabs in a launch whose workgroups are all resident with two on a CU
constexpr int kADistance = 3;   // K-steps the A fragments are requested ahead (more than the ring of B panels has slots)
constexpr int a_distance(int stages) { return stages > kADistance ? stages : kADistance; }
// Tiles of two slabs request their fragments one K-step later, which makes the ring 2 KiB smaller and, with the lists, lets four
// workgroups be resident on a CU instead of three: 256 groups of 32 rows, 26 K-steps, N = 1024 (1024 workgroups): 36.3 -> 26.6 us,
// 60 K-steps, N = 4096: 218 -> 201; launches that were resident before take the same (768 workgroups: 21.4 and 21.1).
constexpr int kADistanceTwo = 2;
constexpr int kLdsBytes = 160 * 1024;
static_assert(4 * tile_lds_bytes<1, kStages, kADistance, true>() <= kLdsBytes && 4 * tile_lds_bytes<1, kStages, kADistance, false>() <= kLdsBytes &&
                  4 * tile_lds_bytes<2, kStages, kADistanceTwo, true>() <= kLdsBytes && 4 * tile_lds_bytes<2, kStages, kADistanceTwo, false>() <= kLdsBytes,
              "four workgroups of one- and two-slab tiles on a CU");
static_assert(3 * tile_lds_bytes<4, kStages, kADistance, true>() <= kLdsBytes, "three of gathered tiles of 3 to 4 slabs");
static_assert(2 * tile_lds_bytes<4, kStagesTall, kADistance, false>() <= kLdsBytes && 2 * tile_lds_bytes<8, kStagesTall, kADistance, false>() <= kLdsBytes,
              "two of taller block tiles");

// A tile without a K-step, up to 64 rows of A without entries, in a launch of block tiles or of lower tiles: zeros, a wave 1 KiB of every fourth row.
// (Lane l asks for the place of row l; asked for one after the other they made the kernel take 4.4 us instead of 2.9: 60 tiles of 16 rows, N = 256.)
__device__ __forceinline__ void zero_tile(const Params &p, const TileDesc td, const int ntile)
{
    static_assert(kTileN == 4 * 64, "a lane writes four columns");
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, n = ntile * kTileN + 4 * lane;
    const int32_t rows = lane < td.n_rows ? p.prow[td.row_begin + lane] : -1;
#pragma unroll
    for (int r = 0; r < kMaxGatherSlabs * kSlabRows; r += 4) {
        const int64_t row = __shfl(rows, r + wave);          // a position of the row list may be padding (-1)
        if (row >= 0 && n < p.N) __builtin_nontemporal_store(float4v{0.f, 0.f, 0.f, 0.f}, reinterpret_cast<float4v *>(p.C + row * p.ldc + n));
    }
}

// Measured on the 16-row workload: two ring slots and four resident workgroups per CU (38 KiB of
// LDS each) beat deeper rings with fewer workgroups; the gather is bound by how many independent
// instruction streams feed the texture-address unit, not by the depth of any one of them.
template <int DT, int S, int NS, int DA, bool GATHER = false>
__global__ void __launch_bounds__(kThreads) vbr_spmm_kernel(const Params p)
{
    __shared__ __attribute__((aligned(1024))) unsigned char smem[tile_lds_bytes<S, NS, DA, GATHER>()];
    int tile, ntile;
    if (!map_workgroup(blockIdx.x, p.n_tiles, p.n_ntiles, p.map, tile, ntile)) return;
    const TileDesc td = p.tiles[tile];
    if constexpr (S <= 2)                                    // see plan_launches
        if (td.n_ks == 0) return zero_tile(p, td, ntile);
    tile_body<DT, S, NS, DA, GATHER>(p, td, ntile, smem);
}

// Tiles of several classes in one launch: the workgroup picks the code of its tile's class.  Registers and LDS are those of
// the largest.  MAXS: the tallest block tile.  RING as above, SLOTS for deep tiles.
template <int DT, int MAXS, int RING, int SLOTS>
__global__ void __launch_bounds__(kThreads) vbr_spmm_mixed_kernel(const Params p)
{
    constexpr int NS1 = RING, DA1 = a_distance(NS1);
    constexpr int NSG = RING > kStages ? kStagesTall : kStages;                    // gathered, 3 to 4 slabs
    constexpr int NS4 = MAXS == 8 ? kStagesTall : NSG, NS8 = RING > kStages ? kStagesTall : kStages;
    constexpr int kLow = std::max(tile_lds_bytes<2, NS1, DA1, true>(), std::max(deep_lds_bytes<2, SLOTS>(), RING > kStages ? deep_lds_bytes<4, 2>() : 0));
    constexpr int k4 = std::max(tile_lds_bytes<4, NSG, kADistance, true>(), tile_lds_bytes<4, NS4, kADistance, false>());
    constexpr int k8 = MAXS == 8 ? tile_lds_bytes<8, NS8, kADistance, false>() : 0;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[std::max(k8, std::max(k4, kLow))];
    int tile, ntile;
    if (!map_workgroup(blockIdx.x, p.n_tiles, p.n_ntiles, p.map, tile, ntile)) return;
    // quarters of a column tile for the tiles that are split; of those that have four workgroups and are not, the first takes all of it
    int quarter;
    const bool four = split_tile(tile, p.whole, p.rest, quarter);
    const TileDesc td = p.tiles[tile];
    if (td.group <= kTileDeep) {
        if (quarter != 0) return;
        const int n0 = ntile * kTileN + (kTileDeep - td.group) * kDeepN;
        if (td.n_slabs <= 1) deep_body<DT, 1, SLOTS>(p, td, n0, smem);
        else deep_body<DT, 2, SLOTS>(p, td, n0, smem);
    } else if (four && td.n_slabs <= split_slabs(RING > kStages) && td.n_ks >= p.split) {
        const int n0 = ntile * kTileN + quarter * kDeepN;
        const bool gathered = td.group == kTileGathered;
        if (gathered && td.n_slabs <= 1) deep_body<DT, 1, SLOTS>(p, td, n0, smem);
        else if (gathered && td.n_slabs <= 2) deep_body<DT, 2, SLOTS>(p, td, n0, smem);
        else if (td.n_slabs <= 1) deep_body<DT, 1, SLOTS, false>(p, td, n0, smem);
        else if (td.n_slabs <= 2) deep_body<DT, 2, SLOTS, false>(p, td, n0, smem);
        else if constexpr (RING > kStages) {
            if (gathered) deep_body<DT, 4, 2>(p, td, n0, smem);
            else deep_body<DT, 4, 2, false>(p, td, n0, smem);
        }
    } else if (quarter != 0) {
        return;
    } else if (td.group == kTileGathered) {
        if (td.n_slabs <= 1) tile_body<DT, 1, NS1, DA1, true>(p, td, ntile, smem);
        else if (td.n_slabs <= 2) tile_body<DT, 2, NS1, DA1, true>(p, td, ntile, smem);
        else tile_body<DT, 4, NSG, kADistance, true, MAXS == 8>(p, td, ntile, smem);
    } else if (td.n_slabs <= 1) tile_body<DT, 1, NS1, DA1>(p, td, ntile, smem);
    else if (td.n_slabs <= 2) tile_body<DT, 2, NS1, DA1>(p, td, ntile, smem);
    else if (MAXS == 4 || td.n_slabs <= 4) tile_body<DT, 4, NS4, kADistance, false, MAXS == 8>(p, td, ntile, smem);
    else if constexpr (MAXS == 8) tile_body<DT, 8, NS8, kADistance>(p, td, ntile, smem);
}

// The deep form for every tile of up to four slabs, for launches whose workgroups would not fill the chip: four times as many,
// each with a quarter of the chain.  64 columns of C per workgroup.
template <int DT, int S, bool GATHER>
__global__ void __launch_bounds__(kThreads) vbr_spmm_split_kernel(const Params p)
{
    constexpr int SLOTS = S <= 2 ? 3 : 2;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[deep_lds_bytes<S, SLOTS>()];
    int tile, ntile;
    if (!map_workgroup(blockIdx.x, p.n_tiles, p.n_ntiles, p.map, tile, ntile)) return;
    deep_body<DT, S, SLOTS, GATHER>(p, p.tiles[tile], ntile * kDeepN, smem);
}

constexpr int kWideWaveN = kWideN / 4;           // C columns per wave of the wide kernel

// Block tiles of 3 to 4 slabs against a wide B.  A workgroup owns 512 columns of C, each of its four waves 128 of them and all rows.
// In the tile kernel a wave's B columns are nobody else's and pass through LDS all the same, for the sake of the transposed read: 16 KiB
// written and 32 KiB read per K-step, which keeps the LDS busier than the matrix unit.  Here a lane loads eight columns of eight rows of B, 8 x 8 values that
// it turns round by itself: 32 byte permutes leave in it, for each of its columns, the eight rows that a lane of a B operand holds, so that
// operand f is columns f, 8 + f, 16 + f ... of the wave's 128, and neither LDS nor other lanes take part.  A row of 16 lanes loads 256 bytes of a row of B.
//   - the row of B for every load stands in a lane of the row of 16, one load for two K-steps, and is added to the lane's column by the DPP of that addition;
//   - the fragments of A, the same for all waves, go through registers into LDS, two K-steps at a time, one slab a wave, two K-steps ahead, with one
//     barrier; 512 columns instead of 256 also halve what is fetched of A, which comes from beyond the L2;
//   - rows of the next K-step are requested as soon as the registers of this one's are free, before its 32 matrix instructions.
// Bound by the load path, 36 KiB a K-step of 64 x 512 (texture-address unit 82 % busy), then by the matrix unit (68 %).
// Blocks of 64 x 64 at 40 %, 8192 x 8192, N = 8192: 473 -> 392 us (with fragments that are always in the L2 371); at 4096 x 4096, N = 4096: 63.4 -> 58.3.
// The same for tiles of one and two slabs is slower (16 x 16 blocks at 10 %, N = 4096: 163 and 200; 32 x 32, 102 and 107): more waves ask for more
// parts of B at a time than stay in the L2.
template <int DT>
__global__ void __launch_bounds__(kThreads, 2) vbr_spmm_wide_kernel(const Params p)
{
    constexpr int S = 4, kBuf = 2 * S * kFragBytes, kOutSlab = kSlabRows * kWideWaveN * 4;
    __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * kOutSlab];      // two buffers of A, then the turned slabs of the four waves
    static_assert(2 * kBuf <= 4 * kOutSlab, "both buffers of A fit");
    int tile, ntile;
    if (!map_workgroup(blockIdx.x, p.n_tiles, p.n_ntiles, p.map, tile, ntile)) return;
    const TileDesc td = p.tiles[tile];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int q = lane >> 4, s16 = lane & 15;
    const int n0 = ntile * kWideN + wave * kWideWaveN;
    const bool live = n0 < p.N;                      // a wave beyond the last column only brings its share of A
    const lds_u8_ptr sm = (lds_u8_ptr)smem;
    const int n_ks = __builtin_amdgcn_readfirstlane(td.n_ks);
    const int32_t c_row = lane < td.n_rows ? p.perm[td.row_begin + lane] : -1;       // C row of row `lane` of the tile

    float4v acc[S][8];
#pragma unroll
    for (int s = 0; s < S; ++s)
#pragma unroll
        for (int f = 0; f < 8; ++f) acc[s][f] = float4v{0.f, 0.f, 0.f, 0.f};

    // A: fragments of slab `wave` (no such slab: the last again, never stored; a row that the last slab does not have: its last one).  Behind the last
    // K-step the loads are out of range and bring zeros.
    const int n_slabs = __builtin_amdgcn_readfirstlane(td.n_slabs);
    const int rows_last = __builtin_amdgcn_readfirstlane(td.n_rows) - (n_slabs - 1) * kSlabRows;
    const uint32_t a_stride = (uint32_t)(((n_slabs - 1) * kFragElems + rows_last * kStepK) * 2);
    const int slab = wave < n_slabs ? wave : n_slabs - 1, rows = slab == n_slabs - 1 ? rows_last : kSlabRows;
    uint32_t a_lane = (uint32_t)((slab * kFragElems + (q * rows + (s16 < rows ? s16 : rows - 1)) * 8) * 2);
    const uint64_t a_addr = reinterpret_cast<uint64_t>(p.vals) + (uint64_t)td.a_off * 16;
    const uint64_t a_base = ((uint64_t)__builtin_amdgcn_readfirstlane((uint32_t)(a_addr >> 32)) << 32) | (uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)a_addr);
    const __amdgpu_buffer_rsrc_t a_rsrc = __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void *>(a_base), 0, (int)((uint32_t)n_ks * a_stride), 0x00020000);
    uint4v stage[2];
    auto load_a = [&]() {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            stage[i] = __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(a_rsrc, (int)a_lane, 0, 0));
            a_lane += a_stride;
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto write_a = [&](int buf) {
#pragma unroll
        for (int i = 0; i < 2; ++i) *(lds_uint4_ptr)(sm + buf * kBuf + (i * S + wave) * kFragBytes + lane * 16) = stage[i];
    };
    auto meet = [&]() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); };      // the loads in flight go on

    if (!live) {
        load_a();
        write_a(0);
        load_a();
        meet();
        for (int k = 0, buf = 1; k < n_ks; k += 2, buf ^= 1) {
            write_a(buf);
            load_a();
            meet();
        }
        return;
    }

    // B: lane (q, s16) loads columns 8 s16 .. 8 s16 + 7 of rows 8 q + j of the K-step in fragment order, j = 0 .. 7.  Lane j + 8 h of a row of 16 looks row j
    // of K-step 2 i + h up for all of them.  (Up to kWideAhead K-steps past the tile's last are looked up, inside the uploaded buffer, and not used.)
    const int last_chunk = (p.N - n0 < kWideWaveN ? p.N - n0 : kWideWaveN) / 8 - 1;
    const uint32_t column = (uint32_t)(s16 <= last_chunk ? s16 : last_chunk) * 16;               // past column N: the last chunk again, never stored
    const uint32_t ldb_bytes = (uint32_t)(p.ldb * 2);
    const char *Bs = reinterpret_cast<const char *>(p.B + n0);
    const __amdgpu_buffer_rsrc_t b_rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(Bs), 0, (int)(p.b_bytes - (uint32_t)n0 * 2), 0x00020000);
    const int lg = p.lg_gran, kk = 16 * (q >> 1) + 4 * (q & 1) + (s16 & 3) + 8 * (s16 >> 2 & 1), in_granule = kk & ((1 << lg) - 1);
    const int32_t *list = p.krow + ((((int64_t)td.ks_begin + (s16 >> 3)) * kStepK + kk) >> lg);
    auto look_up = [&]() -> int32_t {
        const int32_t r = *list;
        list += 2 * kStepK >> lg;
        __builtin_amdgcn_sched_barrier(0);
        return r;
    };
    // the offset of this lane's row of K-step k or k + 1; past the last one: out of range, which brings zeros and costs no traffic
    auto offset = [&](int32_t row, int k) -> uint32_t { return k + (s16 >> 3) < n_ks ? (uint32_t)(row + in_granule) * ldb_bytes : (uint32_t)kNearBytes; };
    uint4v b[8];
    uint32_t turned[8][4];
    auto load_b = [&](uint32_t off) -> uint4v { return __builtin_bit_cast(uint4v, __builtin_amdgcn_raw_buffer_load_b128(b_rsrc, (int)(off + column), 0, 0)); };
    // (the empty statements keep rows in the order written: a wait is for two loads and not for all)
    auto turn = [&](auto j, uint4v &lo, uint4v &hi) {
        asm volatile("" : "+v"(lo), "+v"(hi));
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            turned[2 * w][j.value] = __builtin_amdgcn_perm(hi[w], lo[w], 0x05040100u);
            turned[2 * w + 1][j.value] = __builtin_amdgcn_perm(hi[w], lo[w], 0x07060302u);
        }
        asm volatile("" : "+v"(turned[0][j.value]), "+v"(turned[1][j.value]), "+v"(turned[2][j.value]), "+v"(turned[3][j.value]), "+v"(turned[4][j.value]),
                     "+v"(turned[5][j.value]), "+v"(turned[6][j.value]), "+v"(turned[7][j.value]));
    };
    // one K-step: its rows turned and, in their place, those of the next requested (half h of the offsets); its fragments at `from`
    auto step = [&](lds_u8_ptr from, auto h, uint32_t off) {
        short8v a[S];
#pragma unroll
        for (int s = 0; s < S; ++s) a[s] = *(lds_short8_ptr)(from + s * kFragBytes + lane * 16);
        __builtin_amdgcn_s_setprio(3);
        static_for<4>([&](auto j) {
            turn(j, b[2 * j.value], b[2 * j.value + 1]);
            b[2 * j.value] = load_b(row_lane<8 * h.value + 2 * j.value>(off));
            b[2 * j.value + 1] = load_b(row_lane<8 * h.value + 2 * j.value + 1>(off));
            __builtin_amdgcn_sched_barrier(0);
        });
        __builtin_amdgcn_s_setprio(0);
#pragma unroll
        for (int f = 0; f < 8; ++f) {
            const uint4v bf = {turned[f][0], turned[f][1], turned[f][2], turned[f][3]};
#pragma unroll
            for (int s = 0; s < S; ++s) acc[s][f] = mfma16x16x32<DT>(a[s], __builtin_bit_cast(short8v, bf), acc[s][f]);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    uint32_t off = offset(look_up(), 0);
    load_a();
    static_for<8>([&](auto u) {
        b[u.value] = load_b(row_lane<u.value>(off));
        __builtin_amdgcn_sched_barrier(0);
    });
    int32_t next = look_up();
    write_a(0);
    load_a();
    meet();
    for (int k = 0, buf = 0; k < n_ks; k += 2, buf ^= 1) {
        step(sm + buf * kBuf, constant<1>(), off);
        write_a(buf ^ 1);
        off = offset(next, k + 2);
        next = look_up();
        step(sm + buf * kBuf + S * kFragBytes, constant<0>(), off);
        load_a();
        meet();                                     // the next two K-steps are there, and nobody reads these any more
    }

    // Operand f held every eighth column from f on, so a lane has eight columns in a row of each of its four C rows.  As in the tile kernel the slab is turned
    // round in LDS (the wave's own 8 KiB) and leaves in whole lines, 2 rows x 512 bytes a store.
    const lds_u8_ptr out = sm + wave * kOutSlab;
#pragma unroll
    for (int s = 0; s < S; ++s) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const lds_u8_ptr at = out + i * 2048 + lane * 32;
            *(lds_float4_ptr)at = float4v{acc[s][0][i], acc[s][1][i], acc[s][2][i], acc[s][3][i]};
            *(lds_float4_ptr)(at + 16) = float4v{acc[s][4][i], acc[s][5][i], acc[s][6][i], acc[s][7][i]};
        }
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4v x = *(lds_float4_ptr)(out + i * 2048 + h * 1024 + lane * 16);
                const int32_t row = __shfl(c_row, s * kSlabRows + 4 * (2 * h + (lane >> 5)) + i);
                const int n = n0 + 4 * (lane & 31);
                if (row >= 0 && n < p.N) __builtin_nontemporal_store(x, reinterpret_cast<float4v *>(p.C + row * p.ldc + n));
            }
    }
}

// C rows of tiles without a K-step, the rows of A without entries: zeros.  Bound by what the memory takes, so a workgroup writes whole
// pieces of 4 KiB, one of each of 16 rows (3886 rows of a graph, N = 4096, behind the launch of its other tiles: 27 us in the kernel of the gathered
// tiles, which turns its zeros in LDS like any other result, 25 here; N = 3000: 22 and 17).
__global__ void __launch_bounds__(kThreads) vbr_spmm_zero_rows_kernel(const Params p)
{
    static_assert(kZeroN == 4 * kThreads, "a lane writes four columns");
    const int chunk = blockIdx.x % p.n_ntiles, part = blockIdx.x / p.n_ntiles;
    const TileDesc td = p.tiles[part / kMaxGatherSlabs];
    const int r0 = part % kMaxGatherSlabs * kSlabRows, n = chunk * kZeroN + 4 * threadIdx.x;
    if (n >= p.N) return;
    const const_i32_ptr rows = (const_i32_ptr)p.prow + td.row_begin + r0;
#pragma unroll
    for (int i = 0; i < kSlabRows; ++i) {
        const int64_t row = r0 + i < td.n_rows ? rows[i] : -1;          // a position of the row list may be padding (-1), too
        if (row >= 0) __builtin_nontemporal_store(float4v{0.f, 0.f, 0.f, 0.f}, reinterpret_cast<float4v *>(p.C + row * p.ldc + n));
    }
}

struct PanelParams {
    const PanelDesc *panels;
    const int32_t *pk_meta;   // K-step stream: records {mask, first B row of each granule}
    const int32_t *prow;
    const uint16_t *vals;
    const uint16_t *zfrag;    // 1 KiB of zeros (behind the last fragment): source of the filler loads
    const uint16_t *zeros;    // 256 zero bytes: source of the padding rows of a K-step
    const uint16_t *B;
    float *C;
    int64_t ldb, ldc;
    int32_t N;
    int32_t lg_gran;          // >= 3
    int32_t n_panels;         // T
    int32_t n_ntiles;         // Q = ceil(N / 128)
    ColumnMap map;
};

// Panel kernel: one workgroup (8 waves) owns R slabs (R * 16 rows of short row groups, whatever
// group they belong to) and 128 columns of C, and walks the union of the column blocks of those
// groups.  A B row panel is brought into LDS once per K-step for all R slabs; a slab multiplies only
// in the K-steps where its own groups store a block (mask bit), and only those fragments exist in
// memory.  Waves form a 2 x 4 grid: wave (wr, wc) owns slabs [wr R/2, (wr+1) R/2) x columns
// [32 wc, 32 wc + 32).  A direct-to-LDS load costs the CU about 22 cycles whatever its lane mask, so
// the unit of cost is the load instruction: per K-step 8 for B (1 KiB each) and 8 for A (one
// fragment each; the host splits K-steps that carry more than 8 fragments).
constexpr int kPanelThreads = 512;
template <int DT, int R, int NS, int DA>
__global__ void __launch_bounds__(kPanelThreads) vbr_spmm_panel_kernel(const PanelParams p)
{
    static_assert(NS >= 2 && (NS & (NS - 1)) == 0 && DA == NS - 1, "one ring index for both rings: a power of two, A issued with its B");
    constexpr int kPN = 128;                       // C columns per workgroup
    constexpr int kPRow = kPN * 2;                 // one staged B row: 256 bytes
    constexpr int kPPanel = kStepK * kPRow;        // 8 KiB of B per K-step
    constexpr int kAStage = kPanelMaxFrags * kFragBytes;
    constexpr int NAS = NS;
    constexpr int kBRing = NS * kPPanel;
    constexpr int HS = R / 2;                      // slabs per wave
    // per K-step a wave issues one B load, then one A load; both of K-step ks must have landed
    constexpr int kWait = (NS - 2) * 2;
    static_assert(kWait < 64, "vmcnt is a 6-bit counter");
    static_assert(kPanelMaxFrags == 8, "one fragment load per wave per K-step");
    static_assert(kPanelMetaPad >= NS + 3, "look-ahead of the K-step stream");
    // 2 KiB of slack: the fragment chain reads up to two fragments past the ones it uses
    __shared__ __attribute__((aligned(1024))) unsigned char smem[kBRing + NAS * kAStage + 2 * kFragBytes];

    int tile, ntile;
    if (!map_workgroup(blockIdx.x, p.n_panels, p.n_ntiles, p.map, tile, ntile)) return;
    const PanelDesc pd = p.panels[tile];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wr = wave >> 2, wc = wave & 3;
    const int n0 = ntile * kPN;
    const lds_u8_ptr sm = (lds_u8_ptr)(&smem[0]);
    const uint32_t smem_base = (uint32_t)(uintptr_t)sm;
    const char *zeros = reinterpret_cast<const char *>(p.zeros);
    const int n_ks = pd.n_ks;
    const int q = lane >> 4, s16 = lane & 15;

    float4v acc[HS][2];
#pragma unroll
    for (int s = 0; s < HS; ++s)
#pragma unroll
        for (int f = 0; f < 2; ++f) acc[s][f] = float4v{0.f, 0.f, 0.f, 0.f};

    if (n_ks > 0) {
        // ---- B staging: per K-step every wave issues 1 load: rows 4 wave + (lane / 16) of the
        // K-step, 256 bytes each (16 lanes), into 1 KiB of LDS.  LDS chunk c' of row r holds
        // global chunk c' ^ 2 (r % 8), which spreads the rows of a transposed read over all banks.
        const int lg = p.lg_gran;
        const int gmask = (1 << lg) - 1;
        const int rec = 1 + (kStepK >> lg);                       // int32 per K-step record
        const const_i32_ptr meta = (const_i32_ptr)p.pk_meta + (int64_t)pd.meta_begin * rec;
        // three readers walk the stream: the row lookup of the B loads, the mask of the A loads,
        // the mask of the multiply; each is a pointer that advances by one record per K-step
        const_i32_ptr p_rb = meta + 1 + ((4 * wave) >> lg), p_ma = meta, p_mc = meta;
        const uint32_t ldb_bytes = (uint32_t)(p.ldb * 2);
        const char *Btile = reinterpret_cast<const char *>(p.B) + (int64_t)n0 * 2;
        // chunks at or beyond column N: their lanes fetch the tile's last existing chunk again
        // (the C columns it would feed are never stored, and columns do not mix)
        const int last_chunk = (p.N - n0 < kPN ? p.N - n0 : kPN) / 8 - 1;
        const int rk = 4 * wave + q;                                // this lane's row of the K-step
        const int b_chunk = s16 ^ (2 * (rk & 7));
        const uint32_t b_lane = (uint32_t)(rk & gmask) * ldb_bytes + (b_chunk <= last_chunk ? b_chunk : last_chunk) * 16;
        auto next_rows = [&]() -> int { const int v = *p_rb; p_rb += rec; return v; };
        auto next_ma = [&]() -> uint32_t { const uint32_t v = (uint32_t)*p_ma; p_ma += rec; return v; };
        auto next_mc = [&]() -> uint32_t { const uint32_t v = (uint32_t)*p_mc; p_mc += rec; return v; };
        int rb0, rb1;
        auto issue_b = [&](int slot) {
            const uint32_t sb = smem_base + slot * kPPanel + 4 * wave * kPRow;
            if (rb0 >= 0) {
                dma16_base(b_lane, Btile + (uint64_t)(uint32_t)rb0 * ldb_bytes, sb);
            } else {         // padding rows of the K-step: zeros
                dma16(zeros, sb);
            }
        };
        // ---- A staging: the fragments of a K-step follow each other in memory, one per present
        // slab in rising slab order; fragment i is loaded by wave i.  Every wave issues one load
        // per K-step whatever the count: a wave without a fragment loads 1 KiB of zeros instead.
        const char *a_next = reinterpret_cast<const char *>(p.vals) + pd.a_off * 16;
        const char *zfrag = reinterpret_cast<const char *>(p.zfrag);
        uint32_t mA0, mA1;
        auto issue_a = [&](int slot) {
            const uint32_t sa = smem_base + kBRing + slot * kAStage;
            const int cnt = __builtin_popcount(mA0);
            dma16_base(lane * 16, wave < cnt ? a_next + wave * kFragBytes : zfrag, sa + wave * kFragBytes);
            a_next += cnt * kFragBytes;
        };

        uint32_t b_off[2];
        {
            const int R0 = 16 * (q >> 1) + 4 * (q & 1) + (s16 >> 2);
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const int chunk = 4 * wc + 2 * f + ((s16 & 3) >> 1);
                b_off[f] = R0 * kPRow + ((chunk ^ (2 * (R0 & 7))) << 4) + (s16 & 1) * 8;
            }
        }
        // the LDS reads of a K-step are issued before the next loads (the inline asm keeps that
        // order): B fragments of the wave's 32 columns and the first of its A fragments
        short8v bfrag[2], a_nxt;
        lds_u8_ptr fa;
        auto read_frags = [&](int bslot, int aslot, uint32_t m) {
            const lds_u8_ptr sb = sm + bslot * kPPanel;
            fa = sm + kBRing + aslot * kAStage + __builtin_popcount(m & ((1u << (wr * HS)) - 1u)) * kFragBytes + lane * 16;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const short4v lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(sb + b_off[f]));
                const short4v hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(sb + b_off[f] + 8 * kPRow));
                bfrag[f] = short8v{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
            }
            a_nxt = *(lds_short8_ptr)fa;
        };
        auto multiply = [&](uint32_t mh) {
            // the fragments of this wave's present slabs follow each other: read one ahead
#pragma unroll
            for (int s = 0; s < HS; ++s) {
                if (mh >> s & 1) {
                    const short8v a_cur = a_nxt;
                    fa += kFragBytes;
                    a_nxt = *(lds_short8_ptr)fa;
#pragma unroll
                    for (int f = 0; f < 2; ++f) acc[s][f] = mfma16x16x32<DT>(bfrag[f], a_cur, acc[s][f]);
                }
            }
        };

        // ---- software pipeline: K-steps 0 .. NS-2 are issued up front (B then A each); iteration
        // ks issues K-step ks+NS-1 into the slot K-step ks-1 has left.  K-steps past the end are
        // filler records of the stream (mask 0, rows of the last step), so the loads in flight per
        // wave never change in number.
        rb0 = next_rows();
        rb1 = next_rows();
        mA0 = next_ma();
        mA1 = next_ma();
#pragma unroll
        for (int t = 0; t < NS - 1; ++t) {
            issue_b(t);
            issue_a(t);
            rb0 = rb1; mA0 = mA1;
            rb1 = next_rows();
            mA1 = next_ma();
        }
        uint32_t mC0 = next_mc(), mC1 = next_mc();
        for (int ks = 0; ks < n_ks; ++ks) {
            wait_vmcnt<kWait>();
            __builtin_amdgcn_s_barrier();
            // scalar lookups (issued at the end of earlier iterations) are waited for here, not behind the LDS reads
            asm volatile("" ::"s"(rb0), "s"(mA0), "s"(mC0));
            const int cur = ks & (NS - 1), fill = (ks - 1) & (NS - 1);
            const uint32_t mh = (mC0 >> (wr * HS)) & ((1u << HS) - 1u);      // this wave's slabs
            if (mh != 0) read_frags(cur, cur, mC0);
            issue_b(fill);
            issue_a(fill);
            if (mh != 0) multiply(mh);
            rb0 = rb1; mA0 = mA1; mC0 = mC1;
            rb1 = next_rows();
            mA1 = next_ma();
            mC1 = next_mc();
        }
        wait_vmcnt<0>();
    }

#pragma unroll
    for (int s = 0; s < HS; ++s) {
        const int rr = (wr * HS + s) * kSlabRows + s16;
        const int64_t orig = rr < pd.n_rows ? p.prow[pd.row_begin + rr] : -1;
        if (orig >= 0) {                 // a position of the low-row list may be padding (-1)
            float *crow = p.C + orig * p.ldc;
#pragma unroll
            for (int f = 0; f < 2; ++f) {
                const int n = n0 + wc * 32 + 16 * f + 4 * q;
                if (n < p.N) *reinterpret_cast<float4v *>(crow + n) = acc[s][f];
            }
        }
    }
}


template <int DT>
int launch_all(const vbr *v, const Params &base, PanelParams pp, hipStream_t stream)
{
    Launch plan[VBR_MAX_LAUNCHES];
    const int n = plan_launches(v, base.N, base.ldb % 64 == 0 && (reinterpret_cast<uintptr_t>(base.B) & 127) == 0, plan, base.ldb);
    for (int i = 0; i < n; ++i)
        if (plan[i].grid > INT32_MAX) return VBR_EINVAL;
    for (int i = 0; i < n; ++i) {
        const Launch &L = plan[i];
        Params p = base;
        p.tiles = base.tiles + L.first_tile;
        p.n_tiles = L.n_tiles;
        const dim3 grid((unsigned)L.grid);
        if (L.kind == VBR_LAUNCH_PANEL) {
            pp.map = column_map((uint32_t)pp.n_ntiles, L.even);
            hipLaunchKernelGGL((vbr_spmm_panel_kernel<DT, 8, 4, 3>), grid, dim3(kPanelThreads), 0, stream, pp);
            const hipError_t e = hipGetLastError();
            if (e != hipSuccess) { set_last_hip_error((int)e); return VBR_EHIP; }
            continue;
        }
        if (L.stream) {
            const int rc = launch_stream(v, L, base.B, base.ldb, base.C, base.ldc, base.N, stream);
            if (rc != VBR_OK) return rc;
            continue;
        }
        const bool few = L.few;
        void (*kernel)(Params) = nullptr;
        if (L.kind == VBR_LAUNCH_TILE_MIXED) {
            p.whole = L.whole;
            p.rest = L.rest;
            p.split = L.split;
            p.n_tiles = L.n_tiles + 3 * p.rest;
        } else if (L.split) {
            p.n_ntiles = (p.N + kDeepN - 1) / kDeepN;
        } else if (L.wide) {
            p.n_ntiles = (p.N + kWideN - 1) / kWideN;
        }
        switch (L.kind) {
        case VBR_LAUNCH_TILE_MIXED:
            if (v->class_count[3] > 0) kernel = few ? vbr_spmm_mixed_kernel<DT, 8, kStagesFew, 3> : vbr_spmm_mixed_kernel<DT, 8, kStages, 2>;
            else kernel = few ? vbr_spmm_mixed_kernel<DT, 4, kStagesFew, 3> : vbr_spmm_mixed_kernel<DT, 4, kStages, 2>;
            break;
        case VBR_LAUNCH_GATHER_1:
            kernel = L.split ? vbr_spmm_split_kernel<DT, 1, true> : few ? vbr_spmm_kernel<DT, 1, kStagesFew, kStagesFew, true> : vbr_spmm_kernel<DT, 1, kStages, kADistance, true>;
            break;
        case VBR_LAUNCH_GATHER_2:
            kernel = L.split ? vbr_spmm_split_kernel<DT, 2, true> : few ? vbr_spmm_kernel<DT, 2, kStagesFew, kStagesFew, true> : vbr_spmm_kernel<DT, 2, kStages, kADistanceTwo, true>;
            break;
        case VBR_LAUNCH_GATHER_4:
            kernel = L.split ? vbr_spmm_split_kernel<DT, 4, true> : few ? vbr_spmm_kernel<DT, 4, kStagesTall, kADistance, true> : vbr_spmm_kernel<DT, 4, kStages, kADistance, true>;
            break;
        case VBR_LAUNCH_TILE_1:
            kernel = L.split ? vbr_spmm_split_kernel<DT, 1, false> : few ? vbr_spmm_kernel<DT, 1, kStagesFew, kStagesFew> : vbr_spmm_kernel<DT, 1, kStages, kADistance>;
            break;
        case VBR_LAUNCH_TILE_2:
            kernel = L.split ? vbr_spmm_split_kernel<DT, 2, false> : few ? vbr_spmm_kernel<DT, 2, kStagesFew, kStagesFew> : vbr_spmm_kernel<DT, 2, kStages, kADistanceTwo>;
            break;
        case VBR_LAUNCH_TILE_4:
            kernel = L.split ? vbr_spmm_split_kernel<DT, 4, false> : L.wide ? vbr_spmm_wide_kernel<DT> : vbr_spmm_kernel<DT, 4, kStagesTall, kADistance>;
            break;
        case VBR_LAUNCH_ZERO_ROWS:
            kernel = vbr_spmm_zero_rows_kernel;
            p.n_ntiles = (p.N + kZeroN - 1) / kZeroN;
            break;
        default:
            kernel = vbr_spmm_kernel<DT, 8, kStagesTall, kADistance>;
            break;
        }
        p.map = column_map((uint32_t)p.n_ntiles, L.even);
        hipLaunchKernelGGL(kernel, grid, dim3(kThreads), 0, stream, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) { set_last_hip_error((int)e); return VBR_EHIP; }
    }
    return VBR_OK;
}

}  // namespace
}  // namespace vbrk

extern "C" int vbr_last_hip_error(void) { return vbrk::g_last_hip_error; }

extern "C" int vbr_upload(vbr_t *v, void *buf_dev, void *hip_stream)
{
    if (!v || !buf_dev || (reinterpret_cast<uintptr_t>(buf_dev) & 255) != 0) return VBR_EINVAL;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    char *d = static_cast<char *>(buf_dev);
    const vbrk::DeviceLayout &L = v->lay;
    struct Part { int64_t off; const void *src; size_t bytes; };
    static const unsigned char kZeros[256] = {0};
    const Part rows = v->by_entries ? Part{L.prow_off, v->entries.row.data(), v->entries.row.size() * sizeof(vbrk::EntryRow)} : Part{L.prow_off, v->prow.data(), v->prow.size() * 4};
    const Part cols = v->by_entries ? Part{L.gcol_off, v->entries.entry.get(), v->entries.bytes()} : Part{L.gcol_off, v->gcol.data(), v->gcol.size() * 4};
    const Part parts[11] = {
        cols,
        {L.panels_off, v->panels.data(), v->panels.size() * sizeof(vbrk::PanelDesc)},
        {L.pk_meta_off, v->pk_meta.data(), v->pk_meta.size() * 4},
        rows,
        {L.stream_tiles_off, v->stream_tiles.data(), v->stream_tiles.size() * sizeof(vbrk::StreamTile)},
        {L.stream_steps_off, v->stream_steps.data(), v->stream_steps.size() * sizeof(vbrk::StreamRecord)},
        {L.zeros_off, kZeros, sizeof(kZeros)},
        {L.tiles_off, v->dev_tiles.data(), v->dev_tiles.size() * sizeof(vbrk::TileDesc)},
        {L.krow_off, v->krow.data(), v->krow.size() * 4},
        {L.perm_off, v->perm.data(), v->perm.size() * 4},
        {L.vals_off, v->vals.data(), v->vals.size() * 2},
    };
    for (const Part &pt : parts) {
        if (pt.bytes == 0) continue;
        hipError_t e = hipMemcpyAsync(d + pt.off, pt.src, pt.bytes, hipMemcpyHostToDevice, stream);
        if (e != hipSuccess) { vbrk::set_last_hip_error((int)e); return VBR_EHIP; }
    }
    hipError_t e = hipStreamSynchronize(stream);
    if (e != hipSuccess) { vbrk::set_last_hip_error((int)e); return VBR_EHIP; }
    v->dev = buf_dev;
    return VBR_OK;
}

extern "C" int vbr_spmm(const vbr_t *v, const void *B_dev, int64_t ldb, float *C_dev, int64_t ldc,
                        int64_t N, void *hip_stream)
{
    if (!v) return VBR_EINVAL;
    if (!v->dev) return VBR_ESTATE;
    if (N < 0 || N % 8 != 0 || N > (int64_t)INT32_MAX - 1024) return VBR_EINVAL;
    if (N == 0 || v->n_rows == 0) return VBR_OK;
    if (!B_dev || !C_dev || ldb < N || ldc < N || ldb % 8 != 0 || ldc % 4 != 0) return VBR_EINVAL;
    if (ldb >= ((int64_t)1 << 26)) return VBR_EUNSUPPORTED;   // a lane's offset inside a 32-row granule of B is 32 bits
    if ((reinterpret_cast<uintptr_t>(B_dev) & 15) != 0 || (reinterpret_cast<uintptr_t>(C_dev) & 15) != 0) return VBR_EINVAL;
    const char *d = static_cast<const char *>(v->dev);
    if (v->by_entries) {
        const vbrk::EntryRowsDev rows{reinterpret_cast<const vbrk::EntryRow *>(d + v->lay.prow_off), d + v->lay.gcol_off, v->entries.near};
        const vbrk::EntryLaunch L = vbrk::plan_entry_rows(v->entries.start, v->n_cols, N, ldb % 64 == 0 && (reinterpret_cast<uintptr_t>(B_dev) & 127) == 0);
        return vbrk::launch_entry_rows(L, v->dtype, rows, v->n_rows, v->n_cols, B_dev, ldb, C_dev, ldc, N, hip_stream);
    }
    vbrk::Params p;
    p.tiles = reinterpret_cast<const vbrk::TileDesc *>(d + v->lay.tiles_off);
    p.krow = reinterpret_cast<const int32_t *>(d + v->lay.krow_off);
    p.perm = reinterpret_cast<const int32_t *>(d + v->lay.perm_off);
    p.vals = reinterpret_cast<const uint16_t *>(d + v->lay.vals_off);
    p.B = static_cast<const uint16_t *>(B_dev);
    p.C = C_dev;
    p.ldb = ldb;
    p.ldc = ldc;
    p.N = (int32_t)N;
    p.lg_gran = v->lg_gran;
    p.n_tiles = 0;
    p.n_ntiles = (int32_t)((N + vbrk::kTileN - 1) / vbrk::kTileN);
    vbrk::PanelParams pp;
    pp.panels = reinterpret_cast<const vbrk::PanelDesc *>(d + v->lay.panels_off);
    pp.pk_meta = reinterpret_cast<const int32_t *>(d + v->lay.pk_meta_off);
    pp.zfrag = p.vals + (v->vals.size() - vbrk::kFragElems);
    pp.prow = reinterpret_cast<const int32_t *>(d + v->lay.prow_off);
    pp.vals = p.vals;
    pp.zeros = reinterpret_cast<const uint16_t *>(d + v->lay.zeros_off);
    pp.B = p.B;
    pp.C = C_dev;
    pp.ldb = ldb;
    pp.ldc = ldc;
    pp.N = (int32_t)N;
    pp.lg_gran = v->lg_gran;
    pp.n_panels = (int32_t)v->panels.size();
    pp.n_ntiles = (int32_t)((N + 127) / 128);
    p.gcol = reinterpret_cast<const int32_t *>(d + v->lay.gcol_off);
    p.b_fits24 = (v->n_cols * ldb * 2 + N * 2) < ((int64_t)1 << 32) && v->n_cols <= (1 << 24) && ldb * 2 < (1 << 24) ? 1 : 0;
    p.b_bytes = (uint32_t)vbrk::b_bytes_of(v->n_cols, ldb, N);
    p.prow = pp.prow;
    hipStream_t stream = static_cast<hipStream_t>(hip_stream);
    return v->dtype == VBR_F16 ? vbrk::launch_all<VBR_F16>(v, p, pp, stream) : vbrk::launch_all<VBR_BF16>(v, p, pp, stream);
}
