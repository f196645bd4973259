// Declarations shared by the host-side translation units of the library.
#pragma once

#include "host_threads.h"
#include "vbr_internal.h"

namespace vbrk {

// Canonical-CSR check described in vbr_spmm.h; VBR_OK or VBR_EINVAL.
int validate_csr(const vbr_csr_t *csr, bool need_vals);

int sa1_reorder_impl(const vbr_csr_t *csr, int32_t col_block, double tau, int32_t *perm,
                     int32_t *row_groups, int32_t *n_groups);

// vbr_build without its first checks; schedules: with the stream kernel's where no call takes it, too.
int build_impl(const vbr_csr_t *csr, const int32_t *perm, const int32_t *row_groups, int32_t n_groups, int32_t col_block, vbr_t **out, bool schedules);

// The launches one vbr_spmm call issues for dense width N, in issue order (at most VBR_MAX_LAUNCHES):
// kernel, first tile and number of tiles (or panels) of the launch, grid size; split: 64 columns of C a workgroup,
// whose waves split the K-steps; few: rings of four slots; wide: the wide kernel.  aligned: rows of B begin on a cache line.
// split: 0, or the K-steps from which on its tiles are split, of the mixed kernel `rest` of them from number `whole` on
struct Launch { int32_t kind; int32_t first_tile, n_tiles; int64_t grid; int32_t split = 0; bool few = false; int32_t whole = 0, rest = 0; bool even = false, wide = false, stream = false; };
int plan_launches(const vbr *v, int64_t N, bool aligned, Launch out[VBR_MAX_LAUNCHES], int64_t ldb = 0);      // 0: N
int launch_stream(const vbr *v, const Launch &L, const void *B_dev, int64_t ldb, float *C_dev, int64_t ldc, int64_t N, void *hip_stream);

constexpr int kEntryLongRow = 256;     // entries beyond which a row gets a wave of its own ...
constexpr int kEntryHugeRow = 1024;    // ... and a workgroup of its own

// The rows of a matrix as lists of entries.
void make_entry_rows(const vbr_csr_t *csr, Team &team, EntryRows &out);

// The same on the device.
struct EntryRowsDev {
    const EntryRow *row;
    const void *entry;
    bool near;
};
// six: only six workgroups on a CU at a time, of the eight that fit; together: waves wait for all of their loads of B every eight of them
struct EntryLaunch { int32_t lanes, n_huge, n_long; int64_t waves, grid; bool even, six, together; };
// the launch for dense width N; aligned: rows of B begin on a cache line
EntryLaunch plan_entry_rows(const std::vector<int64_t> &start, int64_t n_cols, int64_t N, bool aligned);
int launch_entry_rows(const EntryLaunch &L, int32_t dtype, const EntryRowsDev &rows, int64_t n_rows, int64_t n_cols,
                      const void *B_dev, int64_t ldb, float *C_dev, int64_t ldc, int64_t N, void *hip_stream);

// Thread-local code of the last failing HIP call.
void set_last_hip_error(int code);

}  // namespace vbrk
