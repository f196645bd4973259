"""Host side of the C-ABI library against the oracle (CPU only, no GPU calls).

sa1_reorder / vbr_build / vbr_get_index / vbr_unpack_block are host code inside the same shared
library as the kernels; perm, row_groups and the VBR index arrays must match the oracle bit for
bit.  Also: the library loads and exports every symbol the header declares, and the error paths.
"""
import ctypes
import os
import re
import shutil
import subprocess

import numpy as np
import pytest

import oracle
from paper_2202_05868_amd import binding, build, synth
from helpers import check_partition_shape, csr_from_rows, random_csr, sa1_sets

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
TAUS = [0.0, 0.1, 0.2, 0.3, 0.4, 0.5, 0.6, 0.7, 0.8, 0.9, 1.0]


def test_library_exports_every_declared_symbol():
    header = open(os.path.join(ROOT, "include", "vbr_spmm.h")).read()
    declared = set(re.findall(r"^(?:const char \*|int64_t |int |void )\s*(\w+)\s*\(", header, flags=re.M))
    assert declared == set(binding.EXPORTS), declared ^ set(binding.EXPORTS)
    lib = ctypes.CDLL(binding.LIB_PATH)
    for name in declared:
        assert hasattr(lib, name), name


def assert_same_blocking(csr, col_block, tau):
    p0, g0 = oracle.sa1(csr, col_block, tau)
    p1, g1 = binding.sa1_reorder(csr, col_block, tau)
    assert np.array_equal(p0, p1), "perm differs"
    assert np.array_equal(g0, g1), "row_groups differ"
    return p1, g1


def assert_same_index(csr, perm, rg, col_block, check_values=True):
    bp0, bc0, bo0 = oracle.vbr_index(csr, perm, rg, col_block)
    v = binding.vbr_build(csr, perm, rg, col_block)
    v.audit()                       # every index the kernels use lies inside what it indexes
    ix = v.index()
    assert np.array_equal(ix["perm"], perm) and np.array_equal(ix["row_groups"], rg)
    assert np.array_equal(ix["blk_ptr"], bp0)
    assert np.array_equal(ix["blk_col"], bc0)
    assert np.array_equal(ix["blk_off"], bo0)
    assert ix["stored_elems"] == bo0[-1] and ix["n_blocks"] == len(bc0)
    if check_values:
        for g in range(len(rg) - 1):
            h = int(rg[g + 1] - rg[g])
            for b in range(int(bp0[g]), int(bp0[g + 1])):
                got = v.unpack_block(b, h, col_block)
                want = oracle.block_bits(csr, perm, rg, g, int(bc0[b]), col_block)
                assert np.array_equal(got, want), (g, b)
    return v


@pytest.mark.parametrize("col_block", [1, 2, 3, 8, 16])
def test_reorder_and_index_match_oracle_on_random_matrices(col_block):
    rng = np.random.default_rng(100 + col_block)
    for trial in range(12):
        n_rows = int(rng.integers(1, 90))
        kb = int(rng.integers(1, 20))
        csr = random_csr(rng, n_rows, kb * col_block, float(rng.choice([0.02, 0.1, 0.3, 0.7])),
                         dtype="bf16" if trial % 2 else "f16")
        for tau in TAUS:
            perm, rg = assert_same_blocking(csr, col_block, tau)
            check_partition_shape(perm, rg, n_rows)
        assert_same_index(csr, perm, rg, col_block)


def test_reorder_matches_set_based_transcription_too():
    rng = np.random.default_rng(9)
    for trial in range(40):
        csr = random_csr(rng, int(rng.integers(1, 12)), 12, 0.3)
        for tau in TAUS:
            p0, g0 = sa1_sets(csr, 2, tau)
            p1, g1 = binding.sa1_reorder(csr, 2, tau)
            assert np.array_equal(p0, p1) and np.array_equal(g0, g1)


def test_more_than_64_column_blocks_and_hash_collisions():
    # patterns {0,3} and {1,2} share the Eq. 5 hash (3) and the length: they must stay apart
    csr = csr_from_rows([[0, 3], [1, 2], [0, 3], [1, 2], [0, 1, 2]], n_cols=4)
    perm, rg = assert_same_blocking(csr, 1, 1.0)
    assert len(rg) - 1 == 3
    rng = np.random.default_rng(2)
    csr = random_csr(rng, 300, 200 * 2, 0.03)        # 200 column blocks: bitsets of 4 words
    for tau in (0.2, 0.5):
        perm, rg = assert_same_blocking(csr, 2, tau)
    assert_same_index(csr, perm, rg, 2)


@pytest.mark.parametrize("n_rows,n_blocks,density", [(3000, 600, 0.004), (3000, 600, 0.02), (2500, 40, 0.5),
                                                     (2000, 130, 0.08)])
def test_reorder_at_sizes_where_both_scan_strategies_run(n_rows, n_blocks, density):
    # sparse quotient rows over many column blocks: candidates come from the column blocks' row
    # lists; dense ones over few blocks: every remaining row is compared.  Rows are drawn from a
    # few hundred base patterns with noise so that merges, refusals and the size cap all occur.
    rng = np.random.default_rng(n_rows + n_blocks)
    base = rng.random((300, n_blocks)) < density
    rows = []
    for i in range(n_rows):
        pat = base[rng.integers(0, 300)] ^ (rng.random(n_blocks) < density * 0.15)
        rows.append((np.nonzero(pat)[0] * 2 + rng.integers(0, 2)).tolist())
    csr = csr_from_rows(rows, n_cols=2 * n_blocks, rng=rng)
    for tau in (0.0, 0.05, 0.3, 0.6, 0.9, 1.0):
        perm, rg = assert_same_blocking(csr, 2, tau)
        check_partition_shape(perm, rg, n_rows)


@pytest.mark.parametrize("threads", ["1", "3", "8"])
@pytest.mark.parametrize("n_rows,n_blocks,density", [(3000, 600, 0.004), (3000, 600, 0.02), (2500, 40, 0.5),
                                                     (2000, 130, 0.08)])
def test_reorder_with_several_host_threads_is_the_sequential_result(monkeypatch, threads, n_rows, n_blocks, density):
    # the candidate search that runs ahead of the greedy pass on several threads must not change
    # a single decision: same inputs as above (merges, refusals and the size cap all occur), the
    # thread count forced through the environment, compared with the oracle
    monkeypatch.setenv("VBR_SA1_THREADS", threads)
    rng = np.random.default_rng(n_rows + n_blocks)
    base = rng.random((300, n_blocks)) < density
    rows = []
    for i in range(n_rows):
        pat = base[rng.integers(0, 300)] ^ (rng.random(n_blocks) < density * 0.15)
        rows.append((np.nonzero(pat)[0] * 2 + rng.integers(0, 2)).tolist())
    csr = csr_from_rows(rows, n_cols=2 * n_blocks, rng=rng)
    for tau in (0.05, 0.3, 0.6, 0.9, 1.0):
        perm, rg = assert_same_blocking(csr, 2, tau)
        check_partition_shape(perm, rg, n_rows)


def test_reorder_threads_on_the_unstructured_workload_reduced(monkeypatch):
    # the workload the parallel search is for: Erdos-Renyi rows, next to no merges
    w = synth.workload("c5", scale=0.25)
    for threads in ("1", "4"):
        monkeypatch.setenv("VBR_SA1_THREADS", threads)
        for tau in (0.1, 0.3):
            assert_same_blocking(w["A"], w["col_block"], tau)


@pytest.mark.parametrize("threads", ["1", "5"])
@pytest.mark.parametrize("n_blocks", [64, 65, 129, 192, 257])
def test_reorder_by_bit_set_scan_and_by_lists_at_the_word_counts_of_the_scan(monkeypatch, threads, n_blocks):
    # bit sets of 1, 2, 4, 4 (padded) and 5 words; a class count that is no multiple of 8; skewed block
    # frequencies (rare blocks make short lists, common ones a bit-set scan), patterns that repeat, merges
    monkeypatch.setenv("VBR_SA1_THREADS", threads)
    rng = np.random.default_rng(n_blocks)
    freq = np.minimum(0.9, 1.5 / (1 + np.arange(n_blocks)))
    base = rng.random((90, n_blocks)) < freq
    rows = [np.nonzero(base[rng.integers(90)] ^ (rng.random(n_blocks) < 0.01))[0] * 2 for _ in range(701)]
    csr = csr_from_rows([r.tolist() for r in rows], 2 * n_blocks)
    for tau in (0.05, 0.3, 0.5, 0.75, 0.99, 1.0):
        p0, g0 = oracle.sa1(csr, 2, tau)
        perm, rg = binding.sa1_reorder(csr, 2, tau)
        assert np.array_equal(perm, p0) and np.array_equal(rg, g0), tau


@pytest.mark.parametrize("threads", ["1", "3"])
@pytest.mark.parametrize("tau", [5e-324, 1e-300, 1e-20, 1e-18, 1e-17])
def test_reorder_at_thresholds_next_to_zero(monkeypatch, threads, tau):
    # blocks of a row divided by the threshold exceed every integer; any block in common is similarity enough, and
    # only the merge limit decides
    monkeypatch.setenv("VBR_SA1_THREADS", threads)
    for n_rows, n_blocks, density in [(50, 20, 0.15), (200, 64, 0.15), (120, 300, 0.02), (60, 30, 0.6)]:
        csr = random_csr(np.random.default_rng(3), n_rows, 2 * n_blocks, density / 2)
        perm, rg = assert_same_blocking(csr, 2, tau)
        curve = binding.sa1_blocking_curve(csr, 2, [tau], 8)
        point = oracle.blocking_curve(csr, 2, [tau], 8)["points"][0]
        assert all(curve[k][0] == point[k] for k in ("n_groups", "n_blocks", "stored_elems", "sum_heights"))


@pytest.mark.parametrize("name,scale,noise", [("c1", 1.0, True), ("c1", 1.0, False), ("c2", 0.25, True),
                                               ("c3", 0.125, True), ("c4", 0.125, True), ("c5", 0.0625, True)])
def test_workloads_small_scale_bit_exact(name, scale, noise):
    w = synth.workload(name, scale=scale, noise=noise)
    for tau in w["taus"]:
        perm, rg = assert_same_blocking(w["A"], w["col_block"], tau)
    v = assert_same_index(w["A"], perm, rg, w["col_block"], check_values=False)
    # values: sampled blocks
    ix = v.index()
    rng = np.random.default_rng(0)
    grp_of_blk = np.repeat(np.arange(ix["n_groups"]), np.diff(ix["blk_ptr"]))
    for b in rng.choice(ix["n_blocks"], size=min(40, ix["n_blocks"]), replace=False):
        g = int(grp_of_blk[b])
        h = int(rg[g + 1] - rg[g])
        assert np.array_equal(v.unpack_block(int(b), h, w["col_block"]),
                              oracle.block_bits(w["A"], perm, rg, g, int(ix["blk_col"][b]), w["col_block"]))


def test_build_accepts_any_valid_partition_and_tall_groups():
    rng = np.random.default_rng(4)
    csr = random_csr(rng, 300, 64, 0.1)
    perm = rng.permutation(300).astype(np.int32)
    rg = np.array([0, 1, 18, 150, 151, 300], dtype=np.int32)     # heights 1, 17, 132, 1, 149
    assert_same_index(csr, perm, rg, 16)
    assert_same_index(csr, np.arange(300, dtype=np.int32), np.array([0, 300], dtype=np.int32), 4)


def test_panels_unpack_exactly():
    # more than 4096 rows in groups shorter than a slab: they are packed as panels; 12 column
    # blocks at high density make nearly every slab present in every K-step (full masks); every
    # stored block must unpack bit-exactly
    rng = np.random.default_rng(77)
    csr = random_csr(rng, 6000, 12 * 8, 0.08)
    perm, rg = assert_same_blocking(csr, 8, 0.9)
    h = np.diff(rg)
    assert h[h < 16].sum() >= 4096
    v = assert_same_index(csr, perm, rg, 8, check_values=False)
    ix = v.index()
    grp_of_blk = np.repeat(np.arange(ix["n_groups"]), np.diff(ix["blk_ptr"]))
    for b in rng.choice(ix["n_blocks"], size=400, replace=False):
        g = int(grp_of_blk[b])
        assert np.array_equal(v.unpack_block(int(b), int(rg[g + 1] - rg[g]), 8),
                              oracle.block_bits(csr, perm, rg, g, int(ix["blk_col"][b]), 8))


def test_empty_rows_and_empty_matrix():
    csr = csr_from_rows([[], [1], [], [1, 5]], n_cols=8)
    perm, rg = assert_same_blocking(csr, 2, 0.5)
    assert_same_index(csr, perm, rg, 2)
    empty = csr_from_rows([[], [], []], n_cols=8)
    perm, rg = assert_same_blocking(empty, 4, 0.5)
    assert len(rg) == 2
    v = assert_same_index(empty, perm, rg, 4)
    assert v.index()["n_blocks"] == 0 and v.device_bytes() >= 256
    none = csr_from_rows([], n_cols=8)                    # no rows at all
    perm, rg = assert_same_blocking(none, 4, 0.5)
    assert perm.size == 0 and rg.tolist() == [0]
    v = binding.vbr_build(none, perm, rg, 4)
    assert v.index()["n_groups"] == 0 and v.device_bytes() >= 256


def test_graph_workload_reduced_bit_exact():
    w = synth.workload("rmat", scale=0.125)
    a = w["A"]
    assert a["n_rows"] == 2048 and 20 < a["nnz"] / a["n_rows"] < 33      # duplicate edges collapse
    for tau in (0.2, 0.4):
        perm, rg = assert_same_blocking(a, w["col_block"], tau)
    assert_same_index(a, perm, rg, w["col_block"], check_values=False)


def test_comparator_handle_checks_its_input():
    csr = csr_from_rows([[0, 1], [2]], n_cols=4)
    h = binding.CsrDev(csr)
    assert binding._lib.csr_device_bytes(h._h) % 256 == 0
    assert binding._lib.csr_spmm(h._h, 256, 8, 256, 8, 8, 0) == -4       # before upload: state error, no GPU touched
    bad = dict(csr)
    bad["col_idx"] = np.array([1, 0, 2], dtype=np.int32)
    with pytest.raises(binding.VbrError):
        binding.CsrDev(bad)


def test_error_paths():
    csr = csr_from_rows([[0, 1], [2]], n_cols=4)
    with pytest.raises(binding.VbrError):
        binding.sa1_reorder(csr, 3, 0.5)                 # 4 % 3 != 0
    with pytest.raises(binding.VbrError):
        binding.sa1_reorder(csr, 2, 1.5)                 # tau out of range
    with pytest.raises(binding.VbrError):
        binding.sa1_reorder(csr, 0, 0.5)
    bad = dict(csr)
    bad["col_idx"] = np.array([1, 0, 2], dtype=np.int32)  # unsorted inside a row
    with pytest.raises(binding.VbrError):
        binding.sa1_reorder(bad, 2, 0.5)
    bad["col_idx"] = np.array([0, 1, 7], dtype=np.int32)  # out of range
    with pytest.raises(binding.VbrError):
        binding.sa1_reorder(bad, 2, 0.5)
    with pytest.raises(binding.VbrError):
        binding.vbr_build(csr, np.array([0, 0], dtype=np.int32), np.array([0, 2], dtype=np.int32), 2)  # not a bijection
    with pytest.raises(binding.VbrError):
        binding.vbr_build(csr, np.array([0, 1], dtype=np.int32), np.array([0, 1, 1, 2], dtype=np.int32), 2)  # empty group
    v = binding.vbr_build(csr, np.array([1, 0], dtype=np.int32), np.array([0, 2], dtype=np.int32), 2)
    # spmm before upload: state error, no GPU touched
    assert binding.vbr_spmm_raw(v, 256, 8, 256, 8, 8, 0) == -4
    assert binding._lib.vbr_strerror(-4) == b"call out of order"


def test_binding_rejects_operands_the_kernels_would_read_or_write_out_of_bounds():
    # the C ABI gets raw addresses; shapes, types and the device are checked in the binding,
    # before anything is launched (CPU tensors suffice: every check precedes the launch)
    import torch
    csr = csr_from_rows([[0, 1], [2], [5]], n_cols=8)
    v = binding.vbr_build(csr, np.arange(3, dtype=np.int32), np.array([0, 3], dtype=np.int32), 2)
    h = binding.CsrDev(csr)
    fake_dev = torch.empty(1, dtype=torch.uint8)          # stands for the uploaded buffer (CPU "device")
    for what, obj in (("vbr_spmm", v), ("csr_spmm", h)):
        def check(b, c, dev=fake_dev):
            return binding._check_operands(what, "f16", obj.n_rows, obj.n_cols, dev, b, c)
        good_b = torch.zeros((8, 16), dtype=torch.float16)
        good_c = torch.zeros((3, 16), dtype=torch.float32)
        assert check(good_b, good_c) is good_c
        assert tuple(check(good_b, None).shape) == (3, 16)
        for b, c in [(torch.zeros((7, 16), dtype=torch.float16), good_c),            # B too short
                     (good_b.to(torch.bfloat16), good_c),                            # wrong type
                     (torch.zeros((16, 8), dtype=torch.float16).t(), good_c),        # column stride
                     (good_b, torch.zeros((2, 16), dtype=torch.float32)),            # C too short
                     (good_b, torch.zeros((4, 16), dtype=torch.float32)),            # C too tall
                     (good_b, torch.zeros((3, 8), dtype=torch.float32)),             # C too narrow
                     (good_b, torch.zeros((3, 16), dtype=torch.float64)),            # C type
                     (good_b, torch.zeros((3, 1), dtype=torch.float32).expand(3, 16)),   # C rows overlap
                     (good_b[:, :8].expand(8, 8)[:, :8].as_strided((8, 8), (0, 1)), torch.zeros((3, 8), dtype=torch.float32))]:
            with pytest.raises(ValueError):
                check(b, c)
        with pytest.raises(binding.VbrError):            # not uploaded
            check(good_b, good_c, dev=None)
        if torch.cuda.is_available():
            with pytest.raises(ValueError):              # uploaded elsewhere than where B and C live
                check(good_b, good_c, dev=torch.empty(1, dtype=torch.uint8, device="cuda:0"))
    # through the public methods: shape errors surface before the state error
    with pytest.raises(ValueError):
        v.spmm(torch.zeros((4, 16), dtype=torch.float16))
    with pytest.raises(binding.VbrError):
        v.spmm(torch.zeros((8, 16), dtype=torch.float16))
    with pytest.raises(ValueError):
        h.spmm(torch.zeros((8, 16), dtype=torch.float16), torch.zeros((9, 16), dtype=torch.float32))


def test_launch_plan_lists_what_a_call_issues():
    # one-slab groups only: one launch of the one-slab tile kernel, 8 tiles x ceil(N / 256) column tiles
    rng = np.random.default_rng(3)
    csr = random_csr(rng, 128, 64, 0.2)
    v = binding.vbr_build(csr, np.arange(128, dtype=np.int32), np.arange(0, 129, 16, dtype=np.int32), 16)
    plan = v.launches(4096)
    assert [p["kernel"] for p in plan] == ["vbr_spmm_kernel<1 slab>"] and plan[0]["tiles"] == 8
    assert plan[0]["workgroups"] == 8 * 16
    assert v.launches(0) == []
    # groups of 16 and of 100 rows: two classes, few tiles -> one mixed launch, which also takes the
    # column-gathered slab the 12 rows left over (a low group) form
    v = binding.vbr_build(csr, np.arange(128, dtype=np.int32), np.array([0, 16, 116, 128], dtype=np.int32), 16)
    plan = v.launches(256)
    assert [p["kernel"] for p in plan] == ["vbr_spmm_mixed_kernel"] and plan[0]["tiles"] == 3
    # thousands of single-row groups over 4 column blocks, every row touching most of them: one
    # panel per 128 rows shares the few B rows there are; the same number of rows with one entry
    # each over many columns: column-gathered slabs, 16 rows each
    big = random_csr(rng, 6000, 64, 0.2)
    v = binding.vbr_build(big, np.arange(6000, dtype=np.int32), np.arange(0, 6001, dtype=np.int32), 16)
    plan = v.launches(256)
    assert [p["kernel"] for p in plan] == ["vbr_spmm_panel_kernel"] and plan[0]["tiles"] == (6000 + 127) // 128
    wide = csr_from_rows([[int(c)] for c in rng.integers(0, 16384, size=6000)], n_cols=16384)
    v = binding.vbr_build(wide, np.arange(6000, dtype=np.int32), np.arange(0, 6001, dtype=np.int32), 16)
    plan = v.launches(256)
    assert [p["kernel"] for p in plan] == ["vbr_spmm_kernel<1 slab, column-gathered>"] and plan[0]["tiles"] == 6000 // 16
    v.audit()


@pytest.mark.parametrize("n_cols", [504, 512, 520, 1016, 1032])
@pytest.mark.parametrize("used", [31, 32, 33, 64])
@pytest.mark.parametrize("last", [True, False])
def test_columns_of_gathered_tiles_found_by_sorting_and_by_marks(n_cols, used, last):
    # a slab of single-row groups, sixteen times whose K-steps are fewer columns than the matrix has, as many, or more; lists that end with a K-step and that do not
    rng = np.random.default_rng(n_cols + used)
    cols = np.arange(n_cols - used, n_cols) if last else np.sort(rng.choice(n_cols, size=used, replace=False))
    rows = [cols[i::16].tolist() for i in range(15)] + [cols[[0, -1]].tolist()]
    csr = csr_from_rows([sorted(set(r) | set(cols[15::16].tolist())) if i == 3 else r for i, r in enumerate(rows)], n_cols)
    perm, rg = np.arange(16, dtype=np.int32), np.arange(17, dtype=np.int32)
    assert_same_index(csr, perm, rg, 8)
    v = binding.vbr_build(csr, perm, rg, 8)
    assert [p["kernel"] for p in v.launches(256)] == ["vbr_spmm_kernel<1 slab, column-gathered>"]
    v.audit()


@pytest.mark.parametrize("dense_rows,panels", [(128 * 10, False), (128 * 24, True)])
def test_a_few_panels_are_not_worth_a_launch_of_their_own(dense_rows, panels):
    # single-row groups over the same 6 column blocks, whose panels need fewer loads than tiles, among rows of two entries anywhere
    rng = np.random.default_rng(8)
    cols = np.concatenate([np.arange(b * 16, b * 16 + 16) for b in (3, 70, 200, 511, 800, 1023)])
    rows = [rng.choice(cols, size=40, replace=False).tolist() for _ in range(dense_rows)]
    rows += [rng.integers(0, 16384, size=2).tolist() for _ in range(6144 - dense_rows)]
    v = binding.vbr_build(csr_from_rows(rows, 16384), np.arange(6144, dtype=np.int32), np.arange(6145, dtype=np.int32), 16)
    v.audit()
    plan = v.launches(256)
    assert (plan[0]["kernel"] == "vbr_spmm_panel_kernel") == panels and len(plan) == 1 + panels


def test_a_matrix_kept_as_entry_rows_reports_its_rows_and_no_tiles():
    csr = csr_from_rows([[int(c)] for c in np.random.default_rng(2).integers(0, 16384, size=9000)], n_cols=16384)
    v = binding.vbr_build(csr, np.arange(9000, dtype=np.int32), np.arange(9001, dtype=np.int32), 16)
    assert [(p["kernel"], p["tiles"]) for p in v.launches(256)] == [("entry_rows_kernel", 9000)]
    assert v.schedule()["n_tiles"] == 9000 and v.schedule()["n_ksteps"] == 0
    assert v.tile_ksteps().size == 0
    kinds, n = np.zeros(3, dtype=np.int32), ctypes.c_int32()
    assert binding._lib.vbr_get_launches(v._h, 256, ctypes.byref(n), kinds.ctypes.data_as(ctypes.c_void_p), None, None) == 0
    assert n.value == 1 and kinds[0] == 10               # a code no other kernel ever had


@pytest.mark.parametrize("n_cols", [65536, 65552])
def test_blocks_of_a_matrix_kept_as_entry_rows_unpack_from_entries_of_one_and_of_two_words(n_cols):
    rng = np.random.default_rng(n_cols)
    rows = [sorted({int(c), int(c) | 15, n_cols - 1}) for c in rng.integers(0, n_cols, size=9000)]
    csr = csr_from_rows(rows, n_cols, rng)
    v = binding.vbr_build(csr, np.arange(9000, dtype=np.int32), np.arange(9001, dtype=np.int32), 16)
    assert [p["kernel"] for p in v.launches(256)] == ["entry_rows_kernel"]
    v.audit()
    ix = v.index()
    for row in [0, 1, 4999, 8999]:
        p0, p1 = csr["row_ptr"][row], csr["row_ptr"][row + 1]
        dense = np.zeros(n_cols, dtype=np.uint16)
        dense[csr["col_idx"][p0:p1]] = csr["vals"][p0:p1]
        for b in range(ix["blk_ptr"][row], ix["blk_ptr"][row + 1]):
            c0 = int(ix["blk_col"][b]) * 16
            assert np.array_equal(np.asarray(v.unpack_block(int(b), 1, 16)).ravel(), dense[c0:c0 + 16])


def full_csr(n_rows, n_cols):
    """Every entry stored: for plans, which look at the pattern alone."""
    return dict(n_rows=n_rows, n_cols=n_cols, nnz=n_rows * n_cols, row_ptr=np.arange(n_rows + 1, dtype=np.int64) * n_cols,
                col_idx=np.tile(np.arange(n_cols, dtype=np.int32), n_rows), vals=np.full(n_rows * n_cols, 0x3c00, dtype=np.uint16), dtype="f16")


@pytest.mark.parametrize("height,n,most", [(16, 256, 300), (32, 256, 208), (64, 256, 128), (50, 256, 128), (16, 248, 200), (32, 248, 150), (64, 248, 128),
                                           (64, 512, 64), (64, 576, 32), (64, 64, 512), (64, 128, 256), (64, 72, 256), (32, 192, 238), (32, 640, 64), (16, 640, 92)])
def test_launches_are_split_up_to_a_number_of_workgroups_that_falls_with_the_height_of_the_tiles(height, n, most):
    # block tiles of 12 K-steps: a workgroup for every 64 columns up to that number of tiles (64 of these four-slab workgroups fit on
    # an L2 domain, and the busiest counts), one for every 256 beyond
    for groups, split in ((most, True), (most + 1, False)):
        csr = full_csr(height * groups, 384)
        v = binding.vbr_build(csr, np.arange(height * groups, dtype=np.int32), np.arange(0, height * groups + 1, height, dtype=np.int32), 32)
        plan = v.launches(n)
        domains = lambda q: 8 * groups * -(-q // 8) if q >= 8 else 8 * -(-groups // (8 // q))
        assert [p["workgroups"] for p in plan] == [domains(-(-n // 64) if split else -(-n // 256))], (groups, plan)


@pytest.mark.parametrize("n_ks,height,n,most", [(4, 16, 512, 64), (11, 32, 512, 64), (4, 64, 256, 128), (11, 64, 576, 32), (8, 16, 72, 256), (3, 16, 512, 0)])
def test_launches_of_short_lists_are_split_while_two_workgroups_on_a_cu_hold_them(n_ks, height, n, most):
    for groups, split in ((max(most, 1), most > 0), (most + 1, False)):
        csr = full_csr(height * groups, 32 * n_ks)
        v = binding.vbr_build(csr, np.arange(height * groups, dtype=np.int32), np.arange(0, height * groups + 1, height, dtype=np.int32), 32)
        plan = v.launches(n)
        domains = lambda q: 8 * groups * -(-q // 8) if q >= 8 else 8 * -(-groups // (8 // q))
        assert [p["workgroups"] for p in plan] == [domains(-(-n // 64) if split else -(-n // 256))], (groups, plan)


@pytest.mark.parametrize("n,most", [(80, 256), (256, 128), (264, 64)])
def test_mixed_launches_are_split_by_the_workgroups_that_have_columns(n, most):
    # the same with tiles of two heights in one launch, four workgroups a column tile, of which those beyond the last column end at once
    for groups, split in ((most, True), (most + 1, False)):
        rg = np.concatenate([[0], [16], 16 + 64 * np.arange(1, groups)]).astype(np.int32)
        v = binding.vbr_build(full_csr(int(rg[-1]), 384), np.arange(rg[-1], dtype=np.int32), rg, 32)
        plan = v.launches(n)
        assert len(plan) == 1 and plan[0]["kernel"] == "vbr_spmm_mixed_kernel"
        assert (plan[0]["workgroups"] > 2 * groups * -(-n // 256)) == split, (groups, plan)


@pytest.mark.parametrize("height,n,long_groups,split", [(64, 248, 65, True), (64, 248, 90, False), (32, 256, 146, True), (32, 256, 147, False)])
def test_tiles_of_short_lists_hardly_count_for_the_split(height, n, long_groups, split):
    # tiles of 12 K-steps among 250 of 32 rows and one K-step
    rows = long_groups * height + 250 * 32
    lens = np.where(np.arange(rows) < long_groups * height, 384, 32)
    row_ptr = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    col = (np.arange(row_ptr[-1]) - np.repeat(row_ptr[:-1], lens)).astype(np.int32)
    csr = dict(n_rows=rows, n_cols=384, nnz=int(row_ptr[-1]), row_ptr=row_ptr, col_idx=col, vals=np.full(col.size, 0x3c00, dtype=np.uint16), dtype="f16")
    rg = np.concatenate([height * np.arange(long_groups + 1), height * long_groups + 32 * np.arange(1, 251)]).astype(np.int32)
    plan = binding.vbr_build(csr, np.arange(rows, dtype=np.int32), rg, 32).launches(n)
    tiles = long_groups + 250
    assert len(plan) == 1 and (plan[0]["workgroups"] >= 3 * tiles if split else plan[0]["workgroups"] <= tiles + 8), plan


@pytest.mark.parametrize("n_cols,entry_bytes", [(65536, 4), (65537, 8)])
def test_a_matrix_kept_as_entries_reports_its_entries_and_holds_no_more(n_cols, entry_bytes):
    rows, each = 9000, 6
    cols = np.sort((np.arange(rows * each) * 7919 % n_cols).reshape(rows, each), axis=1).astype(np.int32)
    csr = dict(n_rows=rows, n_cols=n_cols, nnz=rows * each, row_ptr=np.arange(rows + 1, dtype=np.int64) * each, col_idx=cols.reshape(-1),
               vals=np.full(rows * each, 0x3c00, dtype=np.uint16), dtype="f16")
    v = binding.vbr_build(csr, np.arange(rows, dtype=np.int32), np.arange(rows + 1, dtype=np.int32), 1)
    v.audit()
    assert [p["kernel"] for p in v.launches(256)] == ["entry_rows_kernel"]
    assert v.schedule() == dict(n_tiles=rows, n_ksteps=0, packed_elems=rows * each)
    # the entries, 16 bytes a row, the permutation; sections begin at multiples of 256 bytes
    held = rows * each * entry_bytes + rows * (16 + 4)
    assert held <= v.device_bytes() <= held + 10 * 256


@pytest.mark.parametrize("height,groups,n_ks,n,function", [(64, 128, 5, 1920, "vbr_spmm_wide_kernel"), (64, 128, 5, 1024, "vbr_spmm_kernel"), (64, 43, 10, 5632, "vbr_spmm_wide_kernel"),
                                                           (64, 10, 12, 256, "vbr_spmm_split_kernel"), (32, 300, 5, 1920, "vbr_spmm_kernel"), (16, 10, 12, 256, "vbr_spmm_split_kernel")])
def test_launches_name_the_function_that_runs(height, groups, n_ks, n, function):
    csr = full_csr(height * groups, 32 * n_ks)
    v = binding.vbr_build(csr, np.arange(height * groups, dtype=np.int32), np.arange(0, height * groups + 1, height, dtype=np.int32), 32)
    columns = {"vbr_spmm_wide_kernel": 512, "vbr_spmm_kernel": 256, "vbr_spmm_split_kernel": 64}[function]
    plan = v.launches(n)
    assert [(p["kernel"], p["function"]) for p in plan] == [("vbr_spmm_kernel<%d slab%s>" % (height // 16, "s" * (height > 16)), function)]
    whole = groups * -(-n // columns)              # and the grid is rounded up for the domains
    assert whole <= plan[0]["workgroups"] < 1.6 * whole + 8


def test_launches_are_not_split_where_a_tile_that_cannot_be_takes_longest():
    csr = csr_from_rows([list(range(416))] * 180, 416)
    rg = np.array([0, 100, 120, 140, 160, 180], dtype=np.int32)         # one group of seven slabs, four of two
    v = binding.vbr_build(csr, np.arange(180, dtype=np.int32), rg, 32)
    assert [(p["tiles"], p["workgroups"]) for p in v.launches(256)] == [(5, 8)]


def mixed_heights_and_empty_rows(tiles, n_ks, empty):
    """Row groups of 16 and 128 rows that hold n_ks K-steps of 32 columns, then rows without entries."""
    heights = [128] * 10 + [16] * (tiles - 10)
    full = full_csr(sum(heights), 32 * n_ks)
    csr = dict(full, n_rows=full["n_rows"] + empty, row_ptr=np.concatenate([full["row_ptr"], np.full(empty, full["nnz"], dtype=np.int64)]))
    rg = np.cumsum([0] + heights + ([empty] if empty else [])).astype(np.int32)
    return binding.vbr_build(csr, np.arange(csr["n_rows"], dtype=np.int32), rg, 32)


@pytest.mark.parametrize("tiles,n,split", [(66, 2048, 2), (80, 2048, 16), (81, 2048, 0), (64, 2048, 0), (258, 512, 4), (130, 768, 2), (100, 1280, 2), (97, 1536, 15)])
@pytest.mark.parametrize("empty_tiles", [0, 20])
def test_the_last_tiles_are_split_by_the_tiles_with_entries_on_a_domain(tiles, n, split, empty_tiles):
    # 64 workgroups of such tiles at once on a domain; of eight, two, three, and five and six column tiles, which the domains share; tiles
    # without a K-step run behind the others and do not count
    v = mixed_heights_and_empty_rows(tiles, 4, 64 * empty_tiles)
    plan = v.launches(n)
    q, t = n // 256, tiles + empty_tiles + 3 * split
    whole = {8: t, 2: -(-t // 4), 3: -(-t // 2), 5: 5 * -(-t // 8), 6: 3 * -(-t // 4)}[q]
    assert [(p["kernel"], p["tiles"], p["workgroups"]) for p in plan] == [("vbr_spmm_mixed_kernel", tiles + empty_tiles, 8 * whole)]


@pytest.mark.parametrize("height,col_block,tiles,n_ks,n,empty,kernels", [
    (16, 32, 128, 16, 4096, 2048, ["vbr_spmm_kernel<1 slab>"]), (32, 32, 128, 16, 4096, 2048, ["vbr_spmm_kernel<2 slabs>"]), (16, 32, 600, 3, 512, 1, ["vbr_spmm_kernel<1 slab>"]),
    (16, 4, 512, 3, 1024, 900, ["vbr_spmm_kernel<1 slab, column-gathered>"]), (30, 4, 300, 3, 1024, 9000, ["vbr_spmm_kernel<2 slabs, column-gathered>"]),
    (60, 4, 100, 3, 4096, 1700, ["vbr_spmm_kernel<4 slabs, column-gathered>"]),
    # taller ones run as well in the mixed kernel, and those that are split run in it as they did; lists of one K-step keep their routes
    (64, 32, 100, 3, 8192, 1700, ["vbr_spmm_mixed_kernel"]), (128, 32, 64, 3, 8192, 1100, ["vbr_spmm_mixed_kernel"]), (16, 32, 60, 16, 256, 64, ["vbr_spmm_mixed_kernel"]),
    (16, 32, 128, 1, 4096, 1900, ["vbr_spmm_mixed_kernel"]), (16, 32, 140, 1, 4096, 2048, ["vbr_spmm_kernel<1 slab>", "vbr_spmm_zero_rows_kernel"])])
def test_one_class_of_low_tiles_keeps_its_kernel_beside_tiles_without_entries(height, col_block, tiles, n_ks, n, empty, kernels):
    cols = 32 * n_ks // col_block * col_block
    full = full_csr(height * tiles, cols)
    csr = dict(full, n_rows=full["n_rows"] + empty, row_ptr=np.concatenate([full["row_ptr"], np.full(empty, full["nnz"], dtype=np.int64)]))
    rg = np.append(height * np.arange(tiles + 1), height * tiles + empty).astype(np.int32)
    v = binding.vbr_build(csr, np.arange(csr["n_rows"], dtype=np.int32), rg, col_block)
    v.audit()
    plan = v.launches(n)
    assert [p["kernel"] for p in plan] == kernels and sum(p["tiles"] for p in plan) == tiles + -(-empty // 64)


def test_the_loop_of_one_slab_tiles_with_deep_rings_begins_on_a_fetch_boundary(tmp_path):
    # of the built library's own kernels: the innermost loop around the products, 32-byte pieces
    objdump = "/opt/rocm/llvm/bin/llvm-objdump"
    if not os.path.exists(objdump):
        pytest.skip("no llvm-objdump")
    lib = shutil.copy(binding.LIB_PATH, tmp_path)
    subprocess.run([objdump, "--offloading", lib], cwd=tmp_path, check=True, stdout=subprocess.DEVNULL)
    found = 0
    for part in sorted(tmp_path.glob("*gfx950*")):
        text = subprocess.run([objdump, "-d", str(part)], check=True, capture_output=True, text=True).stdout
        for name, body in re.findall(r"^[0-9a-f]+ <(\S*15vbr_spmm_kernelILi[01]ELi1ELi4E\S*)>:\n((?:.+\n)+)", text, re.M):
            code = [(int(m.group(2), 16), m.group(1), line) for line in body.splitlines() for m in [re.match(r"\s*(\S+).*// ([0-9A-F]+):", line)] if m]
            products = [address for address, op, _ in code if "mfma" in op]
            begins = []
            for address, op, line in code:
                to = re.search(r"\+0x([0-9a-f]+)>", line) if op.startswith(("s_branch", "s_cbranch")) else None
                begin = code[0][0] + int(to.group(1), 16) if to else address + 1
                if any(begin <= x <= address for x in products):
                    begins.append(begin)
            assert max(begins) % 32 == 0, (name, [x % 32 for x in begins])
            found += 1
    assert found == 4


@pytest.mark.parametrize("height,groups,n,domain", [(16, 170, 1352, 129), (16, 170, 1408, 129), (16, 235, 1352, 235), (16, 256, 1288, 256), (16, 235, 1416, 177), (64, 135, 1352, 102), (64, 100, 1352, 100)])
def test_six_column_tiles_with_a_narrow_last_one_are_shared_where_that_saves_a_round(height, groups, n, domain):
    # 128 workgroups of one-slab tiles at once on a domain, 64 of four-slab ones; up to 128 columns in the last
    csr = full_csr(height * groups, 96)
    v = binding.vbr_build(csr, np.arange(height * groups, dtype=np.int32), np.arange(0, height * groups + 1, height, dtype=np.int32), 32)
    assert [p["workgroups"] for p in v.launches(n)] == [8 * domain]


@pytest.mark.parametrize("groups,col_block,blocks,least,most,n", [(64, 16, 6, 1, 6, 0), (65, 16, 40, 1, 40, 0), (127, 32, 30, 1, 2, 0), (128, 64, 30, 30, 30, 8000), (129, 48, 33, 1, 33, 8000),
                                                                  (513, 16, 300, 2, 4, 0), (64, 16, 2000, 1, 1, 0), (70, 16, 900, 700, 900, 8000), (200, 80, 1, 1, 1, 0),
                                                                  (129, 64, 40, 30, 40, 4096), (300, 80, 20, 8, 20, 2552), (520, 48, 24, 10, 20, 1536), (1000, 16, 64, 20, 40, 840)])
def test_schedules_of_one_slab_groups_hold(groups, col_block, blocks, least, most, n):
    # what the audit goes through step by step; lists of one block, of every block, of far apart ones; the last two groups in the row tile behind the others.  n: columns of B
    # that take the schedule, 0: none up to 1024 do (the host check makes it all the same)
    rng = np.random.default_rng(groups + blocks)
    rows = []
    for g in range(groups):
        cols = np.sort(rng.choice(blocks, size=rng.integers(least, most + 1), replace=False))[:, None] * col_block + np.arange(col_block)
        rows += [cols.reshape(-1).tolist()] * 16
    csr = csr_from_rows(rows, blocks * col_block, rng)
    v = binding.vbr_build(csr, rng.permutation(16 * groups).astype(np.int32), (16 * np.arange(groups + 1)).astype(np.int32), col_block)
    v.audit()
    if n:
        assert v.launches(n)[0]["function"] == "vbr_spmm_stream_kernel"
    else:
        assert all(v.launches(k)[0]["function"] != "vbr_spmm_stream_kernel" for k in range(512, 1025, 8))


@pytest.mark.parametrize("groups", [63, 64, 65, 128])
@pytest.mark.parametrize("col_block,blocks", [(16, 1), (16, 2), (32, 1), (48, 1)])
def test_one_slab_groups_of_very_few_columns(groups, col_block, blocks):
    # fewer B rows than a step of the schedules brings
    csr = full_csr(16 * groups, col_block * blocks)
    v = assert_same_index(csr, np.arange(16 * groups, dtype=np.int32), (16 * np.arange(groups + 1)).astype(np.int32), col_block)
    assert v.launches(512)[0]["tiles"] == groups


def test_stream_kernel_waits_for_its_last_products(tmp_path):
    """Its matrix instructions are inline assembly, whose latency the compiler does not see: behind them every other access to an
    accumulator has to find eight wait states, what the compiler itself puts behind such an instruction before its result is read."""
    out = str(tmp_path / "stream.s")
    subprocess.check_call([build.hipcc()] + build.FLAGS + ["--offload-device-only", "-S", "-x", "hip", os.path.join(build.CSRC, "stream_spmm.hip"), "-o", out],
                          stderr=subprocess.DEVNULL)
    products, waited, kernels = 0, True, set()
    for line in open(out):
        head, code = re.match(r"(_Z\w*stream_kernel\w*):", line), line.split(";")[0].strip()
        if head:
            kernels.add(head.group(1))
            waited = True
        elif code.startswith("v_mfma_"):
            products += 1
            waited = False
        elif code.startswith("s_nop") and int(code.split()[1]) >= 7:
            waited = True
        else:
            assert waited or not re.search(r"\ba(\d|\[\d)", code), "%s in %s" % (code, sorted(kernels)[-1])
    # types, stores, groups, column pieces, steps of a turn, K-steps of a step
    assert len(kernels) == 20 and products == 2 * 2 * 8 * 4 * 2 * sum(range(4, 9))


@pytest.mark.parametrize("groups,n,stream", [(64, 4096, False), (128, 2048, False), (256, 4096, True)])
@pytest.mark.parametrize("empty", [0, 10000, 40000])
def test_rows_without_entries_do_not_choose_the_stream_kernel(groups, n, stream, empty):
    # their tiles cost either kernel next to nothing
    csr = full_csr(16 * groups, 768)
    csr = dict(csr, n_rows=16 * groups + empty, row_ptr=np.append(csr["row_ptr"], np.full(empty, csr["nnz"], dtype=np.int64)))
    rg = np.append(16 * np.arange(groups + 1), [csr["n_rows"]] if empty else []).astype(np.int32)
    v = binding.vbr_build(csr, np.arange(csr["n_rows"], dtype=np.int32), rg, 16)
    v.audit()
    assert v.launches(n)[0]["function"] == ("vbr_spmm_stream_kernel" if stream else "vbr_spmm_kernel")


@pytest.mark.parametrize("groups,blocks,used,n,stream", [(1536, 81, 14, 512, False), (1536, 81, 16, 512, False), (1472, 81, 16, 512, True), (1536, 81, 20, 512, True)])
def test_many_row_tiles_have_to_be_clearly_faster_in_the_stream_kernel(groups, blocks, used, n, stream):
    # 24 row tiles of 64 groups and more, and one less
    rng = np.random.default_rng(groups)
    cols = [(np.sort(rng.choice(blocks, size=used, replace=False))[:, None] * 32 + np.arange(32)).reshape(-1) for _ in range(groups)]
    nnz = 16 * 32 * used * groups
    csr = dict(n_rows=16 * groups, n_cols=32 * blocks, nnz=nnz, row_ptr=np.arange(16 * groups + 1, dtype=np.int64) * (32 * used),
               col_idx=np.concatenate([np.tile(c, 16) for c in cols]).astype(np.int32), vals=np.full(nnz, 0x3c00, dtype=np.uint16), dtype="f16")
    v = binding.vbr_build(csr, np.arange(16 * groups, dtype=np.int32), (16 * np.arange(groups + 1)).astype(np.int32), 32)
    v.audit()
    assert v.launches(n)[0]["function"] == ("vbr_spmm_stream_kernel" if stream else "vbr_spmm_kernel")
