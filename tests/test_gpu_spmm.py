"""GPU parity: the HIP path through the C ABI against the CPU oracle on the same seeded inputs.

Bar: perm, row_groups and the VBR index arrays bit-exact; |C - C_ref| <= 1e-4 * sum_k |a_ik||b_kj|
elementwise (C_ref and the bound in binary64 from the original CSR).  Every case, the full-size
workloads included, is compared element by element.
"""
import numpy as np
import pytest

import oracle
from paper_2202_05868_amd import binding, synth, torch_io
from helpers import csr_from_rows, random_csr

pytestmark = pytest.mark.gpu
TOL = 1e-4


def gpu_spmm(csr, perm, rg, col_block, b_bits, ldb_pad=0, ldc_pad=0):
    import torch
    v = binding.vbr_build(csr, perm, rg, col_block)
    v.audit()                       # bounds of everything the kernels index, before anything is launched
    v.upload("cuda:0")
    k, n = b_bits.shape
    if ldb_pad:
        full = np.zeros((k, n + ldb_pad), dtype=np.uint16)
        full[:, :n] = b_bits
        b = torch_io.bits_to_device(full, csr["dtype"])[:, :n]
    else:
        b = torch_io.bits_to_device(b_bits, csr["dtype"])
    c_full = torch.full((csr["n_rows"], n + ldc_pad), float("nan"), dtype=torch.float32, device="cuda:0")
    c = c_full[:, :n]
    v.spmm(b, c)
    torch.cuda.synchronize()
    out = c_full.cpu().numpy()
    if ldc_pad:
        assert np.isnan(out[:, n:]).all(), "wrote outside the N columns"
    return out[:, :n].astype(np.float64), v


def check_c(c, c_ref, s, what=""):
    assert not np.isnan(c).any(), what + ": NaN left in C (rows not written)"
    err = np.abs(c - c_ref)
    bad = err > TOL * s
    assert not bad.any(), "%s: %d elements outside the bound, worst err/bound %.3g" % (
        what, int(bad.sum()), float(np.max(err / np.maximum(s, 1e-300))))


def blocking_bit_exact(csr, col_block, tau):
    p0, g0 = oracle.sa1(csr, col_block, tau)
    perm, rg = binding.sa1_reorder(csr, col_block, tau)
    assert np.array_equal(perm, p0) and np.array_equal(rg, g0)
    return perm, rg


def index_bit_exact(v, csr, perm, rg, col_block):
    bp, bc, bo = oracle.vbr_index(csr, perm, rg, col_block)
    ix = v.index()
    assert np.array_equal(ix["blk_ptr"], bp) and np.array_equal(ix["blk_col"], bc) and np.array_equal(ix["blk_off"], bo)


# --------------------------------------------------------------------------- small, element by element
@pytest.mark.parametrize("col_block", [1, 3, 8, 16, 32, 64])
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_random_matrices_all_column_block_widths(col_block, dtype):
    rng = np.random.default_rng(col_block * 7 + (dtype == "bf16"))
    for m, kb, n, dens, tau in [(70, 9, 64, 0.2, 0.4), (300, 5, 264, 0.05, 0.2), (33, 12, 8, 0.6, 0.7)]:
        csr = random_csr(rng, m, kb * col_block, dens, dtype=dtype)
        b = synth.dense_rhs(rng, kb * col_block, n, dtype)
        perm, rg = blocking_bit_exact(csr, col_block, tau)
        c, v = gpu_spmm(csr, perm, rg, col_block, b)
        index_bit_exact(v, csr, perm, rg, col_block)
        c_ref, s = oracle.spmm(csr, b)
        check_c(c, c_ref, s, "cb=%d %s m=%d n=%d" % (col_block, dtype, m, n))


def test_result_does_not_depend_on_the_row_partition_used():
    rng = np.random.default_rng(5)
    csr = random_csr(rng, 500, 256, 0.04)
    b = synth.dense_rhs(rng, 256, 520, "f16")           # 520: two full column tiles + ragged tail
    c_ref, s = oracle.spmm(csr, b)
    ident = (np.arange(500, dtype=np.int32), np.arange(501, dtype=np.int32))          # every row its own group
    one = (np.arange(500, dtype=np.int32), np.array([0, 500], dtype=np.int32))        # one group of 500 rows
    rnd = (rng.permutation(500).astype(np.int32), np.array([0, 1, 18, 150, 151, 300, 500], dtype=np.int32))
    sa = blocking_bit_exact(csr, 16, 0.3)
    for name, (perm, rg) in [("identity", ident), ("one group", one), ("random", rnd), ("1-SA", sa)]:
        c, v = gpu_spmm(csr, perm, rg, 16, b)
        index_bit_exact(v, csr, perm, rg, 16)
        check_c(c, c_ref, s, name)


def test_short_groups_in_panels():
    # more than 4096 rows in groups shorter than a slab: the panel kernel; few column blocks at
    # high density make nearly every slab present in every K-step (full masks)
    rng = np.random.default_rng(12)
    csr = random_csr(rng, 6000, 12 * 8, 0.08)
    b = synth.dense_rhs(rng, 96, 136, "f16")            # one full 128-column tile + a ragged one
    perm, rg = blocking_bit_exact(csr, 8, 0.9)
    h = np.diff(rg)
    assert h[h < 16].sum() >= 4096                       # enough short rows for panels to be used
    c, v = gpu_spmm(csr, perm, rg, 8, b)
    index_bit_exact(v, csr, perm, rg, 8)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "panels")
    # tall and short groups in one matrix: tiles and panels side by side
    csr = random_csr(rng, 5000, 256, 0.02, dtype="bf16")
    b = synth.dense_rhs(rng, 256, 264, "bf16")
    perm = rng.permutation(5000).astype(np.int32)
    # heights 3, 16, 181, 16, 1, 283, then 4500 rows in groups of 9 (short: they form the panels)
    rg = np.concatenate([[0, 3, 19, 200, 216, 217, 500], np.arange(509, 5001, 9)]).astype(np.int32)
    assert rg[-1] == 5000
    c, v = gpu_spmm(csr, perm, rg, 32, b)
    index_bit_exact(v, csr, perm, rg, 32)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "tiles and panels mixed")


def test_low_rows_packed_both_ways_in_one_matrix():
    # 3072 single-row groups that all touch the same 6 column blocks (one shared panel per 128 rows
    # needs fewest loads), then 3072 rows with two entries each anywhere in 16384 columns (slabs that
    # gather their own columns do), then one tall group: three kernels in one call; the low groups
    # are handed over in scrambled order, so the packing's own ordering of them is at work too
    rng = np.random.default_rng(91)
    n_cols, cb = 16384, 16
    dense_cols = np.concatenate([np.arange(b * cb, (b + 1) * cb) for b in (3, 70, 200, 511, 800, 1023)])
    rows = [sorted(rng.choice(dense_cols, size=40, replace=False).tolist()) for _ in range(3072)]
    rows += [sorted(set(rng.integers(0, n_cols, size=2).tolist())) for _ in range(3072)]
    rows += [sorted(rng.choice(n_cols, size=30, replace=False).tolist()) for _ in range(40)]
    csr = csr_from_rows(rows, n_cols=n_cols, rng=rng)
    m = len(rows)
    low = rng.permutation(6144).astype(np.int32)
    perm = np.concatenate([low, np.arange(6144, m, dtype=np.int32)])
    rg = np.concatenate([np.arange(0, 6145), [m]]).astype(np.int32)
    b = synth.dense_rhs(rng, n_cols, 264, "f16")
    c, v = gpu_spmm(csr, perm, rg, cb, b, ldb_pad=8, ldc_pad=4)
    plan = v.launches(264)
    # some twenty panels, then one launch with the ~200 gathered slabs and the tile of the tall group
    assert plan[0]["kernel"] == "vbr_spmm_panel_kernel" and plan[0]["tiles"] >= 16
    assert len(plan) == 2 and plan[1]["kernel"] == "vbr_spmm_mixed_kernel" and plan[1]["tiles"] >= 150
    index_bit_exact(v, csr, perm, rg, cb)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "panels and gathered slabs")
    ix = v.index()
    for blk in rng.choice(ix["n_blocks"], size=300, replace=False):
        g = int(np.searchsorted(ix["blk_ptr"], blk, side="right") - 1)
        assert np.array_equal(v.unpack_block(int(blk), int(rg[g + 1] - rg[g]), cb),
                              oracle.block_bits(csr, perm, rg, g, int(ix["blk_col"][blk]), cb))


@pytest.mark.parametrize("n,rows_of_hubs,ldb_pad,dtype", [(8, 1, 0, "f16"), (72, 17, 8, "bf16"), (256, 32, 0, "f16"), (1096, 40, 0, "f16")])
def test_tiles_with_long_column_lists_split_their_k_steps(n, rows_of_hubs, ldb_pad, dtype):
    # a few rows with thousands of columns among 1100 short ones: their tiles (one slab, a partial second one)
    # are split over the waves of a workgroup, 64 columns of C each; N below, at and past the 64- and 256-column tiles
    rng = np.random.default_rng(n)
    k = 4800
    lens = [4700 - 37 * i for i in range(rows_of_hubs)] + [int(x) for x in rng.integers(0, 6, size=1100)]
    csr = csr_from_rows([sorted(rng.choice(k, size=x, replace=False).tolist()) for x in lens], k, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, k, n, dtype)
    perm = rng.permutation(len(lens)).astype(np.int32)
    rg = np.arange(len(lens) + 1, dtype=np.int32)
    c, v = gpu_spmm(csr, perm, rg, 16, bits, ldb_pad=ldb_pad, ldc_pad=4)
    assert v.tile_ksteps().max() >= 128
    index_bit_exact(v, csr, perm, rg, 16)
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "hub rows, n=%d" % n)


@pytest.mark.parametrize("n,ldb_pad,dtype", [(1024, 0, "f16"), (1032, 8, "bf16"), (1416, 0, "f16"), (1544, 0, "f16"), (2056, 0, "bf16"), (2568, 0, "f16")])
def test_tiles_with_long_column_lists_among_more_workgroups_than_are_resident(n, ldb_pad, dtype):
    # the same beside 293 tiles of one and two slabs: the rings of launches of up to six and nine to twelve column tiles, and of others
    rng = np.random.default_rng(n)
    k, hubs = 4800, 40
    heights = [17, 16, 20] * 97 + [17, 16]
    rows = [sorted(rng.choice(k, size=4700 - 37 * i, replace=False).tolist()) for i in range(hubs)]
    for g, h in enumerate(heights):
        blocks = np.sort(rng.choice(k // 32, size=1 + g % 3, replace=False))
        rows += [(blocks[:, None] * 32 + np.arange(32)).reshape(-1).tolist()] * h
    csr = csr_from_rows(rows, k, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, k, n, dtype)
    perm, rg = np.arange(len(rows), dtype=np.int32), np.cumsum([0] + [1] * hubs + heights).astype(np.int32)
    c, v = gpu_spmm(csr, perm, rg, 32, bits, ldb_pad=ldb_pad)
    assert [p["kernel"] for p in v.launches(n)] == ["vbr_spmm_mixed_kernel"] and v.tile_ksteps().max() >= 128
    assert v.launches(n)[0]["tiles"] * ((n + 255) // 256) > 1536
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "hub rows among blocks, n=%d" % n)


@pytest.mark.parametrize("n,ldb_pad,dtype", [(8, 0, "f16"), (64, 64, "bf16"), (248, 0, "f16"), (256, 0, "f16"), (1032, 8, "bf16")])
def test_large_matrix_that_shares_nothing_is_multiplied_entry_by_entry(n, ldb_pad, dtype):
    # 8200 rows of 0 to 30 entries anywhere, some of 300 and one of 1500 (a wave, a workgroup for a row)
    rng = np.random.default_rng(n)
    k = 6400
    lens = rng.integers(0, 31, size=8200)
    lens[[5, 77, 4000]], lens[8100] = 300, 1500
    csr = csr_from_rows([sorted(rng.choice(k, size=int(x), replace=False).tolist()) for x in lens], k, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, k, n, dtype)
    perm, rg = rng.permutation(8200).astype(np.int32), np.arange(8201, dtype=np.int32)
    c, v = gpu_spmm(csr, perm, rg, 32, bits, ldb_pad=ldb_pad, ldc_pad=4)
    assert [p["kernel"] for p in v.launches(n)] == ["entry_rows_kernel"]
    index_bit_exact(v, csr, perm, rg, 32)
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "entries, n=%d" % n)
    ix = v.index()
    for blk in rng.choice(ix["n_blocks"], size=100, replace=False):
        g = int(np.searchsorted(ix["blk_ptr"], blk, side="right") - 1)
        assert np.array_equal(v.unpack_block(int(blk), 1, 32), oracle.block_bits(csr, perm, rg, g, int(ix["blk_col"][blk]), 32))


@pytest.mark.parametrize("heights,col_block,n,ldb_pad,dtype", [([16] * 5, 16, 64, 0, "f16"), ([16] * 5, 8, 72, 56, "bf16"), ([27] * 5, 32, 256, 0, "f16"),
                                                               ([32] * 5, 16, 24, 8, "f16"), ([49] * 3, 16, 320, 0, "f16"), ([64] * 3, 8, 64, 0, "bf16"),
                                                               ([16, 40, 3, 64, 23, 9, 100], 16, 320, 0, "f16")])
def test_few_workgroups_with_long_lists_split_their_k_steps(heights, col_block, n, ldb_pad, dtype):
    # groups of one to four slabs, full and partial last ones, every granule width; N below and past 64 columns; then
    # all kinds of tiles in one launch, those of more than four slabs not split
    rng = np.random.default_rng(len(heights) + col_block)
    kb = 1536 // col_block
    rows = []
    for h in heights:
        blocks = rng.choice(kb, size=kb // 2, replace=False)
        cols = np.sort((blocks[:, None] * col_block + np.arange(col_block)).reshape(-1))
        rows += [cols[rng.random(cols.size) < 0.9].tolist() for _ in range(h)]
    csr = csr_from_rows(rows, 1536, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, 1536, n, dtype)
    perm = np.arange(sum(heights), dtype=np.int32)
    rg = np.cumsum([0] + heights).astype(np.int32)
    c, v = gpu_spmm(csr, perm, rg, col_block, bits, ldb_pad=ldb_pad, ldc_pad=4)
    assert len(v.launches(n)) == 1 and v.tile_ksteps().max() >= 12
    index_bit_exact(v, csr, perm, rg, col_block)
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "split K-steps")


@pytest.mark.parametrize("n_ks,n,ldb_pad", [(4, 8, 0), (4, 256, 8), (5, 72, 0), (7, 520, 0), (11, 64, 16)])
@pytest.mark.parametrize("heights,col_block", [([16, 9, 16], 32), ([32, 17, 20], 4), ([64, 33, 50], 8), ([64, 16, 5, 30, 3], 32)])
def test_few_workgroups_with_short_lists_split_their_k_steps(heights, col_block, n_ks, n, ldb_pad):
    # one to four slabs, block tiles and gathered ones, then several classes in one launch: from as many K-steps as a workgroup has
    # waves on up to the last before tiles are split in larger launches too
    rng = np.random.default_rng(n_ks)
    kb = 1024 // col_block
    rows = []
    for h in heights:
        cols = np.sort((rng.choice(kb, size=n_ks * 32 // col_block, replace=False)[:, None] * col_block + np.arange(col_block)).reshape(-1))
        rows += [cols.tolist() for _ in range(h)]
    csr = csr_from_rows(rows, 1024, rng)
    bits = synth.dense_rhs(rng, 1024, n, "f16")
    rg = np.cumsum([0] + heights).astype(np.int32)
    c, v = gpu_spmm(csr, np.arange(len(rows), dtype=np.int32), rg, col_block, bits, ldb_pad=ldb_pad, ldc_pad=4)
    plan = v.launches(n)
    assert len(plan) == 1 and plan[0]["workgroups"] >= plan[0]["tiles"] * -(-n // 64) and v.tile_ksteps().max() >= n_ks
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "short lists")


@pytest.mark.parametrize("heights,col_block,n,dtype,most", [([128] * 10 + [40] * 26 + [16] * 29, 32, 2048, "f16", 64), ([100] * 5 + [30] * 50 + [16] * 14, 32, 1800, "bf16", 64),
                                                            ([64] * 10 + [32, 17] * 24 + [16] * 42, 4, 2040, "f16", 96), ([64] * 50 + [30, 9] * 20 + [16] * 20, 16, 1992, "f16", 96)])
def test_the_last_tiles_of_a_launch_that_does_not_fit_are_split(heights, col_block, n, dtype, most):
    # eight column tiles, one a domain, and a few tiles more than a domain holds at once: the shortest ones, of one and two slabs, block
    # tiles and gathered ones, have four workgroups each; a ragged last column tile, whose last quarters have no columns
    rng = np.random.default_rng(len(heights))
    kb = 512 // col_block
    rows = []
    for i, h in enumerate(heights):
        n_ks = 7 if h > 16 else 4 + i % 3
        cols = np.sort((rng.choice(kb, size=n_ks * 32 // col_block, replace=False)[:, None] * col_block + np.arange(col_block)).reshape(-1))
        rows += [cols.tolist() for _ in range(h)]
    csr = csr_from_rows(rows, 512, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, 512, n, dtype)
    rg = np.cumsum([0] + heights).astype(np.int32)
    c, v = gpu_spmm(csr, np.arange(len(rows), dtype=np.int32), rg, col_block, bits, ldc_pad=4)
    plan = v.launches(n)
    tiles = plan[0]["tiles"]
    assert len(plan) == 1 and plan[0]["kernel"] == "vbr_spmm_mixed_kernel" and most < tiles <= most + most // 4
    assert plan[0]["workgroups"] == 8 * (most + 4 * (tiles - most))
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "the last tiles split")


@pytest.mark.parametrize("tiles,n,split,empty", [(259, 504, 4, 0), (131, 760, 4, 700), (100, 1272, 2, 0), (100, 1280, 2, 640), (97, 1536, 15, 33), (66, 2040, 2, 1000)])
def test_the_last_tiles_are_split_over_fewer_column_tiles_and_before_tiles_without_entries(tiles, n, split, empty):
    # two, three, and five and six column tiles that the domains share; rows without entries behind them, whose tiles have one workgroup
    rng = np.random.default_rng(tiles)
    rows = []
    for t in range(tiles):
        cols = np.sort((rng.choice(16, size=4 + t % 3, replace=False)[:, None] * 32 + np.arange(32)).reshape(-1))
        rows += [cols.tolist() for _ in range(128 if t < 10 else 30 if t % 2 else 16)]
    rg = np.cumsum([0] + [128 if t < 10 else 30 if t % 2 else 16 for t in range(tiles)] + ([empty] if empty else [])).astype(np.int32)
    rows += [[]] * empty
    csr = csr_from_rows(rows, 512, rng)
    order = rng.permutation(len(rows)).astype(np.int32)
    csr = synth.permute_rows(csr, np.argsort(order))
    bits = synth.dense_rhs(rng, 512, n, "f16")
    c, v = gpu_spmm(csr, order, rg, 32, bits, ldc_pad=4)
    plan = v.launches(n)
    q, t = -(-n // 256), tiles + -(-empty // 64) + 3 * split
    domain = {8: t, 2: -(-t // 4), 3: -(-t // 2), 5: 5 * -(-t // 8), 6: 3 * -(-t // 4)}[q]
    assert [(p["kernel"], p["workgroups"]) for p in plan] == [("vbr_spmm_mixed_kernel", 8 * domain)]
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "the last tiles split, %d column tiles" % q)


@pytest.mark.parametrize("n_ks", [5, 6, 8])
@pytest.mark.parametrize("heights,col_block,n", [([32] * 30, 32, 1800), ([16] * 32, 4, 2048), ([32, 20] * 14, 8, 2040), ([64, 100, 16] * 9, 16, 2048), ([30, 9] * 15, 4, 1992)])
def test_lists_about_as_long_as_the_deeper_rings(heights, col_block, n_ks, n):
    # at most one workgroup on a CU and too many to be split: one and two slabs alone, then with four and eight in one launch, block tiles and
    # gathered ones; every third group's list is shorter than the rings
    rng = np.random.default_rng(n_ks)
    kb = 512 // col_block
    rows = []
    for i, h in enumerate(heights):
        ks = n_ks if i % 3 else 1 + i % 4
        cols = np.sort((rng.choice(kb, size=ks * 32 // col_block, replace=False)[:, None] * col_block + np.arange(col_block)).reshape(-1))
        rows += [cols.tolist() for _ in range(h)]
    csr = csr_from_rows(rows, 512, rng)
    bits = synth.dense_rhs(rng, 512, n, "f16")
    rg = np.cumsum([0] + heights).astype(np.int32)
    c, v = gpu_spmm(csr, np.arange(len(rows), dtype=np.int32), rg, col_block, bits, ldc_pad=4)
    plan = v.launches(n)
    assert len(plan) == 1 and plan[0]["workgroups"] <= 256 and v.tile_ksteps().max() >= n_ks
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "deeper rings")


@pytest.mark.parametrize("col_block", [32, 4])
@pytest.mark.parametrize("n_ks,groups,n,dtype", [(1, 5, 264, "f16"), (2, 5, 256, "bf16"), (3, 5, 264, "f16"), (4, 5, 8, "f16"), (7, 5, 264, "bf16"), (26, 131, 1032, "f16")])
def test_two_slab_tiles_at_the_lengths_of_their_rings(col_block, n_ks, groups, n, dtype):
    # block tiles and column-gathered ones of 17 to 32 rows, lists shorter than the rings of B rows and fragments up to long
    # ones in more workgroups than are split or take deeper rings
    rng = np.random.default_rng(n_ks)
    heights = [32, 17, 25, 31, 32] * (groups // 5) + [20] * (groups % 5)
    kb = 1024 // col_block
    rows = []
    for h in heights:
        cols = np.sort((rng.choice(kb, size=n_ks * 32 // col_block, replace=False)[:, None] * col_block + np.arange(col_block)).reshape(-1))
        rows += [cols.tolist() for _ in range(h)]
    csr = csr_from_rows(rows, 1024, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, 1024, n, dtype)
    perm, rg = rng.permutation(len(rows)).astype(np.int32), np.cumsum([0] + heights).astype(np.int32)
    inv = np.argsort(perm)
    csr = synth.permute_rows(csr, inv)               # row perm[i] of the permuted matrix is row i of the groups
    c, v = gpu_spmm(csr, perm, rg, col_block, bits)
    assert [p["kernel"] for p in v.launches(n)] == ["vbr_spmm_kernel<2 slabs%s>" % (", column-gathered" if col_block == 4 else "")]
    assert set(v.tile_ksteps().tolist()) == {n_ks}
    index_bit_exact(v, csr, perm, rg, col_block)
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "two slabs, %d K-steps" % n_ks)


@pytest.mark.parametrize("heights,groups,col_block,n_ks,n,pad,dtype,workgroups", [
    ([33], 128, 32, 4, 2048, 0, "f16", 512), ([64], 128, 16, 5, 1920, 0, "bf16", 512), ([64, 33, 48, 49], 128, 8, 7, 1928, 8, "f16", 512),
    ([50, 64], 128, 24, 6, 1800, 0, "f16", 512), ([40], 128, 64, 6, 1544, 64, "f16", 512), ([35, 64], 126, 40, 9, 2040, 0, "bf16", 504),
    ([33, 41], 192, 16, 4, 2056, 0, "f16", 960), ([61], 64, 32, 11, 4096, 0, "f16", 512)])
def test_long_lists_against_a_wide_b(heights, groups, col_block, n_ks, n, pad, dtype, workgroups):
    # row groups of three and four slabs with full and partial last ones, lists of an even and an odd number of K-steps with and without a partial last one,
    # of one length and (longer than 4) of two; every granule width; the last column tile whole, with waves that have no column, and one that has 8
    rng = np.random.default_rng(n + n_ks)
    n_cols = 40 * 64 if col_block in (40, 64) else 72 * 32
    r, c, row = [], [], 0
    for g in range(groups):
        h, blocks = heights[g % len(heights)], (n_ks - (g % 3 == 1 and n_ks > 4)) * 32 // col_block
        cols = (np.sort(rng.choice(n_cols // col_block, size=blocks, replace=False))[:, None] * col_block + np.arange(col_block)).reshape(-1)
        r.append(np.repeat(np.arange(row, row + h), cols.size))
        c.append(np.tile(cols, h))
        row += h
    r, c = np.concatenate(r), np.concatenate(c)
    csr = synth.csr_from_coo(row, n_cols, r, c, synth.to_bits(rng.uniform(-1, 1, size=r.size).astype(np.float32), dtype), dtype)
    rg = np.cumsum([0] + [heights[g % len(heights)] for g in range(groups)]).astype(np.int32)
    perm = rng.permutation(row).astype(np.int32)
    csr = synth.permute_rows(csr, np.argsort(perm))
    bits = synth.dense_rhs(rng, n_cols, n, dtype)
    out, v = gpu_spmm(csr, perm, rg, col_block, bits, ldb_pad=pad, ldc_pad=pad)
    assert [(p["kernel"], p["workgroups"]) for p in v.launches(n)] == [("vbr_spmm_kernel<4 slabs>", workgroups)]
    c_ref, s = oracle.spmm(csr, bits)
    check_c(out, c_ref, s, "%d K-steps, N = %d" % (n_ks, n))


@pytest.mark.parametrize("groups,col_block,blocks,least,most,empty,n,pad,dtype", [
    (1024, 16, 512, 28, 32, 0, 1024, 0, "f16"), (1024, 16, 512, 36, 40, 0, 1024, 0, "bf16"), (1024, 16, 256, 21, 24, 0, 1024, 64, "f16"), (290, 64, 40, 2, 39, 64, 2040, 0, "bf16"),
    (700, 32, 40, 20, 30, 100, 520, 0, "f16"), (600, 16, 64, 24, 40, 0, 1032, 8, "bf16"), (2048, 16, 32, 14, 18, 0, 512, 0, "f16"), (520, 48, 24, 10, 20, 77, 1032, 0, "f16"),
    (300, 80, 20, 8, 20, 64, 2552, 0, "bf16"), (129, 64, 40, 30, 40, 1, 4096, 0, "f16")])
def test_many_groups_of_one_slab_against_a_wide_b(groups, col_block, blocks, least, most, empty, n, pad, dtype):
    # schedules of four to eight K-steps a step; units of two halves of a block and of one; lists of an even and an odd number of blocks, of one length and of many; the last
    # workgroup with one group, and with waves that have fewer than others; the last column tile of 8, 56 and 64 columns; rows without entries, less than a tile and more
    rng = np.random.default_rng(groups + n)
    r, c = [], []
    for g in range(groups):
        cols = (np.sort(rng.choice(blocks, size=rng.integers(least, most + 1), replace=False))[:, None] * col_block + np.arange(col_block)).reshape(-1)
        r.append(np.repeat(np.arange(16 * g, 16 * g + 16), cols.size))
        c.append(np.tile(cols, 16))
    r, c, rows = np.concatenate(r), np.concatenate(c), 16 * groups + empty
    csr = synth.csr_from_coo(rows, blocks * col_block, r, c, synth.to_bits(rng.uniform(-1, 1, size=r.size).astype(np.float32), dtype), dtype)
    rg = np.append(16 * np.arange(groups + 1), [rows] if empty else []).astype(np.int32)
    perm = rng.permutation(rows).astype(np.int32)
    csr = synth.permute_rows(csr, np.argsort(perm))
    bits = synth.dense_rhs(rng, blocks * col_block, n, dtype)
    out, v = gpu_spmm(csr, perm, rg, col_block, bits, ldb_pad=pad, ldc_pad=pad)
    assert [(p["function"], p["tiles"]) for p in v.launches(n)] == [("vbr_spmm_stream_kernel", groups + -(-empty // 64))]
    c_ref, s = oracle.spmm(csr, bits)
    check_c(out, c_ref, s, "%d groups, N = %d" % (groups, n))
    assert np.all(out[perm[16 * groups:]] == 0.0)


@pytest.mark.parametrize("n,dtype", [(1416, "f16"), (1464, "bf16"), (1472, "f16")])
def test_rows_of_c_that_begin_inside_cache_lines(n, dtype):
    # the stream kernel stores whole lines and parts of lines differently: rows that begin anywhere in a line, at its half, with it; the last column tile of 8, 56 and 64 columns
    import torch
    groups, blocks, k = 512, 128, 64
    rng = np.random.default_rng(n)
    cols = [(np.sort(rng.choice(blocks, size=k, replace=False))[:, None] * 16 + np.arange(16)).reshape(-1) for _ in range(groups)]
    r, c = np.repeat(np.arange(16 * groups), 16 * k), np.concatenate([np.tile(x, 16) for x in cols])
    csr = synth.csr_from_coo(16 * groups, 16 * blocks, r, c, synth.to_bits(rng.uniform(-1, 1, size=r.size).astype(np.float32), dtype), dtype)
    bits = synth.dense_rhs(rng, 16 * blocks, n, dtype)
    c_ref, s = oracle.spmm(csr, bits)
    v = binding.vbr_build(csr, np.arange(16 * groups, dtype=np.int32), (16 * np.arange(groups + 1)).astype(np.int32), 16)
    v.audit()
    assert [p["function"] for p in v.launches(n)] == ["vbr_spmm_stream_kernel"]
    v.upload("cuda:0")
    b = torch_io.bits_to_device(bits, dtype)
    for ldc, shift in [(n, 0), (1472, 0), (1472, 4), (1472, 16), (1488, 0), (1488, 16), (1476, 0), (1484, 8), (1480, 28)]:
        flat = torch.full((16 * groups * ldc + shift,), float("nan"), device="cuda:0")
        assert flat.data_ptr() % 128 == 0
        v.spmm(b, torch.as_strided(flat, (16 * groups, n), (ldc, 1), shift))
        torch.cuda.synchronize()
        out = flat.cpu().numpy()
        rows = out[shift:].reshape(16 * groups, ldc)
        assert np.isnan(out[:shift]).all() and np.isnan(rows[:, n:]).all(), "wrote outside the N columns"
        check_c(rows[:, :n].astype(np.float64), c_ref, s, "N = %d, rows of %d from %d on" % (n, ldc, shift))


@pytest.mark.parametrize("n", [8, 24, 64, 72, 120, 128, 136, 264, 384, 392])
@pytest.mark.parametrize("heights,col_block", [([128, 70, 100], 16), ([128, 70, 40, 18, 33, 16, 3, 9, 2], 16), ([60, 20, 7], 3)])
def test_narrow_column_tiles(heights, col_block, n):
    # the only or the last column tile around the width up to which tall tiles are stored without the way through LDS: block
    # tiles of every height, gathered ones, full and partial slabs, nothing written beside the N columns
    rng = np.random.default_rng(n)
    m = sum(heights)
    csr = random_csr(rng, m, 48 * col_block, 0.1)
    bits = synth.dense_rhs(rng, 48 * col_block, n, "f16")
    perm, rg = rng.permutation(m).astype(np.int32), np.cumsum([0] + heights).astype(np.int32)
    c, v = gpu_spmm(csr, perm, rg, col_block, bits, ldb_pad=8, ldc_pad=12)
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "N = %d" % n)


@pytest.mark.parametrize("tail", [1, 15, 16, 33, 63, 64])
def test_slabs_of_low_rows_that_share_columns_form_taller_tiles(tail):
    # 1024 + tail single-row groups in clusters over the same columns: tiles of 1 to 4 slabs, the last one partial
    rng = np.random.default_rng(tail)
    k, m = 2048, 1024 + tail
    rows = []
    for i in range(m):
        base = 128 * (i // 70 % 16)
        rows.append(sorted(set((base + rng.choice(128, size=50, replace=False)).tolist() + rng.integers(0, k, size=2).tolist())))
    csr = csr_from_rows(rows, k, rng)
    bits = synth.dense_rhs(rng, k, 264, "f16")
    perm, rg = np.arange(m, dtype=np.int32), np.arange(m + 1, dtype=np.int32)
    c, v = gpu_spmm(csr, perm, rg, 4, bits)          # blocks of 4: no panels
    assert v.schedule()["n_tiles"] < m // 32         # most tiles hold more than two slabs
    index_bit_exact(v, csr, perm, rg, 4)
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "taller tiles")


@pytest.mark.parametrize("col_block,n_blocks,density,dtype,n", [(16, 12, 0.03, "f16", 136), (32, 40, 0.01, "bf16", 264),
                                                              (16, 200, 0.004, "f16", 128)])
def test_short_groups_wider_blocks_and_padded_leading_dimensions(col_block, n_blocks, density, dtype, n):
    # thousands of short groups with blocks of 16 and 32 columns (granules of 16 and 32 B rows), few
    # and many column blocks, B and C with padded leading dimensions
    rng = np.random.default_rng(col_block + n_blocks)
    csr = random_csr(rng, 6000, n_blocks * col_block, density, dtype=dtype)
    b = synth.dense_rhs(rng, n_blocks * col_block, n, dtype)
    perm, rg = blocking_bit_exact(csr, col_block, 0.9)
    c, v = gpu_spmm(csr, perm, rg, col_block, b, ldb_pad=8, ldc_pad=4)
    index_bit_exact(v, csr, perm, rg, col_block)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "short groups cb=%d" % col_block)


def test_block_rows_of_exactly_one_slab():
    # the shape of the pruned-weight workload at a size the oracle multiplies whole: 16 x 16 blocks
    # kept at 10 %, every block row is one group of exactly one slab
    rng = np.random.default_rng(31)
    keep = rng.random((256, 64)) < 0.10
    mask = np.kron(keep, np.ones((16, 16), dtype=bool))
    r, cc = np.nonzero(mask)
    vals = synth.to_bits(rng.standard_normal(r.size).astype(np.float32) / 4, "f16")
    csr = synth.csr_from_coo(4096, 1024, r, cc, vals, "f16")
    b = synth.dense_rhs(rng, 1024, 264, "f16", dist="normal")
    perm, rg = blocking_bit_exact(csr, 16, 0.5)
    c, v = gpu_spmm(csr, perm, rg, 16, b)
    index_bit_exact(v, csr, perm, rg, 16)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "block rows of one slab")


@pytest.mark.parametrize("seed", range(16))
def test_random_shapes_partitions_and_widths(seed):
    # random everything: size, block width (fast and slow gather paths), density, dtype, dense
    # width with and without a column tail, padded leading dimensions, and an arbitrary valid row
    # partition with heights from 1 row to several tiles
    rng = np.random.default_rng(1000 + seed)
    col_block = int(rng.choice([1, 2, 4, 5, 8, 12, 16, 24, 32, 48, 64]))
    kb = int(rng.integers(1, 30))
    m = int(rng.integers(1, 700))
    n = 8 * int(rng.integers(1, 80))
    dtype = "bf16" if seed % 2 else "f16"
    csr = random_csr(rng, m, kb * col_block, float(rng.choice([0.01, 0.05, 0.3])), dtype=dtype)
    b = synth.dense_rhs(rng, kb * col_block, n, dtype, dist="normal" if seed % 3 else "uniform")
    cuts = np.unique(np.concatenate([[0, m], rng.integers(0, m + 1, size=int(rng.integers(0, 12)))]))
    if rng.random() < 0.4:                     # plus a run of single-row groups
        lo = int(rng.integers(0, m)); hi = min(m, lo + int(rng.integers(1, 60)))
        cuts = np.unique(np.concatenate([cuts, np.arange(lo, hi + 1)]))
    rg = cuts.astype(np.int32)
    perm = rng.permutation(m).astype(np.int32)
    c, v = gpu_spmm(csr, perm, rg, col_block, b, ldb_pad=8 * int(rng.integers(0, 3)), ldc_pad=4 * int(rng.integers(0, 3)))
    index_bit_exact(v, csr, perm, rg, col_block)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "seed %d cb=%d m=%d n=%d groups=%d" % (seed, col_block, m, n, rg.size - 1))


def test_leading_dimensions_and_overwrite():
    rng = np.random.default_rng(6)
    csr = random_csr(rng, 90, 128, 0.1, dtype="bf16")
    b = synth.dense_rhs(rng, 128, 72, "bf16", dist="normal")
    perm, rg = blocking_bit_exact(csr, 32, 0.5)
    c, _ = gpu_spmm(csr, perm, rg, 32, b, ldb_pad=24, ldc_pad=12)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "padded leading dimensions")


@pytest.mark.parametrize("n", [2048, 2056, 2312, 3592, 4096, 4104])
def test_one_slab_tiles_over_eight_to_seventeen_column_tiles(n):
    # every tile meets every column tile once, however many of these a domain has
    rng = np.random.default_rng(n)
    rows = [[16 * int(b) + i for b in np.sort(rng.choice(40, size=6 + t % 5, replace=False)) for i in range(16)] for t in range(43) for _ in range(16)]
    csr = csr_from_rows(rows, 640, rng)
    bits = synth.dense_rhs(rng, 640, n, "f16")
    c, v = gpu_spmm(csr, np.arange(688, dtype=np.int32), np.arange(0, 689, 16, dtype=np.int32), 16, bits)
    q = -(-n // 256)
    assert [(p["kernel"], p["workgroups"]) for p in v.launches(n)] == [("vbr_spmm_kernel<1 slab>", 8 * {8: 43, 9: 49, 10: 54, 15: 86, 16: 86, 17: 92}[q])]
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "column tiles")


@pytest.mark.parametrize("kind,n,workgroups", [("mixed", 1096, 5 * 10), ("mixed", 1536, 3 * 20), ("mixed", 1408, 77), ("mixed", 1416, 3 * 20), ("mixed", 2304, 77 + 10), ("panel", 640, 5 * 6), ("panel", 1160, 47 + 12),
                                               ("entries", 1216, 563 + 141), ("entries", 1096, 563 + 71)])
def test_column_tiles_that_the_domains_share(kind, n, workgroups):
    # five, six, nine and ten column tiles, not all of them full: mixed tiles, panels and rows of entries
    rng = np.random.default_rng(n)
    if kind == "mixed":
        heights = [64, 30, 9, 16, 33, 48, 16] * 11
        rows = []
        for i, h in enumerate(heights):
            cols = np.sort((rng.choice(24, size=5 + i % 4, replace=False)[:, None] * 32 + np.arange(32)).reshape(-1))
            rows += [cols.tolist() for _ in range(h)]
        csr, rg = csr_from_rows(rows, 768, rng), np.cumsum([0] + heights).astype(np.int32)
    elif kind == "panel":
        csr = random_csr(rng, 6000, 64, 0.2)
        rg = np.arange(6001, dtype=np.int32)
    else:
        csr = csr_from_rows([np.unique(rng.integers(0, 12000, size=1 + i % 5)).tolist() for i in range(9000)], 12000, rng)
        rg = np.arange(9001, dtype=np.int32)
    bits = synth.dense_rhs(rng, csr["n_cols"], n, "f16")
    c, v = gpu_spmm(csr, np.arange(csr["n_rows"], dtype=np.int32), rg, 16 if kind != "mixed" else 32, bits, ldc_pad=4)
    assert v.launches(n)[0]["workgroups"] == 8 * workgroups, v.launches(n)
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "shared column tiles")


@pytest.mark.parametrize("groups,empty,n,kernels", [(70, 1015, 8200, ["vbr_spmm_kernel<1 slab>", "vbr_spmm_zero_rows_kernel"]), (70, 1201, 8200, ["vbr_spmm_mixed_kernel"]),
                                                    (0, 37, 264, ["vbr_spmm_zero_rows_kernel"]), (0, 100, 8, ["vbr_spmm_zero_rows_kernel"])])
def test_tiles_without_entries(groups, empty, n, kernels):
    # in a launch of their own up to a quarter of the others, beyond in the launch of these; nothing but them; the last piece of a row of 8
    # columns, the last rows of a slab and of a tile missing
    rng = np.random.default_rng(empty)
    rows = [[int(16 * (g % 4)) + i for i in range(16)] for g in range(groups) for _ in range(16)] + [[]] * empty
    csr = csr_from_rows(rows, 64, rng)
    bits = synth.dense_rhs(rng, 64, n, "f16")
    rg = np.append(16 * np.arange(groups + 1), 16 * groups + empty).astype(np.int32)
    order = rng.permutation(len(rows)).astype(np.int32)
    csr = synth.permute_rows(csr, np.argsort(order))
    c, v = gpu_spmm(csr, order, rg, 16, bits, ldc_pad=4)
    assert [p["kernel"] for p in v.launches(n)] == kernels
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "tiles without entries")


@pytest.mark.parametrize("height,col_block,tiles,n_ks,n,empty", [(16, 32, 70, 2, 264, 1), (16, 32, 300, 3, 8, 63), (32, 32, 70, 3, 2056, 64), (25, 4, 70, 2, 1032, 65), (16, 4, 70, 3, 520, 200),
                                                                 (16, 32, 40, 20, 1800, 130), (32, 32, 300, 5, 1032, 1500), (60, 4, 40, 3, 1032, 70), (50, 32, 40, 3, 264, 70)])
def test_rows_without_entries_beside_tiles_of_one_class(height, col_block, tiles, n_ks, n, empty):
    # in the kernel of one and two slabs, block tiles and gathered ones, shallow rings and deep ones; of gathered tiles of four slabs; the mixed one
    rng = np.random.default_rng(empty)
    kb = 1024 // col_block
    rows = []
    for t in range(tiles):
        cols = np.sort((rng.choice(kb, size=n_ks * 32 // col_block, replace=False)[:, None] * col_block + np.arange(col_block)).reshape(-1))
        rows += [cols.tolist() for _ in range(height)]
    rows += [[]] * empty
    csr = csr_from_rows(rows, 1024, rng)
    bits = synth.dense_rhs(rng, 1024, n, "f16")
    rg = np.append(height * np.arange(tiles + 1), height * tiles + empty).astype(np.int32)
    order = rng.permutation(len(rows)).astype(np.int32)
    csr = synth.permute_rows(csr, np.argsort(order))
    c, v = gpu_spmm(csr, order, rg, col_block, bits, ldc_pad=4)
    slabs = {16: "1 slab", 25: "2 slabs", 32: "2 slabs", 60: "4 slabs"}.get(height)
    kernel = "vbr_spmm_kernel<%s%s>" % (slabs, ", column-gathered" if col_block == 4 else "") if slabs else "vbr_spmm_mixed_kernel"
    assert [(p["kernel"], p["tiles"]) for p in v.launches(n)] == [(kernel, tiles + -(-empty // 64))]
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c, c_ref, s, "empty rows beside %s" % kernel)
    assert np.all(c[order[height * tiles:]] == 0.0)


def test_empty_rows_get_zeros_and_single_dense_block_is_a_gemm():
    rng = np.random.default_rng(7)
    csr = csr_from_rows([[], [1, 40], [], [2], []], n_cols=64, rng=rng)
    b = synth.dense_rhs(rng, 64, 16, "f16")
    perm, rg = blocking_bit_exact(csr, 16, 0.5)
    c, _ = gpu_spmm(csr, perm, rg, 16, b)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "empty rows")
    assert np.all(c[[0, 2, 4]] == 0.0)
    dense = random_csr(rng, 48, 96, 1.0)
    b = synth.dense_rhs(rng, 96, 128, "f16")
    perm, rg = blocking_bit_exact(dense, 32, 0.5)
    assert len(rg) == 2                                   # one group, three full blocks
    c, _ = gpu_spmm(dense, perm, rg, 32, b)
    a64 = oracle.bits_to_f64(synth.dense_bits(dense), "f16")
    b64 = oracle.bits_to_f64(b, "f16")
    check_c(c, a64 @ b64, np.abs(a64) @ np.abs(b64), "dense block vs numpy GEMM")


def test_identity_like_right_hand_side_reproduces_rows_exactly():
    rng = np.random.default_rng(8)
    csr = random_csr(rng, 64, 64, 0.2)
    eye = synth.to_bits(np.eye(64, dtype=np.float32), "f16")
    perm, rg = blocking_bit_exact(csr, 16, 0.4)
    c, _ = gpu_spmm(csr, perm, rg, 16, eye)
    assert np.array_equal(c, oracle.bits_to_f64(synth.dense_bits(csr), "f16"))


def test_argument_checks_on_the_gpu_entry():
    import torch
    rng = np.random.default_rng(9)
    csr = random_csr(rng, 20, 32, 0.3)
    perm, rg = binding.sa1_reorder(csr, 16, 0.5)
    v = binding.vbr_build(csr, perm, rg, 16).upload("cuda:0")
    b = torch.zeros((32, 16), dtype=torch.float16, device="cuda:0")
    c = torch.zeros((20, 16), dtype=torch.float32, device="cuda:0")
    s = torch.cuda.current_stream().cuda_stream
    assert binding.vbr_spmm_raw(v, b.data_ptr(), 16, c.data_ptr(), 16, 12, s) == -1       # N % 8
    assert binding.vbr_spmm_raw(v, b.data_ptr(), 8, c.data_ptr(), 16, 16, s) == -1        # ldb < N
    assert binding.vbr_spmm_raw(v, b.data_ptr() + 2, 16, c.data_ptr(), 16, 16, s) == -1   # alignment
    assert binding.vbr_spmm_raw(v, b.data_ptr(), 16, c.data_ptr(), 16, 0, s) == 0         # N = 0: nothing to do
    assert binding.vbr_spmm_raw(v, b.data_ptr(), 16, c.data_ptr(), 16, 16, s) == 0
    torch.cuda.synchronize()


@pytest.mark.parametrize("col_block,short", [(16, False), (8, True), (3, False)])
def test_b_rows_no_block_touches_never_reach_c(col_block, short):
    # Column blocks no row of A enters hold NaN and Inf in B.  Padding of K-steps, of partial slabs
    # and of absent slabs must come from zeros, never from whatever B rows happen to be near: C
    # stays finite and within the bound.  (B rows inside a STORED block do meet the block's
    # fill-in zeros: that is the format's semantics, not tested here.)
    import torch
    rng = np.random.default_rng(50 + col_block)
    kb, n = 40, 136
    m = 6000 if short else 300
    dens = 0.004 if short else 0.05
    csr = random_csr(rng, m, kb * col_block, dens)
    # empty the odd column blocks of A
    keep = (csr["col_idx"] // col_block) % 2 == 0
    rows = np.repeat(np.arange(m), np.diff(csr["row_ptr"]))[keep]
    csr = synth.csr_from_coo(m, kb * col_block, rows, csr["col_idx"][keep], csr["vals"][keep], "f16")
    b_bits = synth.dense_rhs(rng, kb * col_block, n, "f16")
    poison = b_bits.copy()
    odd = (np.arange(kb * col_block) // col_block) % 2 == 1
    poison[odd] = np.where(rng.random((int(odd.sum()), n)) < 0.5, 0x7E00, 0x7C00).astype(np.uint16)   # NaN / +Inf
    perm, rg = blocking_bit_exact(csr, col_block, 0.9 if short else 0.4)
    c, v = gpu_spmm(csr, perm, rg, col_block, poison)
    c_ref, s = oracle.spmm(csr, b_bits)          # the clean B: A never reads the poisoned rows
    assert np.isfinite(c).all()
    check_c(c, c_ref, s, "poisoned B rows, cb=%d" % col_block)


def one_row_with_column(kind):
    """A matrix packed as ``kind`` says, its partition and block width, and a column k that one row alone has an entry in;
    then the rows that NaN in row k of B must reach at most: a number of rows, or the rows themselves."""
    rng = np.random.default_rng(17)
    if kind == "gathered":              # single-row groups in clusters over the same columns: tiles of 64 rows
        m, cols, cb = 1100, 2048, 16
        rows = [(128 * (i // 70 % 15) + rng.choice(128, size=50, replace=False)).tolist() for i in range(m)]
        k, limit = cols - 1, 64
        rows[500].append(k)
        perm, rg = np.arange(m, dtype=np.int32), np.arange(m + 1, dtype=np.int32)
    elif kind == "gathered by length":  # a row's columns are those of the next longer one; the rows of five tall groups stand among the others
        cols, cb, low = 4096, 16, 1500
        order = rng.permutation(cols)
        lens = np.concatenate([(100 * rng.random(low) ** 6 + 1).astype(int), rng.integers(150, 250, size=100)])
        lens[77] = 300
        rows = [order[:n].tolist() for n in lens]
        k, limit = int(order[299]), 64
        perm = np.arange(low + 100, dtype=np.int32)
        rg = np.concatenate([np.arange(low + 1), low + 20 * np.arange(1, 6)]).astype(np.int32)
    elif kind.startswith("panels"):     # a K-step is one block of 32 columns, or two of 16
        cb = int(kind.split()[1])
        m, cols = 6000, 14 * cb
        rows = [np.nonzero(rng.random(13 * cb) < 0.2)[0].tolist() for _ in range(m)]
        k, limit = 13 * cb + 3, 16 if cb == 32 else 128
        rows[1234].append(k)
        perm, rg = np.arange(m, dtype=np.int32), np.arange(m + 1, dtype=np.int32)
    elif kind == "blocks":              # groups of 40 rows, blocks half full: every row of the group, no other
        m, cols, cb = 400, 1024, 16
        blocks = [rng.choice(60, size=12, replace=False) for _ in range(10)]
        rows = [[int(c) for b in blocks[i // 40] for c in range(16 * b, 16 * b + 16) if rng.random() < 0.5] for i in range(m)]
        k, limit = cols - 5, np.arange(120, 160)
        rows[130].append(k)
        perm, rg = np.arange(m, dtype=np.int32), np.arange(0, m + 1, 40, dtype=np.int32)
    else:                               # entry rows: the row itself, no other
        m, cols, cb = 9000, 6400, 32
        rows = [rng.choice(cols - 1, size=12, replace=False).tolist() for _ in range(m)]
        k, limit = cols - 1, np.array([4321])
        rows[4321].append(k)
        perm, rg = np.arange(m, dtype=np.int32), np.arange(m + 1, dtype=np.int32)
    return csr_from_rows(rows, cols, rng), perm, rg, cb, k, limit


@pytest.mark.parametrize("kind,kernel", [("gathered", "vbr_spmm_kernel<4 slabs, column-gathered>"), ("gathered by length", "vbr_spmm_kernel<4 slabs, column-gathered>"),
                                         ("panels 16", "vbr_spmm_panel_kernel"), ("panels 32", "vbr_spmm_panel_kernel"),
                                         ("blocks", "vbr_spmm_kernel<4 slabs>"), ("entries", "entry_rows_kernel")])
def test_rows_that_a_nan_in_b_reaches(kind, kernel):
    # what the header says about non-finite values, packing by packing: the row that has an entry in that column, and
    # of the others at most those that share its tile, panel slab or group; all the rest is right to the last element
    csr, perm, rg, cb, k, limit = one_row_with_column(kind)
    rows = np.repeat(np.arange(csr["n_rows"]), np.diff(csr["row_ptr"]))
    own = rows[csr["col_idx"] == k]
    assert own.size == 1
    clean = synth.dense_rhs(np.random.default_rng(3), csr["n_cols"], 72, "f16")
    bits = clean.copy()
    bits[k] = 0x7E00
    c, v = gpu_spmm(csr, perm, rg, cb, bits)
    assert v.launches(72)[0]["kernel"] == kernel
    hit = np.isnan(c).any(axis=1)
    assert np.isnan(c[hit]).all() and hit[own[0]]
    reached = np.nonzero(hit)[0]
    if isinstance(limit, int):
        assert reached.size <= limit, reached.size
    else:
        assert np.array_equal(reached, limit)
    if kind.startswith("gathered") or kind == "panels 16":
        assert reached.size > 16                     # a tile is not one slab, nor is what a K-step of two blocks reaches ...
    if kind == "gathered by length":
        assert (reached >= 1500).any()               # ... nor only of low groups: these have other blocks only
        group = np.searchsorted(rg, reached, side="right") - 1
        stored = {int(np.searchsorted(rg, r, side="right") - 1) for r in rows[csr["col_idx"] // cb == k // cb]}
        assert any(int(g) not in stored for g in group[reached >= 1500])
    c_ref, s = oracle.spmm(csr, clean)
    check_c(c[~hit], c_ref[~hit], s[~hit], "rows a NaN in B does not reach, " + kind)


def test_runs_on_the_given_stream_and_in_a_captured_graph():
    # vbr_spmm only enqueues kernels on the stream it is given (no allocation, no memset, no
    # synchronisation), so it can run on a side stream and be captured into a graph; every replay
    # must reproduce the eager result for the B that is in place at that moment
    import torch
    rng = np.random.default_rng(60)
    w = synth.workload("c3", scale=0.125)            # tall and low groups: several kernels per call
    a, cb = w["A"], w["col_block"]
    perm, rg = binding.sa1_reorder(a, cb, w["taus"][1])
    v = binding.vbr_build(a, perm, rg, cb).upload("cuda:0")
    k, n = w["B"].shape
    b = torch_io.bits_to_device(w["B"], w["dtype"])
    c_ref, s_ref = oracle.spmm(a, w["B"])
    side = torch.cuda.Stream()                        # default priority
    c_side = torch.full((a["n_rows"], n), float("nan"), dtype=torch.float32, device="cuda:0")
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        v.spmm(b, c_side)
    side.synchronize()
    check_c(c_side.cpu().numpy().astype(np.float64), c_ref, s_ref, "side stream")

    c_graph = torch.full_like(c_side, float("nan"))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        v.spmm(b, c_graph)
    for rep in range(3):
        b_bits = synth.dense_rhs(rng, k, n, w["dtype"], dist="normal")
        b.copy_(torch_io.bits_to_device(b_bits, w["dtype"]))       # eager work between the replays
        c_graph.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        c_eager = v.spmm(b, torch.empty_like(c_graph))
        torch.cuda.synchronize()
        assert torch.equal(c_graph, c_eager), "replay %d differs from the eager launch" % rep
        c_ref, s_ref = oracle.spmm(a, b_bits)
        check_c(c_graph.cpu().numpy().astype(np.float64), c_ref, s_ref, "graph replay %d" % rep)


def test_calls_of_several_launches_keep_the_order_of_the_callers_stream_and_replay_in_a_graph():
    # the launches of a multiply follow each other on the caller's stream: work queued before the call
    # (the NaN fill) must be over before any launch writes, work queued after it (the clone) must
    # see every row; a captured graph must carry all of them
    import torch
    rng = np.random.default_rng(61)
    w = synth.workload("rmat")
    a, cb = w["A"], w["col_block"]
    perm, rg = binding.sa1_reorder(a, cb, w["taus"][0])
    v = binding.vbr_build(a, perm, rg, cb).upload("cuda:0")
    k, n = w["B"].shape
    assert len(v.launches(n)) >= 2, v.launches(n)
    b = torch_io.bits_to_device(w["B"], w["dtype"])
    c_ref, s_ref = oracle.spmm(a, w["B"])
    side = torch.cuda.Stream()                        # default priority
    c = torch.empty((a["n_rows"], n), dtype=torch.float32, device="cuda:0")
    side.wait_stream(torch.cuda.current_stream())
    results = []
    with torch.cuda.stream(side):
        for _ in range(6):
            c.fill_(float("nan"))
            v.spmm(b, c)
            results.append(c.clone())
    side.synchronize()
    check_c(results[0].cpu().numpy().astype(np.float64), c_ref, s_ref, "several launches, first call")
    for i, r in enumerate(results[1:]):
        assert torch.equal(r, results[0]), "call %d differs from the first" % (i + 1)

    c_graph = torch.full_like(c, float("nan"))
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        v.spmm(b, c_graph)
    for rep in range(3):
        b_bits = synth.dense_rhs(rng, k, n, w["dtype"])
        b.copy_(torch_io.bits_to_device(b_bits, w["dtype"]))       # eager work between the replays
        c_graph.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        c_eager = v.spmm(b, torch.empty_like(c_graph))
        torch.cuda.synchronize()
        assert torch.equal(c_graph, c_eager), "replay %d differs from the eager launches" % rep
    c_ref, s_ref = oracle.spmm(a, b_bits)
    check_c(c_graph.cpu().numpy().astype(np.float64), c_ref, s_ref, "graph replay")


def test_two_handles_on_two_streams_at_the_same_time():
    # a handle is only read by a multiply and shares nothing with other handles, so two multiplies of several launches
    # each may be in flight at once from different caller streams
    import torch
    rng = np.random.default_rng(62)
    w = synth.workload("rmat")
    a, cb = w["A"], w["col_block"]
    perm, rg = binding.sa1_reorder(a, cb, w["taus"][0])
    k, n = w["B"].shape
    hs = [binding.vbr_build(a, perm, rg, cb).upload("cuda:0") for _ in range(2)]
    assert len(hs[0].launches(n)) >= 2
    bs = [torch_io.bits_to_device(synth.dense_rhs(rng, k, n, w["dtype"]), w["dtype"]) for _ in range(2)]
    alone = [hs[i].spmm(bs[i], torch.empty((a["n_rows"], n), dtype=torch.float32, device="cuda:0")) for i in range(2)]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]          # default priority
    cs = [torch.full_like(alone[0], float("nan")) for _ in range(2)]
    for st in streams:
        st.wait_stream(torch.cuda.current_stream())
    for _ in range(5):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                cs[i].fill_(float("nan"))
                hs[i].spmm(bs[i], cs[i])
    for st in streams:
        st.synchronize()
    for i in range(2):
        assert torch.equal(cs[i], alone[i]), "handle %d: concurrent result differs from the one computed alone" % i
        hs[i].close()


def test_right_hand_side_larger_than_4_gib():
    # B is a 256-column window of a 70 000 x 32 776 tensor (4.6 GB): row bases need 64 bits
    import torch
    rng = np.random.default_rng(41)
    k, n, ld = 70000, 256, 32776
    rows = [sorted(set(rng.integers(0, k, size=40).tolist()) | {0, k - 1}) for _ in range(48)]
    csr = csr_from_rows(rows, n_cols=k, rng=rng)
    b_bits = synth.dense_rhs(rng, k, n, "f16")
    big = torch.zeros((k, ld), dtype=torch.float16, device="cuda:0")
    b = big[:, 1024:1024 + n]
    b.copy_(torch_io.bits_to_device(b_bits, "f16"))
    assert k * ld * 2 > (1 << 32) and b.stride(0) == ld
    for col_block, perm, rg in [(16, np.arange(48, dtype=np.int32), np.array([0, 16, 48], dtype=np.int32)),
                                (8, *binding.sa1_reorder(csr, 8, 0.3))]:
        v = binding.vbr_build(csr, perm, rg, col_block).upload("cuda:0")
        c = torch.full((48, n), float("nan"), dtype=torch.float32, device="cuda:0")
        v.spmm(b, c)
        torch.cuda.synchronize()
        c_ref, s = oracle.spmm(csr, b_bits)
        check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "B beyond 4 GiB, cb=%d" % col_block)
    del big


@pytest.mark.parametrize("n_cols,dtype", [(65536, "f16"), (65536, "bf16"), (70000, "f16"), (70000, "bf16")])
def test_csr_comparator_with_a_right_hand_side_larger_than_4_gib(n_cols, dtype):
    # rows of 0 to 45 entries, the last column among them, of one and of two words, with 64, 128 and 256 columns a wave; rows for a
    # wave and for a workgroup; infinities in rows of B that only the long rows have
    import torch
    rng = np.random.default_rng(n_cols)
    ld = 33000
    short, long = np.repeat(np.arange(46), 4).tolist(), [257, 300, 520, 1030, 1200]
    lists = [np.sort(rng.choice(n_cols - 1000, size=x, replace=False)).tolist() for x in rng.permutation(short)]
    lists = [x[:-1] + [n_cols - 1] if x else x for x in lists]
    big = torch.zeros((n_cols, ld), dtype=torch.float16 if dtype == "f16" else torch.bfloat16, device="cuda:0")
    assert n_cols * ld * 2 > (1 << 32)
    for rows in (lists, lists + [np.sort(rng.choice(n_cols, size=x, replace=False)).tolist() for x in long]):
        csr = csr_from_rows(rows, n_cols, rng, dtype=dtype)
        m = binding.CsrDev(csr).upload("cuda:0")
        for n in (64, 128, 200):
            bits = synth.dense_rhs(rng, n_cols, n, dtype)
            b = big[:, 1000:1000 + n]
            b.copy_(torch_io.bits_to_device(bits, dtype))
            c = m.spmm(b)
            torch.cuda.synchronize()
            c_ref, s = oracle.spmm(csr, bits)
            check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "B beyond 4 GiB, %d rows, n=%d" % (len(rows), n))
            b[n_cols - 1000:n_cols - 1] = float("inf")
            again = m.spmm(b)
            torch.cuda.synchronize()
            assert torch.equal(again.cpu()[:len(lists)], c.cpu()[:len(lists)])
    del big, b


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_long_lists_against_a_wide_b_on_both_sides_of_4_gib(dtype):
    # rows of B up to the last the offsets of the wide kernel reach, and one step beyond, where the tile kernel takes them
    import torch
    rng = np.random.default_rng(7)
    n_cols, n, groups, h, cb = 2560, 1544, 128, 40, 64
    lists = [(np.sort(rng.choice(n_cols // cb - 1, size=2, replace=False)).tolist() + [n_cols // cb - 1]) for _ in range(groups)]
    csr = csr_from_rows([np.concatenate([np.arange(b * cb, (b + 1) * cb) for b in x]).tolist() for x in lists for _ in range(h)], n_cols, rng, dtype=dtype)
    perm, rg = np.arange(groups * h, dtype=np.int32), np.arange(0, groups * h + 1, h, dtype=np.int32)
    v = binding.vbr_build(csr, perm, rg, cb).upload("cuda:0")
    v.audit()
    assert [p["function"] for p in v.launches(n)] == ["vbr_spmm_wide_kernel"]
    bits = synth.dense_rhs(rng, n_cols, n, dtype)
    c_ref, s = oracle.spmm(csr, bits)
    most = ((0xFFFFF000 // 2 - n) // (n_cols - 1)) // 8 * 8
    flat = torch.zeros(n_cols * (most + 8), dtype=torch.float16 if dtype == "f16" else torch.bfloat16, device="cuda:0")
    for ld in (most, most + 8):
        b = flat[:n_cols * ld].view(n_cols, ld)[:, :n]
        b.copy_(torch_io.bits_to_device(bits, dtype))
        c = torch.full((groups * h, n), float("nan"), dtype=torch.float32, device="cuda:0")
        v.spmm(b, c)
        torch.cuda.synchronize()
        check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "ldb = %d" % ld)
    del flat, b


# --------------------------------------------------------------------------- the CSR comparator kernel
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_csr_comparator_matches_oracle(dtype):
    import torch
    rng = np.random.default_rng(21)
    for m, k, n, dens in [(70, 96, 64, 0.2), (301, 160, 520, 0.05), (33, 64, 8, 0.6), (5, 32, 1032, 0.0)]:
        csr = random_csr(rng, m, k, dens, dtype=dtype)
        b_bits = synth.dense_rhs(rng, k, n, dtype)
        h = binding.CsrDev(csr).upload("cuda:0")
        full = np.zeros((k, n + 8), dtype=np.uint16)
        full[:, :n] = b_bits
        b = torch_io.bits_to_device(full, dtype)[:, :n]                      # padded leading dimension
        c_full = torch.full((m, n + 4), float("nan"), dtype=torch.float32, device="cuda:0")
        h.spmm(b, c_full[:, :n])
        torch.cuda.synchronize()
        out = c_full.cpu().numpy()
        assert np.isnan(out[:, n:]).all()
        c_ref, s = oracle.spmm(csr, b_bits)
        check_c(out[:, :n].astype(np.float64), c_ref, s, "csr %s m=%d n=%d" % (dtype, m, n))


@pytest.mark.parametrize("n,ldb_pad,dtype", [(8, 0, "f16"), (128, 0, "bf16"), (136, 8, "f16"), (264, 56, "bf16"), (1160, 0, "f16")])
def test_csr_comparator_at_the_row_lengths_where_it_splits(n, ldb_pad, dtype):
    # a row per 16 (32) lanes, per wave, per workgroup: lengths around a batch of 16 entries, around the
    # limits 256 and 1024, empty rows in between; one column tile and several, a ragged last one, rows of B
    # inside and across cache lines
    import torch
    rng = np.random.default_rng(n)
    k = 2600
    lens = [0, 1, 2, 15, 16, 17, 31, 33, 63, 64, 65, 0, 255, 256, 257, 300, 512, 513, 1023, 1024, 1025, 1300, 2049, 2600, 0] + [5] * 30
    csr = csr_from_rows([sorted(rng.choice(k, size=x, replace=False).tolist()) for x in lens], k, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, k, n + ldb_pad, dtype)
    b = torch_io.bits_to_device(bits, dtype)[:, :n]
    c = torch.full((len(lens), n), float("nan"), dtype=torch.float32, device="cuda:0")
    binding.CsrDev(csr).upload("cuda:0").spmm(b, c)
    torch.cuda.synchronize()
    c_ref, s = oracle.spmm(csr, np.ascontiguousarray(bits[:, :n]))
    check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "csr n=%d" % n)


@pytest.mark.parametrize("n,ldb_pad,dtype", [(64, 0, "bf16"), (128, 0, "f16"), (200, 8, "bf16"), (256, 8, "f16")])
def test_csr_comparator_at_every_length_of_a_rows_end(n, ldb_pad, dtype):
    # four rows of every length, so that a wave has them alone: each way the loads in flight end with 64 columns a wave, of rows for 16 lanes and of the
    # shares of rows for a wave and for a workgroup; infinities in the rows of B that only the longest rows have
    import torch
    rng = np.random.default_rng(n)
    k = 1500
    lens = np.repeat(list(range(46)) + list(range(257, 330, 8)), 4).tolist() + list(range(1025, 1170, 16))
    csr = csr_from_rows([list(range(x)) for x in rng.permutation(lens)], k, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, k, n + ldb_pad, dtype)
    b = torch_io.bits_to_device(bits, dtype)[:, :n]
    m = binding.CsrDev(csr).upload("cuda:0")
    c = m.spmm(b)
    torch.cuda.synchronize()
    c_ref, s = oracle.spmm(csr, np.ascontiguousarray(bits[:, :n]))
    check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "csr n=%d" % n)
    first = 20
    b[first:] = float("inf")
    short = np.diff(csr["row_ptr"]) <= first
    again = m.spmm(b)
    torch.cuda.synchronize()
    assert torch.equal(again.cpu()[short], c.cpu()[short]) and not torch.isfinite(again.cpu()[~short]).any()


@pytest.mark.parametrize("n,ldb_pad,dtype", [(128, 8, "f16"), (200, 8, "bf16"), (120, 0, "bf16"), (208, 0, "f16")])
@pytest.mark.parametrize("long_rows", [False, True])
def test_csr_comparator_at_every_length_of_a_rows_end_in_wide_waves(n, ldb_pad, dtype, long_rows):
    # the same with 128 columns a wave up to N = 128 and 256 beyond: four rows of every length, which a wave has alone; then the shares of rows for a
    # wave and for a workgroup among so many others that the waves stay as wide
    import torch
    rng = np.random.default_rng(n)
    k = 1500
    lens = list(range(257, 330)) + list(range(1025, 1290, 8)) + [600] * 500 if long_rows else np.repeat(np.arange(46), 4).tolist()
    csr = csr_from_rows([list(range(x)) for x in rng.permutation(lens)], k, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, k, n + ldb_pad, dtype)
    b = torch_io.bits_to_device(bits, dtype)[:, :n]
    m = binding.CsrDev(csr).upload("cuda:0")
    c = m.spmm(b)
    torch.cuda.synchronize()
    c_ref, s = oracle.spmm(csr, np.ascontiguousarray(bits[:, :n]))
    check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "csr n=%d" % n)
    first = 300 if long_rows else 20
    b[first:] = float("inf")
    short = np.diff(csr["row_ptr"]) <= first
    again = m.spmm(b)
    torch.cuda.synchronize()
    assert torch.equal(again.cpu()[short], c.cpu()[short]) and not torch.isfinite(again.cpu()[~short]).any()


@pytest.mark.parametrize("rows,n,n_cols,dtype", [(2048, 1024, 20000, "f16"), (2048, 1024, 70000, "bf16"), (4096, 200, 20000, "bf16"), (4096, 200, 70000, "f16"), (4096, 128, 40000, "f16"), (4096, 128, 70000, "bf16")])
def test_csr_comparator_with_waves_that_keep_step(rows, n, n_cols, dtype):
    # rows of 33 to 64 entries of a B that does not stay in an L2, all resident, with 64, 128 and 256 columns a wave and entries of one and of two words
    import torch
    rng = np.random.default_rng(n)
    csr = csr_from_rows([np.sort(rng.choice(n_cols, size=33 + i % 32, replace=False)).tolist() for i in range(rows)], n_cols, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, n_cols, n, dtype)
    c = binding.CsrDev(csr).upload("cuda:0").spmm(torch_io.bits_to_device(bits, dtype))
    torch.cuda.synchronize()
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "csr %d rows, n=%d" % (rows, n))


@pytest.mark.parametrize("n", [24, 72, 208])
@pytest.mark.parametrize("n_cols,dtype", [(65535, "f16"), (65536, "f16"), (65536, "bf16"), (65537, "bf16"), (70000, "f16")])
def test_entries_of_one_and_of_two_words(n_cols, dtype, n):
    # an entry is one word where every column fits its low half: columns on both sides of that, values of either sign, rows of 0 to 40
    # entries that end at the last column, fewer rows than a wave's groups take behind the last full one
    import torch
    rng = np.random.default_rng(n)
    rows = [sorted({n_cols - 1, *rng.integers(0, n_cols, size=x).tolist()}) if x else [] for x in rng.integers(0, 40, size=41)]
    csr = csr_from_rows(rows, n_cols, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, n_cols, n, dtype)
    b = torch_io.bits_to_device(bits, dtype)
    c = binding.CsrDev(csr).upload("cuda:0").spmm(b)
    torch.cuda.synchronize()
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "csr n_cols=%d" % n_cols)


@pytest.mark.parametrize("n,ldb_pad,dtype", [(520, 0, "f16"), (576, 0, "bf16"), (776, 8, "f16"), (1096, 0, "bf16")])
def test_csr_comparator_with_many_long_rows(n, ldb_pad, dtype):
    # rows for a wave and for a workgroup with 128 and 256 columns a wave: none is much longer than the others
    import torch
    rng = np.random.default_rng(n)
    lens = [257, 300, 512, 513, 1023, 1024, 1025, 1300, 2049, 2600, 0, 17] * 3
    csr = csr_from_rows([sorted(rng.choice(2600, size=x, replace=False).tolist()) for x in lens], 2600, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, 2600, n + ldb_pad, dtype)
    b = torch_io.bits_to_device(bits, dtype)[:, :n]
    c = binding.CsrDev(csr).upload("cuda:0").spmm(b)
    torch.cuda.synchronize()
    c_ref, s = oracle.spmm(csr, np.ascontiguousarray(bits[:, :n]))
    check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "csr n=%d" % n)


@pytest.mark.parametrize("n", [520, 1032, 1288])
def test_csr_comparator_with_64_columns_a_wave_of_an_unaligned_b(n):
    # short rows that use every row of a long B often; nine, seventeen and twenty-one column tiles, the last of eight columns
    import torch
    rng = np.random.default_rng(n)
    cols = (rng.integers(0, 16000, size=(12300, 1)) + np.cumsum(rng.integers(1, 600, size=(12300, 10)), axis=1)) % 16000
    csr = csr_from_rows([np.unique(r).tolist() for r in cols], 16000, rng)
    bits = synth.dense_rhs(rng, 16000, n, "f16")
    c = binding.CsrDev(csr).upload("cuda:0").spmm(torch_io.bits_to_device(bits, "f16"))
    torch.cuda.synchronize()
    c_ref, s = oracle.spmm(csr, bits)
    check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "csr n=%d" % n)


@pytest.mark.parametrize("n,ldb_pad,dtype", [(200, 0, "f16"), (456, 0, "f16"), (520, 0, "bf16"), (1096, 0, "f16"), (1848, 8, "f16")])
def test_csr_comparator_with_long_rows_in_wide_waves(n, ldb_pad, dtype):
    # so many entries that 128 and 256 columns a wave are taken: rows for 16 and 32 lanes, for a wave and for a workgroup; rows of B inside and (N = 1848)
    # on cache lines
    import torch
    rng = np.random.default_rng(n)
    lens = ([257, 300, 512, 513, 1023, 1024, 1025, 1100, 0, 17, 256, 255] + [600] * 30) * 30
    csr = csr_from_rows([sorted(rng.choice(2600, size=x, replace=False).tolist()) for x in lens], 2600, rng, dtype=dtype)
    bits = synth.dense_rhs(rng, 2600, n + ldb_pad, dtype)
    b = torch_io.bits_to_device(bits, dtype)[:, :n]
    c = binding.CsrDev(csr).upload("cuda:0").spmm(b)
    torch.cuda.synchronize()
    c_ref, s = oracle.spmm(csr, np.ascontiguousarray(bits[:, :n]))
    check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "csr n=%d" % n)


@pytest.mark.parametrize("n,ldb_pad", [(520, 0), (1032, 0), (512, 0), (296, 24)])
def test_csr_comparator_with_64_columns_a_wave_of_a_long_b(n, ldb_pad):
    # short rows that use every row of a B that does not stay in an L2 often; rows of B inside cache lines and on them
    import torch
    rng = np.random.default_rng(n)
    cols = (rng.integers(0, 17000, size=(12300, 1)) + np.cumsum(rng.integers(1, 600, size=(12300, 10)), axis=1)) % 17000
    csr = csr_from_rows([np.unique(r).tolist() for r in cols], 17000, rng)
    bits = synth.dense_rhs(rng, 17000, n + ldb_pad, "f16")
    c = binding.CsrDev(csr).upload("cuda:0").spmm(torch_io.bits_to_device(bits, "f16")[:, :n])
    torch.cuda.synchronize()
    c_ref, s = oracle.spmm(csr, np.ascontiguousarray(bits[:, :n]))
    check_c(c.cpu().numpy().astype(np.float64), c_ref, s, "csr n=%d" % n)


def test_csr_comparator_and_blocked_path_agree_on_the_graph_workload():
    import torch
    w = synth.workload("rmat", scale=0.125)
    a, cb = w["A"], w["col_block"]
    perm, rg = blocking_bit_exact(a, cb, w["taus"][0])
    c, v = gpu_spmm(a, perm, rg, cb, w["B"])
    index_bit_exact(v, a, perm, rg, cb)
    c_ref, s = oracle.spmm(a, w["B"])
    check_c(c, c_ref, s, "rmat blocked")
    b = torch_io.bits_to_device(w["B"], w["dtype"])
    c2 = binding.CsrDev(a).upload("cuda:0").spmm(b)
    torch.cuda.synchronize()
    check_c(c2.cpu().numpy().astype(np.float64), c_ref, s, "rmat csr")


# --------------------------------------------------------------------------- the five workloads, reduced
@pytest.mark.parametrize("name,scale,noise", [("c1", 1.0, True), ("c1", 1.0, False), ("c2", 0.25, True),
                                               ("c2", 0.25, False), ("c3", 0.125, True), ("c4", 0.125, True),
                                               ("c5", 0.0625, True)])
def test_workloads_reduced_elementwise(name, scale, noise):
    w = synth.workload(name, scale=scale, noise=noise)
    c_ref, s = oracle.spmm(w["A"], w["B"])
    for tau in w["taus"]:
        perm, rg = blocking_bit_exact(w["A"], w["col_block"], tau)
        c, v = gpu_spmm(w["A"], perm, rg, w["col_block"], w["B"])
        index_bit_exact(v, w["A"], perm, rg, w["col_block"])
        check_c(c, c_ref, s, "%s tau=%g" % (name, tau))


# --------------------------------------------------------------------------- wide dense matrices, small A
def test_one_slab_groups_with_eight_or_more_column_tiles():
    # N = 2056: nine 256-column tiles (the last one ragged), so the workgroup -> (tile, column
    # tile) map takes the branch it takes at the full size of the pruned-weight workload
    rng = np.random.default_rng(77)
    keep = rng.random((40, 48)) < 0.15
    mask = np.kron(keep, np.ones((16, 16), dtype=bool))
    r, cc = np.nonzero(mask)
    vals = synth.to_bits(rng.standard_normal(r.size).astype(np.float32) / 4, "f16")
    csr = synth.csr_from_coo(640, 768, r, cc, vals, "f16")
    b = synth.dense_rhs(rng, 768, 2056, "f16", dist="normal")
    perm, rg = blocking_bit_exact(csr, 16, 0.5)
    c, v = gpu_spmm(csr, perm, rg, 16, b)
    index_bit_exact(v, csr, perm, rg, 16)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "one-slab groups, N=2056")


def test_short_groups_with_eight_or_more_column_tiles():
    # short groups (panels) with N = 1032: nine 128-column tiles, the last one 8 columns wide
    rng = np.random.default_rng(78)
    csr = random_csr(rng, 6000, 20 * 16, 0.01)
    b = synth.dense_rhs(rng, 320, 1032, "f16")
    perm, rg = blocking_bit_exact(csr, 16, 0.9)
    h = np.diff(rg)
    assert h[h < 16].sum() >= 4096
    c, v = gpu_spmm(csr, perm, rg, 16, b)
    index_bit_exact(v, csr, perm, rg, 16)
    c_ref, s = oracle.spmm(csr, b)
    check_c(c, c_ref, s, "short groups, N=1032")


# --------------------------------------------------------------------------- full sizes, every element
@pytest.mark.parametrize("name", ["c2", "c3", "c4", "c5", "rmat"])
def test_workloads_full_size_every_element(name):
    # the launch configuration bench.py times, at the full size, every element of C against the
    # oracle; c3 at all three of its thresholds
    w = synth.workload(name)
    a, cb = w["A"], w["col_block"]
    print("full size %s: oracle multiply" % name, flush=True)
    c_ref, s = oracle.spmm(a, w["B"])
    empty = np.nonzero(np.diff(a["row_ptr"]) == 0)[0]
    for tau in w["taus"]:
        print("full size %s tau=%g: library" % (name, tau), flush=True)
        perm, rg = blocking_bit_exact(a, cb, tau)
        c, v = gpu_spmm(a, perm, rg, cb, w["B"])
        index_bit_exact(v, a, perm, rg, cb)
        check_c(c, c_ref, s, "%s full size tau=%g" % (name, tau))
        # rows without entries are exactly zero
        assert np.all(c[empty] == 0.0)
        del c, v


# --------------------------------------------------------------------------- the comparison experiments, reduced
CURVE_TAUS = [0.1, 0.2, 0.3, 0.4, 0.5, 0.6, 0.7, 0.8, 0.9, 1.0]


def blocked_and_csr_against_oracle(a, col_block, tau, b_bits, what):
    import torch
    perm, rg = blocking_bit_exact(a, col_block, tau)
    c, v = gpu_spmm(a, perm, rg, col_block, b_bits)
    index_bit_exact(v, a, perm, rg, col_block)
    c_ref, s = oracle.spmm(a, b_bits)
    check_c(c, c_ref, s, what + " blocked")
    b = torch_io.bits_to_device(b_bits, a["dtype"])
    c2 = binding.CsrDev(a).upload("cuda:0").spmm(b)
    torch.cuda.synchronize()
    check_c(c2.cpu().numpy().astype(np.float64), c_ref, s, what + " csr")


@pytest.mark.parametrize("theta,rho", [(0.1, 0.05), (0.3, 0.5), (0.02, 0.2)])
def test_landscape_point_at_the_selected_threshold(theta, rho):
    # one point of the synthetic landscape A(Delta, theta, rho) at reduced size: the threshold the
    # selection rule picks (same as the oracle's), then both kernels against the oracle
    rng = np.random.default_rng(int(theta * 1000 + rho * 100))
    a = synth.landscape(rng, 1024, 32, theta, rho)
    b_bits = synth.dense_rhs(rng, 1024, 264, "f16")
    sel = binding.sa1_blocking_curve(a, 32, CURVE_TAUS, 32)["selected"]
    assert sel == oracle.blocking_curve(a, 32, CURVE_TAUS, 32)["selected"]
    blocked_and_csr_against_oracle(a, 32, CURVE_TAUS[sel], b_bits, "landscape theta=%g rho=%g" % (theta, rho))


@pytest.mark.parametrize("degree,col_block", [(8, 64), (8, 256), (128, 64), (128, 256), (32, 128)])
def test_graph_grid_points_reduced(degree, col_block):
    # corners and centre of the graph grid (edges per node x column-block width) at 2^11 nodes
    w = synth.workload("rmat", scale=0.125, rmat_degree=degree, rmat_col_block=col_block)
    a = w["A"]
    sel = binding.sa1_blocking_curve(a, col_block, CURVE_TAUS, col_block)["selected"]
    assert sel == oracle.blocking_curve(a, col_block, CURVE_TAUS, col_block)["selected"]
    for tau in {CURVE_TAUS[sel], 0.4}:
        blocked_and_csr_against_oracle(a, col_block, tau, w["B"], "rmat degree=%d cb=%d tau=%g" % (degree, col_block, tau))
