"""What a user of this library has it do, as measured cases.

A program has a sparse matrix in CSR.  It reorders and packs it once (``sa1_reorder``, ``vbr_build``, ``Vbr.upload``),
then multiplies it by dense matrices many times (``Vbr.spmm``).  Before that it may sweep thresholds to choose a
blocking (``sa1_blocking_curve``), and it compares against the multiply straight from CSR (``CsrDev.spmm``).
Accordingly a case has a ``path``:

  multiply   one ``Vbr.spmm`` into an output the program keeps; the packed matrix is in hand
  csr        one ``CsrDev.spmm`` likewise
  setup      a new matrix: reorder, build, upload, first multiply (host work and the copy included)
  curve      one ``sa1_blocking_curve`` over ten thresholds (host work)

and a ``kind`` of matrix.  Kinds, sizes, densities, thresholds and value distributions are those of
``synth.workload`` and of the two experiments (``experiments.landscape``, ``experiments.rmat_grid``), drawn here on
the GPU because that takes milliseconds; ``ragged`` has the odd sizes the tests use.
"""
import math

import numpy as np
import torch

from paper_2202_05868_amd import binding

DEV = "cuda:0"
TAUS = [0.1, 0.2, 0.3, 0.4, 0.5, 0.6, 0.7, 0.8, 0.9, 1.0]
RMAT_PROBS = (0.57, 0.19, 0.19, 0.05)


def listed():
    return [
        # The smallest workload (c1): 32-row groups with noise.  A call is over in about ten microseconds: launch and latency.
        dict(name="small_planted", path="multiply", kind="planted", rows=1024, cols=1024, n=256, cb=32, tau=0.7, dtype="f16",
             height=32, share=0.10, noise=0.005, off_block=False),
        # 64 x 64 blocks with 1 % noise (c2): the threshold leaves thousands of groups lower than a matrix-unit tile.
        dict(name="noisy_planted", path="multiply", kind="planted", rows=8192, cols=8192, n=1024, cb=64, tau=0.6, dtype="f16",
             height=64, share=0.05, noise=0.01, off_block=True),
        # Row groups of 16 to 128 rows, blocks filled to 70 %, bf16 (c3): all tile heights in one matrix.
        dict(name="mixed_heights_bf16", path="multiply", kind="mixed", rows=16384, cols=16384, n=512, cb=32, tau=0.6, dtype="bf16",
             share=0.02, fill=0.7),
        # A pruned weight matrix: 16 x 16 blocks at 10 % (c4), the benchmark's default.
        dict(name="pruned_weight", path="multiply", kind="tiles16", rows=4096, cols=16384, n=4096, cb=16, tau=0.5, dtype="f16",
             share=0.10),
        # No structure at all (c5): the blocking finds nothing.
        dict(name="unstructured", path="multiply", kind="uniform", rows=32768, cols=32768, n=256, cb=32, tau=0.3, dtype="f16",
             density=5e-4),
        # A graph with hubs (rmat): the middle of the graph experiment's grid.
        dict(name="graph", path="multiply", kind="rmat", rows=1 << 14, cols=1 << 14, n=4096, cb=64, tau=0.4, dtype="f16", degree=32),
        # The landscape experiment's corners: few, thinly filled blocks against a narrow B ...
        dict(name="landscape_light", path="multiply", kind="landscape", rows=8192, cols=8192, n=2048, cb=64, tau=0.4, dtype="f16",
             theta=0.01, rho=0.05),
        # ... and many well filled ones against the widest B: the largest multiply.
        dict(name="landscape_heavy", path="multiply", kind="landscape", rows=8192, cols=8192, n=8192, cb=64, tau=0.1, dtype="f16",
             theta=0.4, rho=0.5),
        # Odd row count and group heights, a block width that is not a power of two, B padded to a longer row, N no multiple of a tile.
        dict(name="ragged", path="multiply", kind="ragged", rows=5003, cols=24 * 171, n=1000, cb=24, tau=0.5, dtype="f16", share=0.08,
             fill=0.6),
        # The CSR multiply both experiments put beside the blocked one, on the graph.
        dict(name="csr_graph", path="csr", kind="rmat", rows=1 << 14, cols=1 << 14, n=4096, cb=64, tau=0.4, dtype="f16", degree=32),
        # A matrix seen for the first time, from CSR to the first product.
        dict(name="setup_graph", path="setup", kind="rmat", rows=1 << 14, cols=1 << 14, n=256, cb=64, tau=0.4, dtype="f16", degree=32),
        # The choice of a threshold on a landscape matrix.
        dict(name="curve_landscape", path="curve", kind="landscape", rows=8192, cols=8192, n=8, cb=64, tau=0.1, dtype="f16",
             theta=0.1, rho=0.05),
    ]


def draw(rng):
    def between(lo, hi, q=1):                      # over the logarithm, a multiple of q
        return max(q, int(math.exp(rng.uniform(math.log(lo), math.log(hi))) / q + 0.5) * q)

    path = rng.choice(["multiply"] * 7 + ["csr", "setup", "curve"])
    kind = rng.choice(["planted", "mixed", "tiles16", "uniform", "rmat", "landscape", "ragged"])
    dtype = rng.choice(["f16", "f16", "bf16"])
    if kind == "planted":
        cb = rng.choice([32, 64])
        c = dict(rows=between(1024, 8192, cb), cols=between(1024, 8192, cb), n=between(64, 1024, 8), cb=cb, tau=rng.choice([0.6, 0.7]),
                 height=cb, share=round(rng.uniform(0.05, 0.10), 3), noise=rng.choice([0.0, 0.005, 0.01]), off_block=rng.random() < 0.5)
    elif kind == "mixed":
        c = dict(rows=between(4096, 16384, 16), cols=between(4096, 16384, 32), n=between(128, 1024, 8), cb=32,
                 tau=rng.choice([0.4, 0.6, 0.8]), share=round(rng.uniform(0.02, 0.06), 3), fill=round(rng.uniform(0.5, 0.9), 2))
    elif kind == "tiles16":
        c = dict(rows=between(1024, 4096, 16), cols=between(4096, 16384, 16), n=between(512, 4096, 8), cb=16, tau=0.5,
                 share=round(rng.uniform(0.06, 0.15), 3))
    elif kind == "uniform":
        size = between(8192, 32768, 32)
        c = dict(rows=size, cols=size, n=between(64, 1024, 8), cb=32, tau=0.3, density=round(rng.uniform(2e-4, 8e-4), 6))
    elif kind == "rmat":
        size = 1 << rng.choice([12, 13, 14])
        c = dict(rows=size, cols=size, n=between(512, 4096, 8), cb=rng.choice([64, 128, 256]), tau=rng.choice([0.1, 0.3, 0.4]),
                 degree=between(8, 128))
    elif kind == "landscape":
        size = rng.choice([4096, 6144, 8192])
        c = dict(rows=size, cols=size, n=between(1024, 8192, 8), cb=64, tau=rng.choice([0.1, 0.4]),
                 theta=round(math.exp(rng.uniform(math.log(0.01), math.log(0.4))), 4),
                 rho=round(math.exp(rng.uniform(math.log(0.05), math.log(0.5))), 3))
    else:
        cb = rng.choice([5, 8, 12, 16, 24, 40])
        c = dict(rows=between(1000, 8000) | 1, cols=between(1000, 8000, cb), n=8 * (between(1, 160) | 1), cb=cb, tau=0.5,
                 share=round(rng.uniform(0.03, 0.12), 3), fill=round(rng.uniform(0.4, 0.9), 2))
    if path == "setup":
        c["n"] = min(c["n"], 256)
    if path == "curve":
        c["n"] = 8
    return dict(c, path=path, kind=kind, dtype=dtype)


# ------------------------------------------------------------------------------------------- the inputs
def _heights(case, seed):
    """Heights of the planted row groups, summing to the rows."""
    if case["kind"] in ("planted", "tiles16"):
        h = case.get("height", 16)
        return np.full(case["rows"] // h, h, dtype=np.int64)
    r = np.random.default_rng(seed)
    if case["kind"] == "mixed":
        h = r.choice([16, 32, 64, 128], size=case["rows"] // 16 + 1)
    else:
        h = r.integers(1, 101, size=case["rows"])
    h = h[: int(np.searchsorted(np.cumsum(h), case["rows"])) + 1].astype(np.int64)
    h[-1] -= int(h.sum()) - case["rows"]
    return h


def _positions(case, seed, g):
    """Row and column of every entry, sorted by row, then column; and a factor for each value."""
    m, k, cb, kind = case["rows"], case["cols"], case["cb"], case["kind"]
    scale = 1.0
    if kind == "uniform":
        lin = torch.unique(torch.randint(0, m * k, (int(round(m * k * case["density"])),), generator=g, device=DEV))
    elif kind == "rmat":
        # one quadrant per bit of the node numbers for every edge; duplicates collapse; rows scrambled
        edges = int(m * case["degree"])
        cum = torch.tensor(np.cumsum(RMAT_PROBS)[:3], dtype=torch.float32, device=DEV)
        r = torch.zeros(edges, dtype=torch.int64, device=DEV)
        c = torch.zeros(edges, dtype=torch.int64, device=DEV)
        for _ in range(m.bit_length() - 1):
            quad = torch.bucketize(torch.rand(edges, generator=g, device=DEV), cum, right=True)
            r, c = (r << 1) | (quad >> 1), (c << 1) | (quad & 1)
        lin = torch.unique(torch.randperm(m, generator=g, device=DEV)[r] * k + c)
    else:
        if kind == "landscape":
            # a share theta of all 64 x 64 blocks holds entries, a share rho of the cells of each
            label = torch.arange(m, device=DEV) // 64
            flags = torch.zeros((m // 64) * (k // 64), dtype=torch.bool, device=DEV)
            flags[torch.randperm(flags.numel(), generator=g, device=DEV)[: max(1, round(case["theta"] * flags.numel()))]] = True
            flags, fill = flags.view(m // 64, k // 64), case["rho"]
        else:
            h = torch.from_numpy(_heights(case, seed)).to(DEV)
            label = torch.repeat_interleave(torch.arange(h.numel(), device=DEV), h)
            flags, fill = torch.rand(h.numel(), k // cb, generator=g, device=DEV), case.get("fill", 1.0)
            if kind == "tiles16":                  # every block on its own; the others have a fixed number per group
                flags = flags < case["share"]
            else:
                per = max(1, round(case["share"] * (k // cb)))
                flags = flags <= flags.kthvalue(per, dim=1, keepdim=True).values
        order = torch.arange(m, device=DEV) if kind == "tiles16" else torch.randperm(m, generator=g, device=DEV)
        where = flags[label[order]].repeat_interleave(cb, dim=1)
        planted = where.clone() if case.get("off_block") else None
        if fill < 1.0:
            where &= torch.rand(m, k, generator=g, device=DEV) < fill
        if case.get("noise"):
            extra = int(case["noise"] * int(where.sum()))
            lin = torch.randint(0, m * k, (2 * extra,), generator=g, device=DEV)
            if planted is not None:
                lin = lin[~planted.view(-1)[lin]]
            where.view(-1)[lin[:extra]] = True
        lin = where.view(-1).nonzero().view(-1)
        if kind == "tiles16":                      # magnitudes differ from block to block
            size = torch.randn(flags.shape, generator=g, device=DEV).exp() / 16
            scale = size[label[lin // k], (lin % k) // cb]
    return lin // k, lin % k, scale


def _bits(x, dtype):
    return x.to(torch.float16 if dtype == "f16" else torch.bfloat16)


def _matrix(case, seed, g):
    r, c, scale = _positions(case, seed, g)
    if case["kind"] == "tiles16":
        x = torch.randn(r.numel(), generator=g, device=DEV) * scale
    else:
        x = torch.rand(r.numel(), generator=g, device=DEV) * 2 - 1
    row_ptr = torch.zeros(case["rows"] + 1, dtype=torch.int64, device=DEV)
    row_ptr[1:] = torch.bincount(r, minlength=case["rows"]).cumsum(0)
    return dict(n_rows=case["rows"], n_cols=case["cols"], nnz=int(r.numel()), row_ptr=row_ptr.cpu().numpy(),
                col_idx=c.to(torch.int32).cpu().numpy(), vals=_bits(x, case["dtype"]).view(torch.int16).cpu().numpy().view(np.uint16),
                dtype=case["dtype"])


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    a = _matrix(case, seed, g)
    s = dict(path=case["path"], A=a, cb=case["cb"], tau=case["tau"])
    if case["path"] == "curve":
        return s
    pad = 16 if case["kind"] == "ragged" else 0    # a B that is a slice of a wider one
    x = torch.empty(case["cols"], case["n"] + pad, device=DEV)
    x = x.normal_(generator=g) if case["kind"] in ("mixed", "tiles16") else x.uniform_(-1, 1, generator=g)
    s["B"] = _bits(x, case["dtype"])[:, : case["n"]]
    s["C"] = torch.empty(case["rows"], case["n"], dtype=torch.float32, device=DEV)
    if case["path"] == "csr":
        s["M"] = binding.CsrDev(a).upload(DEV)
    elif case["path"] == "multiply":
        perm, row_groups = binding.sa1_reorder(a, case["cb"], case["tau"])
        s["M"] = binding.vbr_build(a, perm, row_groups, case["cb"]).upload(DEV)
    return s


def run(s):
    if s["path"] in ("multiply", "csr"):
        return s["M"].spmm(s["B"], s["C"])
    if s["path"] == "curve":
        return binding.sa1_blocking_curve(s["A"], s["cb"], TAUS, s["cb"])
    perm, row_groups = binding.sa1_reorder(s["A"], s["cb"], s["tau"])
    c = binding.vbr_build(s["A"], perm, row_groups, s["cb"]).upload(DEV).spmm(s["B"], s["C"])
    group = np.repeat(np.arange(row_groups.size - 1), np.diff(row_groups))          # of every position: one length for all inputs
    return [perm, group, c]


# ------------------------------------------------------------------------------------------- what a pass cannot do without
def _expected(case):
    """Expected entries and expected columns with an entry."""
    m, k, cb, kind = case["rows"], case["cols"], case["cb"], case["kind"]
    if kind == "uniform":
        return m * k * case["density"], k * (1 - math.exp(-m * case["density"]))
    if kind == "rmat":
        lg, edges = m.bit_length() - 1, m * case["degree"]
        a, b, c, d = RMAT_PROBS
        nnz = 0.0
        for i in range(lg + 1):
            for j in range(lg + 1 - i):
                for t in range(lg + 1 - i - j):
                    p = a ** i * b ** j * c ** t * d ** (lg - i - j - t)
                    ways = math.comb(lg, i) * math.comb(lg - i, j) * math.comb(lg - i - j, t)
                    nnz += ways * -math.expm1(edges * math.log1p(-p))
        one = b + d
        return nnz, sum(math.comb(lg, i) * -math.expm1(edges * math.log1p(-(one ** i * (1 - one) ** (lg - i)))) for i in range(lg + 1))
    if kind == "landscape":
        groups, share, fill = m / 64, case["theta"], case["rho"]
    else:
        groups = m / {"planted": case.get("height", 16), "tiles16": 16, "mixed": 60, "ragged": 50.5}[kind]
        share, fill = case["share"], case.get("fill", 1.0)
    return m * k * share * fill * (1 + case.get("noise", 0.0)), k * (1 - (1 - share) ** groups)


def work(case):
    nnz, cols = _expected(case)
    csr = 4 * nnz + 8 * (case["rows"] + 1)         # the structure; values are two bytes more
    if case["path"] == "curve":
        return dict(bytes=csr, flops=0)
    product = 2 * nnz + cols * case["n"] * 2 + case["rows"] * case["n"] * 4
    if case["path"] == "setup":
        return dict(bytes=csr + product + 8 * case["rows"], flops=2 * nnz * case["n"])
    return dict(bytes=csr + product, flops=2 * nnz * case["n"])


def tolerance(case):
    # products of 16-bit values are exact in binary32; what differs is the order of the 32-bit sums
    return "exact" if case["path"] == "curve" else dict(rel=1e-5)
