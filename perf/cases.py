"""The calls whose speed is followed: one dict per case, run through the
package's public entry points on one GPU.

listed() names the cases, draw() gives another one of the same ranges,
prepare() makes what a program holds before the call (matrix handle, vectors),
run() is one pass, exact() the same outputs in 64-bit torch, and work() the
bytes and operations one pass cannot do without.  Matrices are drawn on the
GPU from the seed; sizes and families are those of the package's generators
(stencils, Zipf row lengths with uniform columns, banded Poisson rows, a
block-diagonal batch).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1012_2270_amd as rg
from paper_1012_2270_amd import workloads as W

DEV = "cuda:0"
SIZE = {"f64": 8, "f32": 4, "f16": 2, "bf16": 2}
TORCH = {"f64": torch.float64, "f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
ZIPF_MAX = 10_000
BAND = 500


def listed():
    return [
        # a small system inside an outer loop: one launch, latency counts
        dict(name="spmv_5pt_64_f64", kind="spmv", matrix="5pt", n=64, dtype="f64"),
        # the regular half of the benchmark: a finite-difference operator
        dict(name="spmv_7pt_128_f32", kind="spmv", matrix="7pt", n=128, dtype="f32"),
        # a finite-element-like operator in double precision, odd grid size
        dict(name="spmv_27pt_101_f64", kind="spmv", matrix="27pt", n=101, dtype="f64"),
        # the irregular half of the benchmark: graph-like rows, random columns
        dict(name="spmv_zipf_1m_f32", kind="spmv", matrix="zipf", n=1_000_000, dtype="f32", sigma=512, tau=6),
        # an unstructured banded operator with 16-bit stored values
        dict(name="spmv_band_400k_bf16", kind="spmv", matrix="band", n=400_009, mean=24.0, dtype="bf16", sigma=256),
        # the comparison format on the irregular matrix
        dict(name="hyb_zipf_1m_f32", kind="hyb", matrix="zipf", n=1_000_000, dtype="f32"),
        # several right-hand sides on an irregular matrix, column panels kept
        dict(name="spmm_zipf_1m_k4_f32", kind="spmm", matrix="zipf", n=1_000_000, dtype="f32", sigma=512, tau=12,
             k=4, panels=8),
        # an odd number of right-hand sides on a stencil
        dict(name="spmm_27pt_80_k7_f32", kind="spmm", matrix="27pt", n=80, dtype="f32", k=7),
        # many small and middling independent matrices in one launch
        dict(name="batch_256_f32", kind="batch", count=256, dtype="f32", sigma=256),
        # a training step: values updated, forward, both gradients
        dict(name="train_zipf_1m_f32", kind="train", matrix="zipf", n=1_000_000, dtype="f32", sigma=512, tau=16),
        # a mixed-precision solve of a symmetric positive definite system
        dict(name="cg_27pt_96_bf16", kind="cg", n=96, dtype="bf16"),
        # a matrix assembled on the device, converted and used once
        dict(name="convert_zipf_500k_f32", kind="convert", matrix="zipf", n=500_009, dtype="f32", sigma=512, tau=16),
    ]


def _log(rng, lo, hi):
    """Log-uniform integer, odd about as often as even."""
    return int(math.exp(rng.uniform(math.log(lo), math.log(hi))))


def draw(rng):
    kind = rng.choice(["spmv", "spmv", "spmv", "hyb", "spmm", "spmm", "batch", "train", "cg", "convert"])
    if kind == "batch":
        return dict(kind=kind, count=_log(rng, 8, 256), dtype=rng.choice(["f32", "f64", "bf16"]),
                    sigma=rng.choice([1, 256, 1024]))
    if kind == "cg":
        return dict(kind=kind, n=_log(rng, 16, 96), dtype=rng.choice(["f32", "bf16", "f16"]))
    family = rng.choice(["zipf", "band"] if kind == "train" else ["5pt", "7pt", "27pt", "zipf", "band"])
    dtypes = {"spmm": ["f32", "f32", "f64"], "train": ["f32", "f32", "f64"]}.get(kind, ["f32", "f32", "f64", "f16", "bf16"])
    c = dict(kind=kind, matrix=family, dtype=rng.choice(dtypes))
    small = kind in ("spmm", "convert")
    if family == "5pt":
        c["n"] = _log(rng, 16, 600 if small else 1400)
    elif family == "7pt":
        c["n"] = _log(rng, 8, 80 if small else 128)
    elif family == "27pt":
        c["n"] = _log(rng, 6, 64 if small else 100)
    else:
        c["n"] = _log(rng, 500, 500_000 if small else 1_000_000 if family == "zipf" else 600_000)
        c["sigma"] = rng.choice([1, 256, 512, 4096])
        if family == "zipf":
            c["tau"] = rng.choice([6, 12, 16, 32])
        else:
            c["mean"] = round(rng.uniform(8.0, 40.0 if not small else 24.0), 2)
    if kind == "spmm":
        c["k"] = rng.randint(2, 32)
        if family == "zipf" and rng.random() < 0.5:
            c["panels"] = 8
    return c


# ----------------------------------------------------------------------------
# Matrices (CSR on the GPU, from the seed alone)
# ----------------------------------------------------------------------------
def _gen(seed, salt):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 1009 + salt)
    return g


def _offsets(family):
    if family == "5pt":
        return 2, [(0, a, b) for a in (-1, 0, 1) for b in (-1, 0, 1) if abs(a) + abs(b) <= 1]
    o = [(a, b, c) for a in (-1, 0, 1) for b in (-1, 0, 1) for c in (-1, 0, 1)]
    return 3, o if family == "27pt" else [t for t in o if sum(map(abs, t)) <= 1]


def _stencil(family, n, seed=None):
    """Row pointers, columns and values (float64) of a Dirichlet stencil,
    x fastest: diagonal 4 / 6 / 27, off -1; with a seed, the symmetric positive
    definite variant: off -(1 + u / 4), diagonal 1 plus the row's sum of |off|."""
    dims, offs = _offsets(family)
    rows = n ** dims
    i = torch.arange(rows, device=DEV)
    at = (i // (n * n) if dims == 3 else torch.zeros_like(i), (i // n) % n, i % n)
    disp = [(z * n * n if dims == 3 else 0) + y * n + x for z, y, x in offs]
    order = sorted(range(len(offs)), key=lambda k: disp[k])
    mask = torch.ones(rows, len(offs), dtype=torch.bool, device=DEV)
    col = torch.empty(rows, len(offs), dtype=torch.int32, device=DEV)
    val = torch.empty(rows, len(offs), dtype=torch.float64, device=DEV)
    u = torch.rand(len(offs), rows, generator=_gen(seed, 1), device=DEV, dtype=torch.float64) if seed is not None else None
    centre = None
    for slot, k in enumerate(order):
        for d in range(3):
            if offs[k][d]:
                t = at[d] + offs[k][d]
                mask[:, slot] &= (t >= 0) & (t < n)
        j = i + disp[k]
        col[:, slot] = j.to(torch.int32)
        if disp[k] == 0:
            centre = slot
            val[:, slot] = {"5pt": 4.0, "7pt": 6.0, "27pt": 27.0}[family]
        elif u is None:
            val[:, slot] = -1.0
        else:
            # the entry above the diagonal draws, its mirror image takes the same
            hi = max(slot, len(order) - 1 - slot)
            val[:, slot] = -(1.0 + 0.25 * u[hi][i if slot == hi else j.clamp(0, rows - 1)])
    if u is not None:
        off = torch.where(mask, val.abs(), torch.zeros_like(val))
        off[:, centre] = 0.0
        val[:, centre] = 1.0 + off.sum(1)
    rp = torch.zeros(rows + 1, dtype=torch.int64, device=DEV)
    rp[1:] = mask.sum(1).cumsum(0)
    return rows, rp, col[mask], val[mask]


def _columns(lens, lo, hi, g):
    """lens[r] distinct ascending columns per row, uniform in [lo[r], hi[r])."""
    rows = torch.repeat_interleave(torch.arange(lens.numel(), device=DEV), lens)
    big = int(hi.max()) + 1
    draw_ = lambda r: lo[r] + (torch.rand(r.numel(), generator=g, device=DEV, dtype=torch.float64)  # noqa: E731
                               * (hi[r] - lo[r])).to(torch.int64)
    key = torch.sort(rows * big + draw_(rows))[0]
    while True:
        dup = torch.nonzero(key[1:] == key[:-1]).flatten() + 1
        if dup.numel() == 0:
            return (key % big).to(torch.int32)
        r = key[dup] // big
        key[dup] = r * big + draw_(r)
        key = torch.sort(key)[0]


def _random(lens, lo, hi, g):
    col = _columns(lens, lo, hi, g)
    val = torch.randn(col.numel(), generator=g, device=DEV, dtype=torch.float64)
    rp = torch.zeros(lens.numel() + 1, dtype=torch.int64, device=DEV)
    rp[1:] = lens.cumsum(0)
    return rp, col, val


def _cap(n):
    """Longest row of a Zipf matrix (distinct random columns: at most a quarter of them)."""
    return min(ZIPF_MAX, n // 4)


def _band_bounds(n):
    i = torch.arange(n, device=DEV)
    return (i - BAND).clamp(min=0), (i + BAND + 1).clamp(max=n)


def _matrix(c, seed):
    """(rows, row_ptr, col, val float64 holding what the input dtype holds)."""
    family, n = c["matrix"], c["n"]
    if family in ("5pt", "7pt", "27pt"):
        return _stencil(family, n)
    if family == "zipf":
        # the seed deals the same lengths to other rows: equal sizes for every seed
        lens = np.clip(np.random.default_rng(1).zipf(2.0, size=n), 1, _cap(n)).astype(np.int64)
        lens = torch.from_numpy(np.random.default_rng(seed).permutation(lens)).to(DEV)
        lo, hi = torch.zeros(n, dtype=torch.int64, device=DEV), torch.full((n,), n, device=DEV)
    else:
        lo, hi = _band_bounds(n)
        lens = torch.from_numpy(np.random.default_rng(seed).permutation(np.random.default_rng(1).poisson(c["mean"], n)))
        lens = torch.minimum(lens.to(DEV), hi - lo)
    rp, col, val = _random(lens, lo, hi, _gen(seed, 3))
    return n, rp, col, val if c["dtype"] == "f64" else val.float().double()


def _batch(c, seed):
    """Row counts per matrix and the stacked rows with columns of their own matrix."""
    rng = np.random.default_rng(1)
    ns = np.exp(rng.uniform(math.log(100), math.log(20_000), size=c["count"])).astype(np.int64)
    means = rng.uniform(8.0, 40.0, size=c["count"])
    ns = ns[np.random.default_rng(seed).permutation(c["count"])]
    lo, hi = (torch.cat(v) for v in zip(*[_band_bounds(int(n)) for n in ns]))
    mu = torch.from_numpy(np.repeat(means, ns)).to(DEV, torch.float32)
    lens = torch.minimum(torch.poisson(mu, generator=_gen(seed, 2)).to(torch.int64), hi - lo)
    rp, col, val = _random(lens, lo, hi, _gen(seed, 3))
    return ns, rp, col, val if c["dtype"] == "f64" else val.float().double()


def _vec(n, seed, salt, dtype, k=None):
    v = torch.rand(n if k is None else (n, k), generator=_gen(seed, salt), device=DEV, dtype=torch.float64) * 2 - 1
    return v.to(dtype)


def _vdt(c):
    return torch.float64 if c["dtype"] == "f64" else torch.float32


def _host(n, rp, col, val, dtype):
    return W.CSR(n, n, rp.cpu().numpy(), col.cpu().numpy(), val.to(dtype).cpu().numpy())


def _opts(c, **kw):
    return rg.make_opts(value_dtype=c["dtype"], sigma=c.get("sigma", 1), tau=c.get("tau", -1), **kw)


# ----------------------------------------------------------------------------
# What a program holds, and one pass
# ----------------------------------------------------------------------------
def prepare(case, seed):
    c, kind, vt = case, case["kind"], _vdt(case)
    if kind == "batch":
        ns, rp, col, val = _batch(c, seed)
        rp, col, val = rp.cpu().numpy(), col.cpu().numpy(), val.to(vt).cpu().numpy()
        at = np.concatenate([[0], np.cumsum(ns)])
        mats = []
        for m, n in enumerate(ns):
            p = rp[at[m]:at[m + 1] + 1]
            mats.append(W.CSR(int(n), int(n), p - p[0], col[p[0]:p[-1]], val[p[0]:p[-1]]))
        A = rg.rgcsr_from_csr_batch(mats, opts=_opts(c))
        return dict(c=c, A=A, x=_vec(int(at[-1]), seed, 4, vt), y=torch.empty(int(at[-1]), dtype=vt, device=DEV))
    if kind == "cg":
        n, rp, col, val = _stencil("27pt", c["n"], seed)
        xs = _vec(n, seed, 4, torch.float64)
        b = _product(n, rp, col, val, xs)
        lo = rg.rgcsr_from_csr_device(n, n, rp, col, val.float(), rg.make_opts(value_dtype=c["dtype"]))
        hi = rg.rgcsr_from_csr_device(n, n, rp, col, val, rg.make_opts(value_dtype="f64"))
        return dict(c=c, lo=lo, hi=hi, b=b, n=n)
    n, rp, col, val = _matrix(c, seed)
    s = dict(c=c, n=n)
    if kind == "train":
        s["A"] = rg.rgcsr_from_csr(_host(n, rp, col, val, vt), opts=_opts(c, build_transpose=True))
        s["theta"] = val.to(vt).requires_grad_()
        s["x"] = _vec(n, seed, 4, vt).requires_grad_()
        s["dy"] = _vec(n, seed, 5, vt)
        s["fn"] = rg.spmv_function()
        return s
    s["x"] = _vec(n, seed, 4, vt, c.get("k"))
    if kind == "convert":
        s.update(rp=rp, col=col, val=val.to(vt), opts=_opts(c))
        return s
    if kind == "hyb":
        s["A"] = rg.hyb_from_csr(_host(n, rp, col, val, vt), value_dtype=c["dtype"])
    elif c.get("panels"):
        s["A"] = rg.rgcsr_from_csr(_host(n, rp, col, val, vt), opts=_opts(c, col_panels=c["panels"]))
    else:
        s["A"] = rg.rgcsr_from_csr_device(n, n, rp, col, val.to(vt), _opts(c))
    s["y"] = torch.empty_like(s["x"])
    return s


def run(state):
    s, kind = state, state["c"]["kind"]
    if kind in ("spmv", "batch"):
        rg.rgcsr_spmv(s["A"], s["x"], s["y"])
        return s["y"]
    if kind == "hyb":
        rg.hyb_spmv(s["A"], s["x"], s["y"])
        return s["y"]
    if kind == "spmm":
        rg.rgcsr_spmv_batched(s["A"], s["x"], s["y"])
        return s["y"]
    if kind == "train":
        y = s["fn"].apply(s["theta"], s["x"], s["A"])
        dtheta, dx = torch.autograd.grad(y, (s["theta"], s["x"]), s["dy"])
        return {"y": y.detach(), "dtheta": dtheta, "dx": dx}
    if kind == "cg":
        x = torch.zeros(s["n"], dtype=torch.float64, device=DEV)
        rg.rgcsr_cg_solve(s["lo"], s["hi"], s["b"], x, tol=1e-12)
        return x
    A = rg.rgcsr_from_csr_device(s["n"], s["n"], s["rp"], s["col"], s["val"], s["opts"])
    return A.spmv(s["x"])


# ----------------------------------------------------------------------------
# The same in 64 bits, and what a pass cannot do without
# ----------------------------------------------------------------------------
def _rows(rp):
    return torch.repeat_interleave(torch.arange(rp.numel() - 1, device=DEV), rp[1:] - rp[:-1])


def _product(n, rp, col, val, x):
    x = x.double()
    if x.dim() == 2:
        return torch.stack([_product(n, rp, col, val, x[:, j]) for j in range(x.shape[1])], 1)
    return torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, _rows(rp), val * x[col.long()])


def exact(case, seed):
    c, kind, vt = case, case["kind"], _vdt(case)
    if kind == "cg":
        return _vec(c["n"] ** 3, seed, 4, torch.float64)
    if kind == "batch":
        ns, rp, col, val = _batch(c, seed)
        n = int(ns.sum())
        first = torch.from_numpy(np.repeat(np.cumsum(ns) - ns, ns)).to(DEV)
        return _product(n, rp, col.long() + first[_rows(rp)], val.to(TORCH[c["dtype"]]).double(), _vec(n, seed, 4, vt))
    n, rp, col, val = _matrix(c, seed)
    val = val.to(vt).to(TORCH[c["dtype"]]).double()  # as stored
    x = _vec(n, seed, 4, vt, c.get("k"))
    if kind != "train":
        return _product(n, rp, col, val, x)
    dy, x = _vec(n, seed, 5, vt).double(), x.double()
    rows, cl = _rows(rp), col.long()
    dx = torch.zeros(n, dtype=torch.float64, device=DEV).index_add_(0, cl, val * dy[rows])
    return {"y": _product(n, rp, col, val, x), "dtheta": dy[rows] * x[cl], "dx": dx}


def _nnz(c):
    """Rows and (expected) nonzeros."""
    kind = c["kind"]
    if kind == "batch":
        rows = c["count"] * (20_000 - 100) / math.log(200)
        return rows, rows * 24.0
    family, n = ("27pt" if kind == "cg" else c["matrix"]), c["n"]
    if family == "5pt":
        return n ** 2, 5 * n ** 2 - 4 * n
    if family == "7pt":
        return n ** 3, 7 * n ** 3 - 6 * n ** 2
    if family == "27pt":
        return n ** 3, (3 * n - 2) ** 3
    if family == "zipf":
        cap = _cap(n)
        k = np.arange(1, cap + 1, dtype=np.float64)
        p = 6.0 / math.pi ** 2 / k ** 2
        return n, n * float((k * p).sum() + cap * (1.0 - p.sum()))
    return n, n * c["mean"]


def work(case):
    """Values, 32-bit columns and a row length per row; each vector once.
    A solve counts 100 inner steps: the matrix, ten vectors."""
    c, (rows, nnz), sv = case, _nnz(case), SIZE[case["dtype"]]
    sx = 8 if c["dtype"] == "f64" else 4
    if c["kind"] == "cg":
        return dict(bytes=100 * (nnz * (sv + 4) + rows * 4 * 11), flops=100 * (2 * nnz + 10 * rows))
    if c["kind"] == "train":
        return dict(bytes=nnz * (2 * sx + 4) + rows * (4 + 4 * sx), flops=5 * nnz)
    k = c.get("k", 1)
    return dict(bytes=nnz * (sv + 4) + rows * (4 + 2 * k * sx), flops=2 * nnz * k)
