"""The multiplies whose speed this repository is held to.

A case is one C <- filter_eps(beta*C + alpha*A*B) through the public entry
points, as a program that keeps A, B and C as handles calls it, followed by
the read-out of C's block data into a device tensor (bsmm_copy_out_typed).
Three families cover the range of the benchmarks and tests:

* ``sparse``: square block grids with every block position stored with
  probability ``occ``; one block size or a mix of sizes; U[-1,1] values;
* ``banded``: the same with magnitudes decaying as exp(-|I-J|/50) and blocks
  whose magnitude envelope lies below 1e-10 not stored (the headline
  benchmark's matrices), results filtered at ``eps``;
* ``dense``: every block stored (densified products), square or
  tall-and-skinny, native or emulated on INT8 matrix cores.

Sizes: 460 x 460 in 23-blocks, N = 50,000 in {5,13,23,32}-blocks at 1, 10
and 30 %, N = 8192 in 32-blocks and 1,408 x 1,408 x long K are the
benchmark's own workloads; the others lie between them.
"""
import ctypes

import numpy as np
import torch

from paper_1910_04796_amd import bsmm

DECAY, CUTOFF = 50.0, 1e-10
TORCH_DTYPE = {"f64": torch.float64, "f32": torch.float32}


def _case(name=None, **kw):
    c = dict(family="sparse", m=0, n=0, k=0, sizes="23", occ=1.0, dtype="f64", path="auto", kernel="plain",
             plan=False, entry="multiply", beta=0.0, eps=0.0)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    n50 = dict(family="banded", m=50000, n=50000, k=50000, sizes="5,13,23,32", eps=1e-10)
    return [
        # One small block-sparse product with the library's default options:
        # launches and host work are all there is.
        _case("sparse460_default", m=460, n=460, k=460, occ=0.10),
        # The same product repeated on a fixed pattern with its plan kept
        # (an iterative solver's inner loop), accumulating into C.
        _case("sparse460_plan", m=460, n=460, k=460, occ=0.10, kernel="tuned", plan=True, beta=1.0),
        # A medium product of a mid-size molecule's matrices, accumulating,
        # default options.
        _case("sparse3000_default", m=3000, n=3000, k=3000, sizes="5,13,23", occ=0.25, beta=1.0),
        # Uniform 23-blocks at 20 %: half-filled matrices of one atom kind.
        _case("sparse8000_b23", m=8000, n=8000, k=8000, occ=0.20, kernel="tuned"),
        # The headline family from very sparse to its largest member:
        # linear-scaling matrix functions, results filtered.
        _case("banded_1pct", occ=0.01, kernel="tuned", **n50),
        _case("banded_10pct", occ=0.10, kernel="tuned", **n50),
        _case("banded_30pct", occ=0.30, kernel="tuned", **n50),
        # Single precision, block sizes that the tuning database lacks.
        _case("banded_10pct_f32", family="banded", m=24000, n=24000, k=24000, sizes="6,14,22,30", occ=0.10,
              dtype="f32", kernel="tuned", eps=1e-6),
        # Fully occupied inputs, which the library densifies: the
        # benchmark's square product, and an accumulating ragged one.
        _case("dense8192_b32", family="dense", m=8192, n=8192, k=8192, sizes="32"),
        _case("dense1900_ragged", family="dense", m=1900, n=1700, k=2300, sizes="5,13,22", beta=1.0),
        # The same square product by split-precision emulation.
        _case("dense8192_emul", family="dense", m=8192, n=8192, k=8192, sizes="32", path="emul"),
        # Tall-and-skinny (an eighth of the paper's K), blocks of 22.
        _case("tall_k247808", family="dense", m=1408, n=1408, k=247808, sizes="22"),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["small", "sparse", "banded", "dense", "emul", "tall"])
    mixes = ["5,13,23,32", "6,14,22,30", "5,13,23", "23", "13", "32", "22"]
    kernel = rng.choice(["plain", "tuned"])
    if kind == "small":
        m, n, k = (_log(rng, 150, 1500) for _ in range(3))
        entry, plan = rng.choice([("multiply", False), ("multiply", True), ("noalloc", False)])
        return _case(m=m, n=n, k=k, sizes=rng.choice(mixes), occ=round(rng.uniform(0.05, 0.4), 3), kernel=kernel,
                     plan=plan, entry=entry, beta=rng.choice([0.0, 1.0]), dtype=rng.choice(["f64", "f64", "f32"]))
    if kind == "sparse":
        m, n, k = (_log(rng, 2000, 12000) for _ in range(3))
        return _case(m=m, n=n, k=k, sizes=rng.choice(mixes), occ=round(_log(rng, 20, 300) / 1000, 3), kernel=kernel,
                     beta=rng.choice([0.0, 1.0]), dtype=rng.choice(["f64", "f64", "f32"]))
    if kind == "banded":
        n = _log(rng, 4000, 40000)
        f32 = rng.random() < 0.25
        return _case(family="banded", m=n, n=n, k=n, sizes=rng.choice(mixes[:3]), occ=round(_log(rng, 10, 300) / 1000, 3),
                     kernel="tuned", dtype="f32" if f32 else "f64", eps=1e-6 if f32 else 1e-10)
    if kind == "dense":
        m, n, k = (_log(rng, 200, 8192) for _ in range(3))
        return _case(family="dense", m=m, n=n, k=k, sizes=rng.choice(mixes + ["64", "4"]), beta=rng.choice([0.0, 1.0]),
                     dtype=rng.choice(["f64", "f64", "f32"]))
    if kind == "emul":
        m, n, k = (_log(rng, 400, 8192) for _ in range(3))
        return _case(family="dense", m=m, n=n, k=k, sizes=rng.choice(mixes), path="emul", beta=rng.choice([0.0, 1.0]))
    return _case(family="dense", m=_log(rng, 200, 1500), n=_log(rng, 200, 1500), k=_log(rng, 20000, 250000),
                 sizes=rng.choice(["22", "64", "23", "32"]))


# ------------------------------------------------------------- patterns
def _sizes(rng, total, sizes):
    """Block sizes drawn from the case's mix until they reach `total`."""
    choice = np.array([int(x) for x in sizes.split(",")], np.int32)
    if len(choice) == 1:
        return np.full(max(1, total // int(choice[0])), choice[0], np.int32)
    b = choice[rng.integers(0, len(choice), size=2 * total // int(choice.min()) + 2)]
    return b[:int(np.searchsorted(np.cumsum(b), total)) + 1].astype(np.int32)


def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _inputs(case, seed):
    """Block sizes and, for A and B, the stored positions as a boolean grid
    (the structure, which is the case's own), and the generator of the
    values."""
    rng = np.random.default_rng([case["m"], case["n"], case["k"], int(1e6 * case["occ"])])
    rs = _sizes(rng, case["m"], case["sizes"])
    if case["family"] == "banded":
        ks = ns = rs
    else:
        ks, ns = _sizes(rng, case["k"], case["sizes"]), _sizes(rng, case["n"], case["sizes"])
    pattern = torch.Generator(device=_device()).manual_seed(int(rng.integers(1 << 31)))
    masks = []
    for r, c in ((rs, ks), (ks, ns)):
        if case["family"] == "dense":
            mask = torch.ones((len(r), len(c)), dtype=torch.bool, device=_device())
        else:
            mask = torch.rand((len(r), len(c)), generator=pattern, device=_device()) < case["occ"]
        if case["family"] == "banded":
            d = torch.arange(len(r), device=_device(), dtype=torch.float64)
            sz = torch.as_tensor(r, device=_device()).double()
            env = torch.exp(-(d[:, None] - d[None, :]).abs() / DECAY) * torch.sqrt(sz[:, None] * sz[None, :])
            mask &= env >= CUTOFF
        masks.append(mask)
    # The blocks of C before the filter: an accumulating case starts from a
    # tenth of the positions (a dense one from all of them).
    old = torch.zeros((len(rs), len(ns)), dtype=torch.bool, device=_device())
    if case["beta"] != 0.0:
        old = torch.rand((len(rs), len(ns)), generator=pattern, device=_device()) < (
            2.0 if case["family"] == "dense" else 0.1)
    return rs, ks, ns, masks, old, torch.Generator(device=_device()).manual_seed(int(seed) + 1)


def _product_pattern(masks, old):
    return ((masks[0].float() @ masks[1].float()) > 0) | old


class _Pattern:
    """Block-CSR index of a boolean grid, and where each block's data lie."""

    def __init__(self, rs, cs, mask):
        self.rs, self.cs = rs, cs
        dev = mask.device
        self.rows, self.cols = (x.contiguous() for x in mask.nonzero(as_tuple=True))
        self.row_ptr = np.concatenate([[0], np.cumsum(mask.sum(dim=1).cpu().numpy())]).astype(np.int64)
        self.col_ind = self.cols.cpu().numpy().astype(np.int32)
        self.m = torch.as_tensor(rs, device=dev).long()[self.rows]
        self.n = torch.as_tensor(cs, device=dev).long()[self.cols]
        self.off = torch.cumsum(self.m * self.n, 0) - self.m * self.n
        self.nelems = int((self.m * self.n).sum())
        self.r0 = torch.as_tensor(np.cumsum(rs) - rs, device=dev).long()[self.rows]
        self.c0 = torch.as_tensor(np.cumsum(cs) - cs, device=dev).long()[self.cols]

    def values(self, case, gen):
        dev = self.m.device
        v = torch.empty(self.nelems, dtype=torch.float64, device=dev)
        v.uniform_(-1.0, 1.0, generator=gen)
        if case["family"] == "banded":
            scale = torch.exp(-(self.rows - self.cols).abs().double() / DECAY)
            v *= torch.repeat_interleave(scale, self.m * self.n, output_size=self.nelems)
        return v.to(TORCH_DTYPE[case["dtype"]])

    def pieces(self):
        """(data positions [b, n, m], rows [b, 1, m], columns [b, n, 1]) of
        blocks of one shape, at most 2^25 elements at a time."""
        dev = self.m.device
        for m in sorted(set(int(x) for x in self.rs)):
            for n in sorted(set(int(x) for x in self.cs)):
                idx = ((self.m == m) & (self.n == n)).nonzero().flatten()
                step = max(1, (1 << 25) // (m * n))
                for b in range(0, len(idx), step):
                    i = idx[b:b + step]
                    pos = self.off[i][:, None, None] + torch.arange(m * n, device=dev).view(1, n, m)
                    yield (pos, self.r0[i][:, None, None] + torch.arange(m, device=dev).view(1, 1, m),
                           self.c0[i][:, None, None] + torch.arange(n, device=dev).view(1, n, 1))

    def dense(self, values):
        d = torch.zeros((int(self.rs.sum()), int(self.cs.sum())), dtype=torch.float64, device=values.device)
        for pos, r, c in self.pieces():
            d[r, c] = values[pos].double()
        return d

    def gather(self, dense):
        v = torch.empty(self.nelems, dtype=torch.float64, device=dense.device)
        for pos, r, c in self.pieces():
            v[pos] = dense[r, c]
        return v


def _matrix(pat, values, dtype):
    h = bsmm.bsmm_create_matrix(len(pat.rs), pat.rs, len(pat.cs), pat.cs, len(pat.col_ind), pat.row_ptr, pat.col_ind,
                                values, dtype=dtype)
    return bsmm.Matrix(h, pat.rs, pat.cs, dtype)


# ---------------------------------------------------------------- the case
def prepare(case, seed):
    bsmm.use_torch_allocator()
    for key, value in (("path", case["path"]), ("stack_kernel", case["kernel"]), ("plan_cache", int(case["plan"]))):
        bsmm.bsmm_set_option(key, value)
    rs, ks, ns, masks, old, gen = _inputs(case, seed)
    mats = []
    for r, c, mask in ((rs, ks, masks[0]), (ks, ns, masks[1])):
        pat = _Pattern(r, c, mask)
        mats.append(_matrix(pat, pat.values(case, gen), case["dtype"]))
    if case["beta"] != 0.0:
        pat = _Pattern(rs, ns, old)
        C = _matrix(pat, pat.values(dict(case, family="sparse"), gen), case["dtype"])
    else:
        C = bsmm.Matrix.empty(rs, ns, dtype=case["dtype"])
    if case["entry"] == "noalloc":
        # That entry point takes a C that already holds the pattern.
        bsmm.multiply(0.0, mats[0], mats[1], 1.0, C)
    # The read-out buffer holds every block that the product can have; what
    # a filter leaves of them fills its front.
    m, n = (torch.as_tensor(x, device=_device()).double() for x in (rs, ns))
    most = int(m @ (_product_pattern(masks, old).double() @ n))
    out = torch.zeros(most, dtype=TORCH_DTYPE[case["dtype"]], device="cuda")
    return {"A": mats[0], "B": mats[1], "C": C, "out": out, "case": case, "lib": ctypes.CDLL(bsmm.LIB_PATH)}


def run(state):
    case, C = state["case"], state["C"]
    if case["entry"] == "noalloc":
        bsmm.bsmm_multiply_noalloc(1.0, state["A"].handle, state["B"].handle, case["beta"], C.handle)
    else:
        bsmm.multiply(1.0, state["A"], state["B"], case["beta"], C, case["eps"])
    _, _, nnzb, nelems = C.info()
    if nelems > state["out"].numel():
        raise ValueError("C holds more than the product's blocks")
    status = state["lib"].bsmm_copy_out_typed(
        ctypes.c_void_p(C.handle), None, None, ctypes.c_void_p(state["out"].data_ptr()), 1,
        ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
    if status != 0:
        raise bsmm.BsmmError(status, bsmm.bsmm_last_error())
    return {"data": state["out"], "blocks": nnzb, "elements": nelems}


def work(case):
    """A, B (and an accumulated C) read once, C written once; 2 m n k per
    block product."""
    rs, ks, ns, (ma, mb), old, _ = _inputs(case, 0)
    e = 4.0 if case["dtype"] == "f32" else 8.0
    dev = ma.device
    m, k, n = (torch.as_tensor(x, device=dev).double() for x in (rs, ks, ns))
    am, bn = ma.double().T @ m, mb.double() @ n
    nbytes = float(k @ am) + float(k @ bn)
    hit = _product_pattern((ma, mb), old)
    nbytes += float(m @ (old.double() @ n))
    if case["eps"] > 0.0:
        # Blocks of the product that the filter drops are not written: keep
        # those whose expected squared norm reaches eps^2.
        d = torch.arange(len(rs), device=dev, dtype=torch.float64)
        env = torch.exp(-2.0 * (d[:, None] - d[None, :]).abs() / DECAY) / 3.0
        norm2 = ((ma * env) * k) @ (mb * env)
        hit &= norm2 * m[:, None] * n[None, :] >= case["eps"] ** 2
    nbytes += float(m @ (hit.double() @ n))
    return {"bytes": e * nbytes, "flops": 2.0 * float(torch.sum(k * am * bn))}


def tolerance(case):
    # Measured against `exact`, times about four: FP64 1.6e-16 to 4.4e-16
    # (sparse), 1.7e-15 (dense), 1.7e-14 (dense, k = 247,808); emulation
    # 1.1e-14; FP32 2.2e-7 (sparse), 3.0e-7 (dense, k up to 8192).
    if case["path"] == "emul":
        return {"rel": 5e-14}
    if case["dtype"] == "f32":
        return {"rel": 2e-6 if case["family"] == "dense" else 1e-6}
    if case["family"] == "dense":
        return {"rel": 8e-14 if case["k"] > 20000 else 1e-14}
    return {"rel": 2e-15}


def exact(case, seed):
    rs, ks, ns, masks, old, gen = _inputs(case, seed)
    dense = []
    for r, c, mask in ((rs, ks, masks[0]), (ks, ns, masks[1])):
        pat = _Pattern(r, c, mask)
        dense.append(pat.dense(pat.values(case, gen)))
    X = dense[0] @ dense[1]
    del dense
    hit = _product_pattern(masks, old)
    m, n = (torch.as_tensor(x, device=X.device) for x in (rs, ns))
    most = int(m.double() @ (hit.double() @ n.double()))
    if case["beta"] != 0.0:
        pat = _Pattern(rs, ns, old)
        X += case["beta"] * pat.dense(pat.values(dict(case, family="sparse"), gen))
    if case["eps"] > 0.0:
        # Squared block norms, then the blocks that the filter keeps.
        rb = torch.repeat_interleave(torch.arange(len(rs), device=X.device), m.long())
        cb = torch.repeat_interleave(torch.arange(len(ns), device=X.device), n.long())
        n1 = torch.zeros((len(rs), X.shape[1]), dtype=torch.float64, device=X.device)
        for i in range(0, X.shape[0], 4096):
            n1.index_add_(0, rb[i:i + 4096], X[i:i + 4096].square())
        n2 = torch.zeros((len(rs), len(ns)), dtype=torch.float64, device=X.device)
        n2.index_add_(1, cb, n1)
        hit &= n2 >= case["eps"] ** 2
    data = _Pattern(rs, ns, hit).gather(X)
    return {"data": torch.nn.functional.pad(data, (0, most - data.numel())), "blocks": None, "elements": None}
