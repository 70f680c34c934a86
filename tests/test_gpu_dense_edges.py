"""Edges of the dense path: outputs and depths around the 128-wide tiles,
padding zeros, one part of k or several (a few output tiles with a long k),
accumulation into C, sparse C patterns, FP64 and FP32."""
import numpy as np
import pytest

from oracle import oracle as orc
from synth import BlockCSR, make_matrix, rng_of

from tests.helpers import check_against_oracle, gpu_multiply
from tests.test_launch_rules import dense_parts, rules  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def _cover(total, sizes, rng):
    out = []
    while sum(out) < total:
        out.append(min(int(rng.choice(sizes)), total - sum(out)))
    return np.asarray(out, np.int32)


def _parts(rules, m, n, k, dtype="f64", max_bytes=1 << 31):  # noqa: F811
    """What the library's rule makes of a product: (tiles in one piece, parts
    of k of the others)."""
    import torch
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    size, us = (8, 4.0) if dtype == "f64" else (4, 2.0)
    return dense_parts(rules, -(-m // 128) * -(-n // 128), -(-k // 16), slots, size * 128 * 128, max_bytes, us)[:2]


@pytest.mark.parametrize("beta", [0.0, -2.0])
@pytest.mark.parametrize("m,n,k", [(1, 1, 1), (127, 129, 15), (128, 128, 16), (129, 127, 17), (130, 250, 300),
                                   (64, 40, 2100), (257, 1, 513)])
def test_tile_edges_exact(m, n, k, beta):
    """Integer values: exact for any split of k."""
    rng = rng_of(m + n + k)
    rs, ks, ns = (_cover(x, [9, 22, 32], rng) for x in (m, k, n))
    A, B = make_matrix(rng, rs, ks, 1.0, "int"), make_matrix(rng, ks, ns, 1.0, "int")
    C = make_matrix(rng, rs, ns, 1.0, "int")
    X, st = gpu_multiply(3.0, A, B, beta, C, path="dense")
    assert st["path"] == 2
    check_against_oracle(X, orc.multiply(3.0, A, B, beta, C), 0.0)


@pytest.mark.parametrize("occ", [0.4, 1.0])
def test_split_k_into_blocks(rules, occ):  # noqa: F811
    """Nine tiles with a long k (split), absent blocks of A and B read as
    zero and a C that stores only the product's blocks."""
    rng = rng_of(int(10 * occ))
    rs, ks, ns = _cover(300, [5, 13, 23], rng), _cover(5000, [23, 32], rng), _cover(333, [5, 13, 23], rng)
    A, B = make_matrix(rng, rs, ks, occ * 0.05, "int"), make_matrix(rng, ks, ns, occ, "int")
    X, _ = gpu_multiply(1.0, A, B, 0.0, path="dense")
    assert _parts(rules, 300, 333, 5000)[1] >= 19  # (at least 16 k steps of 16 each)
    assert (len(X.col_ind) == len(rs) * len(ns)) == (occ == 1.0)
    check_against_oracle(X, orc.multiply(1.0, A, B, 0.0), 0.0)


@pytest.mark.parametrize("full", [True, False])
def test_last_round_in_parts(rules, full):  # noqa: F811
    """529 tiles: 512 of them whole, the last ones in parts of k.  A full C,
    and one that lacks blocks of the rows (columns) that A (B) stores nothing
    of, found through the map of its blocks."""
    rng = rng_of(4)
    rs, ks = _cover(23 * 128, [32], rng), _cover(300, [20], rng)
    A, B = make_matrix(rng, rs, ks, 1.0, "int"), make_matrix(rng, ks, rs, 1.0, "int")
    C = make_matrix(rng, rs, rs, 0.5, "int")
    if not full:
        nb, nk = len(rs), len(ks)
        rows, cols = np.arange(nb) % 3 != 1, np.arange(nb) % 4 != 2
        A = _only(A, np.repeat(rows, nk))
        B = _only(B, np.tile(cols, nk))
    X, st = gpu_multiply(1.0, A, B, 2.0, C, path="dense")
    whole, splits = _parts(rules, 23 * 128, 23 * 128, 300)
    assert st["path"] == 2 and whole == 512 and splits == 2
    assert (len(X.col_ind) == len(rs) ** 2) == full
    check_against_oracle(X, orc.multiply(1.0, A, B, 2.0, C), 0.0)


def _only(M, keep):
    """M with the stored blocks of `keep` alone."""
    rows = np.repeat(np.arange(len(M.rbs)), np.diff(M.row_ptr))
    sizes = np.asarray(M.rbs, np.int64)[rows] * np.asarray(M.cbs, np.int64)[M.col_ind]
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=len(M.rbs)))]).astype(np.int64)
    return BlockCSR(M.rbs, M.cbs, rp, M.col_ind[keep], M.data[np.repeat(keep, sizes)])


def test_split_k_f32(rules):  # noqa: F811
    from tests.test_gpu_f32 import _as_f32, _f32_multiply
    rng = rng_of(9)
    rs, ks = _cover(200, [22], rng), _cover(4000, [22], rng)
    A, B = make_matrix(rng, rs, ks, 1.0, "int"), make_matrix(rng, ks, rs, 1.0, "int")
    X, _ = _f32_multiply(1.0, _as_f32(A), _as_f32(B), 0.0, path="dense")
    assert _parts(rules, 200, 200, 4000, "f32")[1] >= 15
    check_against_oracle(X, orc.multiply(1.0, A, B, 0.0), 0.0)  # sums below 2^24: exact in FP32


def test_split_k_within_the_scratch_region(rules):  # noqa: F811
    """The allocation-free multiply of a long k: the parts of k shrink to
    what the scratch region of 64 MiB holds beside the panels."""
    from tests.helpers import lib, set_path
    rng = rng_of(12)
    rs, ks = _cover(256, [32], rng), _cover(14000, [32], rng)
    A, B = make_matrix(rng, rs, ks, 1.0, "int"), make_matrix(rng, ks, rs, 1.0, "int")
    left = (64 << 20) - 2 * 8 * 256 * 14000  # at most; the index arrays take some of it
    assert 2 < _parts(rules, 256, 256, 14000, max_bytes=left - (1 << 20))[1]
    assert _parts(rules, 256, 256, 14000, max_bytes=left)[1] < _parts(rules, 256, 256, 14000)[1]
    b = lib()
    set_path("dense")
    try:
        MA, MB = b.Matrix.from_blocks(A), b.Matrix.from_blocks(B)
        MC = b.Matrix.from_blocks(make_matrix(rng, rs, rs, 1.0, "zeros"))
        b.bsmm_multiply_noalloc(1.0, MA.handle, MB.handle, 0.0, MC.handle)
        X = MC.to_host()
        for M in (MA, MB, MC):
            M.close()
    finally:
        set_path()
    check_against_oracle(X, orc.multiply(1.0, A, B, 0.0), 0.0)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("m,n,k", [(130, 250, 33), (64, 40, 2100)])
def test_k_step_32(m, n, k, dtype):
    """The longer k step (also the way of FP64 panels whose columns lie too
    far apart for the short one's offsets), FP64 and FP32, exact."""
    from tests.helpers import lib
    from tests.test_gpu_f32 import _as_f32, _f32_multiply
    rng = rng_of(m * k)
    rs, ks, ns = (_cover(x, [9, 22, 32], rng) for x in (m, k, n))
    A, B = make_matrix(rng, rs, ks, 1.0, "int"), make_matrix(rng, ks, ns, 1.0, "int")
    lib().bsmm_set_option("dense_kb", "32")
    try:
        if dtype == "f64":
            X, _ = gpu_multiply(3.0, A, B, 0.0, path="dense")
        else:
            X, _ = _f32_multiply(3.0, _as_f32(A), _as_f32(B), 0.0, path="dense")
    finally:
        lib().bsmm_set_option("dense_kb", "16")
    check_against_oracle(X, orc.multiply(3.0, A, B, 0.0), 0.0)


@pytest.mark.parametrize("dtype", ["f64", "f32"])
def test_error_of_split_sums(rules, dtype):  # noqa: F811
    """210 tiles of 128 x 128: an element's sums are cut into parts of k no
    longer than two rounds of workgroups make them.  A chain of L sums of
    random terms, S of them added up, has the relative error
    c u sqrt((L + S) / 2): rounding to nearest of values spread evenly over
    their logarithm has c = 0.425.  Ten per cent above that is allowed (the
    23,040 sampled elements vary by less than one); two parts, which would be
    faster, show 57 % more."""
    import torch
    from tests.test_gpu_f32 import _as_f32, _f32_multiply
    m, n, k = 14 * 128, 15 * 128, 2304
    rng = rng_of(21)
    rs, ks, ns = _cover(m, [64], rng), _cover(k, [64], rng), _cover(n, [64], rng)
    A, B = make_matrix(rng, rs, ks, 1.0), make_matrix(rng, ks, ns, 1.0)
    if dtype == "f32":
        A, B = _as_f32(A), _as_f32(B)
        X, st = _f32_multiply(1.0, A, B, 0.0, path="dense")
    else:
        X, st = gpu_multiply(1.0, A, B, 0.0, path="dense")
    assert st["path"] == 2 and _parts(rules, m, n, k, dtype)[1] >= 5
    slots = 2 * torch.cuda.get_device_properties(0).multi_processor_count
    steps = k // 16
    S = min(-(-2 * slots // 210), steps // 16)
    L = 16 * -(-steps // S)
    rows = rng.choice(m, size=12, replace=False)
    T = orc.to_dense(A)[rows].astype(np.longdouble) @ orc.to_dense(B).astype(np.longdouble)
    D = orc.to_dense(X)[rows] - T
    err = float(np.linalg.norm(D.astype(np.float64)) / np.linalg.norm(T.astype(np.float64)))
    u = 2.0**-24 if dtype == "f32" else 2.0**-53
    assert err <= 1.1 * 0.425 * u * np.sqrt((L + S) / 2)
