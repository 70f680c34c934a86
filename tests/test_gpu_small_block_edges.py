"""Edges of the small-block MFMA kernel's tiles and of the passes around it:
block sides on both sides of the 8-, 16- and 32-wide tiles, products one
deep to beyond two chunks, B read in place and from row-major copies, blocks
moved between layouts in pieces, norms of neighbouring blocks of very
different magnitude."""
import numpy as np
import pytest

from oracle import oracle as orc
from synth import BlockCSR, make_matrix, rng_of

from tests.helpers import check_against_oracle, gpu_multiply, lib, set_path

pytestmark = pytest.mark.gpu


def _matrices(seed, rs, ks, ns, occ, values="uniform"):
    rng = rng_of(seed)
    return make_matrix(rng, rs, ks, occ, values), make_matrix(rng, ks, ns, occ, values)


@pytest.mark.parametrize("kernel", ["plain", "tuned"])
@pytest.mark.parametrize("sizes", [[7, 8, 9], [15, 16, 17], [1, 31, 32, 33], [47, 48, 49], [63, 64, 2]])
def test_tile_edges(sizes, kernel):
    """Integer values: exact whatever the order of the sums."""
    rng = rng_of(len(sizes) + sizes[0])
    rs, ks, ns = (rng.choice(sizes, size=9).astype(np.int32) for _ in range(3))
    A, B = _matrices(sizes[0], rs, ks, ns, 0.6, "int")
    Cin = make_matrix(rng, rs, ns, 0.3, "int")
    X, _ = gpu_multiply(2.0, A, B, -1.0, Cin, path="stack", kernel=kernel)
    check_against_oracle(X, orc.multiply(2.0, A, B, -1.0, Cin), 0.0)


@pytest.mark.parametrize("k", [1, 2, 3, 7, 8, 9, 15, 16, 17, 24, 25, 40])
def test_product_depths(k):
    """Uniform 13- and 23-sided blocks, every product k deep."""
    rng = rng_of(k)
    rs = rng.choice([13, 23], size=10).astype(np.int32)
    A, B = _matrices(k + 100, rs, np.full(12, k, np.int32), rs, 0.7, "int")
    X, _ = gpu_multiply(1.0, A, B, 0.0, path="stack", kernel="tuned")
    check_against_oracle(X, orc.multiply(1.0, A, B, 0.0), 0.0)


@pytest.mark.parametrize("sched", ["static", "dynamic"])
@pytest.mark.parametrize("tile", [1, 32, 200])
@pytest.mark.parametrize("depth,occ", [(1, 1.0), (2, 1.0), (9, 0.8)])
def test_schedule_segments(depth, occ, tile, sched):
    """Schedules of several segments per XCD with an incomplete last one,
    runs taken four, two and one at a time: every C block is written once."""
    rng = rng_of(depth)
    rs, ns = (rng.choice([5, 13, 20], size=s).astype(np.int32) for s in (163, 171))
    A, B = _matrices(depth + 200, rs, np.full(depth, 3, np.int32), ns, occ, "int")
    Cin = make_matrix(rng, rs, ns, 0.2, "int")
    b = lib()
    saved = {k: b.bsmm_get_option(k) for k in ("stack_tile", "stack_sched", "stack_params")}
    b.bsmm_set_option("stack_tile", str(tile))
    b.bsmm_set_option("stack_sched", sched)
    b.bsmm_set_option("stack_params", "16 16 0 4")
    try:
        X, st = gpu_multiply(1.0, A, B, -2.0, Cin, path="stack", kernel="tuned")
    finally:
        for k, v in saved.items():
            b.bsmm_set_option(k, v)
    assert st["n_sched_runs"] > 16 * 256 and st["n_sched_runs"] % 256
    check_against_oracle(X, orc.multiply(1.0, A, B, -2.0, Cin), 0.0)


@pytest.mark.parametrize("at", ["auto", "0", "1"])
@pytest.mark.parametrize("blocks", [70, 20])
@pytest.mark.parametrize("depths", [[1, 7], [8, 13], [5, 23, 24]])
def test_infinities_stay_in_their_rows_and_columns(depths, blocks, at):
    """Infinities anywhere in the blocks reach only the elements of C that
    their rows and columns stand for: values read past a row, a column or the
    depth of a block never do.  One launch (70 x 70 C blocks) and one per
    class, A and B read in place and from row-major copies."""
    rng = rng_of(blocks + depths[0])
    rs = rng.choice([9, 16, 17, 23], size=blocks).astype(np.int32)
    A, B = _matrices(depths[-1], rs, np.asarray(depths, np.int32), rs, 1.0, "int")
    for M, v in ((A, np.inf), (B, -np.inf)):
        M.data[rng.random(M.data.size) < 0.003] = v
    b = lib()
    saved = {k: b.bsmm_get_option(k) for k in ("stack_at", "stack_params")}
    b.bsmm_set_option("stack_at", at)
    b.bsmm_set_option("stack_params", "16 16 0 4")
    try:
        X, st = gpu_multiply(1.0, A, B, 0.0, path="stack", kernel="tuned")
    finally:
        for k, v in saved.items():
            b.bsmm_set_option(k, v)
    assert (st["n_sched_runs"] > 0) == (blocks == 70)
    with np.errstate(invalid="ignore"):
        R = orc.multiply(1.0, A, B, 0.0)
    assert 0.02 < np.isfinite(R.data).mean() < 1.0
    check_against_oracle(X, R, 0.0)


@pytest.mark.parametrize("at", ["0", "1"])
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("k", [1, 3, 5, 7, 9])
def test_first_values_stay_in_their_row_and_column(k, dtype, at):
    """Infinities in the first values of every block of A (the row-major copy
    then begins with row 0) and of B (column 0): lanes whose values of k lie
    past a product's depth must not read them, so only row 0 and column 0 of
    every block of C are not finite."""
    from tests.test_gpu_f32 import _as_f32, _f32_multiply
    rng = rng_of(k)
    rs = rng.choice([9, 16, 17, 23], size=70).astype(np.int32)
    A, B = _matrices(k + 400, rs, np.array([k], np.int32), rs, 1.0, "int")
    A.data[np.cumsum(rs * k) - rs * k] = np.inf
    B.data[np.cumsum(rs * k) - rs * k] = np.inf
    A.data[A.data == 0.0] = 1.0  # (0 x infinity)
    B.data[B.data == 0.0] = 1.0
    b = lib()
    saved = {k: b.bsmm_get_option(k) for k in ("stack_at", "stack_params")}
    b.bsmm_set_option("stack_at", at)
    b.bsmm_set_option("stack_params", "16 16 0 4")
    try:
        if dtype == "f64":
            X, st = gpu_multiply(1.0, A, B, 0.0, path="stack", kernel="tuned")
        else:
            X, st = _f32_multiply(1.0, _as_f32(A), _as_f32(B), 0.0, path="stack", kernel="tuned",
                                 params="16 16 0 4")
    finally:
        for key, v in saved.items():
            b.bsmm_set_option(key, v)
    assert st["n_sched_runs"] > 4096
    with np.errstate(invalid="ignore"):
        R = orc.multiply(1.0, A, B, 0.0)
    first = np.cumsum(rs) - rs
    inner = np.setdiff1d(np.arange(rs.sum()), first)
    assert np.isfinite(orc.to_dense(X)[np.ix_(inner, inner)]).all()
    check_against_oracle(X, R, 0.0)


@pytest.mark.parametrize("nk", [1, 31, 32, 33, 65])
@pytest.mark.parametrize("nbc", [5, 4000, 4001])
def test_product_lists(nk, nbc):
    """Rows of A with as many blocks as one pass over them holds, one less,
    one more and beyond two passes; C with the most block columns of the
    list kernel for short rows and one more: exact, and K ascending (with
    values whose sum depends on the order: the same bits as one product after
    the other)."""
    rng = rng_of(nk + nbc)
    rs, ks, ns = np.array([2, 1, 3], np.int32), np.full(nk, 1, np.int32), np.full(nbc, 1, np.int32)
    A, B = make_matrix(rng, rs, ks, 1.0), make_matrix(rng, ks, ns, 0.7 if nbc < 100 else 0.02)
    A.data[:] = 1.0
    B.data[:] = rng.choice([2.0**53, 1.0, -(2.0**53), 3.0], size=B.data.size)
    X, _ = gpu_multiply(1.0, A, B, 0.0, path="stack")
    D, want = orc.to_dense(B), np.zeros(nbc)
    for k in range(nk):
        want = want + D[k]
    assert np.array_equal(orc.to_dense(X), np.tile(want, (6, 1)))


def test_copied_b_same_bits():
    """Enough products per B block for row-major copies of B: the same bits
    as reading both operands in place (stack_at "1" keeps B in place), and a
    replayed plan copies B's new values."""
    rng = rng_of(5)
    # Two sizes, so that every shape class holds more runs than are split.
    rs, ks = (np.repeat([13, 23], 70).astype(np.int32), rng.choice([5, 17, 32], size=110).astype(np.int32))
    A, B = _matrices(6, rs, ks, rs, 0.6)
    b = lib()
    out = {}
    try:
        for at in ("0", "1"):
            b.bsmm_set_option("stack_at", at)
            out[at] = gpu_multiply(1.5, A, B, 0.0, path="stack", kernel="tuned")
    finally:
        b.bsmm_set_option("stack_at", "auto")
    assert out["0"][1]["n_sched_runs"] > 4096
    assert out["0"][1]["n_products"] >= 48 * len(B.col_ind)
    check_against_oracle(out["0"][0], out["1"][0], 0.0)
    check_against_oracle(out["0"][0], orc.multiply(1.5, A, B, 0.0), 1e-13)
    b.bsmm_set_option("plan_cache", "1")
    set_path("stack", "tuned")
    try:
        MA, MB, MC = b.Matrix.from_blocks(A), b.Matrix.from_blocks(B), b.Matrix.empty(A.rbs, B.cbs)
        b.multiply(1.0, MA, MB, 0.0, MC)
        E1, E2 = b.Matrix.empty(B.rbs, B.rbs), b.Matrix.empty(B.rbs, B.cbs)
        b.multiply(1.0, E1, E2, 2.0, MB)  # B <- 2 B in place
        b.multiply(1.0, MA, MB, 0.0, MC)
        X = MC.to_host()
        for M in (MA, MB, MC, E1, E2):
            M.close()
    finally:
        b.bsmm_set_option("plan_cache", "0")
        set_path()
    check_against_oracle(X, orc.multiply(2.0, A, B, 0.0), 1e-13)


@pytest.mark.parametrize("sizes", [[1], [1, 2, 3], [5, 13], [23, 32, 64]])
def test_moved_blocks(sizes):
    """A filter that drops single blocks and stretches of them, the packed
    read-out, and old blocks moved into a grown pattern."""
    rng = rng_of(sum(sizes))
    rs = rng.choice(sizes, size=40).astype(np.int32)
    one = np.ones(40, np.int32)
    A = make_matrix(rng, rs, one, 0.5)
    B = make_matrix(rng, one, rs, 0.5)
    # Columns of small values: their blocks of C fall below the filter.
    scale = np.where(rng.random(40) < 0.5, 1e-12, 1.0)
    ne = np.repeat(B.col_ind, np.asarray(rs)[B.col_ind])
    B = BlockCSR(B.rbs, B.cbs, B.row_ptr, B.col_ind, B.data * scale[ne])
    b = lib()
    set_path("stack", "tuned")
    try:
        MA, MB, MC = b.Matrix.from_blocks(A), b.Matrix.from_blocks(B), b.Matrix.empty(rs, rs)
        b.multiply(1.0, MA, MB, 0.0, MC, 1e-9)
        X = MC.to_host()
        R = orc.multiply(1.0, A, B, 0.0, filter_eps=1e-9)
        check_against_oracle(X, R, 1e-13)
        b.multiply(1.0, MA, MB, 1.0, MC)
        Y = MC.to_host()
        for M in (MA, MB, MC):
            M.close()
    finally:
        set_path()
    check_against_oracle(Y, orc.multiply(1.0, A, B, 1.0, R), 1e-13)


def test_screen_norms_of_mixed_neighbours():
    """Blocks whose squares overflow, underflow or are ordinary side by side
    (also zero and NaN ones): the screened multiply gives the unscreened
    one's blocks bit for bit."""
    rng = rng_of(77)
    sizes = rng.choice([1, 5, 13, 23], size=24).astype(np.int32)
    A, B = _matrices(78, sizes, sizes, sizes, 0.5)
    per_block = np.asarray(sizes, np.int64)[np.repeat(np.arange(24), np.diff(A.row_ptr))] * sizes[A.col_ind]
    mag = rng.choice([1e-200, 1e-160, 1e-12, 1.0, 0.0, 1e170], size=len(per_block))
    A = BlockCSR(A.rbs, A.cbs, A.row_ptr, A.col_ind, A.data * np.repeat(mag, per_block))
    A.data[int(per_block[:7].sum())] = np.nan
    b = lib()
    out = []
    try:
        for on in ("1", "0"):
            b.bsmm_set_option("prescreen", on)
            out.append(gpu_multiply(1.0, A, B, 0.0, eps=1e-9, path="stack", kernel="tuned")[0])
    finally:
        b.bsmm_set_option("prescreen", "1")
    check_against_oracle(out[0], out[1], 0.0)


@pytest.mark.parametrize("nb,sizes", [(1, [23]), (7, [5, 13, 23, 32]), (60, [3, 8, 17]), (90, [4, 9]),
                                      (92, [4, 9]), (40, list(range(1, 9)))])
def test_classified_stacks(nb, sizes):
    """Stacks of a small C (classified by one workgroup, up to 8,192 blocks
    and 64 classes) and of larger ones: every product once, runs by class and
    C block, K ascending."""
    rng = rng_of(nb)
    rs, ks = rng.choice(sizes, size=nb).astype(np.int32), rng.choice([2, 7], size=nb + 1).astype(np.int32)
    A, B = _matrices(nb + 1, rs, ks, rs, 0.5)
    b = lib()
    set_path("stack", "plain")
    try:
        MA, MB = b.Matrix.from_blocks(A), b.Matrix.from_blocks(B)
        MC = b.Matrix.from_blocks(make_matrix(rng, rs, rs, 0.2, "zeros"))  # also blocks without products
        b.multiply(1.0, MA, MB, 1.0, MC)
        X = MC.to_host()
        st = b.bsmm_inspect_stacks(MA.handle, MB.handle, MC.handle)
        for M in (MA, MB, MC):
            M.close()
    finally:
        set_path()
    a_rows = np.repeat(np.arange(nb), np.diff(A.row_ptr))
    c_rows = np.repeat(np.arange(nb), np.diff(X.row_ptr))
    b_rows = np.repeat(np.arange(nb + 1), np.diff(B.row_ptr))
    want = {(I, K, J) for I, K in zip(a_rows, A.col_ind) for J in B.col_ind[B.row_ptr[K]:B.row_ptr[K + 1]]}
    got = set()
    for r, c in enumerate(st["run_cblk"]):
        p = slice(st["run_ptr"][r], st["run_ptr"][r + 1])
        K = A.col_ind[st["prod_ablk"][p]]
        assert len(K) > 0 and np.all(np.diff(K) > 0)
        assert np.all(a_rows[st["prod_ablk"][p]] == c_rows[c]) and np.all(b_rows[st["prod_bblk"][p]] == K)
        assert np.all(B.col_ind[st["prod_bblk"][p]] == X.col_ind[c])
        got |= {(c_rows[c], k, X.col_ind[c]) for k in K}
    assert got == want and sum(np.diff(st["run_ptr"])) == len(want)
    order = list(zip(st["run_class"], st["run_cblk"]))
    assert order == sorted(order)


def test_threads_and_streams_read_back_their_own_counts():
    """Four host threads, each with its own handles and stream: every
    multiply sees the pattern sizes and class counts of its own product."""
    import threading

    import torch
    b = lib()
    set_path("stack", "plain")
    jobs = []
    for t in range(4):
        rng = rng_of(500 + t)
        rs, ks = rng.choice([5, 13, 23][: t % 3 + 1], size=10 + 7 * t).astype(np.int32), np.full(9 + t, 8, np.int32)
        A, B = _matrices(600 + t, rs, ks, rs, 0.3 + 0.1 * t)
        jobs.append((A, B, orc.multiply(1.0, A, B, 0.0, filter_eps=1e-3 if t == 3 else 0.0), 1e-3 if t == 3 else 0.0))
    failed = []

    def work(A, B, R, eps):
        try:
            stream = torch.cuda.Stream()
            MA, MB = b.Matrix.from_blocks(A, stream=stream), b.Matrix.from_blocks(B, stream=stream)
            for _ in range(8):
                MC = b.Matrix.empty(A.rbs, B.cbs, stream=stream)
                for _ in range(3):
                    b.multiply(1.0, MA, MB, 0.0, MC, eps, stream=stream)
                check_against_oracle(MC.to_host(stream=stream), R, 1e-13)
                MC.close()
            MA.close()
            MB.close()
        except Exception as e:  # noqa: BLE001 - reported by the main thread
            failed.append(repr(e))

    try:
        threads = [threading.Thread(target=work, args=j) for j in jobs]
        for t in threads:
            t.start()
        for t in threads:
            t.join()
    finally:
        set_path()
    assert not failed, failed


@pytest.mark.parametrize("k", [1, 4, 7, 8, 9, 23, 32])
def test_copied_b_f32(k):
    """FP32 with enough products per B block for row-major copies of B: the
    same bits as with both operands in place (stack_at "1"), and the exact
    product of whole numbers."""
    from tests.test_gpu_f32 import _as_f32, _f32_multiply
    rng = rng_of(k)
    rs = rng.choice([6, 14, 22, 31], size=70).astype(np.int32)
    A, B = _matrices(k + 300, rs, np.full(7, k, np.int32), rs, 0.9, "int")
    b = lib()
    out = {}
    try:
        for at in ("0", "1"):
            b.bsmm_set_option("stack_at", at)
            out[at] = _f32_multiply(1.0, _as_f32(A), _as_f32(B), 0.0, path="stack", kernel="tuned",
                                    params="16 16 0 4")
    finally:
        b.bsmm_set_option("stack_at", "auto")
    assert out["0"][1]["n_sched_runs"] > 4096 and out["0"][1]["n_products"] >= 48 * len(B.col_ind)
    check_against_oracle(out["0"][0], out["1"][0], 0.0)
    check_against_oracle(out["0"][0], orc.multiply(1.0, A, B, 0.0), 0.0)


# (C block side, depth of the products): blocks of A and B on both sides of
# the 1,024 elements that one turn through LDS holds, with an odd and an even
# number of rows.
@pytest.mark.parametrize("dtype", ["f64", "f32"])
@pytest.mark.parametrize("n,k", [(32, 32), (32, 33), (31, 33), (31, 35), (23, 44), (23, 45), (23, 46), (22, 47),
                                 (16, 64), (16, 65), (13, 79), (13, 80), (13, 200)])
def test_copied_blocks_of_any_size(n, k, dtype):
    """Row-major copies of blocks deeper than wide, of B (the rule on products
    per B block) and of A (option "stack_at"): the exact product of whole
    numbers."""
    from tests.test_gpu_f32 import _as_f32, _f32_multiply
    rs = np.full(70, n, np.int32)
    A, B = _matrices(n * k, rs, np.full(2, k, np.int32), rs, 0.97, "int")
    R = orc.multiply(1.0, A, B, 0.0)
    b = lib()
    try:
        for at in ("auto", "1"):
            b.bsmm_set_option("stack_at", at)
            if dtype == "f64":
                X, st = gpu_multiply(1.0, A, B, 0.0, path="stack")
            else:
                X, st = _f32_multiply(1.0, _as_f32(A), _as_f32(B), 0.0, path="stack")
            assert st["n_sched_runs"] > 4096 and st["n_products"] >= 48 * len(B.col_ind)
            check_against_oracle(X, R, 0.0)
    finally:
        b.bsmm_set_option("stack_at", "auto")


@pytest.mark.parametrize("kernel", ["plain", "tuned"])
@pytest.mark.parametrize("nb", [3, 4, 8, 40])
@pytest.mark.parametrize("sizes,one_launch", [([5, 23], False), ([5, 13, 23], True), ([6, 14, 22, 30], True)])
def test_few_runs_of_many_classes(sizes, one_launch, nb, kernel):
    """Fewer runs than the scheduled launch asks for: in a plan it takes them
    all the same when they are of more than six classes.  Integer values: exact."""
    nb = max(nb, len(sizes))
    rs = np.resize(np.array(sizes, np.int32), nb)
    A, B = _matrices(nb + 300, rs, rs, rs, 1.0 if nb < 8 else 0.4, "int")
    Cin = make_matrix(rng_of(nb), rs, rs, 0.3, "int")
    b = lib()
    saved = {k: b.bsmm_get_option(k) for k in ("stack_params", "plan_cache")}
    b.bsmm_set_option("stack_params", "16 16 0 4")
    b.bsmm_set_option("plan_cache", "1")
    try:
        X, st = gpu_multiply(2.0, A, B, -1.0, Cin, path="stack", kernel=kernel)
    finally:
        for k, v in saved.items():
            b.bsmm_set_option(k, v)
    assert (st["n_sched_runs"] > 0) == one_launch
    check_against_oracle(X, orc.multiply(2.0, A, B, -1.0, Cin), 0.0)


class RefusingAllocator:
    """Device memory from torch's caching allocator, except requests of
    `least` bytes up to an eighth more (the library rounds sizes up)."""

    def __init__(self):
        import torch
        self.dev = torch.cuda.current_device()
        self.least, self.refused, self.sizes = None, 0, []

    def alloc(self, nbytes, stream):
        import torch
        if self.least and self.least <= nbytes <= self.least + self.least // 8 + 4096:
            self.refused += 1
            return 0
        self.sizes.append(nbytes)
        return torch.cuda.caching_allocator_alloc(nbytes, self.dev, stream if stream else None)

    def dealloc(self, ptr, nbytes, stream):
        import torch
        torch.cuda.caching_allocator_delete(ptr)


@pytest.mark.parametrize("panels", [False, True])
@pytest.mark.parametrize("plan", ["0", "1"])
def test_no_room_for_the_copy_of_b(plan, panels):
    """A product whose copy of B finds no memory reads B in place: the same
    blocks, whether C grows in the call, a plan is kept or C is made in
    several row panels."""
    rng = rng_of(91)
    rs = np.full(70 if not panels else 210, 13, np.int32)
    A, B = _matrices(92, rs, np.full(2, 200, np.int32), rs, 0.97, "int")
    R = orc.multiply(1.0, A, B, 0.0)
    b, ra = lib(), RefusingAllocator()
    b.bsmm_set_allocator(ra.alloc, ra.dealloc)
    saved = {k: b.bsmm_get_option(k) for k in ("plan_cache", "stack_panel")}
    set_path("stack")
    try:
        b.bsmm_set_option("plan_cache", plan)
        if panels:
            b.bsmm_set_option("stack_panel", str(len(R.col_ind)))  # of two products per C block
        MA, MB, MC = b.Matrix.from_blocks(A), b.Matrix.from_blocks(B), b.Matrix.empty(A.rbs, B.cbs)
        ra.least = 8 * (B.data.size + 1)
        for _ in range(2):
            b.multiply(1.0, MA, MB, 0.0, MC)
            st = b.bsmm_last_stats()
            check_against_oracle(MC.to_host(), R, 0.0)
        for M in (MA, MB, MC):
            M.close()
    finally:
        for k, v in saved.items():
            b.bsmm_set_option(k, v)
        set_path()
        b.bsmm_set_allocator()
    assert st["n_sched_runs"] > 4096 and ra.refused > 0
    assert (st["n_row_panels"] > 1) == panels


@pytest.mark.parametrize("nk", [4, 12])
@pytest.mark.parametrize("nbc", [8160, 8161, 8192, 8193, 32736, 32737, 40000])
def test_counts_of_wide_rows(nbc, nk):
    """C rows whose bitmap has fewer words than a workgroup has threads, as
    many and more (256 threads, 1,024 for a few long rows of A), with blocks of
    different widths: blocks, elements, products and flops counted right."""
    rng = rng_of(nbc + nk)
    rs, ks = np.array([2, 1, 3], np.int32), np.full(nk, 2, np.int32)
    ns = rng.choice([1, 2, 5], size=nbc).astype(np.int32)
    A, B = _matrices(nbc, rs, ks, ns, 1.0, "int")
    keep = rng.random(len(B.col_ind)) < 0.01
    keep[[0, nbc - 1]] = True
    rows = np.repeat(np.arange(nk), np.diff(B.row_ptr))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows[keep], minlength=nk))]).astype(np.int64)
    B = BlockCSR(B.rbs, B.cbs, rp, B.col_ind[keep], B.data[np.repeat(keep, 2 * ns[B.col_ind])])
    X, st = gpu_multiply(1.0, A, B, 0.0, path="stack")
    check_against_oracle(X, orc.multiply(1.0, A, B, 0.0), 0.0)
    assert st["n_products"] == 3 * len(B.col_ind) and st["flops"] == 2.0 * 6 * 2 * ns[B.col_ind].sum()
