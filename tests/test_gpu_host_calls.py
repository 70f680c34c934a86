"""Which HIP host calls a multiply makes, seen from a library that stands
before the HIP runtime in a child process: graphs are built for launches that
are worth one, and counts are read back where page-locked memory is refused."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

HOOK = r"""
#include <dlfcn.h>
#include <stddef.h>
int graphs_built = 0;
int hipGraphInstantiate(void **exec, void *graph, void *node, char *log, size_t len) {
    static int (*real)(void **, void *, void *, char *, size_t);
    if (!real) real = dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD), "hipGraphInstantiate");
    ++graphs_built;
    return real(exec, graph, node, log, len);
}
int refuse_pinned = 0, refused = 0;
int hipHostMalloc(void **p, size_t bytes, unsigned flags) {
    static int (*real)(void **, size_t, unsigned);
    if (!real) real = dlsym(dlopen("libamdhip64.so.7", RTLD_LAZY | RTLD_NOLOAD), "hipHostMalloc");
    if (refuse_pinned && bytes == 32768) {  /* the library's own buffers */
        ++refused;
        return 2; /* hipErrorOutOfMemory */
    }
    return real(p, bytes, flags);
}
"""

CHILD = """
import ctypes, sys
hook = ctypes.CDLL(sys.argv[1], mode=ctypes.RTLD_GLOBAL)
import numpy as np
from oracle import oracle as orc
from synth import make_matrix, rng_of
from tests.helpers import check_against_oracle, gpu_multiply, lib
count = ctypes.c_int.in_dll(hook, "graphs_built")
"""


def _run(tmp_path, body):
    (tmp_path / "hook.c").write_text(HOOK)
    so = str(tmp_path / "hook.so")
    subprocess.run(["gcc", "-shared", "-fPIC", "-O1", str(tmp_path / "hook.c"), "-o", so, "-ldl"], check=True)
    (tmp_path / "child.py").write_text(CHILD + body)
    r = subprocess.run([sys.executable, str(tmp_path / "child.py"), so], cwd=ROOT, capture_output=True, text=True,
                       timeout=100, env=dict(os.environ, PYTHONPATH=os.pathsep.join(filter(None, (
                           ROOT, os.environ.get("PYTHONPATH"))))))
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


def test_graph_without_a_plan_for_long_launches_only(tmp_path):
    """Tuned classes that keep a launch each, no plan: long runs of few blocks
    above 64 on a side go into a graph, short ones and short small blocks one
    by one; the product is exact either way."""
    _run(tmp_path, """
for sizes, nk, nb, graph in (([65, 70], 12, 8, 1), ([65, 70], 1, 8, 0), ([65], 12, 8, 0), ([5, 13], 12, 8, 0),
                             ([33, 40, 48, 64], 40, 8, 1), ([33, 40, 48, 64], 2, 8, 0), (list(range(1, 25)), 1, 24, 0)):
    rs, ks = np.resize(np.array(sizes, np.int32), nb), np.full(nk, 32, np.int32)
    rng = rng_of(nk + nb)
    A, B = make_matrix(rng, rs, ks, 1.0, "int"), make_matrix(rng, ks, rs, 1.0, "int")
    before = count.value
    X, st = gpu_multiply(1.0, A, B, 0.0, path="stack", kernel="tuned")
    print(sizes, nk, nb, count.value - before, flush=True)
    assert count.value - before == graph, (sizes, nk, nb)
    check_against_oracle(X, orc.multiply(1.0, A, B, 0.0), 0.0)
""")


def test_counts_without_page_locked_memory(tmp_path):
    """Multiplies that get no page-locked memory read their counts through
    device memory: few and many rows, filtered and screened, a plan, several
    row panels; page-locked memory again once there is some."""
    _run(tmp_path, """
refuse = ctypes.c_int.in_dll(hook, "refuse_pinned")
refused = ctypes.c_int.in_dll(hook, "refused")
b = lib()
def case(seed, nb, eps, **options):
    rng = rng_of(seed)
    rs = rng.choice([3, 5, 8], size=nb).astype(np.int32)
    A, B = make_matrix(rng, rs, rs, min(1.0, 6.0 / nb), "int"), make_matrix(rng, rs, rs, min(1.0, 6.0 / nb), "int")
    saved = {k: b.bsmm_get_option(k) for k in options}
    for k, v in options.items():
        b.bsmm_set_option(k, v)
    try:
        X, _ = gpu_multiply(2.0, A, B, 0.0, eps=eps, path="stack", repeat=2)
    finally:
        for k, v in saved.items():
            b.bsmm_set_option(k, v)
    check_against_oracle(X, orc.multiply(2.0, A, B, 0.0, filter_eps=eps), 0.0)
for on in (1, 0):
    refuse.value = on
    for nb in (4, 200, 1500):
        for eps in (0.0, 100.0):
            before = refused.value
            case(nb, nb, eps)
            assert (refused.value > before) == bool(on), (nb, eps)
            print(on, nb, eps, refused.value, flush=True)
    case(5, 60, 0.0, plan_cache="1")
    case(6, 60, 0.0, stack_panel="300")
""")
