"""Rules of the launches (host code, compiled here with the host compiler).
Parts of k of a dense product: every k step in one part, partial sums within
their bound, and no chain of sums longer than about two rounds of workgroups
make it.  Segments of a schedule: every XCD a like share of the runs."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SRC = """#include "launch_rules.h"
extern "C" void parts(int64_t tiles, int64_t ktiles, int64_t slots, int64_t tile_bytes, int64_t max_bytes,
                      double step_us, int64_t *out) {
    const bsmm::DenseParts d = bsmm::dense_parts(tiles, ktiles, slots, tile_bytes, max_bytes, step_us);
    out[0] = d.whole;
    out[1] = d.splits;
    out[2] = d.kt_per;
}
extern "C" int segment_bits(int64_t n) { return bsmm::schedule_segment_bits(n, 8); }
"""


def build_rules(d):
    (d / "rule.cpp").write_text(SRC)
    so = str(d / "rule.so")
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC",
                    "-I" + os.path.join(ROOT, "paper_1910_04796_amd", "csrc"), str(d / "rule.cpp"), "-o", so],
                   check=True)
    lib = ctypes.CDLL(so)
    lib.parts.argtypes = [ctypes.c_int64] * 5 + [ctypes.c_double, ctypes.POINTER(ctypes.c_int64)]
    lib.segment_bits.argtypes = [ctypes.c_int64]
    return lib


def dense_parts(rules, tiles, ktiles, slots, tile_bytes, max_bytes, step_us):
    """(tiles in one piece, parts of k of the others, k steps of a part)"""
    out = (ctypes.c_int64 * 3)()
    rules.parts(tiles, ktiles, slots, tile_bytes, max_bytes, step_us, out)
    return tuple(out)


@pytest.fixture(scope="module")
def rules(tmp_path_factory):
    return build_rules(tmp_path_factory.mktemp("launch_rules"))


def _cases():
    rng = random.Random(7)
    yield from [(1, 1), (1, 15), (1, 16), (1, 31), (1, 32), (1, 15625), (4, 15625), (210, 144), (255, 144), (256, 144),
                (511, 512), (512, 512), (513, 512), (529, 182), (1023, 64), (1024, 64), (4096, 512)]
    for _ in range(400):
        yield int(2 ** rng.uniform(0, 13)), int(2 ** rng.uniform(0, 15))


@pytest.mark.parametrize("tile_bytes,step_us,slots", [(131072, 4.0, 512), (65536, 2.0, 512), (131072, 4.0, 256)])
@pytest.mark.parametrize("max_bytes", [0, 64 << 20, 1 << 31])
def test_parts_cover_k_and_are_never_too_long(rules, max_bytes, tile_bytes, step_us, slots):
    for tiles, ktiles in _cases():
        whole, splits, per = dense_parts(rules, tiles, ktiles, slots, tile_bytes, max_bytes, step_us)
        case = (tiles, ktiles, whole, splits, per)
        assert 0 <= whole <= tiles and splits >= 1, case
        assert (whole == tiles) == (splits == 1), case
        assert (splits - 1) * per < ktiles <= splits * per, case  # every step once, no empty part
        if splits > 1:
            assert (tiles - whole) * splits * tile_bytes <= max_bytes, case
            assert per >= 8, case
        if whole:
            assert splits == 1 or whole % slots == 0, case
        # The longest chain of sums: that of about two rounds of workgroups of
        # at least 16 steps, unless the partial sums have no room.
        if tiles < slots:
            want = max(1, min(-(-2 * slots // tiles), ktiles // 16, max_bytes // (tiles * tile_bytes)))
            assert (ktiles if whole else per) <= -(-ktiles // want), case


def test_segments_share_the_runs(rules):
    """Segment after segment goes to the next XCD: no XCD has more than an
    eighth of the runs and one segment, and a segment is a small part of that
    share unless it is the smallest there is."""
    rng = random.Random(8)
    sizes = [1, 3, 4, 5, 9, 31, 32, 33, 144, 196, 255, 256, 257, 900, 4096, 4225, 16383, 16384, 10**6, 10**9]
    for n in sizes + [int(2 ** rng.uniform(0, 30)) for _ in range(300)]:
        seg = 1 << rules.segment_bits(n)
        assert 4 <= seg <= 256, n
        assert seg == 4 or n // seg >= 64, n
        assert seg == 256 or n // seg < 130, n
        full, last = divmod(n, seg)
        share = [((full - x + 7) // 8) * seg + (last if full % 8 == x else 0) for x in range(8)]
        assert sum(share) == n and max(share) <= n // 8 + seg, n
