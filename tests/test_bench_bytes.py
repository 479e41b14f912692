"""CPU checks of bench.py's byte accounting: a kernel label is billed for what
the library's present route moves, and not for launches with nothing to do."""
from types import SimpleNamespace

import pytest

import bench
import gen


def _pipe(depth=14, mode=gen.KEY_MORTON, n=10_000_000, tune_build=None, tune_proj=None):
    return SimpleNamespace(g=gen.Grid((0.0, 0.0, 0.0), 1.0, depth, mode), na=n, nb=n, nm=2 * n,
                           tune_build=tune_build, tune_proj=tune_proj)


COUNTS = [9_900_000, 9_900_000, 19_800_000, 18_000_000, 18_100_000, 18_200_000]


def test_tiles_and_buckets_bill_no_sort():
    p = _pipe()
    bill = lambda label: bench.algorithmic_bytes(label, p, COUNTS)
    assert bill("onesweep") == 0 and bill("rle") == 0
    assert bill("bucket_sort") == 8 * 20_000_000 + 12 * 19_800_000
    um, ups = COUNTS[2], COUNTS[3:]
    assert bill("rekey") == 3 * 8 * um
    assert bill("project_tiles") == 3 * 8 * um + 16 * sum(ups)


@pytest.mark.parametrize("kw", [dict(mode=gen.KEY_LINEAR), dict(depth=15), dict(n=400_000),
                                dict(tune_proj=(7, 32))])
def test_projections_by_the_sort_are_billed(kw):
    p = _pipe(**kw)
    um, ups = COUNTS[2], COUNTS[3:]
    passes = -(-2 * p.g.depth // 8)
    assert bench.algorithmic_bytes("project_tiles", p, COUNTS) is None
    assert bench.algorithmic_bytes("onesweep", p, COUNTS) == 3 * passes * 8 * um
    assert bench.algorithmic_bytes("rle", p, COUNTS) == sum(4 * um + 8 * up for up in ups)
    assert bench.algorithmic_bytes("rekey", p, COUNTS) == 3 * 12 * um


def test_builds_by_the_sort_are_billed():
    p = _pipe(n=13_000_000)  # above the bucket rule's end
    assert bench.algorithmic_bytes("bucket_sort", p, COUNTS) is None
    passes = -(-42 // 8)
    assert bench.algorithmic_bytes("onesweep", p, COUNTS) == passes * 16 * 26_000_000
