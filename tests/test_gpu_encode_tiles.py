"""The radix sort of the encoder at the edges of its tiles and of the rule that
chooses them, for one-word and two-word keys; digits with one value, keys
without bits, equal keys (the sort is stable)."""
import numpy as np
import pytest

from _gpu_helpers import check_encoding, to_dev
from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu

LARGE = 4 << 20  # nonzeros from which the larger tiles are used
SHAPES = {
    "one word": (3000, 700, 41),
    "whole word": (1 << 24, 1 << 22, 1 << 18),
    "two words": (1 << 25, 1 << 20, 300000, 731),
    "no bits": (1, 1, 1),
    "one digit of many": (1 << 16, 1, 1),
}


def _tensor(dims, nnz, seed):
    r = np.random.default_rng(seed)
    c = np.stack([np.minimum(r.integers(0, d, nnz), r.integers(0, d, nnz)) for d in dims]).astype(np.uint32)
    c[:, : nnz // 3] = c[:, :1]  # many equal keys
    return synth.SparseCOO(dims, c, r.standard_normal(nnz).astype(np.float32))


def _check(dims, nnz, seed):
    from paper_2509_00280_amd import spt
    t = _tensor(dims, nnz, seed)
    c, v = to_dev(t)
    h = spt.encode(t.dims, c, v)
    check_encoding(h, t)
    h.free()


@pytest.mark.parametrize("shape", sorted(SHAPES))
@pytest.mark.parametrize("nnz", [1, 63, 64, 65, 2047, 2048, 2049, 70_001, 1_100_003])
def test_small_tiles(shape, nnz):
    _check(SHAPES[shape], nnz, nnz)


@pytest.mark.parametrize("shape", ["one word", "two words"])
@pytest.mark.parametrize("nnz", [LARGE - 1, LARGE, LARGE + 4095, LARGE + 8193])
def test_rule_of_the_tiles(shape, nnz):
    _check(SHAPES[shape], nnz, nnz)


@pytest.mark.parametrize("nnz", [2049, LARGE + 1])
def test_out_of_range_is_named(nnz):
    """The first offending nonzero and its mode, whichever tile it is in."""
    from paper_2509_00280_amd import spt
    t = _tensor(SHAPES["one word"], nnz, 3)
    t.coords[1, nnz - 1] = 700
    t.coords[2, nnz // 2] = 41
    c, v = to_dev(t)
    with pytest.raises(spt.SptError, match=rf"2 coordinate\(s\) out of range; first at nonzero {nnz // 2}, mode 2"):
        spt.encode(t.dims, c, v)
