"""The sum of a run that many lane groups of a tile share: the longest chains of
additions that the SEGMENT walk makes, on values that round the same way at
every one of them."""
import numpy as np
import pytest

from _gpu_helpers import to_dev
from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu


def _shape(rank, tile, cols, step):
    """Groups of a wave and waves of a tile's workgroup, and the positions that a group takes
    (cols columns to a lane, step positions at a time)."""
    lanes = -(-rank // cols) if rank >= cols else rank
    per_wave, waves = 64 // lanes, tile // 256
    each = -(-tile // (per_wave * waves))
    return per_wave, waves, -(-each // step) * step


def _bound(rank, tile, cols, step):
    """Additions between a product and its run's sum: a group's steps (a sum for each position of
    a step, then those), the groups of a wave by halves, the waves one after the other."""
    per_wave, waves, each = _shape(rank, tile, cols, step)
    return each // step + step - 1 + int(np.ceil(np.log2(per_wave))) + 1 + waves


def _one_row(nmodes, rank, tile, mantissa, cols, step):
    """A tile of one row, factors of ones, and a value that adds 0.49 of the last place of the full
    sum with every group's part: a chain over the parts loses as much at each of them."""
    each = _shape(rank, tile, cols, step)[2]
    v = 1.0 + 0.49 * 2.0 ** (np.log2(tile) - 1 - mantissa) / each
    r = np.random.default_rng(rank)
    dims = (1,) + (9, 8, 7, 6, 5)[:nmodes - 1]
    c = np.stack([r.integers(0, d, tile) for d in dims]).astype(np.uint32)
    return dims, c, np.full(tile, v)


@pytest.mark.parametrize("rank", [1, 3, 4, 8, 10, 16, 25, 64, 128])
@pytest.mark.parametrize("nmodes", [1, 2, 3, 4, 5, 6])
def test_one_row(nmodes, rank):
    import torch
    from paper_2509_00280_amd import spt
    for tile in (1024, 2048) if nmodes == 6 else (1024, 4096):
        for cache in (False, True):
            step = 2 if nmodes <= 4 else 1
            dims, c, v = _one_row(nmodes, rank, tile, 23, 4 if rank >= 4 else 1, step)
            t = synth.SparseCOO(dims, c, v.astype(np.float32))
            h = spt.encode(dims, *to_dev(t))
            h.set_plan(tile=tile, row_cache=cache)
            out = spt.mttkrp(h, [torch.ones((d, rank), device="cuda") for d in dims], 0).cpu().numpy()
            exact = t.vals.astype(np.float64).sum()
            # and the rounding of the record itself
            tol = (_bound(rank, tile, 4 if rank >= 4 else 1, step) + 1) * 2.0**-24
            assert np.abs(out / exact - 1).max() <= tol, (tile, cache, out / exact - 1)
            h.free()


@pytest.mark.parametrize("rank", [1, 2, 4, 8, 10, 64, 128])
@pytest.mark.parametrize("nmodes", [1, 3, 4, 5])
def test_one_row_fp64(nmodes, rank):
    import torch
    from paper_2509_00280_amd import spt
    cols, step = (2 if rank >= 2 else 1), (2 if nmodes <= 4 else 1)
    tile = 4096
    dims, c, v = _one_row(nmodes, rank, tile, 52, cols, step)
    h = spt.encode(dims, *to_dev(synth.SparseCOO(dims, c, v.astype(np.float32))))
    spt.attach_f64(h, torch.from_numpy(v).cuda())
    ones = [torch.ones((d, rank), device="cuda", dtype=torch.float64) for d in dims]
    out = spt.mttkrp_f64(h, ones, 0).cpu().numpy().astype(np.longdouble)
    exact = np.longdouble(v[0]) * tile
    tol = (_bound(rank, tile, cols, step) + 1) * 2.0**-53
    assert np.abs(out / exact - 1).max() <= tol, out / exact - 1
    h.free()
