"""The SEGMENT walk where the runs of a tile and the lane groups' equal shares
meet: tiles of one run, runs of one nonzero, runs that begin and end inside a
share or go through several, an odd last position, one nonzero past a tile."""
import numpy as np
import pytest

import oracle
from _gpu_helpers import factors_dev, mttkrp_error, to_dev
from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu

# Rows of at most 8193 positive products: a tile's run is a chain of at most 32
# steps (rank 256: 4096 / 64 positions, two accumulators), 64 parts and 9
# records, each addition within 2^-24 (2^-53) of the row's scale.
TOL32 = 2 * (32 + 64 + 9 + 8) * 2.0**-24
TOL64 = 1e-12


def _tensor(rows, nnz, hot, seed):
    r = np.random.default_rng(seed)
    dims = (rows, 61, 47)
    c = np.stack([r.integers(0, d, nnz) for d in dims]).astype(np.uint32)
    c[0, r.random(nnz) < hot] = rows // 2
    return synth.SparseCOO(dims, c, r.random(nnz, dtype=np.float32))


@pytest.mark.parametrize("rank", [1, 3, 16, 64, 256])
@pytest.mark.parametrize("nnz", [1, 2, 63, 1023, 4095, 4096, 4097, 8193])
def test_runs_over_shares(rank, nnz):
    from paper_2509_00280_amd import spt
    for rows, hot in ((1, 0.0), (2, 0.0), (40, 0.6), (9000, 0.0), (9000, 0.97)):
        t = _tensor(rows, nnz, hot, rows + nnz)
        F = [np.abs(f) for f in synth.normal_factors(rank, t.dims, rank)]
        Fd = factors_dev(F)
        c, v = to_dev(t)
        h = spt.encode(t.dims, c, v)
        for plan in (dict(), dict(row_cache=False), dict(tile=1024)):
            if plan:
                h.set_plan(**plan)
            err, bad = mttkrp_error(t, F, 0, spt.mttkrp(h, Fd, 0).cpu().numpy())
            assert bad == 0 and err <= TOL32, (rows, hot, plan, err)
        h.free()


@pytest.mark.parametrize("rank", [1, 2, 127, 128, 129, 130, 255, 256])
@pytest.mark.parametrize("nnz", [1, 4095, 4097])
def test_fp64_ranks(rank, nnz):
    import torch
    from paper_2509_00280_amd import spt
    for rows, hot in ((1, 0.0), (300, 0.5)):
        t = _tensor(rows, nnz, hot, rank + nnz)
        rng = np.random.default_rng(rank)
        vals = rng.random(nnz)
        F = [rng.random((d, rank)) for d in t.dims]
        h = spt.encode(t.dims, *to_dev(t))
        spt.attach_f64(h, torch.from_numpy(vals).cuda())
        out = spt.mttkrp_f64(h, [torch.from_numpy(f).cuda() for f in F], 0).cpu().numpy()
        ref = oracle.mttkrp_f64vals(t.coords, vals, t.dims, F, 0)
        err, bad = oracle.row_error(out, ref, ref)
        assert bad == 0 and err <= TOL64, (rows, hot, err)
        h.free()
