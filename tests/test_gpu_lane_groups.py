"""MTTKRP at ranks where the lane groups have an edge: one to three columns, a
last lane that repeats its neighbour's columns, groups that leave lanes of the
wave over, one group to a wave."""
import pytest

from _gpu_helpers import factors_dev, mttkrp_error, to_dev
from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu

# A row sums at most a few hundred products of at most 6 factors in FP32:
# 300 terms x 2^-24 of the row's scale, and the products' own roundings.
TOL = 2e-5
DIMS = {2: (300, 170), 3: (61, 47, 83), 4: (40, 33, 57, 24), 5: (31, 29, 23, 26, 37), 6: (17, 19, 23, 18, 21, 20)}


@pytest.mark.parametrize("nmodes", sorted(DIMS))
@pytest.mark.parametrize("rank", [1, 2, 3, 4, 5, 7, 10, 21, 25, 50, 63, 65, 129, 255, 256])
def test_every_mode(nmodes, rank):
    from paper_2509_00280_amd import spt
    t = synth.distinct_coo(7 + nmodes, DIMS[nmodes], 5001, ["uniform"] * nmodes, "u01")
    F = synth.normal_factors(rank, t.dims, rank)
    Fd = factors_dev(F)
    c, v = to_dev(t)
    h = spt.encode(t.dims, c, v)
    for plan in (dict(), dict(row_cache=False), dict(tile=1024)):
        if plan:
            h.set_plan(**plan)
        for n in range(nmodes):
            err, bad = mttkrp_error(t, F, n, spt.mttkrp(h, Fd, n).cpu().numpy())
            assert bad == 0 and err <= TOL, (plan, n, err, bad)
    h.free()


@pytest.mark.parametrize("ranks", [(5, 64, 10, 25), (1, 3, 50, 7), (13, 13, 13, 13)])
def test_batch_of_mixed_ranks(ranks):
    import torch
    from paper_2509_00280_amd import spt
    hs, Fs, ts, Fh, outs = [], [], [], [], []
    for i, r in enumerate(ranks):
        nm = 3 + i % 3
        t = synth.distinct_coo(70 + i, DIMS[nm], 4500 + i, ["uniform"] * nm, "u01")
        F = synth.normal_factors(90 + i, t.dims, r)
        ts.append(t)
        Fh.append(F)
        Fs.append(factors_dev(F))
        c, v = to_dev(t)
        hs.append(spt.encode(t.dims, c, v))
    for mode in range(3):
        outs = [torch.empty((t.dims[mode], r), device="cuda") for t, r in zip(ts, ranks)]
        spt.mttkrp_batched(hs, Fs, mode, outs)
        for t, F, o in zip(ts, Fh, outs):
            err, bad = mttkrp_error(t, F, mode, o.cpu().numpy())
            assert bad == 0 and err <= TOL, (mode, err, bad)
    for h in hs:
        h.free()
