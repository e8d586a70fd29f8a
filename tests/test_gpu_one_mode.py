"""Tensors of one mode: the product over the other modes is empty, so a row of
the MTTKRP is the sum of the row's values in every column."""
import numpy as np
import pytest

import oracle
from _gpu_helpers import factors_dev, mttkrp_error, to_dev
from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu

# A row is a sum of at most 2500 positive values; in whatever order they are added,
# that is within 2499 roundings of its size.
TOL = 2500 * 2.0**-24


def _tensor(rows, nnz):
    r = np.random.default_rng(rows + nnz)
    return synth.SparseCOO((rows,), r.integers(0, rows, (1, nnz)).astype(np.uint32), r.random(nnz, dtype=np.float32))


@pytest.mark.parametrize("rank", [1, 3, 16, 64, 256])
@pytest.mark.parametrize("rows,nnz", [(1, 1), (2, 4097), (7, 5000), (5000, 4095), (300_000, 9001)])
def test_mttkrp(rank, rows, nnz):
    import torch
    from paper_2509_00280_amd import spt
    t = _tensor(rows, nnz)
    F = synth.normal_factors(rank, t.dims, rank)
    Fd = factors_dev(F)
    h = spt.encode(t.dims, *to_dev(t))
    for plan in (dict(), dict(tile=1024)):
        if plan:
            h.set_plan(**plan)
        for call in (spt.mttkrp, lambda *a: spt.mttkrp_noalloc(*a, torch.full((rows, rank), np.nan, device="cuda"))):
            err, bad = mttkrp_error(t, F, 0, call(h, Fd, 0).cpu().numpy())
            assert bad == 0 and err <= TOL, (plan, err, bad)
    v = np.random.default_rng(rank).random(nnz)
    spt.attach_f64(h, torch.from_numpy(v).cuda())
    out = spt.mttkrp_f64(h, [f.double() for f in Fd], 0).cpu().numpy()
    ref = oracle.mttkrp_f64vals(t.coords, v, t.dims, [f.astype(np.float64) for f in F], 0)
    err, bad = oracle.row_error(out, ref, ref)
    assert bad == 0 and err <= 1e-12, (err, bad)
    h.free()


@pytest.mark.parametrize("others", [0, 2, 4])
def test_in_a_batch(others):
    """Alone, beside tensors of two modes, and beside tensors of two and six (the kernel of up to 8 modes)."""
    import torch
    from paper_2509_00280_amd import spt
    dims = [(40,), (5000,)] + [(40, 30), (40, 30), (9, 8, 7, 6, 5, 4), (9, 8, 7, 6, 5, 4)][:others]
    ranks = [16, 64, 3, 8, 25, 1]
    ts, hs, Fh, Fd, outs = [], [], [], [], []
    for i, d in enumerate(dims):
        t = synth.distinct_coo(i, d, 500, ["uniform"] * len(d), "u01") if len(d) > 1 else _tensor(d[0], 4500 + i)
        ts.append(t)
        Fh.append(synth.normal_factors(20 + i, d, ranks[i]))
        Fd.append(factors_dev(Fh[-1]))
        hs.append(spt.encode(d, *to_dev(t)))
        outs.append(torch.full((d[0], ranks[i]), np.nan, device="cuda"))
    spt.mttkrp_batched(hs, Fd, 0, outs)
    for t, F, o in zip(ts, Fh, outs):
        err, bad = mttkrp_error(t, F, 0, o.cpu().numpy())
        assert bad == 0 and err <= TOL, (t.dims, err, bad)


def test_rank_one_model():
    """The model of one mode is the row sums themselves: weight and factor their norm and direction, fit 1."""
    import torch
    from paper_2509_00280_amd import spt
    r = np.random.default_rng(5)
    t = synth.SparseCOO((6000,), r.permutation(6000)[None, :4500].astype(np.uint32), r.random(4500, dtype=np.float32))
    ref = oracle.cp_als(t.coords, t.vals, t.dims, [np.ones((6000, 1), np.float32)], iters=2)
    h = spt.encode(t.dims, *to_dev(t))
    F = [[torch.ones((6000, 1), device="cuda")] for _ in range(2)]
    lam, fit, _ = spt.cp_als(h, F[0], 2)
    lams, fits, _ = spt.cp_als_batched([h], [F[1]], 2)
    for l, f, x in ((lam, fit, F[0][0]), (lams[0], fits[0], F[1][0])):
        # each entry is one value, rounded to FP32 twice
        assert abs(float(l[0]) - ref["lam"][0]) <= 1e-6 * ref["lam"][0]
        assert np.abs(x.cpu().numpy() - ref["factors"][0]).max() <= 1e-6
        # the repository's criterion for fits: with nothing left over, the fit is 1 - sqrt of
        # the roundings of the factor's squares
        assert abs(f - 1.0) <= 1e-4
    h.free()
