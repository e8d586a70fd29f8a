"""CP-ALS without a tolerance, whose iterations are read back in groups: what it
returns is the last iteration's, bit for bit that of a run that looks at each."""
import numpy as np
import pytest

import oracle
from _gpu_helpers import factors_dev, to_dev
from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("iters", [1, 2, 31, 32, 33, 64, 65])
def test_same_as_with_a_readback_each(iters):
    """Both runs do the same operations on one plan, with too few records for atomic additions (one
    workgroup sums them all), so they agree in every bit."""
    import torch
    from paper_2509_00280_amd import spt
    t = synth.distinct_coo(5, (60, 50, 40), 6000, ["uniform"] * 3, "u01")
    init = [(np.abs(f) + 0.1).astype(np.float32) for f in synth.normal_factors(3, t.dims, 4)]
    h = spt.encode(t.dims, *to_dev(t))
    got = []
    for tol in (0.0, 1e-300):
        F = factors_dev(init)
        lam, fit, n = spt.cp_als(h, F, iters, tol=tol)
        assert n == iters
        got.append((fit, lam, F))
    assert got[0][0] == got[1][0]
    assert torch.equal(got[0][1], got[1][1])
    assert all(torch.equal(a, b) for a, b in zip(got[0][2], got[1][2]))
    h.free()


@pytest.mark.parametrize("iters", [2, 3, 10, 31, 32])
def test_direct_residual_of_the_last_iteration(iters):
    """A fit above 0.99 is the residual over the nonzeros plus what the model holds elsewhere, which
    takes the last iteration's |Xhat|^2: it is that of the returned model, and the first iteration's
    |Xhat|^2 would have shown."""
    from paper_2509_00280_amd import spt
    dims, R = (30, 20, 10), 4
    rng = np.random.default_rng(iters)
    true = [rng.random((d, R)) + 0.1 for d in dims]
    X = np.einsum("ir,jr,kr->ijk", *true)
    X *= 1.0 + 0.004 * rng.standard_normal(dims)
    # the six smallest cells are left out: the model has mass off the support
    X[X < np.quantile(X, 0.001)] = 0.0
    coords = np.stack(np.nonzero(X)).astype(np.uint32)
    t = synth.SparseCOO(dims, coords, X[tuple(coords)].astype(np.float32))
    init = [(f * (1.0 + 0.1 * rng.standard_normal(f.shape))).astype(np.float32) for f in true]
    h = spt.encode(t.dims, *to_dev(t))
    F = factors_dev(init)
    lam, fit, n = spt.cp_als(h, F, iters)
    h.free()
    assert n == iters and fit > 0.99
    dense = np.zeros(dims)
    dense[tuple(coords)] = t.vals

    def model(lam, F):
        return np.einsum("r,ir,jr,kr->ijk", lam, *[f.astype(np.float64) for f in F])

    xhat = model(lam.cpu().numpy(), [f.cpu().numpy() for f in F])
    norm = np.linalg.norm(dense)
    exact = 1.0 - np.linalg.norm(dense - xhat) / norm
    # |Xhat|^2 is that of the factors before they were rounded to FP32: 3 x 2 roundings
    tol = 6 * 2.0**-24 / (2 * (1.0 - exact))
    assert abs(fit - exact) <= tol, (fit, exact)
    first = oracle.cp_als(t.coords, t.vals, dims, init, iters=1)
    on = dense != 0
    off = np.linalg.norm(model(first["lam"], first["factors"])) ** 2 - (xhat[on] ** 2).sum()
    mistaken = 1.0 - np.sqrt(((dense - xhat)[on] ** 2).sum() + max(off, 0.0)) / norm
    assert abs(mistaken - exact) > 10 * tol
