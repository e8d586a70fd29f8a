"""CP-ALS without a tolerance, which does not wait for an iteration before it starts
the next: what it returns is the last iteration's, bit for bit that of a run that
looks at each, and a solve that fails ends the call soon."""
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


@pytest.mark.parametrize("tol", [0.0, 1e-300])
def test_a_failed_solve_ends_the_call(tol):
    """The first solve is refused: at most one iteration is under way beyond it, of 100 asked for."""
    import torch
    from paper_2509_00280_amd import spt
    t = synth.distinct_coo(6, (60, 50, 40), 6000, ["uniform"] * 3, "u01")
    h = spt.encode(t.dims, *to_dev(t))
    F = factors_dev([np.full((d, 4), np.nan, np.float32) for d in t.dims])
    F[2] = torch.ones_like(F[2])
    h.prepare(4)
    spt.profile_reset(True)
    with pytest.raises(spt.SptError, match="mode 0 not positive definite"):
        spt.cp_als(h, F, 100, tol=tol)
    calls = spt.profile_read()["mttkrp_launches"][:3]
    spt.lib().spt_profile_enable(0)
    assert max(calls) <= 2, calls
    assert torch.equal(F[2], torch.ones_like(F[2])) and torch.isnan(F[0]).all()
    h.free()


def test_calls_of_several_threads():
    """Each call has its own reports: the same models as one call after the other."""
    import threading
    import torch
    from paper_2509_00280_amd import spt
    ts = [synth.distinct_coo(20 + i, (60 + i, 50, 40), 5000, ["uniform"] * 3, "u01") for i in range(6)]
    hs = [spt.encode(t.dims, *to_dev(t)) for t in ts]
    init = [[(np.abs(f) + 0.1).astype(np.float32) for f in synth.normal_factors(i, t.dims, 4)] for i, t in enumerate(ts)]
    alone = []
    for h, f0 in zip(hs, init):
        F = factors_dev(f0)
        alone.append((spt.cp_als(h, F, 9)[1], F))
    got = [None] * len(ts)
    Fs = [factors_dev(f0) for f0 in init]
    torch.cuda.synchronize()

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(5):
                for f, f0 in zip(Fs[i], init[i]):
                    f.copy_(torch.from_numpy(f0))
                fit = spt.cp_als(hs[i], Fs[i], 9)[1]
            s.synchronize()
        got[i] = fit

    threads = [threading.Thread(target=work, args=(i,)) for i in range(len(ts))]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    for i, (fit, F) in enumerate(alone):
        assert got[i] == fit
        assert all(torch.equal(a, b) for a, b in zip(Fs[i], F))
    spt.empty_cache()
