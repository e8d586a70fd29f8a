"""CP-ALS without a tolerance reads its iterations back in groups of 32: the
same decomposition, fit and errors as with a readback each (a tolerance that
no step falls below)."""
import numpy as np
import pytest

from _gpu_helpers import factors_dev, to_dev
from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu

# The two runs differ by the order of FP32 sums only (2^-24 each, a few hundred
# terms), carried through up to 65 iterations of a well-conditioned problem.
TOL = 2e-3


@pytest.mark.parametrize("iters", [1, 31, 32, 33, 65])
def test_groups_of_iterations(iters):
    import torch
    from paper_2509_00280_amd import spt
    t = synth.distinct_coo(5, (60, 50, 40), 6000, ["uniform"] * 3, "u01")
    init = [np.abs(f) + 0.1 for f in synth.normal_factors(3, t.dims, 4)]
    h = spt.encode(t.dims, *to_dev(t))
    got = []
    for tol in (0.0, 1e-300):
        F = factors_dev([f.astype(np.float32) for f in init])
        lam, fit, n = spt.cp_als(h, F, iters, tol=tol)
        assert n == iters
        got.append((fit, [f * lam.to(f.dtype) for f in F]))
    assert abs(got[0][0] - got[1][0]) <= 1e-5
    for a, b in zip(got[0][1], got[1][1]):
        assert torch.linalg.norm(a - b) <= TOL * torch.linalg.norm(b)
    h.free()


@pytest.mark.parametrize("iters", [100, 128, 200])
def test_direct_residual_takes_the_last_iteration(iters):
    """Nearly exact fits come from the residual over the nonzeros and the last
    iteration's |Xhat|^2.  Both runs do the same operations on the same plan, and
    a tensor this small has no atomics: the same fit to rounding in FP64."""
    from paper_2509_00280_amd import spt
    dims, R = (30, 20, 10), 4
    for seed in range(6):
        rng = np.random.default_rng(seed)
        true = [rng.random((d, R)) + 0.1 for d in dims]
        X = np.einsum("ir,jr,kr->ijk", *true)
        coords = np.stack(np.nonzero(np.ones(dims))).astype(np.uint32)
        t = synth.SparseCOO(dims, coords, X[tuple(coords)].astype(np.float32))
        init = [rng.standard_normal((d, R)).astype(np.float32) for d in dims]
        h = spt.encode(t.dims, *to_dev(t))
        fits = []
        for tol in (0.0, 1e-300):
            F = factors_dev(init)
            fits.append(spt.cp_als(h, F, iters, tol=tol)[1:])
        h.free()
        if fits[1][1] == iters:
            assert abs(fits[0][0] - fits[1][0]) <= 1e-9, (seed, fits)


@pytest.mark.parametrize("iters", [1, 40])
def test_failed_solve_leaves_the_factors(iters):
    import torch
    from paper_2509_00280_amd import spt
    t = synth.distinct_coo(6, (60, 50, 40), 6000, ["uniform"] * 3, "u01")
    F = factors_dev([np.full((d, 4), np.nan, np.float32) for d in t.dims])
    F[2] = torch.ones_like(F[2])
    h = spt.encode(t.dims, *to_dev(t))
    with pytest.raises(spt.SptError, match="mode 0 not positive definite"):
        spt.cp_als(h, F, iters)
    assert torch.equal(F[2], torch.ones_like(F[2])) and torch.isnan(F[0]).all()
    h.free()
