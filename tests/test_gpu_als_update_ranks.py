"""The dense ALS update at the edges of its 16-wide blocks, and at row counts
around its slices, tiles and partial sums, against NumPy in FP64."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _update(nmodes, mode, rank, rows, seed):
    import torch
    from paper_2509_00280_amd import spt
    r = np.random.default_rng(seed)
    other = [r.standard_normal((3 * rank + 40 + k, rank)) for k in range(nmodes)]
    grams = np.stack([f.T @ f for f in other])
    M = (100 * r.standard_normal((rows, rank))).astype(np.float32)
    C, lam, retries = spt.als_update(torch.from_numpy(grams).cuda(), mode, torch.from_numpy(M).cuda())
    V = np.ones((rank, rank))
    for k in range(nmodes):
        if k != mode:
            V = V * grams[k]
    ref = np.linalg.solve(V, M.astype(np.float64).T).T
    n = np.linalg.norm(ref, axis=0)
    assert retries == 0
    # V's condition number is below 1e3 (products of well-separated Grams), so
    # FP64 leaves 1e3 x rank x 2^-53 < 1e-11 of the norms; C is rounded to FP32
    # once, half a unit in 2^-23 of entries of at most 1
    np.testing.assert_allclose(lam.cpu().numpy(), n, rtol=1e-10)
    np.testing.assert_allclose(C.cpu().numpy(), ref / n, rtol=1.3e-7, atol=1e-9)


@pytest.mark.parametrize("rank", [1, 2, 3, 4, 5, 10, 15, 16, 17, 25, 31, 32, 33, 47, 48, 49, 63, 64])
def test_every_block_edge(rank):
    _update(3, rank % 3, rank, 1000 + rank, rank)


@pytest.mark.parametrize("rank", [8, 16, 25, 32, 48, 64])
@pytest.mark.parametrize("rows", [65, 127, 128, 129, 255, 257, 512, 513, 1025, 2049, 4097, 70_001])
def test_every_row_edge(rank, rows):
    _update(4, 1, rank, rows, rows)


@pytest.mark.parametrize("rank", [16, 40, 64])
def test_a_failing_pivot_in_any_block(rank):
    """A matrix that is not positive definite from some pivot on is refused, wherever that pivot is."""
    import torch
    from paper_2509_00280_amd import spt
    M = torch.ones((30, rank), device="cuda")
    for bad in (0, 1, 15, 16, rank // 2, rank - 1):
        if bad >= rank:
            continue
        V = np.eye(rank)
        V[bad, bad] = -1.0
        g = torch.from_numpy(np.stack([V, np.ones((rank, rank))])).cuda()
        with pytest.raises(spt.SptError) as e:
            spt.als_update(g, 1, M)
        assert e.value.status == -6
    V = np.eye(rank)
    C, lam, retries = spt.als_update(torch.from_numpy(np.stack([V, V])).cuda(), 1, M)  # and the next call is fine
    assert retries == 0 and np.allclose(lam.cpu().numpy(), np.sqrt(30.0), rtol=1e-12)
