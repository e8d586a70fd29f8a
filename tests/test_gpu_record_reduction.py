"""The record reduction where a row's records meet its edges: rows of one
record, rows that run over many groups and workgroups, chunks of one row,
records that end inside the last group, and outputs that are mostly empty rows
(cleared on the way or by a launch of their own)."""
import numpy as np
import pytest

from _gpu_helpers import factors_dev, mttkrp_error, to_dev
from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu

# Rows of up to 200k products: a tile's run, chunks of at most 64 records and
# the sums over those, each a short chain of FP32 additions.  Random roundings
# of 2^-24 in chains of at most 64 + 64 + 500 terms stay below 628 x 6e-8 of
# the row's scale in the worst case.
TOL = 4e-5


def _tensor(rows, nnz, hot, seed):
    """3 modes; `hot` of the nonzeros in the middle row of mode 0, the others uniform."""
    r = np.random.default_rng(seed)
    dims = (rows, 900, 700)
    c = np.stack([r.integers(0, d, nnz) for d in dims]).astype(np.uint32)
    c[0, r.random(nnz) < hot] = rows // 2
    return synth.SparseCOO(dims, c, r.random(nnz, dtype=np.float32))


@pytest.mark.parametrize("rank", [1, 8, 10, 64, 200])
@pytest.mark.parametrize("rows,nnz,hot", [(1, 1, 0.0), (3, 40, 0.5), (1, 50_000, 0.0), (50, 200_000, 0.9),
                                          (5000, 30_000, 0.3), (400_000, 20_000, 0.1)])
def test_rows_at_every_edge(rank, rows, nnz, hot):
    from paper_2509_00280_amd import spt
    t = _tensor(rows, nnz, hot, rows + rank)
    F = [np.abs(f) for f in synth.normal_factors(rank, t.dims, rank)]
    c, v = to_dev(t)
    h = spt.encode(t.dims, c, v)
    Fd = factors_dev(F)
    for mode in (0, 1):
        err, bad = mttkrp_error(t, F, mode, spt.mttkrp(h, Fd, mode).cpu().numpy())
        assert bad == 0 and err <= TOL, (mode, err, bad)
    h.free()


@pytest.mark.parametrize("noalloc", [False, True])
def test_output_in_a_factors_place(noalloc):
    """An output that shares memory with a factor the call reads: read before it is written."""
    from paper_2509_00280_amd import spt
    r = np.random.default_rng(3)
    dims, nnz, R = (500, 500, 40), 30_000, 16
    t = synth.SparseCOO(dims, np.stack([r.integers(0, d, nnz) for d in dims]).astype(np.uint32),
                        r.random(nnz, dtype=np.float32))
    F = synth.normal_factors(4, dims, R)
    c, v = to_dev(t)
    h = spt.encode(dims, c, v)
    h.prepare(R)
    Fd = factors_dev(F)
    if noalloc:
        spt.mttkrp_noalloc(h, Fd, 0, Fd[1])
    else:
        spt.mttkrp(h, Fd, 0, out=Fd[1])
    err, bad = mttkrp_error(t, F, 0, Fd[1].cpu().numpy())
    assert bad == 0 and err <= TOL, (err, bad)
    h.free()
