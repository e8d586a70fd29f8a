"""The record reduction where a lane group's chunk is more than one round of 8
records: sums carried over rounds, runs that end in a later round, runs through
whole chunks, groups and workgroups."""
import numpy as np
import pytest

from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu

TILE = 1024


def _chunk(rank, cols, records):
    """Records of a lane group's chunk: 512 to a workgroup of 4 waves, while 4096 chunks remain."""
    groups = 4 * (64 // -(-rank // cols))
    chunk = max(8, (512 // groups + 7) & ~7)
    while chunk > 8 and records // chunk < 4096:
        chunk -= 8
    return chunk


# (rank, columns of a lane, nonzeros, chunk expected)
FP32 = [(32, 4, 120_000, 16), (64, 4, 250_000, 32), (128, 4, 500_000, 64), (200, 4, 900_000, 128)]
FP64 = [(16, 2, 120_000, 16), (32, 2, 250_000, 32), (64, 2, 500_000, 64), (129, 4, 900_000, 128)]


def _tensor(nnz, rows, hot, seed):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    dims = (rows, 610, 470)
    c = torch.stack([torch.randint(0, d, (nnz,), generator=g, device="cuda", dtype=torch.int32) for d in dims])
    c[0, torch.rand(nnz, generator=g, device="cuda") < hot] = rows // 3
    v = torch.rand(nnz, generator=g, device="cuda", dtype=torch.float64)
    return dims, c, v


def _reference(dims, c, v, F):
    """Row sums of mode 0 in FP64, a stretch of the nonzeros at a time."""
    import torch
    out = torch.zeros((dims[0], F[1].shape[1]), dtype=torch.float64, device="cuda")
    for a in range(0, v.shape[0], 1 << 18):
        s = slice(a, a + (1 << 18))
        out.index_add_(0, c[0, s].long(), v[s, None] * F[1][c[1, s].long()].double() * F[2][c[2, s].long()].double())
    return out


def _check(dtype, rank, cols, nnz, chunk, rows, hot):
    import torch
    from paper_2509_00280_amd import spt
    dims, c, v = _tensor(nnz, rows, hot, rank)
    F = [torch.rand((d, rank), device="cuda", dtype=dtype) + 0.5 for d in dims]
    # the row's bits lowest in the key: the rows of a tile are spread over the mode
    bits = [(d - 1).bit_length() for d in dims]
    h = spt.encode(dims, c, v.float(), layout=[k for k in range(3) for _ in range(bits[k])])
    h.set_plan(tile=TILE)
    perm = torch.from_numpy(h.export()[2].astype(np.int64)).cuda()
    tile = torch.arange(nnz, device="cuda") // TILE
    records = int(torch.unique(tile * rows + c[0].long()[perm]).shape[0])
    assert _chunk(rank, cols, records) == chunk, records
    if dtype == torch.float64:
        spt.attach_f64(h, v)
        out = spt.mttkrp_f64(h, F, 0)
    else:
        v = v.float().double()
        out = spt.mttkrp(h, F, 0).double()
    ref = _reference(dims, c, v, F)
    # All terms are positive.  A product 3 roundings; a tile's run at most 256
    # additions; a chunk 8 and a join for each round; the groups' parts in FP64;
    # an atomic addition for each workgroup of at least 512 records.
    adds = 3 + 256 + 8 + chunk // 8 + 2 + -(-nnz // TILE) // 512 + 1
    tol = adds * (2.0**-53 if dtype == torch.float64 else 2.0**-24)
    err = float(((out - ref).abs() / ref.clamp(min=1e-300)).max())
    assert bool((out[ref == 0] == 0).all()) and err <= tol, (records, err, tol)
    h.free()


# 1500 rows: runs of a hundred records and more; 40000 rows, one of them hot: runs
# of a few records, and one that goes through groups and workgroups
@pytest.mark.parametrize("rows,hot", [(1500, 0.0), (40_000, 0.1)])
@pytest.mark.parametrize("rank,cols,nnz,chunk", FP32)
def test_fp32(rank, cols, nnz, chunk, rows, hot):
    import torch
    _check(torch.float32, rank, cols, nnz, chunk, rows, hot)


@pytest.mark.parametrize("rows,hot", [(1500, 0.0), (40_000, 0.1)])
@pytest.mark.parametrize("rank,cols,nnz,chunk", FP64)
def test_fp64(rank, cols, nnz, chunk, rows, hot):
    import torch
    _check(torch.float64, rank, cols, nnz, chunk, rows, hot)
