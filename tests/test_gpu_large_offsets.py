"""Record arrays and factors of about 4 GiB and more: a row's index times its
length no longer fits the 32-bit offsets of a structured buffer."""
import pytest

pytestmark = pytest.mark.gpu


def _rows_once(rows, nnz, others, seed):
    """nnz nonzeros in mode-0 rows of their own (a record each), anywhere in the other modes."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    c = [torch.randperm(rows, generator=g, device="cuda")[:nnz].to(torch.int32)]
    c += [torch.randint(0, d, (nnz,), generator=g, device="cuda", dtype=torch.int32) for d in others]
    return torch.stack(c), torch.rand(nnz, generator=g, device="cuda") + 0.5, g


def _stretches(nnz):
    return [slice(a, a + (1 << 18)) for a in range(0, nnz, 1 << 18)]


def _product(c, v, F, mode, s):
    p = v[s, None].double().expand(-1, F[1].shape[1])
    for k, f in enumerate(F):
        if k != mode:
            p = p * f[c[k, s].long()].double()
    return p


def _check_large_output(out, c, v, F, eps):
    """Mode 0: a row is one product, rounded once for each factor (FP64, where the reference
    rounds alike: the repository's criterion for it, 1e-12)."""
    import torch
    seen = torch.zeros(out.shape[0], dtype=torch.bool, device="cuda")
    for s in _stretches(v.shape[0]):
        ref = _product(c, v, F, 0, s)
        err = float(((out[c[0, s].long()].double() - ref).abs() / ref).max())
        assert err <= (len(F) * eps if out.dtype == torch.float32 else 1e-12), (s, err)
        seen[c[0, s].long()] = True
    assert bool((out[~seen] == 0).all())


def _check_large_factor(out, c, v, F, eps):
    """Mode 1: rows of all of the large factor.  All terms are positive; a row's are added in
    chains of at most 256 (a run's) and a few dozen (a chunk of at most 128 records) at a time."""
    import torch
    rows = out.shape[0]
    ref = torch.zeros(out.shape, dtype=torch.float64, device="cuda")
    for s in _stretches(v.shape[0]):
        order = torch.argsort(c[1, s], stable=True)
        ref += torch.segment_reduce(_product(c, v, F, 1, s)[order], "sum", lengths=torch.bincount(c[1, s], minlength=rows),
                                    axis=0, unsafe=True)
    err = float(((out.double() - ref).abs() / ref).max())
    assert err <= max(320 * eps, 1e-12), err


# rows of 1 KiB: 2^32 bytes of records and factor exactly, and more
@pytest.mark.parametrize("rows,nnz", [(1 << 22, 1 << 22), (5_000_000, 4_600_000)])
@pytest.mark.parametrize("dtype,rank", [("float32", 256), ("float64", 128)])
@pytest.mark.parametrize("others", [(2000,), (50, 40), (20, 10, 10), (10, 5, 8, 5), (5, 4, 5, 4, 5)])
def test_one_tensor(others, dtype, rank, rows, nnz):
    import torch
    from paper_2509_00280_amd import spt
    dt = getattr(torch, dtype)
    c, v, g = _rows_once(rows, nnz, others, rank)
    dims = (rows,) + others
    F = [torch.rand((d, rank), generator=g, device="cuda", dtype=dt) + 0.5 for d in dims]
    h = spt.encode(dims, c, v)
    eps = torch.finfo(dt).eps / 2
    plans, call = [dict(), dict(row_cache=False, tile=1024)], spt.mttkrp
    if dtype == "float64":
        spt.attach_f64(h, v.double())
        plans, call = plans[:1], spt.mttkrp_f64
    for plan in plans:
        if plan:
            h.set_plan(**plan)
        _check_large_output(call(h, F, 0), c, v, F, eps)
        _check_large_factor(call(h, F, 1), c, v, F, eps)
    h.free()


@pytest.mark.parametrize("others", [(50, 40), (20, 10, 10), (10, 5, 8, 5)])
def test_in_a_batch(others):
    """A large member beside a small one."""
    import torch
    from paper_2509_00280_amd import spt
    ts, hs, Fs = [], [], []
    for rows, nnz, rank in ((18_000_000, 17_000_000, 64), (3000, 2000, 16)):
        c, v, g = _rows_once(rows, nnz, others, rank)
        ts.append((c, v))
        hs.append(spt.encode((rows,) + others, c, v))
        Fs.append([torch.rand((d, rank), generator=g, device="cuda") + 0.5 for d in (rows,) + others])
    for mode, check in ((0, _check_large_output), (1, _check_large_factor)):
        outs = [torch.empty_like(F[mode]) for F in Fs]
        spt.mttkrp_batched(hs, Fs, mode, outs)
        for (c, v), F, o in zip(ts, Fs, outs):
            check(o, c, v, F, 2.0**-24)
    for h in hs:
        h.free()
