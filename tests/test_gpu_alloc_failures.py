"""Batched CP-ALS and the server when an allocation fails: every allocation of a
call in turn is refused once by the allocator hook."""
import threading

import numpy as np
import pytest

from _gpu_helpers import cpd_error, factors_dev, to_dev, to_host
from paper_2509_00280_amd import synth

pytestmark = pytest.mark.gpu

E_OOM = -5
TOL = 1e-4  # the repository's criterion for CP-ALS factors and fits


class FailingHook:
    """Fresh memory for every request, kept until the end; refuses the one that `refuse` counts down to."""

    def __init__(self, spt):
        import torch
        self.lock, self.kept, self.refuse, self.refused = threading.Lock(), [], 0, False

        def _alloc(nbytes, stream, ctx):
            with self.lock:
                self.refuse -= 1
                if self.refuse == 0:
                    self.refused = True
                    return None
                x = torch.empty(int(nbytes), dtype=torch.uint8, device="cuda")
                self.kept.append(x)
                return x.data_ptr()

        self.hooks = (spt.ALLOC_FN(_alloc), spt.RELEASE_FN(lambda ptr, stream, ctx: None))

    def arm(self, k):
        with self.lock:
            self.refuse, self.refused = k, False


@pytest.fixture
def hook():
    import torch
    from paper_2509_00280_amd import spt
    h = FailingHook(spt)
    assert spt.lib().spt_set_allocator(h.hooks[0], h.hooks[1], None) == 0
    yield h
    torch.cuda.synchronize()
    spt.use_torch_allocator(False)


def _member(i):
    t = synth.distinct_coo(30 + i, (80 + i, 60, 40), 4000, ["uniform"] * 3, "u01")
    return t, [(np.abs(f) + 0.1).astype(np.float32) for f in synth.normal_factors(i, t.dims, 8)]


def test_batch(hook):
    import torch
    from paper_2509_00280_amd import spt
    members = [_member(i) for i in range(2)]
    hs = [spt.encode(t.dims, *to_dev(t)) for t, _ in members]
    for h in hs:
        h.prepare(8, batched=True)
    ref = []
    for (t, f0), h in zip(members, hs):
        F = factors_dev(f0)
        lam, fit, _ = spt.cp_als(h, F, 4)
        ref.append((to_host(F), lam.cpu().numpy(), fit))
    Fs = [factors_dev(f0) for _, f0 in members]
    k = 0
    while True:
        k += 1
        print("refused allocation", k, flush=True)
        hook.arm(k)
        try:
            lams, fits, _ = spt.cp_als_batched(hs, Fs, 4)
            break
        except spt.SptError as e:
            assert hook.refused and e.status == E_OOM
            for F, (_, f0) in zip(Fs, members):
                assert all(np.array_equal(a, b) for a, b in zip(to_host(F), f0))
    assert not hook.refused and k > 10
    for F, lam, fit, (rF, rlam, rfit) in zip(Fs, lams, fits, ref):
        err, lerr = cpd_error(to_host(F), lam.cpu().numpy(), rF, rlam)
        assert err <= TOL and lerr <= TOL and abs(fit - rfit) <= TOL


def test_server(hook):
    """A request joins one that runs, and an allocation fails on the way: each request ends with its
    model or refused for memory, and the next one is served."""
    from paper_2509_00280_amd import spt
    (ta, fa), (tb, fb) = _member(3), _member(4)
    ref = {}
    for name, t, f0, iters in (("a", ta, fa, 40), ("b", tb, fb, 4)):
        h = spt.encode(t.dims, *to_dev(t))
        F = factors_dev(f0)
        lam, fit, _ = spt.cp_als(h, F, iters)
        ref[name] = (to_host(F), lam.cpu().numpy(), fit)
        h.free()
    server = spt.Server(1 << 34, 4)
    served = refused = 0
    try:
        for k in range(1, 90):
            print("refused allocation", k, flush=True)
            hook.arm(0)
            tickets = [("a", server.submit(ta.dims, ta.coords, ta.vals, fa, 40))]
            hook.arm(k)
            tickets.append(("b", server.submit(tb.dims, tb.coords, tb.vals, fb, 4)))
            for name, ticket in tickets:
                res, F, lam = server.wait(ticket)
                if res["status"] != 0:
                    assert res["status"] == E_OOM and hook.refused, (k, name, res)
                    refused += 1
                    continue
                served += 1
                # 40 iterations carry the roundings of FP32 further than 4: fits only
                assert abs(res["fit"] - ref[name][2]) <= TOL, (k, name, res, ref[name][2])
                if name == "b":
                    err, lerr = cpd_error(F, lam, ref[name][0], ref[name][1])
                    assert err <= TOL and lerr <= TOL, (k, err, lerr)
    finally:
        server.close()
    assert served > 60 and refused > 20, (served, refused)
