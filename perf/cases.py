"""The work whose speed matters: sizes, inputs and one pass of each case.

A case is a dict of plain values.  ``listed()`` names the cases that are
followed from change to change, ``draw(rng)`` gives one more of the same
ranges, ``prepare(case, seed)`` makes what a program holds before the call,
``run(state)`` is one pass through the public entry points, ``work(case)`` is
what the pass cannot do without and ``exact(case, seed)`` is its result in 64
bits from plain torch.

Kinds:
  mttkrp   every mode's MTTKRP, one after the other, of a tensor that is
           encoded and prepared (the sweep that an ALS loop repeats)
  encode   a new COO tensor to its linearized form, out again as keys, values
           and order, and decoded back to coordinates
  solve    a new COO tensor to its CP model: encode, then CP-ALS iterations
  als      CP-ALS iterations on a tensor that is kept encoded and prepared
  batch    CP-ALS of many kept tensors in lock step
  update   one dense ALS mode update of a caller that forms M itself
"""
import ctypes
import math
import random

import numpy as np
import torch

from paper_2509_00280_amd import spt

DEV = "cuda"


# ------------------------------------------------------------------ the cases
def listed():
    return [
        # the smallest configuration of the repository (its smoke check): every
        # call is a few microseconds of work, so launches and host time count
        dict(name="mttkrp small r16", kind="mttkrp", dims="200x150x100", nnz=20_000, zipf="0,0,0",
             vals="u01", shuffle=False, rank=16, dtype="f32"),
        # an exploratory decomposition: a small rank that is no multiple of 4,
        # four modes, 128-bit keys, labels in no order (a flickr-4d shape)
        dict(name="mttkrp flickr4d r10", kind="mttkrp", dims="319700x28200000x1600000x731", nnz=3_000_000,
             zipf="1.1,1.1,1.1,1.1", vals="u01", shuffle=True, rank=10, dtype="f32"),
        # five modes and an odd rank: log records (who, what, where, hour, kind)
        dict(name="mttkrp 5d r25", kind="mttkrp", dims="60000x9000x1200x168x20", nnz=5_000_000,
             zipf="1.2,1.2,1.1,0,0", vals="lognormal", shuffle=True, rank=25, dtype="f32"),
        # the ratings benchmark at full size
        dict(name="mttkrp ratings r32", kind="mttkrp", dims="480000x18000x2000", nnz=100_000_000,
             zipf="1.1,1.1,0", vals="int1to5", shuffle=False, rank=32, dtype="f32"),
        # the headline tensor at full size: factors larger than the Infinity Cache
        dict(name="mttkrp skewed4d r64", kind="mttkrp", dims="2000000x100000x50000x24", nnz=150_000_000,
             zipf="1.3,1.3,1.3,0", vals="lognormal", shuffle=False, rank=64, dtype="f32"),
        # the paper's own precision and rank on a Table I shape (deli-3d, 128-bit keys)
        dict(name="mttkrp deli3d f64 r16", kind="mttkrp", dims="532900x17300000x2500000", nnz=20_000_000,
             zipf="1.1,1.1,1.1", vals="u01", shuffle=True, rank=16, dtype="f64"),
        # loading a data set: one-word keys
        dict(name="encode reddit 30M", kind="encode", dims="8200000x177000x8100000", nnz=30_000_000,
             zipf="1.1,1.1,1.1", vals="u01", shuffle=True),
        # loading a middling tensor with 128-bit keys
        dict(name="encode flickr4d 1M", kind="encode", dims="319700x28200000x1600000x731", nnz=1_000_000,
             zipf="1.1,1.1,1.1,1.1", vals="u01", shuffle=True),
        # the small configuration's decomposition, repeated from new starting
        # points on a kept tensor: launches and the R x R solve count
        dict(name="als small r16", kind="als", dims="200x150x100", nnz=20_000, zipf="0,0,0", vals="u01",
             shuffle=False, rank=16, iters=10),
        # a middling request from COO to model, as the serving workload draws them
        dict(name="solve 2M r48", kind="solve", dims="120000x30000x4000x300", nnz=2_000_000,
             zipf="1.2,1.2,1.2,1.2", vals="u01", shuffle=False, rank=48, iters=10),
        # many independent decompositions (the batch workload, an eighth of its members)
        dict(name="batch 32 r16/32", kind="batch", count=32, nnz_lo=10_000, nnz_hi=5_000_000, dim_lo=50,
             dim_hi=200_000, zipf="1.2", shape_seed=4, ranks="16,32", iters=10),
        # the dense half of an ALS step alone, at the largest rank it takes
        dict(name="update 100k r64", kind="update", rows=100_000, nmodes=4, rank=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _draw_shape(rng, nnz, nmodes, shortest, most):
    """Mode lengths of at least ``shortest`` and at most ``most`` together, room for nnz nonzeros, 128-bit keys."""
    while True:
        dims = [_log_int(rng, shortest, 5_000_000) for _ in range(nmodes)]
        if math.prod(dims) >= 64 * nnz and sum(dims) <= most and sum((d - 1).bit_length() for d in dims) <= 128:
            return dims


def draw(rng):
    kind = rng.choice(["mttkrp", "mttkrp", "mttkrp", "mttkrp", "encode", "als", "solve", "solve", "batch", "update"])
    if kind == "update":
        return dict(kind=kind, rows=_log_int(rng, 100, 2_000_000), nmodes=rng.choice([3, 4, 5]),
                    rank=rng.choice([4, 8, 10, 16, 24, 25, 32, 48, 50, 64]))
    if kind == "batch":
        return dict(kind=kind, count=rng.randint(3, 32), nnz_lo=10_000, nnz_hi=_log_int(rng, 100_000, 3_000_000),
                    dim_lo=50, dim_hi=_log_int(rng, 2_000, 200_000), zipf="%.2f" % rng.uniform(0.8, 1.3),
                    shape_seed=rng.randrange(1 << 20), ranks=rng.choice(["16,32", "8", "10,25", "16,48", "64"]),
                    iters=rng.choice([5, 10]))
    # decompositions have 3 or 4 modes: with 5, ALS from N(0,1) on this few nonzeros often ends not positive definite
    nmodes = rng.choice({"mttkrp": [3, 3, 3, 4, 4, 5], "encode": [2, 3, 4, 5, 6]}.get(kind, [3, 4]))
    hi = {"mttkrp": 30_000_000, "encode": 30_000_000, "als": 3_000_000, "solve": 3_000_000}[kind]
    model = kind in ("als", "solve")
    nnz = _log_int(rng, 20_000 if model else 5_000, hi) | 1
    # a model has modes longer than its rank, and several nonzeros to each of their rows
    dims = _draw_shape(rng, nnz, nmodes, *((100, nnz // 4) if model else (20, 8 * nnz + 100_000)))
    c = dict(kind=kind, dims="x".join(str(d) for d in dims), nnz=nnz,
             zipf=",".join("0" if rng.random() < 0.25 else "%.2f" % rng.uniform(0.8, 1.3) for _ in dims),
             vals=rng.choice(["u01", "int1to5"] if model else ["u01", "int1to5", "lognormal"]), shuffle=rng.random() < 0.5)
    if kind == "encode":
        return c
    c["rank"] = rng.choice([8, 10, 16, 16, 20, 25, 32, 32, 48, 50, 64])
    if kind == "mttkrp":
        c["dtype"] = "f64" if rng.random() < 0.25 else "f32"
        if rng.random() < 0.1:
            c["rank"] = rng.choice([100, 128])
    else:
        c["iters"] = rng.choice([3, 5, 10])
    return c


# ------------------------------------------------------------------ inputs
def _dims(case):
    return [int(d) for d in case["dims"].split("x")]


def _zipfs(case):
    return [float(z) for z in case["zipf"].split(",")]


def _labels(gen, n, count, s):
    """Labels in {0..n-1}: uniform (s = 0) or a bounded power law of exponent s, label 0 the most
    frequent (the inverse distribution function of x^-s over [1, n + 1), rounded down)."""
    if s == 0:
        return torch.randint(0, n, (count,), generator=gen, device=DEV)
    u = torch.rand(count, generator=gen, device=DEV, dtype=torch.float64)
    x = (n + 1.0) ** u if s == 1 else (u * ((n + 1.0) ** (1 - s) - 1) + 1) ** (1 / (1 - s))
    return (x.long() - 1).clamp_(0, n - 1)


def _coo(seed, dims, nnz, zipfs, vals, shuffle):
    """A COO tensor of nnz cells in random order: int32 (nmodes, nnz), float32 (nnz,).

    The cells are distinct, drawn from the modes' laws in rounds; what twelve
    rounds leave open in a crowded corner is filled with uniform cells."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed))
    coords = torch.zeros((len(dims), 0), dtype=torch.int32, device=DEV)
    for _ in range(12):
        m = int(1.5 * (nnz - coords.shape[1])) + 64
        c = torch.stack([_labels(gen, d, m, s).to(torch.int32) for d, s in zip(dims, zipfs)])
        coords = torch.cat([coords, c], dim=1)
        cell = torch.zeros(coords.shape[1], dtype=torch.int64, device=DEV)
        for n, d in enumerate(dims):  # the cell's number, modulo 2^64 in a box larger than that
            cell = cell * (d | 1) + coords[n]
        cell, order = torch.sort(cell, stable=True)
        head = torch.ones_like(cell, dtype=torch.bool)
        head[1:] = cell[1:] != cell[:-1]
        coords = coords[:, order[head].sort().values]
        if coords.shape[1] >= nnz:
            break
    rest = nnz - coords.shape[1]
    if rest > 0:
        c = torch.stack([_labels(gen, d, rest, 0).to(torch.int32) for d in dims])
        coords = torch.cat([coords, c], dim=1)
    coords = coords[:, :nnz].contiguous()
    if shuffle:
        for n, d in enumerate(dims):
            coords[n] = torch.randperm(d, generator=gen, device=DEV).to(torch.int32)[coords[n].long()]
    if vals == "u01":
        v = torch.rand(nnz, generator=gen, device=DEV)
    elif vals == "int1to5":
        v = torch.randint(1, 6, (nnz,), generator=gen, device=DEV).to(torch.float32)
    else:
        v = torch.randn(nnz, generator=gen, device=DEV).exp_()
    return coords, v


def _factors(seed, dims, rank, law, dtype=torch.float32):
    """N(0,1) starting points of a decomposition, or the U(0,1) factors of a nonnegative one.

    A sweep by itself takes the latter: with N(0,1) rows that have nothing to
    do with the data, the sums of the busiest rows of a skewed tensor cancel
    to a hundredth of their terms, and FP32 leaves four digits of them."""
    gen = torch.Generator(device=DEV)
    gen.manual_seed(int(seed) + 0x5EED)
    make = torch.randn if law == "normal" else torch.rand
    return [make((d, rank), generator=gen, device=DEV, dtype=dtype) for d in dims]


def _members(case):
    """Shapes of a batch: (dims, nnz, rank) of every member, fixed by the case."""
    r = random.Random(case["shape_seed"])
    ranks = [int(x) for x in case["ranks"].split(",")]
    out = []
    for _ in range(case["count"]):
        nm = r.choice([3, 4])
        nnz = _log_int(r, case["nnz_lo"], case["nnz_hi"])
        while True:
            dims = [_log_int(r, case["dim_lo"], case["dim_hi"]) for _ in range(nm)]
            if math.prod(dims) >= 64 * nnz and sum(dims) <= nnz:
                break
        out.append((dims, nnz, r.choice(ranks)))
    return out


def _update_inputs(case, seed):
    R = case["rank"]
    other = _factors(seed, [40 * R + 64 * k for k in range(case["nmodes"])], R, "normal")
    grams = torch.stack([f.double().T @ f.double() for f in other]).contiguous()
    M = _factors(seed + 1, [case["rows"]], R, "normal")[0] * 100.0
    return grams, M


def prepare(case, seed):
    kind = case["kind"]
    if kind == "update":
        grams, M = _update_inputs(case, seed)
        return dict(case=case, grams=grams, M=M, C=torch.empty_like(M),
                    lam=torch.empty(case["rank"], dtype=torch.float64, device=DEV))
    if kind == "batch":
        ts, inits, shapes = [], [], []
        for i, (dims, nnz, R) in enumerate(_members(case)):
            c, v = _coo(seed * 1000 + i, dims, nnz, [float(case["zipf"])] * len(dims), "u01", False)
            t = spt.encode(dims, c, v)
            t.prepare(R, batched=True)
            ts.append(t)
            inits.append(_factors(seed * 1000 + i, dims, R, "normal"))
            shapes.append((dims, R))
        # every member's factors and weights are views of one buffer each
        init = torch.cat([f.reshape(-1) for fl in inits for f in _aligned(fl)])
        work = torch.empty_like(init)
        lists, at = [], 0
        for dims, R in shapes:
            fl = []
            for d in dims:
                fl.append(work[at:at + d * R].view(d, R))
                at += -(-d * R // 4) * 4
            lists.append(fl)
        lam = torch.empty(sum(R for _, R in shapes), dtype=torch.float64, device=DEV)
        return dict(case=case, tensors=ts, init=init, work=work, factors=lists,
                    lam=lam, lams=list(lam.split([R for _, R in shapes])))
    dims = _dims(case)
    coords, vals = _coo(seed, dims, case["nnz"], _zipfs(case), case["vals"], case["shuffle"])
    s = dict(case=case, dims=dims)
    if kind == "encode":
        nnz, words = case["nnz"], _key_words(dims)
        return dict(s, coords=coords, vals=vals, keys=torch.empty(nnz * words, dtype=torch.int64, device=DEV),
                    out_vals=torch.empty(nnz, device=DEV), perm=torch.empty(nnz, dtype=torch.int32, device=DEV),
                    back=torch.empty((len(dims), nnz), dtype=torch.int32, device=DEV))
    R = case["rank"]
    if kind == "mttkrp":
        dt = torch.float64 if case["dtype"] == "f64" else torch.float32
        t = spt.encode(dims, coords, vals)
        t.prepare(R)
        if case["dtype"] == "f64":
            spt.attach_f64(t, vals.double())
        return dict(s, tensor=t, factors=_factors(seed, dims, R, "uniform", dt),
                    outs=[torch.empty((d, R), dtype=dt, device=DEV) for d in dims])
    s.update(init=_factors(seed, dims, R, "normal"), lam=torch.empty(R, dtype=torch.float64, device=DEV))
    s["factors"] = [torch.empty_like(f) for f in s["init"]]
    if kind == "als":
        t = spt.encode(dims, coords, vals)
        t.prepare(R)
        return dict(s, tensor=t)
    return dict(s, coords=coords, vals=vals)


def _aligned(factors):
    """Flat copies padded to 16 bytes, so that views of their concatenation are aligned."""
    return [torch.nn.functional.pad(f.reshape(-1), (0, -f.numel() % 4)) for f in factors]


def _key_words(dims):
    return 2 if sum((d - 1).bit_length() for d in dims) > 64 else 1


# ------------------------------------------------------------------ one pass
def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "mttkrp":
        call = spt.mttkrp_f64 if case["dtype"] == "f64" else spt.mttkrp
        for n, out in enumerate(s["outs"]):
            call(s["tensor"], s["factors"], n, out=out)
        return s["outs"]
    if kind == "encode":
        # the export and decode of the C interface, into device buffers
        t = spt.encode(s["dims"], s["coords"], s["vals"])
        stream = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
        ptr = lambda x: ctypes.c_void_p(x.data_ptr())  # noqa: E731
        for st in (spt.lib().spt_tensor_export(t.handle, ptr(s["keys"]), ptr(s["out_vals"]), ptr(s["perm"]), stream),
                   spt.lib().spt_tensor_decode(t.handle, ptr(s["back"]), stream)):
            if st != 0:
                raise RuntimeError(spt.lib().spt_last_error())
        t.free()
        return dict(keys=s["keys"], vals=s["out_vals"], perm=s["perm"], coords=s["back"])
    if kind == "update":
        C, lam, retries = spt.als_update(s["grams"], case["nmodes"] - 1, s["M"], C=s["C"], lam=s["lam"])
        return dict(C=C, lam=lam, retries=retries)
    # The model is kept in FP32, factors and weights alike: the weights come
    # out of an FP32 MTTKRP, whatever type they are handed over in.
    if kind == "batch":
        s["work"].copy_(s["init"])
        _, fits, _ = spt.cp_als_batched(s["tensors"], s["factors"], case["iters"], lams=s["lams"])
        return dict(factors=s["work"], weights=s["lam"].float(), fits=np.array(fits, dtype=np.float32))
    for f, f0 in zip(s["factors"], s["init"]):
        f.copy_(f0)
    t = s["tensor"] if kind == "als" else spt.encode(s["dims"], s["coords"], s["vals"])
    _, fit, _ = spt.cp_als(t, s["factors"], case["iters"], lam=s["lam"])
    if kind == "solve":
        t.free()
    return dict(factors=s["factors"], weights=s["lam"].float(), fit=fit)


# ------------------------------------------------------------------ what a pass cannot do without
def _touched(n, s, nnz):
    """Expected distinct labels of nnz draws from the mode's law (a sum over a log grid of labels)."""
    if s == 0:
        return n * -math.expm1(-nnz / n)
    grid = np.unique(np.round(np.geomspace(1, n, 400)).astype(np.int64)).astype(np.float64)
    norm = np.trapezoid(grid ** -s, grid) + 0.5 * (1 + n ** -s)
    hit = -np.expm1(-nnz * grid ** -s / norm)
    return min(float(n), float(np.trapezoid(hit, grid)) + 1.0)


def _sweep(dims, zipfs, nnz, rank, item):
    """Bytes and flops of one all-mode MTTKRP: the encoding once a mode, touched factor rows, outputs."""
    rows = [_touched(d, z, nnz) for d, z in zip(dims, zipfs)]
    N = len(dims)
    b = N * nnz * (8 * _key_words(dims) + item)
    for n in range(N):
        b += (sum(rows) - rows[n] + dims[n]) * rank * item
    return b, float(N) * N * nnz * rank


def _als(dims, zipfs, nnz, rank, iters):
    b, f = _sweep(dims, zipfs, nnz, rank, 4)
    b += sum(dims) * rank * 4  # the new factors
    f += sum(dims) * 4.0 * rank * rank + len(dims) * 4.0 * rank ** 3
    return iters * b, iters * f


def _encode(dims, nnz):
    return nnz * (4 * len(dims) + 4 + 8 * _key_words(dims) + 8)


def work(case):
    kind = case["kind"]
    if kind == "update":
        R = case["rank"]
        return {"bytes": case["rows"] * R * 8 + (case["nmodes"] + 1) * R * R * 8,
                "flops": case["rows"] * 4.0 * R * R + 4.0 * R ** 3}
    if kind == "batch":
        b = f = 0.0
        for dims, nnz, R in _members(case):
            x, y = _als(dims, [float(case["zipf"])] * len(dims), nnz, R, case["iters"])
            b, f = b + x, f + y
        return {"bytes": b, "flops": f}
    dims, zipfs, nnz = _dims(case), _zipfs(case), case["nnz"]
    if kind == "encode":
        return {"bytes": _encode(dims, nnz) + 4 * len(dims) * nnz, "flops": 0}
    if kind == "mttkrp":
        b, f = _sweep(dims, zipfs, nnz, case["rank"], 8 if case["dtype"] == "f64" else 4)
    else:
        b, f = _als(dims, zipfs, nnz, case["rank"], case["iters"])
        b += _encode(dims, nnz) if kind == "solve" else 0
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------ the same in 64 bits
class _Mode:
    """Nonzeros ordered by one mode's row, cut into runs of at most 64 of one row, level by level."""

    def __init__(self, row, rows):
        self.row, self.order = row.long().sort(stable=True)
        self.rows = rows

    def sum(self, coords, vals, F, mode):
        R = F[(mode + 1) % len(F)].shape[1]
        step = max(1, (1 << 29) // R)
        parts, heads = [], []
        for a in range(0, self.row.shape[0], step):
            o = self.order[a:a + step]
            p = vals[o, None].expand(-1, R).clone()
            for k, f in enumerate(F):
                if k != mode:
                    p *= f[coords[k, o].long()]
            p, h = self._fold(p, self.row[a:a + step])
            parts.append(p)
            heads.append(h)
        p, h = torch.cat(parts), torch.cat(heads)
        while h.shape[0] > 1 and bool((h[1:] == h[:-1]).any()):
            p, h = self._fold(p, h)
        out = torch.zeros((self.rows, R), dtype=torch.float64, device=DEV)
        out[h] = p
        return out

    @staticmethod
    def _fold(p, row):
        """Sums over runs of at most 64 consecutive equal rows."""
        i = torch.arange(row.shape[0], device=DEV)
        new = torch.ones_like(row, dtype=torch.bool)
        new[1:] = row[1:] != row[:-1]
        start = torch.where(new, i, 0).cummax(0).values
        cut = ((i - start) % 64 == 0).nonzero().squeeze(1)
        lengths = torch.diff(cut, append=torch.tensor([row.shape[0]], device=DEV))
        return torch.segment_reduce(p, "sum", lengths=lengths, axis=0, unsafe=True), row[cut]


def _als64(coords, vals, dims, F, iters):
    N = len(dims)
    modes = [_Mode(coords[n], dims[n]) for n in range(N)]
    F = [f.double() for f in F]
    G = [f.T @ f for f in F]
    x2 = (vals * vals).sum()
    fit = lam = None
    for _ in range(iters):
        for n in range(N):
            M = modes[n].sum(coords, vals, F, n)
            V = torch.ones_like(G[0])
            for k in range(N):
                if k != n:
                    V = V * G[k]
            C = torch.cholesky_solve(M.T.contiguous(), torch.linalg.cholesky(V)).T.contiguous()
            lam = C.norm(dim=0)
            lam = torch.where(lam > 0, lam, torch.ones_like(lam))
            F[n] = C / lam
            G[n] = F[n].T @ F[n]
        H = torch.ones_like(G[0])
        for g in G:
            H = H * g
        r2 = x2 + lam @ H @ lam - 2.0 * (M * F[-1] * lam).sum()
        fit = float(1.0 - torch.sqrt(r2.clamp(min=0) / x2))
    return F, lam, fit


def exact(case, seed):
    kind = case["kind"]
    if kind == "encode":
        return None  # whole numbers, and values that are moved, not computed
    if kind == "update":
        grams, M = _update_inputs(case, seed)
        V = grams[:-1].prod(dim=0)
        C = torch.cholesky_solve(M.double().T.contiguous(), torch.linalg.cholesky(V)).T
        lam = C.norm(dim=0)
        return dict(C=C / lam, lam=lam, retries=None)
    if kind == "batch":
        flat, lams, fits = [], [], []
        for i, (dims, nnz, R) in enumerate(_members(case)):
            c, v = _coo(seed * 1000 + i, dims, nnz, [float(case["zipf"])] * len(dims), "u01", False)
            F, lam, fit = _als64(c, v.double(), dims, _factors(seed * 1000 + i, dims, R, "normal"), case["iters"])
            flat += _aligned(F)
            lams.append(lam)
            fits.append(fit)
        return dict(factors=torch.cat(flat), weights=torch.cat(lams), fits=np.array(fits))
    dims = _dims(case)
    c, v = _coo(seed, dims, case["nnz"], _zipfs(case), case["vals"], case["shuffle"])
    v = v.double()
    if kind == "mttkrp":
        dt = torch.float64 if case["dtype"] == "f64" else torch.float32
        F = [f.double() for f in _factors(seed, dims, case["rank"], "uniform", dt)]
        return [_Mode(c[n], dims[n]).sum(c, v, F, n) for n in range(len(dims))]
    F, lam, fit = _als64(c, v, dims, _factors(seed, dims, case["rank"], "normal"), case["iters"])
    return dict(factors=F, weights=lam, fit=fit)
