"""The work that a program using this library has it do, as measurable cases:
sparse MTTKRP, tensor-times-matrix and tensor-times-matrix-chain on an F-COO
build, CP-ALS sweeps, the gradients of a CP model at the nonzeros, and the
build itself.  Sizes follow the synthetic workloads of ``synth`` (the tensors
of ``CONFIGS`` at up to 20M nonzeros) and the ranks of the paper's sweep
(8..64), with ranks between the powers of two that users ask for as often.

Inputs are drawn on the GPU: unique coordinates, uniform or with a truncated
Zipf(1.1) skew per mode, in a shuffled order, values U(0, 1) (planted CP values
for the gradient cases), factors N(0, 1).  A case fixes how its nonzeros share
rows (so that its outputs keep their size); the indices these rows go by, the
order of the nonzeros, the values and the factors come from the seed.
"""
import math

import numpy as np
import torch

from paper_1705_09905_amd import CPAtNonzeros, CPMSELoss, Tensor, cp_als

SKEW = 1.1


def listed():
    def case(name, kind, dims, nnz, rank, dtype="f32", skew=True, mode=0, **more):
        return dict(name=name, kind=kind, dims="x".join(map(str, dims)), nnz=nnz, rank=rank, dtype=dtype, skew=skew,
                    mode=mode, blocks=more.get("blocks", 0))

    zipf3, zipf4 = (100_000, 80_000, 60_000), (50_000, 20_000, 5_000, 1_000)
    return [
        # a call on a small tensor inside a serving loop: latency and launches
        case("mttkrp-small-10k-r8", "mttkrp", (200, 150, 100), 10_000, 8, skew=False),
        # the headline operation on the benchmark's skewed tensor
        case("mttkrp-zipf-20m-r32", "mttkrp", zipf3, 20_000_000, 32),
        # a rank and a nonzero count that no tile or vector width divides, four modes
        case("mttkrp-order4-4m-r25", "mttkrp", zipf4, 4_000_003, 25, mode=1),
        # factors too large for a cache, in the layout for them, bfloat16 storage
        case("mttkrp-uniform-20m-r16-xcd-bf16", "mttkrp", (200_000, 150_000, 100_000), 20_000_000, 16, "bf16",
             skew=False, blocks=8),
        # the second headline operation: short fibres, an output larger than the input
        case("ttm-zipf-20m-r16", "ttm", zipf3, 20_000_000, 16, mode=2),
        # the Tucker kernel: 16 x 16 Kronecker columns per row
        case("ttmc-zipf-10m-r16", "ttmc", zipf3, 10_000_000, 16),
        # CP-ALS from a fresh start, two sweeps: a small tensor ...
        case("cpals-small-10k-r8", "cpals", (200, 150, 100), 10_000, 8, skew=False),
        # ... and an order-4 one with bfloat16 factors
        case("cpals-order4-10m-r32-bf16", "cpals", zipf4, 10_000_000, 32, "bf16"),
        # one training step of gradient CP (loss and all gradients), fused residual
        case("grad-zipf-20m-r64", "grad", (1_000_000, 500_000, 50_000), 20_000_000, 64),
        # ... and of a model at the nonzeros under the program's own loss
        case("adjoint-zipf-5m-r16", "adjoint", zipf3, 5_000_000, 16),
        # a few thousand rows at a rank of ten, as in exploratory fits
        case("ttm-ragged-300k-r10-bf16", "ttm", (3_001, 2_003, 997), 300_007, 10, "bf16", mode=1),
        # the build on the GPU of one mode and its first use
        case("build-zipf-20m-r16", "build", zipf3, 20_000_000, 16),
    ]


def draw(rng):
    """One more case: every kind, orders 3 and 4, 10k to 20M nonzeros, ranks
    3..64 (16 per mode for the chain product), both storage types, odd sizes."""
    kind = rng.choice(["mttkrp", "mttkrp", "mttkrp", "ttm", "ttm", "ttmc", "cpals", "grad", "adjoint", "build"])
    order = 3 if kind in ("ttmc", "grad", "build") else rng.choice([3, 3, 4])
    top = {"mttkrp": 20e6, "ttm": 20e6, "ttmc": 10e6, "cpals": 10e6, "grad": 20e6, "adjoint": 5e6, "build": 20e6}[kind]
    nnz = int(math.exp(rng.uniform(math.log(10e3), math.log(top))))
    if kind == "ttmc":
        rank = rng.choice([4, 5, 8, 10, 12, 16])
    elif rng.random() < 0.5:
        rank = 8 * rng.randint(1, 8)
    else:
        rank = int(math.exp(rng.uniform(math.log(3), math.log(65))))
    # the listed cases' nonzeros x rank bound the drawn ones'
    most = {"ttm": 320e6, "adjoint": 80e6, "cpals": 320e6, "build": 320e6, "mttkrp": 640e6}.get(kind, 1.3e9)
    rank = max(3, min(rank, int(most / nnz)))
    low = max(40, int(nnz ** (0.55 if order == 3 else 0.45)))
    dims = [int(math.exp(rng.uniform(math.log(low), math.log(10 * low)))) for _ in range(order)]
    return dict(kind=kind, dims="x".join(map(str, dims)), nnz=nnz, rank=rank, dtype=rng.choice(["f32", "f32", "bf16"]),
                skew=rng.random() < 0.6, mode=rng.randrange(order),
                blocks=8 if kind == "mttkrp" and nnz > 2e6 and rng.random() < 0.3 else 0)


# ---- inputs ----------------------------------------------------------------

def _dims(case):
    return [int(d) for d in case["dims"].split("x")]


def _tdtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


def _pattern(case):
    """nnz unique coordinates: one int64 column per mode."""
    dims, nnz = _dims(case), case["nnz"]
    g = torch.Generator(device="cuda").manual_seed(1)
    cdfs = None
    if case["skew"]:
        w = [torch.arange(1, d + 1, dtype=torch.float64, device="cuda") ** -SKEW for d in dims]
        cdfs = [torch.cumsum(x / x.sum(), 0) for x in w]
    keys = torch.empty(0, dtype=torch.int64, device="cuda")
    while keys.numel() < nnz:
        n = max(1024, int(1.2 * (nnz - keys.numel())) + 64)
        key = torch.zeros(n, dtype=torch.int64, device="cuda")
        for m, d in enumerate(dims):
            if cdfs is None:
                c = torch.randint(0, d, (n,), generator=g, device="cuda")
            else:
                u = torch.rand(n, generator=g, dtype=torch.float64, device="cuda")
                c = torch.searchsorted(cdfs[m], u).clamp_(max=d - 1)
            key = key * d + c
        keys = torch.unique(torch.cat([keys, key]))
    keys = keys[torch.randperm(keys.numel(), generator=g, device="cuda")[:nnz]]
    cols = []
    for d in reversed(dims):
        cols.append(keys % d)
        keys = keys // d
    return cols[::-1]


def _coords(case, g):
    """The case's coordinates with the seed's indices and order."""
    order = torch.randperm(case["nnz"], generator=g, device="cuda")
    return [torch.randperm(d, generator=g, device="cuda")[c[order]] for c, d in zip(_pattern(case), _dims(case))]


def _chunks(n, rank):
    step = max(1, (1 << 26) // rank)
    return [slice(s, min(n, s + step)) for s in range(0, n, step)]


def _rows(cols, factors, sl, skip=-1):
    """Products of the factors' rows at the nonzeros of `sl` (all modes but `skip`)."""
    p = None
    for m, f in enumerate(factors):
        if m != skip:
            r = f[cols[m][sl]]
            p = r if p is None else p * r
    return p


def _inputs(case, seed):
    """(coordinate columns, float32 values, factors in the storage type)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    cols = _coords(case, g)
    normal = lambda r: [torch.randn(d, r, generator=g, device="cuda") for d in _dims(case)]  # noqa: E731
    if case["kind"] in ("grad", "adjoint"):
        planted, vals = normal(8), torch.empty(case["nnz"], device="cuda")
        for sl in _chunks(case["nnz"], 8):
            vals[sl] = _rows(cols, planted, sl).sum(1)
        vals += 0.1 * torch.randn(case["nnz"], generator=g, device="cuda")
        factors = [0.5 * f for f in normal(case["rank"])]
    else:
        vals = torch.rand(case["nnz"], generator=g, device="cuda")
        factors = normal(case["rank"])
    if case["kind"] not in ("cpals", "grad"):  # those two keep float32 masters and take the storage type as an option
        factors = [f.to(_tdtype(case)) for f in factors]
    return cols, vals, factors


class _State:
    pass


def prepare(case, seed):
    """The tensor's handle with the builds its program keeps, and the factors."""
    cols, vals, factors = _inputs(case, seed)
    s = _State()
    s.case, s.factors = case, factors
    s.tensor = Tensor([c.to(torch.int32).cpu().numpy() for c in cols], vals.cpu().numpy(), _dims(case))
    kind, mode = case["kind"], case["mode"]
    if kind in ("mttkrp", "ttmc"):
        s.tensor.build(mode, "mttkrp", device=True, xcd_blocks=case["blocks"])
    elif kind == "ttm":
        s.tensor.build(mode, "ttm", device=True)
    elif kind in ("cpals", "grad", "adjoint"):
        for m in range(s.tensor.order):
            s.tensor.build(m, "mttkrp", device=True)
    if kind == "adjoint":
        s.target = vals
    if kind in ("grad", "adjoint"):
        for f in s.factors:
            f.requires_grad_(True)
    return s


def run(s):
    case, t, f = s.case, s.tensor, s.factors
    kind, mode, rank = case["kind"], case["mode"], case["rank"]
    if kind == "mttkrp":
        return t.spmttkrp(mode, f)
    if kind == "ttm":
        return t.spttm(mode, f[mode])
    if kind == "ttmc":
        return t.spttmc(mode, f)
    if kind == "build":
        t.build(mode, "mttkrp", device=True)
        return t.spmttkrp(mode, f)
    if kind == "cpals":
        # the weights as the program keeps them beside its factors: float32
        # (they come in float64, computed from float32 sums)
        r = cp_als(t, rank, 2, f, dtype=case["dtype"], build=False)
        return dict(factors=r["factors"], lam=r["lam"].float(), fits=r["fits"], used_pinv=r["used_pinv"])
    if kind == "grad":
        loss = CPMSELoss.apply(t, case["dtype"], *f)
        return dict(loss=loss.detach().float(), grads=list(torch.autograd.grad(loss, f)))
    xhat = CPAtNonzeros.apply(t, *f)
    # the program's own loss: the derivative of its mean square, here
    g = (xhat.detach() - s.target) / t.nnz
    return dict(xhat=xhat.detach(), grads=list(torch.autograd.grad(xhat, f, g)))


# ---- what a pass cannot do without -------------------------------------------

def _segments(case):
    """Fibres of a TTM case: the rows of its output."""
    cols = _pattern(case)
    key = torch.zeros_like(cols[0])
    for m, d in enumerate(_dims(case)):
        if m != case["mode"]:
            key = key * d + cols[m]
    return torch.unique(key).numel()


def work(case):
    kind, mode, dims, nnz, r = case["kind"], case["mode"], _dims(case), case["nnz"], case["rank"]
    n, size = len(dims), 4 if case["dtype"] == "f32" else 2
    rest = sum(dims) - dims[mode]

    def mttkrp(m, extra=0.0):
        return nnz * (4 * n + 1 / 8 + extra) + (sum(dims) - dims[m]) * r * size + dims[m] * r * 4

    if kind == "mttkrp":
        return dict(bytes=mttkrp(mode), flops=nnz * r * n)
    if kind == "ttm":
        return dict(bytes=nnz * (8 + 1 / 8) + dims[mode] * r * size + _segments(case) * r * 4, flops=2 * nnz * r)
    if kind == "ttmc":
        w = r ** (n - 1)
        return dict(bytes=nnz * (4 * n + 1 / 8) + rest * r * size + dims[mode] * w * 4, flops=2 * nnz * w)
    if kind == "cpals":
        one = sum(mttkrp(m) for m in range(n)) + 2 * sum(dims) * r * size
        return dict(bytes=2 * one, flops=2 * n * nnz * r * n + 2 * 4 * sum(dims) * r * r)
    if kind == "grad":
        return dict(bytes=sum(mttkrp(m) + dims[m] * r * size for m in range(n)), flops=n * nnz * r * (n + 4))
    if kind == "adjoint":
        model = nnz * (4 * n + 4) + sum(dims) * r * size
        return dict(bytes=model + sum(mttkrp(m, 4) for m in range(n)), flops=nnz * r * (n + n * n))
    # build: the coordinates and values read, the encoded arrays and the permutation written
    return dict(bytes=nnz * (4 * n + 4) + nnz * (4 * n + 4 + 1 / 8) + mttkrp(mode), flops=nnz * r * n)


# ---- the same in 64 bits -------------------------------------------------------

def _sum64(at, n, width, rows):
    """out[at[e]] += rows(e) in float64: running sums over the nonzeros sorted
    by `at`, so that a row that a tenth of them share is no chain of atomics."""
    out = torch.zeros(n, width, dtype=torch.float64, device="cuda")
    at, order = torch.sort(at)
    for sl in _chunks(at.numel(), width):
        a = at[sl]
        sums = rows(order[sl]).T.contiguous().cumsum(1)
        ends = torch.cat([a[1:] != a[:-1], a.new_ones(1, dtype=torch.bool)]).nonzero()[:, 0]
        sums = sums[:, ends]
        out[a[ends]] += torch.diff(sums, dim=1, prepend=torch.zeros_like(sums[:, :1])).T
    return out


def _mttkrp64(case, cols, vals, factors, mode):
    return _sum64(cols[mode], _dims(case)[mode], factors[0].shape[1],
                  lambda e: _rows(cols, factors, e, mode) * vals[e, None])


def _model64(case, cols, factors):
    out = torch.empty(case["nnz"], dtype=torch.float64, device="cuda")
    for sl in _chunks(case["nnz"], factors[0].shape[1]):
        out[sl] = _rows(cols, factors, sl).sum(1)
    return out


def exact(case, seed):
    cols, vals, factors = _inputs(case, seed)
    kind, mode, dims, nnz = case["kind"], case["mode"], _dims(case), case["nnz"]
    if kind == "grad":  # the kernels read the factors in the storage type
        factors = [f.to(_tdtype(case)) for f in factors]
    vals, factors = vals.double(), [f.double() for f in factors]
    if kind in ("mttkrp", "build"):
        return _mttkrp64(case, cols, vals, factors, mode)
    if kind == "ttm":
        key = torch.zeros_like(cols[0])
        for m, d in enumerate(dims):
            if m != mode:
                key = key * d + cols[m]
        fibres, at = torch.unique(key, return_inverse=True)
        return _sum64(at, fibres.numel(), case["rank"], lambda e: factors[mode][cols[mode][e]] * vals[e, None])
    if kind == "ttmc":
        others = [m for m in range(len(dims)) if m != mode]

        def kron(e):
            p = vals[e, None]
            for m in others:
                p = (p[:, :, None] * factors[m][cols[m][e]][:, None, :]).flatten(1)
            return p

        return _sum64(cols[mode], dims[mode], case["rank"] ** len(others), kron)
    if kind == "cpals":
        return _als64(case, cols, vals, factors)
    xhat = _model64(case, cols, factors)
    g = (xhat - vals) / nnz
    grads = [_mttkrp64(case, cols, g, factors, m) for m in range(len(dims))]
    if kind == "grad":
        return dict(loss=((xhat - vals) ** 2).sum() / (2 * nnz), grads=grads)
    return dict(xhat=xhat, grads=grads)


def _als64(case, cols, vals, factors):
    """Two sweeps of CP-ALS with 2-norm columns; the fit after each."""
    n, norm = len(factors), vals.norm()
    grams, fits = [f.T @ f for f in factors], []
    for _ in range(2):
        for m in range(n):
            M = _mttkrp64(case, cols, vals, factors, m)
            v = torch.ones_like(grams[0])
            for k in range(n):
                if k != m:
                    v = v * grams[k]
            a = torch.linalg.solve(v, M.T).T
            lam = a.norm(dim=0)
            factors[m] = (a / lam).contiguous()
            grams[m] = factors[m].T @ factors[m]
        v = torch.ones_like(grams[0])
        for k in range(n):
            v = v * grams[k]
        left = norm ** 2 + lam @ v @ lam - 2 * ((M * factors[-1]).sum(0) @ lam)
        fits.append(float(1 - left.clamp(min=0).sqrt() / norm))
    return dict(factors=factors, lam=lam, fits=fits, used_pinv=[None, None])
