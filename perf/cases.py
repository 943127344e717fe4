"""The workloads this framework is timed on, through its public entry points.

``listed`` names them, ``draw`` gives one more of the same ranges,
``prepare`` makes what a program holds before a call (a plan or network, its
state and workspace), ``run`` is one pass, ``work`` the bytes and operations a
pass cannot do without, and ``exact`` the same results in 64-bit torch.

A case is one of six kinds:

* ``rod``    ge.Plan.step_n on one rod (two-point groups), with constant or
             moving walls and with or without a source; the compensated pair
             is read back as FP64, as a checkpoint of such a run is;
* ``sdc``    ge.Plan.step_n with sub-domains of k nodes (the paper's own form);
* ``batch``  ge.Batch.solve on many independent rods of uneven length;
* ``grid``   ge.step2d_n on the unit square;
* ``jump``   ge.Net.jump: inference of the learned 64-level propagator;
* ``grads``  ge.Net.grads: forward, loss and backward of a training minibatch.

Every call advances the state in place from level 0; a repeated pass goes on
from where the last one ended.
"""
import math

import numpy as np
import torch

from paper_1310_3422_amd import ge

NMODES = 16

# The dearest listed pass in point-levels (the moving-wall rod): a drawn case
# of a sweep stays below a quarter of it.
MOST = (1 << 27) * 600


def listed():
    return [
        # the smallest call: a rod of one window for a few levels, as an
        # interactive or coupled program steps it (latency)
        dict(name="rod_step_fp32", kind="rod", n=1001, r=0.8, levels=16, precision="fp32",
             moving=False, source=False),
        # the closed-form check of the method: sin(pi x), 1024 points, 1000 levels
        dict(name="rod_1024_fp64", kind="rod", n=1024, r=1.0, levels=1000, precision="fp64",
             moving=False, source=False),
        # the paper's timing experiment at its node count, 1200 time rows: a
        # rod too small to fill the chip
        dict(name="rod_262655_fp64", kind="rod", n=262655, r=2.0, levels=1200, precision="fp64",
             moving=False, source=False),
        # a large rod, FP64, library defaults
        dict(name="rod_2p24_fp64", kind="rod", n=1 << 24, r=2.0, levels=2000, precision="fp64",
             moving=False, source=False),
        # the headline workload: the largest rod, moving wall and source
        dict(name="rod_2p27_walls_fp64", kind="rod", n=1 << 27, r=4.0, levels=600,
             precision="fp64", moving=True, source=True),
        # the same problem in the compensated FP32 pair, a ragged length
        dict(name="rod_walls_fp32c", kind="rod", n=(1 << 24) + 77, r=4.0, levels=600,
             precision="fp32c", moving=True, source=True),
        # the paper's scheme: sub-domains of 16 nodes, FP64
        dict(name="sdc_k16_fp64", kind="sdc", n=(1 << 24) - 1, k=16, r=2.0, levels=1000,
             precision="fp64"),
        # a production batch: 4096 uneven rods, FP32, 2000 levels in one launch
        dict(name="batch_4096_fp32", kind="batch", nrods=4096, nmin=256, nmax=65536, rmin=0.25,
             rmax=4.0, levels=2000, precision="fp32"),
        # what the surrogate's training data and re-checks ask of the batch
        # sweep: rods of 4096 points, 64 levels, FP64
        dict(name="batch_ge64_fp64", kind="batch", nrods=1024, nmin=4096, nmax=4096, rmin=0.5,
             rmax=2.0, levels=64, precision="fp64"),
        # two dimensions, FP64, library depth
        dict(name="grid_4096_fp64", kind="grid", nx=4096, ny=4096, rx=2.0, ry=2.0, levels=200,
             precision="fp64"),
        # surrogate inference
        dict(name="jump_1024", kind="jump", width=4096, batch=1024),
        # one training minibatch of the surrogate
        dict(name="grads_64", kind="grads", width=4096, batch=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["rod", "rod", "rod", "sdc", "batch", "batch", "grid", "grid", "jump",
                       "grads"])
    most = MOST // 4
    if kind == "rod":
        n = _log_int(rng, 512, 1 << 25)
        levels = min(_log_int(rng, 16, 2000), most // n)
        return dict(kind=kind, n=n, r=round(rng.uniform(0.25, 4.0), 3), levels=levels,
                    precision=rng.choice(["fp64", "fp64", "fp32", "fp32c"]),
                    moving=rng.random() < 0.5, source=rng.random() < 0.4)
    if kind == "sdc":
        k = rng.choice([2, 4, 8, 16, 16])
        n = 2 * k * _log_int(rng, 512 // k, (1 << 23) // k) - 1
        levels = min(_log_int(rng, 16, 1200), most // 2 // n)
        return dict(kind=kind, n=n, k=k, r=round(rng.uniform(0.25, 4.0), 3), levels=levels,
                    precision=rng.choice(["fp64", "fp64", "fp32"]))
    if kind == "batch":
        nmin = _log_int(rng, 200, 4096)
        return dict(kind=kind, nrods=_log_int(rng, 16, 2048), nmin=nmin,
                    nmax=min(65536, nmin * _log_int(rng, 1, 64)), rmin=0.25, rmax=4.0,
                    levels=_log_int(rng, 16, 1000),
                    precision=rng.choice(["fp32", "fp32", "fp64", "fp32c"]))
    if kind == "grid":
        return dict(kind=kind, nx=_log_int(rng, 64, 4096), ny=_log_int(rng, 64, 4096),
                    rx=round(rng.uniform(0.25, 4.0), 3), ry=round(rng.uniform(0.25, 4.0), 3),
                    levels=_log_int(rng, 8, 200), precision=rng.choice(["fp64", "fp64", "fp32"]))
    width = 128 * _log_int(rng, 4, 32)
    return dict(kind=kind, width=width,
                batch=_log_int(rng, 1, 1024) if kind == "jump" else _log_int(rng, 2, 128))


# ---- inputs ----------------------------------------------------------------
def _device():
    return "cuda" if torch.cuda.is_available() else "cpu"


def _f64(a):
    return torch.as_tensor(np.ascontiguousarray(a, dtype=np.float64)).to(_device())


def _rounded(u, precision):
    """The values a state of this precision starts from."""
    return u.float().double() if precision == "fp32" else u


def _rod_data(case, seed):
    """u0, wall values per level (or constants), source factors and profile:
    sine modes with coefficients z_k / k^2 on top of the steady state of the
    first wall values; g_L(t) = gl + sin(2 pi t), f = exp(-t) x (1 - x)."""
    rng = np.random.default_rng(seed)
    z = rng.standard_normal(NMODES)
    gl, gr = (float(v) for v in rng.uniform(-1.0, 1.0, 2))
    n, levels = case["n"], case["levels"]
    x = torch.arange(1, n + 1, dtype=torch.float64, device=_device()) / (n + 1)
    u0 = gl + (gr - gl) * x
    for k in range(1, NMODES + 1):
        u0 += (z[k - 1] / (k * k)) * torch.sin(k * math.pi * x)
    h = 1.0 / (n + 1)
    tau = case["r"] * h * h
    t = np.arange(levels + 1, dtype=np.float64) * tau
    moving, source = case.get("moving", False), case.get("source", False)
    b = x * (1.0 - x) if source else None
    if source and case["precision"] != "fp64":
        b = b.float().double()
    return dict(u0=_rounded(u0, case["precision"]), gl=gl, gr=gr, tau=tau,
                gl_t=gl + np.sin(2.0 * math.pi * t) if moving else None,
                gr_t=np.full(levels + 1, gr) if moving else None,
                b=b, a=np.exp(-(t[:-1] + 0.5 * tau)) if source else None)


def _batch_data(case, seed):
    """Rod table (N log-uniform, the case's own; r uniform, walls uniform in
    [-1, 1]) and the packed initial values, rods aligned to 4 values, zeros
    between them."""
    nr = case["nrods"]
    rng = np.random.default_rng([nr, case["nmin"], case["nmax"]])
    n = np.rint(np.exp(rng.uniform(math.log(case["nmin"]), math.log(case["nmax"]), nr)))
    n = n.astype(np.int64)
    rng = np.random.default_rng(seed)
    r = rng.uniform(case["rmin"], case["rmax"], nr)
    gl, gr = rng.uniform(-1.0, 1.0, nr), rng.uniform(-1.0, 1.0, nr)
    z = rng.standard_normal((nr, NMODES))
    offsets = np.zeros(nr + 1, dtype=np.int64)
    offsets[1:] = np.cumsum((n + 3) // 4 * 4)
    dev = _device()
    rod = torch.repeat_interleave(torch.arange(nr, device=dev),
                                  torch.as_tensor(np.diff(offsets)).to(dev))
    i = torch.arange(int(offsets[-1]), device=dev) - torch.as_tensor(offsets).to(dev)[rod] + 1
    nn = torch.as_tensor(n).to(dev)[rod]
    inside = i <= nn
    x = i.double() / (nn + 1).double()
    u0 = torch.zeros_like(x)
    zt = _f64(z)
    for k in range(1, NMODES + 1):
        u0 += (zt[:, k - 1] / (k * k))[rod] * torch.sin(k * math.pi * x)
    u0 = torch.where(inside, u0, torch.zeros_like(u0))
    return dict(n=n, offsets=offsets, r=r, gl=gl, gr=gr, u0=_rounded(u0, case["precision"]))


def _grid_data(case, seed):
    """Smooth separable modes plus rough values; walls uniform in [-1, 1]."""
    rng = np.random.default_rng(seed)
    nx, ny = case["nx"], case["ny"]
    x = np.arange(1, nx + 1) / (nx + 1)
    y = np.arange(1, ny + 1) / (ny + 1)
    k = np.arange(1, 9)
    z = rng.standard_normal((8, 8)) / np.outer(k, k)
    u0 = (_f64(np.sin(math.pi * np.outer(y, k))) @ _f64(z)) @ _f64(np.sin(math.pi * np.outer(k, x)))
    gen = torch.Generator(device=_device()).manual_seed(int(seed))
    u0 += 0.05 * torch.randn(ny, nx, dtype=torch.float64, device=_device(), generator=gen)
    walls = tuple(float(v) for v in rng.uniform(-1.0, 1.0, 4))
    return dict(u0=_rounded(u0, case["precision"]), walls=walls)


LAYERS = [(2, 64), (64, 64), (64, 64), (64, 64), (64, 64), (64, 1)]
DILATIONS = [1, 2, 4, 8, 16, 1]


def _net_data(case, seed):
    """He-style weights with small biases, rods of sine modes up to a cutoff
    with zero walls (r in [0.5, 2]) and, for training, states 64 levels on
    (each mode damped by its own rate)."""
    rng = np.random.default_rng(seed)
    flat = []
    for li, (ci, co) in enumerate(LAYERS):
        std = math.sqrt(2.0 / (5 * ci)) * (0.1 if li == 5 else 1.0)
        flat += [(rng.standard_normal((5, co, ci)) * std).ravel(), 0.05 * rng.standard_normal(co)]
    params = np.concatenate(flat).astype(np.float32)
    w, nb, modes = case["width"], case["batch"], 64
    r = rng.uniform(0.5, 2.0, nb)
    k = np.arange(1, modes + 1, dtype=np.float64)
    z = rng.standard_normal((nb, modes)) / (k * k)
    basis = _f64(np.sin(math.pi * np.outer(k, np.arange(1, w + 1) / (w + 1))))
    lam = 2.0 - 2.0 * np.cos(math.pi * k / (w + 1))
    u = (_f64(z) @ basis).float()
    u64 = (_f64(z * np.exp(-64.0 * np.outer(r, lam))) @ basis).float()
    return dict(params=params, u=u, u64=u64, r=torch.as_tensor(r).float().to(_device()))


# ---- one pass --------------------------------------------------------------
def _pair(u0):
    """FP64 values as the compensated pair of ge_comp_from_fp64's layout."""
    return ge.comp_from_fp64(u0)


def prepare(case, seed):
    kind = case["kind"]
    if kind in ("rod", "sdc"):
        d = _rod_data(case, seed)
        p = case["precision"]
        b = d["b"] if d["b"] is None else d["b"].to(ge.state_dtype(p))
        plan = ge.Plan(case["n"], case["r"], p, g_left=d["gl"], g_right=d["gr"], src_b=b,
                       k=case.get("k", 0))
        u = _pair(d["u0"]) if p == "fp32c" else d["u0"].to(ge.state_dtype(p))
        dev = lambda a: None if a is None else _f64(a)  # noqa: E731
        return dict(case=case, plan=plan, u=u, ws=plan.new_workspace(), gl=dev(d["gl_t"]),
                    gr=dev(d["gr_t"]), a=dev(d["a"]))
    if kind == "batch":
        d = _batch_data(case, seed)
        p = case["precision"]
        batch = ge.Batch(d["n"], d["offsets"], d["r"], d["gl"], d["gr"], p)
        u = _pair(d["u0"]) if p == "fp32c" else d["u0"].to(ge.state_dtype(p))
        return dict(case=case, batch=batch, u=u, ws=batch.new_workspace(),
                    total=int(d["offsets"][-1]))
    if kind == "grid":
        d = _grid_data(case, seed)
        u = d["u0"].to(ge.state_dtype(case["precision"])).contiguous()
        return dict(case=case, u=u, ws=torch.empty_like(u).view(torch.uint8), walls=d["walls"])
    d = _net_data(case, seed)
    net = ge.Net(width=case["width"], max_batch=case["batch"], seed=1)
    net.set_params(d["params"])
    return dict(case=case, net=net, u=d["u"].reshape(-1), u64=d["u64"].reshape(-1), r=d["r"],
                out=torch.empty_like(d["u"].reshape(-1)))


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind in ("rod", "sdc"):
        u = state["plan"].step_n(state["u"], 0, case["levels"], workspace=state["ws"],
                                 g_left_t=state["gl"], g_right_t=state["gr"], src_a_t=state["a"])
        return ge.comp_to_fp64(u, case["n"]) if case["precision"] == "fp32c" else u
    if kind == "batch":
        u = state["batch"].solve(state["u"], 0, case["levels"], state["ws"])
        return ge.comp_to_fp64(u, state["total"]) if case["precision"] == "fp32c" else u
    if kind == "grid":
        return ge.step2d_n(state["u"], case["nx"], case["ny"], case["rx"], case["ry"], 0,
                           case["levels"], case["precision"], state["walls"],
                           workspace=state["ws"])
    if kind == "jump":
        return state["net"].jump(state["u"], state["r"], out=state["out"])
    return state["net"].grads(state["u"], state["u64"], state["r"])


# ---- what a pass cannot do without -----------------------------------------
def work(case):
    """The state read once and written once (and a source profile read), and
    the operations of the scheme as the paper's formulas need them at least:
    a pair's two points take 4 subtractions and 4 multiply-adds in second
    differences, 6 flops a point and level (8 with a source, 12 for the pair
    with its compensation), a sub-domain node 5, a grid point 12; the network
    2 x 5 x c_in x c_out a point and layer, three times that with a backward."""
    kind = case["kind"]
    if kind in ("jump", "grads"):
        points = case["width"] * case["batch"]
        flops = points * sum(2 * 5 * ci * co for ci, co in LAYERS)
        if kind == "jump":
            return dict(bytes=points * 8 + 83201 * 2, flops=flops)
        first = points * 2 * 5 * 2 * 64      # the input takes no gradient
        return dict(bytes=points * 8 + 83201 * 6, flops=3 * flops - first)
    p = case["precision"]
    size = {"fp64": 8, "fp32": 4, "fp32c": 8}[p]
    per = {"fp64": 6, "fp32": 6, "fp32c": 12}[p]
    if kind == "grid":
        points, per = case["nx"] * case["ny"], 12
    elif kind == "batch":
        if case["nmin"] == case["nmax"]:
            mean = case["nmin"]
        else:
            mean = (case["nmax"] - case["nmin"]) / math.log(case["nmax"] / case["nmin"])
        points = case["nrods"] * mean
    else:
        points = case["n"]
        if kind == "sdc":
            per = 5
    nbytes = 2 * size * points
    if case.get("source"):
        nbytes += (8 if p == "fp64" else 4) * points
        per += 2
    if p == "fp32c":
        nbytes += 8 * points                 # the FP64 values read back
    return dict(bytes=float(nbytes), flops=float(per * points * case["levels"]))


# ---- the same results in 64 bits -------------------------------------------
def _level(U, r, p, west, east, src=None):
    """One level of parity p along the last axis of U (walls in its first and
    last place, holding the level's old values); west, east: the new ones.
    Explicit part of the old neighbours, then each pair's 2x2 solve; a point
    left alone beside a wall takes Eq. (1) or (2)."""
    n = U.shape[-1] - 2
    first = 1 + p
    pairs = (n - p) // 2
    last = first + 2 * pairs                       # one past the paired points
    V = U.clone()
    if pairs:
        a, b = U[..., first:last:2], U[..., first + 1:last:2]
        l, g = U[..., first - 1:last - 1:2], U[..., first + 2:last + 1:2]
        va = a + r * (l - a)
        vb = b + r * (g - b)
        if src is not None:
            va += src[first:last:2]
            vb += src[first + 1:last:2]
        d = (vb - va) * (r / (1.0 + 2.0 * r))
        V[..., first:last:2] = va + d
        V[..., first + 1:last:2] = vb - d
    if p:
        v = U[..., 1] + r * (U[..., 2] - U[..., 1])
        if src is not None:
            v = v + src[1]
        V[..., 1] = v + (r / (1.0 + r)) * (west - v)
    if last == n:
        v = U[..., n] + r * (U[..., n - 1] - U[..., n])
        if src is not None:
            v = v + src[n]
        V[..., n] = v + (r / (1.0 + r)) * (east - v)
    V[..., 0], V[..., -1] = west, east
    return V


def _exact_rod(case, seed):
    d = _rod_data(case, seed)
    L = case["levels"]
    gl = d["gl_t"] if d["gl_t"] is not None else np.full(L + 1, d["gl"])
    gr = d["gr_t"] if d["gr_t"] is not None else np.full(L + 1, d["gr"])
    n = case["n"]
    U = torch.empty(n + 2, dtype=torch.float64, device=_device())
    U[1:-1] = d["u0"]
    U[0], U[-1] = gl[0], gr[0]
    B = torch.zeros_like(U) if d["b"] is not None else None
    if B is not None:
        B[1:-1] = d["tau"] * d["b"]
    for m in range(L):
        src = B * d["a"][m] if B is not None else None
        U = _level(U, case["r"], m & 1, gl[m + 1], gr[m + 1], src)
    return U[1:-1].clone()


def _exact_sdc(case, seed):
    """Sub-domains as rows: node j of couple i at S[j, i]."""
    d = _rod_data(case, seed)
    n, k, r, c = case["n"], case["k"], case["r"], 2 * case["k"]
    e = (n + 1) // c
    nodes = torch.empty(n + 1, dtype=torch.float64, device=_device())
    nodes[0] = d["gl"]
    nodes[1:] = d["u0"]
    S = nodes.reshape(e, c).t().contiguous()
    gl, gr = d["gl"], d["gr"]
    den, q = 1.0 + 2.0 * r, 1.0 + r

    def pair(l, a, b, g):
        va, vb = a + r * (l - a), b + r * (g - b)
        t = (vb - va) * (r / den)
        return va + t, vb - t

    def chain(new, own, old):                      # predecessor at the new level
        return (r * new + (1.0 - r) * own + r * old) / q

    for m in range(case["levels"]):
        V = torch.empty_like(S)
        if m % 2 == 0:
            right, left = S[0].clone(), S[c - 1].clone()
            if e > 1:
                v, w = pair(S[c - 2, :-1], S[c - 1, :-1], S[0, 1:], S[1, 1:])
                left[:-1], right[1:] = v, w
            right[0] = gl
            left[-1] = chain(torch.tensor(gr, dtype=torch.float64, device=S.device),
                             S[c - 1, -1], S[c - 2, -1])
            V[0], V[c - 1] = right, left
            for j in range(1, k):
                V[j] = chain(V[j - 1], S[j], S[j + 1])
            for j in range(c - 2, k - 1, -1):
                V[j] = chain(V[j + 1], S[j], S[j - 1])
        else:
            V[k - 1], V[k] = pair(S[k - 2], S[k - 1], S[k], S[k + 1])
            before = torch.cat([torch.full_like(S[0, :1], gl), S[c - 1, :-1]])
            after = torch.cat([S[0, 1:], torch.full_like(S[0, :1], gr)])
            for j in range(k - 2, -1, -1):
                V[j] = chain(V[j + 1], S[j], S[j - 1] if j > 0 else before)
            V[0, 0] = gl
            for j in range(k + 1, c):
                V[j] = chain(V[j - 1], S[j], S[j + 1] if j < c - 1 else after)
        S = V
    return S.t().reshape(-1)[1:].clone()


def _exact_batch(case, seed):
    """All rods in one array, walls in the places around each rod, every rod's
    left wall at an even place, so that one stride-2 view pairs them all; the
    points alone beside a wall are put right afterwards."""
    d = _batch_data(case, seed)
    n, nr, L = d["n"], case["nrods"], case["levels"]
    dev = _device()
    base = np.zeros(nr + 1, dtype=np.int64)
    base[1:] = np.cumsum((n + 2 + 1) // 2 * 2)
    total = int(base[-1]) + 2
    place = np.repeat(base[:-1] - d["offsets"][:-1] + 1, n) + np.concatenate(
        [np.arange(o, o + c) for o, c in zip(d["offsets"][:-1], n)])
    packed = np.concatenate([np.arange(o, o + c) for o, c in zip(d["offsets"][:-1], n)])
    place, packed = torch.as_tensor(place).to(dev), torch.as_tensor(packed).to(dev)
    U = torch.zeros(total, dtype=torch.float64, device=dev)
    U[place] = d["u0"][packed]
    west, east = torch.as_tensor(base[:-1]).to(dev), torch.as_tensor(base[:-1] + n + 1).to(dev)
    gl, gr, r1 = _f64(d["gl"]), _f64(d["gr"]), _f64(d["r"])
    rod = torch.repeat_interleave(torch.arange(nr, device=dev),
                                  torch.as_tensor(np.diff(base)).to(dev))
    R = torch.ones(total, dtype=torch.float64, device=dev)
    R[:rod.numel()] = r1[rod]
    kap = R / (1.0 + 2.0 * R)
    U[west], U[east] = gl, gr
    odd = torch.as_tensor(n & 1).to(dev).bool()
    for m in range(L):
        p = m & 1
        f, t = 1 + p, total - 1 - (total - 2 - p) % 2
        a, b, l, g = U[f:t:2], U[f + 1:t:2], U[f - 1:t - 1:2], U[f + 2:t + 1:2]
        ra, rb = R[f:t:2], R[f + 1:t:2]
        va, vb = torch.addcmul(a, ra, l - a), torch.addcmul(b, rb, g - b)
        w = (vb - va) * kap[f:t:2]
        V = U.clone()
        V[f:t:2] = va + w
        V[f + 1:t:2] = vb - w
        if p:
            v = U[west + 1] + r1 * (U[west + 2] - U[west + 1])
            V[west + 1] = v + (r1 / (1.0 + r1)) * (gl - v)
        alone = odd if p == 0 else ~odd
        i, rr = east[alone] - 1, r1[alone]
        v = U[i] + rr * (U[i - 1] - U[i])
        V[i] = v + (rr / (1.0 + rr)) * (gr[alone] - v)
        V[west], V[east] = gl, gr
        U = V
    out = torch.zeros_like(d["u0"])
    out[packed] = U[place]
    return out


def _exact_grid(case, seed):
    d = _grid_data(case, seed)
    gw, g_e, gs, gn = d["walls"]
    u = d["u0"]
    for m in range(case["levels"]):
        U = torch.nn.functional.pad(u, (1, 1))
        U[:, 0], U[:, -1] = gw, g_e
        u = _level(U, case["rx"], m & 1, gw, g_e)[:, 1:-1]
        U = torch.nn.functional.pad(u, (0, 0, 1, 1)).t()
        U[:, 0], U[:, -1] = gs, gn
        u = _level(U, case["ry"], m & 1, gs, gn)[:, 1:-1].t()
    return u.contiguous()


def _gelu(z):
    return 0.5 * z * (1.0 + torch.tanh(math.sqrt(2.0 / math.pi) * (z + 0.044715 * z ** 3)))


def _exact_net(case, seed):
    d = _net_data(case, seed)
    nb, w = case["batch"], case["width"]
    part = max(1, (1 << 20) // w)                  # rods at once
    P = _f64(d["params"])
    if case["kind"] == "grads":
        P.requires_grad_(True)
    layers, at = [], 0
    for ci, co in LAYERS:
        layers.append((P[at:at + 5 * co * ci].reshape(5, co, ci), P[at + 5 * co * ci:][:co]))
        at += 5 * co * ci + co
    outs, loss = [], 0.0
    for i in range(0, nb, part):
        u, r = d["u"][i:i + part].double(), d["r"][i:i + part].double()
        up = torch.nn.functional.pad(u, (1, 1))
        D = up[:, :-2] - 2.0 * up[:, 1:-1] + up[:, 2:]
        s = D.square().mean(1).sqrt()
        h = torch.stack([D / s[:, None], ((r - 1.25) / 0.75)[:, None].expand_as(D)], 2)
        for li, (W, b) in enumerate(layers):
            dl = DILATIONS[li]
            hp = torch.nn.functional.pad(h, (0, 0, 2 * dl, 2 * dl))
            pre = b
            for t in range(5):
                pre = pre + (hp[:, t * dl:t * dl + w].reshape(-1, h.shape[2])
                             @ W[t].t()).reshape(h.shape[0], w, -1)
            h = pre if li == 5 else _gelu(pre) if li == 0 else h + _gelu(pre)
        step = (64.0 * r * s)[:, None]
        if case["kind"] == "jump":
            outs.append(u + step * h[:, :, 0])
        else:
            part_loss = (h[:, :, 0] - (d["u64"][i:i + part].double() - u) / step).square().sum()
            part_loss = part_loss / (nb * w)
            part_loss.backward(retain_graph=True)
            loss += float(part_loss.detach())
    if case["kind"] == "jump":
        return torch.cat(outs).reshape(-1)
    return torch.tensor([loss], dtype=torch.float64), P.grad.detach()


def exact(case, seed):
    kind = case["kind"]
    if kind == "rod":
        return _exact_rod(case, seed)
    if kind == "sdc":
        return _exact_sdc(case, seed)
    if kind == "batch":
        return _exact_batch(case, seed)
    if kind == "grid":
        return _exact_grid(case, seed)
    return _exact_net(case, seed)
