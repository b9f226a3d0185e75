"""The calls that this library's users make, as cases that can be timed and compared.

A case is an operation (one call of ``paper_2011_13824_amd.lirpa.Network``) on a network with a
batch of sub-domains:

* ``bound``     lower bounds of every property row; with the intermediate bounds and stability
                codes where ``lu`` is set (a root's, or those a search branches on);
* ``child``     bounds of sub-domains whose parents' intermediate bounds are known;
* ``ul``        lower and upper bounds in one call;
* ``grad``      bounds and the gradient with respect to the lower slopes;
* ``optimize``  a fresh projected-Adam run on the lower slopes;
* ``bab``       the batched branch-and-bound search on one property.

The networks are the four of this repository's configurations (``tiny``, ``base``, ``wide``,
``deep``), the small ragged convolution of its tests (``small``), one-channel 28x28 images
through the same kind of two-convolution net (``gray``), and fully connected layers (``mlp``).
"""
from __future__ import annotations

import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2011_13824_amd import lirpa
from paper_2011_13824_amd import workloads as wl

NETS = {
    "tiny": wl.ARCHS["tiny"],
    "base": wl.ARCHS["base"],
    "wide": wl.ARCHS["wide"],
    "deep": wl.ARCHS["deep"],
    "small": [wl.conv(2, 9, 4, 3, 2, 1), wl.conv(4, 5, 3, 2, 1, 0), wl.fc(48, 7), wl.fc(7, 3)],
    "gray": [wl.conv(1, 28, 16, 4, 2, 1), wl.conv(16, 14, 32, 4, 2, 1), wl.fc(1568, 100),
             wl.fc(100, 10)],
    "mlp": [wl.fc(784, 256), wl.fc(256, 256), wl.fc(256, 10)],
}
# the box radius each network is used at: 2/255 on images, as in the repository's workloads
EPS = {"tiny": 0.1, "small": 0.05, "mlp": 0.01}


def listed():
    return [
        # the smallest call: a handful of launches, so latency is what counts
        dict(name="tiny_bound", op="bound", net="tiny", B=64, S=1, splits=6, alpha=False, lu=False,
             steps=0),
        # the first call of every search: one sub-domain, no splits, everything reported
        dict(name="base_root", op="bound", net="base", B=1, S=9, splits=0, alpha=False, lu=True,
             steps=0),
        # a batch of sub-domains with the heuristic slopes (Base of the configurations)
        dict(name="base_bound", op="bound", net="base", B=400, S=9, splits=10, alpha=False,
             lu=False, steps=0),
        # a batch with given slopes (Wide of the configurations)
        dict(name="wide_bound", op="bound", net="wide", B=1024, S=9, splits=16, alpha=True,
             lu=False, steps=0),
        # the net with four convolutions (Deep of the configurations)
        dict(name="deep_bound", op="bound", net="deep", B=1024, S=9, splits=16, alpha=False,
             lu=False, steps=0),
        # children of a search step, bounded from their parents
        dict(name="base_child", op="child", net="base", B=129, S=1, splits=10, alpha=True,
             lu=True, steps=0),
        # a user's own optimiser: bounds and gradient per call
        dict(name="base_grad", op="grad", net="base", B=400, S=9, splits=10, alpha=True, lu=False,
             steps=0),
        # another image size, ragged against every tile
        dict(name="gray_bound", op="bound", net="gray", B=255, S=9, splits=12, alpha=False,
             lu=True, steps=0),
        # a fully connected net, bounds and gradient
        dict(name="mlp_grad", op="grad", net="mlp", B=200, S=9, splits=12, alpha=True, lu=False,
             steps=0),
        # one iteration of a search on Deep: its children optimised for the paper's 10 steps
        dict(name="deep_opt", op="optimize", net="deep", B=64, S=9, splits=16, alpha=False,
             lu=False, steps=10),
        # the headline workload (the benchmark's default)
        dict(name="wide_opt", op="optimize", net="wide", B=2048, S=9, splits=16, alpha=False,
             lu=False, steps=20),
        # a whole search, with the heuristic slopes
        dict(name="base_bab", op="bab", net="base", B=64, S=1, splits=0, alpha=False, lu=False,
             steps=10),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# the largest drawn batch (and step count) of each operation, so that no drawn case costs more
# than the largest listed one
MOST = {
    "bound": dict(tiny=4096, base=1024, wide=1024, deep=1024, small=2048, gray=1024, mlp=1024),
    "child": dict(base=1024, wide=512, deep=512, gray=512),
    "ul": dict(base=1024, wide=512, deep=512, gray=512),
    "grad": dict(tiny=1024, base=512, wide=512, deep=256, small=512, gray=256, mlp=512),
    "optimize": dict(base=256, wide=256, deep=64, gray=64),
    "bab": dict(base=64),
}


def draw(rng):
    op = rng.choice(["bound", "bound", "bound", "child", "ul", "grad", "grad", "optimize",
                     "optimize", "bab"])
    net = rng.choice(sorted(MOST[op]))
    B = _log_int(rng, 8 if op == "bab" else 1, MOST[op][net])
    n_out = NETS[net][-1]["out_c"]
    S = 1 if op == "bab" else rng.choice([1, n_out - 1, rng.randint(1, n_out - 1)])
    steps = rng.randint(2, 10) if op in ("optimize", "bab") else 0
    alpha = op == "grad" or (op in ("bound", "child", "ul") and rng.random() < 0.5)
    return dict(op=op, net=net, B=B, S=S, splits=0 if op == "bab" else rng.randint(0, 16),
                alpha=alpha, lu=op == "bound" and rng.random() < 0.5, steps=steps)


# ---- inputs --------------------------------------------------------------------------------

def _forward64(layers, X):
    """Pre-activations of every ReLU layer for a batch of inputs, in 64 bits on the host."""
    a, pre = torch.as_tensor(X, dtype=torch.float64), []
    for t in layers[:-1]:
        W, b = torch.as_tensor(t["W"]).double(), torch.as_tensor(t["b"]).double()
        if t["kind"] == wl.CONV:
            a = F.conv2d(a.reshape(len(X), t["in_c"], t["in_h"], t["in_w"]), W, b,
                         stride=t["stride"], padding=t["pad"])
        else:
            a = a.reshape(len(X), -1) @ W.T + b
        pre.append(a.reshape(len(X), -1))
        a = a.clamp(min=0)
    return torch.cat(pre, 1).numpy()


def _inputs(case, seed):
    """Everything on the host: layers, x0, eps, C, split, alpha."""
    arch = NETS[case["net"]]
    layers = wl.make_layers(arch, seed)
    rng = np.random.default_rng([seed, 0xCA5E])
    n0, B = wl.n_in(arch[0]), 1 if case["op"] == "bab" else case["B"]
    x0 = rng.uniform(0.0, 1.0, size=n0).astype(np.float32)
    eps = float(np.float32(EPS.get(case["net"], wl.EPS_CIFAR)))
    C = wl.margin_spec(arch[-1]["out_c"], int(rng.integers(0, arch[-1]["out_c"])))
    C = np.ascontiguousarray(C[:case["S"]])
    n_relu = wl.num_relu(layers)
    split = None
    if case["splits"]:
        # a search splits neurons that are not stable: those seen with both signs in the box
        X = x0 + eps * rng.choice([-1.0, 1.0], size=(32, n0))
        pre = _forward64(layers, X)
        cand = np.flatnonzero((pre.min(0) < 0) & (pre.max(0) > 0))
        split = wl.make_splits(B, n_relu, case["splits"], seed, cand)
    alpha = None
    if case["alpha"]:
        # slopes as an optimiser leaves them: in [0, 1], a good part of them at the ends
        alpha = np.clip(rng.normal(0.5, 0.4, size=(B, n_relu)), 0, 1).astype(np.float32)
    return layers, x0, eps, C, split, alpha


def _parent_split(split, seed):
    """The parents' splits: each child's with one split of it undone."""
    rng = np.random.default_rng([seed, 0xFA])
    out = split.copy()
    for row in out:
        idx = np.flatnonzero(row)
        if idx.size:
            row[rng.choice(idx)] = 0
    return out


def prepare(case, seed):
    layers, x0, eps, C, split, alpha = _inputs(case, seed)
    dev = lambda a: None if a is None else torch.as_tensor(a).to("cuda")  # noqa: E731
    net = lirpa.Network(layers)
    st = dict(case=case, net=net, x0=dev(x0), eps=eps, C=dev(C), split=dev(split),
              alpha=dev(alpha))
    if case["op"] == "child":
        ps = None if split is None else dev(_parent_split(split, seed))
        _, st["lp"], st["up"] = net.bound(st["x0"], eps, st["C"], split=ps, alpha=st["alpha"],
                                          B=case["B"], want_lu=True)
    if case["op"] == "bab":
        st["c"] = dev(np.ascontiguousarray(C[0]))
    if case["op"] == "optimize":
        st["slopes"] = torch.empty((case["B"], net.n_relu), device="cuda")
        st["m"], st["v"] = torch.empty_like(st["slopes"]), torch.empty_like(st["slopes"])
    return st


def run(st):
    c, net = st["case"], st["net"]
    box = (st["x0"], st["eps"], st["C"])
    if c["op"] == "bound":
        return net.bound(*box, split=st["split"], alpha=st["alpha"], B=c["B"], want_lu=c["lu"],
                         want_codes=c["lu"])
    if c["op"] == "child":
        return net.bound_child(*box, st["split"], st["alpha"], st["lp"], st["up"])
    if c["op"] == "ul":
        return net.bound_ul(*box, split=st["split"], alpha=st["alpha"], B=c["B"])
    if c["op"] == "grad":
        return net.bound_grad(*box, st["split"], st["alpha"])
    if c["op"] == "optimize":
        lb = net.optimize(*box, st["split"], st["slopes"], st["m"], st["v"], steps=c["steps"],
                          fresh=True)
        return lb, st["slopes"], st["m"], st["v"]
    r = net.bab(st["x0"], st["eps"], st["c"], batch=c["B"], max_iters=c["steps"])
    return {k: r[k] for k in ("f_lo", "f_hi", "status", "iterations", "domains_bounded",
                              "domains_left")}


# ---- what a pass cannot do without -------------------------------------------------------------

def _pass_flops(arch, k, rows):
    """Flops of `rows` rows of h^(k) taken back to the input: every layer below k once, over the
    entries that the row can reach (a row of a convolution's output has a window)."""
    flops, side = 0.0, 0 if arch[k - 1]["kind"] == wl.FC else 1
    for m in range(k, 0, -1):
        t = arch[m - 1]
        if t["kind"] == wl.FC:
            flops += 0 if m == k else 2.0 * rows * t["out_c"] * t["in_c"]
            side = 0  # every entry from here on
            continue
        s = t["out_h"] if side == 0 else min(side, t["out_h"])
        if m < k:
            flops += 2.0 * rows * s * s * t["out_c"] * t["in_c"] * t["k"] ** 2
        side = 0 if side == 0 else (s - 1) * t["stride"] + t["k"]
    return flops


def work(case):
    arch, op, B, S = NETS[case["net"]], case["op"], case["B"], case["S"]
    n = wl.num_relu(arch)
    mid = sum(_pass_flops(arch, k, 2.0 * wl.n_out(arch[k - 1])) for k in range(2, len(arch)))
    fin = _pass_flops(arch, len(arch), 1.0)
    fin += 2.0 * arch[-1]["out_c"] * arch[-1]["in_c"]
    weights = 4.0 * sum(int(np.prod(wl.weight_shape(t))) for t in arch)
    rows = dict(ul=2 * S).get(op, S)
    flops = B * (mid + rows * fin)
    state = B * n * (1.0 * bool(case["splits"]) + 4.0 * case["alpha"])
    out = 4.0 * B * rows
    if op == "child":
        state, out = state + 8.0 * B * n, out + 9.0 * B * n
    if case["lu"] and op == "bound":
        out += 9.0 * B * n
    if op == "grad":
        flops, out = 2 * flops, out + 4.0 * B * n
    if op == "optimize":
        flops, out = (2 * case["steps"] + 1) * flops, out + 12.0 * B * n
    if op == "bab":  # the root, then two children of each sub-domain picked, both sides
        count = 1.0 + 2 * sum(min(B, 1 << i) for i in range(case["steps"]))
        flops, state, out = count * (mid + 2 * fin), 0.0, 24.0
    return {"bytes": weights + state + out, "flops": flops}


def tolerance(case):
    # about four times what the path shows against exact() over the ranges of draw().  A row whose
    # A_x entry is within rounding of zero has two valid gradients, and Adam's first steps take
    # the sign of gradients that are within rounding of zero: a few slopes then move the other way.
    if case["op"] == "bab":
        return {"rel": 1e-4, "max": 1e-3}
    if case["op"] == "optimize":
        return {"rel": 3e-3, "max": 0.9}
    if case["op"] == "grad":
        return {"rel": 1e-4, "max": 0.05}
    return {"rel": 3e-5, "max": 1e-4, "differ": 1e-4}


# ---- the same in 64 bits, in plain torch -------------------------------------------------------

def _dense(t):
    """A layer's matrix [n_out, n_in] and bias [n_out] in 64 bits on the GPU."""
    W, b = torch.as_tensor(t["W"]).double(), torch.as_tensor(t["b"]).double()
    if t["kind"] == wl.FC:
        return W.to("cuda"), b.to("cuda")
    ci, hi, wi, co, ho, wo = (t[x] for x in ("in_c", "in_h", "in_w", "out_c", "out_h", "out_w"))
    M = torch.zeros((co, ho, wo, ci, hi, wi), dtype=torch.float64)
    for y in range(ho):
        for x in range(wo):
            for dy in range(t["k"]):
                for dx in range(t["k"]):
                    iy, ix = y * t["stride"] + dy - t["pad"], x * t["stride"] + dx - t["pad"]
                    if 0 <= iy < hi and 0 <= ix < wi:
                        M[:, y, x, :, iy, ix] = W[:, :, dy, dx]
    M = M.reshape(co * ho * wo, -1).to("cuda")
    return M, b.to("cuda").repeat_interleave(ho * wo)


def _relax(l, u, split, alpha):
    """(lower slope, upper slope, upper intercept, code) per neuron."""
    code = torch.full(l.shape, 5, dtype=torch.int8, device=l.device)
    code[l >= 0] = 4
    code[u <= 0] = 3
    if split is not None:
        code[split < 0] = 2
        code[split > 0] = 1
    one, zero = torch.ones_like(l), torch.zeros_like(l)
    uns, act = code == 5, (code == 1) | (code == 4)
    gap = torch.where(uns, u - l, one)
    up = torch.where(uns, u / gap, torch.where(act, one, zero))
    cut = torch.where(uns, -l * u / gap, zero)
    if alpha is None:
        return up, up, cut, code
    return torch.where(uns, alpha, up), up, cut, code


def _low(mats, rel, rows, const, k, x0, eps):
    """Lower bounds of the rows [b, r, n_k] of h^(k) (const their constants [r])."""
    A, beta = rows, const
    for m in range(k, 0, -1):
        W, b = mats[m - 1]
        beta = beta + A @ b
        A = A @ W
        if m > 1:
            lo, up, cut, _ = rel[m - 2]
            neg = A < 0
            beta = beta + torch.where(neg, A, torch.zeros_like(A)).matmul(cut.unsqueeze(-1)).squeeze(-1)
            A = A * torch.where(neg, up.unsqueeze(1), lo.unsqueeze(1))
    return A @ x0 + beta - eps * A.abs().sum(-1)


def _bounds(mats, x0, eps, C, split, alpha, lp=None, up=None):
    """(lb, l, u, codes) of a few sub-domains."""
    sizes = [M.shape[0] for M, _ in mats]
    nb = next(t.shape[0] for t in (split, alpha, lp, torch.zeros(1, 1)) if t is not None)
    rel, ls, us, o = [], [], [], 0
    for k in range(1, len(mats)):
        n, (W, b) = sizes[k - 1], mats[k - 1]
        if k == 1:
            mid, rad = W @ x0 + b, eps * W.abs().sum(1)
            l, u = (mid - rad).expand(nb, n), (mid + rad).expand(nb, n)
        else:
            # the first step from the unit rows is the matrix itself
            l = _open(mats, rel, W.expand(nb, *W.shape), b, k, x0, eps)
            u = -_open(mats, rel, (-W).expand(nb, *W.shape), -b, k, x0, eps)
        if lp is not None:
            l, u = torch.maximum(l, lp[:, o:o + n]), torch.minimum(u, up[:, o:o + n])
        rel.append(_relax(l, u, None if split is None else split[:, o:o + n],
                          None if alpha is None else alpha[:, o:o + n]))
        ls, us, o = ls + [l], us + [u], o + n
    W, b = mats[-1]
    lb = _open(mats, rel, (C @ W).expand(nb, C.shape[0], W.shape[1]), C @ b, len(mats), x0, eps)
    return lb, torch.cat(ls, 1), torch.cat(us, 1), torch.cat([r[3] for r in rel], 1)


def _open(mats, rel, A, beta, k, x0, eps):
    """Lower bounds of rows already taken through T_k: A over g^(k-1), constants beta."""
    if k > 1:
        lo, up, cut, _ = rel[k - 2]
        neg = A < 0
        beta = beta + (torch.where(neg, A, torch.zeros_like(A)) * cut.unsqueeze(1)).sum(-1)
        A = torch.where(neg, A * up.unsqueeze(1), A * lo.unsqueeze(1))
        return _low(mats, rel, A, beta, k - 1, x0, eps)
    return A @ x0 + beta - eps * A.abs().sum(-1)


def exact(case, seed):
    op, B, arch = case["op"], case["B"], NETS[case["net"]]
    per = sum(_dense_flops(arch, k) for k in range(2, len(arch)))
    count = {"optimize": 4.0 * case["steps"] + 1, "grad": 4.0, "child": 2.0}.get(op, 1.0)
    if op == "bab" or B * per * count > 5e14:
        return None
    layers, x0, eps, C, split, alpha = _inputs(case, seed)
    mats = [_dense(t) for t in layers]
    d = lambda a: None if a is None else torch.as_tensor(a).to("cuda")  # noqa: E731
    x0, C, split = d(x0).double(), d(C).double(), d(split)
    alpha = None if alpha is None else d(alpha).double()
    pieces = []
    few = 1 if op in ("grad", "optimize") else max(1, min(B, int(1.0e8 / _widest(arch))))
    par = None
    if op == "child":
        par = None if split is None else d(_parent_split(split.cpu().numpy(), seed))
    cut = lambda t, i, j: None if t is None else t[i:j]  # noqa: E731
    for i in range(0, B, few):
        j = min(B, i + few)
        s, a = cut(split, i, j), cut(alpha, i, j)
        if s is None and a is None and j - i > 1:  # the batch is what the masks say
            s = torch.zeros((j - i, wl.num_relu(layers)), dtype=torch.int8, device="cuda")
        if op == "grad":
            pieces.append(_grad64(mats, x0, eps, C, s, a))
        elif op == "optimize":
            pieces.append(_adam64(mats, x0, eps, C, s, case["steps"]))
        elif op == "ul":
            lb = _bounds(mats, x0, eps, torch.cat([C, -C]), s, a)[0]
            pieces.append((lb[:, :C.shape[0]], -lb[:, C.shape[0]:]))
        elif op == "child":
            _, lp, up, _ = _bounds(mats, x0, eps, C, cut(par, i, j), a)
            if lp.shape[0] < j - i:
                lp, up = lp.expand(j - i, -1), up.expand(j - i, -1)
            pieces.append(_bounds(mats, x0, eps, C, s, a, lp, up))
        else:
            pieces.append(_bounds(mats, x0, eps, C, s, a))
    out = tuple(torch.cat(p) for p in zip(*pieces))
    if op == "child":
        return out[:3] + (None,)
    if op == "bound":
        return out[:3] + (None,) if case["lu"] else out[0]
    return out


def _dense_flops(arch, k):
    n, f = wl.n_out(arch[k - 1]), 0.0
    for t in arch[:k - 1]:
        f += 4.0 * n * wl.n_out(t) * wl.n_in(t)
    return f


def _widest(arch):
    n = [wl.n_in(arch[0])] + [wl.n_out(t) for t in arch]
    return max(n[k] * max(n[:k]) for k in range(1, len(arch)))


def _grad64(mats, x0, eps, C, split, alpha):
    a = alpha.clone().requires_grad_(True)
    lb = _bounds(mats, x0, eps, C, split, a)[0]
    g, = torch.autograd.grad(lb.sum(), a)
    return lb.detach(), g


def _adam64(mats, x0, eps, C, split, steps, lr=float(np.float32(0.1)),
            b1=float(np.float32(0.9)), b2=float(np.float32(0.999)), tiny=float(np.float32(1e-8))):
    _, l, u, _ = _bounds(mats, x0, eps, C, split, None)
    gap = torch.where((l < 0) & (u > 0), u - l, torch.ones_like(l))
    a = torch.where(u <= 0, torch.zeros_like(l), torch.where(l >= 0, torch.ones_like(l), u / gap))
    m, v, best = torch.zeros_like(a), torch.zeros_like(a), None
    for t in range(steps + 1):
        if t == steps:
            lb = _bounds(mats, x0, eps, C, split, a)[0]
        else:
            lb, g = _grad64(mats, x0, eps, C, split, a)
        best = lb if best is None else torch.maximum(best, lb)
        if t < steps:
            m, v = b1 * m + (1 - b1) * g, b2 * v + (1 - b2) * g * g
            up = (m / (1 - b1 ** (t + 1))) / ((v / (1 - b2 ** (t + 1))).sqrt() + tiny)
            a = (a + lr * up).clamp(0, 1)
    return best, a, m, v
