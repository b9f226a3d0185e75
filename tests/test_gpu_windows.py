"""Receptive-field passes of convolution chains of any geometry, against the fp64 oracle: bounds,
intermediate bounds and gradients of nets whose windows have every edge the kernel handles
(strides 1 to 4, kernels 1 to 7 larger than the map, taps that do not divide by the stride,
channel counts off the 4, 8 and 16 of its tiles, up to four convolutions), and of one whose
windows do not fit on chip (the dense stages).  The fc nets do the same for the fully connected
stages: widths off every tile, and a layer too narrow for the split kernels.  Their few rows here
run on one tile of rows a block, whatever their LDS panels would hold; test_fc_row_tiles runs the
first two on two and four tiles.  The net nets run the one-launch bound of small fully connected
nets.  The slab nets end their intermediate pass 4, whose rows come from a fully connected layer of
even width off the 16 rows of a block, in the two convolutions' kernel.

Tolerance: a bound is at most four chained fp32 sums of up to 2,000 terms, each within 8e-7 of its
2-norm (the fp32 matrix instruction's measured error at that length); with a factor 3 for
cancellation 1e-5 (1 + |ref|).  Gradients: the same, normwise, with the kink rule of the gradient
tests."""
import re

import numpy as np
import pytest
import torch

from oracle import bab, ref
from paper_2011_13824_amd import lirpa
from paper_2011_13824_amd import workloads as wl
from tests import helpers as H
from tests.test_gpu_grad import check_grad, dev, heuristic_alpha, one_sided

pytestmark = pytest.mark.gpu

NETS = {
    "stride2-k3": [wl.conv(2, 9, 5, 3, 2, 1), wl.conv(5, 5, 9, 3, 1, 1), wl.fc(225, 6),
                   wl.fc(6, 3)],
    "k7-stride4": [wl.conv(1, 11, 17, 7, 4, 3), wl.conv(17, 3, 6, 2, 1, 0), wl.fc(24, 5),
                   wl.fc(5, 3)],
    "four-convs": [wl.conv(5, 7, 3, 3, 1, 1), wl.conv(3, 7, 10, 3, 2, 0), wl.conv(10, 3, 8, 2, 1, 1),
                   wl.conv(8, 4, 20, 4, 2, 1), wl.fc(80, 3)],
    "k-over-map": [wl.conv(3, 6, 8, 5, 3, 2), wl.conv(8, 2, 33, 1, 1, 0), wl.fc(132, 3)],
    "wide-channels": [wl.conv(3, 6, 40, 3, 1, 1), wl.conv(40, 6, 12, 3, 2, 1), wl.fc(108, 3)],
    "conv-last": [wl.conv(1, 6, 4, 4, 2, 1), wl.conv(4, 3, 16, 3, 1, 1), wl.conv(16, 3, 1, 3, 1, 0)],
    "fc-four-tiles": [wl.fc(70, 250), wl.fc(250, 67), wl.fc(67, 3)],
    "fc-two-tiles": [wl.fc(50, 330), wl.fc(330, 54), wl.fc(54, 3)],
    "fc-one-tile": [wl.fc(20, 850), wl.fc(850, 20), wl.fc(20, 31), wl.fc(31, 3)],
    "net-edges": [wl.fc(1, 64), wl.fc(64, 1), wl.fc(1, 33), wl.fc(33, 3)],
    "net-eight-layers": [wl.fc(7, 5), wl.fc(5, 6), wl.fc(6, 7), wl.fc(7, 8), wl.fc(8, 9),
                         wl.fc(9, 10), wl.fc(10, 11), wl.fc(11, 3)],
    "net-two-layers": [wl.fc(20, 16), wl.fc(16, 3)],
    "off-chip": [wl.conv(1, 4, 64, 7, 1, 3), wl.conv(64, 4, 2, 7, 1, 3), wl.fc(32, 3)],
    "slab-8-16": [wl.conv(3, 32, 8, 4, 2, 1), wl.conv(8, 16, 16, 4, 2, 1), wl.fc(1024, 30),
                  wl.fc(30, 34), wl.fc(34, 3)],
    "slab-16-32": [wl.conv(3, 32, 16, 4, 2, 1), wl.conv(16, 16, 32, 4, 2, 1), wl.fc(2048, 30),
                   wl.fc(30, 18), wl.fc(18, 3)],
    "gray": [wl.conv(1, 28, 16, 4, 2, 1), wl.conv(16, 14, 32, 4, 2, 1), wl.fc(1568, 100),
             wl.fc(100, 3)],
}


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    lirpa.load()


def close(name, got, want, tol=1e-5):
    excess = np.abs(got - want) - tol * (1 + np.abs(want))
    print(f"{name}: max |gpu - oracle| = {np.abs(got - want).max():.3g}", flush=True)
    assert np.all(excess <= 0), f"{name}: off by {excess.max():.3g} beyond tolerance"


@pytest.mark.parametrize("name", sorted(NETS))
@pytest.mark.parametrize("B", [1, 7])
def test_windows(name, B):
    arch = NETS[name]
    layers = wl.random_net(arch, 5 + len(name))
    rng = np.random.default_rng(len(name))
    x0 = rng.uniform(0, 1, wl.n_in(arch[0])).astype(np.float32)
    eps = 0.1
    C = wl.margin_spec(3, 1) if wl.n_out(arch[-1]) == 3 else np.ones((1, 1), np.float32)
    rnet = ref.RefNet(layers)
    split = wl.make_splits(B, rnet.n_relu, 6, B, ref.root_unstable(rnet, x0, eps, C))
    alpha = rng.uniform(0.05, 0.95, (B, rnet.n_relu)).astype(np.float32)
    net = lirpa.Network(layers)
    for a in (None, alpha):
        lb, l, u = net.bound(dev(x0), eps, dev(C), dev(split), dev(a), want_lu=True)
        lr, llr, ulr, _ = ref.bound(rnet, x0, eps, C, split, a)
        close(f"{name} lb", lb.cpu().double().numpy(), lr)
        close(f"{name} l", l.cpu().double().numpy(), llr)
        close(f"{name} u", u.cpu().double().numpy(), ulr)
    lb, g = net.bound_grad(dev(x0), eps, dev(C), dev(split), dev(alpha))
    lr, gr = ref.bound_grad(rnet, x0, eps, C, split, alpha)
    close(f"{name} grad lb", lb.cpu().double().numpy(), lr)
    check_grad(f"{name} grad", g.cpu().double().numpy(), gr, split,
               lambda b, j: one_sided(rnet, x0, eps, C, split, alpha, b, j))


# Fully connected stages take two tiles of 16 rows a block from 16,384 rows on and four from 32,768:
# the first pass's rows here, two per neuron with slopes (134 and 108), 54 without
@pytest.mark.parametrize("name,B", [("fc-four-tiles", 125), ("fc-four-tiles", 251),
                                    ("fc-two-tiles", 309), ("fc-two-tiles", 617)])
def test_fc_row_tiles(name, B):
    arch = NETS[name]
    layers = wl.random_net(arch, B)
    rng = np.random.default_rng(B)
    x0 = rng.uniform(0, 1, wl.n_in(arch[0])).astype(np.float32)
    eps, C, some = 0.1, wl.margin_spec(3, 1), [0, 1, B // 2, B - 2, B - 1]
    rnet = ref.RefNet(layers)
    split = wl.make_splits(B, rnet.n_relu, 6, B)
    alpha = rng.uniform(0.05, 0.95, (B, rnet.n_relu)).astype(np.float32)
    net = lirpa.Network(layers)
    for a in (None, alpha):
        got = net.bound(dev(x0), eps, dev(C), dev(split), dev(a), want_lu=True)
        want = ref.bound(rnet, x0, eps, C, split[some], None if a is None else a[some])
        for what, g, w in zip(("lb", "l", "u"), got, want):
            close(f"{name} {B} {what}", g.cpu().double().numpy()[some], w)
    lb, g = net.bound_grad(dev(x0), eps, dev(C), dev(split), dev(alpha))
    lr, gr = ref.bound_grad(rnet, x0, eps, C, split[some], alpha[some])
    close(f"{name} {B} grad lb", lb.cpu().double().numpy()[some], lr)
    check_grad(f"{name} {B} grad", g.cpu().double().numpy()[some], gr, split[some],
               lambda b, j: one_sided(rnet, x0, eps, C, split[some], alpha[some], b, j))


SOME = ["four-convs", "k7-stride4", "conv-last", "off-chip", "fc-two-tiles"]


@pytest.mark.parametrize("slopes", [False, True])
@pytest.mark.parametrize("name", SOME)
def test_other_entry_points(name, slopes):
    # bounds from a parent's and bounds of both sides
    arch, B = NETS[name], 5
    layers = wl.random_net(arch, 3)
    rng = np.random.default_rng(3)
    x0 = rng.uniform(0, 1, wl.n_in(arch[0])).astype(np.float32)
    eps, C = 0.1, np.eye(wl.n_out(arch[-1]), dtype=np.float32)
    rnet = ref.RefNet(layers)
    split = wl.make_splits(B, rnet.n_relu, 6, B)
    alpha = rng.uniform(0.05, 0.95, (B, rnet.n_relu)).astype(np.float32) if slopes else None
    net = lirpa.Network(layers)
    # (the parent: the same sub-domain without its splits)
    _, lp, up, _ = ref.bound(rnet, x0, eps, C, np.zeros_like(split), alpha)
    lp, up = lp.astype(np.float32), up.astype(np.float32)
    got = net.bound_child(dev(x0), eps, dev(C), dev(split), dev(alpha), dev(lp), dev(up))
    want = ref.bound_child(rnet, x0, eps, C, split, alpha, lp, up)
    for what, g, w in zip(("lb", "l", "u"), got, want):
        close(f"{name} child {what}", g.cpu().double().numpy(), w)
    lo, hi = net.bound_ul(dev(x0), eps, dev(C), dev(split), dev(alpha))
    close(f"{name} ul lb", lo.cpu().double().numpy(), ref.bound(rnet, x0, eps, C, split, alpha)[0])
    close(f"{name} ul ub", hi.cpu().double().numpy(),
          -ref.bound(rnet, x0, eps, -C, split, alpha)[0])


@pytest.mark.parametrize("name", SOME)
def test_optimize_step(name):
    # a fresh start: the heuristic bound, the gradient there (ten times the first moment), and the
    # bound at the slopes after the step
    arch, B = NETS[name], 3
    layers = wl.random_net(arch, 4)
    rng = np.random.default_rng(4)
    x0 = rng.uniform(0, 1, wl.n_in(arch[0])).astype(np.float32)
    eps, C = 0.1, np.eye(wl.n_out(arch[-1]), dtype=np.float32)
    rnet = ref.RefNet(layers)
    split = wl.make_splits(B, rnet.n_relu, 6, B)
    net = lirpa.Network(layers)
    a = torch.empty((B, rnet.n_relu), device="cuda")
    m, v = torch.empty_like(a), torch.empty_like(a)
    best, trace = net.optimize(dev(x0), eps, dev(C), dev(split), a, m, v, steps=1, fresh=True,
                               trace=True)
    lr, l, u, _ = ref.bound(rnet, x0, eps, C, split)
    a0 = heuristic_alpha(l, u).astype(np.float32)
    gr = ref.bound_grad(rnet, x0, eps, C, split, a0)[1]
    close(f"{name} start", trace[0].cpu().double().numpy(), lr)
    check_grad(f"{name} gradient", 10 * m.cpu().double().numpy(), gr, split,
               lambda b, j: one_sided(rnet, x0, eps, C, split, a0, b, j))
    end = ref.bound(rnet, x0, eps, C, split, a.cpu().numpy())[0]
    close(f"{name} end", trace[1].cpu().double().numpy(), end)
    assert torch.equal(best, trace.max(0).values)


@pytest.mark.parametrize("kw", [dict(), dict(root_steps=2, steps=2)])
def test_search_without_room_for_fragments(kw):
    # the search's least workspace, where its calls run without their packed weights or in chunks:
    # its course on the heuristic slopes is the oracle's, with optimised ones the full workspace's
    layers = wl.random_net(H.small_conv_arch(), 21)
    x0 = np.random.default_rng(21).uniform(0, 1, wl.n_in(layers[0])).astype(np.float32)
    c = wl.margin_spec(3, 2)[1]
    net = lirpa.Network(layers)
    p = lirpa.lirpa_bab_params(8, 100, 3, kw.get("root_steps", 0), kw.get("steps", 0), 0.1, 0.9,
                               0.999, 1e-8)
    full = lirpa.lirpa_bab_workspace_bytes(net.handle, p)

    def search(room):
        r = lirpa.lirpa_bab(net.handle, dev(x0), 0.05, dev(c), p,
                            torch.empty(room, dtype=torch.uint8, device="cuda"), room)
        return {k: getattr(r, k) for k, _ in r._fields_}

    with pytest.raises(lirpa.LirpaError) as ei:
        search(256)
    need = int(re.search(r"needs (\d+)", str(ei.value)).group(1))
    assert need <= full
    got, want = search(need), search(full)
    if not kw:
        want = bab.bab(ref.RefNet(layers), x0, 0.05, c, 8, 100, 3)
    print(f"{need} of {full} bytes: {got}", flush=True)
    for k in ("status", "iterations", "domains_bounded", "domains_left"):
        assert got[k] == want[k], k
    for k in ("f_lo", "f_hi"):
        assert abs(got[k] - want[k]) <= 1e-4 * (1 + abs(want[k])), k


@pytest.mark.parametrize("convs", [8, 10, 16])
def test_many_convolutions(convs):
    # every convolution has weight fragments of its own in each direction, and a set-up launch
    # carries 16 of them: 8 layers fill one launch in a gradient call, 10 one and a part of the
    # next, 16 one in a bound and two in a gradient.  (Up to 17 chained sums where the nets above
    # have four: four times their tolerance.)
    arch = [wl.conv(1, 6, 4, 3, 1, 1)] + [wl.conv(4, 6, 4, 3, 1, 1)] * (convs - 1) + [wl.fc(144, 3)]
    layers = wl.random_net(arch, convs)
    x0 = np.random.default_rng(convs).uniform(0, 1, 36).astype(np.float32)
    eps, C = 0.16 / convs, wl.margin_spec(3, 0)
    rnet = ref.RefNet(layers)
    alpha = np.random.default_rng(1).uniform(0.05, 0.95, (2, rnet.n_relu)).astype(np.float32)
    net = lirpa.Network(layers)
    for a in (None, alpha):
        lb = net.bound(dev(x0), eps, dev(C), None, dev(a), B=2)
        lr = ref.bound(rnet, x0, eps, C, None, a)[0]
        close(f"{convs} lb", lb.cpu().double().numpy(), np.broadcast_to(lr, (2, 2)), 4e-5)
    lb, g = net.bound_grad(dev(x0), eps, dev(C), None, dev(alpha))
    lr, gr = ref.bound_grad(rnet, x0, eps, C, None, alpha)
    close(f"{convs} grad lb", lb.cpu().double().numpy(), lr, 4e-5)
    check_grad(f"{convs} grad", g.cpu().double().numpy(), gr, None,
               lambda b, j: one_sided(rnet, x0, eps, C, None, alpha, b, j))


# net, the layer whose weights are scaled, their largest value: bounds of that layer beyond fp32's
# range, and in the fifth case all of them and every partial sum inside it (sum |a| b_up is beyond).
# "gray" with layer 0 scaled: layer 1's bounds are inside the range and their intercepts beyond it;
# the bounds after the next layer's
OVERFLOWS = [("fc-four-tiles", 1, 3e37), ("base", 2, 3e37), ("deep", 3, 3e37), ("deep", 4, 3e37),
             ("deep", 4, 1e36), ("gray", 0, 1e36)]


@pytest.mark.parametrize("name,layer,scale", OVERFLOWS)
def test_overflowing_bounds_are_infinite(name, layer, scale):
    # a pass with one row per neuron gives -inf and +inf where the bounds leave fp32's range, as
    # one with two rows does, and never a NaN.  (Partial sums may leave it where the bound itself
    # does not: then the bound is infinite on its sound side.)
    layers = wl.random_net(NETS.get(name) or wl.ARCHS[name], 4)
    W = layers[layer]["W"].astype(np.float64)
    layers[layer]["W"] = (W * (scale / np.abs(W).max())).astype(np.float32)
    x0 = np.random.default_rng(1).uniform(0, 1, wl.n_in(layers[0])).astype(np.float32)
    C = np.eye(wl.n_out(layers[-1]), dtype=np.float32)
    net = lirpa.Network(layers)
    _, l, u = net.bound(dev(x0), 0.05, dev(C), None, None, B=1, want_lu=True)
    want = ref.bound(ref.RefNet(layers), x0, 0.05, C, None, None)
    layer = max(layer, 1)
    o = sum(wl.relu_sizes(layers)[:layer])
    top = float(np.finfo(np.float32).max)
    for what, side, got, ref_ in (("l", -1, l, want[1]), ("u", 1, u, want[2])):
        g = got.cpu().double().numpy()[0, o:o + wl.n_out(layers[layer])]
        r = ref_[0, o:o + len(g)]
        beyond = side * r > 1.01 * top
        print(f"{name} {what}: {beyond.sum()} of {len(g)} beyond, {np.isinf(g).sum()} infinite, "
              f"{np.isnan(g).sum()} NaN", flush=True)
        assert not np.isnan(g).any(), f"{name} {what}"
        assert np.all(g[beyond] == side * np.inf), f"{name} {what}"
        assert np.all(side * (g - r) >= -1e-5 * np.abs(r)), f"{name} {what}: inside the bound"
        if name == "deep" and scale < 3e37:
            assert np.isfinite(g).all(), f"{name} {what}"


@pytest.mark.parametrize("few", [1, 15, 16, 31, 32])
@pytest.mark.parametrize("slopes", [False, True])
def test_pass2_by_ones_and_by_eights(few, slopes):
    # up to 31 sub-domains without slopes, 15 with them, the pass takes one window a block, beyond
    # that eight: the same sums, bit for bit
    w = wl.base()
    net = lirpa.Network(w.layers)
    rng = np.random.default_rng(0)
    split = dev(wl.make_splits(40, net.n_relu, 9, 1))
    a = dev(rng.uniform(0, 1, (40, net.n_relu)).astype(np.float32)) if slopes else None
    cut = lambda t: None if t is None else t[:few].contiguous()  # noqa: E731
    want = net.bound(dev(w.x0), w.eps, dev(w.C), split, a, want_lu=True)
    got = net.bound(dev(w.x0), w.eps, dev(w.C), cut(split), cut(a), want_lu=True)
    for x, y in zip(got, want):
        assert torch.equal(x, y[:few])


@pytest.mark.parametrize("layer,scale", [(1, 2e38), (2, 1e38)])
def test_overflow_in_one_launch(layer, scale):
    # the 4-32-32-2 net, bounded in one launch: the terms in x0 are part of layer 1's constants, so
    # coefficients over x beyond fp32's range give -inf, not inf - inf, and no bound on the wrong
    # side
    layers = wl.random_net(wl.ARCHS["tiny"], 4)
    W = layers[layer]["W"].astype(np.float64)
    layers[layer]["W"] = (W * (scale / np.abs(W).max())).astype(np.float32)
    x0 = np.random.default_rng(1).uniform(0, 1, 4).astype(np.float32)
    C = np.eye(2, dtype=np.float32)
    net = lirpa.Network(layers)
    lb, l, u = (t.cpu().double().numpy() for t in net.bound(dev(x0), 0.05, dev(C), None, None, B=1,
                                                            want_lu=True))
    lr, llr, ulr, _ = ref.bound(ref.RefNet(layers), x0, 0.05, C, None, None)
    print([int(np.isinf(a).sum()) for a in (lb, l, u)], "infinite", flush=True)
    if layer == 2:
        assert not np.isnan(lb).any()
        assert np.all(lb - lr <= 1e-5 * np.abs(lr))
    assert not np.any(l == np.inf) and not np.any(u == -np.inf)


# widths, sub-domains, spec rows on each side of every line of the one-launch rule: sub-domains of
# a two-layer net, of a net wider than 48 with and without slopes, few and many spec rows
NET_LINES = [([20, 16, 3], 256, 2), ([20, 16, 3], 257, 2), ([48, 49, 3], 512, 31),
             ([48, 49, 3], 513, 31), ([48, 49, 3], 513, 32), ([48, 49, 3], 1024, 2),
             ([48, 49, 3], 1025, 2), ([48, 48, 5, 3], 1025, 2), ([64, 7, 5, 3], 2, 32),
             ([64, 7, 5, 3], 2, 33), ([64, 9, 3], 127, 999), ([64, 9, 3], 128, 999),
             ([48, 9, 3], 127, 999), ([48, 9, 3], 128, 999), ([20, 16, 3], 2, 480),
             ([20, 16, 3], 2, 481), ([60, 60, 60, 3], 2, 64), ([60, 60, 60, 3], 2, 65),
             ([65, 7, 5, 3], 2, 1)]


@pytest.mark.parametrize("slopes", [False, True])
@pytest.mark.parametrize("widths,B,S", NET_LINES)
def test_one_launch_rule(widths, B, S, slopes):
    layers = wl.random_net([wl.fc(a, b) for a, b in zip(widths, widths[1:])], 2)
    rng = np.random.default_rng(B + S)
    x0 = rng.uniform(0, 1, widths[0]).astype(np.float32)
    C = rng.normal(size=(S, 3)).astype(np.float32)
    rnet = ref.RefNet(layers)
    split = wl.make_splits(B, rnet.n_relu, 3, B)
    alpha = rng.uniform(0, 1, (B, rnet.n_relu)).astype(np.float32) if slopes else None
    net = lirpa.Network(layers)
    lb, l, u = net.bound(dev(x0), 0.1, dev(C), dev(split), dev(alpha), want_lu=True)
    lr, llr, ulr, _ = ref.bound(rnet, x0, 0.1, C, split, alpha)
    close("lb", lb.cpu().double().numpy(), lr)
    close("l", l.cpu().double().numpy(), llr)
    close("u", u.cpu().double().numpy(), ulr)


@pytest.mark.parametrize("mode", ["bound", "grad"])
def test_workspace_without_room_for_fragments(mode):
    # a workspace that holds one sub-domain but not the split weight fragments beside it: the
    # dense stages run, with the same results
    layers = wl.random_net(NETS["off-chip"], 3)
    rng = np.random.default_rng(3)
    x0 = rng.uniform(0, 1, wl.n_in(layers[0])).astype(np.float32)
    C = wl.margin_spec(3, 0)
    rnet = ref.RefNet(layers)
    alpha = rng.uniform(0.05, 0.95, (2, rnet.n_relu)).astype(np.float32)
    net = lirpa.Network(layers)
    S = C.shape[0]
    full = lirpa.lirpa_workspace_bytes(net.handle, S, 1, 1 if mode == "grad" else 0)
    for room in (full, full - 256):  # the fragments, 147 KB of it at least, are the last to fit
        ws = torch.empty(room, dtype=torch.uint8, device="cuda")
        lb = torch.empty((2, S), device="cuda")
        if mode == "grad":
            g = torch.empty((2, rnet.n_relu), device="cuda")
            lirpa.lirpa_bound_grad(net.handle, dev(x0), 0.1, dev(C), S, 2, None, dev(alpha), 1, lb,
                                   g, ws, room)
            lr, gr = ref.bound_grad(rnet, x0, 0.1, C, None, alpha)
            check_grad("grad", g.cpu().double().numpy(), gr, None,
                       lambda b, j: one_sided(rnet, x0, 0.1, C, None, alpha, b, j))
        else:
            lirpa.lirpa_bound(net.handle, dev(x0), 0.1, dev(C), S, 2, None, dev(alpha), lb, None,
                              None, None, ws, room)
            lr = ref.bound(rnet, x0, 0.1, C, None, alpha)[0]
        close(f"{mode} lb", lb.cpu().double().numpy(), lr)


def test_least_workspace_is_the_one_named():
    # the refusal of a workspace that is too small names what one sub-domain needs at least
    layers = wl.random_net(NETS["off-chip"], 3)
    net = lirpa.Network(layers)
    x0, C = dev(np.full(16, 0.5, np.float32)), dev(wl.margin_spec(3, 0))
    lb = torch.empty((2, 2), device="cuda")

    def call(room):
        lirpa.lirpa_bound(net.handle, x0, 0.1, C, 2, 2, None, None, lb, None, None, None,
                          torch.empty(room, dtype=torch.uint8, device="cuda"), room)

    with pytest.raises(lirpa.LirpaError) as ei:
        call(256)
    assert ei.value.code == lirpa.LIRPA_ENOMEM
    need = int(re.search(r"need (\d+)", str(ei.value)).group(1))
    call(need)
    with pytest.raises(lirpa.LirpaError) as ei:
        call(need - 1)
    assert ei.value.code == lirpa.LIRPA_ENOMEM


@pytest.mark.parametrize("B,S", [(1, 1), (5, 7), (129, 2), (1024, 1), (1025, 3)])
def test_few_spec_rows(B, S):
    # fewer than 8 spec rows, padded to 8 up to 1,024 sub-domains and in stages beyond: the rows
    # of the call with all 9, whose blocks need no padding (the same sums up to their order: 1e-5)
    w = wl.base()
    rng = np.random.default_rng(B)
    net = lirpa.Network(w.layers)
    alpha = dev(rng.uniform(0, 1, (B, net.n_relu)).astype(np.float32))
    want = net.bound(dev(w.x0), w.eps, dev(w.C), None, alpha).cpu().double().numpy()
    lb = net.bound(dev(w.x0), w.eps, dev(w.C[:S]), None, alpha)
    close("lb", lb.cpu().double().numpy(), want[:, :S])
    lo, up = net.bound_ul(dev(w.x0), w.eps, dev(w.C[:S]), None, alpha)
    close("ul lb", lo.cpu().double().numpy(), want[:, :S])
    neg = net.bound(dev(w.x0), w.eps, dev(-w.C), None, alpha).cpu().double().numpy()
    close("ul ub", up.cpu().double().numpy(), -neg[:, :S])
