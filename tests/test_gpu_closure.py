"""GPU tests of the learned coarse closure (BF16 matrix-core forward and
backward kernels) against the CPU oracle, and of what the trained network
gains over the plain coarse run.

Parity is checked twice:
- against the oracle emulating the GPU's bfloat16 storage (inputs, weights,
  activations, back-propagated activations): the remaining differences are
  FP32 accumulation order and tanh rounding, which can flip single bfloat16
  roundings. Bars about 10x the measured differences (1e-5..4e-5): forward
  5e-4 relative l2, loss 1e-5 relative, each gradient block 3e-4;
- against the plain FP64 network (no rounding anywhere, its gradient pinned
  by finite differences): the GPU may be no farther from it than the
  bfloat16 storage itself puts the emulated network (computed in the test),
  plus 25% and an FP32-accumulation floor of 2e-4."""

import numpy as np
import pytest

import oracle as O
from oracle import closure as OC
from oracle.pipeline import build_ns
from workloads import density_current_config, closure_config
from workloads.fields import smooth_ns_state

pytestmark = pytest.mark.gpu


def say(*a):
    print(*a, flush=True)


@pytest.fixture(scope="module")
def setup():
    import torch
    from paper_1509_02615_amd import rbffd as R
    from paper_1509_02615_amd import pipeline as P
    ctx = R.Context(0)
    cfg = density_current_config("cartesian", 400.0)
    nd = cfg["nodes"]
    om, o_idx, o_W, o_Ww = build_ns(cfg)
    E = 3
    states = [smooth_ns_state(nd, seed=20 + k).astype(np.float32).astype(np.float64) for k in range(E)]
    closed = np.stack([O.ghost_closure(om, s).astype(np.float32).astype(np.float64) for s in states], axis=1)
    gm = P.ns_model(ctx, cfg, torch.from_numpy(o_idx).int().cuda(), torch.from_numpy(o_W).cuda(),
                    torch.from_numpy(o_Ww).cuda(), field_dtype=R.F32, weight_dtype=R.F32, ensemble=E)
    return dict(R=R, P=P, ctx=ctx, cfg=cfg, nd=nd, o_idx=o_idx, gm=gm, closed=closed, E=E)


def _closure(st, params, in_scale, out_scale, act=OC.TANH):
    import torch
    R = st["R"]
    nodef = st["nd"].xy[:st["nd"].n_active, 1] / st["nd"].height
    return R.Closure(st["ctx"], st["gm"], torch.from_numpy(params.astype(np.float32)).cuda(),
                     torch.from_numpy(nodef).cuda(), in_scale, out_scale, activation=act), nodef


IN_SCALE = [10.0, 10.0, 5.0, 1e-3]
OUT_SCALE = [0.05, 0.05, 0.02, 1e-5]


BLOCKS = [("W1", OC.OW1, OC.OB1), ("b1", OC.OB1, OC.OW2), ("W2", OC.OW2, OC.OB2), ("b2", OC.OB2, OC.OW3),
          ("W3", OC.OW3, OC.OW3 + 4 * OC.HID), ("b3", OC.OB3, OC.OB3 + 4)]


def _rel(a, b):
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


@pytest.mark.parametrize("act", [OC.TANH, OC.RELU])
def test_closure_forward_and_gradient_parity(setup, act):
    """The fused forward kernel (closure_forward) and the layer-by-layer
    kernels of the gradient against the oracle: the bfloat16-emulating one
    (tight bars) and the plain FP64 network (bars from the bfloat16 effect)."""
    import torch
    st = setup
    say(f"closure: forward and gradient vs the oracle, cartesian 400 m, E = 3, activation {act}")
    rng = np.random.default_rng(4)
    p = OC.init_params(seed=5).astype(np.float64)
    p[OC.OB1:OC.OW2] = rng.normal(0, 0.1, OC.HID)
    p[OC.OB3:OC.OB3 + 4] = rng.normal(0, 0.1, 4)
    p = p.astype(np.float32)
    p64 = p.astype(np.float64)
    cl, nodef = _closure(st, p, IN_SCALE, OUT_SCALE, act)
    s = torch.from_numpy(st["closed"].astype(np.float32)).cuda().contiguous()
    na, E = st["nd"].n_active, st["E"]
    X = OC.features(st["closed"], st["o_idx"], nodef, IN_SCALE)
    Ye = OC.forward(p64, X, emulate=True, act=act)[0][:, :4]
    Yp = OC.forward(p64, X, emulate=False, act=act)[0][:, :4]
    got = cl.forward(s).cpu().numpy().reshape(na * E, 4) / np.array(OUT_SCALE)
    e_em, e_pl, e_bf = _rel(got, Ye), _rel(got, Yp), _rel(Ye, Yp)
    say(f"   forward rel-l2: vs emulated {e_em:.2e}, vs plain FP64 {e_pl:.2e} (bfloat16 effect {e_bf:.2e})")
    assert e_em < 5e-4
    assert e_pl <= 1.25 * e_bf + 2e-4
    T = rng.normal(0, 1, (na * E, 4))
    loss_e, g_e = OC.loss_and_grad(p64, X, T, emulate=True, act=act)
    loss_p, g_p = OC.loss_and_grad(p64, X, T, emulate=False, act=act)
    g, loss = cl.gradient(s, torch.from_numpy(T.astype(np.float32)).cuda().reshape(na, E, 4).contiguous())
    g = g.cpu().numpy().astype(np.float64)
    say(f"   loss gpu {loss:.8f} emulated {loss_e:.8f} plain {loss_p:.8f}")
    assert abs(loss - loss_e) <= 1e-5 * loss_e
    assert abs(loss - loss_p) <= 1.25 * abs(loss_e - loss_p) + 1e-5 * loss_p
    for name, a, b in BLOCKS:
        e_em, e_pl, e_bf = _rel(g[a:b], g_e[a:b]), _rel(g[a:b], g_p[a:b]), _rel(g_e[a:b], g_p[a:b])
        say(f"   grad {name}: vs emulated {e_em:.2e}, vs plain FP64 {e_pl:.2e} (bfloat16 effect {e_bf:.2e})")
        assert e_em < 3e-4, name
        assert e_pl <= 1.25 * e_bf + 2e-4, name
    assert np.all(g[OC.OW3 + 4 * OC.HID:OC.OB3] == 0.0)


def test_closure_tuner_shapes_are_bit_identical(setup):
    """Every launch shape of the fused forward kernel (tiles per wavefront,
    wavefronts per block, occupancy) computes the same correction bit for
    bit; the tuner keeps one of them."""
    import torch
    st = setup
    say("closure tuner: every forward launch shape bit-identical")
    p = OC.init_params(seed=5)
    cl, _ = _closure(st, p, IN_SCALE, OUT_SCALE, OC.RELU)
    s = torch.from_numpy(st["closed"].astype(np.float32)).cuda().contiguous()
    ref = cl.forward(s)
    for shape in range(5):
        got, us = cl.tune(s, shape)
        assert got == shape
        assert torch.equal(cl.forward(s), ref), shape
        say(f"   shape {shape}: {us:.1f} us per call")
    chosen, us = cl.tune(s)
    assert 0 <= chosen < 5 and torch.equal(cl.forward(s), ref)


def test_closure_training_lowers_the_loss(setup):
    import torch
    st = setup
    say("closure: 60 Adam steps on one batch lower the loss")
    cl, _ = _closure(st, OC.init_params(seed=1), IN_SCALE, OUT_SCALE)
    s = torch.from_numpy(st["closed"].astype(np.float32)).cuda().contiguous()
    # learnable targets: smooth functions of each node's own fields
    own = torch.from_numpy(st["closed"][:st["nd"].n_active].astype(np.float32)).cuda()
    sc = torch.tensor(IN_SCALE, device="cuda")
    T = torch.tanh(own / sc) + 0.5 * torch.tanh(own / sc).roll(1, dims=2)
    losses = [cl.train_step(s, T.contiguous(), 3e-3) for _ in range(60)]
    say(f"   loss {losses[0]:.4f} -> {losses[-1]:.4f}")
    assert losses[-1] < 0.2 * losses[0]


def test_closure_fallback_keeps_the_plain_step(setup):
    """A correction that is not finite leaves the plain coarse step."""
    import torch
    st = setup
    R = st["R"]
    say("closure: non-finite network output -> plain coarse step for every member")
    p = OC.init_params(seed=1)
    p[OC.OB3] = np.nan
    cl, _ = _closure(st, p, IN_SCALE, OUT_SCALE)
    s0 = torch.from_numpy(st["closed"].astype(np.float32)).cuda().contiguous()
    s1, s2 = s0.clone(), s0.clone()
    R.rbffd_step(st["ctx"], st["gm"], s1, 0.0, 1.0, 2, R.RK4)
    t, fb = cl.step(s2, 0.0, 1.0, 2, R.RK4)
    assert fb == 2 * st["E"]
    na = st["nd"].n_active
    assert torch.equal(s1[:na], s2[:na])


def test_learned_closure_beats_plain_coarse_run():
    """The whole learned part at the workload's 256 seeded members: a fine
    (50 m) ensemble of the same method, restricted to the coarse (400 m)
    nodes, gives one-step correction targets over the first 150 s; the
    library's kernels train the relu network on 192 members; on the 64
    held-out members the corrected coarse run is closer to the fine run than
    the plain coarse run at 30, 60, 120 and 150 s, and at 150 s by a wide
    margin.

    The window ends where the 400 m run stops resolving the current (its
    error doubles between 120 and 150 s and reaches 0.57 by 300 s): trained
    on the later, 30x larger corrections as well, the network's absolute
    error swamps the early, small ones."""
    from paper_1509_02615_amd import rbffd as R
    from paper_1509_02615_amd import closure as CL
    ctx = R.Context(0)
    cc = closure_config(n_members=256, n_train=192)
    say(f"learned closure: fine ensemble 256 x {cc['fine']['nodes'].n_active} nodes, 150 s; 192 train, 64 held out")
    q = CL.quality_run(ctx, cc, log=say)
    say(f"   training {q['train_s']:.1f} s, loss {q['loss_first']:.3f} -> {q['loss_last']:.3f}")
    res = q["errors"]
    for c, (ep, ec) in res.items():
        say(f"   t = {c:4d} s: theta' rel-l2 vs fine, plain {ep:.4f}, with closure {ec:.4f}")
    say(f"   corrected coarse run {q['corrected_run_s']:.2f} s for 64 members vs fine run {q['fine_run_s']:.1f} s for 256")
    assert q["fallbacks"] == 0
    assert all(res[c][1] < res[c][0] for c in (30, 60, 120, 150))
    assert res[150][1] < 0.6 * res[150][0]


import time  # noqa: E402


@pytest.mark.parametrize("nx, nz, n, E, act", [(10, 5, 13, 1, OC.RELU),      # one tile of 64 samples, not full
                                               (16, 4, 13, 1, OC.TANH),      # exactly one tile
                                               (24, 9, 37, 77, OC.RELU),     # more tiles than compute units, a remainder
                                               (24, 9, 21, 7, OC.TANH)])
def test_closure_gradient_tile_edges(nx, nz, n, E, act):
    """The fused training kernel at the edges of its 64-sample tiles and for
    stencils shorter than 37, against the bfloat16-emulating oracle; the
    padding parameters (nonzero here) get no gradient.

    Bar: FP32 sums of up to 160 terms are off by at most 160 x 2^-24 of their
    size, against a bfloat16 spacing of 2^-8, so about 1% of the stored values
    at most round the other way, each by 2^-8: sqrt(0.01) 2^-8 = 4e-4 relative
    l2 per layer, over three layers 1.2e-3."""
    import torch
    from paper_1509_02615_amd import rbffd as R
    h = 1.0 / nx
    i, j = np.meshgrid(np.arange(nx), np.arange(nz))
    xy = np.stack([i.ravel() * h, j.ravel() * h], 1)
    na = len(xy)
    ghost = np.concatenate([xy[:nx] - [0.0, h], xy[-nx:] + [0.0, h]])
    xy = np.concatenate([xy, ghost])
    bnd = np.concatenate([np.arange(nx), na - nx + np.arange(nx)]).astype(np.int32)
    ctx = R.Context(0)
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()              # noqa: E731
    ops = [(R.DX, 0, 0), (R.DZ, 0, 0), (R.LAP, 0, 0), (R.HYPERLAP, 3, 7)]
    idx, W, _, _ = R.rbffd_weights(ctx, dev(xy), ops, n, 7, 2, period_x=1.0, n_centers=na)
    _, Ww, _, _ = R.rbffd_weights(ctx, dev(xy), [(R.DZ, 0, 0), (R.DZZ, 0, 0)], n, 7, 2, period_x=1.0, centers=dev(bnd))
    model = R.Model(ctx, R.PHYS_NS, idx, W, dev(xy), na, field_dtype=R.F32, weight_dtype=R.F32, ensemble=E,
                    hv_coeff=0.0, consts=dict(c_p=1004.0, c_v=717.0, R_d=287.0, g=9.81, theta_bar=300.0, mu=75.0),
                    bnd_nodes=dev(bnd), bnd_ghosts=dev((na + np.arange(2 * nx)).astype(np.int32)),
                    bnd_normal=dev(np.zeros(2 * nx, np.int32)), bnd_d1=Ww[0].contiguous(), bnd_d2=Ww[1].contiguous())
    rng = np.random.default_rng(7)
    p = OC.init_params(seed=3)
    for a, b in ((OC.OB1, OC.OW2), (OC.OB2, OC.OW3), (OC.OB3, OC.OB3 + 4)):
        p[a:b] = rng.normal(0, 0.1, b - a)
    state = (rng.normal(0, 1, (len(xy), E, 4)) * np.array(IN_SCALE)).astype(np.float32)
    nodef = xy[:na, 1].astype(np.float32).astype(np.float64)
    cl = R.Closure(ctx, model, dev(p), dev(nodef), IN_SCALE, OUT_SCALE, activation=act)
    T = rng.normal(0, 1, (na * E, 4)).astype(np.float32)
    g, loss = cl.gradient(dev(state), dev(T.reshape(na, E, 4)))
    g = g.cpu().numpy().astype(np.float64)
    X = OC.features(state.astype(np.float64), idx.cpu().numpy(), nodef, IN_SCALE)
    loss_e, g_e = OC.loss_and_grad(p.astype(np.float64), X, T.astype(np.float64), emulate=True, act=act)
    say(f"closure gradient, {na * E} samples, n = {n}: loss {loss:.8f} against {loss_e:.8f}")
    assert abs(loss - loss_e) <= 1e-4 * loss_e
    for name, a, b in BLOCKS:
        say(f"   {name}: {_rel(g[a:b], g_e[a:b]):.2e}")
        assert _rel(g[a:b], g_e[a:b]) < 1.2e-3, name
    assert np.all(g[OC.OW1:OC.OB1].reshape(OC.HID, OC.KIN)[:, 149:] == 0.0)
    assert np.all(g[OC.OW3 + 4 * OC.HID:OC.OB3] == 0.0) and np.all(g[OC.OB3 + 4:] == 0.0)
    g2, loss2 = cl.gradient(dev(state), dev(T.reshape(na, E, 4)))
    assert loss2 == loss and np.array_equal(g2.cpu().numpy().astype(np.float64), g)   # fixed summation order


def test_closure_gradient_of_nan_activations(setup):
    """relu's derivative is 0 where the activation is not above 0, and a NaN is
    not: with one NaN hidden unit in layer 1, which makes all of layer 2 and the
    outputs NaN, nothing flows back through either layer. The loss and the
    output layer's gradient are NaN; the biases and weights below get exactly 0
    (but for the W2 column that multiplies the NaN unit itself)."""
    import torch
    st = setup
    p = OC.init_params(seed=5)
    p[OC.OB1 + 5] = np.nan
    cl, _ = _closure(st, p, IN_SCALE, OUT_SCALE, OC.RELU)
    s = torch.from_numpy(st["closed"].astype(np.float32)).cuda().contiguous()
    T = torch.zeros((st["nd"].n_active, st["E"], 4), dtype=torch.float32, device="cuda")
    g, loss = cl.gradient(s, T)
    g = g.cpu().numpy()
    assert np.isnan(loss)
    assert np.all(np.isnan(g[OC.OB3:OC.OB3 + 4])) and np.all(np.isnan(g[OC.OW3:OC.OW3 + 4 * OC.HID]))
    W2 = g[OC.OW2:OC.OB2].reshape(OC.HID, OC.HID)
    assert np.all(np.isnan(W2[:, 5])) and np.all(np.delete(W2, 5, 1) == 0.0)
    assert np.all(g[OC.OB2:OC.OW3] == 0.0)
    assert np.all(g[OC.OW1:OC.OW2] == 0.0)


def test_closure_fallback_of_one_member_in_one_step(setup):
    """A member whose correction is not finite keeps the plain step, the others
    are corrected, and a member that was bad in one step is corrected again in
    the next: member 1 carries a spike of theta' whose input overflows before
    the first step and, smoothed by it, no longer before the second (the
    network's theta' weights are 0, so a finite input does nothing and an
    infinite one makes NaN). The corrected states are dt times the forward pass
    added to plain steps, to a few FP32 roundings."""
    import torch
    st = setup
    R, na, E, dt = st["R"], st["nd"].n_active, st["E"], 1.0
    p = OC.init_params(seed=2)
    p[OC.OW1:OC.OB1].reshape(OC.HID, OC.KIN)[:, 2:4 * OC.NSLOT:4] = 0.0
    y0 = torch.from_numpy(st["closed"].astype(np.float32)).cuda().contiguous()
    spike = na // 2 + 40
    y0[spike, 1, 2] += 60.0
    R.rbffd_ghost(st["ctx"], st["gm"], y0)
    y1 = y0.clone()
    R.rbffd_step(st["ctx"], st["gm"], y1, 0.0, dt, 1, R.RK4)

    def largest(y):                                        # largest theta' input of each member
        th = y[..., 2].double()
        d = th[torch.from_numpy(st["o_idx"]).cuda().long()] - th[:na, None]
        return torch.maximum(d.abs().amax((0, 1)), th[:na].abs().amax(0)).cpu().numpy()
    f0, f1 = largest(y0), largest(y1)
    say(f"closure: one bad member, largest theta' inputs {f0} then {f1}")
    # (the threshold lies between them, further from both than BF16's spacing of 2^-8)
    assert f1[1] < 0.98 * f0[1] and max(f0[0], f0[2], f1[0], f1[2]) < 0.98 * f1[1]
    scale = list(IN_SCALE)
    scale[2] = float(np.sqrt(f0[1] * f1[1]) / np.finfo(np.float32).max)
    cl, _ = _closure(st, p, scale, OUT_SCALE, OC.RELU)
    want, fallbacks = y0.clone(), []
    for k in range(2):
        R.rbffd_ghost(st["ctx"], st["gm"], want)
        corr = cl.forward(want)
        good = torch.isfinite(corr).all(dim=2).all(dim=0)
        fallbacks.append([int(e) for e in torch.nonzero(~good)])
        R.rbffd_step(st["ctx"], st["gm"], want, 0.0, dt, 1, R.RK4)
        want[:na, good] += dt * corr[:, good]
    assert fallbacks == [[1], []]
    got = y0.clone()
    assert cl.step(got, 0.0, dt, 1, R.RK4)[1] == 1
    assert torch.equal(got[:na, 1], y1[:na, 1])
    assert not torch.equal(got[:na, 0], y1[:na, 0]) and not torch.equal(got[:na, 2], y1[:na, 2])
    got = y0.clone()
    assert cl.step(got, 0.0, dt, 2, R.RK4)[1] == 1
    for f in range(4):
        size = want[:na, :, f].abs().amax()
        assert float((got[:na, :, f] - want[:na, :, f]).abs().amax() / size) < 1e-5, f
