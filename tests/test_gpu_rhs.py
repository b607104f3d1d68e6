"""GPU parity of the ghost closure, the fused right-hand side and the RK
stages against the CPU oracle, through the C ABI.

Tolerances: FP64 paths agree with the oracle to 1e-12 relative l2 per field
for one evaluation (rounding-order differences only) and to 1e-9 after a
multi-step run; the FP32-field path (FP32 weights, the divergence and the
hyperviscosity sums in FP64 on corrected weights) meets 1e-6 per field on
FP32-representable inputs, also on a developed flow; BF16 weights (Dx and Dz
with an 8-bit correction, about 16 significant bits; Lap 8 bits) are held to
2e-3 per field."""

import numpy as np
import pytest

import oracle as O
from oracle.pipeline import build_ns, build_advection
from workloads import advection_config, density_current_config, scale_config
from workloads.fields import smooth_ns_state

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a HIP device"
    from paper_1509_02615_amd import rbffd
    return rbffd


@pytest.fixture(scope="module")
def ctx(R):
    return R.Context(0)


def say(*a):
    print(*a, flush=True)


def dev(a, dtype):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(dtype).cuda()


def host(t):
    return t.double().cpu().numpy()


_NS_CACHE = {}


def ns_case(layout, h, translating=False):
    key = (layout, h, translating)
    if key not in _NS_CACHE:
        from workloads import translating_config
        cfg = (translating_config if translating else density_current_config)(layout, h)
        model, idx, W, Ww = build_ns(cfg)
        _NS_CACHE[key] = (cfg, model, idx, W, Ww)
    return _NS_CACHE[key]


def gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=0, wdt=0, E=1, hv=None):
    import torch
    nd = cfg["nodes"]
    n = idx.shape[1]
    Wwall = Ww.reshape(2, -1, n)
    return R.Model(ctx, R.PHYS_NS, dev(idx, torch.int32), dev(W, torch.float64), dev(nd.xy, torch.float64),
                   nd.n_active, field_dtype=fdt, weight_dtype=wdt, ensemble=E,
                   hv_coeff=cfg["hv_coeff"] if hv is None else hv, consts=cfg["consts"],
                   bnd_nodes=dev(nd.bnd_nodes, torch.int32), bnd_ghosts=dev(nd.bnd_ghosts, torch.int32),
                   bnd_normal=dev(nd.bnd_normal, torch.int32),
                   bnd_d1=dev(Wwall[0], torch.float64), bnd_d2=dev(Wwall[1], torch.float64))


def rel_fields(a, b, rows):
    return [np.linalg.norm(a[rows, f] - b[rows, f]) / np.linalg.norm(b[rows, f]) for f in range(a.shape[1])]


def test_rhs_parity_background_wind(R, ctx):
    import torch
    say("rhs: translating density current (u_bar = 20 m/s), hexagonal 400 m, FP64")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0, translating=True)
    gm = gpu_ns(R, ctx, cfg, idx, W, Ww)
    st = smooth_ns_state(cfg["nodes"], seed=8)
    ref, _ = O.ns_rhs(om, st)
    s = dev(st, torch.float64).reshape(gm.state_shape()).contiguous()
    out = torch.empty_like(s)
    R.rbffd_rhs(ctx, gm, 0.0, s, out)
    got = host(out).reshape(st.shape)
    errs = rel_fields(got, ref, np.arange(cfg["nodes"].n_active))
    say(f"   rel-l2 per field {['%.1e' % e for e in errs]}")
    assert max(errs) <= 1e-12


@pytest.mark.parametrize("layout", ["cartesian", "hexagonal", "scattered"])
def test_ghost_closure_parity(R, ctx, layout):
    import torch
    say(f"closure: {layout} 400 m, FP64, smooth seeded state")
    cfg, om, idx, W, Ww = ns_case(layout, 400.0)
    gm = gpu_ns(R, ctx, cfg, idx, W, Ww)
    st = smooth_ns_state(cfg["nodes"], seed=2)
    ref = O.ghost_closure(om, st)
    s = dev(st, torch.float64).reshape(gm.state_shape()).contiguous()
    R.rbffd_ghost(ctx, gm, s)
    got = host(s).reshape(st.shape)
    g = cfg["nodes"].ghost_nodes.ravel()
    for f in range(4):
        err = np.abs(got[g, f] - ref[g, f]).max() / max(np.abs(ref[g, f]).max(), 1e-300)
        assert err <= 1e-12, (f, err)
    wall = cfg["nodes"].wall_nodes.ravel()
    assert np.all(got[wall, 1] == 0.0)


_BOX_CACHE = {}


def box_case(layout):
    """The rising-bubble box (four walls) at 400 m."""
    if layout not in _BOX_CACHE:
        from workloads import bubble_config
        cfg = bubble_config(layout, 400.0)
        model, idx, W, Ww = build_ns(cfg)
        _BOX_CACHE[layout] = (cfg, model, idx, W, Ww)
    return _BOX_CACHE[layout]


def box_state(nd, seed):
    """Seeded smooth state on the box: u, w ~ 15 m/s, theta' ~ 10 K, pi' ~ 1e-3."""
    rng = np.random.Generator(np.random.PCG64(seed))
    x, z = nd.xy[:, 0] / nd.width, nd.xy[:, 1] / nd.height
    s = np.zeros((nd.n_total, 4))
    for f, amp in enumerate([15.0, 15.0, 10.0, 1e-3]):
        for _ in range(3):
            kx, kz = rng.integers(1, 4, 2)
            px, pz = rng.uniform(0, 2 * np.pi, 2)
            s[:, f] += rng.uniform(-1, 1) * amp / 3 * np.cos(np.pi * kx * x + px) * np.cos(np.pi * kz * z + pz)
    s[nd.n_active:] = 0.0
    return s


@pytest.mark.parametrize("layout", ["cartesian", "hexagonal", "scattered"])
def test_box_ghost_closure_parity(R, ctx, layout):
    """Four walls (Section 6.5): lateral rows close u with d2/dx2 and w,
    theta', pi' with d/dx; corner rows of two walls share one coupled solve."""
    import torch
    say(f"closure: rising-bubble box {layout} 400 m, FP64")
    cfg, om, idx, W, Ww = box_case(layout)
    nd = cfg["nodes"]
    gm = gpu_ns(R, ctx, cfg, idx, W, Ww)
    st = box_state(nd, seed=4)
    ref = O.ghost_closure(om, st)
    s = dev(st, torch.float64).reshape(gm.state_shape()).contiguous()
    R.rbffd_ghost(ctx, gm, s)
    got = host(s).reshape(st.shape)
    g = nd.bnd_ghosts
    for f in range(4):
        err = np.abs(got[g, f] - ref[g, f]).max() / max(np.abs(ref[g, f]).max(), 1e-300)
        say(f"   field {f}: max ghost error / max ghost {err:.1e}")
        assert err <= 1e-12, (f, err)
    zn = nd.bnd_normal == 0
    assert np.all(got[nd.bnd_nodes[zn], 1] == 0.0) and np.all(got[nd.bnd_nodes[~zn], 0] == 0.0)


@pytest.mark.parametrize("layout,fdt,tol", [("cartesian", 0, 1e-12), ("hexagonal", 0, 1e-12),
                                            ("scattered", 0, 1e-12), ("cartesian", 1, 1e-6)])
def test_box_rhs_parity(R, ctx, layout, fdt, tol):
    import torch
    say(f"rhs: rising-bubble box {layout} 400 m, field/weight dtype {fdt}")
    cfg, om, idx, W, Ww = box_case(layout)
    nd = cfg["nodes"]
    gm = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=fdt, wdt=fdt)
    st = box_state(nd, seed=5)
    if fdt == 1:
        st = st.astype(np.float32).astype(np.float64)
    ref, _ = O.ns_rhs(om, st)
    s = dev(st, torch.float64 if fdt == 0 else torch.float32).reshape(gm.state_shape()).contiguous()
    out = torch.full_like(s, float("nan"))
    R.rbffd_rhs(ctx, gm, 0.0, s, out)
    got = host(out).reshape(st.shape)
    errs = rel_fields(got, ref, np.arange(nd.n_active))
    say(f"   rel-l2 per field {['%.1e' % e for e in errs]}")
    assert max(errs) <= tol
    k = nd.kinds()[:nd.n_active]
    assert np.all(got[:nd.n_active][(k & 1) > 0, 1] == 0.0) and np.all(got[:nd.n_active][(k & 4) > 0, 0] == 0.0)


def test_box_steps_parity(R, ctx):
    """30 RK4 steps of the rising bubble (FP64), Cartesian 400 m, against the
    oracle's integration."""
    import torch
    say("steps: rising bubble, cartesian 400 m, 30 RK4 steps, FP64")
    cfg, om, idx, W, Ww = box_case("cartesian")
    gm = gpu_ns(R, ctx, cfg, idx, W, Ww)
    yref, _ = O.integrate(lambda t, y: O.ns_rhs(om, y)[0], cfg["state0"], 0.0, cfg["dt"], 30, "rk4")
    s = dev(cfg["state0"], torch.float64).reshape(gm.state_shape()).contiguous()
    R.rbffd_step(ctx, gm, s, 0.0, cfg["dt"], 30, R.RK4)
    got = host(s).reshape(yref.shape)
    na = cfg["nodes"].n_active
    errs = [np.linalg.norm(got[:na, f] - yref[:na, f]) / np.linalg.norm(yref[:na, f]) for f in range(4)]
    say(f"   rel-l2 per field {['%.1e' % e for e in errs]}")
    assert max(errs) <= 1e-10


@pytest.mark.parametrize("layout,h", [("cartesian", 400.0), ("hexagonal", 400.0), ("scattered", 400.0),
                                      ("hexagonal", 200.0)])
def test_rhs_parity_fp64(R, ctx, layout, h):
    import torch
    say(f"rhs: {layout} {h} m, FP64 fields and weights")
    cfg, om, idx, W, Ww = ns_case(layout, h)
    gm = gpu_ns(R, ctx, cfg, idx, W, Ww)
    st = smooth_ns_state(cfg["nodes"], seed=3)
    ref, _ = O.ns_rhs(om, st)
    s = dev(st, torch.float64).reshape(gm.state_shape()).contiguous()
    out = torch.full_like(s, float("nan"))
    R.rbffd_rhs(ctx, gm, 0.0, s, out)
    got = host(out).reshape(st.shape)
    na = cfg["nodes"].n_active
    errs = rel_fields(got, ref, np.arange(na))
    say(f"   rel-l2 per field {['%.1e' % e for e in errs]}")
    assert max(errs) <= 1e-12
    assert np.all(got[na:] == 0.0)


@pytest.mark.parametrize("wdt,tol", [(1, 1e-6), (2, 2e-3)])
@pytest.mark.parametrize("h", [400.0, 200.0])
def test_rhs_parity_reduced_precision(R, ctx, wdt, tol, h):
    import torch
    say(f"rhs: hexagonal {h} m, FP32 fields, weight dtype {wdt}, tol {tol}")
    cfg, om, idx, W, Ww = ns_case("hexagonal", h)
    gm = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=1, wdt=wdt)
    st = smooth_ns_state(cfg["nodes"], seed=4).astype(np.float32).astype(np.float64)
    ref, _ = O.ns_rhs(om, st)
    s = dev(st, torch.float32).reshape(gm.state_shape()).contiguous()
    out = torch.empty_like(s)
    R.rbffd_rhs(ctx, gm, 0.0, s, out)
    got = host(out).reshape(st.shape)
    errs = rel_fields(got, ref, np.arange(cfg["nodes"].n_active))
    say(f"   rel-l2 per field {['%.2e' % e for e in errs]}")
    assert max(errs) <= tol


@pytest.mark.parametrize("h", [400.0, 200.0])
def test_rhs_parity_developed_state(R, ctx, h):
    """One right-hand side on a developed flow: the hexagonal density
    current integrated by the oracle to t = 300 s (stored by
    tests/golden/make_developed_states.py; Section 6.4), in FP64, FP32 fields
    and weights (on the FP32-rounded state) and BF16 weights, against the
    oracle on the same input."""
    import os
    import torch
    say(f"rhs: developed hexagonal {h} m state at t = 300 s (oracle run), FP64 / FP32 / BF16 weights")
    cfg, om, idx, W, Ww = ns_case("hexagonal", h)
    path = os.path.join(os.path.dirname(__file__), "golden", f"developed_hexagonal_{int(h)}m_300s.npz")
    st64 = np.load(path)["state"]
    na = cfg["nodes"].n_active
    assert st64.shape == (cfg["nodes"].n_total, 4) and np.abs(st64[:na, 2]).max() > 5.0
    for fdt, wdt, tol in ((0, 0, 1e-12), (1, 1, 1e-6), (1, 2, 2e-3)):
        st = st64 if fdt == 0 else st64.astype(np.float32).astype(np.float64)
        ref, _ = O.ns_rhs(om, st)
        gm = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=fdt, wdt=wdt)
        s = dev(st, torch.float64 if fdt == 0 else torch.float32).reshape(gm.state_shape()).contiguous()
        out = torch.full_like(s, float("nan"))
        R.rbffd_rhs(ctx, gm, 300.0, s, out)
        got = host(out).reshape(st.shape)
        errs = rel_fields(got, ref, np.arange(na))
        say(f"   fields {fdt} weights {wdt}: rel-l2 per field {['%.2e' % e for e in errs]} (bar {tol})")
        assert max(errs) <= tol
        del gm


def test_fp32_model_rejects_hyperviscosity_weights_beyond_fp32(R, ctx):
    """The FP32 and BF16 layouts store the Lap^k weights as an FP32 value
    plus a relative correction, so weights outside the FP32 normal range are
    rejected at model creation (EINVAL); FP64 weights take them."""
    say("model: FP32 and BF16 layouts reject Lap^k weights beyond the FP32 range, FP64 accepts them")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0)
    Wbig = W.copy()
    Wbig[3] *= 1e60   # weights of about 1e-16 at 400 m end beyond 3.4e38
    for wdt in (1, 2):
        with pytest.raises(R.RbffdError) as e:
            gpu_ns(R, ctx, cfg, idx, Wbig, Ww, fdt=1, wdt=wdt)
        assert e.value.code == R.EINVAL
    gpu_ns(R, ctx, cfg, idx, Wbig, Ww, fdt=0, wdt=0).close()


def test_rhs_independent_of_node_order(R, ctx):
    """Neighbour indices travel as 16-bit offsets j - i, with an escape to the
    full index beyond +-32767. A random order of the active nodes of the 50 m
    hexagonal channel (about 150k nodes, most offsets beyond that range)
    gives the same tendency node for node, bit for bit (FP64, FP32 and BF16
    weights)."""
    import torch
    from paper_1509_02615_amd import pipeline as P
    say("rhs: random order of the 50 m hexagonal channel's active nodes, same tendency bit for bit")
    cfg = density_current_config("hexagonal", 50.0)
    nd = cfg["nodes"]
    na, N = nd.n_active, nd.n_total
    xy, idx, W, Ww, _ = P.ns_weights(ctx, cfg)
    rng = np.random.default_rng(12)
    order = rng.permutation(na)                    # new node k is old node order[k]
    new_of_old = np.arange(N)
    new_of_old[order] = np.arange(na)
    order_t, map_t = dev(order, torch.int64), dev(new_of_old, torch.int64)
    idx2 = map_t[idx.long()[order_t]].int().contiguous()
    W2 = W[:, order_t].contiguous()
    xy2 = xy.clone()
    xy2[:na] = xy[order_t]
    far = (idx2.long() - torch.arange(na, device="cuda")[:, None]).abs() > 32767
    say(f"   {float(far.float().mean()):.0%} of the offsets beyond +-32767")
    assert float(far.float().mean()) > 0.5
    st = smooth_ns_state(nd, seed=5)
    st2 = st.copy()
    st2[:na] = st[order]
    Wwall = Ww.reshape(2, -1, idx.shape[1])
    for fdt, wdt, dt in ((R.F64, R.F64, torch.float64), (R.F32, R.F32, torch.float32),
                         (R.F32, R.BF16, torch.float32)):
        outs = []
        for ix, w, x, s, bn in ((idx, W, xy, st, nd.bnd_nodes), (idx2, W2, xy2, st2, new_of_old[nd.bnd_nodes])):
            m = R.Model(ctx, R.PHYS_NS, ix, w, x, na, field_dtype=fdt, weight_dtype=wdt, hv_coeff=cfg["hv_coeff"],
                        consts=cfg["consts"], bnd_nodes=dev(bn, torch.int32),
                        bnd_ghosts=dev(nd.bnd_ghosts, torch.int32), bnd_normal=dev(nd.bnd_normal, torch.int32),
                        bnd_d1=Wwall[0].contiguous(), bnd_d2=Wwall[1].contiguous())
            sv = dev(s, dt).reshape(m.state_shape()).contiguous()
            o = torch.empty_like(sv)
            R.rbffd_rhs(ctx, m, 0.0, sv, o)
            outs.append(o.reshape(N, 4))
            m.close()
        assert torch.equal(outs[1][:na], outs[0][:na][order_t]), (fdt, wdt)


def test_centre_slot_skip_is_exact(R, ctx):
    """Centre-subtracted sums give the centre slot a zero term, so a model
    whose stencils all start with their own node streams only the other
    slots. Swapping the first two slots of one interior stencil makes the
    model keep every slot (more bytes per node); the tendency is the same
    bit for bit (FP64, FP32, BF16 weights)."""
    import torch
    say("rhs: centre slot left out of the stream vs kept, same tendency bit for bit")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0)
    nd = cfg["nodes"]
    assert (idx[:, 0] == np.arange(idx.shape[0])).all()
    k = nd.n_active // 2
    assert k not in set(nd.bnd_nodes.tolist())
    idx2, W2 = idx.copy(), W.copy()
    idx2[k, [0, 1]] = idx2[k, [1, 0]]
    W2[:, k, [0, 1]] = W2[:, k, [1, 0]]
    st = smooth_ns_state(nd, seed=21)
    for fdt, wdt, dt in ((R.F64, R.F64, torch.float64), (R.F32, R.F32, torch.float32),
                         (R.F32, R.BF16, torch.float32)):
        outs, bpn = [], []
        for ix, w in ((idx, W), (idx2, W2)):
            m = gpu_ns(R, ctx, cfg, ix, w, Ww, fdt=fdt, wdt=wdt)
            s = dev(st, dt).reshape(m.state_shape()).contiguous()
            o = torch.empty_like(s)
            R.rbffd_rhs(ctx, m, 0.0, s, o)
            outs.append(o)
            bpn.append(m.bytes_per_node())
            m.close()
        assert bpn[0] < bpn[1], (fdt, wdt, bpn)
        assert torch.equal(outs[0], outs[1]), (fdt, wdt)


def test_rhs_rest_state_is_zero(R, ctx):
    import torch
    say("rhs: hydrostatic rest gives exactly zero tendency (FP64 and FP32)")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0)
    for fdt, wdt, dt in ((0, 0, torch.float64), (1, 1, torch.float32)):
        gm = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=fdt, wdt=wdt)
        s = torch.zeros(gm.state_shape(), dtype=dt, device="cuda")
        out = torch.full_like(s, 1.0)
        R.rbffd_rhs(ctx, gm, 0.0, s, out)
        assert torch.count_nonzero(out).item() == 0


def test_ensemble_members_equal_single_runs(R, ctx):
    import torch
    say("rhs: ensemble E=3 (FP32) equals three single-member evaluations bit for bit")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0)
    states = [smooth_ns_state(cfg["nodes"], seed=10 + k).astype(np.float32) for k in range(3)]
    g1 = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=1, wdt=1)
    singles = []
    for st in states:
        s = dev(st, torch.float32).reshape(g1.state_shape()).contiguous()
        o = torch.empty_like(s)
        R.rbffd_rhs(ctx, g1, 0.0, s, o)
        singles.append(o.reshape(-1, 4))
    g3 = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=1, wdt=1, E=3)
    s3 = dev(np.stack(states, axis=1), torch.float32).contiguous()
    o3 = torch.empty_like(s3)
    R.rbffd_rhs(ctx, g3, 0.0, s3, o3)
    for k in range(3):
        assert torch.equal(o3[:, k, :], singles[k])


@pytest.mark.parametrize("E", [16, 64])
def test_large_ensemble_members_match_single_runs(R, ctx, E):
    """From 16 members on, the ghost closure runs one member per lane with
    its sums in slot order (and from 64 the stage kernel one member per
    wavefront): each member agrees with its single-member run to FP32
    rounding."""
    import torch
    say(f"rhs: ensemble E={E} (FP32) vs single-member evaluations, rel-l2 <= 1e-6 per member")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0)
    states = [smooth_ns_state(cfg["nodes"], seed=30 + k).astype(np.float32) for k in range(E)]
    g1 = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=1, wdt=1)
    gE = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=1, wdt=1, E=E)
    sE = dev(np.stack(states, axis=1), torch.float32).contiguous()
    oE = torch.empty_like(sE)
    R.rbffd_rhs(ctx, gE, 0.0, sE, oE)
    worst = 0.0
    for k in range(0, E, 5):
        s = dev(states[k], torch.float32).reshape(g1.state_shape()).contiguous()
        o = torch.empty_like(s)
        R.rbffd_rhs(ctx, g1, 0.0, s, o)
        a, b = oE[:, k, :].double(), o.reshape(-1, 4).double()
        for c in range(4):
            worst = max(worst, float(torch.linalg.norm(a[:, c] - b[:, c]) / torch.linalg.norm(b[:, c])))
    say(f"   worst per-field rel-l2 {worst:.2e}")
    assert worst <= 1e-6


def test_advection_rhs_and_bell_run(R, ctx):
    import torch
    say("transport: 64x64 rhs at t=0.7 and the full 2000-step RK4 bell run (FP64)")
    cfg = advection_config(64)
    om, idx, W, status = build_advection(cfg)
    nd = cfg["nodes"]
    gm = R.Model(ctx, R.PHYS_ADVECTION, dev(idx, torch.int32), dev(W, torch.float64), dev(nd.xy, torch.float64),
                 nd.n_active, hv_coeff=cfg["hv_coeff"], vel_u=dev(cfg["U"], torch.float64),
                 vel_v=dev(cfg["V"], torch.float64), vel_period=cfg["vel_period"])
    psi = cfg["psi0"]
    ref = om(0.7, psi)
    s = dev(psi, torch.float64).reshape(gm.state_shape()).contiguous()
    out = torch.empty_like(s)
    R.rbffd_rhs(ctx, gm, 0.7, s, out)
    got = host(out).ravel()
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 1e-12
    yref, _ = O.integrate(om, psi, 0.0, cfg["dt"], 2000, "rk4")
    t = R.rbffd_step(ctx, gm, s, 0.0, cfg["dt"], 2000, R.RK4)
    assert abs(t - 5.0) < 1e-12
    y = host(s).ravel()
    d = np.linalg.norm(y - yref) / np.linalg.norm(yref)
    e_gpu, e_ref = O.rel_l2(y, psi), O.rel_l2(yref, psi)
    say(f"   run diff {d:.2e}; bell-return error gpu {e_gpu:.6f} oracle {e_ref:.6f}")
    assert d <= 1e-9 and abs(e_gpu - e_ref) <= 1e-9


def test_advection_mirror_boundary_parity(R, ctx):
    """Section 6.1 mirror boundary: ghosts copy their mirror sources before
    every right-hand side; rhs at t = 0.7 and the 2000-step bell run against
    the oracle (FP64), 64 x 64 nodes + 804 ghosts."""
    import torch
    from paper_1509_02615_amd import pipeline as P
    say("transport: 64x64 with mirror ghosts, rhs at t=0.7 and the 2000-step RK4 bell run (FP64)")
    cfg = advection_config(64, mirror=True)
    om, idx, W, status = build_advection(cfg)
    nd = cfg["nodes"]
    gm = P.advection_model(ctx, cfg, dev(idx, torch.int32), dev(W, torch.float64))
    psi = cfg["psi0"]
    ref = om(0.7, psi)
    s = dev(psi, torch.float64).reshape(gm.state_shape()).contiguous()
    out = torch.full_like(s, float("nan"))
    R.rbffd_rhs(ctx, gm, 0.7, s, out)
    got = host(out).ravel()
    na = nd.n_active
    assert np.linalg.norm(got - ref) / np.linalg.norm(ref) <= 1e-12 and np.all(got[na:] == 0.0)
    assert np.array_equal(host(s).ravel()[na:], psi[nd.mirror_src])
    yref, _ = O.integrate(om, om.mirror(psi), 0.0, cfg["dt"], 2000, "rk4")
    R.rbffd_step(ctx, gm, s, 0.0, cfg["dt"], 2000, R.RK4)
    y = host(s).ravel()
    d = np.linalg.norm(y[:na] - yref[:na]) / np.linalg.norm(yref[:na])
    e_gpu, e_ref = O.rel_l2(y[:na], psi[:na]), O.rel_l2(yref[:na], psi[:na])
    say(f"   run diff {d:.2e}; bell-return error gpu {e_gpu:.6f} oracle {e_ref:.6f}")
    assert d <= 1e-9 and abs(e_gpu - e_ref) <= 1e-9


@pytest.mark.parametrize("tableau", ["rk4", "wsrk3"])
def test_ns_steps_parity(R, ctx, tableau):
    import torch
    say(f"step: hexagonal 400 m density current, 20 steps {tableau}, FP64 and FP32")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0)
    f = lambda t, y: O.ns_rhs(om, y)[0]                                    # noqa: E731
    yref, _ = O.integrate(f, cfg["state0"], 0.0, cfg["dt"], 20, tableau)
    yref = O.ghost_closure(om, yref)
    na = cfg["nodes"].n_active
    tab = R.RK4 if tableau == "rk4" else R.WSRK3
    for fdt, wdt, dt, tol in ((0, 0, torch.float64, 1e-9), (1, 1, torch.float32, 2e-5)):
        gm = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=fdt, wdt=wdt)
        s = dev(cfg["state0"], dt).reshape(gm.state_shape()).contiguous()
        t = R.rbffd_step(ctx, gm, s, 0.0, cfg["dt"], 20, tab)
        assert abs(t - 20 * cfg["dt"]) < 1e-12
        R.rbffd_ghost(ctx, gm, s)
        got = host(s).reshape(yref.shape)
        errs = rel_fields(got, yref, np.arange(na))
        say(f"   field dtype {fdt}: rel-l2 per field {['%.1e' % e for e in errs]}")
        assert max(errs) <= tol


def test_step_reports_nonfinite(R, ctx):
    import torch
    say("step: a NaN in the state is reported as ENONFINITE")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0)
    gm = gpu_ns(R, ctx, cfg, idx, W, Ww)
    st = cfg["state0"].copy()
    st[500, 2] = np.nan
    s = dev(st, torch.float64).reshape(gm.state_shape()).contiguous()
    with pytest.raises(R.RbffdError) as e:
        R.rbffd_step(ctx, gm, s, 0.0, cfg["dt"], 3, R.RK4)
    assert e.value.code == R.ENONFINITE


def test_full_size_scale_rhs_sampled(R, ctx):
    """2048 x 256 hexagonal channel (524,288 nodes): the whole GPU path
    (search, weights, closure, fused RHS) against the oracle evaluated
    node by node at sampled nodes away from the walls, in FP64, FP32 and
    with BF16 weights, each in the launch shape the tuner picks (as the
    benchmark runs it)."""
    import torch
    from paper_1509_02615_amd import pipeline as P
    say("full size: 2048x256 channel, GPU search+weights+rhs, 160 sampled nodes, FP64 and FP32")
    cfg = scale_config()
    nd = cfg["nodes"]
    xy, idx, W, Ww, (st_a, st_w) = P.ns_weights(ctx, cfg)
    assert int(st_a.abs().sum()) == 0 and int(st_w.abs().sum()) == 0
    state = smooth_ns_state(nd, seed=6).astype(np.float32).astype(np.float64)
    rng = np.random.default_rng(1)
    rows = rng.integers(6 * nd.nx, (nd.nz - 6) * nd.nx, 160)
    ops = [(O.DX, 0, 0), (O.DZ, 0, 0), (O.LAP, 0, 0), (O.HYPERLAP, 3, 7)]
    o_idx = O.knn(nd.xy, rows, 37, nd.period_x)
    o_W, _ = O.all_weights(nd.xy, o_idx, rows, 7, 4, ops, nd.period_x)
    ref = O.ns_tendency(state, rows, o_idx, o_W[0], o_W[1], o_W[2], o_W[3], nd.xy[rows, 1],
                        np.zeros(len(rows), bool), cfg["consts"], cfg["hv_coeff"])
    assert np.array_equal(idx[torch.from_numpy(rows).cuda()].cpu().numpy(), o_idx)
    for fdt, wdt, dt, tol in ((0, 0, torch.float64, 1e-12), (1, 1, torch.float32, 1e-6),
                              (1, 2, torch.float32, 2e-3)):
        gm = P.ns_model(ctx, cfg, idx, W, Ww, xy=xy, field_dtype=fdt, weight_dtype=wdt)
        s = dev(state, dt).reshape(gm.state_shape()).contiguous()
        out = torch.empty_like(s)
        shape, _ = R.rbffd_model_tune(ctx, gm, s)
        R.rbffd_rhs(ctx, gm, 0.0, s, out)
        got = host(out).reshape(-1, 4)[rows]
        errs = [np.linalg.norm(got[:, f] - ref[:, f]) / np.linalg.norm(ref[:, f]) for f in range(4)]
        say(f"   field dtype {fdt}, weight dtype {wdt}, shape {shape}: rel-l2 per field over samples "
            f"{['%.2e' % e for e in errs]}")
        assert max(errs) <= tol


@pytest.mark.parametrize("fdt,wdt", [(0, 0), (1, 1), (1, 2)])
def test_tuned_shape_gives_identical_results(R, ctx, fdt, wdt):
    """rbffd_model_tune only changes the launch shape (block size, slot
    unrolling, load caching), never a thread's arithmetic: results are
    bit-identical before and after tuning."""
    import torch
    say(f"tune: hexagonal 400 m, field dtype {fdt}, weight dtype {wdt}")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0)
    gm = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=fdt, wdt=wdt)
    dt = torch.float64 if fdt == 0 else torch.float32
    s = dev(smooth_ns_state(cfg["nodes"], seed=5), dt).reshape(gm.state_shape()).contiguous()
    o1 = torch.empty_like(s)
    R.rbffd_rhs(ctx, gm, 0.0, s, o1)
    shape, us = R.rbffd_model_tune(ctx, gm, s)
    say(f"   chosen shape {shape}, {us:.1f} us per launch")
    assert 0 <= shape < 6 and us > 0
    o2 = torch.empty_like(s)
    R.rbffd_rhs(ctx, gm, 0.0, s, o2)
    assert torch.equal(o1, o2)
    s1 = s.clone()
    R.rbffd_step(ctx, gm, s1, 0.0, cfg["dt"], 3, R.RK4)     # graph recaptured with the new shape
    assert torch.isfinite(s1).all()


def test_every_forced_shape_and_morton_order_identical(R, ctx):
    """A 64-member model has twelve launch shapes (six shapes, each in row
    order and in Morton order of the coordinates): forcing each one in
    turn gives the same tendency bit for bit, and a shape out of range is
    refused without changing the kept one."""
    import torch
    E = 64
    say(f"tune: every forced stage-kernel shape, E={E} (FP32), hexagonal 400 m")
    cfg, om, idx, W, Ww = ns_case("hexagonal", 400.0)
    gE = gpu_ns(R, ctx, cfg, idx, W, Ww, fdt=1, wdt=1, E=E)
    states = [smooth_ns_state(cfg["nodes"], seed=60 + k).astype(np.float32) for k in range(E)]
    sE = dev(np.stack(states, axis=1), torch.float32).contiguous()
    ref = torch.empty_like(sE)
    R.rbffd_rhs(ctx, gE, 0.0, sE, ref)
    for shape in range(12):
        got, us = R.rbffd_model_tune(ctx, gE, sE, shape)
        assert got == shape and us > 0
        out = torch.empty_like(sE)
        R.rbffd_rhs(ctx, gE, 0.0, sE, out)
        assert torch.equal(out, ref), shape
    for bad in (12, -2):
        with pytest.raises(R.RbffdError):
            R.rbffd_model_tune(ctx, gE, sE, bad)
    out = torch.empty_like(sE)
    R.rbffd_rhs(ctx, gE, 0.0, sE, out)
    assert torch.equal(out, ref)


def test_measurement_helpers(R, ctx):
    """The streaming copy copies; the matrix-core probe rejects a short
    output, writes a finite value per thread and reports its flop count."""
    import torch
    say("measurement helpers: stream copy and matrix-core probe")
    src = torch.arange(1 << 20, dtype=torch.float32, device="cuda")
    dst = torch.empty_like(src)
    R.rbffd_stream_copy(ctx, dst, src)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)
    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    with pytest.raises(R.RbffdError):
        R.rbffd_mfma_probe(ctx, torch.empty(16, dtype=torch.float32, device="cuda"), 1)
    for shape in (0, 1):
        out = torch.full((1024 * n_cu,), float("nan"), dtype=torch.float32, device="cuda")
        flops = R.rbffd_mfma_probe(ctx, out, 10, shape)
        torch.cuda.synchronize()
        assert flops == 4 * n_cu * 4 * 10 * 4 * 2 * 16 * 16 * 32 * (1 if shape == 0 else 2)
        assert bool(torch.isfinite(out).all())


def test_full_size_wall_rows_match_the_oracle(R, ctx):
    """2048 x 256 channel (2 x 2,048 wall rows): the tendency at 288 sampled
    nodes of the three rows next to each wall, whose stencils reach the
    ghosts, against the oracle with its own Section 5.2 ghost solve over
    every boundary row: FP64 1e-12, FP32 1e-6 (FP32-representable inputs),
    BF16 weights 2e-3, rel-l2 per field over the samples.

    The oracle is handed the nodes of the 12 rows nearest each wall and all
    ghosts, renumbered. That is the whole node set for these stencils: the
    test checks that every oracle stencil's 37th neighbour is nearer than
    the nearest node left out, so the stencils, weights and ghost values are
    those of the full channel, and it checks the GPU stencils against them."""
    import torch
    from oracle.pipeline import ns_ops, wall_ops
    from paper_1509_02615_amd import pipeline as P
    say("full size: 2048x256 channel, sampled wall-adjacent rows against the oracle's ghost closure")
    cfg = scale_config()
    nd = cfg["nodes"]
    na, nx, nz, n = nd.n_active, nd.nx, nd.nz, cfg["n"]
    xy, idx, W, Ww, (st_a, st_w) = P.ns_weights(ctx, cfg)
    assert int(st_a.abs().sum()) == 0 and int(st_w.abs().sum()) == 0
    state = smooth_ns_state(nd, seed=8).astype(np.float32).astype(np.float64)
    # the oracle's node set: the rows near the walls, then every ghost
    row_of = np.arange(na) // nx
    near = 12
    sub_active = np.nonzero((row_of < near) | (row_of >= nz - near))[0]
    sub = np.concatenate([sub_active, np.arange(na, nd.n_total)])
    to_sub = np.full(nd.n_total, -1, np.int64)
    to_sub[sub] = np.arange(len(sub))
    oxy = nd.xy[sub]
    assert np.all(nd.bnd_normal == 0)
    bnd, ghosts = to_sub[nd.bnd_nodes], to_sub[nd.bnd_ghosts]
    rng = np.random.default_rng(3)
    samp_full = np.concatenate([r * nx + rng.choice(nx, 48, replace=False) for r in (0, 1, 2, nz - 3, nz - 2, nz - 1)])
    samp = to_sub[samp_full]
    idx_b = O.knn(oxy, bnd, n, nd.period_x)
    idx_s = O.knn(oxy, samp, n, nd.period_x)
    z_lo = nd.xy[:na][row_of == near][:, 1].min()
    z_hi = nd.xy[:na][row_of == nz - near - 1][:, 1].max()
    for centres, st in ((bnd, idx_b), (samp, idx_s)):
        c, nb = oxy[centres], oxy[st]
        dx = nb[:, :, 0] - c[:, None, 0]
        dx -= nd.period_x * np.round(dx / nd.period_x)
        radius = np.sqrt((dx ** 2 + (nb[:, :, 1] - c[:, None, 1]) ** 2).max(axis=1))
        gap = np.minimum(np.abs(z_lo - c[:, 1]), np.abs(c[:, 1] - z_hi))
        assert np.all(radius < 0.9 * gap)
    gpu_idx = host(idx).astype(np.int64)
    assert np.array_equal(to_sub[gpu_idx[samp_full]], idx_s)
    assert np.array_equal(to_sub[gpu_idx[nd.bnd_nodes]], idx_b)
    Wb, st_b = O.all_weights(oxy, idx_b, bnd, cfg["m"], cfg["l"], wall_ops(0), nd.period_x)
    Ws, st_s = O.all_weights(oxy, idx_s, samp, cfg["m"], cfg["l"], ns_ops(cfg), nd.period_x)
    assert st_b.sum() == 0 and st_s.sum() == 0
    rows_idx = np.zeros((len(sub_active), n), np.int64)
    rows_idx[bnd] = idx_b
    walls = O.WallRows(rows_idx, len(sub_active), len(sub), bnd, ghosts, nd.bnd_normal, Wb[0], Wb[1], cfg["consts"])
    closed = O.ghost_closure(walls, state[sub])
    ref = O.ns_tendency(closed, samp, idx_s, Ws[0], Ws[1], Ws[2], Ws[3], oxy[samp, 1], walls.zwall[samp],
                        cfg["consts"], cfg["hv_coeff"])
    for fdt, wdt, dt, tol in ((0, 0, torch.float64, 1e-12), (1, 1, torch.float32, 1e-6),
                              (1, 2, torch.float32, 2e-3)):
        gm = P.ns_model(ctx, cfg, idx, W, Ww, xy=xy, field_dtype=fdt, weight_dtype=wdt)
        s = dev(state, dt).reshape(gm.state_shape()).contiguous()
        out = torch.empty_like(s)
        R.rbffd_rhs(ctx, gm, 0.0, s, out)
        got = host(out).reshape(-1, 4)[samp_full]
        errs = [np.linalg.norm(got[:, f] - ref[:, f]) / np.linalg.norm(ref[:, f]) for f in range(4)]
        say(f"   field dtype {fdt}, weight dtype {wdt}: rel-l2 per field over the wall-adjacent samples "
            f"{['%.2e' % e for e in errs]}")
        assert max(errs) <= tol


def test_full_size_ghost_closure_holds_the_wall_conditions(R, ctx):
    """2048 x 256 channel (2 x 2,048 wall rows): after the ghost closure
    every wall row's own conditions hold to rounding with the model's wall
    weights (Section 5.2: the ghost values are what makes them hold):
    du/dz = dtheta'/dz = 0, dpi'/dz = g theta'_B / (c_p theta_bar (theta_bar +
    theta'_B)), w_B = 0 and d2w/dz2 = 0. A property that holds at any size:
    it checks the windowed W_G^-1 solve on the full walls, FP64 and FP32."""
    import torch
    from paper_1509_02615_amd import pipeline as P
    say("full size: ghost closure on 2 x 2048 wall rows, wall conditions to rounding (FP64, FP32)")
    cfg = scale_config()
    nd = cfg["nodes"]
    c = cfg["consts"]
    xy, idx, W, Ww, _ = P.ns_weights(ctx, cfg)
    n = idx.shape[1]
    rows = nd.bnd_nodes
    assert np.all(nd.bnd_normal == 0)  # channel: both walls normal to z
    I = idx.cpu().numpy()[rows]                           # the wall rows' stencils (ghosts included)
    D = host(Ww).reshape(2, -1, n)                        # Dz and Dzz weights of the wall rows
    base = smooth_ns_state(nd, seed=7)
    for fdt, dt, tol in ((R.F64, torch.float64, 1e-12), (R.F32, torch.float32, 1e-5)):
        gm = P.ns_model(ctx, cfg, idx, W, Ww, xy=xy, field_dtype=fdt, weight_dtype=fdt)
        s = dev(base, dt).reshape(gm.state_shape()).contiguous()
        R.rbffd_ghost(ctx, gm, s)
        y = host(s).reshape(-1, 4).astype(np.float64)
        assert np.all(y[rows, 1] == 0.0)                  # w on the walls
        thb = y[rows, 2]
        bc = c["g"] * thb / (c["c_p"] * c["theta_bar"] * (c["theta_bar"] + thb))
        worst = 0.0
        for f, d, target in ((0, D[0], 0.0), (1, D[1], 0.0), (2, D[0], 0.0), (3, D[0], bc)):
            terms = d * y[I, f]
            r = np.abs(terms.sum(1) - target) / (np.abs(terms).sum(1) + np.abs(target))
            worst = max(worst, float(r.max()))
            assert r.max() <= tol, (fdt, f, float(r.max()))
        say(f"   field dtype {fdt}: worst relative wall-condition residual {worst:.2e}")
        gm.close()


@pytest.mark.parametrize("n", [2, 4, 13, 37])
@pytest.mark.parametrize("na, E", [(61, 1), (321, 3), (321, 16), (21, 64), (700, 70)])
def test_split_slots(R, ctx, na, E, n):
    """Small launches split each node's slots over several wavefronts: every
    remainder of nodes and slots (parts without a slot included), against
    plain FP64 sums over arbitrary stencils and weights, both physics. Bars:
    each sum's rounding, (n + 8) 2^-53 of the summed magnitudes (FP32 fields:
    2^-23, for its weights, differences and products)."""
    import torch
    rng = np.random.default_rng(100 * n + na)
    idx = rng.integers(0, na, (na, n)).astype(np.int32)
    if na % 2:
        idx[:, 0] = np.arange(na)                 # the centre slot left out of the stream, or kept
    W = rng.normal(0, 1, (4, na, n))
    xy = rng.uniform(0, 1, (na, 2))
    c = dict(c_p=1004.0, c_v=717.0, R_d=287.0, g=9.81, theta_bar=300.0, mu=0.7, u_bar=0.3)
    for fdt, dt, eps in ((R.F64, np.float64, 2.0 ** -53), (R.F32, np.float32, 2.0 ** -23)):
        y = rng.normal(0, 1, (na, E, 4)).astype(dt)
        m = R.Model(ctx, R.PHYS_NS, dev(idx, torch.int32), dev(W, torch.float64), dev(xy, torch.float64), na,
                    field_dtype=fdt, weight_dtype=fdt, ensemble=E, hv_coeff=0.4, consts=c)
        s = torch.from_numpy(y).cuda()
        f = torch.empty_like(s)
        R.rbffd_rhs(ctx, m, 0.0, s, f)
        y = y.astype(np.float64)
        d = y[idx] - y[:, None]                                       # [na][n][E][4]
        D = np.einsum("qik,ikef->qief", W, d)
        A = np.einsum("qik,ikef->qief", np.abs(W), np.abs(d)) + np.abs(D)
        u, w, th, pi = [y[..., q] for q in range(4)]
        pib = (1.0 - c["g"] * xy[:, 1] / (c["c_p"] * c["theta_bar"]))[:, None]
        ua, cpt = u + c["u_bar"], c["c_p"] * (c["theta_bar"] + th)
        rcv, dpb = c["R_d"] / c["c_v"], -c["g"] / (c["c_p"] * c["theta_bar"])

        def tend(X, a, sign):
            x, z, lp, hv = X
            r = np.empty_like(y)
            r[..., 0] = sign * (a(ua) * x[..., 0] + a(w) * z[..., 0] + a(cpt) * x[..., 3]) + c["mu"] * lp[..., 0]
            r[..., 1] = (sign * (a(ua) * x[..., 1] + a(w) * z[..., 1] + a(cpt) * z[..., 3])
                         + a(c["g"] * th / c["theta_bar"]) + c["mu"] * lp[..., 1])
            r[..., 2] = sign * (a(ua) * x[..., 2] + a(w) * z[..., 2]) + c["mu"] * lp[..., 2]
            r[..., 3] = sign * (a(ua) * x[..., 3] + a(w) * (a(np.float64(dpb)) + z[..., 3])
                                + a(rcv * (pib + pi)) * (x[..., 0] + z[..., 1]))
            return r + 0.4 * hv
        want, mag = tend(D, lambda v: v, -1.0), tend(A, np.abs, 1.0)
        err = np.abs(host(f) - want)
        say(f"split slots: NS na {na}, E {E}, n {n}, {dt.__name__}: {(err / np.maximum(mag, 1e-300)).max() / eps:.2f} eps")
        assert np.all(err <= (n + 8) * eps * mag)
        U, V = rng.normal(0, 1, (2, na))
        psi = rng.normal(0, 1, (na, E, 1)).astype(dt)
        m = R.Model(ctx, R.PHYS_ADVECTION, dev(idx, torch.int32), dev(W[:3], torch.float64), dev(xy, torch.float64), na,
                    field_dtype=fdt, ensemble=E, hv_coeff=0.4, vel_u=dev(U, torch.float64), vel_v=dev(V, torch.float64),
                    vel_period=5.0)
        s = torch.from_numpy(psi).cuda()
        f = torch.empty_like(s)
        R.rbffd_rhs(ctx, m, 0.25, s, f)
        adv = W[0] * U[idx] + W[1] * V[idx]
        g = psi.astype(np.float64)[idx][..., 0]
        cs = np.cos(np.pi * 0.25 / 5.0)
        want = -cs * np.einsum("ik,ike->ie", adv, g) + 0.4 * np.einsum("ik,ike->ie", W[2], g)
        mag = (np.einsum("ik,ike->ie", np.abs(W[0] * U[idx]) + np.abs(W[1] * V[idx]), np.abs(g))
               + 0.4 * np.einsum("ik,ike->ie", np.abs(W[2]), np.abs(g)))
        err = np.abs(host(f)[..., 0] - want)
        say(f"   transport: {(err / np.maximum(mag, 1e-300)).max() / eps:.2f} eps")
        assert np.all(err <= (n + 8) * eps * mag)


CONSTS = dict(c_p=1004.0, c_v=717.0, R_d=287.0, g=9.81, theta_bar=300.0, mu=0.7, u_bar=0.3)
NS_TYPES = {"f64": (0, 0), "f32": (1, 1), "bf16": (1, 2)}


def _random_ns(R, ctx, kind, na, E, n, seed=0):
    """A model of arbitrary stencils and weights without walls (the centre in
    slot 0 of every stencil, so that it is left out of the stream), its state,
    stencils, weights and nodes, all on the device."""
    import torch
    fdt, wdt = NS_TYPES[kind]
    g = torch.Generator(device="cuda")
    g.manual_seed(1000 * n + seed)
    idx = torch.randint(0, na, (na, n), generator=g, device="cuda", dtype=torch.int32)
    idx[:, 0] = torch.arange(na, device="cuda", dtype=torch.int32)
    W = torch.randn((4, na, n), generator=g, device="cuda", dtype=torch.float64)
    xy = torch.rand((na, 2), generator=g, device="cuda", dtype=torch.float64)
    y = torch.randn((na, E, 4), generator=g, device="cuda", dtype=torch.float64 if fdt == 0 else torch.float32)
    m = R.Model(ctx, R.PHYS_NS, idx, W, xy, na, field_dtype=fdt, weight_dtype=wdt, ensemble=E, hv_coeff=0.4,
                consts=CONSTS)
    return m, y, idx.long(), W, xy


def _tendency64(y, idx, W, xy):
    """The Navier-Stokes tendency of _random_ns in FP64, and the magnitude of
    what it sums."""
    import torch
    c, y = CONSTS, y.double()
    d = y[idx] - y[:, None]                                            # [na][n][E][4]
    D = [(w[:, :, None, None] * d).sum(1) for w in W]
    A = [(w.abs()[:, :, None, None] * d.abs()).sum(1) + x.abs() for w, x in zip(W, D)]
    u, w, th, pi = y.unbind(-1)
    pib = (1.0 - c["g"] * xy[:, 1] / (c["c_p"] * c["theta_bar"]))[:, None]
    ua, cpt = u + c["u_bar"], c["c_p"] * (c["theta_bar"] + th)
    rcv, dpb = c["R_d"] / c["c_v"], -c["g"] / (c["c_p"] * c["theta_bar"])

    def tend(X, a, s):
        x, z, lp, hv = X
        r = torch.stack([s * (a(ua) * x[..., 0] + a(w) * z[..., 0] + a(cpt) * x[..., 3]) + c["mu"] * lp[..., 0],
                         s * (a(ua) * x[..., 1] + a(w) * z[..., 1] + a(cpt) * z[..., 3])
                         + a(c["g"] * th / c["theta_bar"]) + c["mu"] * lp[..., 1],
                         s * (a(ua) * x[..., 2] + a(w) * z[..., 2]) + c["mu"] * lp[..., 2],
                         s * (a(ua) * x[..., 3] + a(w) * (abs(dpb) if s > 0 else dpb) + a(w) * z[..., 3]
                              + a(rcv * (pib + pi)) * (x[..., 0] + z[..., 1]))], -1)
        return r + 0.4 * hv
    return tend(D, lambda v: v, -1.0), tend(A, torch.abs, 1.0)


def _rhs(R, ctx, m, y):
    import torch
    f = torch.empty_like(y)
    R.rbffd_rhs(ctx, m, 0.25, y.clone(), f)
    return f


def _random_transport(R, ctx, na, E, n, ng=0, fdt=0):
    """A transport model of arbitrary stencils and weights (and ng mirror
    ghosts), its state and, for the reference, stencils, the folded velocity
    weights, the Lap^k weights and the ghosts' sources."""
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(7 * n + na)
    idx = torch.randint(0, na + ng, (na, n), generator=g, device="cuda", dtype=torch.int32)
    W = torch.randn((3, na, n), generator=g, device="cuda", dtype=torch.float64)
    xy = torch.rand((na + ng, 2), generator=g, device="cuda", dtype=torch.float64)
    U, V = torch.randn((2, na + ng), generator=g, device="cuda", dtype=torch.float64)
    src = torch.randint(0, na, (ng,), generator=g, device="cuda", dtype=torch.int32)
    y = torch.randn((na + ng, E, 1), generator=g, device="cuda", dtype=torch.float64 if fdt == 0 else torch.float32)
    m = R.Model(ctx, R.PHYS_ADVECTION, idx, W, xy, na, field_dtype=fdt, ensemble=E, hv_coeff=0.4, vel_u=U.contiguous(),
                vel_v=V.contiguous(), vel_period=5.0, mirror_src=src if ng else None)
    j = idx.long()
    return m, y, j, W[0] * U[j] + W[1] * V[j], W[2], src.long()


@pytest.mark.parametrize("kind", ["f64", "f32", "bf16"])
def test_members_of_full_launches_are_not_split(R, ctx, kind):
    """Whether slots are split goes by all units of a launch, members included:
    15 members of 30,000 nodes fill the chip as 16 do, and each member has the
    same bits in both (fewer than 16 members went by their nodes alone, and a
    chip full of split units takes up to a third longer). Transport as well."""
    import torch
    na, n = 30000, 13
    m16, y, *_ = _random_ns(R, ctx, kind, na, 16, n)
    f16 = _rhs(R, ctx, m16, y)
    m15, _, *_ = _random_ns(R, ctx, kind, na, 15, n)
    f15 = _rhs(R, ctx, m15, y[:, :15].contiguous())
    assert torch.equal(f15, f16[:, :15])
    fdt = NS_TYPES[kind][0]
    m16, y, *_ = _random_transport(R, ctx, na, 16, n, fdt=fdt)
    f16 = _rhs(R, ctx, m16, y)
    m15, _, *_ = _random_transport(R, ctx, na, 15, n, fdt=fdt)
    assert torch.equal(_rhs(R, ctx, m15, y[:, :15].contiguous()), f16[:, :15])


@pytest.mark.parametrize("kind, E, units", [
    ("f64", 1, 3583), ("f64", 1, 3584), ("f64", 3, 5120), ("f64", 3, 5121), ("f64", 3, 6912), ("f64", 3, 6913),
    ("f32", 1, 5734), ("f32", 1, 5735), ("f32", 5, 8192), ("f32", 5, 8193), ("f32", 5, 11059), ("f32", 5, 11060),
    ("bf16", 1, 5734), ("bf16", 1, 5735), ("bf16", 2, 8193), ("bf16", 17, 8193),
    ("f64", 64, 3583), ("f64", 64, 3584), ("f32", 64, 2943), ("f32", 64, 2944), ("bf16", 64, 4095), ("bf16", 64, 4096)])
def test_split_limits(R, ctx, kind, E, units):
    """Launches just below and just above each limit of slot splitting, with
    FP64, FP32 and BF16 weights and members in lanes or by wavefront, against
    plain FP64 sums. Bars: each sum's rounding, (n + 8) 2^-53 of the summed
    magnitudes (FP32 fields: 2^-23), and BF16 weights' own 2^-16."""
    n = 9
    na = (64 * units - 63) // E + 1 if E < 64 else units              # the last unit holds a few pairs
    assert (na * E + 63) // 64 == units
    m, y, idx, W, xy = _random_ns(R, ctx, kind, na, E, n, units)
    want, mag = _tendency64(y, idx, W, xy)
    got = _rhs(R, ctx, m, y).double()
    bar = (n + 8) * 2.0 ** (-53 if kind == "f64" else -23) + (2.0 ** -16 if kind == "bf16" else 0.0)
    worst = float(((got - want).abs() / mag).max())
    say(f"split limits: {kind}, E {E}, {units} units ({na} nodes): {worst / bar:.3f} of the bar")
    assert worst <= bar


@pytest.mark.parametrize("kind, E", [("f64", 1), ("f32", 1), ("bf16", 1), ("f64", 64), ("f32", 64), ("bf16", 64)])
def test_forced_shapes_of_full_launches_identical(R, ctx, kind, E):
    """Every launch shape of the unsplit stage kernels (for 64 members in row
    and in Morton order) gives the same tendency bit for bit, and the tuner
    keeps one of them."""
    import torch
    na = 64 * 5800 - 9 if E == 1 else 4200
    m, y, *_ = _random_ns(R, ctx, kind, na, E, 9)
    ref = _rhs(R, ctx, m, y)
    for shape in range(12 if E == 64 else 6):
        got, us = R.rbffd_model_tune(ctx, m, y.clone(), shape)
        assert got == shape and us > 0
        assert torch.equal(_rhs(R, ctx, m, y), ref), shape
    R.rbffd_model_tune(ctx, m, y.clone())
    assert torch.equal(_rhs(R, ctx, m, y), ref)


@pytest.mark.parametrize("E, units", [(1, 767), (1, 768), (15, 767), (15, 768), (3, 2310)])
def test_transport_split_limit(R, ctx, E, units):
    """Transport right-hand sides and RK4 steps with mirror ghosts just below
    and above the limit of slot splitting, against plain FP64 sums (13 slots).
    Bars: (n + 8) 2^-53 of the summed magnitudes for one right-hand side; three
    steps sum 12 of them, each in a state a few 2^-53 off, at |dt f| << |y|:
    1e-13 relative l2."""
    import torch
    n, ng = 13, 500
    na = (64 * units - 63) // E + 1
    m, y, idx, adv, hv, src = _random_transport(R, ctx, na, E, n, ng)

    def f(t, v, mag=False):
        v = torch.cat([v, v[src]])[idx]                                # [na][n][E]
        a = torch.abs if mag else (lambda x: x)
        cs = np.cos(np.pi * t / 5.0)
        return (-a(torch.tensor(cs)) * (-1.0 if mag else 1.0) * (a(adv)[..., None] * a(v)).sum(1)
                + 0.4 * (a(hv)[..., None] * a(v)).sum(1))
    v0 = y[:na, :, 0].clone()
    got = _rhs(R, ctx, m, y)[..., 0]
    err, mag = (got[:na] - f(0.25, v0)).abs(), f(0.25, v0, True)
    say(f"transport split limit: E {E}, {units} units: {float((err / mag).max()) * 2.0 ** 53:.2f} eps")
    assert bool((err <= (n + 8) * 2.0 ** -53 * mag).all()) and bool((got[na:] == 0.0).all())
    dt, v = 1e-3, v0
    s = y.clone()
    R.rbffd_step(ctx, m, s, 0.1, dt, 3, R.RK4)
    for k in range(3):
        t = 0.1 + k * dt
        k1 = f(t, v)
        k2 = f(t + dt / 2, v + dt / 2 * k1)
        k3 = f(t + dt / 2, v + dt / 2 * k2)
        v = v + dt / 6 * (k1 + 2 * k2 + 2 * k3 + f(t + dt, v + dt * k3))
    off = float(torch.linalg.norm(s[:na, :, 0] - v) / torch.linalg.norm(v))
    say(f"   three RK4 steps: {off:.1e}")
    assert off <= 1e-13
    assert torch.equal(s[na:, :, 0], s[src, :, 0])


@pytest.mark.parametrize("kind, E", [("f64", 1), ("f32", 1), ("bf16", 3), ("f32", 64)])
def test_tuner_names_a_split_launch_once(R, ctx, kind, E):
    """Split launches have no block size, so shapes 0, 3 and 4 are one launch, and
    1 and 2: the tuner times each launch once and returns the first shape of its
    kind; every shape can still be forced."""
    m, y, *_ = _random_ns(R, ctx, kind, 900, E, 9)
    for _ in range(12):
        shape, us = R.rbffd_model_tune(ctx, m, y)
        assert shape % 6 in (0, 1, 5) and us > 0
    for shape in range(6):
        assert R.rbffd_model_tune(ctx, m, y, shape)[0] == shape
