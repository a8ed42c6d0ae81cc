"""GPU parity of the step with the SI's network (Q -> 300 -> 300 -> 100 -> Q,
LeakyReLU) against the FP64 oracle, through the C ABI: float32 over several
steps on small grids with ragged rows, bf16 / fp16 against the oracle's
emulated rounding, and one step at the 3-D throughput size (D3Q19 256^3) and
at a size where work items wrap over several rows per wavefront, on sampled
nodes the oracle computes one by one."""
import numpy as np
import pytest

import oracle
from lbm_cases import (plain_rounding_config, kernel_emulation, lib_config, random_state, rel_l2, to_canonical,
                       to_shifted)
from paper_2403_18466_amd import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def lbm():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2403_18466_amd import lbm as m
    m.load_library()
    return m


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.float32)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.detach().cpu().numpy().astype(np.float64)


def wide_params(Q, seed, scale=0.05):
    return inputs.random_params_net(inputs.net_widths(Q, 0, "paper"), seed, scale=scale)


def run_gpu(lbm, ocfg, g0, theta, nsteps, prec="fp32"):
    L = lbm.Lattice(lib_config(ocfg, prec))
    assert L.n_param == ocfg.n_params
    A = dev(to_shifted(g0, ocfg.lattice))
    out = L.step(A, dev(theta), nsteps)
    res = to_canonical(host(out), ocfg.lattice)
    L.close()
    return res


@pytest.mark.parametrize("lat,shape,batch,force,nsteps", [
    ("D2Q9", (1, 20, 70), 2, 0, 4),
    ("D2Q9", (1, 9, 130), 1, 1, 4),
    ("D3Q19", (5, 6, 70), 2, 0, 2),
    ("D3Q19", (4, 5, 9), 1, 2, 3),
])
def test_wide_fp32_parity(lbm, lat, shape, batch, force, nsteps):
    nz, ny, nx = shape
    kw = {}
    if force == 1:
        kw = dict(force_kind=1, force_amp=1e-4, force_k=1)
    elif force == 2:
        kw = dict(force_kind=2, force_amp=5e-5, force_k=1)
    ocfg = oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=batch, tau=0.55, hidden=300,
                         net="paper", out_scale=0.25, **kw)
    theta = wide_params(ocfg.Q, seed=50)
    g0 = random_state(ocfg, 51, scale=0.03)
    want = oracle.run(ocfg, g0, theta.astype(np.float64), nsteps)
    got = run_gpu(lbm, ocfg, g0, theta, nsteps)
    bgk = oracle.run(oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=batch, tau=0.55, **kw),
                     g0, None, nsteps)
    err = rel_l2(got, want)
    net_effect = rel_l2(bgk, want)
    print(f"{lat} {shape} x{batch} force {force}: rel L2 {err:.2e} after {nsteps} steps "
          f"(the network changes the state by {net_effect:.2e})")
    assert net_effect > 1e-3
    assert err < 1e-5
    # mass and momentum totals are conserved by the collision and by streaming
    c = np.array(oracle.tables(lat)[0], np.float64)
    one = run_gpu(lbm, ocfg, g0, theta, 1)
    d = one - g0
    assert abs(d.sum()) < 1e-6 * np.abs(g0).sum()
    if force == 0:
        assert np.abs(np.einsum("bqzyx,qa->a", d, c)).max() < 1e-6 * np.abs(g0).sum()


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("lat,shape", [("D2Q9", (1, 40, 70)), ("D3Q19", (4, 6, 20))])
def test_wide_reduced_precision(lbm, prec, lat, shape):
    """One step with 16-bit operands against the oracle's emulated rounding;
    the same criterion as for the small network: the L2 gap is a small
    fraction of the rounding effect itself, and the largest deviation is
    bounded relative to the largest update."""
    nz, ny, nx = shape
    base = dict(lattice=lat, nx=nx, ny=ny, nz=nz, batch=1, tau=0.51, hidden=300, net="paper",
                out_scale=0.5)
    ocfg_x = oracle.Config(**base)
    theta = inputs.glorot_params_net(inputs.net_widths(ocfg_x.Q, 0, "paper"), seed=1)
    g0 = random_state(ocfg_x, 52, scale=0.05)
    got = run_gpu(lbm, ocfg_x, g0, theta, 1, prec=prec)
    kcfg, kth = kernel_emulation(ocfg_x, theta, prec)
    emu = oracle.step(kcfg, g0, kth)
    plain = oracle.step(plain_rounding_config(ocfg_x, prec), g0, theta.astype(np.float64))
    exact = oracle.step(ocfg_x, g0, theta.astype(np.float64))
    upd = np.abs(exact - g0).max()
    l2_emu = np.linalg.norm(got - emu)
    l2_round = np.linalg.norm(emu - exact)
    vs_exact = np.linalg.norm(got - exact) / np.linalg.norm(plain - exact)
    max_emu = np.abs(got - emu).max() / upd
    max_exact = np.abs(got - exact).max() / upd
    print(f"{prec} {lat}: L2 |gpu-emulated| / L2 |emulated-fp64| = {l2_emu / l2_round:.3f}; "
          f"L2 |gpu-fp64| / L2 |plain-fp64| = {vs_exact:.3f}; "
          f"max |gpu-emulated| {max_emu:.2e}, max |gpu-fp64| {max_exact:.2e} of max |update|")
    assert l2_emu < 0.25 * l2_round
    assert vs_exact < 1.5
    assert max_emu < (2e-3 if prec == "bf16" else 5e-4)
    assert max_exact < (1e-2 if prec == "bf16" else 2e-3)


def _sampled_case(lat, n):
    """(oracle config, canonical float32 state, pull-shifted state, points)."""
    if lat == "D3Q19":
        nx = ny = nz = n
        ocfg = oracle.Config(lattice="D3Q19", nx=n, ny=n, nz=n, tau=0.51, hidden=300, net="paper",
                             out_scale=2.0 ** -6)
        u = inputs.solenoidal_spectrum_velocity((n, n, n), 4.0, 0.04, seed=0)
        g = oracle.init_equilibrium(ocfg, np.ones((1, n, n, n)), u[None])
    else:
        nx, ny, nz = n, 96, 1
        ocfg = oracle.Config(nx=nx, ny=ny, tau=0.51, hidden=300, net="paper", out_scale=2.0 ** -6)
        u = inputs.fourier_modes_velocity(nx, ny, kmax=4, umax=0.05, seed=0)
        g = oracle.init_equilibrium(ocfg, np.ones((1, 1, ny, nx)), u[None, :, None])
    del u
    g32 = g.astype(np.float32)
    del g
    c = np.array(oracle.tables(lat)[0])
    A = np.empty_like(g32)
    for q in range(ocfg.Q):
        A[0, q] = np.roll(g32[0, q], shift=(-c[q, 2], -c[q, 1], -c[q, 0]), axis=(0, 1, 2))
    rng = np.random.default_rng(53)
    pts = [(0, 0, 0), (nz - 1, ny - 1, nx - 1), (0, ny - 1, 63), (nz - 1, 0, 64)]
    pts += [tuple(p) for p in rng.integers(0, [nz, ny, nx], size=(28, 3))]
    return ocfg, g32, A, pts


@pytest.mark.parametrize("lat,n", [("D3Q19", 256), ("D2Q9", 2048)])
def test_wide_one_step_sampled(lbm, lat, n):
    """D3Q19 256^3 is the 3-D throughput workload (solenoidal field with
    E(k) ~ k^4 exp(-2 (k/4)^2), u_rms 0.04, tau 0.51, s_out 2^-6, Glorot
    weights, bf16); D2Q9 2048 x 96 makes every wavefront walk two work items
    (the second one past the end for some), which small grids never do."""
    ocfg, g32, A, pts = _sampled_case(lat, n)
    Q = ocfg.Q
    theta = inputs.glorot_params_net(inputs.net_widths(Q, 0, "paper"), seed=1)
    L = lbm.Lattice(lib_config(ocfg, "bf16"))
    out = L.step(torch.from_numpy(A).cuda(), torch.from_numpy(theta).cuda(), 1)
    _, _, diag = L.moments(out, want_fields=False)
    torch.cuda.synchronize()
    assert int(diag[0, 2].item()) == 0
    c = np.array(oracle.tables(lat)[0], np.float64)
    tot_in = A.astype(np.float64).sum(axis=(0, 2, 3, 4))
    tot_out = out.double().sum(dim=(0, 2, 3, 4)).cpu().numpy()
    assert abs(tot_out.sum() - tot_in.sum()) < 1e-6 * np.abs(A).sum()
    assert np.abs(c.T @ (tot_out - tot_in)).max() < 1e-6 * np.abs(A).sum()
    del A
    zs, ys, xs = (np.array([p[i] for p in pts]) for i in range(3))
    got = out[0].cpu().numpy()[:, zs, ys, xs].astype(np.float64)
    kw = dict(lattice=lat, nx=1, ny=1, nz=1, tau=0.51, hidden=300, net="paper", out_scale=2.0 ** -6)
    one_x = oracle.Config(**kw)
    one_q, kth = kernel_emulation(one_x, theta, "bf16")
    th64 = theta.astype(np.float64)
    want, exact, pre = [], [], []
    for z, y, x in pts:
        gg = g32[0, :, z, y, x].astype(np.float64).reshape(1, Q, 1, 1, 1)
        want.append(oracle.collide(one_q, gg, kth)[0, :, 0, 0, 0])
        exact.append(oracle.collide(one_x, gg, th64)[0, :, 0, 0, 0])
        pre.append(gg[0, :, 0, 0, 0])
    want, exact, pre = np.array(want).T, np.array(exact).T, np.array(pre).T
    e_upd = np.linalg.norm(got - want) / np.linalg.norm(exact - pre)
    gap = np.linalg.norm(want - exact) / np.linalg.norm(exact - pre)
    e_state = np.linalg.norm(got - want) / np.linalg.norm(want)
    print(f"{lat} n={n} bf16: state rel L2 {e_state:.2e}; |gpu - emulated| / |update| {e_upd:.2e}; "
          f"emulated rounding / |update| {gap:.2e}")
    assert e_state < 1e-4 and e_upd < 0.5 * gap
    L.close()


def gpu_adjoint(lbm, ocfg, g, lam1, theta, prec="fp32"):
    L = lbm.Lattice(lib_config(ocfg, prec))
    lam0, dth = L.step_backward(dev(to_shifted(g, ocfg.lattice)), dev(theta),
                                dev(to_shifted(lam1, ocfg.lattice)))
    out = to_canonical(host(lam0), ocfg.lattice), host(dth)
    L.close()
    return out


def _blocks(Q):
    """Offsets of the eight parameter blocks [W1 b1 W2 b2 W3 b3 W4 b4]."""
    o, offs = 0, [0]
    for nin, nout in ((Q, 300), (300, 300), (300, 100), (100, Q)):
        o += nin * nout
        offs.append(o)
        o += nout
        offs.append(o)
    return offs


@pytest.mark.parametrize("lat,shape,batch,force", [
    ("D2Q9", (1, 9, 20), 2, 0),
    ("D2Q9", (1, 16, 70), 1, 1),
    ("D3Q19", (4, 5, 6), 2, 0),
    ("D3Q19", (5, 5, 5), 1, 2),
])
def test_wide_adjoint_fp32_parity(lbm, lat, shape, batch, force):
    """lam^n and dtheta of one step against the oracle's reverse pass, every
    parameter block separately (the node count is not a multiple of the
    64-row tiles, so padded rows are exercised too)."""
    nz, ny, nx = shape
    kw = {1: dict(force_kind=1, force_amp=1e-3, force_k=1),
          2: dict(force_kind=2, force_amp=1e-3, force_k=1)}.get(force, {})
    ocfg = oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=batch, tau=0.55, hidden=300,
                         net="paper", out_scale=0.25, **kw)
    theta = wide_params(ocfg.Q, seed=54)
    g = random_state(ocfg, 55, scale=0.03)
    lam1 = random_state(ocfg, 56, scale=1.0)
    want, wdth = oracle.step_adjoint(ocfg, g, lam1, theta.astype(np.float64))
    got, gdth = gpu_adjoint(lbm, ocfg, g, lam1, theta)
    e_lam, e_th = rel_l2(got, want), rel_l2(gdth, wdth)
    print(f"{lat} {shape} x{batch} force {force}: lam rel L2 {e_lam:.2e}, dtheta rel L2 {e_th:.2e}")
    assert e_lam < 1e-5 and e_th < 1e-5
    offs = _blocks(ocfg.Q)
    for a, b in zip(offs[:-1], offs[1:]):
        assert np.abs(wdth[a:b]).max() > 0
        assert rel_l2(gdth[a:b], wdth[a:b]) < 1e-4, (a, b)


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_wide_adjoint_reduced_precision(lbm, prec):
    """16-bit operands against the oracle's emulated-rounding adjoint; the
    GPU also rounds its backward operands (dY, dZ), so the bounds are
    stated, as for the small network."""
    ocfg = oracle.Config(lattice="D3Q19", nx=9, ny=6, nz=5, batch=1, tau=0.51, hidden=300,
                         net="paper", out_scale=0.25)
    theta = inputs.glorot_params_net(inputs.net_widths(19, 0, "paper"), seed=1)
    g = random_state(ocfg, 57, scale=0.03)
    lam1 = random_state(ocfg, 58, scale=1.0)
    kcfg, kth = kernel_emulation(ocfg, theta, prec)
    want, wdth = oracle.step_adjoint(kcfg, g, lam1, kth)
    got, gdth = gpu_adjoint(lbm, ocfg, g, lam1, theta, prec=prec)
    e_lam, e_th = rel_l2(got, want), rel_l2(gdth, wdth)
    print(f"{prec}: lam rel L2 {e_lam:.2e}, dtheta rel L2 {e_th:.2e}")
    assert e_lam < (2e-3 if prec == "bf16" else 3e-4)
    assert e_th < (2e-2 if prec == "bf16" else 3e-3)


def test_wide_adjoint_4335_nodes(lbm):
    """bf16 adjoint on 4335 nodes (68 node tiles of 64 in the products, the
    last one ragged) against the oracle's emulated-rounding adjoint, every
    parameter block on its own."""
    ocfg = oracle.Config(lattice="D3Q19", nx=17, ny=17, nz=15, batch=1, tau=0.51, hidden=300,
                         net="paper", out_scale=0.25)
    theta = inputs.glorot_params_net(inputs.net_widths(19, 0, "paper"), seed=1)
    g = random_state(ocfg, 57, scale=0.03)
    lam1 = random_state(ocfg, 58, scale=1.0)
    kcfg, kth = kernel_emulation(ocfg, theta, "bf16")
    want, wdth = oracle.step_adjoint(kcfg, g, lam1, kth)
    got, gdth = gpu_adjoint(lbm, ocfg, g, lam1, theta, prec="bf16")
    e_lam, e_th = rel_l2(got, want), rel_l2(gdth, wdth)
    offs = _blocks(ocfg.Q)
    errs = [rel_l2(gdth[a:b], wdth[a:b]) for a, b in zip(offs[:-1], offs[1:])]
    print(f"4335 nodes: lam rel L2 {e_lam:.2e}, dtheta rel L2 {e_th:.2e}, blocks " +
          " ".join(f"{e:.1e}" for e in errs))
    assert e_lam < 2e-3
    assert e_th < 2e-2
    for e in errs:
        assert e < 5e-2


def test_wide_unrolled_gradient(lbm):
    """6 unrolled steps of the SI's network on D3Q19 (forced), fp32, the
    population loss on a node subset: the parameter gradient against the
    oracle's reverse pass through all steps."""
    from paper_2403_18466_amd import training
    ocfg = oracle.Config(lattice="D3Q19", nx=7, ny=6, nz=5, batch=1, tau=0.55, hidden=300,
                         net="paper", out_scale=0.25, force_kind=2, force_amp=5e-5, force_k=1)
    theta = wide_params(19, seed=59)
    g0, gt = random_state(ocfg, 60, 0.02), random_state(ocfg, 61, 0.02)
    nodes = np.random.default_rng(62).choice(210, size=50, replace=False).astype(np.int32)
    wl, wth, _ = oracle.unrolled_loss_and_grad(
        ocfg, g0, theta.astype(np.float64), None, 6, 3,
        loss_fn=lambda g: oracle.loss_population_sse(ocfg, g, gt, nodes))
    L = lbm.Lattice(lib_config(ocfg))
    nd = torch.from_numpy(nodes).cuda()
    T = dev(to_shifted(gt, "D3Q19"))
    loss, dth, _ = training.unrolled_loss_and_grad(
        L, dev(to_shifted(g0, "D3Q19")), dev(theta), None, 6, 3,
        loss_fn=lambda A: L.loss_population_sse(A, T, nd))
    err = rel_l2(host(dth), wth)
    print(f"wide network, 6 unrolled steps: loss {loss.item():.6e} vs {wl:.6e}, dtheta rel L2 {err:.2e}")
    assert abs(loss.item() - wl) <= 1e-5 * wl
    assert err < 1e-5
    L.close()


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("lat,shape,batch,force", [
    ("D2Q9", (1, 3, 5), 1, 0),      # less than one 16-node tile
    ("D2Q9", (1, 8, 8), 1, 1),      # exactly one workgroup of 64 nodes
    ("D3Q19", (5, 13, 1), 1, 0),    # one node more (65), a dimension of 1
    ("D3Q19", (3, 7, 31), 2, 2),    # 1302 nodes: several node ranges, fewer than 8
    ("D3Q19", (15, 17, 17), 1, 0),  # 4335 nodes: eight ranges and more
])
def test_wide_adjoint_16bit_edges(lbm, lat, shape, batch, force, prec):
    """The 16-bit adjoint where its node tiles, workgroups and node ranges
    end, against the oracle's emulated-rounding adjoint.  The GPU also rounds
    dY and dZ1-dZ3 to the operand format (relative 2^-9 / 2^-12 each): bars of
    ten such roundings for dtheta, a tenth of that for lam, whose network part
    carries the factor s_out."""
    nz, ny, nx = shape
    kw = {1: dict(force_kind=1, force_amp=1e-3, force_k=1),
          2: dict(force_kind=2, force_amp=1e-3, force_k=1)}.get(force, {})
    ocfg = oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=batch, tau=0.55, hidden=300,
                         net="paper", out_scale=0.25, **kw)
    theta = inputs.glorot_params_net(inputs.net_widths(ocfg.Q, 0, "paper"), seed=7)
    g = random_state(ocfg, 71, scale=0.03)
    lam1 = random_state(ocfg, 72, scale=1.0)
    kcfg, kth = kernel_emulation(ocfg, theta, prec)
    want, wdth = oracle.step_adjoint(kcfg, g, lam1, kth)
    got, gdth = gpu_adjoint(lbm, ocfg, g, lam1, theta, prec=prec)
    e_lam, e_th = rel_l2(got, want), rel_l2(gdth, wdth)
    print(f"{lat} {shape} x{batch} {prec}: lam rel L2 {e_lam:.2e}, dtheta rel L2 {e_th:.2e}")
    assert e_lam < (2e-3 if prec == "bf16" else 3e-4)
    assert e_th < (2e-2 if prec == "bf16" else 3e-3)


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_wide_adjoint_16bit_beyond_cache(lbm, prec):
    """A batch whose records exceed the last-level cache (non-temporal
    accesses, 64 node ranges) against its fields one by one (within it, 32
    ranges): lam node by node the same bits; dtheta the same sums in another
    order, some 100 float32 roundings of 2^-24 in quadrature (6e-7), bar 1e-5."""
    cfg = dict(lattice="D2Q9", nx=157, ny=160, nz=1, tau=0.55, hidden=300, net="paper",
               out_scale=0.25)
    ocfg, one = oracle.Config(batch=3, **cfg), oracle.Config(batch=1, **cfg)
    theta = inputs.glorot_params_net(inputs.net_widths(9, 0, "paper"), seed=7)
    g = random_state(ocfg, 73, scale=0.03)
    lam1 = random_state(ocfg, 74, scale=1.0)
    got, gdth = gpu_adjoint(lbm, ocfg, g, lam1, theta, prec=prec)
    sums = np.zeros_like(gdth)
    for b in range(3):
        lam, dth = gpu_adjoint(lbm, one, g[b:b + 1], lam1[b:b + 1], theta, prec=prec)
        np.testing.assert_array_equal(got[b:b + 1], lam)
        sums += dth
    assert rel_l2(gdth, sums) < 1e-5


def test_wide_adjoint_16bit_at_rest(lbm):
    """A fluid at rest and zero biases: every pre-activation is exactly 0, where
    the derivative is the slope, so b3's gradient is slope W4^T dY and the
    weight gradients vanish."""
    ocfg = oracle.Config(lattice="D3Q19", nx=6, ny=5, nz=4, batch=1, tau=0.55, hidden=300,
                         net="paper", out_scale=0.25)
    theta = inputs.glorot_params_net(inputs.net_widths(19, 0, "paper"), seed=7)
    g = random_state(ocfg, 73) * 0.0
    lam1 = random_state(ocfg, 74, scale=1.0)
    want, wdth = oracle.step_adjoint(ocfg, g, lam1, theta.astype(np.float64))
    got, gdth = gpu_adjoint(lbm, ocfg, g, lam1, theta, prec="bf16")
    offs = _blocks(19)
    b3, w4 = slice(offs[5], offs[6]), slice(offs[6], offs[7])
    assert np.abs(wdth[b3]).max() > 0 and np.abs(wdth[w4]).max() == 0
    assert rel_l2(gdth[b3], wdth[b3]) < 2e-2
    assert np.abs(gdth[w4]).max() == 0
    assert rel_l2(got, want) < 2e-3


def test_wide_adjoint_sequence_packs_theta(lbm):
    """A sequence packs theta once for all its steps; a later call with other
    parameters uses those.  lam equals the step-by-step result bit for bit."""
    ocfg = oracle.Config(lattice="D3Q19", nx=7, ny=6, nz=5, batch=1, tau=0.55, hidden=300,
                         net="paper", out_scale=0.25)
    L = lbm.Lattice(lib_config(ocfg, "bf16"))
    states = [dev(to_shifted(random_state(ocfg, 80 + k), "D3Q19")) for k in range(3)]
    lam = dev(to_shifted(random_state(ocfg, 90, scale=1.0), "D3Q19"))
    for seed in (1, 2):
        th = dev(inputs.glorot_params_net(inputs.net_widths(19, 0, "paper"), seed=seed))
        a, b = lam.clone(), torch.empty_like(lam)
        d = torch.zeros(L.n_param, dtype=torch.float32, device="cuda")
        res = lbm.lbm_step_backward_seq(L.ctx, L.cfg, states, th, a, b, d, L.workspace())
        l, e = lam, torch.zeros_like(d)
        for s in reversed(states):
            l, e = L.step_backward(s, th, l, dtheta=e)
        assert torch.equal(res, l)
        assert torch.equal(d, e)
    L.close()


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("lat,shape,batch,force", [
    ("D2Q9", (1, 1, 3), 1, 0),      # a few nodes of one block
    ("D2Q9", (1, 5, 13), 1, 1),     # 65 nodes: a second block with one node
    ("D3Q19", (4, 5, 10), 3, 2),    # 600 nodes, three fields in one block range
    ("D3Q19", (33, 32, 33), 1, 2),  # 545 blocks on 512 workgroups: some take a second one
])
def test_wide_step_16bit_blocks(lbm, lat, shape, batch, force, prec):
    """The step by blocks of 64 nodes where its blocks and its workgroups' walks
    end: 300 repeats give the same bits, and the result lies within half the
    rounding effect of the kernels' scheme (as the other 16-bit rows)."""
    nz, ny, nx = shape
    kw = {1: dict(force_kind=1, force_amp=1e-3, force_k=1),
          2: dict(force_kind=2, force_amp=1e-3, force_k=1)}.get(force, {})
    ocfg = oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=batch, tau=0.55, hidden=300,
                         net="paper", out_scale=0.25, **kw)
    theta = inputs.glorot_params_net(inputs.net_widths(ocfg.Q, 0, "paper"), seed=7)
    g = random_state(ocfg, 75, scale=0.03)
    L = lbm.Lattice(lib_config(ocfg, prec))
    A, th = dev(to_shifted(g, lat)), dev(theta)
    out = L.step(A, th, 1)
    for _ in range(300):
        again = L.step(A, th, 1)
    assert torch.equal(out, again)
    got = to_canonical(host(out), lat)
    L.close()
    oracle.set_threads(8)
    try:
        kcfg, kth = kernel_emulation(ocfg, theta, prec)
        want = oracle.step(kcfg, g, kth)
        exact = oracle.step(ocfg, g, theta.astype(np.float64))
    finally:
        oracle.set_threads(1)
    gap, eff = np.linalg.norm(got - want), np.linalg.norm(want - exact)
    print(f"{lat} {shape} x{batch} {prec}: |gpu - emulated| / rounding effect {gap / eff:.2e}")
    assert gap < 0.5 * eff


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("lat,shape,batch,force", [
    ("D2Q9", (1, 16, 126), 128, 0),
    ("D2Q9", (1, 16, 126), 128, 1),
    ("D3Q19", (8, 8, 62), 64, 0),
    ("D3Q19", (8, 8, 62), 64, 2),
])
def test_wide_step_kernels_same_bits(lbm, lat, shape, batch, force, prec):
    """The two kernels of the 16-bit step, by row items and by blocks of 64
    nodes, against each other, two steps: the fields of a large batch advanced
    together and one by one.  On 256 compute units the whole batch has 4096
    ragged row items (two per wavefront) and some 254,000 nodes, 7.8 blocks
    per place for one: row items by a factor of 1.3 in the rule; a field
    alone (32 or 64 items, at most 63 blocks) runs by blocks by a factor of 2."""
    nz, ny, nx = shape
    kw = {1: dict(force_kind=1, force_amp=1e-3, force_k=1),
          2: dict(force_kind=2, force_amp=1e-3, force_k=1)}.get(force, {})
    theta = dev(inputs.glorot_params_net(inputs.net_widths(9 if lat == "D2Q9" else 19, 0, "paper"),
                                         seed=7))

    def lattice(n):
        return lbm.Lattice(lib_config(oracle.Config(
            lattice=lat, nx=nx, ny=ny, nz=nz, batch=n, tau=0.55, hidden=300, net="paper",
            out_scale=0.25, **kw), prec))

    A = dev(to_shifted(random_state(oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=batch,
                                                  tau=0.55), 76, scale=0.03), lat))
    L, one = lattice(batch), lattice(1)
    full = L.step(A, theta, 2)
    for b in range(0, batch, 7):
        assert torch.equal(one.step(A[b:b + 1], theta, 2), full[b:b + 1]), b
    L.close()
    one.close()


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
def test_wide_adjoint_16bit_128_ranges(lbm, prec):
    """373,248 nodes, 128 node ranges, the last one empty.  Against its fields
    one by one, as test_wide_adjoint_16bit_beyond_cache: lam the same bits,
    dtheta the same sums in another order, bar 1e-5."""
    cfg = dict(lattice="D3Q19", nx=24, ny=24, nz=18, tau=0.55, hidden=300, net="paper",
               out_scale=0.25)
    L = lbm.Lattice(lib_config(oracle.Config(batch=36, **cfg), prec))
    one = lbm.Lattice(lib_config(oracle.Config(batch=1, **cfg), prec))
    theta = dev(inputs.glorot_params_net(inputs.net_widths(19, 0, "paper"), seed=7))
    gen = torch.Generator(device="cuda").manual_seed(77)
    A = torch.randn(L.cfg.state_shape, generator=gen, device="cuda") * 0.03
    lam1 = torch.randn(L.cfg.state_shape, generator=gen, device="cuda")
    lam, dth = L.step_backward(A, theta, lam1)
    sums = torch.zeros(L.n_param, dtype=torch.float64, device="cuda")
    for b in range(36):
        l, d = one.step_backward(A[b:b + 1], theta, lam1[b:b + 1])
        assert torch.equal(lam[b:b + 1], l), b
        sums += d
    assert rel_l2(host(dth), host(sums)) < 1e-5
    L.close()
    one.close()


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("lat,shape,batch", [("D2Q9", (1, 5, 13), 1), ("D3Q19", (33, 32, 33), 1)])
def test_wide_16bit_repeats(lbm, lat, shape, batch, prec):
    """Every one of 300 repeats of the step by blocks and of 100 of the adjoint
    gives the bits of the first (a race on the activations in LDS or on the
    next block's populations would show in some of them)."""
    nz, ny, nx = shape
    ocfg = oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=batch, tau=0.55, hidden=300,
                         net="paper", out_scale=0.25)
    L = lbm.Lattice(lib_config(ocfg, prec))
    th = dev(inputs.glorot_params_net(inputs.net_widths(ocfg.Q, 0, "paper"), seed=7))
    A = dev(to_shifted(random_state(ocfg, 75, scale=0.03), lat))
    lam1 = dev(to_shifted(random_state(ocfg, 78, scale=1.0), lat))
    out, (lam, dth) = L.step(A, th, 1), L.step_backward(A, th, lam1)
    differs = torch.zeros(3, dtype=torch.int64, device="cuda")
    for _ in range(300):
        differs[0] += (L.step(A, th, 1) != out).any()
    for _ in range(100):
        l, d = L.step_backward(A, th, lam1)
        differs[1] += (l != lam).any()
        differs[2] += (d != dth).any()
    assert differs.tolist() == [0, 0, 0]
    L.close()


@pytest.mark.parametrize("lat,shape,batch", [
    ("D2Q9", (1, 3, 5), 1), ("D2Q9", (1, 40, 41), 1), ("D3Q19", (16, 16, 17), 1),
    ("D3Q19", (32, 32, 32), 1), ("D3Q19", (44, 44, 44), 1), ("D3Q19", (24, 24, 18), 36),
])
def test_wide_adjoint_16bit_workspace(lbm, lat, shape, batch):
    """The workspace holds one record per node (3,200 bytes) and at most 128
    gradient slabs, and the adjoint stays inside it: bytes behind the stated
    size keep their values."""
    nz, ny, nx = shape
    ocfg = oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=batch, tau=0.55, hidden=300,
                         net="paper", out_scale=0.25)
    L = lbm.Lattice(lib_config(ocfg, "bf16"))
    nodes, need = nx * ny * nz * batch, lbm.lbm_workspace_bytes(L.ctx)
    assert need <= 3200 * (nodes + 63) + 546 * 1024 * min(128, nodes // 256 + 1)
    ws = torch.full((need + (1 << 20),), 0x5A, dtype=torch.uint8, device="cuda")
    th = dev(inputs.glorot_params_net(inputs.net_widths(ocfg.Q, 0, "paper"), seed=7))
    gen = torch.Generator(device="cuda").manual_seed(79)
    A = torch.randn(L.cfg.state_shape, generator=gen, device="cuda") * 0.03
    lam1 = torch.randn(L.cfg.state_shape, generator=gen, device="cuda")
    lam, dth = torch.empty_like(A), torch.zeros_like(th)
    lbm.lbm_step_backward(L.ctx, L.cfg, A, th, lam1, lam, dth, ws[:need])
    assert bool((ws[need:] == 0x5A).all())
    assert bool(torch.isfinite(lam).all()) and bool(torch.isfinite(dth).all())
    L.close()


@pytest.mark.parametrize("prec", ["bf16", "fp16"])
@pytest.mark.parametrize("n", [44, 70])
def test_wide_adjoint_16bit_large_reference(lbm, n, prec):
    """dtheta where the records leave the cache (44^3, 64 node ranges) and
    with 128 ranges (70^3), against the same products in float64 with the
    operands rounded where the kernels round them.  What is left are float32
    sums (some 1e-6), the operands that they tip to the next 16-bit value (one
    in a few thousand, each by 2^-9 or 2^-12), and with those, once in a million,
    the sign of a pre-activation: bar 1e-3, every parameter block on its own."""
    ocfg = oracle.Config(lattice="D3Q19", nx=n, ny=n, nz=n, tau=0.55, hidden=300, net="paper",
                         out_scale=0.25)
    L = lbm.Lattice(lib_config(ocfg, prec))
    theta = dev(inputs.glorot_params_net(inputs.net_widths(19, 0, "paper"), seed=7))
    theta += 0.01 * torch.randn(theta.shape, device="cuda",
                                generator=torch.Generator(device="cuda").manual_seed(80))
    gen = torch.Generator(device="cuda").manual_seed(81)
    A = torch.randn(L.cfg.state_shape, generator=gen, device="cuda") * 0.03
    lam1 = torch.randn(L.cfg.state_shape, generator=gen, device="cuda")
    _, got = L.step_backward(A, theta, lam1)
    L.close()

    dt = {"bf16": torch.bfloat16, "fp16": torch.float16}[prec]
    rnd = lambda t: t.float().to(dt).double()
    offs = _blocks(19)
    par = [theta[a:b].double() for a, b in zip(offs, offs[1:] + [theta.numel()])]
    W1, W2, W3, W4 = (rnd(p).reshape(s) for p, s in
                      zip(par[::2], ((300, 19), (300, 300), (100, 300), (19, 100))))
    c = np.array(lbm.lbm_lattice_tables("D3Q19")[0])
    g = torch.stack([torch.roll(A[0, q], shifts=(int(c[q, 2]), int(c[q, 1]), int(c[q, 0])),
                                dims=(0, 1, 2)).reshape(-1) for q in range(19)], dim=1)
    X = rnd(g)
    act = lambda z: rnd(torch.where(z > 0, z, 0.01 * z))
    H1 = act(X @ W1.T + rnd(par[1]))
    H2 = act(H1 @ W2.T + par[3])
    H3 = act(H2 @ W3.T + par[5])
    mu = lam1[0].reshape(19, -1).T.double()
    cd = torch.from_numpy(c.astype(np.float64)).cuda()
    nu = mu - mu.sum(1, keepdim=True) / 19 - (mu @ cd) @ cd.T / 10
    dY = rnd(0.25 / 0.55 * nu)
    back = lambda d, W, H: rnd(d @ W * torch.where(H > 0, 1.0, 0.01))
    dZ3 = back(dY, W4, H3)
    dZ2 = back(dZ3, W3, H2)
    dZ1 = back(dZ2, W2, H1)
    want = []
    for d, x in ((dZ1, X), (dZ2, H1), (dZ3, H2), (dY, H3)):
        want += [(d.T @ x).reshape(-1), d.sum(0)]
    errs = [((got[a:a + w.numel()].double() - w).norm() / w.norm()).item() for a, w in zip(offs, want)]
    print(f"{n}^3 {prec}: blocks " + " ".join(f"{e:.1e}" for e in errs))
    assert sum(w.numel() for w in want) == theta.numel()
    assert max(errs) < 1e-3
