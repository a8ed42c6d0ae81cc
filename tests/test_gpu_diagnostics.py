"""GPU parity of the diagnostics against the FP64 oracle: structure
functions of a velocity field, and the sums of the moment-space analysis
for one step of each collision (BGK, the two networks, Smagorinsky)."""
import numpy as np
import pytest

import oracle
from lbm_cases import lib_config, params, random_state, to_canonical, to_shifted
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


@pytest.mark.parametrize("lat,shape", [("D2Q9", (1, 30, 70)), ("D3Q19", (6, 7, 9))])
def test_structure_functions(lbm, lat, shape):
    nz, ny, nx = shape
    ocfg = oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=2)
    u = np.random.default_rng(91).normal(0, 0.05, (2, ocfg.D, nz, ny, nx)).astype(np.float32)
    lmax, pmax = min(shape[1:] if lat == "D2Q9" else shape), 6
    want, wabs = oracle.structure_functions(ocfg, u.astype(np.float64), lmax, pmax)
    L = lbm.Lattice(lib_config(ocfg))
    S = torch.empty((pmax, lmax), dtype=torch.float64, device="cuda")
    Sa = torch.empty_like(S)
    nws = lbm.lbm_structure_functions_workspace_bytes(L.ctx, lmax, pmax)
    assert nws == 8 * lmax * 64 * 2 * pmax
    ud = torch.from_numpy(u).cuda()
    # a workspace one double short is refused before anything is launched
    short = torch.empty(nws // 8 - 1, dtype=torch.float64, device="cuda")
    with pytest.raises(lbm.LBMError) as e:
        lbm.lbm_structure_functions(L.ctx, L.cfg, ud, lmax, pmax, S, Sa, short)
    assert e.value.status == lbm.LBM_ERR_WORKSPACE
    ws = torch.empty(nws // 8, dtype=torch.float64, device="cuda")
    lbm.lbm_structure_functions(L.ctx, L.cfg, ud, lmax, pmax, S, Sa, ws)
    got, gabs = S.cpu().numpy(), Sa.cpu().numpy()
    assert np.abs(got - want).max() <= 1e-12 * np.abs(wabs).max(axis=1, keepdims=True).max()
    assert np.all(np.abs(gabs - wabs) <= 1e-12 * wabs)
    # a smaller second call in the same workspace
    want2, wabs2 = oracle.structure_functions(ocfg, u.astype(np.float64), 3, 2)
    S2 = torch.empty((2, 3), dtype=torch.float64, device="cuda")
    Sa2 = torch.empty_like(S2)
    lbm.lbm_structure_functions(L.ctx, L.cfg, ud, 3, 2, S2, Sa2, ws)
    assert np.all(np.abs(Sa2.cpu().numpy() - wabs2) <= 1e-12 * wabs2)
    assert np.abs(S2.cpu().numpy() - want2).max() <= 1e-12 * np.abs(wabs2).max()
    L.close()


@pytest.mark.parametrize("kind", ["bgk", "tanh", "paper", "smagorinsky", "bgk-forced"])
def test_mrt_moment_sums(lbm, kind):
    from paper_2403_18466_amd import diagnostics
    kw = dict(lattice="D3Q19", nx=9, ny=6, nz=5, batch=2, tau=0.55)
    theta = None
    if kind == "tanh":
        kw.update(hidden=64, out_scale=0.25)
        theta = params(19, 64, seed=92, kind="random")
    elif kind == "paper":
        kw.update(hidden=300, net="paper", out_scale=0.25)
        theta = inputs.random_params_net(inputs.net_widths(19, 0, "paper"), 93, scale=0.05)
    elif kind == "smagorinsky":
        kw.update(collision="smagorinsky", smag_cs=0.17)
    elif kind == "bgk-forced":
        kw.update(force_kind=2, force_amp=1e-3, force_k=1)
    ocfg = oracle.Config(**kw)
    g = random_state(ocfg, 94, 0.03)
    L = lbm.Lattice(lib_config(ocfg))
    A = torch.from_numpy(to_shifted(g, "D3Q19").astype(np.float32)).cuda()
    th = torch.from_numpy(theta).cuda() if theta is not None else None
    A1 = L.step(A, th, 1)
    stats = torch.empty((19, 5), dtype=torch.float64, device="cuda")
    lbm.lbm_mrt_moment_sums(L.ctx, A, A1, stats)
    got = stats.cpu().numpy()
    torch.cuda.synchronize()
    g1 = to_canonical(A1.cpu().numpy().astype(np.float64), "D3Q19")
    want = oracle.mrt_moment_sums(ocfg, g.astype(np.float32).astype(np.float64), g1)
    scale = np.abs(want).max(axis=1, keepdims=True) + 1e-30
    assert np.abs(got - want).max() <= 1e-5 * scale.max()
    res = diagnostics.relaxation_from_sums(got, 2 * 9 * 6 * 5)
    if kind.startswith("bgk"):
        for name in ("pxy", "pxx", "e", "qx", "mx"):
            assert abs(res[name][0] - 0.55) < 1e-4, (name, res[name])
    print(kind, {k: round(v[0], 4) for k, v in res.items() if not np.isnan(v[0])})
    L.close()


@pytest.mark.parametrize("lat,shape,batch,lmax,pmax", [
    ("D2Q9", (1, 2, 3), 1, 2, 1),        # fewer nodes than a wavefront
    ("D2Q9", (1, 19, 41), 3, 19, 8),     # four separations per thread, the last group short
    ("D3Q19", (17, 18, 37), 1, 16, 7),   # the smallest lmax of that form
    ("D3Q19", (16, 50, 50), 1, 15, 5),   # the largest of the other; 40,000 nodes, 64 x 512 threads
    ("D3Q19", (16, 50, 50), 1, 16, 3),   # every separation wraps in z at lmax = nz
])
def test_structure_functions_edges(lbm, lat, shape, batch, lmax, pmax):
    """Grid and separation counts at the ends of the kernel's groups, every
    power: within 1e-12 of the oracle (float64 sums in another order)."""
    nz, ny, nx = shape
    ocfg = oracle.Config(lattice=lat, nx=nx, ny=ny, nz=nz, batch=batch)
    u = np.random.default_rng(95).normal(0, 0.05, (batch, ocfg.D, nz, ny, nx)).astype(np.float32)
    want, wabs = oracle.structure_functions(ocfg, u.astype(np.float64), lmax, pmax)
    L = lbm.Lattice(lib_config(ocfg))
    S = torch.empty((pmax, lmax), dtype=torch.float64, device="cuda")
    Sa = torch.empty_like(S)
    ws = torch.empty(lbm.lbm_structure_functions_workspace_bytes(L.ctx, lmax, pmax) // 8,
                     dtype=torch.float64, device="cuda")
    lbm.lbm_structure_functions(L.ctx, L.cfg, torch.from_numpy(u).cuda(), lmax, pmax, S, Sa, ws)
    assert np.all(np.abs(Sa.cpu().numpy() - wabs) <= 1e-12 * wabs)
    assert np.all(np.abs(S.cpu().numpy() - want) <= 1e-12 * wabs)
    L.close()


@pytest.mark.parametrize("shape,batch", [((1, 1, 2), 1), ((3, 43, 2), 1), ((47, 40, 36), 1)])
def test_mrt_moment_sums_edges(lbm, shape, batch):
    """One block of a few nodes, a second block of two nodes (258), and more
    nodes (67,680) than threads: the sums over the nodes against the oracle."""
    nz, ny, nx = shape
    ocfg = oracle.Config(lattice="D3Q19", nx=nx, ny=ny, nz=nz, batch=batch, tau=0.55)
    g = random_state(ocfg, 96, 0.03)
    L = lbm.Lattice(lib_config(ocfg))
    A = torch.from_numpy(to_shifted(g, "D3Q19").astype(np.float32)).cuda()
    A1 = L.step(A, None, 1)
    stats = torch.empty((19, 5), dtype=torch.float64, device="cuda")
    lbm.lbm_mrt_moment_sums(L.ctx, A, A1, stats)
    got = stats.cpu().numpy()
    L.close()
    want = oracle.mrt_moment_sums(ocfg, g.astype(np.float32).astype(np.float64),
                                  to_canonical(A1.cpu().numpy().astype(np.float64), "D3Q19"))
    assert np.abs(got - want).max() <= 1e-5 * np.abs(want).max()


@pytest.mark.parametrize("lat,shape", [("D2Q9", (1, 30, 41)), ("D3Q19", (17, 19, 18))])
@pytest.mark.parametrize("lmax", [3, 17])
def test_structure_function_orders_agree(lbm, lat, shape, lmax):
    """The sums of an order do not depend on how many more are asked for (1 to
    12 sums per separation go through the wavefront's reduction, for one or
    four separations): the same bits."""
    nz, ny, nx = shape
    L = lbm.Lattice(lbm.Config(lattice=lat, nx=nx, ny=ny, nz=nz))
    u = torch.from_numpy(np.random.default_rng(96).normal(0, 0.05, (1, L.cfg.D, nz, ny, nx))
                         .astype(np.float32)).cuda()
    ws = torch.empty(lbm.lbm_structure_functions_workspace_bytes(L.ctx, lmax, 8) // 8,
                     dtype=torch.float64, device="cuda")
    got = {}
    for pmax in range(1, 9):
        S, Sa = (torch.full((pmax, lmax), float("nan"), dtype=torch.float64, device="cuda")
                 for _ in range(2))
        lbm.lbm_structure_functions(L.ctx, L.cfg, u, lmax, pmax, S, Sa, ws)
        got[pmax] = S.cpu(), Sa.cpu()
    for pmax in range(1, 8):
        for a, b in zip(got[pmax], got[8]):
            assert torch.equal(a, b[:pmax]), pmax
    L.close()
