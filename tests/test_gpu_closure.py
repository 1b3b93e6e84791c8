"""GPU tests of the learned subgrid closure against the CPU oracle.

Tolerances:
  * bfloat16 inference: the oracle follows the kernel's precision steps
    (normalised features, weights and hidden activations rounded to
    bfloat16, nearest-even) but sums in FP64 and uses the FP64 erf; the
    kernel sums in FP32 with an FP32 erf approximation (|error| <= 1.5e-7)
    and holds the gradient features in FP32 before normalising them.  A hidden activation whose FP32
    and FP64 values straddle a bfloat16 rounding boundary differs by one
    bfloat16 ulp (2^-8 relative); these are rare (~1e-7 / 4e-3 per value),
    so the output error is held to 1e-3 of the output norm per component,
    and 2e-2 of each component's largest value point-wise.
  * FP32 training kernels against the FP64 oracle: sums of up to a few
    hundred FP32 products, relative 1e-4 on the gradient; Adam updates of a
    few steps, relative 1e-3 on the parameter change.
  * filter: FP64 on both sides, relative 1e-12.
"""
import numpy as np
import pytest

from chorus_inputs import box_mesh, cubed_sphere_shell, mlp_init, random_velocity, uniform_noise

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch


@pytest.fixture(scope="module")
def ch(torch_dev):
    import paper_1503_00834_amd as ch
    return ch


@pytest.fixture(scope="module")
def cl(oracle_mod):
    from oracle import closure
    return closure


def _state(om, seed, vel=0.2):
    """Polytrope with a seeded smooth velocity field and entropy noise."""
    Q, _ = om.polytrope(0.7, 1.0, noise=uniform_noise(om.n_solpts, seed), amp=1e-2)
    xyz, _ = om.solpts()
    u = random_velocity(xyz, seed + 1, amp=vel)
    Q = Q.reshape(5, -1)
    Q[1:4] = Q[0] * u
    Q[4] += 0.5 * Q[0] * (u ** 2).sum(0)
    return Q.reshape(5, om.E, om.np)


def _shell_case(oracle_mod, seed=3):
    beta = 0.7
    ri, ro = beta / (1 - beta), 1 / (1 - beta)
    m = cubed_sphere_shell(3, 2, ri, ro)
    om = oracle_mod.OracleMesh(m, 3)
    Q0, pars = om.polytrope(beta, 1.0)
    return m, om, pars, _state(om, seed)


def _norm_from(cl, X, T=None):
    """Normalisation from feature statistics (oracle side data)."""
    norm = np.zeros(70)
    norm[0:20] = X.mean(0)
    norm[20:40] = 1.0 / np.maximum(X.std(0), 1e-12)
    if T is not None:
        norm[40:55] = T.mean(0)
        norm[55:70] = T.std(0)
    else:
        norm[40:55] = np.linspace(-0.1, 0.1, 15)
        norm[55:70] = np.linspace(0.5, 1.5, 15)
    return norm


def _dev(torch, a, dtype=None):
    import torch as t
    return t.from_numpy(np.ascontiguousarray(a)).to(dtype or t.float64).cuda()


def test_infer_bf16_matches_oracle(ch, cl, oracle_mod, torch_dev):
    torch = torch_dev
    m, om, pars, Q = _shell_case(oracle_mod)
    ph_o = oracle_mod.phys(GM=pars["GM"], omega=1.0, nu=1e-3, kappa=1e-3)
    raw = cl.features(om, ph_o, Q)
    params = mlp_init(11) * 1.5
    params[1280:1344] = np.linspace(-0.3, 0.3, 64)     # non-zero biases
    params[5440:5504] = np.linspace(0.2, -0.2, 64)
    params[6464:6479] = np.linspace(-0.05, 0.05, 15)
    norm = _norm_from(cl, raw)
    want = cl.infer_bf16(params, norm, raw)              # [n][15]
    want64 = cl.infer_fp64(params, norm, raw)
    model = ch.chorus_closure_pack(_dev(torch, params, torch.float32), _dev(torch, norm, torch.float32))
    phys = ch.physics(GM=pars["GM"], omega=1.0, nu=1e-3, kappa=1e-3, closure=ch.CHORUS_CLOSURE_MLP,
                      closure_model=model)
    cm = ch.mesh_from_arrays(m, 3).upload()
    ws = cm.workspace(phys)
    sgs = torch.zeros((15, cm.n_solpts), dtype=torch.float32, device="cuda")
    ch.chorus_closure_infer(cm, phys, _dev(torch, Q.reshape(5, -1)), sgs, ws)
    # features through the ABI (FP32 rounding of the FP64 values)
    X = torch.zeros((cm.n_solpts, 20), dtype=torch.float32, device="cuda")
    ch.chorus_closure_features(cm, phys, _dev(torch, Q.reshape(5, -1)), X, ws)
    torch.cuda.synchronize()
    got = sgs.cpu().numpy().T.astype(np.float64)
    Xg = X.cpu().numpy().astype(np.float64)
    assert np.allclose(Xg, raw.astype(np.float32).astype(np.float64), rtol=1e-6,
                       atol=1e-6 * np.abs(raw).max(0))
    for k in range(15):
        scale = np.abs(want[:, k]).max()
        err = np.linalg.norm(got[:, k] - want[:, k])
        assert err <= 1e-3 * np.linalg.norm(want[:, k]) + 1e-7 * scale, (k, err)
        assert np.abs(got[:, k] - want[:, k]).max() <= 2e-2 * scale, k
    # and the bfloat16 network is within bfloat16 accuracy of the FP64 one
    rel = np.linalg.norm(got - want64) / np.linalg.norm(want64)
    assert rel < 3e-2, rel
    print("closure inference: rel err vs bf16 oracle %.2e, vs FP64 network %.2e" % (
        np.linalg.norm(got - want) / np.linalg.norm(want), rel))


def test_closure_residual_matches_oracle(ch, cl, oracle_mod, torch_dev):
    torch = torch_dev
    m, om, pars, Q = _shell_case(oracle_mod, seed=5)
    kw = dict(GM=pars["GM"], omega=1.0, nu=1e-3, kappa=1e-3)
    ph_o = oracle_mod.phys(**kw)
    raw = cl.features(om, ph_o, Q)
    params = mlp_init(12) * 1.5
    norm = _norm_from(cl, raw)
    norm[55:70] *= 0.5
    norm[40:43] = 0.0
    norm[55:58] = 0.0        # no subgrid mass flux
    tau = cl.sgs_field(om, ph_o, Q, params, norm)
    R_cl = om.residual(ph_o, Q, tau)
    R_pl = om.residual(ph_o, Q)
    model = ch.chorus_closure_pack(_dev(torch, params, torch.float32), _dev(torch, norm, torch.float32))
    phys = ch.physics(closure=ch.CHORUS_CLOSURE_MLP, closure_model=model, **kw)
    cm = ch.mesh_from_arrays(m, 3).upload()
    ws = cm.workspace(phys)
    R = torch.empty((5, cm.n_solpts), dtype=torch.float64, device="cuda")
    ch.chorus_sd_residual(cm, phys, _dev(torch, Q.reshape(5, -1)), R, ws)
    torch.cuda.synchronize()
    Rg = R.cpu().numpy().reshape(5, om.E, om.np)
    for v in range(5):
        d = np.linalg.norm(R_cl[v] - R_pl[v])
        err = np.linalg.norm(Rg[v] - R_cl[v])
        assert err <= 2e-3 * d + 1e-11 * np.linalg.norm(R_cl[v]), (v, err, d)
    # the closure changes the residual by far more than the tolerance
    assert np.linalg.norm(R_cl[1:] - R_pl[1:]) > 1e-3 * np.linalg.norm(R_pl[1:])


def test_closure_odd_element_count(ch, cl, oracle_mod, torch_dev):
    """27 hexes (a curved periodic box): the network pass's last block of
    two elements holds one; inference and the closure residual against the
    oracle, to the tolerances above."""
    torch = torch_dev
    m = box_mesh(3, 3, 3, periodic=(True,) * 3, curve=0.03)
    om = oracle_mod.OracleMesh(m, 3)
    assert om.E == 27
    xyz, _ = om.solpts()
    x, y, z = xyz
    rho = 1 + 0.2 * np.sin(2 * np.pi * (x + y))
    u = np.stack([0.3 * np.cos(2 * np.pi * z), -0.2 * np.sin(2 * np.pi * x), 0.25 * np.cos(2 * np.pi * y)])
    Q = np.stack([rho, rho * u[0], rho * u[1], rho * u[2],
                  2.5 + 0.1 * np.sin(2 * np.pi * z) + 0.5 * rho * (u ** 2).sum(0)]).reshape(5, om.E, om.np)
    kw = dict(nu=1e-3, kappa=1e-3)
    ph_o = oracle_mod.phys(**kw)
    raw = cl.features(om, ph_o, Q)
    params = mlp_init(14) * 1.5
    norm = _norm_from(cl, raw)
    norm[40:43] = 0.0
    norm[55:58] = 0.0
    want = cl.infer_bf16(params, norm, raw)
    model = ch.chorus_closure_pack(_dev(torch, params, torch.float32), _dev(torch, norm, torch.float32))
    phys = ch.physics(closure=ch.CHORUS_CLOSURE_MLP, closure_model=model, **kw)
    cm = ch.mesh_from_arrays(m, 3).upload()
    ws = cm.workspace(phys)
    sgs = torch.zeros((15, cm.n_solpts), dtype=torch.float32, device="cuda")
    ch.chorus_closure_infer(cm, phys, _dev(torch, Q.reshape(5, -1)), sgs, ws)
    R = torch.empty((5, cm.n_solpts), dtype=torch.float64, device="cuda")
    ch.chorus_sd_residual(cm, phys, _dev(torch, Q.reshape(5, -1)), R, ws)
    torch.cuda.synchronize()
    got = sgs.cpu().numpy().T.astype(np.float64)
    for k in range(3, 15):
        scale = np.abs(want[:, k]).max()
        assert np.linalg.norm(got[:, k] - want[:, k]) <= 1e-3 * np.linalg.norm(want[:, k]) + 1e-7 * scale, k
        # the last element (alone in its block) on its own
        last = slice((om.E - 1) * om.np, om.E * om.np)
        assert np.abs(got[last, k] - want[last, k]).max() <= 2e-2 * scale, k
    tau = cl.sgs_field(om, ph_o, Q, params, norm)
    R_cl = om.residual(ph_o, Q, tau)
    R_pl = om.residual(ph_o, Q)
    Rg = R.cpu().numpy().reshape(5, om.E, om.np)
    for v in range(5):
        d = np.linalg.norm(R_cl[v] - R_pl[v])
        err = np.linalg.norm(Rg[v] - R_cl[v])
        assert err <= 2e-3 * d + 1e-11 * np.linalg.norm(R_cl[v]), (v, err, d)
    assert np.linalg.norm(R_cl[1:] - R_pl[1:]) > 1e-3 * np.linalg.norm(R_pl[1:])


def test_closure_on_a_large_mesh(ch, cl, oracle_mod, torch_dev):
    """2,873 hexes, above the wide lift pass (10 elements per CU of 256) and odd
    (the last block of two elements holds one): the closure residual against
    the oracle (a wrong last element would be 1.9e-2 of the closure's part, ten
    times the bound)."""
    torch = torch_dev
    m = box_mesh(13, 13, 17, periodic=(True,) * 3, curve=0.01)
    om = oracle_mod.OracleMesh(m, 3)
    assert om.E == 2873
    x, y, z = om.solpts()[0]
    rho = 1 + 0.2 * np.sin(2 * np.pi * (x + y))
    u = np.stack([0.3 * np.cos(2 * np.pi * z), -0.2 * np.sin(2 * np.pi * x), 0.25 * np.cos(2 * np.pi * y)])
    Q = np.stack([rho, rho * u[0], rho * u[1], rho * u[2],
                  2.5 + 0.1 * np.sin(2 * np.pi * z) + 0.5 * rho * (u ** 2).sum(0)]).reshape(5, om.E, om.np)
    kw = dict(nu=1e-3, kappa=1e-3)
    ph_o = oracle_mod.phys(**kw)
    params = mlp_init(14) * 1.5
    norm = _norm_from(cl, cl.features(om, ph_o, Q))
    norm[40:70] *= 2e-3  # a subgrid flux of the flux's own size
    model = ch.chorus_closure_pack(_dev(torch, params, torch.float32), _dev(torch, norm, torch.float32))
    phys = ch.physics(closure=ch.CHORUS_CLOSURE_MLP, closure_model=model, **kw)
    cm = ch.mesh_from_arrays(m, 3).upload()
    ws = cm.workspace(phys)
    Qd = _dev(torch, Q.reshape(5, -1))
    Rd = torch.empty_like(Qd)
    ch.chorus_sd_residual(cm, phys, Qd, Rd, ws)
    torch.cuda.synchronize()
    want = om.residual(ph_o, Q, cl.sgs_field(om, ph_o, Q, params, norm))
    plain = om.residual(ph_o, Q)
    Rg = Rd.cpu().numpy().reshape(5, om.E, om.np)
    for v in range(5):
        d = np.linalg.norm(want[v] - plain[v])
        err = np.linalg.norm(Rg[v] - want[v])
        assert err <= 2e-3 * d + 1e-11 * np.linalg.norm(want[v]), (v, err, d)
    # the mass part of the subgrid flux (the lift's fifth component) counts
    assert np.linalg.norm(want[0] - plain[0]) > 1e-2 * np.linalg.norm(plain[0])


def test_closure_rk_steps_match_oracle(ch, cl, oracle_mod, torch_dev):
    """Two SSP-RK3 steps with the closure re-evaluated at every stage."""
    torch = torch_dev
    m, om, pars, Q = _shell_case(oracle_mod, seed=7)
    kw = dict(GM=pars["GM"], omega=1.0, nu=1e-3, kappa=1e-3)
    ph_o = oracle_mod.phys(**kw)
    raw = cl.features(om, ph_o, Q)
    params = mlp_init(13)
    norm = _norm_from(cl, raw)
    norm[40:43] = 0.0
    norm[55:58] = 0.0
    dt = 2e-3

    def R(q):
        return om.residual(ph_o, q, cl.sgs_field(om, ph_o, q, params, norm))
    q = Q.copy()
    for _ in range(2):
        q1 = q + dt * R(q)
        q2 = 0.75 * q + 0.25 * (q1 + dt * R(q1))
        q = q / 3.0 + 2.0 / 3.0 * (q2 + dt * R(q2))
    model = ch.chorus_closure_pack(_dev(torch, params, torch.float32), _dev(torch, norm, torch.float32))
    phys = ch.physics(closure=ch.CHORUS_CLOSURE_MLP, closure_model=model, **kw)
    cm = ch.mesh_from_arrays(m, 3).upload()
    ws = cm.workspace(phys)
    Qd = _dev(torch, Q.reshape(5, -1))
    ch.chorus_rk_step(cm, phys, Qd, dt, 2, ws)
    torch.cuda.synchronize()
    got = Qd.cpu().numpy().reshape(5, om.E, om.np)
    for v in range(5):
        dq = np.linalg.norm(q[v] - Q[v])
        assert np.linalg.norm(got[v] - q[v]) <= 2e-3 * dq + 1e-13 * np.linalg.norm(q[v]), v


def test_closure_ssp54_step_matches_oracle(ch, cl, oracle_mod, torch_dev):
    """One step of the five-stage SSP method with the closure re-evaluated at
    every stage (the oracle's Shu-Osher table, stage sums written out)."""
    torch = torch_dev
    m, om, pars, Q = _shell_case(oracle_mod, seed=9)
    kw = dict(GM=pars["GM"], omega=1.0, nu=1e-3, kappa=1e-3)
    ph_o = oracle_mod.phys(**kw)
    raw = cl.features(om, ph_o, Q)
    params = mlp_init(15)
    norm = _norm_from(cl, raw)
    norm[40:43] = 0.0
    norm[55:58] = 0.0
    dt = 3e-3
    alpha, beta = oracle_mod.ssp54_table()

    def R(q):
        return om.residual(ph_o, q, cl.sgs_field(om, ph_o, q, params, norm))
    u = [Q.copy()]
    L = []
    for i in range(5):
        L.append(R(u[i]))
        u.append(sum(alpha[i, k] * u[k] + dt * beta[i, k] * L[k] for k in range(i + 1)))
    q = u[5]
    model = ch.chorus_closure_pack(_dev(torch, params, torch.float32), _dev(torch, norm, torch.float32))
    phys = ch.physics(closure=ch.CHORUS_CLOSURE_MLP, closure_model=model, integrator=ch.CHORUS_SSPRK54, **kw)
    cm = ch.mesh_from_arrays(m, 3).upload()
    ws = cm.workspace(phys)
    Qd = _dev(torch, Q.reshape(5, -1))
    ch.chorus_rk_step(cm, phys, Qd, dt, 1, ws)
    torch.cuda.synchronize()
    got = Qd.cpu().numpy().reshape(5, om.E, om.np)
    for v in range(5):
        dq = np.linalg.norm(q[v] - Q[v])
        assert np.linalg.norm(got[v] - q[v]) <= 2e-3 * dq + 1e-13 * np.linalg.norm(q[v]), v


@pytest.mark.parametrize("n", [1, 17, 64, 300])
def test_grad_matches_oracle(ch, cl, torch_dev, n):
    torch = torch_dev
    rng = np.random.default_rng(21 + n)
    X = rng.normal(size=(n, 20))
    T = rng.normal(size=(n, 15))
    params = mlp_init(14) * 1.2
    params[1280:1344] = rng.normal(0, 0.1, 64)
    p32 = params.astype(np.float32).astype(np.float64)
    X32 = X.astype(np.float32).astype(np.float64)
    T32 = T.astype(np.float32).astype(np.float64)
    g_want = cl.grad(p32, X32, T32)
    l_want = cl.loss(p32, X32, T32)
    ws = ch.closure_train_workspace(n)
    grad = torch.zeros(6479, dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    ch.chorus_closure_grad(_dev(torch, X, torch.float32), _dev(torch, T, torch.float32),
                           _dev(torch, params, torch.float32), grad, loss, ws)
    torch.cuda.synchronize()
    g = grad.cpu().numpy().astype(np.float64)
    assert abs(loss.item() - l_want) <= 1e-5 * l_want
    for lo, hi in ((0, 1280), (1280, 1344), (1344, 5440), (5440, 5504), (5504, 6464), (6464, 6479)):
        err = np.linalg.norm(g[lo:hi] - g_want[lo:hi])
        assert err <= 1e-4 * np.linalg.norm(g_want[lo:hi]), (lo, err)


@pytest.mark.parametrize("n", [15, 16, 33, 8192, 8209])
def test_grad_at_group_edges(ch, cl, torch_dev, n):
    """One group of 16 samples and its neighbours; the largest batch with one
    group per block (8,192) and one where blocks take a second group."""
    torch = torch_dev
    rng = np.random.default_rng(61 + n)
    X = rng.normal(size=(n, 20)).astype(np.float32)
    T = rng.normal(size=(n, 15)).astype(np.float32)
    p = (mlp_init(14) * 1.2).astype(np.float32)
    g_want = cl.grad(p, X, T)
    ws = ch.closure_train_workspace(n)
    grad = torch.zeros(6479, dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    ch.chorus_closure_grad(_dev(torch, X, torch.float32), _dev(torch, T, torch.float32),
                           _dev(torch, p, torch.float32), grad, loss, ws)
    torch.cuda.synchronize()
    g = grad.cpu().numpy().astype(np.float64)
    assert abs(loss.item() - cl.loss(p, X, T)) <= 1e-5 * loss.item()
    for lo, hi in ((0, 1280), (1280, 1344), (1344, 5440), (5440, 5504), (5504, 6464), (6464, 6479)):
        err = np.linalg.norm(g[lo:hi] - g_want[lo:hi])
        assert err <= 1e-4 * np.linalg.norm(g_want[lo:hi]), (lo, err)


@pytest.mark.parametrize("n", [1, 17, 33, 4096])
def test_grad_in_the_smallest_workspace(ch, cl, torch_dev, n):
    """The least workspace of a batch (273 floats per sample and a partial
    gradient per 64, in 256-byte parts): fewer blocks than groups at 33 and
    4,096 samples; one byte less is refused."""
    torch = torch_dev
    rng = np.random.default_rng(71 + n)
    X = rng.normal(size=(n, 20)).astype(np.float32)
    T = rng.normal(size=(n, 15)).astype(np.float32)
    p = (mlp_init(14) * 1.2).astype(np.float32)
    up = lambda b: (b + 255) // 256 * 256
    least = 4 * up(256 * n) + up(64 * n) + up(4 * n) + up(4 * 6480 * ((n + 63) // 64)) + 256
    full = ch.closure_train_workspace(n).numel()
    assert least <= full <= 1.3 * least
    ws = torch.full((least + 4096,), 255, dtype=torch.uint8, device="cuda")
    grad = torch.zeros(6479, dtype=torch.float32, device="cuda")
    loss = torch.zeros(1, dtype=torch.float32, device="cuda")
    args = (_dev(torch, X, torch.float32), _dev(torch, T, torch.float32), _dev(torch, p, torch.float32), grad, loss)
    with pytest.raises(ch.ChorusError):
        ch.chorus_closure_grad(*args, ws[:least - 1])
    ch.chorus_closure_grad(*args, ws[:least])
    torch.cuda.synchronize()
    assert bool((ws[least:] == 255).all())
    g, g_want = grad.cpu().numpy().astype(np.float64), cl.grad(p, X, T)
    assert abs(loss.item() - cl.loss(p, X, T)) <= 1e-5 * loss.item()
    for lo, hi in ((0, 1280), (1280, 1344), (1344, 5440), (5440, 5504), (5504, 6464), (6464, 6479)):
        err = np.linalg.norm(g[lo:hi] - g_want[lo:hi])
        assert err <= 1e-4 * np.linalg.norm(g_want[lo:hi]), (lo, err)


def _least_train_workspace(n):
    """Bytes a batch of n samples needs: 273 floats per sample and a partial
    gradient of 6,480 floats per 64, in 256-byte parts."""
    up = lambda b: (b + 255) // 256 * 256
    return 4 * up(256 * n) + up(64 * n) + up(4 * n) + up(4 * 6480 * ((n + 63) // 64)) + 256


@pytest.mark.parametrize("n", [16, 17, 33, 1000, 4096, 8188, 8853, 17000])
def test_training_does_not_depend_on_the_workspace_size(ch, cl, torch_dev, n):
    """The batch alone fixes the order of the sums: gradients, losses and an
    Adam trajectory are bitwise the same in the smallest workspace (rows for
    fewer blocks than the batch has from 17 to 8,853 samples, 40 too few at
    8,188), in one with a row more, in one of the queried size and in one of a
    larger batch; and the gradient is the oracle's."""
    torch = torch_dev
    rng = np.random.default_rng(81 + n)
    X = _dev(torch, rng.normal(size=(n, 20)), torch.float32)
    T = _dev(torch, rng.normal(size=(n, 15)), torch.float32)
    p = _dev(torch, mlp_init(14) * 1.2, torch.float32)
    idx = torch.from_numpy(rng.integers(0, n, 3 * n).astype(np.int32)).cuda()
    least = _least_train_workspace(n)
    full = ch.closure_train_workspace(n).numel()
    outs = []
    for size in (least, least + 4 * 6480, full, _least_train_workspace(1 << 16)):
        ws = torch.full((size,), 255, dtype=torch.uint8, device="cuda")
        grad, loss = torch.zeros(6479, device="cuda"), torch.zeros(1, device="cuda")
        ch.chorus_closure_grad(X, T, p, grad, loss, ws)
        q, m, v, L = p.clone(), torch.zeros_like(p), torch.zeros_like(p), torch.zeros(3, device="cuda")
        ch.chorus_closure_train(X, T, idx, n, 3, q, m, v, 0, (1e-3, 0.9, 0.999, 1e-8), L, ws)
        torch.cuda.synchronize()
        outs.append((grad, loss, q, m, v, L))
    for other in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(outs[0], other))
    g, want = outs[0][0].cpu().numpy().astype(np.float64), cl.grad(*(t.cpu().numpy() for t in (p, X, T)))
    for lo, hi in ((0, 1280), (1280, 1344), (1344, 5440), (5440, 5504), (5504, 6464), (6464, 6479)):
        assert np.linalg.norm(g[lo:hi] - want[lo:hi]) <= 1e-4 * np.linalg.norm(want[lo:hi]), lo


def test_train_matches_oracle_and_is_deterministic(ch, cl, torch_dev):
    torch = torch_dev
    rng = np.random.default_rng(31)
    n, batch, iters = 500, 96, 12
    X = rng.normal(size=(n, 20)).astype(np.float32)
    teacher = mlp_init(15) * 2.0
    T, _ = cl.forward(teacher, X.astype(np.float64))
    T = T.astype(np.float32)
    idx = np.concatenate([rng.permutation(n) for _ in range(3)])[: batch * iters].astype(np.int32)
    p0 = mlp_init(16).astype(np.float32)
    hyper = (2e-3, 0.9, 0.999, 1e-8)
    want, _, _, losses_want = cl.train(p0.astype(np.float64), X.astype(np.float64), T.astype(np.float64),
                                       idx, batch, lr=hyper[0], b1=hyper[1], b2=hyper[2], eps=hyper[3])
    outs = []
    for _ in range(2):
        P = _dev(torch, p0, torch.float32)
        M = torch.zeros_like(P)
        V = torch.zeros_like(P)
        L = torch.zeros(iters, dtype=torch.float32, device="cuda")
        ws = ch.closure_train_workspace(batch)
        ch.chorus_closure_train(_dev(torch, X, torch.float32), _dev(torch, T, torch.float32),
                                torch.from_numpy(idx).cuda(), batch, iters, P, M, V, 0, hyper, L, ws)
        torch.cuda.synchronize()
        outs.append((P.cpu().numpy(), L.cpu().numpy()))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])
    got, losses = outs[0][0].astype(np.float64), outs[0][1].astype(np.float64)
    assert np.allclose(losses, losses_want, rtol=1e-4)
    dW = want - p0
    assert np.linalg.norm(got - want) <= 2e-3 * np.linalg.norm(dW)


def test_train_rejects_out_of_range_indices(ch, torch_dev):
    """A sample index outside [0, n) is an argument error, found before any
    training kernel reads through the indices; the parameters stay as
    they were."""
    torch = torch_dev
    n, batch, iters = 200, 64, 3
    rng = np.random.default_rng(41)
    X = torch.from_numpy(rng.normal(size=(n, 20)).astype(np.float32)).cuda()
    T = torch.from_numpy(rng.normal(size=(n, 15)).astype(np.float32)).cuda()
    P = torch.as_tensor(mlp_init(3), dtype=torch.float32).cuda()
    P0 = P.clone()
    M, V = torch.zeros_like(P), torch.zeros_like(P)
    L = torch.zeros(iters, dtype=torch.float32, device="cuda")
    ws = ch.closure_train_workspace(batch)
    for bad in (n, -1):
        idx = torch.zeros(batch * iters, dtype=torch.int32, device="cuda")
        idx[batch * iters - 1] = bad
        with pytest.raises(ch.ChorusError) as ei:
            ch.chorus_closure_train(X, T, idx, batch, iters, P, M, V, 0, (1e-3, 0.9, 0.999, 1e-8), L, ws)
        assert ei.value.status == -1
        torch.cuda.synchronize()
        assert torch.equal(P, P0)
    # in range: trains
    idx = torch.from_numpy(rng.integers(0, n, batch * iters).astype(np.int32)).cuda()
    ch.chorus_closure_train(X, T, idx, batch, iters, P, M, V, 0, (1e-3, 0.9, 0.999, 1e-8), L, ws)
    torch.cuda.synchronize()
    assert not torch.equal(P, P0)


def test_pack_rejects_nonfinite(ch, torch_dev):
    torch = torch_dev
    params = mlp_init(17).astype(np.float32)
    params[2000] = np.nan
    norm = np.ones(70, dtype=np.float32)
    with pytest.raises(ch.ChorusError) as ei:
        ch.chorus_closure_pack(torch.from_numpy(params).cuda(), torch.from_numpy(norm).cuda())
    assert ei.value.status == -5


def test_filter_matches_oracle(ch, cl, oracle_mod, torch_dev):
    torch = torch_dev
    beta = 0.7
    ri, ro = beta / (1 - beta), 1 / (1 - beta)
    m = cubed_sphere_shell(2, 1, ri, ro)
    of, oc = oracle_mod.OracleMesh(m, 6), oracle_mod.OracleMesh(m, 3)
    Q = _state(of, 9, vel=0.3)
    jf, jc = of.geometry()[0], oc.geometry()[0]
    Qb_want, tau_want = cl.sgs_target(Q, jf, jc, 6, 3, oracle_mod.basis(6)[0], oracle_mod.basis(3)[0], 5 / 3)
    mf = ch.mesh_from_arrays(m, 6).upload()
    mc = ch.mesh_from_arrays(m, 3).upload()
    Qb = torch.zeros((5, mc.n_solpts), dtype=torch.float64, device="cuda")
    tau = torch.zeros((15, mc.n_solpts), dtype=torch.float64, device="cuda")
    ch.chorus_closure_filter(mf, mc, 5 / 3, _dev(torch, Q.reshape(5, -1)), Qb, tau)
    torch.cuda.synchronize()
    Qb, tau = Qb.cpu().numpy().reshape(5, -1), tau.cpu().numpy().reshape(15, -1)
    Qb_want, tau_want = Qb_want.reshape(5, -1), tau_want.reshape(15, -1)
    for v in range(5):
        assert np.linalg.norm(Qb[v] - Qb_want[v]) <= 1e-12 * np.linalg.norm(Qb_want[v])
    assert np.abs(tau[0:3]).max() == 0.0
    for k in range(3, 15):
        assert np.linalg.norm(tau[k] - tau_want[k]) <= 1e-10 * np.linalg.norm(tau_want[k]) + 1e-14, k


def test_closure_call_errors(ch, cl, oracle_mod, torch_dev):
    torch = torch_dev
    m, om, pars, Q = _shell_case(oracle_mod)
    model = ch.chorus_closure_pack(torch.from_numpy(mlp_init(18).astype(np.float32)).cuda(),
                                   torch.ones(70, dtype=torch.float32, device="cuda"))
    cm4 = ch.mesh_from_arrays(m, 4).upload()
    phys = ch.physics(GM=pars["GM"], closure=ch.CHORUS_CLOSURE_MLP, closure_model=model)
    ws = cm4.workspace(phys)
    Q4 = torch.ones((5, cm4.n_solpts), dtype=torch.float64, device="cuda")
    with pytest.raises(ch.ChorusError) as ei:
        ch.chorus_sd_residual(cm4, phys, Q4, torch.empty_like(Q4), ws)
    assert ei.value.status == -3
    pm = ch.physics(GM=pars["GM"], closure=ch.CHORUS_CLOSURE_MLP, closure_model=model,
                    precision=ch.CHORUS_MIXED)
    with pytest.raises(ch.ChorusError) as ei:
        ch.chorus_rk_step(cm4, pm, Q4, 1e-3, 1, ws)
    assert ei.value.status == -3
    p0 = ch.physics(GM=pars["GM"], closure=ch.CHORUS_CLOSURE_MLP)
    with pytest.raises(ch.ChorusError) as ei:
        ch.chorus_sd_residual(cm4, p0, Q4, torch.empty_like(Q4), ws)
    assert ei.value.status == -1


@pytest.mark.parametrize("nf,nc", [(3, 2), (4, 2), (5, 2), (6, 2), (4, 3), (5, 3), (6, 3)])
def test_filter_every_order_pair(ch, cl, oracle_mod, torch_dev, nf, nc):
    """Every pair of orders on a box of 15 elements (a last block of the
    kernel that holds several elements is partly empty); FP64 on both sides,
    relative 1e-12 of each component's norm."""
    torch = torch_dev
    m = box_mesh(5, 3, 1, lengths=(1.0, 1.1, 0.9), curve=0.03)
    of, oc = oracle_mod.OracleMesh(m, nf), oracle_mod.OracleMesh(m, nc)
    rng = np.random.default_rng(10 * nf + nc)
    n = of.n_solpts
    Q = np.empty((5, n))
    Q[0] = 1.0 + 0.2 * rng.random(n)
    Q[1:4] = 0.3 * rng.standard_normal((3, n))
    Q[4] = 2.5 + 0.2 * rng.random(n)
    Qb_w, tau_w = cl.sgs_target(Q.reshape(5, of.E, -1), of.geometry()[0], oc.geometry()[0], nf, nc,
                                oracle_mod.basis(nf)[0], oracle_mod.basis(nc)[0], 5 / 3)
    mf, mc = ch.mesh_from_arrays(m, nf).upload(), ch.mesh_from_arrays(m, nc).upload()
    Qb = torch.empty((5, mc.n_solpts), dtype=torch.float64, device="cuda")
    tau = torch.empty((15, mc.n_solpts), dtype=torch.float64, device="cuda")
    ch.chorus_closure_filter(mf, mc, 5 / 3, _dev(torch, Q), Qb, tau)
    torch.cuda.synchronize()
    Qb_w, tau_w = Qb_w.reshape(5, -1), tau_w.reshape(15, -1)
    for v in range(5):
        assert np.linalg.norm(Qb[v].cpu().numpy() - Qb_w[v]) <= 1e-12 * np.linalg.norm(Qb_w[v]), v
    got = tau.cpu().numpy()
    assert np.all(got[0:3] == 0.0)
    for k in range(3, 15):
        assert np.linalg.norm(got[k] - tau_w[k]) <= 1e-12 * np.linalg.norm(tau_w[k]), k
