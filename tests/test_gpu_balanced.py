"""Balanced mode (CHORUS_BALANCED): the residual R(Q) - R(Q0) about a
registered background Q0, on both paths, against the oracle's R(Q) - R(Q0)
(the oracle evaluates the residual twice; the subtraction is the whole
definition), and the background as an exact discrete steady state."""
import numpy as np
import pytest

from chorus_inputs import cubed_sphere_shell, uniform_noise

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


def _dev(torch, a):
    return torch.from_numpy(np.ascontiguousarray(a.reshape(5, -1))).cuda()


def _case(oracle_mod, N, seed=4):
    """Shell (beta 0.7, 3 x 2 panels), the polytrope at rest as background,
    the state with an entropy perturbation and a seeded velocity field."""
    beta = 0.7
    ri, ro = beta / (1 - beta), 1 / (1 - beta)
    m = cubed_sphere_shell(3, 2, ri, ro)
    om = oracle_mod.OracleMesh(m, N)
    Q0, pars = om.polytrope(beta, 1.0)
    Q, _ = om.polytrope(beta, 1.0, noise=uniform_noise(om.n_solpts, seed), amp=1e-3)
    rng = np.random.default_rng(seed + 1)
    Q[1:4] = 1e-3 * Q[0] * rng.uniform(-1, 1, size=Q[1:4].shape)
    Q[4] += 0.5 * (Q[1:4] ** 2).sum(0) / Q[0]
    kw = dict(GM=pars["GM"], omega=1.0, nu=1e-3, kappa=1e-3, kappa_r=1e-4, T_top=pars["chi_o"], F_bottom=0.01)
    return m, om, Q0, Q, kw


def _balanced_residual(ch, torch, cm, phys, Q0, Q):
    ws = cm.workspace(phys)
    ch.chorus_set_background(cm, phys, _dev(torch, Q0), ws)
    R = torch.empty_like(_dev(torch, Q))
    ch.chorus_sd_residual(cm, phys, _dev(torch, Q), R, ws)
    torch.cuda.synchronize()
    return R.cpu().numpy(), ws


@pytest.mark.parametrize("N", [3, 4])
def test_balanced_fp64_matches_oracle(ch, oracle_mod, torch_dev, N):
    """FP64: R(Q) - R(Q0) against the oracle's, to 1e-12 of its norm or 2x
    the oracle's one-ulp floor of the difference (L2 and max norm)."""
    from test_gpu_parity import assert_parity, perturbed_oracle, ulp_perturb
    torch = torch_dev
    m, om, Q0, Q, kw = _case(oracle_mod, N)
    cm = ch.mesh_from_arrays(m, N).upload()
    Rg, _ = _balanced_residual(ch, torch, cm, ch.physics(flags=ch.CHORUS_BALANCED, **kw), Q0, Q)
    op = oracle_mod.phys(**kw)
    ref = om.residual(op, Q) - om.residual(op, Q0)
    pom = perturbed_oracle(oracle_mod, m, N)
    pert = pom.residual(op, ulp_perturb(Q)) - pom.residual(op, ulp_perturb(Q0, seed=9))
    assert_parity(Rg, ref, pert, "balanced fp64 N=%d" % N)


@pytest.mark.parametrize("N,panel_n,radial_n", [(3, 13, 3), (4, 13, 2), (6, 9, 2)])
def test_balanced_fp64_on_large_meshes(ch, oracle_mod, torch_dev, N, panel_n, radial_n):
    """The same in the element passes (shells above 10, 7 and 3 elements per
    CU of 256), and one SSPRK(5,4) step, whose fourth stage writes two
    registers: the oracle's stage sums with R(Q) - R(Q0) written out."""
    from test_gpu_parity import assert_parity, perturbed_oracle, ulp_perturb
    torch = torch_dev
    beta, dt = 0.7, 1e-3
    m = cubed_sphere_shell(panel_n, radial_n, beta / (1 - beta), 1 / (1 - beta))
    om = oracle_mod.OracleMesh(m, N)
    assert om.E > 256 * {3: 10, 4: 7, 6: 3}[N]
    Q0, pars = om.polytrope(beta, 1.0)
    Q, _ = om.polytrope(beta, 1.0, noise=uniform_noise(om.n_solpts, 4), amp=1e-3)
    rng = np.random.default_rng(5)
    Q[1:4] = 1e-3 * Q[0] * rng.uniform(-1, 1, size=Q[1:4].shape)
    Q[4] += 0.5 * (Q[1:4] ** 2).sum(0) / Q[0]
    kw = dict(GM=pars["GM"], omega=1.0, nu=1e-3, kappa=1e-3, kappa_r=1e-4, T_top=pars["chi_o"], F_bottom=0.01)
    phys = ch.physics(flags=ch.CHORUS_BALANCED, integrator=ch.CHORUS_SSPRK54, **kw)
    cm = ch.mesh_from_arrays(m, N).upload()
    Rg, ws = _balanced_residual(ch, torch, cm, phys, Q0, Q)
    Qd = _dev(torch, Q)
    ch.chorus_rk_step(cm, phys, Qd, dt, 1, ws)
    torch.cuda.synchronize()
    op = oracle_mod.phys(**kw)
    alpha, bet = oracle_mod.ssp54_table()

    def both(mesh, q, q0):
        r0 = mesh.residual(op, q0)
        u, L = [q], []
        for i in range(5):
            L.append(mesh.residual(op, u[i]) - r0)
            u.append(sum(alpha[i, k] * u[k] + dt * bet[i, k] * L[k] for k in range(i + 1)))
        return L[0], (u[5] - q).reshape(5, -1)
    ref, step = both(om, Q, Q0)
    pert, pstep = both(perturbed_oracle(oracle_mod, m, N), ulp_perturb(Q), ulp_perturb(Q0, seed=9))
    assert_parity(Rg, ref, pert, "balanced fp64 N=%d E=%d" % (N, om.E))
    assert_parity(Qd.cpu().numpy() - Q.reshape(5, -1), step, pstep, "balanced step N=%d E=%d" % (N, om.E))


@pytest.mark.parametrize("N", [3, 4])
def test_balanced_mixed_matches_oracle(ch, oracle_mod, torch_dev, N):
    """Mixed: the FP32 perturbation residual alone against the oracle's
    R(Q) - R(Q0): L2 2e-5 and max-norm 1e-4 relative per variable."""
    torch = torch_dev
    m, om, Q0, Q, kw = _case(oracle_mod, N)
    cm = ch.mesh_from_arrays(m, N).upload()
    Rg, _ = _balanced_residual(ch, torch, cm, ch.physics(precision=ch.CHORUS_MIXED, flags=ch.CHORUS_BALANCED,
                                                          **kw), Q0, Q)
    op = oracle_mod.phys(**kw)
    ref = (om.residual(op, Q) - om.residual(op, Q0)).reshape(5, -1)
    for v in range(5):
        d = Rg[v] - ref[v]
        l2 = np.linalg.norm(d) / np.linalg.norm(ref[v])
        mx = np.abs(d).max() / np.abs(ref[v]).max()
        print("balanced mixed N=%d var %d: L2 %.2e max %.2e" % (N, v, l2, mx))
        assert l2 <= 2e-5 and mx <= 1e-4, (v, l2, mx)


@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_balanced_background_is_steady(ch, oracle_mod, torch_dev, precision):
    """The registered background is a discrete steady state: the balanced
    residual at Q = Q0 is exactly zero, and three SSP-RK3 steps from Q0
    leave it unchanged to rounding.  Without the flag the same background
    has a truncation-sized residual."""
    torch = torch_dev
    m, om, Q0, _, kw = _case(oracle_mod, 3)
    cm = ch.mesh_from_arrays(m, 3).upload()
    prec = ch.CHORUS_MIXED if precision == "mixed" else ch.CHORUS_FP64
    phys = ch.physics(precision=prec, flags=ch.CHORUS_BALANCED, **kw)
    R, ws = _balanced_residual(ch, torch, cm, phys, Q0, Q0)
    assert np.array_equal(R, np.zeros_like(R)), np.abs(R).max()
    Qd = _dev(torch, Q0)
    ch.chorus_rk_step(cm, phys, Qd, 0.01, 3, ws)
    torch.cuda.synchronize()
    Q0r = Q0.reshape(5, -1)
    # momentum is zero in Q0: measured against the density scale
    scale = np.maximum(np.abs(Q0r).max(axis=1), np.abs(Q0r[0]).max())
    dev = np.abs(Qd.cpu().numpy() - Q0r).max(axis=1) / scale
    print("%s: max relative change of the background over 3 balanced steps: %s" % (precision, dev))
    assert (dev <= 1e-14).all(), dev
    Rp = om.residual(oracle_mod.phys(**kw), Q0).reshape(5, -1)
    assert np.abs(Rp[1:4]).max() > 1e-6  # the imbalance the flag removes


def test_balanced_call_order_errors(ch, oracle_mod, torch_dev):
    """The FP64 path with the flag needs a background registered with this
    workspace and the same physics; a background registered without the flag
    does not serve a balanced call, nor the other way round."""
    torch = torch_dev
    m, om, Q0, Q, kw = _case(oracle_mod, 3)
    cm = ch.mesh_from_arrays(m, 3).upload()
    bal = ch.physics(flags=ch.CHORUS_BALANCED, **kw)
    plain = ch.physics(**kw)
    ws = cm.workspace(bal)
    R = torch.empty_like(_dev(torch, Q))
    with pytest.raises(ch.ChorusError) as ei:
        ch.chorus_sd_residual(cm, bal, _dev(torch, Q), R, ws)
    assert ei.value.status == -6
    ch.chorus_set_background(cm, plain, _dev(torch, Q0), ws)
    with pytest.raises(ch.ChorusError) as ei:
        ch.chorus_rk_step(cm, bal, _dev(torch, Q), 1e-3, 1, ws)
    assert ei.value.status == -6
    ch.chorus_set_background(cm, bal, _dev(torch, Q0), ws)
    ch.chorus_sd_residual(cm, bal, _dev(torch, Q), R, ws)
    mx = ch.physics(precision=ch.CHORUS_MIXED, **kw)
    with pytest.raises(ch.ChorusError) as ei:
        ch.chorus_sd_residual(cm, mx, _dev(torch, Q), R, ws)
    assert ei.value.status == -6
