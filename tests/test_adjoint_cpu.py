"""The hand-written adjoint of the step, checked on the host (double precision) against
central finite differences of the very step body the kernels run. Every Jacobian column
of the state, the commands, the damping and the added mass (through the Coriolis and
current terms and through the mass inverse) is compared."""
import numpy as np
import pytest

import synth
from paper_2503_09203_amd import mgx

DT = 0.01


def class_flat(c, dt=DT, deadzone=None):
    """The host diagnostic's class layout: k-scaled layout columns (with the shaft torque in
    the moment rows), lag factors, dead zones, inertia, r_b, g0, dt, reverse-gain ratios."""
    e = c.e / np.linalg.norm(c.e, axis=1, keepdims=True)
    react = np.zeros(c.m) if c.reaction is None else c.reaction
    Bk = np.zeros((6, 8))
    Bk[:3, :c.m] = (e * c.k[:, None]).T
    Bk[3:, :c.m] = ((np.cross(c.r, e) + react[:, None] * e) * c.k[:, None]).T
    alpha = np.zeros(8)
    alpha[:c.m] = 1 - np.exp(-dt / c.tau)
    dz = np.zeros(8)
    if deadzone is not None:
        dz[:c.m] = deadzone
    rev = np.ones(8)
    if c.k_rev is not None:
        rev[:c.m] = c.k_rev / c.k
    return np.concatenate([Bk.ravel(), alpha, dz, c.inertia, c.rb, [c.g0, dt], rev])


def rec_flat(c, mass, added, dlin, dquad, buoy, current, dt=DT):
    Mrb = np.array([mass] * 3 + list(c.inertia))
    return np.concatenate([dt / (Mrb + added), [mass], added, dlin, dquad, [mass * c.g0 - buoy, buoy], current])


def setup(seed, m=6, omega_scale=1.0, variants=False):
    rng = np.random.default_rng(seed)
    c = synth.draw_class(m, 7)
    if variants:
        c = synth.propeller_variants(c)
    mass, added, dlin, dquad, buoy = c.mass, c.added.copy(), c.dlin.copy(), c.dquad.copy(), c.buoy * 1.01
    current = rng.normal(0, 0.3, 3)
    q = rng.normal(size=4)
    q /= np.linalg.norm(q)
    nu = rng.normal(0, 0.3, 6)
    nu[3:] *= omega_scale
    state = np.concatenate([rng.normal(0, 1, 3), q, nu, rng.uniform(-0.9, 0.9, m)])
    a = rng.uniform(-0.95, 0.95, m)
    xbar = rng.normal(size=13 + m)
    return c, (mass, added, dlin, dquad, buoy, current), state, a, xbar


def fd_columns(fun, x0, h):
    cols = []
    for i in range(len(x0)):
        xp, xm = x0.copy(), x0.copy()
        xp[i] += h
        xm[i] -= h
        cols.append((fun(xp) - fun(xm)) / (2 * h))
    return np.array(cols)  # [n_in, n_out]


@pytest.mark.parametrize("seed,flags,dz,omega,variants", [(0, 0, None, 1.0, False), (1, mgx.FLAG_NO_AMC, None, 1.0, False),
                                                           (2, 0, 0.1, 1.0, False), (3, 0, None, 30.0, False),
                                                           (4, mgx.FLAG_LAG_EULER, None, 1.0, False),
                                                           (6, 0, "class", 1.0, True)])
def test_step_vjp_matches_finite_differences(seed, flags, dz, omega, variants):
    c, prm, state, a, xbar = setup(seed, omega_scale=omega, variants=variants)
    m = c.m
    cls = class_flat(c, deadzone=c.deadzone if dz == "class" else dz)
    if flags & mgx.FLAG_LAG_EULER:
        cls[48:48 + m] = DT / c.tau
    rec = rec_flat(c, *prm)
    s1, xb, ab, gp = mgx.mgx_host_step_vjp(m, flags, cls, rec, state, a, xbar)
    h = 1e-6

    def out_state(x):
        return mgx.mgx_host_step_vjp(m, flags, cls, rec, x, a, xbar)[0]

    J = fd_columns(out_state, state, h)               # d(out)/d(state_i)
    fd_xb = J @ xbar
    scale = np.abs(fd_xb).max()
    assert np.allclose(xb, fd_xb, rtol=1e-5, atol=1e-6 * scale), np.abs(xb - fd_xb).max()

    def out_act(u):
        return mgx.mgx_host_step_vjp(m, flags, cls, rec, state, u, xbar)[0]

    fd_ab = fd_columns(out_act, a, h) @ xbar
    assert np.allclose(ab, fd_ab, rtol=1e-5, atol=1e-6 * np.abs(fd_ab).max())

    mass, added, dlin, dquad, buoy, current = prm

    def out_params(th):
        r = rec_flat(c, mass, th[12:18], th[:6], th[6:12], buoy, current)
        return mgx.mgx_host_step_vjp(m, flags, cls, r, state, a, xbar)[0]

    theta = np.concatenate([dlin, dquad, added])
    fd_th = fd_columns(out_params, theta, 1e-6) @ xbar
    Mrb = np.array([mass] * 3 + list(c.inertia))
    dtMinv = DT / (Mrb + added)
    g_total = np.concatenate([gp[:12], gp[12:18] - gp[18:24] * dtMinv ** 2 / DT])
    sc = np.abs(fd_th).max()
    assert np.allclose(g_total, fd_th, rtol=1e-5, atol=1e-6 * sc), np.abs(g_total - fd_th).max()


@pytest.mark.parametrize("variants", [False, True])
def test_step_body_on_host_is_the_documented_map(variants):
    """The host evaluation of the kernels' step body agrees with the FP64 oracle (same
    inputs in double): both implement the same step, with and without the propeller
    variants (dead zone, reverse gain, shaft torque)."""
    import oracle
    c, prm, state, a, xbar = setup(5, variants=variants)
    mass, added, dlin, dquad, buoy, current = prm
    cls = class_flat(c, deadzone=c.deadzone)
    s1 = mgx.mgx_host_step_vjp(c.m, 0, cls, rec_flat(c, *prm), state, a, xbar)[0]
    p = synth.EnvParams(np.array([mass]), added[:, None], dlin[:, None], dquad[:, None], np.array([buoy]),
                        current[:, None])
    env = oracle.make_envs(c, p, DT)
    x = np.zeros(oracle.STATE_LEN)
    x[:13 + c.m] = state
    ref = oracle.step(env, x, a)
    assert np.allclose(s1, ref[:13 + c.m], rtol=1e-12, atol=1e-14)


@pytest.mark.parametrize("rate", [0.0, 1e-12, 1e-3, 10.0, 49.9, 50.1, 400.0])
@pytest.mark.parametrize("norm2", [1.0, 1.0 + 0.9e-5, 1.0 - 1.1e-5, 4.0])
def test_double_attitude_series_and_their_fallbacks(rate, norm2):
    """The double step's attitude increment and normalisation on both sides of the series'
    limits (50 rad/s at this step, |q|^2 within 1e-5 of 1) against the closed forms: a body
    without forces turns by exp(dt w / 2) and comes out normalised, to 4 units of the last
    place; the adjoint of the attitude against central differences of the closed form."""
    dt, m = 0.01, 1
    w = rate * np.array([0.6, -0.64, 0.48])
    q = np.sqrt(norm2) * np.array([0.5, 0.1, -0.7, 0.5]) / np.linalg.norm([0.5, 0.1, -0.7, 0.5])
    # one idle thruster; no forces reach the body (dt M^-1 = 0)
    cls = np.concatenate([np.zeros(48), np.ones(8), np.zeros(8), np.ones(3), np.zeros(3), [9.81, dt], np.ones(8)])
    rec = np.zeros(30)
    x = np.concatenate([np.zeros(3), q, np.zeros(3), w, np.zeros(m)])

    def turned(w):
        half = 0.5 * dt * np.linalg.norm(w)
        d = np.concatenate([[np.cos(half)], 0.5 * dt * np.sinc(half / np.pi) * w])
        p = np.array([q[0] * d[0] - q[1:] @ d[1:], *(q[0] * d[1:] + d[0] * q[1:] + np.cross(q[1:], d[1:]))])
        return p / np.linalg.norm(p)

    xbar = np.zeros(13 + m)
    xbar[3:7] = [0.3, -0.2, 0.9, 0.4]
    s, xb, _, _ = mgx.mgx_host_step_vjp(m, 0, cls, rec, x, np.zeros(m), xbar)
    np.testing.assert_allclose(s[3:7], turned(w), rtol=0, atol=4 * 2.0 ** -53)
    h = 1e-6 * max(1.0, rate)
    fd = [(turned(w + h * e) - turned(w - h * e)) @ xbar[3:7] / (2 * h) for e in np.eye(3)]
    # rounding 2^-53 / h, and the third derivative (dt / 2)^3 h^2
    np.testing.assert_allclose(xb[10:13], fd, rtol=0, atol=8 * 2.0 ** -53 / h + (0.5 * dt) ** 3 * h * h)


@pytest.mark.parametrize("n,n_pad", [([70], [128]), ([64, 1, 130], [64, 64, 192])])
def test_positions_are_the_gather_of_the_padded_layout(n, n_pad):
    """DiffRollout.positions and its derivatives (reverse, forward, vmap) against the index
    gather it stands for: copies only, so equal."""
    import types

    import torch
    from paper_2503_09203_amd.autograd import DiffRollout
    ro = DiffRollout.__new__(DiffRollout)
    ro.b = types.SimpleNamespace(n=n, n_pad=n_pad)
    off = np.cumsum([0] + n_pad)
    idx = torch.as_tensor(np.concatenate(
        [np.stack([3 * o + j * p + np.arange(k) for j in range(3)]) for k, p, o in zip(n, n_pad, off)], axis=1))
    g = torch.Generator().manual_seed(3)
    x = torch.randn((5, 3 * sum(n_pad)), generator=g)
    v = torch.randn((5, 3, sum(n)), generator=g)
    ref = lambda p: p[:, idx]
    for fn in (lambda f: f(x), lambda f: f(x.t().contiguous().t()), lambda f: torch.func.vjp(f, x)[1](v)[0],
               lambda f: torch.func.jvp(f, (x,), (2 * x,))[1],
               lambda f: torch.func.vmap(f)(torch.stack([x, 2 * x])), lambda f: f(x[..., None].expand(-1, -1, 2))):
        assert torch.equal(fn(ro.positions), fn(ref))
    assert ro.positions(x).data_ptr() != x.data_ptr() and ro.positions(x).is_contiguous()
    with pytest.raises(Exception):
        ro.positions(x[:, :-1 - (n_pad[-1] - n[-1])])


def test_position_index_map():
    """DiffRollout.pos_idx gathers the positions' rows as positions() does."""
    import types

    import torch
    from paper_2503_09203_amd.autograd import DiffRollout
    ro = DiffRollout.__new__(DiffRollout)
    ro.b = types.SimpleNamespace(n=[64, 1, 130], n_pad=[64, 64, 192], device="cpu")
    x = torch.randn((5, 3 * 320), generator=torch.Generator().manual_seed(3))
    assert ro.pos_idx.dtype == torch.int64 and ro.pos_idx.shape == (3, 195)
    assert torch.equal(x[:, ro.pos_idx], ro.positions(x))
