"""GPU parity of the viscous part of the right-hand side (Sec. II.B: the diffusion term of
Eq. 5 by particle strength exchange, Vreman's sub-grid viscosity) and of the velocity
gradient it needs, against the FP64 oracle: element-wise at sizes the oracle finishes in
seconds (several tiles plus a ragged tail), on sampled outputs at the benchmark's full size,
and through properties (conservation, the closed-form Gaussian limit)."""
import numpy as np
import pytest

import oracle
import paper_2511_11430_amd as vpm
from paper_2511_11430_amd import workloads as W

from gpu_helpers import TOL, dev, host, prepare, rel_l2, say

pytestmark = pytest.mark.gpu
KINDS = ["f64", "f32c"]


def _random_set(n, seed, spread=0.3):
    rng = np.random.default_rng([5151, seed])
    x = rng.uniform(-spread, spread, (3, n))
    g = rng.normal(0, 1e-3, (3, n))
    s = rng.uniform(0.02, 0.06, n)
    return x, g, s


def _J(grad):
    """(9, n) row-major gradients to (3, 3, n)."""
    return host(grad).reshape(3, 3, -1)


# ------------------------------------------------------------------ velocity gradient

@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [2, 37, 1537])
@pytest.mark.parametrize("scheme,rule", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_gradient_small_sets(kind, n, scheme, rule, gpu):
    x, g, s = prepare(_random_set(n, n), kind)
    say(f"gradient {kind} n={n} scheme={scheme} rule={rule}")
    u, d, J = vpm.vpm_eval_velocity_gradient(dev(x, kind), dev(g, kind), dev(s, kind), scheme=scheme,
                                             sigma_rule=rule)
    uo, do = oracle.eval_pairs(x, g, s, scheme=scheme, sigma_rule=rule)
    Jo = oracle.velocity_gradient(x, g, s, sigma_rule=rule)
    assert rel_l2(host(u), uo) <= TOL[kind]
    assert rel_l2(host(d), do) <= TOL[kind]
    assert rel_l2(_J(J), Jo) <= TOL[kind]


@pytest.mark.parametrize("kind", KINDS)
def test_gradient_agrees_with_the_stretching_call(kind, gpu):
    c = W.config2(n=20000)
    x, g, s = prepare([c["x"], c["gamma"], c["sigma"]], kind)
    X, G, S = dev(x, kind), dev(g, kind), dev(s, kind)
    u0, d0 = vpm.vpm_eval_velocity_stretching(X, G, S)
    u1, d1, J = vpm.vpm_eval_velocity_gradient(X, G, S)
    say(f"gradient vs stretching call {kind}")
    assert rel_l2(host(u1), host(u0)) <= TOL[kind]
    assert rel_l2(host(d1), host(d0)) <= TOL[kind]
    # the divergence of the velocity vanishes: tr J is rounding-level against |J|
    Jh = _J(J)
    tr = np.einsum("aat->t", Jh)
    assert np.linalg.norm(tr) <= 10 * TOL[kind] * np.linalg.norm(Jh)


@pytest.mark.parametrize("kind", KINDS)
def test_gradient_source_split_and_batched(kind, gpu):
    import torch
    c = W.config2(n=20000)
    x, g, s = prepare([c["x"], c["gamma"], c["sigma"]], kind)
    X, G, S = dev(x, kind), dev(g, kind), dev(s, kind)
    # 64 particles as explicit targets, each skipping itself: a small target set whose sources
    # are split into chunks (partial sums in the workspace)
    idx = np.sort(np.random.default_rng(8).choice(x.shape[1], 64, replace=False))
    ex = torch.tensor(idx, dtype=torch.int32, device="cuda")
    need = vpm.vpm_workspace_size(vpm.F64 if kind == "f64" else vpm.F32C, [0, x.shape[1]], [0, 64],
                                  self_eval=False, gradient=True)
    assert need > 0
    say(f"gradient split {kind} workspace {need}")
    u, d, J = vpm.vpm_eval_velocity_gradient(X, G, S, dev(x[:, idx], kind), dev(g[:, idx], kind),
                                             dev(s[idx], kind), tgt_exclude=ex)
    uo, do = oracle.eval_pairs(x, g, s, x_tgt=x[:, idx], gam_tgt=g[:, idx], excl=idx)
    Jo = oracle.velocity_gradient(x, g, s, x_tgt=x[:, idx], excl=idx)
    assert rel_l2(host(u), uo) <= TOL[kind]
    assert rel_l2(host(d), do) <= TOL[kind]
    assert rel_l2(_J(J), Jo) <= TOL[kind]
    # three independent sets in one persistent launch
    sizes = [700, 2300, 1100]
    sets = [prepare(_random_set(m, 100 + k), kind) for k, m in enumerate(sizes)]
    xb = np.concatenate([a[0] for a in sets], 1)
    gb = np.concatenate([a[1] for a in sets], 1)
    sb = np.concatenate([a[2] for a in sets])
    off = [0, *np.cumsum(sizes).tolist()]
    say(f"gradient batched {kind} sizes {sizes}")
    u, d, J = vpm.vpm_eval_velocity_gradient(dev(xb, kind), dev(gb, kind), dev(sb, kind), src_off=off)
    Jh = _J(J)
    for k in range(3):
        a, b = off[k], off[k + 1]
        Jo = oracle.velocity_gradient(xb[:, a:b], gb[:, a:b], sb[a:b])
        _, do = oracle.eval_pairs(xb[:, a:b], gb[:, a:b], sb[a:b])
        assert rel_l2(Jh[:, :, a:b], Jo) <= TOL[kind]
        assert rel_l2(host(d)[:, a:b], do) <= TOL[kind]


@pytest.mark.parametrize("kind", KINDS)
def test_gradient_full_size_sampled(kind, gpu):
    c = W.config3()
    x, g, s = prepare([c["x"], c["gamma"], c["sigma"]], kind)
    say(f"gradient config3 {kind} N={x.shape[1]}")
    u, d, J = vpm.vpm_eval_velocity_gradient(dev(x, kind), dev(g, kind), dev(s, kind))
    idx = c["sample"][:: 32]  # 128 of the seeded sample targets
    Jo = oracle.velocity_gradient(x, g, s, x_tgt=x[:, idx], excl=idx)
    _, do = oracle.eval_pairs(x, g, s, x_tgt=x[:, idx], gam_tgt=g[:, idx], excl=idx)
    eJ, ed = rel_l2(_J(J)[:, :, idx], Jo), rel_l2(host(d)[:, idx], do)
    say(f"config3 gradient {kind}: rel-L2 J {eJ:.3e} dgamma {ed:.3e}")
    assert eJ <= TOL[kind] and ed <= TOL[kind]


# ------------------------------------------------------------------ Vreman

@pytest.mark.parametrize("kind", KINDS)
def test_vreman(kind, gpu):
    rng = np.random.default_rng(17)
    n = 3001
    Jn = rng.normal(size=(3, 3, n)) * 10.0 ** rng.uniform(-2, 3, size=n)
    Jn[:, :, 0] = 0.0               # zero gradient
    Jn[:, :, 1] = 0.0
    Jn[0, 1, 1] = 4.0               # pure shear: the model vanishes
    sig = rng.uniform(0.01, 0.05, n)
    Jn, sig = prepare([Jn.reshape(9, n), sig], kind)
    say(f"vreman {kind} n={n}")
    nut = vpm.vpm_sgs_vreman(dev(Jn, kind), dev(sig, kind), W.C_V)
    ref = oracle.vreman(Jn.reshape(3, 3, n), sig, W.C_V)
    got = host(nut)
    assert got[0] == 0.0 and got[1] == 0.0
    assert rel_l2(got, ref) <= TOL[kind]


# ------------------------------------------------------------------ PSE

@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n", [1, 37, 1537])
@pytest.mark.parametrize("with_nut", [False, True])
def test_pse_small_sets(kind, n, with_nut, gpu):
    x, g, s = _random_set(n, 40 + n, spread=0.08)
    rng = np.random.default_rng([77, n])
    vol = W.particle_volume(s) * rng.uniform(0.5, 1.5, n)
    nut = W.eddy_viscosity_field(n, n) if with_nut else None
    arrs = prepare([x, g, s, vol] + ([nut] if with_nut else []), kind)
    x, g, s, vol = arrs[:4]
    nut = arrs[4] if with_nut else None
    say(f"pse {kind} n={n} nu_t={with_nut}")
    d = vpm.vpm_eval_diffusion(dev(x, kind), dev(g, kind), dev(s, kind), dev(vol, kind), W.NU_AIR,
                               None if nut is None else dev(nut, kind))
    do = oracle.pse(x, g, s, vol, W.NU_AIR, nut)
    if n == 1:
        assert np.all(host(d) == 0.0)
        return
    assert rel_l2(host(d), do) <= TOL[kind]


def test_pse_gaussian_lattice_closed_form(gpu):
    """FP64 PSE of a Gaussian vorticity field on a lattice equals the closed-form convolution
    (2 nu / sigma^2) [(zeta_sigma * omega) - omega] V up to the spectrally small lattice error."""
    h, sig, L, nu, w0, M = 1.0, 1.5, 2.0, 1.5e-5, 0.7, 14
    k = np.arange(-M, M + 1) * h
    X, Y, Z = np.meshgrid(k, k, k, indexing="ij")
    x = np.stack([X.ravel(), Y.ravel(), Z.ravel()])
    n = x.shape[1]
    r2 = (x ** 2).sum(0)
    om = w0 * np.exp(-r2 / (2 * L * L))
    gam = np.zeros((3, n))
    gam[2] = om * h ** 3
    say(f"pse lattice n={n}")
    d = host(vpm.vpm_eval_diffusion(dev(x, "f64"), dev(gam, "f64"), dev(np.full(n, sig), "f64"),
                                    dev(np.full(n, h ** 3), "f64"), nu))
    conv = w0 * (L * L / (L * L + sig * sig)) ** 1.5 * np.exp(-r2 / (2 * (L * L + sig * sig)))
    ref = 2 * nu / sig ** 2 * (conv - om) * h ** 3
    inner = r2 <= (2 * L) ** 2
    assert np.abs(d[2, inner] - ref[inner]).max() <= 1e-9 * np.abs(ref[inner]).max()
    assert np.abs(d[:2]).max() <= 1e-12 * np.abs(ref).max()


@pytest.mark.parametrize("kind", KINDS)
def test_pse_batched_and_accumulate(kind, gpu):
    import torch
    sizes = [300, 1800, 5, 900]
    sets = [_random_set(m, 200 + k, spread=0.06) for k, m in enumerate(sizes)]
    x = np.concatenate([a[0] for a in sets], 1)
    g = np.concatenate([a[1] for a in sets], 1)
    s = np.concatenate([a[2] for a in sets])
    vol = W.particle_volume(s)
    x, g, s, vol = prepare([x, g, s, vol], kind)
    off = [0, *np.cumsum(sizes).tolist()]
    base = np.random.default_rng(5).normal(0, 1e-3, (3, x.shape[1]))
    base = prepare([base], kind)[0]
    out = dev(base, kind)
    say(f"pse batched {kind} sizes {sizes}")
    vpm.vpm_eval_diffusion(dev(x, kind), dev(g, kind), dev(s, kind), dev(vol, kind), W.NU_AIR, dgamma_out=out,
                           accumulate=True, off=off)
    torch.cuda.synchronize()
    got = host(out) - base
    for k in range(len(sizes)):
        a, b = off[k], off[k + 1]
        do = oracle.pse(x[:, a:b], g[:, a:b], s[a:b], vol[a:b], W.NU_AIR)
        # the accumulated result is compared after removing the base it was added to
        assert np.linalg.norm(got[:, a:b] - do) <= TOL[kind] * np.linalg.norm(do) + \
            4 * np.finfo(np.float32 if kind == "f32c" else np.float64).eps * np.linalg.norm(base[:, a:b])


@pytest.mark.parametrize("kind", KINDS)
def test_pse_full_size_sampled_and_conservation(kind, gpu):
    c = W.config3()
    n = c["x"].shape[1]
    vol = W.particle_volume(c["sigma"])
    nut = W.eddy_viscosity_field(n, 3)
    x, g, s, vol, nut = prepare([c["x"], c["gamma"], c["sigma"], vol, nut], kind)
    say(f"pse config3 {kind} N={n}")
    d = host(vpm.vpm_eval_diffusion(dev(x, kind), dev(g, kind), dev(s, kind), dev(vol, kind), W.NU_AIR,
                                    dev(nut, kind)))
    idx = c["sample"][:: 16]
    do = oracle.pse(x, g, s, vol, W.NU_AIR, nut, targets=idx)
    e = rel_l2(d[:, idx], do)
    tot = np.abs(d.sum(1)).max() / np.abs(d).sum(1).max()
    say(f"config3 pse {kind}: rel-L2 {e:.3e}, |sum dGamma| / sum |dGamma| {tot:.3e}")
    assert e <= TOL[kind]
    assert tot <= (1e-13 if kind == "f64" else 1e-5)


@pytest.mark.parametrize("kind", KINDS)
def test_viscous_chain_small(kind, gpu):
    """gradient -> Vreman -> PSE on one set, each side computing its own eddy viscosity."""
    c = W.config2(n=4000)
    vol = W.particle_volume(c["sigma"])
    x, g, s, vol = prepare([c["x"], c["gamma"], c["sigma"], vol], kind)
    X, G, S, V = dev(x, kind), dev(g, kind), dev(s, kind), dev(vol, kind)
    say(f"viscous chain {kind}")
    _, d, J = vpm.vpm_eval_velocity_gradient(X, G, S)
    nut = vpm.vpm_sgs_vreman(J, S, W.C_V)
    vpm.vpm_eval_diffusion(X, G, S, V, W.NU_AIR, nut, dgamma_out=d, accumulate=True)
    Jo = oracle.velocity_gradient(x, g, s)
    nuto = oracle.vreman(Jo, s, W.C_V)
    _, do = oracle.eval_pairs(x, g, s)
    do = do + oracle.pse(x, g, s, vol, W.NU_AIR, nuto)
    assert rel_l2(host(nut), nuto) <= TOL[kind]
    assert rel_l2(host(d), do) <= TOL[kind]


@pytest.mark.parametrize("kind", KINDS)
# a group of 64 targets and its neighbours, one tile of 256 records per wavefront and one more, and
# both widths of the workgroup
@pytest.mark.parametrize("n", [63, 65, 257, 1025, 4097, 65601])
def test_diffusion_at_group_sizes(kind, n, gpu):
    rng = np.random.default_rng([41, n])
    if n < 10000:
        x, g, s = _random_set(n, 43)
    else:
        w = W.hover_wake(n, 1, 0.02, 10, rng)
        x, g, s = w["x"], w["gamma"], w["sigma"]
    x, g, s, vol, nut = prepare([x, g, s, W.particle_volume(s), rng.uniform(0.0, 1e-4, n)], kind)
    say(f"diffusion {kind} n={n}")
    d = vpm.vpm_eval_diffusion(dev(x, kind), dev(g, kind), dev(s, kind), dev(vol, kind), W.NU_AIR, dev(nut, kind))
    idx = np.unique(np.concatenate([[0, n - 1], rng.integers(0, n, 300)]))
    ref = oracle.pse(x, g, s, vol, W.NU_AIR, nut, targets=idx)
    assert rel_l2(host(d)[:, idx], ref) <= TOL[kind]


def test_diffusion_in_more_than_one_launch(gpu):
    """More target groups than one launch takes (2^18 of 64): random targets of a scattered set, and the last
    ones of the sorted order, which the second launch has."""
    n = 17_000_003
    rng = np.random.default_rng(47)
    x = rng.uniform(0.0, 1.0, (3, n))
    g, s = rng.normal(0, 1e-6, (3, n)), np.full(n, 7e-4)
    x, g, s, vol = prepare([x, g, s, np.full(n, 1.0 / n)], "f32c")
    say(f"diffusion n={n}")
    d = vpm.vpm_eval_diffusion(dev(x, "f32c"), dev(g, "f32c"), dev(s, "f32c"), dev(vol, "f32c"), W.NU_AIR)
    # the last of the Morton order lie at the far corner
    last = np.argsort(x.sum(0))[-40:]
    idx = np.unique(np.concatenate([[0, n - 1], last, rng.integers(0, n, 60)]))
    ref = oracle.pse(x, g, s, vol, W.NU_AIR, targets=idx)
    assert rel_l2(host(d)[:, idx], ref) <= TOL["f32c"]
    assert rel_l2(host(d)[:, last], oracle.pse(x, g, s, vol, W.NU_AIR, targets=last)) <= TOL["f32c"]
