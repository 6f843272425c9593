"""GPU parity of the Cartesian FMM (Sec. II.B) against the FP64 oracle FMM (same tree, same
expansions: equal to rounding), its limits (no far field: the direct sum), edge cases, and at
full size its error against the direct sums."""
import time

import numpy as np
import pytest

import oracle
import paper_2511_11430_amd as vpm
from paper_2511_11430_amd import workloads as W

from gpu_helpers import TOL, dev, host, prepare, rel_l2, say

pytestmark = pytest.mark.gpu
KINDS = ["f64", "f32c"]


def _wake(n, kind, seed_n=None):
    c = W.config3(n=n)
    return prepare([c["x"], c["gamma"], c["sigma"]], kind)


@pytest.mark.parametrize("kind", KINDS)
# orders 1 and 2: the M2L's per-group sums outgrow its LDS grid; 15 to 20: one group per
# workgroup whose wavefronts share the terms' walks in pieces (every such order, grids beyond
# 64 KiB from 18 on); depth 7: mostly single-particle leaves
@pytest.mark.parametrize("level,order", [(2, 4), (3, 8), (4, 6), (4, 12), (6, 5), (3, 1), (3, 2), (3, 16), (5, 14),
                                         (7, 3), (3, 18), (2, 20), (3, 20), (2, 15), (2, 17), (2, 19)])
def test_fmm_matches_oracle_fmm(kind, level, order, gpu):
    x, g, s = _wake(4999, kind)
    say(f"fmm {kind} level={level} order={order}")
    u, d = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), level, order)
    uo, do = oracle.fmm(x, g, s, level, order)
    eu, ed = rel_l2(host(u), uo), rel_l2(host(d), do)
    say(f"  rel-L2 u {eu:.2e} dgamma {ed:.2e}")
    assert eu <= TOL[kind] and ed <= TOL[kind]


@pytest.mark.parametrize("kind", KINDS)
def test_fmm_classical_scheme(kind, gpu):
    x, g, s = _wake(3001, kind)
    u, d = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), 3, 7, scheme=vpm.CLASSICAL)
    uo, do = oracle.fmm(x, g, s, 3, 7, oracle.CLASSICAL)
    assert rel_l2(host(u), uo) <= TOL[kind] and rel_l2(host(d), do) <= TOL[kind]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("level", [0, 1])
def test_fmm_without_far_field_equals_direct(kind, level, gpu):
    x, g, s = _wake(2500, kind)
    u, d = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), level, 4)
    uo, do = oracle.eval_pairs(x, g, s)
    assert rel_l2(host(u), uo) <= TOL[kind] and rel_l2(host(d), do) <= TOL[kind]


@pytest.mark.parametrize("kind", KINDS)
def test_fmm_edge_cases(kind, gpu):
    import torch
    tdt = torch.float64 if kind == "f64" else torch.float32
    # no particles
    z = torch.zeros((3, 0), dtype=tdt, device="cuda")
    u, d = vpm.vpm_fmm_eval(z, z.clone(), torch.zeros(0, dtype=tdt, device="cuda"), 4, 8)
    assert u.shape == (3, 0)
    # one particle: nothing acts on it
    one = dev(np.array([[0.3], [0.1], [-0.2]]), kind)
    u, d = vpm.vpm_fmm_eval(one, dev(np.ones((3, 1)), kind), dev(np.array([0.05]), kind), 3, 6)
    assert np.all(host(u) == 0) and np.all(host(d) == 0)
    # all particles at one point (empty box) and a strided view with ld > n
    rng = np.random.default_rng(4)
    x = np.zeros((3, 40)) + 0.5
    g, s = rng.normal(size=(3, 40)), np.full(40, 0.1)
    u, d = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), 5, 4)
    uo, do = oracle.fmm(x, g, s, 5, 4)
    assert rel_l2(host(u), uo) <= TOL[kind] and rel_l2(host(d), do) <= TOL[kind]
    xs, gs, ss = _wake(1700, kind)
    X = torch.zeros((3, 1800), dtype=tdt, device="cuda")
    G = torch.zeros_like(X)
    X[:, :1700] = dev(xs, kind)
    G[:, :1700] = dev(gs, kind)
    u, d = vpm.vpm_fmm_eval(X[:, :1700], G[:, :1700], dev(ss, kind), 3, 6)
    uo, do = oracle.fmm(xs, gs, ss, 3, 6)
    assert rel_l2(host(u), uo) <= TOL[kind] and rel_l2(host(d), do) <= TOL[kind]


@pytest.mark.parametrize("kind", KINDS)
# more particles than the near field gives sixteen wavefronts per 64 targets; leaves from one
# particle to many units; every width of the M2L's term blocks
@pytest.mark.parametrize("level,order", [(4, 4), (4, 8), (5, 10), (4, 12), (4, 14)])
def test_fmm_many_units_matches_oracle_fmm(kind, level, order, gpu):
    x, g, s = _wake(33001, kind)
    say(f"fmm units {kind} level={level} order={order}")
    u, d, J = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), level, order, want_grad=True)
    u2, d2 = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), level, order)
    uo, do, Jo = oracle.fmm(x, g, s, level, order, want_grad=True)
    for got, ref in ((u, uo), (d, do), (J, Jo.reshape(9, -1)), (u2, uo), (d2, do)):
        assert rel_l2(host(got), ref) <= TOL[kind]


@pytest.mark.parametrize("kind", KINDS)
# one tile of the sort, whole and with an empty part; one, two, three and four levels above the tile
@pytest.mark.parametrize("n", [1023, 1025, 2048, 2049, 8191, 8193, 16385])
def test_fmm_at_sort_sizes(kind, n, gpu):
    x, g, s = _wake(n, kind)
    order = np.random.default_rng([53, n]).permutation(x.shape[1])
    x, g, s = x[:, order], g[:, order], s[order]
    say(f"fmm sort {kind} n={n}")
    u, d = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), 6, 2)
    uo, do = oracle.fmm(x, g, s, 6, 2)
    assert rel_l2(host(u), uo) <= TOL[kind] and rel_l2(host(d), do) <= TOL[kind]


def test_fmm_full_size_against_direct(gpu):
    """The 1,048,576-particle forward-flight wake at depth 6 (leaf width 6.5 sigma_max) and
    orders 12 and 18: the FP32C FMM against the FP64 oracle's direct sums at 512 sampled
    particles, and against the GPU's direct FP32C sums on every particle; order 18 within 1e-5
    for both outputs."""
    import torch
    c = W.config3()
    x, g, s = prepare([c["x"], c["gamma"], c["sigma"]], "f32c")
    X, G, S = dev(x, "f32c"), dev(g, "f32c"), dev(s, "f32c")
    ws = torch.empty(vpm.vpm_fmm_workspace_size(X.shape[1], 6, 12, torch.float32), dtype=torch.uint8, device="cuda")
    u, d = vpm.vpm_fmm_eval(X, G, S, 6, 12, workspace=ws)
    torch.cuda.synchronize()
    t = time.perf_counter()
    u, d = vpm.vpm_fmm_eval(X, G, S, 6, 12, workspace=ws, u_out=u, dgamma_out=d)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t) * 1e3
    ud, dd = vpm.vpm_eval_velocity_stretching(X, G, S)
    eu, ed = rel_l2(host(u), host(ud)), rel_l2(host(d), host(dd))
    idx = np.sort(np.random.default_rng(7).choice(x.shape[1], 512, replace=False))
    uo, do = oracle.eval_pairs(x, g, s, x_tgt=x[:, idx], gam_tgt=g[:, idx], excl=idx)
    su, sd = rel_l2(host(u)[:, idx], uo), rel_l2(host(d)[:, idx], do)
    say(f"fmm 1M: {ms:.1f} ms; vs direct GPU u {eu:.2e} dgamma {ed:.2e}; vs oracle (512) u {su:.2e} dgamma {sd:.2e}")
    assert np.all(np.isfinite(host(u))) and np.all(np.isfinite(host(d)))
    # truncation of the far field: about x0.6 per order on this wake (measured 2.5e-5 and
    # 1.0e-4 at order 12)
    assert max(eu, su) <= 1e-4 and max(ed, sd) <= 3e-4
    # and it converges at full size: order 8 is clearly worse
    u8, d8 = vpm.vpm_fmm_eval(X, G, S, 6, 8)
    e8 = max(rel_l2(host(u8), host(ud)), rel_l2(host(d8), host(dd)))
    say(f"  order 8: {e8:.2e}")
    assert e8 > 3 * max(eu, ed)
    del ws
    # order 18 is the setting within the direct path's 1e-5 for both outputs (measured 1.6e-6
    # and 8.6e-6 against the direct FP32C sums), here also against the oracle's sample
    ws18 = torch.empty(vpm.vpm_fmm_workspace_size(X.shape[1], 6, 18, torch.float32), dtype=torch.uint8,
                       device="cuda")
    u18, d18 = vpm.vpm_fmm_eval(X, G, S, 6, 18, workspace=ws18)
    e18u, e18d = rel_l2(host(u18), host(ud)), rel_l2(host(d18), host(dd))
    s18u, s18d = rel_l2(host(u18)[:, idx], uo), rel_l2(host(d18)[:, idx], do)
    say(f"  order 18: vs direct GPU u {e18u:.2e} dgamma {e18d:.2e}; vs oracle (512) u {s18u:.2e} dgamma {s18d:.2e}")
    assert max(e18u, e18d, s18u, s18d) <= 1e-5


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("scheme", [vpm.TRANSPOSED, vpm.CLASSICAL])
@pytest.mark.parametrize("level,order", [(1, 4), (3, 8), (4, 10)])
def test_fmm_velocity_gradient_matches_oracle(kind, scheme, level, order, gpu):
    x, g, s = _wake(3333, kind)
    u, d, J = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), level, order, scheme=scheme, want_grad=True)
    uo, do, Jo = oracle.fmm(x, g, s, level, order, scheme, want_grad=True)
    eu, ed, ej = rel_l2(host(u), uo), rel_l2(host(d), do), rel_l2(host(J), Jo.reshape(9, -1))
    say(f"fmm grad {kind} scheme={scheme} level={level} order={order}: u {eu:.1e} dgamma {ed:.1e} J {ej:.1e}")
    assert max(eu, ed, ej) <= TOL[kind]


def test_fmm_velocity_gradient_full_size(gpu):
    """1M wake, depth 6, order 12: J against the direct gradient kernel, and the viscous
    right-hand side built on it (Vreman, PSE) against the one built on the direct gradient."""
    import torch
    c = W.config3()
    x, g, s = prepare([c["x"], c["gamma"], c["sigma"]], "f32c")
    X, G, S = dev(x, "f32c"), dev(g, "f32c"), dev(s, "f32c")
    u, d, J = vpm.vpm_fmm_eval(X, G, S, 6, 12, want_grad=True)
    torch.cuda.synchronize()
    t = time.perf_counter()
    vpm.vpm_fmm_eval(X, G, S, 6, 12, u_out=u, dgamma_out=d, grad_out=J)
    torch.cuda.synchronize()
    ms = (time.perf_counter() - t) * 1e3
    ud, dd, Jd = vpm.vpm_eval_velocity_gradient(X, G, S)
    ej = rel_l2(host(J), host(Jd))
    nut_f = vpm.vpm_sgs_vreman(J, S, W.C_V)
    nut_d = vpm.vpm_sgs_vreman(Jd, S, W.C_V)
    en = rel_l2(host(nut_f), host(nut_d))
    say(f"fmm 1M with gradient: {ms:.1f} ms; J vs direct {ej:.2e}; Vreman nu_t {en:.2e}")
    assert ej <= 3e-4 and en <= 3e-4


def _helix(n):
    """Particles along a helix, most of them alone in a cell of the deepest grid (1024 per axis)."""
    t = (np.arange(n) + 0.5) / n
    rng = np.random.default_rng(n)
    x = np.stack([0.5 * np.cos(6 * np.pi * t), 0.5 * np.sin(6 * np.pi * t), t - 0.5])
    return x, rng.normal(0, 1e-3, (3, n)), rng.uniform(1e-4, 2e-4, n)


def _cube(n):
    rng = np.random.default_rng(n)
    return rng.uniform(-1.0, 1.0, (3, n)), rng.normal(0, 1e-3, (3, n)), rng.uniform(0.005, 0.01, n)


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("scheme", [vpm.TRANSPOSED, vpm.CLASSICAL])
# more occupied cells on several levels, work items and 64-particle units than the launches have workgroups
# (4096, and 16384 wavefronts for the units' boxes): every kernel takes further ones in strides
@pytest.mark.parametrize("make,n,level,order", [(_cube, 20001, 6, 3), (_helix, 9001, 10, 7)])
def test_fmm_of_more_cells_than_workgroups(kind, scheme, make, n, level, order, gpu):
    x, g, s = prepare(make(n), kind)
    lo, hi = x.min(1), x.max(1)
    half = (hi - lo).max() / 2
    cell = np.floor((x - ((lo + hi) / 2 - half)[:, None]) / (2 * half / 2 ** level)).clip(0, 2 ** level - 1)
    leaves = len(np.unique(cell, axis=1).T)
    say(f"fmm many cells {kind} {make.__name__} level={level} order={order}: {leaves} leaves")
    assert leaves > (16384 if make is _cube else 8000)
    u, d, J = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), level, order, scheme=scheme, want_grad=True)
    uo, do, Jo = oracle.fmm(x, g, s, level, order, scheme, want_grad=True)
    assert rel_l2(host(u), uo) <= TOL[kind] and rel_l2(host(d), do) <= TOL[kind]
    assert rel_l2(host(J).reshape(9, -1), Jo.reshape(9, -1)) <= TOL[kind]
    u, d = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), level, order, scheme=scheme)
    assert rel_l2(host(u), uo) <= TOL[kind] and rel_l2(host(d), do) <= TOL[kind]


def test_high_order_fmm_of_more_cells_than_workgroups(gpu):
    """The same for the M2L of orders from 13 on (the oracle takes most of the time: one evaluation, at inputs
    that both types hold)."""
    x, g, s = prepare(_helix(4601), "f32c")
    say("fmm many cells, order 13")
    uo, do = oracle.fmm(x, g, s, 10, 13)
    for kind in KINDS:
        u, d = vpm.vpm_fmm_eval(dev(x, kind), dev(g, kind), dev(s, kind), 10, 13)
        assert rel_l2(host(u), uo) <= TOL[kind] and rel_l2(host(d), do) <= TOL[kind]
