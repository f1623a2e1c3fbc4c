"""GPU parity of scenario A (lead time, FIFO) through the C ABI against the oracle.

Tolerances (normwise, relative to max |V| of the oracle):
  FP64 backup       1e-12  (same arithmetic up to summation order)
  FP32 storage      1e-6   per sweep (FP32 rounding of V plus FP32 weights)
  converged V       1e-5   (max-abs relative error of the FP32 schedule), per config
Policies must match wherever the oracle's best-minus-second Q gap exceeds 1e-6
(1e-9 for single FP64 backups, where both sides see the same V).
"""
import numpy as np
import pytest

import workloads as W
from oracle.oracle import Oracle
from paper_2303_10672_amd import pvi

pytestmark = pytest.mark.gpu

SMALL = [
    W.scenario_a(m=2, L=1, a_max=10, d_max=20),
    W.scenario_a(m=1, L=1, a_max=6, d_max=9),
    W.scenario_a(m=1, L=2, a_max=5, d_max=8),
    W.scenario_a(m=3, L=1, a_max=7, d_max=15),
    W.scenario_a(m=3, L=2, a_max=12, d_max=30,
                 demand={"kind": "gamma", "mean": [4.0], "cv": [1.5]}),
    W.scenario_a(m=4, L=1, a_max=6, d_max=12),
    W.scenario_a(m=2, L=3, a_max=5, d_max=4),     # d_max < a_max: clipped demand paths
    W.scenario_a(m=5, L=1, a_max=4, d_max=25),
    W.scenario_a(m=2, L=1, a_max=31, d_max=40),   # 32 actions: the widest kernel
    W.scenario_a(m=3, L=1, a_max=25, d_max=33,
                 demand={"kind": "negbin", "mean": [6.0], "n": [3.0]}),
    # the two action counts with exact-count kernels (no padded actions computed)
    W.scenario_a(m=3, L=1, a_max=20, d_max=30,
                 demand={"kind": "gamma", "mean": [4.0], "cv": [1.5]}),
    W.scenario_a(m=3, L=2, a_max=10, d_max=20),
]
IDS = [f"m{s['m']}L{s['L']}R{s['a_max'][0] + 1}D{s['d_max'][0]}" for s in SMALL]


def relerr(a, b):
    return float(np.abs(a - b).max() / max(np.abs(b).max(), 1e-300))


@pytest.mark.parametrize("sc", SMALL, ids=IDS)
def test_one_backup_fp64(sc):
    o = Oracle(sc)
    m = pvi.mdp_create(sc)
    for seed in range(2):
        V = W.random_values(o.n_states, seed=seed)
        Vo, pio, gapo = o.sweep(V)
        Vg, pig, gapg = pvi.vi_backup(m, V, "fp64")
        assert relerr(Vg, Vo) < 1e-12
        clear = gapo > 1e-9
        assert np.array_equal(pig[clear], pio[clear])
        assert np.allclose(gapg[clear], gapo[clear], rtol=1e-8, atol=1e-8)


@pytest.mark.parametrize("sc", SMALL, ids=IDS)
def test_tiles_per_wavefront_do_not_change_results(sc, monkeypatch):
    """Small instances run with two tiles per wavefront; the full floor(64 / R) tiles
    (the grouping of large instances, with short groups padded) must give the same
    bits: one FP64 and one FP32 backup, and a converged solve with its policy."""
    o = Oracle(sc)
    V = W.random_values(o.n_states, seed=4)
    runs = []
    for force in (None, str(max(1, min(16, 64 // (sc["a_max"][0] + 1))))):
        if force is None:
            monkeypatch.delenv("PVI_A_GROUP", raising=False)
        else:
            monkeypatch.setenv("PVI_A_GROUP", force)
        m = pvi.mdp_create(sc)
        monkeypatch.delenv("PVI_A_GROUP", raising=False)
        b64 = pvi.vi_backup(m, V, "fp64")
        b32 = pvi.vi_backup(m, V, "fp32")
        res = pvi.vi_solve(m, precision="fp64")
        runs.append((b64, b32, res["sweeps_fp64"], pvi.value_get(m), pvi.policy_get(m)))
    (a64, a32, asw, aV, ap), (g64, g32, gsw, gV, gp) = runs
    for x, y in zip(a64 + a32, g64 + g32):
        assert np.array_equal(x, y)
    assert asw == gsw and np.array_equal(aV, gV)
    assert np.array_equal(ap[0], gp[0]) and np.array_equal(ap[1], gp[1])
    assert relerr(a64[0], o.sweep(V)[0]) < 1e-12


@pytest.mark.parametrize("prec", ["fp32", "fp32_wide"])
@pytest.mark.parametrize("sc", SMALL, ids=IDS)
def test_one_backup_fp32(sc, prec):
    o = Oracle(sc)
    m = pvi.mdp_create(sc)
    V = W.random_values(o.n_states, seed=3)
    Vo, pio, gapo = o.sweep(V)
    Vg, pig, _ = pvi.vi_backup(m, V, prec)
    assert relerr(Vg, Vo) < 1e-6, relerr(Vg, Vo)
    clear = gapo > 1e-9
    assert np.array_equal(pig[clear], pio[clear])   # the policy comes from the FP64 Q


@pytest.mark.parametrize("sc", SMALL, ids=IDS)
def test_converged_fp64_matches_oracle_exactly(sc):
    o = Oracle(sc)
    ref = o.solve()
    m = pvi.mdp_create(sc)
    res = pvi.vi_solve(m, precision="fp64")
    assert res["sweeps_fp64"] == ref["sweeps"]
    V = pvi.value_get(m)
    assert relerr(V, ref["V"]) < 1e-12
    pol, gap = pvi.policy_get(m)
    clear = ref["gap"] > 1e-6
    assert np.array_equal(pol[clear], ref["pi"][clear])
    assert res["final_span"] < res["threshold"]


def vhat(V, res, gamma):
    return V + gamma / (1.0 - gamma) * 0.5 * (res["dmax"] + res["dmin"])


@pytest.mark.parametrize("prec", ["fp64", "fp32"])
def test_result_vhat_shift_and_device_time(prec):
    """vhat_shift is gamma/(1-gamma) times the mean of the last increments, and V plus
    it lies within MacQueen's half-width gamma/(1-gamma) (dmax - dmin)/2 of V* (the
    oracle's own bound midpoint at a span of 1e-11, which the span rule alone does not
    bring near V*); device_ms is the solve's stream time, within its wall time."""
    sc = SMALL[0]
    g = sc["gamma"]
    tight = Oracle(sc).solve(thr=1e-11)
    star = vhat(tight["V"], tight, g)
    m = pvi.mdp_create(sc)
    res = pvi.vi_solve(m, precision=prec)
    k = g / (1.0 - g)
    assert res["vhat_shift"] == pytest.approx(k * 0.5 * (res["dmax"] + res["dmin"]), rel=1e-15)
    half = k * 0.5 * (res["dmax"] - res["dmin"])
    err = np.abs(pvi.value_get(m) + res["vhat_shift"] - star).max()
    assert err <= half + 1e-9 * np.abs(star).max()
    assert 0.0 < res["device_ms"] <= res["wall_ms"]


@pytest.mark.parametrize("prec", ["fp32", "fp32_wide"])
@pytest.mark.parametrize("sc", SMALL, ids=IDS)
def test_converged_fp32_schedule(sc, prec):
    o = Oracle(sc)
    tight = o.solve(thr=1e-11)
    ref = o.solve()
    g = sc["gamma"]
    m = pvi.mdp_create(sc)
    res = pvi.vi_solve(m, precision=prec)
    assert res["final_span"] < res["threshold"]
    assert res["sweeps_fp64"] >= 1
    V = pvi.value_get(m)
    err = relerr(vhat(V, res, g), vhat(ref["V"], ref, g))
    assert err < 1e-5, err
    pol, _ = pvi.policy_get(m)
    clear = tight["gap"] > 1e-6
    assert np.array_equal(pol[clear], tight["pi"][clear])


@pytest.mark.parametrize("prec", ["fp64", "fp32", "fp32_wide"])
def test_fixed_sweeps(prec):
    sc = SMALL[4]
    o = Oracle(sc)
    ref = o.solve(fixed_sweeps=7)
    m = pvi.mdp_create(sc)
    res = pvi.vi_solve(m, precision=prec, fixed_sweeps=7)
    assert res["sweeps_fp32"] + res["sweeps_fp64"] == 7
    V = pvi.value_get(m)
    tol = 1e-12 if prec == "fp64" else 1e-5
    assert relerr(V, ref["V"]) < tol


def test_v0_resume_matches_uninterrupted():
    sc = SMALL[4]
    m = pvi.mdp_create(sc)
    pvi.vi_solve(m, precision="fp64", fixed_sweeps=10)
    V10 = pvi.value_get(m)
    pvi.vi_solve(m, precision="fp64", fixed_sweeps=4)
    V4 = pvi.value_get(m)
    pvi.vi_solve(m, precision="fp64", fixed_sweeps=6, v0=V4)
    assert np.array_equal(pvi.value_get(m), V10)


def test_newsvendor_closed_form_on_gpu():
    from scipy import stats
    sc = W.scenario_a(m=1, L=1, a_max=10, d_max=20)
    g, c = sc["gamma"], sc["costs"]
    pmf = np.array([stats.poisson.pmf(d, 4.0) for d in range(20)] + [stats.poisson.sf(19, 4.0)])
    d = np.arange(21)
    G = np.array([-(c["short"] * np.maximum(d - x, 0) + c["waste"] * np.maximum(x - d, 0)) @ pmf
                  for x in range(11)])
    h = -c["var"][0] * np.arange(11) + g * G
    V_star = G + h.max() / (1.0 - g)
    for prec in ("fp64", "fp32", "fp32_wide"):
        m = pvi.mdp_create(sc)
        res = pvi.vi_solve(m, precision=prec)
        V = pvi.value_get(m)
        assert relerr(vhat(V, res, g), V_star) < 1e-9
        pol, _ = pvi.policy_get(m)
        assert np.all(pol == 2)


def test_determinism_bit_identical():
    sc = SMALL[4]
    outs = []
    for _ in range(2):
        m = pvi.mdp_create(sc)
        pvi.vi_solve(m, precision="fp32")
        outs.append((pvi.value_get(m), pvi.policy_get(m)[0]))
    assert np.array_equal(outs[0][0], outs[1][0]) and np.array_equal(outs[0][1], outs[1][1])


def test_max_sweeps_not_converged_keeps_results():
    sc = SMALL[4]
    m = pvi.mdp_create(sc)
    with pytest.raises(pvi.PviError) as e:
        pvi.vi_solve(m, precision="fp64", max_sweeps=2)
    assert e.value.status == pvi.PVI_E_NOT_CONVERGED
    V = pvi.value_get(m)
    assert np.all(np.isfinite(V))


# each compiled action count and the counts on both sides of it; the last has more than 2,048
# wavefronts of one tile, whose states are finished in two parts
SPLITS = [W.scenario_a(m=m, L=L, a_max=R - 1, d_max=20, demand={
              "kind": "gamma", "mean": [0.4 * R + 1.0], "cv": [0.8]})
          for R in (1, 2, 8, 9, 11, 12, 16, 17, 21, 24, 25, 32)
          for m, L in ((1, 1), (2, 2), (3, 1))] + [W.scenario_a(m=4, L=2, a_max=12, d_max=25)]


@pytest.mark.parametrize("sc", SPLITS, ids=[f"m{s['m']}L{s['L']}R{s['a_max'][0] + 1}"
                                            for s in SPLITS])
def test_actions_split_over_lanes_equal_whole_tiles(sc, monkeypatch):
    """One tile per wavefront (actions split over lanes) against the oracle and, bit for bit,
    against several tiles per wavefront; short chunks of the path give the same bits too."""
    o = Oracle(sc)
    R = sc["a_max"][0] + 1
    V = W.random_values(o.n_states, seed=7)
    ref = o.sweep(V)[0]
    runs = []
    for G, CH in ((1, 64), (1, 3), (2, 5), (min(16, 64 // R), 1)):
        monkeypatch.setenv("PVI_A_GROUP", str(G))
        monkeypatch.setenv("PVI_A_CHUNK", str(CH))
        m = pvi.mdp_create(sc)
        runs.append([x for prec in ("fp64", "fp32", "fp32_wide")
                     for x in pvi.vi_backup(m, V, prec)])
    assert relerr(runs[0][0], ref) < 1e-12
    for prec in (3, 6):
        assert relerr(runs[0][prec], ref) < 1e-6
    for other in runs[1:]:
        for x, y in zip(runs[0], other):
            assert np.array_equal(x, y)


# 17 to 20 orders take the split kernel of 21: (1, 2) has one life class, (3, 1) rows in parts
@pytest.mark.parametrize("m,L", [(1, 2), (2, 2), (3, 1)])
@pytest.mark.parametrize("R", [18, 19, 20])
def test_rows_of_21_serve_fewer_orders(R, m, L, monkeypatch):
    sc = W.scenario_a(m=m, L=L, a_max=R - 1, d_max=20, demand={
        "kind": "gamma", "mean": [0.4 * R + 1.0], "cv": [0.8]})
    test_actions_split_over_lanes_equal_whole_tiles(sc, monkeypatch)
    o = Oracle(sc)
    V = W.random_values(o.n_states, seed=11)
    _, pi, gap = o.sweep(V)[:3]
    monkeypatch.setenv("PVI_A_GROUP", "1")
    out = pvi.vi_backup(pvi.mdp_create(sc), V)
    clear = gap > 1e-9 * np.abs(V).max()
    assert np.array_equal(out[1][clear], pi[clear])


@pytest.mark.parametrize("value", [np.nan, np.inf, -np.inf, -1e301])
@pytest.mark.parametrize("m,L", [(1, 2), (3, 2)])
def test_values_that_are_no_numbers_split_over_lanes(m, L, value, monkeypatch):
    """11 orders, four lanes of three actions: the twelfth is no action whatever V holds.  The
    packed kernel, compiled for 11 actions, has no padding."""
    n = 11 ** (m + L - 1)
    rng = np.random.default_rng(m)
    for share in (0.02, 0.5, 1.0):
        V = W.random_values(n, seed=2)
        V[rng.random(n) < share] = value
        runs = []
        for G in (1, 2):
            monkeypatch.setenv("PVI_A_GROUP", str(G))
            h = pvi.mdp_create(W.scenario_a(m=m, L=L, a_max=10, d_max=15))
            runs.append([x for prec in ("fp64", "fp32", "fp32_wide")
                         for x in pvi.vi_backup(h, V, prec)])
        for x, y in zip(*runs):
            assert np.array_equal(x, y, equal_nan=x.dtype == np.float64)
