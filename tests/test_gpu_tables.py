"""The table kernel (numeric tables and chain patterns of a segment) at the
sizes where its forms change: items that enumerate bottom slots (chains of 6
bits and more once a segment has over 256 patterns), pattern parts (over 4096
patterns by the plan's bound), zone records beyond the LDS stage (tables and
patterns in two launches).  Every mask's error and band slack against the
oracle: both evaluate sums of at most a few dozen voltage changes of order
0.01 in FP64, which round below 1e-14; the tolerance is the 1e-9 p.u. that the
decisions are specified to."""
import numpy as np
import pytest

import oracle
from synth_feeders import make_feeder

pytestmark = pytest.mark.gpu

TOL = 1e-9


@pytest.fixture(scope="module")
def okr():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    import paper_2510_19608_amd as okr
    okr.lib()
    return okr


def check(okr, f, precision="fp64", per_segment=256):
    """Decisions, and sampled masks of every segment at the state the earlier
    decisions left, against the oracle."""
    V, I, st, _ = oracle.powerflow(f)
    assert st == 0
    out = okr.reduce_feeder(f, dump=True, precision=precision, want_vhat=False)
    state = np.ones(f["n"], np.uint8)
    rng = np.random.default_rng(0)
    for g, s in enumerate(out["segments"]):
        e, slack, k = out["scores"][g]
        masks = np.unique(np.r_[0, (1 << k) - 1, s["mask"], rng.integers(0, 1 << k, per_segment)]).astype(np.uint32)
        want = oracle.score_masks(f, V, I, state, g, masks)
        np.testing.assert_allclose(e[masks], want["e_loc"], rtol=0, atol=TOL, err_msg=f"segment {g}")
        fin = np.isfinite(want["slack_loc"])
        np.testing.assert_allclose(slack[masks][fin], want["slack_loc"][fin], rtol=0, atol=TOL)
        from synth_feeders import dfs_preorder
        order = [int(v) for v in dfs_preorder(f["parent"]) if f["segment"][v] == g]
        for j, v in enumerate(order):
            if s["mask"] >> j & 1:
                state[v] = 0
    return out


@pytest.mark.parametrize("k", [5, 6, 8, 9, 12, 13])
def test_long_chains(okr, k):
    """Deep laterals: chains of up to k bits, from one pattern per thread to
    several parts."""
    print(f"tables: long chains k={k}", flush=True)
    f = make_feeder("c1", k, n=45, n_eligible=None, seg_size=(k, k), snapshots=3, p_deep=0.93, e_bar=2e-4, kappa=0.25)
    check(okr, f)


def zone_feeder(n, leaves):
    """A three-phase feeder whose node 1 carries everything else: reducing it
    moves every other node."""
    f = make_feeder("c1", 3, n=n, n_eligible=None, p_single=0.0, p_two=0.0, snapshots=2, kappa=1 / 64)
    parent = np.asarray(f["parent"]).copy()
    parent[1:3] = [0, 1]
    parent[3:] = np.maximum(parent[3:], 2)
    Yd = np.zeros_like(f["Y_diag"])
    for i in range(1, n):
        Yd[i] -= f["Y_off"][i]
        Yd[parent[i]] -= f["Y_off"][i]
    seg = np.full(n, -1, np.int32)
    nchild = np.bincount(parent[1:], minlength=n)
    seg[[1] + [int(v) for v in np.flatnonzero(nchild == 0)[:leaves]]] = 0
    return dict(f, parent=parent, Y_diag=Yd, segment=seg, eligible=(seg >= 0).astype(np.uint8), n_segments=1,
                v_min=0.9, v_max=1.1, e_bar=3e-4)


@pytest.mark.parametrize("n", [20, 90, 350, 900])
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_many_zone_entries(okr, n, precision):
    """One short chain above 50 to 2,700 zone entries: in the LDS stage, partly
    beyond it, and with tables and patterns in separate launches."""
    print(f"tables: zone entries n={n} {precision}", flush=True)
    f = zone_feeder(n, 5)
    if precision == "fp64":
        check(okr, f, per_segment=64)
    else:
        a = okr.reduce_feeder(f, precision=precision, want_vhat=False)
        b = okr.reduce_feeder(f, want_vhat=False)
        assert [s["mask"] for s in a["segments"]] == [s["mask"] for s in b["segments"]]
        np.testing.assert_array_equal(a["err_per_snapshot"], b["err_per_snapshot"])


@pytest.mark.parametrize("snapshots", [2, 31, 32, 33, 70])
def test_smice_snapshot_lanes(okr, snapshots):
    """SMICE sums taken by 32 lanes per mask: fewer snapshots than lanes, as
    many, one more, several rounds.  Sums of up to a few hundred errors of order
    1e-3: the tolerance is the tests' 1e-11 for SMICE sums (rounding 1e-16 each)."""
    print(f"tables: smice snapshots={snapshots}", flush=True)
    f = make_feeder("c1", 2, n=24, n_eligible=None, seg_size=(4, 6), snapshots=snapshots, scale=(0.3, 1.0), e_bar=2e-4)
    V, I, st, _ = oracle.powerflow(f)
    keep, dec, _ = oracle.search(f, V, I, secondary="smice")
    assert st == 0 and not any(d["ambiguous"] for d in dec)
    out = okr.reduce_feeder(f, secondary="smice")
    for s, d in zip(out["segments"], dec):
        assert s["mask"] == d["mask"]
        assert abs(s["smice_rise"] - d["smice_rise"]) < 1e-11
    np.testing.assert_array_equal(out["kept"], keep)


@pytest.mark.parametrize("n,S,p_deep,kappa,moves", [
    (64, 3, 0.5, 0.5, 70), (65, 1, 0.97, 0.5, 70), (129, 2, 0.97, 0.5, 24), (700, 2, 0.9, 0.05, 80)])
def test_greedy_cluster_list(okr, n, S, p_deep, kappa, moves):
    """Greedy search at the edges of the cluster list's runs of 64 and of the
    intervals that one wave scores alone (a 700-node trunk), in both scoring
    forms: the oracle's moves where it is small enough, and the same moves in
    both forms.  SMICE sums at most S * n errors that agree within the load
    flow's 1e-13."""
    from oracle import greedy as G
    print(f"greedy cluster list: n={n} S={S} p_deep={p_deep}", flush=True)
    f = make_feeder("c2", n, n=n, snapshots=S, p_deep=p_deep, kappa=kappa)
    V, I, st, _ = oracle.powerflow(f)
    assert st == 0
    outs = [okr.greedy(f, e_bar=5e-3, vhat=V, max_iter=moves, incremental=inc) for inc in (False, True)]
    ids = [[(s["cand"], s["s"], s["r"], s["n_cand"], s["n_feasible"]) for s in o["steps"]] for o in outs]
    assert ids[0] == ids[1] and len(ids[0]) > 10
    for key in ("smice", "emax"):
        np.testing.assert_allclose([s[key] for s in outs[1]["steps"]], [s[key] for s in outs[0]["steps"]], rtol=0,
                                   atol=TOL)
    if n <= 129:
        sup, steps, err = G.greedy(f, V, I, e_bar=5e-3, max_iter=moves)
        assert ids[0] == [(s["cand"], s["s"], s["r"], s["n_cand"], s["n_feasible"]) for s in steps]
        for o in outs:
            np.testing.assert_array_equal(o["super"], sup)
            np.testing.assert_allclose([s["smice"] for s in o["steps"]], [s["smice"] for s in steps], rtol=0, atol=TOL)
            np.testing.assert_allclose(o["err_per_snapshot"], err, rtol=0, atol=TOL)


@pytest.mark.parametrize("n,p_deep", [(2, 0.5), (64, 0.5), (65, 0.9), (320, 0.5), (321, 0.5), (1023, 0.5), (1024, 0.5), (1025, 0.5), (2100, 0.6)])
def test_prefix_sum_load_flow(okr, n, p_deep):
    """Load flow and fixed-current solve by prefix sums at the edges of the
    waves and of the forms (up to 320 nodes a thread per node and phase, up to
    1024 a thread per node; above, phase by phase), 3 snapshots.  The oracle's load flow stops at the same
    1e-13, so the voltages differ by less than ten times that; the identity
    assignment solved at the load flow's own currents gives its voltages back
    within the same bound."""
    print(f"load flow: n={n} p_deep={p_deep}", flush=True)
    f = make_feeder("c2", n, n=n, snapshots=3, p_deep=p_deep, kappa=0.2)
    V, I, st, it = oracle.powerflow(f)
    assert st == 0
    out = okr.reduce_feeder(f, want_vhat=True)
    np.testing.assert_allclose(out["Vhat"], V, rtol=0, atol=1e-12)
    err, mx = okr.evaluate_assignment(f, np.arange(n))
    assert mx == err.max() and mx < 1e-12


@pytest.mark.parametrize("n", [65, 1025])
def test_evaluation_of_given_voltages(okr, n):
    """An evaluation with V^ given takes the aggregate, fixed solve and errors
    as launches of their own: the identity assignment gives the oracle's V^
    back (bound as above)."""
    print(f"evaluation, V^ given: n={n}", flush=True)
    f = make_feeder("c2", n, n=n, snapshots=3, kappa=0.2)
    V, I, st, _ = oracle.powerflow(f)
    assert st == 0
    err, mx = okr.evaluate_assignment(f, np.arange(n), vhat=V)
    assert mx == err.max() and mx < 1e-12


def test_load_flow_beyond_prefix_sums(okr):
    """An 18,000-node feeder (over 9600 nodes on a phase): the breadth-first
    load flow of the search, and the level-by-level load flow and fixed-current
    solve of an evaluation (bounds as above; a wide band keeps the heavily
    loaded feeder valid)."""
    print("load flow: n=18000", flush=True)
    f = make_feeder("c3", 0, n=18000, snapshots=2, v_min=0.5, v_max=1.5)
    assert max(int((f["phase"] >> p & 1).sum()) for p in range(3)) > 9600
    V, I, st, _ = oracle.powerflow(f)
    assert st == 0
    out = okr.reduce_feeder(f, want_vhat=True)
    np.testing.assert_allclose(out["Vhat"], V, rtol=0, atol=1e-12)
    err, _ = okr.evaluate_assignment(f, np.arange(f["n"]))
    assert err.max() < 1e-12


def test_load_flow_more_snapshots_than_compute_units(okr):
    """257 snapshots of a 1100-node feeder: the phase-by-phase load flow in
    blocks of 512 threads, two on a compute unit (bound as above)."""
    print("load flow: n=1100, 257 snapshots", flush=True)
    f = make_feeder("c2", 3, n=1100, snapshots=257, kappa=0.2, seg_size=(6, 8))
    V, I, st, _ = oracle.powerflow(f)
    assert st == 0
    out = okr.reduce_feeder(f, want_vhat=True)
    np.testing.assert_allclose(out["Vhat"], V, rtol=0, atol=1e-12)


@pytest.mark.parametrize("S", [255, 257])
def test_snapshot_pairs_with_a_remainder(okr, S):
    """Two snapshots per block of the table kernel with one block's second
    half empty, and the lists' and patterns' folds over both."""
    print(f"tables: {S} snapshots", flush=True)
    f = make_feeder("c1", 5, n=30, snapshots=S, e_bar=5e-4, kappa=0.25)
    check(okr, f, per_segment=64)
