"""Per-mask scores against references that share no kernel with them.

FP64 and factored searches score every mask from chain pattern tables, so
comparing the two compares a path with itself.  Here sampled masks of every
segment (the empty and the full one and the chosen one among them) are scored
by the oracle at the state that the earlier decisions left, over the forms that
the launches take: one or two snapshots per block, pattern parts and enumerated
bottom slots, 2, 4 or 8 tiles per wave, patterns beyond the combine's LDS stage,
one chunk lane or eight.  The decisions are compared, bit for bit, with those of
the short-list scoring, which walks every chain for every listed mask.

Tolerances: both sides add up at most a few dozen voltage changes of order 0.01
in FP64 (below 1e-14); 1e-9 p.u. is what the decisions are specified to."""
import numpy as np
import pytest

import oracle
from synth_feeders import dfs_preorder, make_feeder

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


def check_samples(f, out, per_segment):
    V, I, st, _ = oracle.powerflow(f)
    assert st == 0
    state = np.ones(f["n"], np.uint8)
    rng = np.random.default_rng(1)
    order = [int(v) for v in dfs_preorder(f["parent"])]
    for g, s in enumerate(out["segments"]):
        e, slack, k = out["scores"][g]
        masks = np.unique(np.r_[0, (1 << k) - 1, s["mask"], rng.integers(0, 1 << k, per_segment)]).astype(np.uint32)
        want = oracle.score_masks(f, V, I, state, g, masks)
        np.testing.assert_allclose(e[masks], want["e_loc"], rtol=0, atol=TOL, err_msg=f"segment {g}")
        fin = np.isfinite(want["slack_loc"])
        np.testing.assert_allclose(slack[masks][fin], want["slack_loc"][fin], rtol=0, atol=TOL, err_msg=f"segment {g}")
        assert (slack[masks][~fin] > 1e300).all()
        assert s["e_loc"] == e[s["mask"]]
        for j, v in enumerate([v for v in order if f["segment"][v] == g]):
            if s["mask"] >> j & 1:
                state[v] = 0


# chunks of 1 to 8 segments: 2 to 8 tiles per wave; 248, 256 and 264 (segment,
# snapshot) pairs in the widest launch, on both sides of two snapshots per block
LONG = dict(snapshots=4, seg_size=(19, 20), e_bar=2e-4)
WIDE = dict(seg_size=(6, 8), e_bar=2e-4)


@pytest.mark.parametrize("cfg,seed,over,per", [
    ("c2", 0, {}, 20), ("c2", 1, dict(e_bar=1e-4), 20), ("c2", 2, LONG, 24), ("c4", 0, dict(LONG, n=400), 24),
    ("c2", 3, dict(WIDE, snapshots=31), 4), ("c2", 3, dict(WIDE, snapshots=32), 4),
    ("c2", 3, dict(WIDE, snapshots=33), 4)])
def test_sampled_masks_of_every_segment(okr, cfg, seed, over, per):
    print(f"sampled masks: {cfg} seed {seed} {over}", flush=True)
    f = make_feeder(cfg, seed, **over)
    ref = okr.reduce_feeder(f, dump=True, want_vhat=False, lanes=1)
    check_samples(f, ref, per)
    for kw in (dict(lanes=8), dict(lanes=8, precision="factored")):
        out = okr.reduce_feeder(f, dump=True, want_vhat=False, **kw)
        for g in ref["scores"]:
            for a, b in zip(out["scores"][g], ref["scores"][g]):
                np.testing.assert_array_equal(a, b, err_msg=f"segment {g} {kw}")
        assert [(s["mask"], s["e_loc"], s["e_min"]) for s in out["segments"]] == \
               [(s["mask"], s["e_loc"], s["e_min"]) for s in ref["segments"]]
        np.testing.assert_array_equal(out["err_per_snapshot"], ref["err_per_snapshot"])


@pytest.mark.parametrize("cfg,seed,over", [
    ("c2", 0, dict(seg_size=(8, 12))), ("c2", 5, dict(n=300, snapshots=40, seg_size=(3, 9), e_bar=1e-4)),
    ("c4", 2, dict(n=700, snapshots=6, seg_size=(8, 12), v_min=0.9, v_max=1.1, e_bar=1e-4))])
def test_patterns_against_walked_chains(okr, cfg, seed, over):
    """A surrogate search whose list holds every mask of every segment decides
    from scores walked chain by chain, mask by mask: the pattern tables' decisions
    and errors must be the same bits."""
    from paper_2510_19608_amd import surrogate
    print(f"walked chains: {cfg} seed {seed} {over}", flush=True)
    f = make_feeder(cfg, seed, **over)
    seg = np.asarray(f["segment"])
    top = 1 << int(np.bincount(seg[seg >= 0]).max())
    a = okr.reduce_feeder(f, want_vhat=False)
    b = okr.reduce_feeder(f, want_vhat=False, surrogate=surrogate.init_params(seed), top_k=top)
    listed = [s for s in b["segments"] if s["n_scored"] == 1 << s["k"]]
    assert len(listed) > len(b["segments"]) // 2  # (a segment that reduces nothing is enumerated after its list)
    for key in ("mask", "e_loc", "e_min", "ambiguous"):
        assert [s[key] for s in a["segments"]] == [s[key] for s in b["segments"]]
    np.testing.assert_array_equal(a["err_per_snapshot"], b["err_per_snapshot"])
    np.testing.assert_array_equal(a["Yk_diag"], b["Yk_diag"])


@pytest.mark.parametrize("snapshots", [2, 63, 64, 65, 130])
def test_smice_snapshots_over_the_lanes(okr, snapshots):
    """SMICE sums by a wave per mask, its lanes the snapshots: fewer than 64, as
    many, one more, a third round.  Sums of up to a few hundred errors of order
    1e-3 (rounding 1e-16 each): 1e-11."""
    print(f"smice lanes: {snapshots} snapshots", flush=True)
    f = make_feeder("c1", 2, n=24, n_eligible=None, seg_size=(4, 6), snapshots=snapshots, scale=(0.3, 1.0), e_bar=2e-4)
    V, I, st, _ = oracle.powerflow(f)
    keep, dec, _ = oracle.search(f, V, I, secondary="smice")
    assert st == 0 and not any(d["ambiguous"] for d in dec)
    out = okr.reduce_feeder(f, secondary="smice")
    for s, d in zip(out["segments"], dec):
        assert s["mask"] == d["mask"]
        assert abs(s["smice_rise"] - d["smice_rise"]) < 1e-11
    np.testing.assert_array_equal(out["kept"], keep)
