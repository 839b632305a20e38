"""Load flow and fixed-current solve of feeders with uneven branches: some
subtrees (leaves and laterals of up to 40 nodes) carry a load 1e6 times smaller
behind impedances 1e6 times larger, so that their own voltage drops stay what
they were while their currents are 1e-6 of the others'.  Reference: the same
sweeps in 80-bit arithmetic."""
import numpy as np
import pytest

from synth_feeders import dfs_preorder, make_feeder

pytestmark = pytest.mark.gpu

R = 1e6

# Rounding of a converged voltage: V0 - D rounds once at |V| ~ 1 (1.1e-16 per
# component); D, below 0.1 p.u., is a sum of at most 40 rounded steps
# (40 * 1.1e-16 * 0.1 = 4.4e-16) of drops z J whose factors carry about 20
# roundings each (2 * 20 * 1.1e-16 * 0.1 = 4.4e-16); the iteration stops at
# 1e-15 with a contraction below 0.3 (4e-16 left).  In all below 2e-15.
TOL = 2e-15
# Stopped at the default 1e-13: 0.3 / 0.7 * 1e-13 left in V^, as much in |V^|.
TOL_STOP = 1e-13


@pytest.fixture(scope="module")
def okr():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("GPU tests need a visible MI355X")
    import paper_2510_19608_amd as okr
    okr.lib()
    return okr


def uneven(f, seed, share=0.05, r=R):
    """The feeder with about `share` of its nodes at the top of a light subtree."""
    n, parent = f["n"], np.asarray(f["parent"])
    rng = np.random.default_rng(seed)
    order = [int(v) for v in dfs_preorder(parent)]
    pos = np.empty(n, int)
    pos[order] = np.arange(n)
    size = np.ones(n, int)
    for v in reversed(order[1:]):
        size[parent[v]] += size[v]
    light = np.zeros(n, bool)
    tops = np.flatnonzero(size <= min(40, n // 8 + 1))
    for v in rng.permutation(tops[tops > 0])[:max(1, int(share * n))]:
        light[order[pos[v]:pos[v] + size[v]]] = True
    Yo, S = np.array(f["Y_off"]), np.array(f["S_load"])
    Yo[light] /= r
    S[:, light] /= r
    Yd = np.zeros_like(Yo)
    for i in range(1, n):
        Yd[i] -= Yo[i]
        Yd[parent[i]] -= Yo[i]
    return dict(f, Y_off=Yo, Y_diag=Yd, S_load=S), light


class Exact:
    """The two sweeps of a radial network in 80-bit arithmetic, all snapshots at once."""

    def __init__(self, f):
        self.f, self.n, self.parent = f, f["n"], np.asarray(f["parent"])
        depth = np.zeros(self.n, int)
        for v in dfs_preorder(self.parent)[1:]:
            depth[v] = depth[self.parent[v]] + 1
        self.levels = [np.flatnonzero(depth == d) for d in range(1, depth.max() + 1)]
        self.on = (np.asarray(f["phase"])[:, None] >> np.arange(3)) & 1 == 1
        z = np.zeros((self.n, 3, 3), complex)
        for i in range(1, self.n):
            ix = np.flatnonzero(self.on[i])
            z[np.ix_([i], ix, ix)] = np.linalg.inv(-f["Y_off"][i][np.ix_(ix, ix)])
        self.z = z.astype(np.clongdouble)
        self.V0 = np.asarray(f["V0"]).astype(np.clongdouble)

    def currents(self, V):
        I = np.zeros(V.shape, np.clongdouble)
        S = np.asarray(self.f["S_load"]).astype(np.clongdouble)
        I[:, self.on] = np.conj(S[:, self.on] / V[:, self.on])
        I[:, 0] = 0
        return I

    def solve(self, I):
        J, V = I.copy(), np.zeros_like(I)
        for v in reversed(self.levels):
            np.add.at(J, (slice(None), self.parent[v]), J[:, v])
        V[:, 0] = self.V0 * self.on[0]
        for v in self.levels:
            d = sum(self.z[v][None, :, :, c] * J[:, v, c][:, :, None] for c in range(3))
            V[:, v] = (V[:, self.parent[v]] - d) * self.on[v]
        return V

    def flow(self):
        V = np.broadcast_to(self.V0 * self.on, np.asarray(self.f["S_load"]).shape).astype(np.clongdouble)
        for _ in range(100):
            W = self.solve(self.currents(V))
            step, V = np.abs(W - V).max(), W
            if step < 1e-17:
                return V
        raise AssertionError("the reference load flow did not converge")

    def errors(self, Vh, I, sup):
        """Largest error per snapshot of an assignment at the load currents I."""
        A = np.zeros_like(I)
        np.add.at(A, (slice(None), sup), I)
        e = np.abs(np.abs(Vh) - np.abs(self.solve(A)[:, sup])) * self.on
        return e.max(axis=(1, 2)).astype(float)


def reduced(f):
    """Every eligible node moved to its nearest kept ancestor."""
    sup = np.arange(f["n"])
    for v in dfs_preorder(f["parent"]):
        if f["eligible"][v]:
            sup[v] = sup[f["parent"][v]]
    return sup


CASES = [(30, 3, 0.5), (64, 2, 0.97), (300, 3, 0.5), (320, 2, 0.9), (321, 2, 0.9), (1000, 3, 0.0), (1024, 2, 0.9),
         (1025, 2, 0.9), (1100, 257, 0.5), (2100, 3, 0.9), (6000, 2, 0.5)]


@pytest.mark.parametrize("n,S,p_deep", CASES)
def test_light_branches_keep_their_bits(okr, n, S, p_deep):
    """Every form of the load flow (up to 320 nodes, up to 1024, phase by phase,
    that in pairs of blocks), and the evaluation of an assignment after it and at
    given voltages."""
    print(f"uneven load flow: n={n} S={S} p_deep={p_deep}", flush=True)
    f = make_feeder("c2", n, n=n, snapshots=S, p_deep=p_deep, kappa=2.0 ** -6 if n > 1000 or p_deep > 0.5 else 0.2,
                    seg_size=(6, 8), v_min=0.5, v_max=1.5)
    f, light = uneven(f, n)
    assert light.any()
    x = Exact(f)
    V = x.flow()
    assert np.abs(V - x.V0 * x.on).max() < 0.1
    even = okr.reduce_feeder(make_feeder("c2", n, n=n, snapshots=S, p_deep=p_deep, seg_size=(6, 8), v_min=0.5,
                                         v_max=1.5, kappa=f["kappa"]), want_vhat=False)
    out = okr.reduce_feeder(f, want_vhat=False)
    assert out["pf_iterations"] <= even["pf_iterations"]
    out = okr.reduce_feeder(f, pf_tol=1e-15)
    worst = float(np.abs(out["Vhat"] - V).max())
    sup = reduced(f)
    want = x.errors(V, x.currents(V), sup)
    err, _ = okr.evaluate_assignment(f, sup)
    Vd = V.astype(np.complex128)
    given, _ = okr.evaluate_assignment(f, sup, vhat=Vd)
    Vd = Vd.astype(np.clongdouble)
    want_given = x.errors(Vd, x.currents(Vd), sup)
    print(f"  |V - ref| {worst:.2e}, evaluation {np.abs(err - want).max():.2e}, "
          f"at given voltages {np.abs(given - want_given).max():.2e}", flush=True)
    assert worst <= TOL
    assert np.abs(err - want).max() <= TOL_STOP
    assert np.abs(given - want_given).max() <= TOL


def without_phase_a(n, S, nan_at):
    """A feeder of phases b and c alone whose loads are NaN at one node."""
    f = make_feeder("c2", n, n=n, snapshots=S, p_single=0.0, p_two=0.0, kappa=2.0 ** -6, seg_size=(6, 8), v_min=0.5,
                    v_max=1.5)
    parent, Yo, S_load = np.asarray(f["parent"]), np.array(f["Y_off"]), np.array(f["S_load"])
    for i in range(1, n):
        z = np.linalg.inv(-Yo[i])[1:, 1:]
        Yo[i] = 0
        Yo[i, 1:, 1:] = -np.linalg.inv(z)
    Yd = np.zeros_like(Yo)
    for i in range(1, n):
        Yd[i] -= Yo[i]
        Yd[parent[i]] -= Yo[i]
    S_load[:, :, 0] = 0
    S_load[-1, nan_at, 2] = np.nan
    return dict(f, phase=np.full(n, 6, np.uint8), Y_off=Yo, Y_diag=Yd, S_load=S_load)


@pytest.mark.parametrize("n", [30, 320, 1000, 1100, 18000])
def test_nan_load_is_no_convergence(okr, n):
    """A load flow that turns NaN is reported as diverged in every form, also
    where the lanes of an absent phase hold zeros beside the NaN ones."""
    print(f"NaN load: n={n}", flush=True)
    f = without_phase_a(n, 2, n - 1)
    with pytest.raises(okr.OkrError) as e:
        okr.reduce_feeder(f, want_vhat=False)
    assert "converge" in str(e.value)
    with pytest.raises(okr.OkrError) as e:
        okr.evaluate_assignment(f, np.arange(n))
    assert "converge" in str(e.value)


@pytest.mark.parametrize("n,S", [(9600, 2), (9601, 2), (4902, 257), (4903, 257)])
def test_phase_lists_at_the_edges_of_lds(okr, n, S):
    """Three-phase feeders at the largest list that a block's LDS holds (9600
    entries and their rows' sums), one more (level by level), and at the largest
    that two blocks share a compute unit with (4902).  The oracle's load flow
    stops at the same 1e-13, so the voltages differ by less than ten times that."""
    import oracle
    print(f"phase lists: n={n} S={S}", flush=True)
    f = make_feeder("c2", 1, n=n, snapshots=S, p_single=0.0, p_two=0.0, p_deep=0.5, kappa=2.0 ** -7, seg_size=(4, 6),
                    v_min=0.5, v_max=1.5)
    V, _, st, _ = oracle.powerflow(f)
    assert st == 0
    out = okr.reduce_feeder(f, want_vhat=True)
    np.testing.assert_allclose(out["Vhat"], V, rtol=0, atol=1e-12)
    err, _ = okr.evaluate_assignment(f, np.arange(n))
    assert err.max() < 1e-12
