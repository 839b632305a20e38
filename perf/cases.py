"""The work users have this library do, as cases that can be timed and compared.

Four kinds of case, each through the package's public entry points:

  reduce     the segment-exhaustive search of a feeder (``Reducer.run``), in
             its precisions, keys and launch forms;
  greedy     Algorithm 1, the single-move search (``Greedy.run``);
  evaluate   a fixed reduction scored over many scenarios
             (``Greedy.evaluate``);
  surrogate  one training batch's gradient and a forward pass over many rows
             (``okr_surrogate_grad``, ``surrogate.predict``).

Feeders come from the seeded generator, so a case's topology, impedances and
loads all follow from the seed.  The voltage band of the 6000- and 8400-node
generators is 0.90-1.10 p.u., so that every seed's base network is inside it
and the search makes its decisions.
"""
import math

import numpy as np
import torch

from paper_2510_19608_amd import (SURR_FEATURES, SURR_PARAMS, Greedy, Reducer, okr_surrogate_grad,
                                  okr_surrogate_workspace, surrogate)
from synth_feeders import CONFIGS, extreme_scenarios, hourly_feeder, make_feeder

DEVICE = "cuda:0"
DECISIONS = (("mask", np.uint32), ("e_loc", np.float64), ("key_gap", np.float64), ("smice_rise", np.float64))


def _reduce(name, cfg, *, n=0, S=0, seg_lo=0, seg_hi=0, e_bar=0.003, precision="fp64", secondary="maxerr",
            graph=False, replan=False):
    c = CONFIGS[cfg]
    return dict(name=name, kind="reduce", cfg=cfg, n=n or c.n, S=S or c.snapshots, seg_lo=seg_lo or c.seg_size[0],
                seg_hi=seg_hi or c.seg_size[1], e_bar=e_bar, precision=precision, secondary=secondary, graph=graph,
                replan=replan)


def listed():
    return [
        # the 30-bus, 4,096-candidate feeder of the tests and the smoke run,
        # planned on each call: the smallest call, all latency
        _reduce("reduce_30", "c1", e_bar=3e-4, replan=True),
        # the benchmark's headline search
        _reduce("reduce_1000", "c2"),
        # a bound that binds and Algorithm 1's key (SMICE), replayed as a graph
        _reduce("reduce_1000_smice", "c2", e_bar=1e-4, secondary="smice", graph=True),
        # the factored form, as a serving loop replays it
        _reduce("reduce_1000_factored", "c2", precision="factored", graph=True),
        # the 6000-node feeder at a bound that binds: FP64 and mixed precision
        _reduce("reduce_6000", "c3", e_bar=7e-5),
        _reduce("reduce_6000_mixed", "c3", e_bar=7e-5, precision="mixed", graph=True),
        # the largest search: 8400 nodes, 288 snapshots, segments of up to 20
        _reduce("reduce_8400", "c4"),
        _reduce("reduce_8400_factored", "c4", precision="factored"),
        # Algorithm 1 on a sub-feeder and on a whole one (the paper's sizes),
        # two extreme hours of a week
        dict(name="greedy_1000", kind="greedy", cfg="c2", n=1000, S=2, e_bar=0.003),
        dict(name="greedy_5591", kind="greedy", cfg="c3", n=5591, S=2, e_bar=0.001),
        # the robustness study: a reduction scored over a week of hours
        dict(name="evaluate_1000_168h", kind="evaluate", cfg="c2", n=1000, S=168),
        # the ranking network: a training batch and a ranking pass
        dict(name="surrogate_4096_65536", kind="surrogate", batch=4096, rows=65536),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["reduce"] * 7 + ["greedy", "evaluate", "surrogate"])
    if kind == "surrogate":
        return dict(kind=kind, batch=64 * _log_int(rng, 1, 128), rows=_log_int(rng, 64, 65536))
    if kind == "greedy":
        n = _log_int(rng, 30, 3000)
        return dict(kind=kind, cfg="c2" if n <= 1000 else "c3", n=n, S=2, e_bar=10 ** rng.uniform(-4, -2))
    if kind == "evaluate":
        n = _log_int(rng, 30, 8400)
        return dict(kind=kind, cfg="c2" if n <= 1000 else "c3", n=n, S=rng.randint(1, 168))
    n = _log_int(rng, 30, 8400)
    cfg = "c2" if n <= 1000 else rng.choice(["c3", "c4"])
    hi = rng.randint(8, 18 if n > 1000 else 16)
    precision = rng.choice(["fp64", "fp64", "factored", "mixed"])
    c = _reduce("", cfg, n=n, S=_log_int(rng, 1, 288), seg_lo=rng.choice([min(8, hi), hi]), seg_hi=hi,
                e_bar=10 ** rng.uniform(-4, -2), precision=precision,
                secondary="maxerr" if precision == "mixed" else rng.choice(["maxerr", "maxerr", "smice"]),
                graph=rng.random() < 0.5, replan=rng.random() < 0.3)
    del c["name"]
    return c


# ---- inputs ---------------------------------------------------------------

def _feeder(case, seed):
    if case["kind"] == "reduce":
        over = {} if case["cfg"] == "c1" else dict(seg_size=(case["seg_lo"], case["seg_hi"]))
        f = make_feeder(case["cfg"], seed, n=case["n"], snapshots=case["S"], e_bar=case["e_bar"], **over)
    else:
        f = hourly_feeder(case["cfg"], seed, n=case["n"])
        if case["kind"] == "greedy":
            f = extreme_scenarios(f)
        else:
            f = dict(f, snapshots=case["S"], S_load=np.ascontiguousarray(f["S_load"][:case["S"]]))
    if case["cfg"] in ("c3", "c4"):
        f = dict(f, v_min=0.90, v_max=1.10)
    return f


def _eligible_reduced(f):
    """Every eligible node moved to its nearest kept ancestor."""
    sup = np.arange(f["n"], dtype=np.int32)
    for i in _top_down(f["parent"]):
        if f["eligible"][i]:
            sup[i] = sup[f["parent"][i]]
    return sup


def _surrogate_inputs(case, seed):
    """Rows as the search's feature extraction leaves them (16 used features of
    order one, the rest zero), targets ln(error) and a network part-trained."""
    g = np.random.default_rng(seed)
    X = np.zeros((max(case["rows"], case["batch"]), SURR_FEATURES), np.float32)
    X[:, :16] = g.normal(0.3, 0.6, (X.shape[0], 16))
    t = (-9.0 + 1.5 * X[:, 0] - X[:, 3] + 0.3 * g.normal(size=X.shape[0])).astype(np.float32)
    return X, t


def prepare(case, seed):
    if case["kind"] == "surrogate":
        X, t = _surrogate_inputs(case, seed)
        X, t = torch.from_numpy(X).to(DEVICE), torch.from_numpy(t).to(DEVICE)
        B = case["batch"]
        return dict(case=case, X=X[:case["rows"]].contiguous(), Xb=X[:B].contiguous(), tb=t[:B].contiguous(),
                    params=surrogate.init_params(seed, DEVICE, b3=-9.0),
                    grads=torch.empty(SURR_PARAMS, dtype=torch.float32, device=DEVICE),
                    work=torch.empty(okr_surrogate_workspace(B), dtype=torch.uint8, device=DEVICE))
    f = _feeder(case, seed)
    if case["kind"] == "reduce":
        # a case's segment count depends on its seed: the decisions are handed
        # on in arrays of the node count
        return dict(case=case, R=Reducer(f, device=DEVICE, precision=case["precision"], secondary=case["secondary"],
                                         graph=case["graph"]),
                    decisions={key: np.zeros(f["n"], kind) for key, kind in DECISIONS})
    s = dict(case=case, G=Greedy(f, device=DEVICE))
    if case["kind"] == "evaluate":
        s["super"] = _eligible_reduced(f)
    return s


def run(state):
    case = state["case"]
    if case["kind"] == "reduce":
        R = state["R"]
        R.run(replan=case["replan"])
        seg = np.frombuffer(R.out_seg, dtype=R.out_seg._type_)[:R.sizes.n_segments]
        for key, a in state["decisions"].items():
            a[:len(seg)] = seg[key]
        return dict(super=R.out_super, kept_parent=R.out_kp, Yk_diag=R.out_Ykd, Yk_off=R.out_Yko, err=R.out_err,
                    max_err=R.res.max_err, n_kept=R.res.n_kept, **state["decisions"])
    if case["kind"] == "greedy":
        r = state["G"].run(case["e_bar"])
        steps, cand, smice = r["steps"], np.full(case["n"], -1, np.int32), np.zeros(case["n"])
        cand[:len(steps)] = [s["cand"] for s in steps]
        smice[:len(steps)] = [s["smice"] for s in steps]
        return dict(super=r["super"], err=r["err_per_snapshot"], max_err=r["max_err"], cand=cand, smice=smice)
    if case["kind"] == "evaluate":
        err, mx = state["G"].evaluate(state["super"])
        return dict(err=err, max_err=mx)
    loss = okr_surrogate_grad(state["params"], state["Xb"], state["tb"], state["grads"], state["work"])
    return dict(loss=loss, grads=state["grads"], y=surrogate.predict(state["params"], state["X"]))


# ---- what a pass cannot do without ----------------------------------------

def work(case):
    """Bytes: each input read once, each output written once.  Flops: a load
    flow of 8 iterations (per node, phase and snapshot: a load current, a sum
    and a 3x3 product), and per candidate one comparison per node that it
    reduces; for Algorithm 1 a state update per move; for the network its
    multiply-adds."""
    if case["kind"] == "surrogate":
        macs = 32 * 256 + 256 * 256 + 256
        rows, B = case["rows"], case["batch"]
        return dict(bytes=4 * (SURR_FEATURES * (rows + B) + B + rows + 3 * SURR_PARAMS),
                    flops=2.0 * macs * (rows + 3 * B))
    n, S = case["n"], case["S"]
    d = dict(bytes=n * S * 48 + 2 * n * 144 + 8 * S, flops=8.0 * n * S * 3 * 40)
    if case["kind"] == "reduce":
        k = 0.5 * (case["seg_lo"] + case["seg_hi"])
        segments = max(1.0, (0.4 if case["cfg"] == "c1" else 0.77) * n / k)
        masks = sum(2.0 ** j for j in range(case["seg_lo"], case["seg_hi"] + 1)) / (case["seg_hi"] - case["seg_lo"] + 1)
        d["bytes"] += 2 * n * 144 + 8 * n + 64 * segments
        d["flops"] += segments * masks * k
    elif case["kind"] == "greedy":
        d["bytes"] += 52 * n
        d["flops"] += 0.9 * n * (n * S * 3.0)
    return d


# ---- the same in 64 bits, from the definitions ----------------------------

def _top_down(parent):
    """Node ids, parents first (breadth-first)."""
    kids = [[] for _ in parent]
    for i in range(1, len(parent)):
        kids[int(parent[i])].append(i)
    order = [0]
    for v in order:
        order.extend(kids[v])
    return order


class _Net:
    """A feeder's tree by levels, its branch impedances and the two sweeps of
    a radial network, over all snapshots at once."""

    def __init__(self, f):
        self.dev = DEVICE if torch.cuda.is_available() else "cpu"
        self.f, self.n = f, f["n"]
        self.parent = np.asarray(f["parent"])
        self.order = _top_down(self.parent)
        depth = np.zeros(self.n, int)
        for i in self.order[1:]:
            depth[i] = depth[self.parent[i]] + 1
        by = [np.flatnonzero(depth == d) for d in range(1, depth.max() + 1)]
        self.levels = [(self._t(v), self._t(self.parent[v])) for v in by]
        self.present = (np.asarray(f["phase"])[:, None] >> np.arange(3)) & 1 == 1
        self.z = np.zeros((self.n, 3, 3), complex)
        for i in range(1, self.n):
            ix = np.flatnonzero(self.present[i])
            self.z[np.ix_([i], ix, ix)] = np.linalg.inv(-f["Y_off"][i][np.ix_(ix, ix)])
        self.zt = self._t(self.z)
        self.on = self._t(self.present)[:, None, :]
        # [node][snapshot][phase], so that a level is a contiguous gather
        self.S_load = self._t(np.ascontiguousarray(np.asarray(f["S_load"]).transpose(1, 0, 2)))
        self.V0 = self._t(np.asarray(f["V0"]))

    def _t(self, a):
        return torch.from_numpy(np.ascontiguousarray(a)).to(self.dev)

    def solve(self, I):
        """Voltages with the injected load currents I fixed."""
        J = I.clone()
        for v, p in reversed(self.levels):
            J.index_add_(0, p, J[v])
        V = torch.zeros_like(I)
        V[0] = self.V0
        for v, p in self.levels:
            V[v] = V[p] - (self.zt[v][:, None, :, :] * J[v][:, :, None, :]).sum(-1)
        return V * self.on

    def flow(self):
        """Constant-power load flow: (V, I)."""
        V = (self.V0 * torch.ones_like(self.S_load)) * self.on
        for _ in range(100):
            I = torch.where(self.on, (self.S_load / torch.where(self.on, V, torch.ones_like(V))).conj(), 0.0)
            W = self.solve(I)
            step = float((W - V).abs().max())
            V = W
            if step <= 1e-13:
                break
        return V, torch.where(self.on, (self.S_load / torch.where(self.on, V, torch.ones_like(V))).conj(), 0.0)

    def reduced(self, Vh, I, sup):
        """(largest error per snapshot, state voltages) of an assignment."""
        s = self._t(np.asarray(sup, np.int64))
        A = torch.zeros_like(I).index_add_(0, s, I)
        V = self.solve(A)
        e = (Vh.abs() - V[s].abs()).abs() * self.on
        return e.amax(dim=(0, 2)), V


def _kron(net, kept):
    """Kept parents and Y blocks of the radial reduced network."""
    kp = np.full(net.n, -1, np.int32)
    yd, yo = np.zeros((net.n, 3, 3), complex), np.zeros((net.n, 3, 3), complex)
    for i in range(1, net.n):
        if not kept[i]:
            continue
        z, a = net.z[i].copy(), net.parent[i]
        while not kept[a]:
            z, a = z + net.z[a], net.parent[a]
        kp[i] = a
        ix = np.flatnonzero(net.present[i])
        y = np.zeros((3, 3), complex)
        y[np.ix_(ix, ix)] = np.linalg.inv(z[np.ix_(ix, ix)])
        yo[i] = -y
        yd[i] += y
        yd[a] += y
    return kp, yd, yo


def _top_masks(net, f, Vh, I):
    """The assignment when every segment takes all of its nodes, or None where
    one of them may not (then the decisions need the enumeration)."""
    sup = np.arange(net.n)
    reduced = np.zeros(net.n, bool)
    for g in range(int(f["segment"].max()) + 1):
        reduced |= f["segment"] == g
        for i in net.order[1:]:
            sup[i] = sup[net.parent[i]] if reduced[i] else i
        e, V = net.reduced(Vh, I, sup)
        kept = net._t(~reduced)[:, None, None] & net.on
        m = V.abs()
        if not (float(e.max()) < f["e_bar"] - 1e-9 and float(torch.where(kept, m, 1.0).amin()) > f["v_min"] + 1e-9
                and float(torch.where(kept, m, 1.0).amax()) < f["v_max"] - 1e-9):
            return None
    return sup


def _one_segment(net, f, Vh, I):
    """The decision over every subset of a single segment: most reduced nodes,
    then the smallest error, then the lowest mask.  Levels are tried from the
    top, so the first with a feasible subset decides.  The error over all
    nodes orders the subsets as the error over the affected ones does where
    the unaffected nodes' error is zero, as it is with one segment."""
    pre, stack = [], [0]
    kids = [[] for _ in range(net.n)]
    for i in range(1, net.n):
        kids[net.parent[i]].append(i)
    while stack:
        v = stack.pop()
        pre.append(v)
        stack.extend(reversed(kids[v]))
    nodes = [v for v in pre if f["segment"][v] == 0]
    Z = np.zeros((net.n, net.n, 3, 3), complex)  # impedance of the common path to the slack
    for i in net.order[1:]:
        p = net.parent[i]
        Z[i] = Z[p]
        Z[:, i] = Z[:, p]
        Z[i, i] = Z[p, p] + net.z[i]
    Vh, I = Vh[:, 0].cpu().numpy(), I[:, 0].cpu().numpy()
    Zm = Z.transpose(0, 2, 1, 3).reshape(3 * net.n, 3 * net.n)
    V0 = np.tile(np.asarray(f["V0"]), net.n)
    on = net.present.reshape(-1)
    for level in range(len(nodes), -1, -1):
        masks = [m for m in range(1 << len(nodes)) if bin(m).count("1") == level]
        sups, A = np.empty((len(masks), net.n), int), np.zeros((len(masks), net.n, 3), complex)
        for q, m in enumerate(masks):
            red = {v for j, v in enumerate(nodes) if m >> j & 1}
            sup = sups[q]
            for i in net.order:
                sup[i] = sup[net.parent[i]] if i in red else i
            np.add.at(A[q], sup, I)
        V = ((V0 - A.reshape(len(masks), -1) @ Zm.T) * on).reshape(len(masks), net.n, 3)
        mag = np.abs(V)
        e = np.abs(np.abs(Vh)[None] - np.take_along_axis(mag, sups[:, :, None].repeat(3, 2), 1) * net.present)
        e = e.max(axis=(1, 2))
        kept = (sups == np.arange(net.n))[:, :, None] & net.present[None]
        lo, hi = np.where(kept, mag, 1.0).min(axis=(1, 2)), np.where(kept, mag, 1.0).max(axis=(1, 2))
        best = np.flatnonzero((e <= f["e_bar"]) & (lo >= f["v_min"]) & (hi <= f["v_max"]))
        if len(best):
            near = best[e[best] <= e[best].min() + 1e-11]
            return sups[near.min()], masks[near.min()]
    return None, None


def exact(case, seed):
    if case["kind"] == "greedy":
        return None
    if case["kind"] == "surrogate":
        X, t = (torch.from_numpy(a).double() for a in _surrogate_inputs(case, seed))
        p = surrogate.init_params(seed, "cpu", b3=-9.0).double().requires_grad_()
        a = np.cumsum([256 * 32, 256, 256 * 256, 256, 256])
        W1, b1, W2, b2, w3, b3 = torch.tensor_split(p, a.tolist())

        def net(x):
            h = torch.nn.functional.gelu(x @ W1.view(256, 32).T + b1)
            return torch.nn.functional.gelu(h @ W2.view(256, 256).T + b2) @ w3 + b3
        B = case["batch"]
        loss = ((net(X[:B]) - t[:B]) ** 2).mean()
        loss.backward()
        with torch.no_grad():
            return dict(loss=float(loss), grads=p.grad, y=net(X[:case["rows"]]))
    f = _feeder(case, seed)
    net = _Net(f)
    Vh, I = net.flow()
    if case["kind"] == "evaluate":
        e, _ = net.reduced(Vh, I, _eligible_reduced(f))
        return dict(err=e.cpu().numpy(), max_err=float(e.max()))
    if case["cfg"] == "c1" and case["secondary"] == "maxerr" and case["S"] == 1:
        sup, m = _one_segment(net, f, Vh, I)
        mask = [m]
    else:
        sup = _top_masks(net, f, Vh, I)
        if sup is not None:
            mask = [(1 << int((f["segment"] == g).sum())) - 1 for g in range(int(f["segment"].max()) + 1)]
    if sup is None:
        return None
    e, _ = net.reduced(Vh, I, sup)
    kept = np.asarray(sup) == np.arange(net.n)
    mask = np.pad(np.array(mask, np.uint32), (0, net.n - len(mask)))
    kp, yd, yo = _kron(net, kept)
    return dict(super=np.asarray(sup, np.int32), kept_parent=kp, Yk_diag=yd, Yk_off=yo, err=e.cpu().numpy(),
                max_err=float(e.max()), n_kept=int(kept.sum()), mask=mask, e_loc=None, key_gap=None, smice_rise=None)
