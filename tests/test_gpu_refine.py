"""GPU parity of the max-flow guided refinement (Sec. 3.4): edge classes, guided moves, the
column gather and whole refinement rounds, through the C-ABI, against the CPU oracle on the
same seeded inputs.  Everything here is integer or byte work and must be bit-exact.  The edge
classes do not depend on which maximum flow is used, so the GPU's classes (from its own
push-relabel flow) must equal the oracle's (from Edmonds-Karp)."""
import os
import sys

import numpy as np
import pytest

from oracle import hxo
from paper_2502_07903_amd import hx
from paper_2502_07903_amd import inputs as I
from tests import helpers as Hh

pytestmark = pytest.mark.gpu
N_THREADS = max(1, min(16, os.cpu_count() or 1))


def say(msg: str) -> None:
    print(f"[gpu] {msg}", flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def torch():
    import torch as T
    if not T.cuda.is_available():
        pytest.fail("GPU tests need a ROCm GPU (torch.cuda.is_available() is False)")
    hx.lib()
    return T


def gpu_classes(torch, dp):
    """Score dp on the GPU with a flow assignment, then its edge classes."""
    ws = hx.Workspace.for_problem(dp, flows=True)
    hx.score(dp, ws)
    mp, md, mpd = ws.net.dims
    N = dp.n_cand
    node = torch.full((mp + md, N), 0xEE, dtype=torch.uint8, device="cuda")
    kv = torch.full((mpd, N), 0xEE, dtype=torch.uint8, device="cuda")
    hx.edge_classes(ws.net, ws.flow_value, ws.kv_flow, node, kv)
    torch.cuda.synchronize()
    return ws, node, kv


def compare_classes(fn, got_node, got_kv, want):
    mp = fn["dims"][0]
    for n in range(fn["n_p"].shape[0]):
        P, D = int(fn["n_p"][n]), int(fn["n_d"][n])
        rows = list(range(P)) + [mp + j for j in range(D)]
        assert np.array_equal(got_node[rows, n], want["node_cls"][rows, n]), f"node classes differ at {n}"
        assert np.array_equal(got_kv[:P * D, n], want["kv_cls"][:P * D, n]), f"KV classes differ at {n}"


@pytest.mark.parametrize("cfg,n", [(1, 256), (2, 1024), (3, 2048), (4, 512), (5, 48)])
def test_edge_classes_workloads(torch, cfg, n):
    prob = I.make_problem(cfg, n_cand=n)
    say(f"edge classes: workload {cfg}, N={n}")
    dp = hx.DeviceProblem.upload(prob)
    ws, node, kv = gpu_classes(torch, dp)
    fn = ws.net.host()
    want_fn = hxo.build_flownet(prob, hxo.cost_eval(prob))
    Hh.compare_flownet(fn, want_fn)
    compare_classes(fn, node.cpu().numpy(), kv.cpu().numpy(), hxo.edge_classes(want_fn))


def test_edge_classes_random_networks(torch):
    """Random capacities, including zeros and unbounded edges, over P, D <= 12."""
    rng = np.random.default_rng(91)
    N, mp, md = 1500, 12, 12
    mpd = mp * md
    fn = dict(n_p=rng.integers(0, mp + 1, N).astype(np.int32), n_d=rng.integers(0, md + 1, N).astype(np.int32),
              dims=(mp, md, mpd))
    for k, rows in (("src_cap", mp), ("p_cap", mp), ("d_cap", md), ("sink_cap", md), ("kv_cap", mpd),
                    ("p_slot", mp), ("d_slot", md)):
        hi = rng.choice([1, 3, 50, 10 ** 5], size=N)
        fn[k] = (rng.random((rows, N)) * (hi[None, :] + 1)).astype(np.int32)
        if k in ("src_cap", "sink_cap"):
            fn[k] = np.where(rng.random((rows, N)) < 0.5, Hh.CAP_MAX, fn[k]).astype(np.int32)
    nb = hx.FlowNetBuffers.from_host(fn)
    fv = torch.empty(N, dtype=torch.int32, device="cuda")
    kvf = torch.zeros((mpd, N), dtype=torch.int32, device="cuda")
    cut = torch.zeros((mp + md, N), dtype=torch.uint8, device="cuda")
    hx.maxflow_batch(nb, fv, kvf, cut)
    node = torch.full((mp + md, N), 0xEE, dtype=torch.uint8, device="cuda")
    kv = torch.full((mpd, N), 0xEE, dtype=torch.uint8, device="cuda")
    say(f"edge classes: {N} random networks")
    hx.edge_classes(nb, fv, kvf, node, kv)
    torch.cuda.synchronize()
    compare_classes(fn, node.cpu().numpy(), kv.cpu().numpy(), hxo.edge_classes(fn))


@pytest.mark.parametrize("P,D,room", [(1, 1, 0), (31, 31, 0), (30, 33, 0), (32, 32, 0), (31, 33, 1), (31, 32, 3), (62, 64, 0),
                                      (64, 64, 0), (120, 62, 0), (95, 66, 0), (200, 30, 0), (25, 230, 0), (230, 25, 0)])
def test_edge_classes_closure_blocks(torch, P, D, room):
    """Networks of P x D nodes around the closure's sizes: one to five words a row, the last vertices on
    either side of a 64-pivot block, one wavefront or four per network (by the room of the arrays),
    with capacities small enough that edges saturate everywhere; every class equal to the oracle's."""
    rng = np.random.default_rng([91, P, D])
    N, mp, md = (21 if P + D < 132 else 4), P + room, D
    mpd = mp * md
    fn = dict(n_p=np.full(N, P, np.int32), n_d=np.full(N, D, np.int32), dims=(mp, md, mpd))
    for k, rows in (("src_cap", mp), ("p_cap", mp), ("d_cap", md), ("sink_cap", md), ("kv_cap", mpd),
                    ("p_slot", mp), ("d_slot", md)):
        hi = rng.choice([1, 3, 50, 10 ** 5], size=N)
        fn[k] = (rng.random((rows, N)) * (hi[None, :] + 1)).astype(np.int32)
        if k in ("src_cap", "sink_cap"):
            fn[k] = np.where(rng.random((rows, N)) < 0.5, Hh.CAP_MAX, fn[k]).astype(np.int32)
    fn["n_p"][::5] = np.maximum(P - np.arange(len(fn["n_p"][::5])), 0)
    nb = hx.FlowNetBuffers.from_host(fn)
    fv = torch.empty(N, dtype=torch.int32, device="cuda")
    kvf = torch.zeros((mpd, N), dtype=torch.int32, device="cuda")
    say(f"edge classes: {P} x {D} nodes, room {room}")
    hx.maxflow_batch(nb, fv, kvf)
    node = torch.full((mp + md, N), 0xEE, dtype=torch.uint8, device="cuda")
    kv = torch.full((mpd, N), 0xEE, dtype=torch.uint8, device="cuda")
    hx.edge_classes(nb, fv, kvf, node, kv)
    torch.cuda.synchronize()
    compare_classes(fn, node.cpu().numpy(), kv.cpu().numpy(), hxo.edge_classes(fn))


def test_edge_classes_beyond_closure_rows(torch):
    """A network of more than 255 nodes gets no classes (node rows 0); its neighbours do."""
    mp, md = 200, 100
    fn = dict(n_p=np.array([200, 1], np.int32), n_d=np.array([100, 1], np.int32), dims=(mp, md, mp * md))
    for k, rows in (("src_cap", mp), ("p_cap", mp), ("d_cap", md), ("sink_cap", md), ("kv_cap", mp * md),
                    ("p_slot", mp), ("d_slot", md)):
        fn[k] = np.zeros((rows, 2), np.int32)
    fn["src_cap"][0, 1] = fn["p_cap"][0, 1] = fn["kv_cap"][0, 1] = fn["sink_cap"][0, 1] = 10
    fn["d_cap"][0, 1] = 4
    nb = hx.FlowNetBuffers.from_host(fn)
    fv = torch.tensor([0, 4], dtype=torch.int32, device="cuda")           # zero capacities: zero flow
    kvf = torch.zeros((mp * md, 2), dtype=torch.int32, device="cuda")
    kvf[0, 1] = 4
    node = torch.full((mp + md, 2), 0xEE, dtype=torch.uint8, device="cuda")
    kv = torch.full((mp * md, 2), 0xEE, dtype=torch.uint8, device="cuda")
    hx.edge_classes(nb, fv, kvf, node, kv)
    torch.cuda.synchronize()
    node = node.cpu().numpy()
    assert (node[:, 0] == 0).all()
    want = hxo.edge_classes({k: (np.ascontiguousarray(v[..., 1:]) if isinstance(v, np.ndarray) else v)
                             for k, v in fn.items()})
    assert node[0, 1] == want["node_cls"][0, 0] and node[mp, 1] == want["node_cls"][mp, 0]
    assert node[mp, 1] & 1                                                 # the decode node is the bottleneck


def _parents(torch, cfg, idx):
    prob = I.make_problem(cfg, n_cand=int(max(idx)) + 1).subset(np.asarray(idx))
    dp = hx.DeviceProblem.upload(prob)
    ws, node, _ = gpu_classes(torch, dp)
    return prob, dp, ws, node


@pytest.mark.parametrize("cfg,idx,n_child", [(1, [0], 1), (1, [3, 5, 8], 1000), (2, list(range(7)), 4097),
                                             (3, [11, 40], 3001), (5, [0], 131072), (5, [2, 9, 17], 2000)])
def test_guided_moves_parity(torch, cfg, idx, n_child):
    prob, dp, ws, node = _parents(torch, cfg, idx)
    rnd_h = I.move_draws(cfg, 7, n_child)
    rnd = torch.as_tensor(rnd_h.view(np.int64)).to("cuda")
    ca = torch.full((prob.n_gpus, n_child), 0xEE, dtype=torch.uint8, device="cuda")
    cr = torch.full((prob.max_groups, n_child), 0xEE, dtype=torch.uint8, device="cuda")
    mv = torch.full((n_child,), -7, dtype=torch.int32, device="cuda")
    say(f"guided moves: workload {cfg}, parents {idx}, {n_child} children")
    hx.guided_moves(dp, ws.net, node, rnd, ca, cr, mv)
    torch.cuda.synchronize()
    fn = hxo.build_flownet(prob, hxo.cost_eval(prob))
    want = hxo.guided_moves(prob.n_gpus, prob.max_groups, prob.granularity, prob.assign, prob.role, fn,
                            hxo.edge_classes(fn), rnd_h)
    got_m = mv.cpu().numpy()
    bad = np.flatnonzero(got_m != want["move"])
    assert bad.size == 0, f"moves differ at {bad[:5].tolist()}: {got_m[bad[:5]]} vs {want['move'][bad[:5]]}"
    assert np.array_equal(ca.cpu().numpy(), want["assign"])
    assert np.array_equal(cr.cpu().numpy(), want["role"])
    say(f"guided moves: types {np.bincount(got_m & 0xFF, minlength=4).tolist()}")


def test_gather(torch):
    prob = I.make_problem(2, n_cand=300)
    dp = hx.DeviceProblem.upload(prob)
    index = np.array([5, 299, 0, -1, 300, 5, 17], np.int32)
    idx = torch.as_tensor(index).to("cuda")
    da = torch.zeros((prob.n_gpus, len(index)), dtype=torch.uint8, device="cuda")
    dr = torch.zeros((prob.max_groups, len(index)), dtype=torch.uint8, device="cuda")
    hx.gather_candidates(dp, idx, da, dr)
    torch.cuda.synchronize()
    ok = (index >= 0) & (index < 300)
    want_a = np.where(ok[None, :], prob.assign[:, np.clip(index, 0, 299)], I.UNUSED)
    want_r = np.where(ok[None, :], prob.role[:, np.clip(index, 0, 299)], I.UNUSED)
    assert np.array_equal(da.cpu().numpy(), want_a)
    assert np.array_equal(dr.cpu().numpy(), want_r)


def _oracle_round(prob_parent, rnd_h):
    """One refinement round on the CPU oracle: the parent's classes, its children, their
    scores and the best child."""
    fn = hxo.build_flownet(prob_parent, hxo.cost_eval(prob_parent))
    cls = hxo.edge_classes(fn)
    ch = hxo.guided_moves(prob_parent.n_gpus, prob_parent.max_groups, prob_parent.granularity,
                          prob_parent.assign, prob_parent.role, fn, cls, rnd_h)
    import dataclasses
    child_prob = dataclasses.replace(prob_parent, assign=ch["assign"], role=ch["role"])
    res = hxo.score_batch(child_prob, n_threads=N_THREADS)
    return ch, res


@pytest.mark.parametrize("cfg,n_child,rounds", [(2, 2048, 4), (5, 2048, 3)])
def test_refiner_rounds(torch, cfg, n_child, rounds):
    """Whole rounds on the device (hx.Refiner: score parent with flows, classes, guided moves,
    score children, gather the best) against the same loop on the oracle, round by round."""
    import dataclasses
    prob = I.make_problem(cfg, n_cand=64)
    res0 = hxo.score_batch(prob, n_threads=N_THREADS)
    start = res0["best"][0]
    dp = hx.DeviceProblem.upload(prob)
    ref = hx.Refiner.create(dp, start, n_child)
    parent = prob.subset(np.array([start]))
    value = res0["best"][1]
    for r in range(rounds):
        rnd_h = I.move_draws(cfg, r, n_child)
        say(f"refiner: workload {cfg}, round {r}, {n_child} children")
        ref.round(torch.as_tensor(rnd_h.view(np.int64)).to("cuda"))
        torch.cuda.synchronize()
        ch, res = _oracle_round(parent, rnd_h)
        assert np.array_equal(ref.move.cpu().numpy(), ch["move"]), f"round {r}: moves differ"
        assert np.array_equal(ref.child_ws.flow_value.cpu().numpy(), res["flow_value"]), f"round {r}: flows differ"
        best = tuple(int(x) for x in ref.child_ws.best.cpu().numpy())
        assert best == res["best"], f"round {r}: best {best} vs {res['best']}"
        assert best[1] >= value, "a round may never lose the parent's score"
        value = best[1]
        parent = dataclasses.replace(parent, assign=np.ascontiguousarray(ch["assign"][:, best[0]:best[0] + 1]),
                                     role=np.ascontiguousarray(ch["role"][:, best[0]:best[0] + 1]))
        assert np.array_equal(ref.parent.tensors["assign"].cpu().numpy(), parent.assign)
        assert np.array_equal(ref.parent.tensors["role"].cpu().numpy(), parent.role)


def test_profile_sees_refinement_kernels(torch):
    prob = I.make_problem(2, n_cand=16)
    dp = hx.DeviceProblem.upload(prob)
    ref = hx.Refiner.create(dp, 0, 512)
    rnd = torch.as_tensor(I.move_draws(2, 0, 512).view(np.int64)).to("cuda")
    hx.profile(True)
    ref.round(rnd)
    prof = hx.profile_read()
    hx.profile(False)
    for name in ("classes", "moves", "gather"):
        assert prof[name][1] == 1 and prof[name][0] > 0.0, (name, prof[name])
