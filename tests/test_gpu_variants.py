"""GPU parity of the cost-model variants against the oracle, through the C-ABI: with the
pipelined decode capacity (HX_VARIANT_PIPELINED) every strategy choice, batch limit,
capacity and latency, the networks built on them, every flow value and the best candidate
must equal the oracle's (integers bit-exact, latencies to 1e-5 relative and expected
bit-identical)."""
import dataclasses
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
PIPE = 1


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


def _gpu(torch, prob):
    dp = hx.DeviceProblem.upload(prob)
    assert dp.space.variant == prob.variant
    ws = hx.Workspace.for_problem(dp)
    hx.score(dp, ws)
    torch.cuda.synchronize()
    return ({k: getattr(ws.cost, k).cpu().numpy() for k in ("tp", "pp", "bmax", "cap", "lat")}, ws.net.host(),
            ws.flow_value.cpu().numpy(), tuple(int(x) for x in ws.best.cpu().numpy()))


@pytest.mark.parametrize("cfg,n", [(1, None), (2, None), (3, None), (3, 4097), (4, 4096), (2, 1)])
def test_pipelined_parity(torch, cfg, n):
    prob = dataclasses.replace(I.make_problem(cfg, n_cand=n), variant=PIPE)
    say(f"pipelined decode capacity: workload {cfg}, N={prob.n_cand}")
    cost, fn, fv, best = _gpu(torch, prob)
    want = hxo.score_batch(prob, n_threads=N_THREADS)
    for k in ("tp", "pp", "bmax", "cap"):
        bad = cost[k] != want["cost"][k]
        assert not bad.any(), f"{k} differs at {np.argwhere(bad)[:5].tolist()}"
    rel = np.abs(cost["lat"] - want["cost"]["lat"]) / np.maximum(np.abs(want["cost"]["lat"]), 1e-300)
    assert (rel <= 1e-5).all()
    assert np.array_equal(cost["lat"], want["cost"]["lat"])
    Hh.compare_flownet(fn, want["flownet"])
    assert np.array_equal(fv, want["flow_value"])
    assert best == want["best"]
    # the variant moves decode capacities only, and only up
    base = hxo.cost_eval(dataclasses.replace(prob, variant=0))
    dec = prob.role == I.DECODE
    assert (cost["cap"][dec] >= base["cap"][dec]).all()
    assert np.array_equal(cost["cap"][prob.role == I.PREFILL], base["cap"][prob.role == I.PREFILL])


def test_pipelined_per_gpu_nodes(torch):
    """Per-GPU flow nodes (128 GPUs) with the variant, on a seeded sample of round 0."""
    prob = dataclasses.replace(I.make_problem(5, n_cand=1024), variant=PIPE)
    say("pipelined decode capacity: per-GPU nodes, N=1024")
    cost, fn, fv, best = _gpu(torch, prob)
    want = hxo.score_batch(prob, n_threads=N_THREADS)
    for k in ("tp", "pp", "bmax", "cap", "lat"):
        assert np.array_equal(cost[k], want["cost"][k]), k
    assert np.array_equal(fv, want["flow_value"])
    assert best == want["best"]


def test_unknown_variant_rejected(torch):
    prob = dataclasses.replace(I.make_problem(1, n_cand=4), variant=8)
    dp = hx.DeviceProblem.upload(prob)
    ws = hx.Workspace.for_problem(dp)
    with pytest.raises(hx.HxError) as e:
        hx.cost_eval(dp, ws.cost)
    assert e.value.code == hx.HX_EINVAL


ORDER = 2


@pytest.mark.parametrize("cfg,n,variant", [(1, None, ORDER), (2, None, ORDER), (3, 16384, ORDER), (4, 2048, ORDER),
                                           (4, 8191, ORDER), (2, 777, ORDER | PIPE), (3, 4096, ORDER | PIPE)])
def test_kv_order_parity(torch, cfg, n, variant):
    """KV stage-order search (alone and with the pipelined capacity), exact at every pipeline depth
    up to 8 stages: KV capacities, flows and the best candidate equal the oracle's; every KV
    capacity is at least the ascending-order one."""
    prob = dataclasses.replace(I.make_problem(cfg, n_cand=n), variant=variant)
    say(f"KV stage-order search: workload {cfg}, N={prob.n_cand}, variant {variant}")
    cost, fn, fv, best = _gpu(torch, prob)
    want = hxo.score_batch(prob, n_threads=N_THREADS)
    for k in ("tp", "pp", "bmax", "cap", "lat"):
        assert np.array_equal(cost[k], want["cost"][k]), k
    Hh.compare_flownet(fn, want["flownet"])
    assert np.array_equal(fv, want["flow_value"])
    assert best == want["best"]
    asc = hxo.build_flownet(dataclasses.replace(prob, variant=variant & ~ORDER),
                            hxo.cost_eval(dataclasses.replace(prob, variant=variant & ~ORDER)))
    up, ud, upd = Hh.used_rows(fn)
    assert (fn["kv_cap"][upd] >= asc["kv_cap"][upd]).all()


@pytest.mark.parametrize("tiles,spare", [(256, 1), (257, 1), (3, 5)])
def test_kv_order_large_grids(torch, tiles, spare):
    """The stage-order search over more (edge, candidate) cells than one launch has lanes for: 2,048
    candidates of workload 4 (256 KV rows) repeated 256 times are 2^27 cells, 257 times more than that,
    with the arrays' own rows; and arrays with five times the rows a network can have.  Every repetition's
    KV rows, flow values and the best equal those of the 2,048 candidates alone."""
    n = 2048
    prob = dataclasses.replace(I.make_problem(4, n_cand=n), variant=ORDER)
    dp = hx.DeviceProblem.upload(prob)
    one = hx.Workspace.for_problem(dp)
    hx.score_batch(dp, one)
    many = dp.with_candidates(dp.tensors["assign"].repeat(1, tiles), dp.tensors["role"].repeat(1, tiles))
    ws = hx.Workspace.for_problem(many)
    mp, md, mpd = ws.net.dims
    ws.net = hx.FlowNetBuffers.empty((mp, md, mpd * spare), n * tiles, fill=-1)
    say(f"KV stage-order search: {mpd * spare} rows x {n * tiles} candidates")
    hx.score_batch(many, ws)
    torch.cuda.synchronize()
    used = torch.arange(mpd, device="cuda")[:, None] < (one.net.n_p * one.net.n_d)[None, :]
    kv = ws.net.kv_cap.view(mpd * spare, tiles, n)
    for i in range(tiles):
        assert bool((~used | (kv[:mpd, i] == one.net.kv_cap)).all()), f"repetition {i}"
    assert bool((kv[mpd:] == -1).all())
    assert bool((ws.flow_value.view(tiles, n) == one.flow_value).all())
    assert ws.best.tolist() == one.best.tolist()


def test_kv_order_single_slot(torch):
    """One group slot: networks that have no KV row."""
    a, r = I.placement_from_groups([list(range(8))], [I.PREFILL], 8, 1)
    for variant in (0, ORDER):
        prob = dataclasses.replace(Hh.problem(Hh.cluster_c1(), Hh.MODELS["opt30b"], a, r), variant=variant)
        dp = hx.DeviceProblem.upload(prob)
        ws = hx.Workspace.for_problem(dp)
        ws.net = hx.FlowNetBuffers.empty((1, 1, 1), 1, fill=-1)
        for call in (hx.score, hx.score_batch):
            call(dp, ws)
            torch.cuda.synchronize()
            assert (ws.net.n_p.tolist(), ws.net.n_d.tolist(), ws.net.kv_cap.tolist()) == ([1], [0], [[-1]])
            assert ws.flow_value.tolist() == [0] and ws.best.tolist() == [0, 0]


@pytest.mark.parametrize("dpp", [8, 4])
def test_kv_order_deep_hidden_pairing(torch, dpp):
    """Eight one-GPU prefill stages against eight or four one-GPU decode stages whose fast links
    follow a hidden pairing (the oracle's hand-derived case): the searched KV edge carries every
    overlapping block on a 300 GB/s link, 6 layers each."""
    pi = [3, 6, 0, 7, 2, 5, 1, 4]
    G = 16
    beta = np.full((G, G), 10e9)
    for i in range(8):
        for t in range(8):
            if (pi[i] == t) if dpp == 8 else (pi[i] // 2 == t):
                beta[i, 8 + t] = beta[8 + t, i] = 300e9
    np.fill_diagonal(beta, 0.0)
    tt = np.array([I.GPU_TYPES["A"]], np.float64)
    cl = I.Cluster(np.zeros(G, np.int32), tt[:, 0].copy(), tt[:, 1].copy(), tt[:, 2].copy(),
                   np.ascontiguousarray(beta.reshape(-1)), np.zeros(G * G))
    a, r = I.placement_from_groups([list(range(8)), list(range(8, 8 + dpp))], [I.PREFILL, I.DECODE], G, 2)
    prob = Hh.problem(cl, dict(I.OPT_30B), a, r, s_in=512.0, s_out=128.0, tp=(1,), pp=(4, 8))
    prob = dataclasses.replace(prob, variant=ORDER)
    say(f"KV stage-order search: 8 x {dpp} hidden pairing")
    cost, fn, fv, best = _gpu(torch, prob)
    want = hxo.score_batch(prob)
    assert cost["pp"][0, 0] == 8 and cost["pp"][1, 0] == dpp
    V6 = 2.0 * 512.0 * 7168 * 2 * 6
    assert int(fn["kv_cap"][0, 0]) == int(np.floor(1000.0 / (V6 / 300e9)))
    Hh.compare_flownet(fn, want["flownet"])
    assert np.array_equal(fv, want["flow_value"])


def test_kv_order_crossed_links(torch):
    """The hand-derived crossed-link case: the searched order pairs the 300 GB/s links."""
    G = 4
    beta = np.full((G, G), 10e9)
    for a, b in ((0, 3), (1, 2)):
        beta[a, b] = beta[b, a] = 300e9
    np.fill_diagonal(beta, 0.0)
    t = np.array([I.GPU_TYPES["A"]], np.float64)
    cl = I.Cluster(np.zeros(G, np.int32), t[:, 0].copy(), t[:, 1].copy(), t[:, 2].copy(),
                   np.ascontiguousarray(beta.reshape(-1)), np.zeros(G * G))
    a, r = I.placement_from_groups([[0, 1], [2, 3]], [I.PREFILL, I.DECODE], 4, 2)
    for variant, bw in ((0, 10e9), (ORDER, 300e9)):
        prob = dataclasses.replace(Hh.problem(cl, dict(I.OPT_30B), a, r, tp=(1,), pp=(2,)), variant=variant)
        _, fn, _, _ = _gpu(torch, prob)
        V = 2.0 * 512.0 * 7168 * 2 * 24
        assert int(fn["kv_cap"][0, 0]) == int(np.floor(1000.0 / (V / bw)))


ASYM = 4


@pytest.mark.parametrize("cfg,n,variant", [(1, None, ASYM), (2, None, ASYM), (3, None, ASYM), (4, 4096, ASYM),
                                           (3, 8192, ASYM | PIPE), (2, 777, ASYM | PIPE)])
def test_asym_parity(torch, cfg, n, variant):
    """Asymmetric layer split (alone and with the pipelined capacity): every strategy, capacity,
    latency, KV edge, flow and the best candidate equal the oracle's."""
    prob = dataclasses.replace(I.make_problem(cfg, n_cand=n), variant=variant)
    say(f"asymmetric layer split: workload {cfg}, N={prob.n_cand}, variant {variant}")
    cost, fn, fv, best = _gpu(torch, prob)
    want = hxo.score_batch(prob, n_threads=N_THREADS)
    for k in ("tp", "pp", "bmax", "cap"):
        bad = cost[k] != want["cost"][k]
        assert not bad.any(), f"{k} differs at {np.argwhere(bad)[:5].tolist()}"
    assert np.array_equal(cost["lat"], want["cost"]["lat"])
    Hh.compare_flownet(fn, want["flownet"])
    assert np.array_equal(fv, want["flow_value"])
    assert best == want["best"]


def test_asym_per_gpu_nodes(torch):
    prob = dataclasses.replace(I.make_problem(5, n_cand=1024), variant=ASYM)
    say("asymmetric layer split: per-GPU nodes, N=1024")
    cost, fn, fv, best = _gpu(torch, prob)
    want = hxo.score_batch(prob, n_threads=N_THREADS)
    for k in ("tp", "pp", "bmax", "cap", "lat"):
        assert np.array_equal(cost[k], want["cost"][k]), k
    assert np.array_equal(fv, want["flow_value"])


def test_asym_with_kv_order_rejected(torch):
    prob = dataclasses.replace(I.make_problem(1, n_cand=4), variant=ASYM | ORDER)
    dp = hx.DeviceProblem.upload(prob)
    ws = hx.Workspace.for_problem(dp)
    with pytest.raises(hx.HxError) as e:
        hx.cost_eval(dp, ws.cost)
    assert e.value.code == hx.HX_EINVAL
