"""hx_score_batch, the whole scoring path in one value-only call, through the C-ABI: on every
workload its cost outputs, node counts, flow values and best equal the four calls' bit for bit
(and every node and KV row too at replica granularity); on per-GPU networks whose KV edges bind
(slow links) the networks it hands to push-relabel are solved to the oracle's values; ragged
batch sizes and request classes."""
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


def _both(torch, prob):
    """(four calls, one call): host copies of every output."""
    dp = hx.DeviceProblem.upload(prob)
    out = []
    for fused in (False, True):
        ws = hx.Workspace.for_problem(dp, flows=False)
        for t in (ws.flow_value, ws.best, ws.net.kv_cap):
            t.fill_(-7)
        if fused:
            hx.score_batch(dp, ws)
        else:
            hx.score(dp, ws)
        torch.cuda.synchronize()
        out.append(dict(cost={k: getattr(ws.cost, k).cpu().numpy() for k in ("tp", "pp", "bmax", "cap", "lat", "members")},
                        net=ws.net.host(), flow_value=ws.flow_value.cpu().numpy(),
                        best=tuple(int(x) for x in ws.best.cpu().numpy())))
    return out


def _same(a, b, granularity):
    for k in a["cost"]:
        assert np.array_equal(a["cost"][k].view(np.uint8), b["cost"][k].view(np.uint8)), f"cost {k} differs"
    assert np.array_equal(a["net"]["n_p"], b["net"]["n_p"]) and np.array_equal(a["net"]["n_d"], b["net"]["n_d"])
    if granularity == 0:  # per-GPU networks settled from the link table keep their rows unwritten
        up, ud, upd = Hh.used_rows(a["net"])
        for k in ("p_slot", "src_cap", "p_cap"):
            assert np.array_equal(a["net"][k][up], b["net"][k][up]), k
        for k in ("d_slot", "d_cap", "sink_cap"):
            assert np.array_equal(a["net"][k][ud], b["net"][k][ud]), k
        assert np.array_equal(a["net"]["kv_cap"][upd], b["net"]["kv_cap"][upd])
    bad = np.flatnonzero(a["flow_value"] != b["flow_value"])
    assert bad.size == 0, f"flow values differ at {bad[:8].tolist()}"
    assert a["best"] == b["best"]


@pytest.mark.parametrize("cfg,n", [(1, None), (2, None), (3, None), (4, None), (5, None), (3, 1), (5, 7), (5, 777),
                                   (2, 4097)])
def test_score_batch_matches_four_calls(torch, cfg, n):
    prob = I.make_problem(cfg, n_cand=n)
    say(f"hx_score_batch vs four calls: workload {cfg}, N={prob.n_cand}")
    four, one = _both(torch, prob)
    _same(four, one, prob.granularity)
    # and the oracle, on the whole batch (workloads 1-3) or a sample
    idx = np.arange(prob.n_cand) if cfg <= 3 else np.unique(np.concatenate(
        [np.random.default_rng(cfg).choice(prob.n_cand, min(prob.n_cand, 1024), replace=False), [one["best"][0]]]))
    want = hxo.score_batch(prob.subset(idx), n_threads=N_THREADS)
    assert np.array_equal(one["flow_value"][idx], want["flow_value"])
    if cfg <= 3:
        assert one["best"] == want["best"]


def test_score_batch_request_classes_per_gpu(torch):
    prob = I.make_problem(5, n_cand=2048)
    prob = dataclasses.replace(prob, classes=I.length_classes(I.WORKLOADS[5], 4))
    say("hx_score_batch vs four calls: per-GPU networks, four request classes")
    four, one = _both(torch, prob)
    _same(four, one, 1)


def test_score_batch_per_gpu_binding_kv(torch):
    """The 128-GPU cluster with every link 100 times slower: KV edges fall below the node shares,
    so networks are handed to push-relabel with their KV rows; their values equal the oracle's
    (a sample) and the four calls' (all)."""
    prob = I.make_problem(5, n_cand=2048)
    cl = dataclasses.replace(prob.cluster, beta=np.ascontiguousarray(np.asarray(prob.cluster.beta) * 0.01))
    prob = dataclasses.replace(prob, cluster=cl)
    say("hx_score_batch: per-GPU networks with binding KV edges")
    four, one = _both(torch, prob)
    _same(four, one, 1)
    dp = hx.DeviceProblem.upload(prob)
    ws = hx.Workspace.for_problem(dp, flows=False)
    st = hx.maxflow_stats(_net_of(torch, dp, ws), torch.empty_like(ws.flow_value))
    assert st["push_relabel"] > 100, st
    idx = np.random.default_rng(51).choice(prob.n_cand, 96, replace=False)
    want = hxo.score_batch(prob.subset(idx), n_threads=N_THREADS)
    assert np.array_equal(one["flow_value"][idx], want["flow_value"])


def _net_of(torch, dp, ws):
    """The full network of the batch (the four calls' cost model and builder), for the counters."""
    hx.cost_eval(dp, ws.cost)
    hx.build_flownet(dp, ws.cost, ws.net)
    torch.cuda.synchronize()
    return ws.net


@pytest.mark.parametrize("cfg,sizes", [(3, (65536, 1, 1023, 1025, 4097)), (5, (131072, 777))])
def test_score_batch_argmax_over_workgroups(torch, cfg, sizes):
    """The value-only call's argmax: for replica networks each max-flow wavefront folds its best
    candidate into one of the workspace's slots (zeroed by the call's first kernel) and one
    workgroup reduces them; for per-GPU networks the batch is split over up to 256 workgroups and
    the last one to finish reduces their winners (its counter lives in the workspace). With the
    workspace filled with garbage before every call, and batch sizes from one candidate up, the
    best equals the single-workgroup argmax of hx_best_candidate over the same flow values, and
    the first maximum of the host copy."""
    full = I.make_problem(cfg)
    for n in sizes:
        prob = full if n == full.n_cand else full.subset(np.arange(n))
        say(f"hx_score_batch argmax: workload {cfg}, N={n}")
        dp = hx.DeviceProblem.upload(prob)
        ws = hx.Workspace.for_problem(dp, flows=False)
        for rep in range(3):
            ws.cost.workspace.fill_(0xA5 if rep % 2 == 0 else 0xFF)
            ws.best.fill_(-7)
            hx.score_batch(dp, ws)
            torch.cuda.synchronize()
            fv = ws.flow_value.cpu().numpy()
            got = tuple(int(x) for x in ws.best.cpu().numpy())
            first = int(np.flatnonzero(fv == fv.max())[0])
            assert got == (first, int(fv.max())), (n, rep, got)
            one = torch.full_like(ws.best, -7)
            hx.best_candidate(ws.flow_value, one, dp.n_cand)
            torch.cuda.synchronize()
            assert tuple(int(x) for x in one.cpu().numpy()) == got


@pytest.mark.parametrize("cfg", [3, 5])
def test_score_batch_argmax_ties(torch, cfg):
    """Ties for the best flow across slots and workgroups: the best candidate's placement copied
    to indices spread over the batch (both ends included) must give the lowest of those indices;
    a batch whose every flow is 0 (every group's role cleared) must give index 0."""
    full = I.make_problem(cfg, n_cand=16384)
    dp0 = hx.DeviceProblem.upload(full)
    ws0 = hx.Workspace.for_problem(dp0, flows=False)
    hx.score_batch(dp0, ws0)
    torch.cuda.synchronize()
    b, bv = (int(x) for x in ws0.best.cpu().numpy())
    N = full.n_cand
    for spots in ((N - 1, 9000, 4097, 1025), (0, N - 1), (b + 1, N - 1)):
        spots = [x for x in spots if 0 <= x < N]
        assign, role = full.assign.copy(), full.role.copy()
        for x in spots:
            assign[:, x] = full.assign[:, b]
            role[:, x] = full.role[:, b]
        prob = dataclasses.replace(full, assign=assign, role=role)
        say(f"hx_score_batch argmax ties: workload {cfg}, best {b} copied to {spots}")
        dp = hx.DeviceProblem.upload(prob)
        ws = hx.Workspace.for_problem(dp, flows=False)
        ws.cost.workspace.fill_(0xFF)
        hx.score_batch(dp, ws)
        torch.cuda.synchronize()
        got = tuple(int(x) for x in ws.best.cpu().numpy())
        assert got == (min(spots + [b]), bv), (spots, got)
    role = np.full_like(full.role, 0xFF)
    prob = dataclasses.replace(full, role=role)
    say(f"hx_score_batch argmax: workload {cfg}, every flow 0")
    dp = hx.DeviceProblem.upload(prob)
    ws = hx.Workspace.for_problem(dp, flows=False)
    ws.cost.workspace.fill_(0xA5)
    hx.score_batch(dp, ws)
    torch.cuda.synchronize()
    assert not ws.flow_value.cpu().numpy().any()
    assert tuple(int(x) for x in ws.best.cpu().numpy()) == (0, 0)


@pytest.mark.parametrize("cfg,n,variant,classes", [(3, 4096, 0, 4), (2, None, 4, 0), (3, 8192, 1, 0), (2, 1000, 2, 0),
                                                   (4, 2048, 5, 0), (4, 1000, 0, 4), (2, 777, 1, 3)])
def test_score_batch_replica_variants(torch, cfg, n, variant, classes):
    """Replica networks under the cost-model variants (request classes, the asymmetric split,
    the pipelined capacity, the stage-order search, asymmetric + pipelined; request classes on
    32 group slots, whose KV edges go through the packed list, and three classes with the
    pipelined capacity on 16 GPUs, many feasible edges per candidate): the fused call's outputs
    equal the four calls', and the oracle's flow values on a sample."""
    prob = I.make_problem(cfg, n_cand=n)
    if variant:
        prob = dataclasses.replace(prob, variant=variant)
    if classes:
        prob = dataclasses.replace(prob, classes=I.length_classes(I.WORKLOADS[cfg], classes))
    say(f"hx_score_batch vs four calls: workload {cfg}, N={prob.n_cand}, variant {variant}, classes {classes}")
    four, one = _both(torch, prob)
    _same(four, one, prob.granularity)
    idx = np.unique(np.concatenate([np.random.default_rng(cfg + variant).choice(prob.n_cand, min(prob.n_cand, 512),
                                                                              replace=False), [one["best"][0]]]))
    want = hxo.score_batch(prob.subset(idx), n_threads=N_THREADS)
    assert np.array_equal(one["flow_value"][idx], want["flow_value"])


@pytest.mark.parametrize("variant", [0, 4])
def test_score_batch_listed_kv_maximum_cluster(torch, variant):
    """255 GPUs (four mask words per group) and 32 group slots: the largest networks whose KV
    edges the fused call lists for one lane per edge, here with alpha and beta read from memory
    (too many GPUs to stage them); with the asymmetric split (variant 4) the walk's extra LDS
    sends them back to one lane per (edge, candidate).  Rows and values equal the four calls',
    and the oracle's."""
    from tests.test_gpu_parity import max_cluster_problem
    prob = max_cluster_problem(32, 96, 32)
    if variant:
        prob = dataclasses.replace(prob, variant=variant)
    say(f"hx_score_batch vs four calls: 255 GPUs, 32 slots, N={prob.n_cand}, variant {variant}")
    four, one = _both(torch, prob)
    _same(four, one, prob.granularity)
    want = hxo.score_batch(prob, n_threads=N_THREADS)
    assert np.array_equal(one["flow_value"], want["flow_value"])
    assert one["best"] == want["best"]


def _feasible_problem(gpus, groups, n, slow, seed):
    """Placements of an OPT-30B cluster of 48-80 GB GPUs, most of whose groups have a strategy, so
    that both sides have several nodes; links slow times slower (KV edges below the node capacities)."""
    rng = np.random.default_rng([2502, gpus, groups, n, seed])
    nodes = (gpus + 3) // 4
    inter = np.triu(rng.uniform(5.0, 25.0, (nodes, nodes)), 1) * 1e9
    tab = np.array([I.GPU_TYPES[c] for c in "DEF"])
    cl = I.cluster_from_nodes(np.repeat(np.arange(nodes) % 3, 4)[:gpus].astype(np.int32), tab, inter + inter.T)
    cl = dataclasses.replace(cl, beta=np.ascontiguousarray(cl.beta / slow))
    assign = rng.integers(0, groups, (gpus, n)).astype(np.uint8)
    assign[rng.random((gpus, n)) < 0.05] = I.UNUSED
    role = rng.integers(0, 2, (groups, n)).astype(np.uint8)
    role[rng.random((groups, n)) < 0.05] = I.UNUSED
    return I.Problem(cl, dict(I.OPT_30B), 700.0, 150.0, I._mask((1, 2, 3, 4, 8)), I._mask(range(1, 9)), 0, groups, assign,
                     role)


@pytest.mark.parametrize("gpus,groups,n,slow,room", [
    (8, 2, 5, 1, 0), (9, 3, 17, 200, 0), (33, 7, 1000, 200, 0), (65, 16, 16384, 300, 0), (40, 17, 16385, 300, 3),
    (64, 31, 777, 2000, 40), (129, 32, 500, 2000, 0), (24, 32, 32769, 1, 0), (64, 33, 300, 2000, 0)])
def test_score_batch_replica_networks(torch, gpus, groups, n, slow, room):
    """The fused network kernel around its branches: batch sizes on both sides of the switches of its
    candidates per workgroup, group slots from two to one past its limit, 1 to 4 mask words, arrays
    with more room than the slots need (room), and slow links, whose networks no closed form settles.
    Rows, values and best equal the four calls' and, on a sample, the oracle's."""
    prob = _feasible_problem(gpus, groups, n, slow, 1)
    say(f"hx_score_batch networks: {gpus} GPUs, {groups} slots, N={n}, links / {slow}, room {room}")
    dp = hx.DeviceProblem.upload(prob)
    mp, md, mpd = hx.flownet_dims(groups, gpus, 0)
    out = []
    for fused in (False, True):
        ws = hx.Workspace.for_problem(dp, flows=False)
        ws.net = hx.FlowNetBuffers.empty((mp + room, md + room, max(mpd, 1) + room), n, fill=-7)
        ws.cost.workspace.fill_(0xA5)
        (hx.score_batch if fused else hx.score)(dp, ws)
        torch.cuda.synchronize()
        out.append(dict(cost={k: getattr(ws.cost, k).cpu().numpy() for k in ("tp", "pp", "bmax", "cap", "lat", "members")},
                        net=ws.net.host(), flow_value=ws.flow_value.cpu().numpy(),
                        best=tuple(int(x) for x in ws.best.cpu().numpy())))
    _same(out[0], out[1], 0)
    rows = np.arange(max(mpd, 1) + room)[:, None]
    past = rows >= (out[1]["net"]["n_p"].astype(np.int64) * out[1]["net"]["n_d"])[None, :]
    assert (out[1]["net"]["kv_cap"][past] == -7).all(), "a KV row past n_p n_d was written"
    st = hx.maxflow_stats(ws.net, torch.empty_like(ws.flow_value))
    say(f"paths: {st}")
    if slow > 1 and groups > 3:  # a side of one node is a star
        assert st["min_cut"] + st["push_relabel"] > n // 20, st
    idx = np.random.default_rng(5).choice(n, min(n, 128), replace=False)
    want = hxo.score_batch(prob.subset(idx), n_threads=N_THREADS)
    assert np.array_equal(out[1]["flow_value"][idx], want["flow_value"])


@pytest.mark.parametrize("groups,n,every", [(8, 3, 1), (8, 70000, 1), (16, 65, 1), (16, 30000, 1), (32, 3, 1), (32, 20000, 1),
                                            (16, 4096, 1500), (16, 4096, 300), (8, 4096, 50), (32, 4096, 9)])
def test_score_batch_listed_networks(torch, groups, n, every):
    """The last kernel of the fused call from one listed network up: every candidate with groups of four
    GPUs, which all have a strategy, over links too slow for them (so no closed form settles it), or every
    n-th one and the others without a decode group; fewer and more listed than its workgroups take at
    once.  Flow values equal the four calls', best is the first maximum, call after call on a dirty
    workspace."""
    gpus = 4 * groups
    rng = np.random.default_rng([2502, groups, n, every])
    inter = np.triu(rng.uniform(3.0, 25.0, (groups, groups)), 1) * 1e9
    tab = np.array([I.GPU_TYPES[c] for c in "AB"])
    cl = I.cluster_from_nodes(np.repeat(np.arange(groups) % 2, 4).astype(np.int32), tab, inter + inter.T)
    cl = dataclasses.replace(cl, beta=np.ascontiguousarray(cl.beta / 1000))
    assign = np.argsort(rng.random((n, gpus)), 1).argsort(1).T // 4
    role = np.repeat((np.arange(groups) % 2)[:, None], n, 1)
    role[:, np.arange(n) % every != 0] = I.PREFILL
    prob = I.Problem(cl, dict(I.OPT_30B), 1024.0, 256.0, I._mask((1, 2, 4, 8)), I._mask(range(1, 9)), 0, groups,
                     np.ascontiguousarray(assign, np.uint8), np.ascontiguousarray(role, np.uint8))
    dp = hx.DeviceProblem.upload(prob)
    ws = hx.Workspace.for_problem(dp, flows=False)
    hx.score(dp, ws)
    st = hx.maxflow_stats(ws.net, torch.empty_like(ws.flow_value))
    want = ws.flow_value.cpu().numpy()
    say(f"hx_score_batch: {groups} slots, N={n}, every {every}: {st}")
    listed = st["min_cut"] + st["push_relabel"]
    assert listed > 0.5 * n / every and listed <= -(-n // every)
    for fill in (0xA5, 0xFF):
        ws.cost.workspace.fill_(fill)
        ws.flow_value.fill_(-7)
        hx.score_batch(dp, ws)
        torch.cuda.synchronize()
        got = ws.flow_value.cpu().numpy()
        assert np.array_equal(got, want)
        assert ws.best.tolist() == [int(np.argmax(want)), int(want.max())]


def test_score_batch_concurrent_streams(torch):
    """Independent calls in flight on three streams (each with its own workspace and outputs, the
    inputs shared): every stream's flow values and best equal a single-stream call's, call after
    call (the library keeps no state between calls)."""
    prob = I.make_problem(3)
    dp = hx.DeviceProblem.upload(prob)
    ref = hx.Workspace.for_problem(dp, flows=False)
    hx.score_batch(dp, ref)
    torch.cuda.synchronize()
    want_fv, want_best = ref.flow_value.cpu().numpy(), tuple(int(x) for x in ref.best.cpu().numpy())
    streams = [torch.cuda.Stream() for _ in range(3)]
    wss = [hx.Workspace.for_problem(dp, flows=False) for _ in range(3)]
    say("hx_score_batch on three streams at once, 12 calls")
    for s in range(12):
        hx.score_batch(dp, wss[s % 3], stream=streams[s % 3])
    torch.cuda.synchronize()
    for w in wss:
        assert np.array_equal(w.flow_value.cpu().numpy(), want_fv)
        assert tuple(int(x) for x in w.best.cpu().numpy()) == want_best
