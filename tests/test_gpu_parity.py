"""GPU parity: the HIP library (through its C ABI) against the CPU oracle on the same seeded inputs.

Sizes are chosen so the oracle finishes in seconds while every kernel still sees several tiles, ragged
tails and (where the workload drifts) real splits.  Each of the five benchmark configurations appears
with its own storage type, group size, cluster count and budget, on a few of its units.
"""
import ctypes
import json
import os
import sys
from fractions import Fraction

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import parity  # noqa: E402
from parity import DEV, Tally, check_attention, compare_build, compare_retrieval, compare_state, make_pair, run_trajectory, to_dev  # noqa: E402
from paper_2511_07427_amd import binding  # noqa: E402
from paper_2511_07427_amd.binding import LAUNCH_SEPARATE, LAUNCH_SPLIT_KERNEL, launch_shape  # noqa: E402
from paper_2511_07427_amd.workload import CONFIGS, WorkloadSpec, generate  # noqa: E402

pytestmark = pytest.mark.gpu
GOLD = os.path.join(os.path.dirname(__file__), "golden")


def say(*a):
    print(*a, flush=True)


# --------------------------------------------------------------------------- the five configurations

def test_cfg1_tiny_f32_full_trajectory():
    s = CONFIGS["tiny"]
    r = run_trajectory(s, [0], s.steps, check_every=1, full_every=16)
    say("tiny:", {k: r[k] for k in ("worst_rel", "ties", "oracle_low_margin", "splits", "clusters")})
    assert r["splits"] > 0


def test_cfg1_tiny_with_variance_trigger_and_small_buffer():
    s = CONFIGS["tiny"].scaled(var_alpha=1.2, buffer_max=4)
    r = run_trajectory(s, [0], s.steps, budget=128, check_every=1, full_every=16)
    say("tiny/var:", {k: r[k] for k in ("worst_rel", "ties", "splits", "forced", "clusters")})
    assert r["splits"] > 0 and r["forced"] > 0


def test_cfg2_llama_shaped_f16():
    s = CONFIGS["llama3_8b"]
    r = run_trajectory(s, [0, 17, 255], 384, check_every=4, full_every=64)
    say("llama:", {k: r[k] for k in ("worst_rel", "ties", "splits", "forced", "clusters")})


def test_cfg3_qwen_shaped_bf16_group_of_7():
    s = CONFIGS["qwen25_7b"]
    r = run_trajectory(s, [0, 111], 768, check_every=8, full_every=128)
    say("qwen:", {k: r[k] for k in ("worst_rel", "ties", "splits", "forced", "clusters")})
    assert r["splits"] > 0


def test_cfg4_batched_shaped_f16():
    s = CONFIGS["batched16"]
    r = run_trajectory(s, [3, 64], 128, check_every=4, full_every=64)
    say("batched:", {k: r[k] for k in ("worst_rel", "ties", "splits", "forced", "clusters")})


def test_cfg5_long_shaped_bf16_group_of_8():
    s = CONFIGS["long131k"].scaled(kmeans_iters=3)
    r = run_trajectory(s, [5], 192, check_every=8, full_every=96)
    say("long:", {k: r[k] for k in ("worst_rel", "ties", "splits", "forced", "clusters")})


# --------------------------------------------------------------------------- launch shapes of the retrieval

@pytest.mark.parametrize("name,units,steps,launch", [
    ("llama3_8b", [1, 2], 96, launch_shape(1)),                          # one kernel per retrieval, G = 4
    ("qwen25_7b", [3], 160, launch_shape(1)),                            # one kernel per retrieval, G = 7
    ("llama3_8b", [4], 64, launch_shape(1, 0, LAUNCH_SEPARATE)),         # separate kernels, no split-KV
    ("long131k", [2], 48, launch_shape(3, 8)),                           # split-KV with prefetching wavefronts
    ("llama3_8b", [5, 6], 64, launch_shape(5, 16, LAUNCH_SEPARATE)),     # split-KV, 16 wavefronts, odd split count
])
def test_every_launch_shape_of_retrieve_attend(name, units, steps, launch):
    s = CONFIGS[name]
    if name == "long131k":
        s = s.scaled(kmeans_iters=2)
    if name == "llama3_8b":
        s = s.scaled(max_cluster_factor=8)
    r = run_trajectory(s, units, steps, check_every=1, full_every=32, step_call="mixed", launch=launch)
    say(name, hex(launch), {k: r[k] for k in ("worst_rel", "ties", "splits", "clusters")})


@pytest.mark.parametrize("name,units,steps,launch", [
    ("llama3_8b", [7, 8, 9], 160, launch_shape(1)),                        # the whole step in one kernel, G = 4
    ("qwen25_7b", [5, 6], 256, launch_shape(1)),                           # the same with G = 7
    ("llama3_8b", [7, 8, 9], 160, launch_shape(1, 0, LAUNCH_SPLIT_KERNEL)),   # retrieval + append in one kernel, splits in their own
    ("batched16", [9], 64, launch_shape(0, 0, LAUNCH_SEPARATE)),           # separate kernels behind the same call
])
def test_whole_step_call_matches_the_three_calls(name, units, steps, launch):
    s = CONFIGS[name]
    r = run_trajectory(s, units, steps, check_every=1, full_every=32, step_call="one", launch=launch)
    say(name, hex(launch), {k: r[k] for k in ("worst_rel", "ties", "splits", "forced", "clusters")})
    assert r["splits"] > 0 or name == "batched16"


@pytest.mark.parametrize("launch", [launch_shape(1), 0])
def test_long_run_through_the_whole_step_call_with_several_splits_per_step(launch):
    # the steady state of the benchmark configuration in its launch shape (one workgroup per unit, the whole
    # step in one kernel) and in the one that the library takes for so few units (two workgroups per unit): small
    # clusters, several due splits of one unit in one step (decided by separate wavefronts while the pages are
    # streamed)
    s = CONFIGS["llama3_8b"]
    r = run_trajectory(s, [16, 17, 18, 19, 20, 21, 22, 23], 2560, check_every=32, full_every=640, step_call="one",
                       launch=launch)
    say("long:", launch, {k: r[k] for k in ("worst_rel", "ties", "splits", "forced", "clusters", "most_splits_in_a_step")})
    assert r["splits"] > 2000 and r["most_splits_in_a_step"] >= 3


@pytest.mark.parametrize("launch", [launch_shape(1), 0])
def test_long_run_through_the_whole_step_call_group_of_7(launch):
    # the same for the kernel variant that holds up to 8 query heads per KV head (bf16, G = 7; four workgroups per unit)
    s = CONFIGS["qwen25_7b"]
    r = run_trajectory(s, [30, 31, 32, 33], 2048, check_every=32, full_every=512, step_call="one", launch=launch)
    say("long, G = 7:", launch, {k: r[k] for k in ("worst_rel", "ties", "splits", "forced", "clusters", "most_splits_in_a_step")})
    assert r["splits"] > 500 and r["most_splits_in_a_step"] >= 2


@pytest.mark.parametrize("dtype,step_call", [("f16", "one"), ("bf16", "one"), ("f32", "three"), ("f16", "three")])
def test_splits_of_large_clusters(dtype, step_call):
    # prefill clusters of several dozen to a few hundred entries that the drift splits early: up to 64 entries of a
    # 16-bit type (32 of float32) one wavefront each, four side by side; up to 128 (64) one wavefront each, two
    # side by side; larger ones by the whole workgroup.  The sizes of the clusters that were split are taken from
    # the oracle's records before and after every step.
    s = CONFIGS["llama3_8b"].scaled(dtype=dtype, prefill=1536, n_clusters_init=20, var_alpha=1.02, max_cluster_factor=16,
                                    kmeans_iters=4, budget=512)
    units, steps = [0, 1, 2, 3], 192
    w = generate(s, units=units, steps=steps)
    ix, o = make_pair(s, len(units), max_tokens=s.prefill + steps)
    ix.dynakv_build_index(to_dev(w["K0"], s.dtype), to_dev(w["V0"], s.dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    o.build_index(w["K0"], w["V0"], w["init_idx"])
    st = parity.Stepper(ix, o, s, w, None, None)
    compare_build(ix, o, st.tally, s.prefill)
    parents = []
    for t in range(steps):
        before = [o.clusters(k) for k in range(len(units))]
        st.step(t, step_call == "one", attention=t % 4 == 0, full=t % 32 == 0 or t == steps - 1)
        for k in range(len(units)):
            after = o.clusters(k)
            if len(after["n"]) > len(before[k]["n"]):
                m0 = before[k]["n"] + before[k]["b"]
                m1 = (after["n"] + after["b"])[:len(m0)]
                parents += [int(x) for x in m0[m1 < m0]]
    r = st.report()
    small = 32 if dtype == "f32" else 64
    hist = dict(one_per_lane=sum(p <= small for p in parents), two_per_lane=sum(small < p <= 2 * small for p in parents),
                workgroup=sum(p > 2 * small for p in parents))
    say("large clusters,", dtype, step_call, hist, {k: r[k] for k in ("worst_rel", "ties", "splits", "forced", "clusters")})
    assert hist["two_per_lane"] >= 3 and hist["workgroup"] >= 1 and (hist["one_per_lane"] >= 3 or dtype == "f32")


@pytest.mark.parametrize("dtype,step_call", [("f16", "one"), ("bf16", "one"), ("f16", "three"), ("f32", "three")])
def test_splits_of_degenerate_large_clusters(dtype, step_call):
    # one large cluster per unit that the size trigger flags at the first append and that is split at once
    # (B_max = 0): 100 equal keys (no second seed: unflagged with exact statistics), 99 equal keys and one apart
    # (split 99 / 1, the second seed is the lowest of 99 equally far members), two values of 60 keys each, and 129
    # equal keys (workgroup path)
    N0, d = 160, 128
    s = WorkloadSpec("degenerate", dtype, 4, 2, N0, 2, 2, 64, 6, 0.05, var_alpha=0.0, size_factor=1.0, buffer_max=0,
                     kmeans_iters=2, max_cluster_factor=8, seed=77)
    w = generate(s, steps=2)
    a = np.full(d, 5.0, np.float32)
    apart = a.copy(); apart[0] = 8.0
    b = a.copy(); b[:4] += 0.5
    K0 = w["K0"].copy()
    sizes = (100, 100, 120, 129)
    K0[0, :100] = a
    K0[1, :100] = a; K0[1, 57] = apart
    K0[2, :120:2] = a; K0[2, 1:120:2] = b
    K0[3, :129] = a
    init = np.array([[0, n] for n in sizes], np.int32)
    w = dict(w, K0=K0, init_idx=init)
    w["Knew"] = w["Knew"].copy(); w["Knew"][0, :] = a
    ix, o = make_pair(s, 4, max_tokens=N0 + 2)
    ix.dynakv_build_index(to_dev(K0, dtype), to_dev(w["V0"], dtype), torch.from_numpy(init).to(DEV))
    o.build_index(K0, w["V0"], init)
    st = parity.Stepper(ix, o, s, w, None, None)
    compare_build(ix, o, st.tally, N0)
    assert [int(o.clusters(k)["n"][0]) for k in range(4)] == list(sizes)
    for t in range(2):
        st.step(t, step_call == "one", attention=True, full=True)
    r = st.report()
    say("degenerate clusters,", dtype, step_call, {k: r[k] for k in ("worst_rel", "ties", "splits", "failed", "clusters")})
    assert r["failed"] == 2 and r["splits"] >= 2
    c1, c2 = o.clusters(1), o.clusters(2)
    assert {1, 100} <= set(c1["n"].tolist()) and {60, 61} <= set(c2["n"].tolist())


@pytest.mark.parametrize("name,sample,steps,iters", [
    ("llama3_8b", [0, 131, 255], 1280, None),     # what the benchmark times
    ("llama3_8b", [0, 100, 255], 8256, None),     # ... over its whole horizon (warm-up and timed steps)
    ("batched16", [0, 77, 127], 96, None),
    ("qwen25_7b", [0, 58, 111], 512, None),
    ("long131k", [6], 96, 3),                     # separate kernels, 4 workgroups per unit in gather + attention
])
def test_full_size_configurations_on_sampled_units(name, sample, steps, iters):
    # all units of the configuration, default launch shape, one whole-step call per step; the oracle follows
    # a few of the units (k-means shortened where the oracle's prefill would take minutes)
    s = CONFIGS[name] if iters is None else CONFIGS[name].scaled(kmeans_iters=iters)
    r = parity.run_full_size(s, sample, steps, check_every=32 if steps < 4096 else 64, full_every=256 if steps < 4096 else 512)
    say("full size, %s:" % name, r)
    assert r["splits"] > 0 or name in ("batched16", "long131k")


# --------------------------------------------------------------------------- late windows of the full horizons

@pytest.mark.parametrize("name,sample,start,steps", [
    ("batched16", [0, 77, 127], 24576 - 64, 64),     # the end of the window the configuration times (128 units, ~7200 clusters each)
    ("qwen25_7b", [0, 58, 111], 30000 - 64, 64),     # 112 units, ~12000 clusters each
    ("long131k", [0, 5], 114688 - 48, 48),           # 8 units, 131 072 entries each
])
def test_late_window_of_the_full_horizon(name, sample, start, steps):
    """All units of the configuration run alone from prefill to `start` (whole-step calls, the launch shape the
    benchmark times, cluster capacity for the full horizon); the state is then exported, the oracle imports the
    sampled units, and the last steps of the horizon run side by side under the parity protocol."""
    from paper_2511_07427_amd.workload import FULL_HORIZON_FACTOR
    s = CONFIGS[name].scaled(max_cluster_factor=FULL_HORIZON_FACTOR[name])
    r = parity.run_window(s, sample, start, steps, check_every=8)
    say("late window, %s:" % name, r)
    assert r["splits"] > 0 and min(r["clusters"]) > 4 * s.n_clusters_init


# --------------------------------------------------------------------------- hand-worked fixtures, padded to d = 128

def _pad(a):
    a = np.asarray(a, np.float32)
    out = np.zeros(a.shape[:-1] + (128,), np.float32)
    out[..., :a.shape[-1]] = a
    return out


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_hand_examples_on_the_gpu(dtype):
    g1 = json.load(open(os.path.join(GOLD, "hand_example_1_retrieve.json")))
    g3 = json.load(open(os.path.join(GOLD, "hand_example_3_split.json")))
    tdt = binding.TORCH_DTYPES[dtype]
    scale = float(1 / np.sqrt(2))
    # example 1: build, score, select, attend
    cfg = binding.Config(1, 1, dtype, 2, 8, 64, kmeans_iters=3, softmax_scale=scale)
    ix = binding.Index(cfg, DEV)
    K = torch.from_numpy(_pad(g1["keys"]))[None].to(DEV).to(tdt)
    V = torch.from_numpy(_pad(g1["values"]))[None].to(DEV).to(tdt)
    ix.dynakv_build_index(K, V, torch.tensor([g1["init_idx"]], dtype=torch.int32, device=DEV))
    st = ix.dynakv_export_state()
    assert st["size"][0, :2].tolist() == g1["clusters"]["n"]
    np.testing.assert_allclose(st["centroids"][0, :2, :2].numpy(), np.array(g1["clusters"]["centroids"], np.float32), rtol=1e-6)
    np.testing.assert_allclose(st["m2"][0, :2].numpy(), g1["clusters"]["M2"], rtol=1e-6)
    assert st["members"][0, :6].tolist() == sum(g1["clusters"]["members"], [])
    q = torch.from_numpy(_pad([[g1["query"]]])).to(DEV).to(tdt)
    out = torch.empty(1, 1, 128, device=DEV)
    lse = torch.empty(1, 1, device=DEV)
    ix.dynakv_retrieve_attend(q, 2, out, lse)
    st = ix.dynakv_export_state(binding._STATE_FIELDS)
    assert st["selected"][0, :st["n_selected"][0]].tolist() == g1["budget_2"]["selected"]
    assert st["gathered"][0, :st["n_gathered"][0]].tolist() == g1["budget_2"]["gather"]
    np.testing.assert_allclose(st["scores"][0, :2].numpy(), g1["scores"], rtol=1e-6)
    np.testing.assert_array_equal(st["keys"][0, :6].float().numpy(), _pad(g1["keys"]))
    np.testing.assert_array_equal(st["values"][0, :6].float().numpy(), _pad(g1["values"]))
    np.testing.assert_allclose(out[0, 0, :2].cpu().numpy(), g1["budget_2"]["out"], atol=2e-3 * 0.80443)
    ix.dynakv_retrieve_attend(q, 6, out, lse)
    st = ix.dynakv_export_state()
    # the same entries as the worked example; the library attends the clusters in its own order (ascending id)
    got = st["gathered"][0, :st["n_gathered"][0]].tolist()
    assert sorted(got) == sorted(g1["budget_6"]["gather"])
    order = st["selected"][0, :st["n_selected"][0]].tolist()
    assert sorted(order) == sorted(g1["budget_6"]["selected"]) if "selected" in g1["budget_6"] else len(order) == 2
    assert got == sum((g1["clusters"]["members"][j] for j in order), [])
    # example 3: append, flag, split
    cfg = binding.Config(1, 1, dtype, 2, 8, 64, kmeans_iters=3, var_alpha=1.5, buffer_max=16, softmax_scale=scale)
    ix = binding.Index(cfg, DEV)
    K = torch.from_numpy(_pad(g3["keys"]))[None].to(DEV).to(tdt)
    ix.dynakv_build_index(K, K, torch.tensor([g3["init_idx"]], dtype=torch.int32, device=DEV))
    ix.dynakv_retrieve_attend(q, 4, out, lse)
    k = torch.from_numpy(_pad([g3["new_key"]])).to(DEV).to(tdt)
    ix.dynakv_append(k, k)
    st = ix.dynakv_export_state()
    assert (st["flag"][0, 0], st["buffered"][0, 0], st["size"][0, 0], st["last_assign"][0]) == (1, 1, 4, 0)
    ix.dynakv_split()
    st = ix.dynakv_export_state()
    assert st["n_clusters"][0] == 3 and st["counters"][0, 0] == 1
    for ch in (g3["split"]["stay"], g3["split"]["moved"]):
        j = ch["id"]
        lo, hi = st["offsets"][0, j], st["offsets"][0, j + 1]
        assert st["members"][0, lo:hi].tolist() == ch["members"]
        np.testing.assert_allclose(st["centroids"][0, j, :2].numpy(), np.array(ch["centroid"], np.float32), rtol=1e-6)
        assert st["m2"][0, j] == pytest.approx(ch["M2"], abs=1e-9) and st["size"][0, j] == ch["n"]


# --------------------------------------------------------------------------- budgets, dense limit, degenerate shapes

def _dense(Q, K, V, scale):
    q, k, v = (torch.from_numpy(np.asarray(a, np.float64)) for a in (Q, K, V))
    lg = scale * torch.einsum("ugd,utd->ugt", q, k)
    return torch.einsum("ugt,utd->ugd", torch.softmax(lg, -1), v).numpy(), torch.logsumexp(lg, -1).numpy()


def _build_pair(s, w, n_units, K0=None, init=None, **over):
    ix, o = make_pair(s, n_units, **over)
    K0 = w["K0"] if K0 is None else K0
    init = w["init_idx"] if init is None else init
    ix.dynakv_build_index(to_dev(K0, s.dtype), to_dev(w["V0"], s.dtype), torch.from_numpy(init).to(DEV))
    o.build_index(K0, w["V0"], init)
    t = Tally()
    compare_build(ix, o, t, K0.shape[1])
    return ix, o, t


@pytest.mark.parametrize("dtype,G,N0,M0", [("f16", 4, 1000, 37), ("bf16", 16, 300, 300), ("f32", 1, 530, 1), ("f16", 5, 16, 16)])
def test_budget_edges_and_dense_limit(dtype, G, N0, M0):
    s = WorkloadSpec("edge", dtype, 2, G, N0, 40, M0, 10 ** 6, 8, 0.05, var_alpha=1.3, size_factor=2.0, seed=77)
    w = generate(s)
    ix, o, tally = _build_pair(s, w, 2, kmeans_iters=4)
    out = torch.empty(2, G, 128, device=DEV)
    lse = torch.empty(2, G, device=DEV)
    Qd, Kd, Vd = to_dev(w["Q"], dtype), to_dev(w["Knew"], dtype), to_dev(w["Vnew"], dtype)
    biggest = int(o.clusters(0)["n"].max())
    budgets = [0, 1, max(1, biggest - 1), biggest, N0 // 3, N0 - 1, N0 + 100, 10 ** 6]
    for t in range(s.steps):
        B = budgets[t % len(budgets)]
        ix.dynakv_retrieve_attend(Qd[t], B, out, lse)
        oo, ol = o.retrieve_attend(w["Q"][t], B)
        dirty = compare_retrieval(ix, o, tally, "edge step %d budget %d" % (t, B), Q=w["Q"][t], budget=B)
        keep = [u for u in range(2) if u not in dirty]
        check_attention(out.cpu().numpy()[keep], lse.cpu().numpy()[keep], oo[keep], ol[keep], "edge step %d budget %d" % (t, B))
        if B >= N0 + t:   # everything retrieved: dense attention over the whole cache
            allK = np.concatenate([w["K0"], w["Knew"][:t].transpose(1, 0, 2)], 1)
            allV = np.concatenate([w["V0"], w["Vnew"][:t].transpose(1, 0, 2)], 1)
            ref, rl = _dense(w["Q"][t], allK, allV, 1 / np.sqrt(128))
            check_attention(out.cpu().numpy(), lse.cpu().numpy(), ref, rl, "dense step %d" % t)
            assert not dirty
        ix.dynakv_append(Kd[t], Vd[t]); o.append(w["Knew"][t], w["Vnew"][t])
        ix.dynakv_split(); o.split()
        dirty |= compare_state(ix, o, tally, "edge step %d" % t, full=True, skip=dirty)
        parity.resync(ix, o, None, dirty, tally)
    say("edges", dtype, G, N0, M0, dict(tally))


@pytest.mark.parametrize("launch", [0, launch_shape(0, 0, LAUNCH_SEPARATE)])
def test_selection_with_equal_scores_and_large_active_sets(launch):
    """The selection's special paths: every score equal (a zero query: ids decide, and the cut falls inside the
    group of equal scores), and active sets of more than a thousand clusters."""
    s = WorkloadSpec("sel", "f16", 2, 4, 4096, 4, 1400, 10 ** 6, 8, 0.05, var_alpha=0.0, size_factor=0.0, seed=31)
    w = generate(s)
    ix, o, tally = _build_pair(s, w, 2, kmeans_iters=2, launch=launch)
    out = torch.empty(2, 4, 128, device=DEV)
    lse = torch.empty(2, 4, device=DEV)
    zero = np.zeros_like(w["Q"][0])
    cases = [("all equal", zero, B) for B in (0, 1, 7, 100, 2500, 4095, 4096, 10 ** 6)]
    cases += [("large set", w["Q"][1], B) for B in (3000, 3500, 4096, 10 ** 6)]
    cases += [("mid set", w["Q"][2], B) for B in (1, 64, 1024, 2048)]
    for what, Q, B in cases:
        ix.dynakv_retrieve_attend(to_dev(Q, "f16"), B, out, lse)
        oo, ol = o.retrieve_attend(Q, B)
        dirty = compare_retrieval(ix, o, tally, "%s budget %d" % (what, B), Q=Q, budget=B)
        assert not dirty or what != "all equal"      # exact ties go by id on both sides: never a disagreement
        keep = [u for u in range(2) if u not in dirty]
        check_attention(out.cpu().numpy()[keep], lse.cpu().numpy()[keep], oo[keep], ol[keep], "%s budget %d" % (what, B))
    st = ix.dynakv_export_state(["n_selected"])
    say("selection paths", hex(launch), "last active set:", st["n_selected"].tolist(), dict(tally))


@pytest.mark.parametrize("dtype,M0,kw", [("f16", 7100, {}), ("bf16", 7400, {}), ("f16", 900, dict(search_copy=1)), ("f32", 1025, {})])
def test_selection_from_contenders(dtype, M0, kw):
    """Capacity for more clusters than the selection keeps in LDS: it runs on the clusters that the coarse histogram lets
    through.  Equal scores within (7100) and beyond (7400) what that list holds, a first cluster over budget, cuts
    anywhere, and everything selected."""
    s = WorkloadSpec("contenders", dtype, 2, 4, M0 + 300, 4, M0, 10 ** 6, 8, 0.05, var_alpha=0.0, size_factor=0.0, seed=41)
    w = generate(s)
    ix, o, tally = _build_pair(s, w, 2, kmeans_iters=1, max_clusters=16400, **kw)
    out = torch.empty(2, 4, 128, device=DEV)
    lse = torch.empty(2, 4, device=DEV)
    zero = np.zeros_like(w["Q"][0])
    cases = [("all equal", zero, B) for B in (0, 1, 7, 2500)] + [("cut", w["Q"][1 + B % 3], B) for B in (1, 2, 65, 1000, 3900)]
    if M0 + 300 < 4096:
        cases.append(("all", w["Q"][1], 10 ** 6))       # (a selection of more than 4096 clusters sets the error word)
    for what, Q, B in cases:
        ix.dynakv_retrieve_attend(to_dev(Q, dtype), B, out, lse)
        oo, ol = o.retrieve_attend(Q, B)
        dirty = compare_retrieval(ix, o, tally, "%s budget %d" % (what, B), Q=Q, budget=B)
        assert not dirty or what == "cut"               # exact ties go by id on both sides: never a disagreement
        keep = [u for u in range(2) if u not in dirty]
        check_attention(out.cpu().numpy()[keep], lse.cpu().numpy()[keep], oo[keep], ol[keep], "%s budget %d" % (what, B))
    assert ix.dynakv_export_state(["error"])["error"].tolist() == [0, 0]
    say("selection from contenders", dtype, M0, dict(tally))


def test_group_sum_custom_scale_all_resident_and_huge_logits():
    s = WorkloadSpec("opts", "f16", 3, 3, 700, 64, 24, 200, 6, 0.1, var_alpha=1.2, size_factor=0.0, buffer_max=0, seed=99)
    r = run_trajectory(s, range(3), 64, group_reduce=1, softmax_scale=0.05, kmeans_iters=5, full_every=8)
    say("opts:", {k: r[k] for k in ("worst_rel", "ties", "splits", "clusters")})
    assert r["splits"] > 0
    ix, o, w = r["index"], r["oracle"], r["workload"]
    Q = w["Q"][0] * 200.0                      # logits far beyond exp's range without max subtraction
    out = torch.empty(3, 3, 128, device=DEV)
    lse = torch.empty(3, 3, device=DEV)
    ix.dynakv_retrieve_attend(to_dev(Q, "f16"), 300, out, lse)
    from paper_2511_07427_amd.workload import round_to_dtype
    Qr = round_to_dtype(Q, "f16")
    oo, ol = o.retrieve_attend(Qr, 300)
    dirty = compare_retrieval(ix, o, Tally(), "huge logits", Q=Qr, budget=300)
    keep = [u for u in range(3) if u not in dirty]
    assert torch.isfinite(out).all() and torch.isfinite(lse).all()
    den = np.maximum(np.abs(oo).max(-1), 1e-6)
    assert (np.abs(out.cpu().numpy() - oo).max(-1) / den)[keep].max() <= 2e-3
    assert np.abs(lse.cpu().numpy() - ol)[keep].max() <= 2e-3 * np.abs(ol).max()


@pytest.mark.parametrize("dtype,kw", [("bf16", dict(search_copy=1)), ("f16", dict(search_copy=1, score_round=1)),
                                      ("bf16", dict(score_round=1)), ("f16", dict(update_mode=1))])
def test_readings_behind_config_fields(dtype, kw):
    """Both settings of the two readings that are configuration fields on both sides (which copy of the centroids the
    searches read, whether scores are rounded to float32 before they are compared), and the static-update mode."""
    s = CONFIGS["llama3_8b"].scaled(dtype=dtype, prefill=1536, n_clusters_init=96, budget=384, var_alpha=1.3)
    r = run_trajectory(s, [0, 1, 2], 160, check_every=2, full_every=40, step_call="mixed", kmeans_iters=4, **kw)
    say("readings", dtype, kw, {k: r[k] for k in ("worst_rel", "ties", "splits", "clusters")})
    if kw.get("update_mode"):
        assert r["splits"] == 0 and r["clusters"] == [96, 96, 96]
    else:
        assert r["splits"] > 0


@pytest.mark.parametrize("dtype,N0,M0", [("f16", 8292, 8192), ("bf16", 700, 640), ("f32", 700, 700)])
def test_token_level_mode(dtype, N0, M0):
    """The baseline without clustering: every entry its own cluster (retrieval = exact top-B over tokens), appended
    entries become new clusters; more clusters than the selection keeps in LDS, and the capacity error at the end."""
    s = CONFIGS["llama3_8b"].scaled(dtype=dtype, prefill=N0, n_clusters_init=M0, budget=300, max_cluster_factor=1)
    r = run_trajectory(s, [0, 1], 40, check_every=1, full_every=10, step_call="mixed", update_mode=2, kmeans_iters=1,
                       max_clusters=M0 + 36)
    say("token level", dtype, {k: r[k] for k in ("worst_rel", "ties", "splits", "clusters")})
    ix, o = r["index"], r["oracle"]
    st = ix.dynakv_export_state(["error", "n_clusters", "n_tokens", "size"])
    assert r["splits"] == 0 and st["n_clusters"].tolist() == [M0 + 36] * 2 and st["n_tokens"].tolist() == [N0 + 36] * 2
    assert st["error"].tolist() == [binding.ERR_CLUSTERS] * 2 and o.error(0) == 2
    assert int(st["size"][:, M0:M0 + 36].min()) == 1


@pytest.mark.parametrize("dtype,kw", [("f16", {}), ("bf16", {}), ("f32", {}), ("f16", dict(search_copy=1))])
def test_chunked_prefill_extension(dtype, kw):
    """dynakv_extend_index: k-means on the first chunk, the second chunk (drifted keys) added entry by entry with every
    cluster resident; compared with the oracle's extension, then decode steps go on from the extended index."""
    s = CONFIGS["llama3_8b"].scaled(dtype=dtype, prefill=1024, n_clusters_init=48, budget=300, var_alpha=1.25, drift_std=0.1)
    U, n2, steps = 3, 384, 24
    w = generate(s, units=range(U), steps=n2 + steps)
    ix, o = make_pair(s, U, max_tokens=1024 + n2 + steps, kmeans_iters=4, **kw)
    ix.dynakv_build_index(to_dev(w["K0"], dtype), to_dev(w["V0"], dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    o.build_index(w["K0"], w["V0"], w["init_idx"])
    tally = Tally()
    compare_build(ix, o, tally, 1024)
    K1, V1 = np.ascontiguousarray(w["Knew"][:n2].transpose(1, 0, 2)), np.ascontiguousarray(w["Vnew"][:n2].transpose(1, 0, 2))
    ix.dynakv_extend_index(to_dev(K1, dtype), to_dev(V1, dtype))
    o.extend(K1, V1)
    # the extension takes hundreds of decisions between two comparisons: a tie in any of them shows as a different
    # partition with no single margin to blame, so the comparison is strict (none occurred on these inputs)
    st = ix.dynakv_export_state(["n_clusters", "n_tokens", "flag", "members", "offsets", "error"])
    for u in range(U):
        M = o.num_clusters(u)
        off, mem = o.members(u)
        assert st["n_clusters"][u] == M > 48 and st["n_tokens"][u] == 1024 + n2 and st["error"][u] == 0
        assert int(st["flag"][u].sum()) == 0
        np.testing.assert_array_equal(st["offsets"][u, :M + 1].numpy(), off)
        np.testing.assert_array_equal(st["members"][u, :1024 + n2].numpy(), mem)
    assert not compare_state(ix, o, tally, "after the extension", assign=False)
    w2 = {k: (v[n2:] if k in ("Q", "Knew", "Vnew") else v) for k, v in w.items()}
    sp = parity.Stepper(ix, o, s, w2, None, 300)
    sp.tally = tally
    for t in range(steps):
        sp.step(t, t % 2 == 1, attention=True, full=(t % 8 == 0 or t == steps - 1))
    say("chunked prefill", dtype, kw, sp.report())


@pytest.mark.parametrize("dtype,launch", [("f16", 0), ("bf16", launch_shape(2, 0, LAUNCH_SEPARATE)), ("f32", 0)])
def test_coretrieval_placement(dtype, launch):
    """dynakv_place_by_coretrieval (Section 5.1, Eq. 8): co-retrieval probabilities and placement chain against the
    oracle's; the page pool then follows the chain, everything else (partition, statistics, retrieval results) is
    as before, and decode steps go on under the parity protocol."""
    s = CONFIGS["llama3_8b"].scaled(dtype=dtype, prefill=1536, n_clusters_init=64, budget=400, var_alpha=1.3)
    U, R, steps = 3, 24, 32
    w = generate(s, units=range(U), steps=R + steps)
    ix, o = make_pair(s, U, max_tokens=1536 + steps, kmeans_iters=4, launch=launch)
    K0, V0 = to_dev(w["K0"], dtype), to_dev(w["V0"], dtype)
    ix.dynakv_build_index(K0, V0, torch.from_numpy(w["init_idx"]).to(DEV))
    o.build_index(w["K0"], w["V0"], w["init_idx"])
    tally = Tally()
    compare_build(ix, o, tally, 1536)
    out0, lse0 = torch.empty(U, s.group_size, 128, device=DEV), torch.empty(U, s.group_size, device=DEV)
    q_probe = to_dev(w["Q"][R], dtype)
    ix.dynakv_retrieve_attend(q_probe, 400, out0, lse0)
    before = ix.dynakv_export_state(["offsets", "members", "centroids", "m2", "size", "gathered", "n_gathered", "first_page"])
    P, order = ix.dynakv_place_by_coretrieval(K0, V0, to_dev(w["Q"][:R], dtype), 400)
    Po, oo = o.coretrieval(w["Q"][:R], 400)
    np.testing.assert_allclose(P.cpu().numpy(), Po, rtol=1e-6, atol=1e-9)
    np.testing.assert_array_equal(order.cpu().numpy(), oo)
    assert float(P.sum()) == pytest.approx(U, rel=1e-4) and int((P > 0).sum()) > 0
    out1, lse1 = torch.empty_like(out0), torch.empty_like(lse0)
    ix.dynakv_retrieve_attend(q_probe, 400, out1, lse1)
    after = ix.dynakv_export_state(["offsets", "members", "centroids", "m2", "size", "gathered", "n_gathered", "first_page", "error"])
    assert not after["error"].any()
    for k in ("offsets", "members", "centroids", "m2", "size", "gathered", "n_gathered"):
        assert torch.equal(before[k], after[k]), k
    assert torch.allclose(out0, out1, rtol=1e-6, atol=1e-7) and torch.allclose(lse0, lse1, atol=1e-6)
    fp, sz, ch = after["first_page"].numpy(), after["size"].numpy(), order.cpu().numpy()
    assert not np.array_equal(before["first_page"].numpy(), fp)
    for u in range(U):                                  # the pool follows the chain: each cluster right after its predecessor
        nxt = 0
        for j in ch[u]:
            if sz[u, j] > 0:
                assert fp[u, j] == nxt
                nxt += (sz[u, j] + 15) // 16
    o.retrieve_attend(w["Q"][R], 400)                   # the oracle's active set as the library's
    w2 = {k: (v[R:] if k in ("Q", "Knew", "Vnew") else v) for k, v in w.items()}
    sp = parity.Stepper(ix, o, s, w2, None, 400)
    sp.tally = tally
    for t in range(steps):
        sp.step(t, t % 2 == 0, attention=True, full=(t % 8 == 0 or t == steps - 1))
    say("co-retrieval placement", dtype, hex(launch), sp.report())
    # an index that has moved on since it was built is refused
    ix.dynakv_place_by_coretrieval(K0, V0, to_dev(w["Q"][:2], dtype), 400)
    st = ix.dynakv_export_state(["error"])
    assert st["error"].tolist() == [binding.ERR_PLACE] * U


@pytest.mark.parametrize("dtype,built_before", [("f16", False), ("bf16", True), ("f32", False)])
def test_coretrieval_placement_after_an_import(dtype, built_before):
    """A snapshot taken right after the build counts as a built index: placing the importing index (new, or built
    earlier on another prompt of the same size) gives what placing the exporting one gives.  A unit whose snapshot names
    a position beyond the keys at hand is refused."""
    N0, M0, Mcap, U = 1100, 70, 300, 3
    s = WorkloadSpec("place", dtype, U, 4, N0, 8, M0, 300, 6, 0.05, var_alpha=1.5, size_factor=0.0, seed=17)
    w, other = generate(s), generate(s.scaled(seed=18))
    a, _ = make_pair(s, U, max_tokens=N0 + 40, max_clusters=Mcap, kmeans_iters=3)
    b, _ = make_pair(s, U, max_tokens=N0 + 40, max_clusters=Mcap, kmeans_iters=3)
    K, V = to_dev(w["K0"], dtype), to_dev(w["V0"], dtype)
    a.dynakv_build_index(K, V, torch.from_numpy(w["init_idx"]).to(DEV))
    snap = a.dynakv_export_state(binding.IMPORT_FIELDS, to_cpu=False)
    if built_before:
        b.dynakv_build_index(to_dev(other["K0"], dtype), to_dev(other["V0"], dtype), torch.from_numpy(other["init_idx"]).to(DEV))
    b.dynakv_import_state(snap)
    Qref = to_dev(w["Q"], dtype)
    got = []
    for ix in (a, b):
        P, order = ix.dynakv_place_by_coretrieval(K, V, Qref, 300)
        out, lse = torch.empty(U, 4, 128, device=DEV), torch.empty(U, 4, device=DEV)
        ix.dynakv_retrieve_attend(Qref[0], 300, out, lse)
        st = ix.dynakv_export_state(("error", "size", "offsets", "members", "keys", "values", "first_page", "n_gathered", "gathered"))
        got.append((P.cpu(), order.cpu(), out.cpu(), lse.cpu(), st))
    (Pa, oa, xa, la, sa), (Pb, ob, xb, lb, sb) = got
    assert torch.equal(Pa, Pb) and torch.equal(oa, ob)
    for k in sa:
        assert torch.equal(sa[k], sb[k]), k
    assert not sa["error"].any() and torch.equal(sa["keys"][:, :N0], K.cpu()) and torch.equal(sa["values"][:, :N0], V.cpu())
    # the same entries in the same order; only which wavefront takes a tile differs: float32 sums of up to 300 terms
    assert torch.allclose(xa, xb, rtol=3e-5, atol=3e-6) and torch.allclose(la, lb, rtol=3e-5)
    snap["members"][1, 5] = N0 + 7
    b.dynakv_import_state(snap)
    before = b.dynakv_export_state(("members", "first_page"))
    b.dynakv_place_by_coretrieval(K, V, Qref, 300)
    after = b.dynakv_export_state(("members", "first_page", "error"))
    assert after["error"].tolist() == [0, binding.ERR_PLACE, 0]
    assert torch.equal(before["members"], after["members"]) and torch.equal(before["first_page"][1], after["first_page"][1])
    assert torch.equal(after["first_page"][0], sa["first_page"][0])


@pytest.mark.parametrize("dtype,W,k", [("f16", 32, 4), ("bf16", 128, 32), ("f32", 20, 3)])
def test_local_update_mode(dtype, W, k):
    """The local-update baseline: new entries are clusters of their own until a window is full, its own k-means then
    replaces them; several windows, mixed call styles, the prefill's clusters untouched."""
    s = CONFIGS["llama3_8b"].scaled(dtype=dtype, prefill=1024, n_clusters_init=40, budget=300, max_cluster_factor=8, drift_std=0.08)
    steps = 2 * W + 9
    r = run_trajectory(s, [0, 1], steps, check_every=1, full_every=7, step_call="mixed", update_mode=3, local_window=W,
                       local_clusters=k, kmeans_iters=3)
    say("local update", dtype, W, k, {x: r[x] for x in ("worst_rel", "ties", "splits", "clusters")})
    assert r["clusters"] == [40 + 2 * k + 9] * 2 and r["splits"] == 0


def test_capacity_limits_set_the_error_word_and_keep_state():
    s = WorkloadSpec("cap", "f16", 1, 2, 64, 8, 4, 32, 4, 0.5, var_alpha=0.5, size_factor=0.0, buffer_max=0,
                     max_cluster_factor=1, seed=5)
    w = generate(s)
    ix, o, tally = _build_pair(s, w, 1, max_tokens=68)
    assert ix.export_status == binding.OK
    Kd, Vd = to_dev(w["Knew"], "f16"), to_dev(w["Vnew"], "f16")
    for t in range(8):                          # 4 appends fit, then max_tokens; splits have no free cluster id
        ix.dynakv_append(Kd[t], Vd[t]); o.append(w["Knew"][t], w["Vnew"][t])
        ix.dynakv_split(); o.split()
        assert not compare_state(ix, o, tally, "cap step %d" % t)
    st = ix.dynakv_export_state(["error", "n_tokens", "n_clusters"])
    assert ix.export_status == binding.ECAPACITY      # the sticky words leave the device as a status
    assert st["n_tokens"][0] == 68 and st["n_clusters"][0] == 4
    assert st["error"][0] & binding.ERR_TOKENS and st["error"][0] & binding.ERR_CLUSTERS
    assert "capacity" in binding.load().dynakv_strerror(binding.ECAPACITY).decode()


@pytest.mark.parametrize("launch", [0, launch_shape(0, 0, LAUNCH_SEPARATE)])
def test_whole_step_call_at_the_capacity_limits(launch):
    s = WorkloadSpec("cap", "f16", 1, 2, 64, 8, 4, 32, 4, 0.5, var_alpha=0.5, size_factor=0.0, buffer_max=0,
                     max_cluster_factor=1, seed=5)
    w = generate(s)
    ix, o, tally = _build_pair(s, w, 1, max_tokens=68, launch=launch)
    Qd, Kd, Vd = to_dev(w["Q"], "f16"), to_dev(w["Knew"], "f16"), to_dev(w["Vnew"], "f16")
    out = torch.empty(1, 2, 128, device=DEV)
    lse = torch.empty(1, 2, device=DEV)
    for t in range(8):
        ix.dynakv_decode_step(Qd[t], 32, out, lse, Kd[t], Vd[t])
        oo, ol = o.retrieve_attend(w["Q"][t], 32)
        assert not compare_retrieval(ix, o, tally, "cap step %d" % t, gather=False, Q=w["Q"][t], budget=32)
        check_attention(out.cpu().numpy(), lse.cpu().numpy(), oo, ol, "cap step %d" % t)
        o.append(w["Knew"][t], w["Vnew"][t]); o.split()
        assert not compare_state(ix, o, tally, "cap step %d" % t)
    st = ix.dynakv_export_state(["error", "n_tokens"])
    assert st["n_tokens"][0] == 68 and st["error"][0] & binding.ERR_TOKENS and ix.export_status == binding.ECAPACITY


def test_initial_positions_out_of_range_or_repeated_set_the_error_word():
    s = CONFIGS["tiny"].scaled(prefill=300, n_clusters_init=12)
    w = generate(s, steps=1)
    ix, _ = make_pair(s, 1)
    K0, V0 = to_dev(w["K0"], "f32"), to_dev(w["V0"], "f32")
    for bad, want in ((None, 0), ((3, 300), binding.ERR_INIT), ((5, -1), binding.ERR_INIT), ((7, "dup"), binding.ERR_INIT)):
        init = w["init_idx"].copy()
        if bad:
            init[0, bad[0]] = init[0, 0] if bad[1] == "dup" else bad[1]
        ix.dynakv_build_index(K0, V0, torch.from_numpy(init).to(DEV))
        st = ix.dynakv_export_state(["error", "n_clusters", "n_tokens"])
        assert st["error"][0] == want and st["n_clusters"][0] == 12 and st["n_tokens"][0] == 300, bad
        assert ix.export_status == (binding.ECAPACITY if want else binding.OK)


def test_prefill_with_a_wide_key_range():
    """Keys whose exponents span far more bits than a float64 sum keeps exact (bfloat16, a few keys scaled far up
    and far down): the centres are still float64 sums of the members."""
    s = WorkloadSpec("wide", "bf16", 2, 2, 1500, 4, 24, 256, 6, 0.05, var_alpha=0.0, size_factor=0.0, seed=123)
    w = generate(s)
    K0 = w["K0"].copy()
    K0[:, 5] *= 2.0 ** 30
    K0[:, 77] *= 2.0 ** 30
    K0[:, 300:303] *= 2.0 ** -40
    ix, o, tally = _build_pair(s, w, 2, K0=K0, kmeans_iters=5)
    say("wide range", dict(tally))


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_prefill_with_coinciding_centres(dtype):
    """Keys drawn from a handful of distinct vectors, so that many initial centres coincide: points whose nearest
    centre is one of several equal ones (lowest id wins on both sides: exact ties are not disagreements)."""
    s = WorkloadSpec("dup", dtype, 2, 2, 900, 4, 40, 256, 6, 0.05, var_alpha=0.0, size_factor=0.0, seed=321)
    w = generate(s)
    K0 = w["K0"].copy()
    for u, distinct in enumerate((3, 11)):
        base = K0[u, :distinct].copy()
        K0[u, :600] = base[np.arange(600) % distinct]          # the remaining 300 keys stay as drawn
    init = np.tile(np.arange(40, dtype=np.int32), (2, 1))      # the first 40 keys: 3 resp. 11 distinct centres
    ix, o, tally = _build_pair(s, w, 2, K0=K0, init=init, kmeans_iters=4)
    assert tally["tie_kmeans"] == 0


@pytest.mark.parametrize("dtype,N0,M0", [
    ("f16", 257, 1), ("f16", 300, 31), ("bf16", 321, 33), ("f16", 4100, 64), ("bf16", 1025, 65), ("f32", 130, 33),
    ("f16", 3000, 2),          # hundreds of keys move from one cluster to the other at once
    ("bf16", 5000, 17),        # and from many clusters to many
    ("f16", 9000, 2100),       # more than 8192 float16 keys: whether sums may follow the moves depends on their range
    ("bf16", 8300, 8192)])     # the most centres: counts of the sort for four wavefronts only
def test_prefill_partition_at_the_edges_of_tiles_and_chunks(dtype, N0, M0):
    """Labels, centres and statistics of the k-means where the last tile of 32 centres, chunk of 64 points or run of 16
    clusters is partly filled; memberships exactly as the oracle's."""
    s = WorkloadSpec("edges", dtype, 2, 2, N0, 4, M0, 256, 6, 0.05, var_alpha=0.0, size_factor=0.0, seed=N0 + M0)
    ix, o, tally = _build_pair(s, generate(s), 2, kmeans_iters=3 if M0 > 2000 else 5)
    assert tally["tie_kmeans"] == 0


@pytest.mark.parametrize("dtype,scale", [("f16", 0.0), ("bf16", 0.0), ("f32", 0.0), ("f16", 2.0 ** -24), ("bf16", 1e-20), ("bf16", 1e-38)])
@pytest.mark.parametrize("M0", [2, 3, 40])
def test_prefill_with_keys_of_zero_and_at_the_end_of_the_range(dtype, scale, M0):
    """Equal distances of zero go to the lowest id, and distances that float32 cannot tell from zero are told apart in
    float64.  Where the keys are zero, the second unit also holds entries of ordinary size."""
    N0 = 200
    s = WorkloadSpec("zero", dtype, 2, 2, N0, 4, M0, 64, 4, 0.05, var_alpha=1.5, size_factor=0.0, seed=9)
    w = generate(s)
    rng = np.random.default_rng(3)
    q = lambda a: torch.from_numpy(a.astype(np.float32)).to(binding.TORCH_DTYPES[dtype]).float().numpy()  # noqa: E731
    w["K0"][0] = q(rng.integers(-2, 3, (N0, 128)) * np.float32(scale))
    w["K0"][1, :N0 if scale else 120] = q(rng.standard_normal((N0 if scale else 120, 128)) * np.float32(scale))
    w["init_idx"][:] = np.arange(M0)
    ix, o = make_pair(s, 2, kmeans_iters=3)
    ix.dynakv_build_index(to_dev(w["K0"], dtype), to_dev(w["V0"], dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    o.build_index(w["K0"], w["V0"], w["init_idx"])
    st = ix.dynakv_export_state(["offsets", "members", "error"])
    assert not st["error"].any()
    for u in range(2):
        off, mem = o.members(u)
        np.testing.assert_array_equal(st["offsets"][u, :M0 + 1].numpy(), off)
        np.testing.assert_array_equal(st["members"][u, :N0].numpy(), mem)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("bad", [(np.inf,), (-np.inf, np.inf), (np.nan, np.inf)])
def test_prefill_with_keys_that_are_not_finite(dtype, bad):
    """Such a key is at no finite distance from any centre: the lowest id takes it, its centre is then nearest to
    no other key, and the partition of all others is the oracle's."""
    U, N0, M0 = 2, 700, 12
    s = WorkloadSpec("inf", dtype, U, 2, N0, 4, M0, 256, 6, 0.05, var_alpha=1.5, size_factor=0.0, seed=77)
    w = generate(s)
    for i, x in enumerate(bad):
        w["K0"][:, 300 + 170 * i, 5 + 40 * i] = x
    ix, o = make_pair(s, U, kmeans_iters=5)
    ix.dynakv_build_index(to_dev(w["K0"], dtype), to_dev(w["V0"], dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    o.build_index(w["K0"], w["V0"], w["init_idx"])
    st = ix.dynakv_export_state(["size", "offsets", "members", "centroids", "error"])
    assert not st["error"].any()
    for u in range(U):
        off, mem = o.members(u)
        np.testing.assert_array_equal(st["offsets"][u, :M0 + 1].numpy(), off)
        np.testing.assert_array_equal(st["members"][u, :N0].numpy(), mem)
        c = o.clusters(u)["centroids"]
        np.testing.assert_allclose(st["centroids"][u, :M0].numpy(), c, rtol=1e-6, atol=1e-6)
        assert not np.isfinite(c[0]).all() and np.isfinite(c[1:]).all()


@pytest.mark.parametrize("dtype,M0,N0", [("bf16", 65, 700), ("bf16", 513, 1200), ("bf16", 1100, 2000), ("f16", 600, 9000), ("f32", 40, 300)])
@pytest.mark.parametrize("distinct", [0, 30])
def test_prefill_forms_all_sums_anew_and_reseeds(dtype, M0, N0, distinct):
    """Units whose sums are not order-free (one coordinate at the end of the type's range; more than 8192 float16 keys need
    that check), with one and with several workgroups to a unit; with few distinct keys most clusters run empty in every
    iteration and choose one after the other, more of them than there are keys at any distance."""
    s = WorkloadSpec("anew", dtype, 2, 2, N0, 4, M0, 64, 4, 0.05, var_alpha=1.5, size_factor=0.0, seed=M0 + distinct)
    w = generate(s)
    if distinct:
        w["K0"][1] = w["K0"][1, np.random.default_rng(2).integers(0, distinct, N0)]
    w["K0"][:, 3, 17] = 2.0 ** -24 if dtype == "f16" else 1e-30
    w["K0"][0, 9] *= 40.0
    w["K0"] = torch.from_numpy(w["K0"]).to(binding.TORCH_DTYPES[dtype]).float().numpy()
    ix, o = make_pair(s, 2, kmeans_iters=3 if N0 > 5000 else 5)
    ix.dynakv_build_index(to_dev(w["K0"], dtype), to_dev(w["V0"], dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    o.build_index(w["K0"], w["V0"], w["init_idx"])
    st = ix.dynakv_export_state(["offsets", "members", "centroids", "error"])
    assert not st["error"].any()
    for u in range(2):
        moff, mem = o.members(u)
        np.testing.assert_array_equal(st["offsets"][u, :M0 + 1].numpy(), moff)
        np.testing.assert_array_equal(st["members"][u, :N0].numpy(), mem)
        # sums of the same numbers in the same order, rounded to float32 once
        np.testing.assert_allclose(st["centroids"][u, :M0].numpy(), o.clusters(u)["centroids"], rtol=1.2e-7, atol=0)


@pytest.mark.parametrize("dtype,M0,N0,offset", [
    ("f16", 60, 700, 2), ("f16", 150, 1000, 200), ("bf16", 129, 513, 30), ("f16", 300, 1000, 15), ("bf16", 700, 1500, 200), ("f16", 5, 400, 8000)])
def test_prefill_where_most_keys_have_many_candidates(dtype, M0, N0, offset):
    """Keys about a common offset far beyond their spread, which the 16-bit filter hardly tells apart, and keys of a few
    values each, where every key has several equal centres: such keys are decided among all centres in float64, with one,
    two or four wavefronts to a batch of them."""
    s = WorkloadSpec("offset", dtype, 2, 2, N0, 4, M0, 64, 4, 0.05, var_alpha=1.5, size_factor=0.0, n_outliers=0, seed=M0)
    w = generate(s)
    rng = np.random.default_rng(1)
    w["K0"][0] += offset * rng.standard_normal((1, 128)).astype(np.float32)
    w["K0"][1] = w["K0"][1, :M0 // 4][rng.integers(0, M0 // 4, N0)]
    w["K0"] = torch.from_numpy(w["K0"]).to(binding.TORCH_DTYPES[dtype]).float().numpy()
    ix, o = make_pair(s, 2, kmeans_iters=4)
    ix.dynakv_build_index(to_dev(w["K0"], dtype), to_dev(w["V0"], dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    o.build_index(w["K0"], w["V0"], w["init_idx"])
    st = ix.dynakv_export_state(["offsets", "members", "error"])
    assert not st["error"].any()
    for u in range(2):
        moff, mem = o.members(u)
        np.testing.assert_array_equal(st["offsets"][u, :M0 + 1].numpy(), moff)
        np.testing.assert_array_equal(st["members"][u, :N0].numpy(), mem)


def _blocked_sqdist(x, r):
    """The library's float64 squared distance: blocks of 8 coordinates by fused multiply-adds, block sums left to right."""
    total = 0.0
    for k in range(16):
        blk = 0.0
        for e in range(8):
            t = float(x[8 * k + e]) - float(r[8 * k + e])
            blk = float(Fraction(t) * Fraction(t) + Fraction(blk))
        total += blk
    return total


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("M0", [2, 3, 7])
def test_prefill_decides_equal_distances_by_one_order_of_summation(dtype, M0):
    """Centres that are block rotations of each other are equally far from a key whose blocks are all alike, up to the
    rounding of the sum: with two of them (pair comparison) and with more (all centres) that decides as in one fixed
    order.  The reseeding's farthest key likewise: two equal centres, candidates that are rotations of each other."""
    rng = np.random.default_rng(5 + M0)
    q = lambda a: torch.from_numpy(a.astype(np.float32)).to(binding.TORCH_DTYPES[dtype]).float().numpy()  # noqa: E731
    # magnitudes over a range whose squares do not fit 53 bits together
    a = q(rng.standard_normal((16, 8)) * np.exp2(rng.integers(-14, 4, (16, 8))))
    same = q(np.tile(rng.standard_normal((90, 1, 8)) * np.exp2(rng.integers(-14, 3, (90, 1, 8))), (1, 16, 1)))
    rot = np.stack([np.roll(a, 2 * j + 1, axis=0) for j in range(M0)])
    K = np.concatenate([rot, same]).reshape(1, -1, 128).astype(np.float32)
    U = 1

    def labels(K, init, iters):
        ix = binding.Index(binding.Config(U, 2, dtype, len(init), 4 * len(init), K.shape[1], iters), DEV)
        Kd = to_dev(K, dtype)
        ix.dynakv_build_index(Kd, Kd, torch.tensor([init], dtype=torch.int32, device=DEV))
        st = ix.dynakv_export_state(["offsets", "members"])
        lab = np.zeros(K.shape[1], int)
        for j in range(len(init)):
            lab[st["members"][0, st["offsets"][0, j]:st["offsets"][0, j + 1]].numpy()] = j
        return lab

    got = labels(K, list(range(M0)), 1)
    want = [int(np.argmin([_blocked_sqdist(x, r) for r in K[0, :M0]])) for x in K[0]]
    np.testing.assert_array_equal(got, want)
    assert len(set(want[M0:])) > 1                       # the rounding does decide
    if M0 == 7:
        K2 = np.concatenate([np.zeros((2, 16, 8), np.float32)] + [np.roll(a, j, axis=0)[None] for j in range(16)]).reshape(1, -1, 128)
        d = [_blocked_sqdist(x, K2[0, 0]) for x in K2[0]]
        assert len(set(d[2:])) > 1
        got = labels(K2, [0, 1], 2)
        assert np.flatnonzero(got).tolist() == [int(np.argmax(d))]


def test_rebuild_resets_the_index_and_runs_are_deterministic():
    s = CONFIGS["tiny"].scaled(prefill=777, n_clusters_init=19)
    w = generate(s, steps=8)
    ix, o = make_pair(s, 1)
    K0, V0, init = to_dev(w["K0"], "f32"), to_dev(w["V0"], "f32"), torch.from_numpy(w["init_idx"]).to(DEV)
    ix.dynakv_build_index(K0, V0, init)
    for t in range(8):
        ix.dynakv_append(to_dev(w["Knew"][t], "f32"), to_dev(w["Vnew"][t], "f32"))
    a = ix.dynakv_export_state()
    ix.dynakv_build_index(K0, V0, init)
    o.build_index(w["K0"], w["V0"], w["init_idx"])
    compare_build(ix, o, Tally(), 777)
    for t in range(8):
        ix.dynakv_append(to_dev(w["Knew"][t], "f32"), to_dev(w["Vnew"][t], "f32"))
    b = ix.dynakv_export_state()
    for k in a:
        assert torch.equal(a[k], b[k]), k


def test_timing_aid_brackets_an_even_sample_of_the_launches():
    s = CONFIGS["llama3_8b"].scaled(prefill=512, n_clusters_init=32, budget=128)
    U = 2
    w = generate(s, units=range(U), steps=32)
    ix = binding.Index(binding.Config(U, s.group_size, s.dtype, 32, 128, 512 + 32, 3, 16, 0, s.var_alpha, s.size_factor, 0.0), DEV)
    ix.dynakv_build_index(to_dev(w["K0"], s.dtype), to_dev(w["V0"], s.dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    Qd, Kd, Vd = to_dev(w["Q"], s.dtype), to_dev(w["Knew"], s.dtype), to_dev(w["Vnew"], s.dtype)
    out, lse = torch.empty(U, s.group_size, 128, device=DEV), torch.empty(U, s.group_size, device=DEV)
    lib = binding.load()
    assert lib.dynakv_profile_sample(ix._h, 0, 1) == binding.EINVAL and lib.dynakv_profile_sample(ix._h, 4, 5) == binding.EINVAL
    t = 0
    for every, run, steps, want in ((1, 1, 6, 6), (4, 2, 10, 6), (4, 4, 7, 4), (3, 1, 6, 2)):
        ix.dynakv_profile_sample(every, run)
        ix.dynakv_profile_enable(16)
        for _ in range(steps):
            ix.dynakv_decode_step(Qd[t], 128, out, lse, Kd[t], Vd[t])
            t += 1
        n, ms = ix.dynakv_profile_read()
        assert n == want and 0.0 < ms < 50.0, (every, run, steps, n, ms)
    ix.dynakv_profile_sample(1, 1)
    ix.dynakv_profile_enable(0)


# --------------------------------------------------------------------------- exported and imported state

@pytest.mark.parametrize("dtype,N0,M0,Mcap", [("f16", 1501, 3, 67), ("f32", 700, 65, 65), ("bf16", 333, 333, 9000)])
def test_snapshot_round_trip(dtype, N0, M0, Mcap):
    """Export, import into a second index and export again: clusters of many pages (chains past the inline page table),
    capacities that are no multiple of a table tile, far more slots than clusters."""
    s = WorkloadSpec("snap", dtype, 3, 2, N0, 4, M0, 256, 6, 0.05, var_alpha=1.5, size_factor=0.0, seed=99 + N0)
    w = generate(s)
    a, _ = make_pair(s, 3, max_clusters=Mcap, kmeans_iters=2)
    b, _ = make_pair(s, 3, max_clusters=Mcap, kmeans_iters=2)
    a.dynakv_build_index(to_dev(w["K0"], dtype), to_dev(w["V0"], dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    a.dynakv_retrieve_attend(to_dev(w["Q"][0], dtype), 256, torch.empty(3, 2, 128, device=DEV), None)
    x = a.dynakv_export_state(binding.IMPORT_FIELDS, to_cpu=False)
    b.dynakv_import_state(x)
    y = b.dynakv_export_state(binding.IMPORT_FIELDS + ("error",), to_cpu=False)
    assert int(y["error"].abs().sum()) == 0
    for k in x:
        assert torch.equal(x[k], y[k]), k
    K = to_dev(w["K0"], dtype)
    for u in range(3):
        m = x["members"][u, :N0].long()
        assert torch.equal(torch.sort(m).values, torch.arange(N0, device=DEV))
        assert torch.equal(x["keys"][u, :N0], K[u])


@pytest.mark.parametrize("dtype", ["f16", "f32"])
def test_snapshot_and_retrieval_of_many_clusters(dtype):
    """More clusters than one round of the snapshots' prefix sums (8192) and one trip of the selection's passes over all
    scores (16384) take: the snapshot comes out of the index as it went in, and retrievals are the oracle's."""
    U, N, Mcap, Ncap, Ms = 2, 41003, 21003, 41010, (20001, 8193)
    gen = torch.Generator(device=DEV).manual_seed(5)
    rnd = lambda *a: torch.randn(*a, generator=gen, device=DEV)  # noqa: E731
    K, V = rnd(U, Ncap, 128).to(binding.TORCH_DTYPES[dtype]), rnd(U, Ncap, 128).to(binding.TORCH_DTYPES[dtype])
    K[:, N:], V[:, N:] = 0, 0
    i32 = lambda *a: torch.zeros(*a, dtype=torch.int32, device=DEV)  # noqa: E731
    x = dict(n_clusters=torch.tensor(Ms, dtype=torch.int32, device=DEV), n_tokens=torch.full((U,), N, dtype=torch.int32, device=DEV),
             tau=torch.tensor([1.5, 2.5], dtype=torch.float64, device=DEV), centroids=torch.zeros(U, Mcap, 128, device=DEV),
             size=i32(U, Mcap), buffered=i32(U, Mcap), flag=i32(U, Mcap), m2=torch.zeros(U, Mcap, dtype=torch.float64, device=DEV),
             offsets=i32(U, Mcap + 1), members=i32(U, Ncap), n_selected=i32(U), selected=torch.full((U, Mcap), -1, dtype=torch.int32, device=DEV),
             keys=K, values=V)
    for u, M in enumerate(Ms):
        label = torch.cat([torch.arange(M, device=DEV), torch.randint(0, M, (N - M,), generator=gen, device=DEV)])
        label = label[torch.randperm(N, generator=gen, device=DEV)]
        order = torch.argsort(label, stable=True)
        stored = torch.bincount(label, minlength=M).int()
        flag = (torch.arange(M, device=DEV) % 977 == 5).int()
        x["flag"][u, :M] = flag
        x["buffered"][u, :M] = torch.where((flag > 0) & (stored > 1), torch.ones_like(stored), torch.zeros_like(stored))
        x["size"][u, :M] = stored - x["buffered"][u, :M]
        x["m2"][u, :M] = torch.rand(M, generator=gen, device=DEV).double()
        x["offsets"][u, 1:M + 1] = stored.cumsum(0).int()
        x["offsets"][u, M + 1:] = N
        x["members"][u, :N] = order.int()
        x["centroids"][u, :M] = torch.zeros(M, 128, device=DEV).index_add_(0, label, K[u, :N].float()) / stored[:, None]
        x["n_selected"][u] = 3000
        x["selected"][u, :3000] = torch.randperm(M, generator=gen, device=DEV)[:3000].int()
    s = WorkloadSpec("many", dtype, U, 4, N, 7, 8, 2500, 8, 0.05, var_alpha=1.5, size_factor=0.0)
    ix, o = make_pair(s, U, max_tokens=Ncap, max_clusters=Mcap)
    ix.dynakv_import_state(x)
    y = ix.dynakv_export_state(binding.IMPORT_FIELDS + ("error",), to_cpu=False)
    assert not y["error"].any()
    for k in x:
        assert torch.equal(x[k], y[k]), k
    tally = Tally()
    parity.resync(ix, o, None, {0, 1}, tally)
    out, lse = torch.empty(U, 4, 128, device=DEV), torch.empty(U, 4, device=DEV)
    for t, budget in enumerate((1, 60, 2500, 4900)):
        Q = K[:, 100 * t, None].float() + 0.5 * rnd(U, 4, 128)
        Qs = Q.to(binding.TORCH_DTYPES[dtype])
        Qn = Qs.float().cpu().numpy()
        ix.dynakv_retrieve_attend(Qs.contiguous(), budget, out, lse)
        oo, ol = o.retrieve_attend(Qn, budget)
        dirty = compare_retrieval(ix, o, tally, "budget %d" % budget, Q=Qn, budget=budget)
        keep = [u for u in range(U) if u not in dirty]
        check_attention(out.cpu().numpy()[keep], lse.cpu().numpy()[keep], oo[keep], ol[keep], "budget %d" % budget)
    assert not ix.dynakv_export_state(["error"])["error"].any()
    say("many clusters", dtype, dict(tally))


def test_snapshot_arrays_need_their_element_alignment_only():
    """Centroids of a snapshot at an address that is a multiple of four bytes and no more, out and in."""
    s = WorkloadSpec("align", "f16", 2, 2, 300, 4, 21, 100, 6, 0.05, var_alpha=1.5, size_factor=0.0, seed=31)
    w = generate(s)
    a, b = (make_pair(s, 2, max_clusters=90, kmeans_iters=2)[0] for _ in range(2))
    a.dynakv_build_index(to_dev(w["K0"], "f16"), to_dev(w["V0"], "f16"), torch.from_numpy(w["init_idx"]).to(DEV))
    x = a.dynakv_export_state(binding.IMPORT_FIELDS, to_cpu=False)
    flat = torch.full((2 * 90 * 128 + 2,), 5.0, device=DEV)
    odd = flat[1:-1].view(2, 90, 128)
    assert odd.data_ptr() % 16 == 4
    st = binding._State(**{k: (odd.data_ptr() if k == "centroids" else None) for k in binding._STATE_FIELDS})
    assert a._lib.dynakv_export_state(a._h, ctypes.byref(st), torch.cuda.current_stream().cuda_stream) == binding.OK
    assert torch.equal(odd, x["centroids"]) and flat[0] == 5.0 and flat[-1] == 5.0
    b.dynakv_import_state(dict(x, centroids=odd))
    y = b.dynakv_export_state(binding.IMPORT_FIELDS, to_cpu=False)
    assert torch.equal(y["centroids"], x["centroids"]) and torch.equal(y["members"], x["members"])


@pytest.mark.parametrize("dtype,launch,Mcap,kw", [
    ("f16", 0, 200, {}), ("bf16", launch_shape(2, 0, LAUNCH_SEPARATE), 200, {}), ("f32", 0, 200, {}),
    ("f16", 0, 17000, {}), ("f16", 0, 200, dict(search_copy=1)), ("bf16", LAUNCH_SPLIT_KERNEL, 200, {})])
def test_units_refused_by_the_first_import_are_empty(dtype, launch, Mcap, kw):
    """On a handle without a state an import that refuses a unit leaves it empty, whatever the workspace held: every
    later call is defined on it (exports of nothing, zeros, refused appends) and its neighbours are as if alone."""
    N0, M0, U = 500, 20, 3
    s = WorkloadSpec("refuse", dtype, U, 2, N0, 6, M0, 100, 6, 0.05, var_alpha=1.5, size_factor=0.0, seed=23)
    w = generate(s)
    a, b = (make_pair(s, U, max_clusters=Mcap, kmeans_iters=2, launch=launch, **kw)[0] for _ in range(2))
    K, V = to_dev(w["K0"], dtype), to_dev(w["V0"], dtype)
    a.dynakv_build_index(K, V, torch.from_numpy(w["init_idx"]).to(DEV))
    snap = a.dynakv_export_state(binding.IMPORT_FIELDS, to_cpu=False)
    snap["n_clusters"][0], snap["n_tokens"][2] = Mcap + 1, -1
    b.workspace.fill_(0x5A)
    b.dynakv_import_state(snap)
    st = b.dynakv_export_state(binding.IMPORT_FIELDS + ("error", "counters", "last_assign", "n_gathered", "first_page"))
    assert st["error"].tolist() == [binding.ERR_IMPORT, 0, binding.ERR_IMPORT]
    for u in (0, 2):
        for k in ("n_clusters", "n_tokens", "n_selected", "n_gathered", "tau", "size", "offsets", "members", "centroids", "counters"):
            assert not st[k][u].any(), k
    Q, kn, vn = (to_dev(w[k], dtype) for k in ("Q", "Knew", "Vnew"))
    outs = []
    for ix in (a, b):
        out, lse = torch.full((6, U, 2, 128), 7.0, device=DEV), torch.full((6, U, 2), 7.0, device=DEV)
        for t in range(4):
            ix.dynakv_decode_step(Q[t], 100, out[t], lse[t], kn[t], vn[t])
        ix.dynakv_retrieve_attend(Q[4], 100, out[4], lse[4])
        ix.dynakv_append(kn[4], vn[4])
        ix.dynakv_split()
        ix.dynakv_extend_index(kn[5][:, None].contiguous(), vn[5][:, None].contiguous())
        ix.dynakv_retrieve_attend(Q[5], 100, out[5], lse[5])
        outs.append((out.cpu(), lse.cpu()))
    (oa, la), (ob, lb) = outs
    assert torch.allclose(oa[:, 1], ob[:, 1], rtol=3e-5, atol=3e-6) and torch.allclose(la[:, 1], lb[:, 1], rtol=3e-5)
    assert not ob[:, [0, 2]].any() and bool((lb[:, [0, 2]] == -float("inf")).all())
    sa, sb = (ix.dynakv_export_state(("error", "n_clusters", "n_tokens", "size", "members", "offsets")) for ix in (a, b))
    assert sb["error"].tolist() == [binding.ERR_IMPORT | binding.ERR_TOKENS, 0, binding.ERR_IMPORT | binding.ERR_TOKENS]
    assert sb["n_tokens"].tolist() == [0, N0 + 6, 0]
    for k in ("n_clusters", "size", "members", "offsets"):
        assert torch.equal(sa[k][1], sb[k][1]) and not sb[k][[0, 2]].any(), k
    b.dynakv_place_by_coretrieval(K, V, Q[:2].contiguous(), 100)     # nothing to place in any of them
    assert all(e & binding.ERR_PLACE for e in b.dynakv_export_state(["error"])["error"].tolist())


@pytest.mark.parametrize("name,launch", [("llama3_8b", 0), ("tiny", 0), ("qwen25_7b", launch_shape(2, 0, LAUNCH_SEPARATE))])
def test_imported_state_continues_like_the_exporting_index(name, launch):
    """dynakv_export_state -> dynakv_import_state into a second index: both then take the same steps and must
    agree on every decision and, since both run the same kernels on the same values, on every exported bit
    except the page-dependent gather order inside a step."""
    s = CONFIGS[name].scaled(prefill=1024, n_clusters_init=48, budget=256, var_alpha=1.25 if name != "tiny" else 0.0)
    U = 3
    w = generate(s, units=range(U), steps=96)
    mk = lambda: binding.Index(binding.Config(U, s.group_size, s.dtype, 48, 192, 1024 + 96, 4, 4, 0, s.var_alpha,
                                              s.size_factor, 0.0, launch=launch), DEV)
    a, b = mk(), mk()
    a.dynakv_build_index(to_dev(w["K0"], s.dtype), to_dev(w["V0"], s.dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    Qd, Kd, Vd = to_dev(w["Q"], s.dtype), to_dev(w["Knew"], s.dtype), to_dev(w["Vnew"], s.dtype)
    oa, la = torch.empty(U, s.group_size, 128, device=DEV), torch.empty(U, s.group_size, device=DEV)
    ob, lb = torch.empty_like(oa), torch.empty_like(la)
    for t in range(48):
        a.dynakv_decode_step(Qd[t], 256, oa, la, Kd[t], Vd[t])
    a.dynakv_retrieve_attend(Qd[48], 256, oa, la)              # the active set travels with the state
    snap = a.dynakv_export_state(binding.IMPORT_FIELDS, to_cpu=False)
    if name == "llama3_8b":
        assert int(snap["flag"].sum()) > 0                     # flagged clusters and their buffers are part of it
    b.dynakv_import_state(snap)
    fields = ("n_clusters", "n_tokens", "error", "tau", "centroids", "size", "buffered", "flag", "m2", "offsets", "members",
              "keys", "values")
    sa, sb = a.dynakv_export_state(fields), b.dynakv_export_state(fields)
    for k in fields:
        assert torch.equal(sa[k], sb[k]), "right after the import: " + k
    for ix in (a, b):
        ix.dynakv_append(Kd[48], Vd[48]); ix.dynakv_split()
    for t in range(49, 96):
        a.dynakv_decode_step(Qd[t], 256, oa, la, Kd[t], Vd[t])
        b.dynakv_decode_step(Qd[t], 256, ob, lb, Kd[t], Vd[t])
        assert torch.allclose(oa, ob, rtol=2e-3, atol=1e-6) and torch.allclose(la, lb, atol=2e-3), t
    sa, sb = a.dynakv_export_state(fields + ("scores", "n_selected", "n_gathered")), b.dynakv_export_state(fields + ("scores", "n_selected", "n_gathered"))
    for k in sa:
        assert torch.equal(sa[k], sb[k]), k
    assert int(sa["n_clusters"].max()) > 48
    # an inconsistent snapshot is refused unit by unit and leaves the index as it was
    snap["n_clusters"][1] = 10 ** 6
    snap["offsets"][2, 1] += 1
    b.dynakv_import_state(snap)
    sb2 = b.dynakv_export_state(("error", "n_clusters", "n_tokens", "members"))
    assert b.export_status == binding.ECAPACITY
    assert sb2["error"].tolist() == [0, binding.ERR_IMPORT, binding.ERR_IMPORT]
    assert torch.equal(sb2["members"][1:], sb["members"][1:]) and torch.equal(sb2["n_tokens"][1:], sb["n_tokens"][1:])
    assert int(sb2["n_tokens"][0]) == 1024 + 48
