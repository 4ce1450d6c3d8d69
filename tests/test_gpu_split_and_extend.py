"""GPU parity of splits over every way a cluster can be split and of the chunked prefill across its batches, from snapshots that
put each size at the edge where the next way begins."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import parity  # noqa: E402
from parity import DEV, Tally, compare_build, compare_state, make_pair, to_dev  # noqa: E402
from paper_2511_07427_amd import binding  # noqa: E402
from paper_2511_07427_amd.binding import LAUNCH_SEPARATE, launch_shape  # noqa: E402
from paper_2511_07427_amd.workload import CONFIGS, WorkloadSpec, generate  # noqa: E402

pytestmark = pytest.mark.gpu
D = 128


def snapshot(dtype, sizes, flagged, max_clusters, capacity, gen, offset=0.0, tau=1.0):
    """One state for all units: unit u's clusters hold sizes[u][j] entries (the first flagged[u] of them flagged, with one entry
    buffered), each cluster a walk away from a mean of its own, all keys about a common offset."""
    U = len(sizes)
    dt = binding.TORCH_DTYPES[dtype]
    rnd = lambda *s: torch.randn(*s, generator=gen, device=DEV)  # noqa: E731
    i32 = lambda *s: torch.zeros(*s, dtype=torch.int32, device=DEV)  # noqa: E731
    st = dict(n_clusters=i32(U), n_tokens=i32(U), tau=torch.full((U,), tau, dtype=torch.float64, device=DEV),
              centroids=torch.zeros(U, max_clusters, D, device=DEV), size=i32(U, max_clusters), buffered=i32(U, max_clusters),
              flag=i32(U, max_clusters), m2=torch.zeros(U, max_clusters, dtype=torch.float64, device=DEV),
              offsets=i32(U, max_clusters + 1), members=i32(U, capacity), keys=torch.zeros(U, capacity, D, dtype=dt, device=DEV),
              values=torch.zeros(U, capacity, D, dtype=dt, device=DEV))
    for u, sz in enumerate(sizes):
        M, n = len(sz), sum(sz)
        label = torch.repeat_interleave(torch.arange(M, device=DEV), torch.tensor(sz, device=DEV))
        K = rnd(M, D)[label] + 0.3 * rnd(n, D) + offset * rnd(1, D)
        start = 0
        for j in range(flagged[u]):
            K[start:start + sz[j]] += (0.4 * rnd(sz[j], D) * (8.0 / sz[j]) ** 0.5).cumsum(0)
            start += sz[j]
        label = label[torch.randperm(n, generator=gen, device=DEV)]       # positions of a cluster's entries: anywhere
        order = torch.argsort(label, stable=True)
        keys = torch.empty_like(K)
        keys[order] = K
        st["keys"][u, :n], st["values"][u, :n] = keys.to(dt), rnd(n, D).to(dt)
        stored = torch.tensor(sz, dtype=torch.int32, device=DEV)
        st["n_clusters"][u], st["n_tokens"][u] = M, n
        st["flag"][u, :flagged[u]] = 1
        st["buffered"][u, :flagged[u]] = 1
        st["size"][u, :M] = stored - st["buffered"][u, :M]
        st["offsets"][u, 1:M + 1] = stored.cumsum(0).int()
        st["offsets"][u, M + 1:] = n
        st["members"][u, :n] = order.int()
        mean = torch.zeros(M, D, dtype=torch.float64, device=DEV).index_add_(0, label, st["keys"][u, :n].double()) / stored[:, None]
        st["centroids"][u, :M] = mean.float()
        st["m2"][u, :M] = torch.zeros(M, dtype=torch.float64, device=DEV).index_add_(
            0, label, (st["keys"][u, :n].double() - mean.float().double()[label]).square().sum(1))
    return st


def pair(dtype, sizes, flagged, max_clusters, extra=0, offset=0.0, seed=3, tau=1.0, **over):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    cap = max(sum(s) for s in sizes) + extra
    s = WorkloadSpec("edges", dtype, len(sizes), 2, cap, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=0, seed=seed)
    ix, o = make_pair(s, len(sizes), max_tokens=cap, max_clusters=max_clusters, **over)
    ix.dynakv_import_state(snapshot(dtype, sizes, flagged, max_clusters, cap, gen, offset, tau))
    tally = Tally()
    parity.resync(ix, o, None, set(range(len(sizes))), tally)
    return ix, o, tally, gen


SIZES = [2, 3, 5, 15, 16, 17, 32, 33, 63, 64, 65, 96, 97, 128, 129, 160, 161, 192, 255, 256, 257, 300]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("offset", [0.0, 30.0])
def test_splits_at_the_edges_of_every_path(dtype, offset):
    """One flagged cluster per unit of every size at which another path begins (16, 32, 64, 128, 160 and 256 entries), also with
    keys about an offset that the float32 filters of the 2-means cannot see past."""
    sizes = [[m, 7, 1, 12] for m in SIZES]
    ix, o, tally, _ = pair(dtype, sizes, [1] * len(sizes), 16, offset=offset)
    ix.dynakv_split()
    o.split()
    dirty = compare_state(ix, o, tally, "split", assign=False)
    ties = tally.get("tie_split", 0) + tally.get("tie_trigger", 0)
    print("split edges", dtype, offset, dict(tally), flush=True)
    assert len(dirty) <= ties and ties <= 2
    assert int(ix.dynakv_export_state(["n_clusters"])["n_clusters"].sum()) >= 5 * len(sizes) - 2


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("sizes,flagged", [((10, 200, 12, 8, 60, 31), 6), ((150, 9), 2), ((2, 2, 3, 130), 4), ((20, 300, 40), 3)])
def test_statistics_beside_a_large_cluster_are_float64_sums(dtype, sizes, flagged):
    """A plan with a cluster above 128 entries (64 of float32) takes the squares of all its children in float64: M2 is off by the
    roundings of two float64 sums of m * 128 squares in different orders, not by those of float32 squares (up to 2^-18)."""
    ix, o, tally, _ = pair(dtype, [list(sizes)] * 3, [flagged] * 3, 40, offset=3.0)
    ix.dynakv_split()
    o.split()
    assert not compare_state(ix, o, tally, "beside a large one", assign=False)
    print("beside a large cluster", dtype, sizes, dict(tally), flush=True)
    assert tally["m2_rel"] <= 2 * 128 * max(sizes) * 2.0 ** -53


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("scale,sizes", [(1e17, (6, 10, 14)), (1e17, (40, 26, 100)), (1e18, (20, 60, 8)), (1e19, (200, 40, 12)), (1e19, (140, 6, 20)),
                                         (1e19, (300, 20, 40))])
def test_splits_where_squared_distances_leave_float32(dtype, scale, sizes):
    """Keys so far apart that their squared distances reach 1e36 to 1e40, every one of them there twice (so that several members are
    farthest): such a cluster is split like any other."""
    sizes = list(sizes)
    cap = sum(sizes)
    gen = torch.Generator(device=DEV).manual_seed(71)
    st = snapshot(dtype, [sizes] * 2, [3] * 2, 16, cap, gen)
    off, mem = st["offsets"], st["members"].long()
    for u in range(2):
        for j, m in enumerate(sizes):
            a = mem[u, int(off[u, j]):int(off[u, j + 1])]
            x = (scale * (st["keys"][u, a[:m // 2]].float() - st["centroids"][u, j])).to(st["keys"].dtype)
            st["keys"][u, a] = torch.cat([x, x.flip(0)])
            st["centroids"][u, j] = st["keys"][u, a].double().mean(0).float()
    s = WorkloadSpec("far", dtype, 2, 2, cap, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=0, seed=71)
    ix, o = make_pair(s, 2, max_tokens=cap, max_clusters=16)
    ix.dynakv_import_state(st)
    tally = Tally()
    parity.resync(ix, o, None, {0, 1}, tally)
    ix.dynakv_split()
    o.split()
    assert not compare_state(ix, o, tally, "far apart", assign=False)
    assert ix.dynakv_export_state(["n_clusters"])["n_clusters"].tolist() == [6, 6]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("offset", [8.0, 100.0])
def test_small_clusters_about_a_large_offset(dtype, offset):
    """Clusters of up to 16 entries whose spread is of the order of what float32 inner products can tell apart: whatever they
    cannot decide goes to float64."""
    sizes = [[3 + (u + j) % 14 for j in range(7)] for u in range(64)]
    ix, o, tally, _ = pair(dtype, sizes, [7] * 64, 24, offset=offset)
    ix.dynakv_split()
    o.split()
    dirty = compare_state(ix, o, tally, "offset", assign=False)
    print("small clusters", dtype, offset, dict(tally), flush=True)
    assert len(dirty) <= tally.get("tie_split", 0) <= 4


# (value, members) of clusters whose 2-means ends on an exact tie: centres p and q with a member at (p + q) / 2, where sum * (1 / n)
# is not sum / n
TIED = [((0, 3), (1, 150), (4, 1), (5, 5), (7, 89), (9, 5)), ((2, 6), (3, 96), (5, 3), (6, 12), (7, 111), (11, 3)),
        ((1, 25), (2, 75), (7, 5), (10, 6), (12, 89), (15, 4)), ((6, 20), (7, 125), (11, 5), (14, 12), (15, 40), (19, 3)),
        ((2, 6), (3, 114), (5, 3), (6, 12), (7, 9), (11, 3)), ((3, 8), (5, 93), (9, 4), (10, 2), (13, 12), (16, 2))]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_a_member_halfway_between_the_centres_goes_to_the_first(dtype):
    """Centres of a round are rounded as a division rounds them: all values here are small whole numbers, every comparison is
    exact, and the tie goes to side A whatever path the cluster takes."""
    units = [(t, sign) for t in TIED for sign in (1, -1)]
    sizes = [[sum(n for _, n in t), 3] for t, _ in units]
    cap = max(sum(x) for x in sizes)
    gen = torch.Generator(device=DEV).manual_seed(41)
    st = snapshot(dtype, sizes, [1] * len(units), 8, cap, gen)
    for u, (t, sign) in enumerate(units):
        x = sign * torch.cat([torch.full((n,), float(v), device=DEV) for v, n in t])
        x = x[torch.randperm(len(x), generator=gen, device=DEV)]
        keys = torch.zeros(len(x), D, device=DEV)
        keys[:, 5] = x
        st["keys"][u, st["members"][u, :len(x)].long()] = keys.to(st["keys"].dtype)
    s = WorkloadSpec("tied", dtype, len(units), 2, cap, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=0, seed=41)
    ix, o = make_pair(s, len(units), max_tokens=cap, max_clusters=8)
    ix.dynakv_import_state(st)
    tally = Tally()
    parity.resync(ix, o, None, set(range(len(units))), tally)
    ix.dynakv_split()
    o.split()
    assert not compare_state(ix, o, tally, "tied", assign=False)
    assert ix.dynakv_export_state(["n_clusters"])["n_clusters"].tolist() == [3] * len(units)


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_splits_of_several_clusters_at_once(dtype):
    """Plans that mix sizes: four small ones side by side, wide ones two at a time, one that takes the whole workgroup before,
    between and after them, one beyond the staging rows among them, more than one round of each."""
    sizes = [[9, 12, 30, 4, 8, 20, 3], [100, 50, 40, 9, 60], [10, 200, 12, 8], [180, 10, 150, 90, 70, 60], [20, 300, 40],
             [2, 2, 2, 2, 2, 2, 2, 2, 2, 130], [6] * 70]
    flagged = [6, 4, 3, 6, 3, 10, 66]
    ix, o, tally, _ = pair(dtype, sizes, flagged, 160)
    ix.dynakv_split()
    o.split()
    dirty = compare_state(ix, o, tally, "split", assign=False)
    print("several splits", dtype, dict(tally), flush=True)
    assert not dirty
    assert not ix.dynakv_export_state(["flag"])["flag"].any()


@pytest.mark.parametrize("dtype,M,n,Mcap", [
    ("f16", 1, 1, 8), ("bf16", 60, 15, 200), ("f16", 60, 16, 200), ("f16", 60, 33, 200), ("bf16", 640, 20, 900), ("f16", 641, 20, 900),
    ("bf16", 1281, 20, 1500), ("f16", 2561, 12, 2700), ("bf16", 5121, 6, 5300), ("f16", 10234, 8, 10300), ("bf16", 10240, 5, 10300),
    ("f16", 10218, 8, 10300), ("f16", 10221, 8, 10300), ("f16", 5096, 12, 5300), ("bf16", 5100, 9, 5300), ("f16", 5101, 9, 5300),
    ("bf16", 70, 2, 200), ("f16", 70, 3, 200), ("f32", 70, 20, 200), ("f16", 3, 70, 90), ("bf16", 600, 90, 900)])
def test_extension_across_batches(dtype, M, n, Mcap):
    """dynakv_extend_index against the oracle where its batches change size (620, 1260, .. clusters) or end: one entry, two, three, one batch,
    a remainder, a split inside a batch, entries that follow one another into one cluster, the last cluster that a batch can hold
    and the first that it cannot."""
    U = 2
    sizes = [[1 + (j * 7 + u) % 3 for j in range(M)] for u in range(U)]
    # (tau: about what the clusters' own entries give, so that some of the new entries flag theirs)
    ix, o, tally, gen = pair(dtype, sizes, [0] * U, Mcap, extra=n, tau=7.0)
    st = ix.dynakv_export_state(["keys"], to_cpu=False)["keys"].float()
    pick = torch.randint(0, min(M, 12), (U, n), generator=gen, device=DEV)      # few clusters: most entries meet one that has just changed
    K = torch.gather(st, 1, pick[:, :, None].expand(-1, -1, D)) + 0.25 * torch.randn(U, n, D, generator=gen, device=DEV)
    K[:, ::5] += 0.3 * torch.randn(U, (n + 4) // 5, D, generator=gen, device=DEV)
    K = K.to(binding.TORCH_DTYPES[dtype])
    V = torch.randn(U, n, D, generator=gen, device=DEV).to(K.dtype)
    ix.dynakv_extend_index(K.contiguous(), V.contiguous())
    o.extend(K.float().cpu().numpy(), V.float().cpu().numpy())
    dirty = compare_state(ix, o, tally, "extension", assign=False)
    out = ix.dynakv_export_state(["n_clusters", "n_tokens", "error"])
    print("extension", dtype, M, n, out["n_clusters"].tolist(), dict(tally), flush=True)
    assert not dirty and not out["error"].any()
    if n >= 20:
        assert int(out["n_clusters"].min()) > M

@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
def test_extension_of_an_index_that_holds_flagged_clusters(dtype):
    """Flagged clusters from before the call (a snapshot's; none, one, two and one that cannot be split) are split along with the
    first entry, which goes elsewhere; the entries that follow in the same batch go to them."""
    n = 40
    sizes = [[40, 30, 9, 12, 6, 20, 3, 11]] * 5
    flagged = [1, 2, 1, 0, 2]
    gen = torch.Generator(device=DEV).manual_seed(17)
    cap = sum(sizes[0]) + n
    s = WorkloadSpec("flagged", dtype, 5, 2, cap, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=16, seed=17)
    ix, o = make_pair(s, 5, max_tokens=cap, max_clusters=100)
    st = snapshot(dtype, sizes, flagged, 100, cap, gen, 0.0, 9.0)
    off, mem = st["offsets"], st["members"].long()
    st["keys"][2, mem[2, :40]] = st["keys"][2, mem[2, :1]]           # unit 2: all entries equal, statistics that are not theirs
    ix.dynakv_import_state(st)
    tally = Tally()
    parity.resync(ix, o, None, set(range(5)), tally)
    K = torch.empty(5, n, D, device=DEV)
    for u in range(5):
        for t in range(n):
            j = (4, 0, 0, 1, 0, 2, 1, 0)[t % 8]
            at = int(off[u, j]) + (5 * t) % sizes[u][j]
            K[u, t] = st["keys"][u, mem[u, at]].float() + 0.15 * torch.randn(D, generator=gen, device=DEV)
    K = K.to(binding.TORCH_DTYPES[dtype])
    V = torch.randn(5, n, D, generator=gen, device=DEV).to(K.dtype)
    ix.dynakv_extend_index(K.contiguous(), V)
    o.extend(K.float().cpu().numpy(), V.float().cpu().numpy())
    assert not compare_state(ix, o, tally, "extension", assign=False)
    e = ix.dynakv_export_state(["n_clusters", "flag", "error", "keys", "values"])
    print("flagged before the extension", dtype, e["n_clusters"].tolist(), dict(tally), flush=True)
    assert not e["flag"].any() and not e["error"].any()
    N = sum(sizes[0])
    assert torch.equal(e["keys"][:, N:], K.cpu()) and torch.equal(e["values"][:, N:], V.cpu())
    Q = (K[:, :2].float() + 0.1 * torch.randn(5, 2, D, generator=gen, device=DEV)).to(K.dtype).contiguous()
    out, lse = torch.empty(5, 2, D, device=DEV), torch.empty(5, 2, device=DEV)
    for budget in (50, 1000):
        ix.dynakv_retrieve_attend(Q, budget, out, lse)
        oo, ol = o.retrieve_attend(Q.float().cpu().numpy(), budget)
        assert not parity.compare_retrieval(ix, o, tally, "after it", Q=Q.float().cpu().numpy(), budget=budget)
        parity.check_attention(out.cpu().numpy(), lse.cpu().numpy(), oo, ol, "after it")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_extension_takes_entries_that_are_not_finite_as_an_append_does(dtype, bad):
    """Such an entry is at no finite distance from any cluster: it goes to the lowest id, in a chunk as in an append."""
    sizes, n = [[6, 5, 7, 4, 6, 5, 3, 4]] * 2, 12
    cap = sum(sizes[0]) + n
    gen = torch.Generator(device=DEV).manual_seed(31)
    st = snapshot(dtype, sizes, [0, 0], 40, cap, gen, 0.0, 9.0)
    K = (st["keys"][:, :n].float() + 0.1 * torch.randn(2, n, D, generator=gen, device=DEV)).to(binding.TORCH_DTYPES[dtype])
    K[:, 3, 17] = bad
    V = torch.randn(2, n, D, generator=gen, device=DEV).to(K.dtype)
    s = WorkloadSpec("bad", dtype, 2, 2, cap, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=0, seed=31)
    a, b = (make_pair(s, 2, max_tokens=cap, max_clusters=40)[0] for _ in range(2))
    for ix in (a, b):
        ix.dynakv_import_state(st)
    a.dynakv_extend_index(K.contiguous(), V)
    for t in range(n):
        b.dynakv_append(K[:, t].contiguous(), V[:, t].contiguous())
        b.dynakv_split()
    ea, eb = (ix.dynakv_export_state(["n_clusters", "size", "offsets", "members", "error"]) for ix in (a, b))
    for k in ea:
        assert torch.equal(ea[k], eb[k]), k
    for u in range(2):
        off, mem = ea["offsets"][u], ea["members"][u]
        assert sum(sizes[0]) + 3 in mem[off[0]:off[1]].tolist()


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_extension_after_decode_steps_that_leave_flags(dtype):
    """A chunk after decode steps whose delayed splits are still due."""
    s = CONFIGS["llama3_8b"].scaled(dtype=dtype, prefill=1024, n_clusters_init=48, budget=120, var_alpha=1.1, drift_std=0.1, buffer_max=40)
    U, steps, n = 4, 96, 64
    w = generate(s, units=range(U), steps=steps + n)
    ix, o = make_pair(s, U, max_tokens=1024 + steps + n, kmeans_iters=4)
    ix.dynakv_build_index(to_dev(w["K0"], dtype), to_dev(w["V0"], dtype), torch.from_numpy(w["init_idx"]).to(DEV))
    o.build_index(w["K0"], w["V0"], w["init_idx"])
    sp = parity.Stepper(ix, o, s, w)
    compare_build(ix, o, sp.tally, 1024)
    for t in range(steps):
        sp.step(t, True, attention=False, full=t == steps - 1)
    left = ix.dynakv_export_state(["flag"])["flag"].sum(1).tolist()
    K1, V1 = (np.ascontiguousarray(w[k][steps:].transpose(1, 0, 2)) for k in ("Knew", "Vnew"))
    ix.dynakv_extend_index(to_dev(K1, dtype), to_dev(V1, dtype))
    o.extend(K1, V1)
    assert not compare_state(ix, o, sp.tally, "extension", assign=False)
    e = ix.dynakv_export_state(["flag", "error"])
    print("extension after steps", dtype, left, dict(sp.tally), flush=True)
    assert min(left) >= 1 and not e["flag"].any() and not e["error"].any()


def workgroups_per_unit(dtype, units, budget, capacity, step):
    """What the single kernel takes (launch_retrieve_fused)."""
    f32, most = dtype == "f32", 8 if units <= 32 else 4 if units <= 64 else 2 if units <= 128 else 1
    kib = min(budget, capacity) * (1 if f32 else 0.5)
    worth = 256 if units <= 16 or f32 else 768 if step else 256 if units <= 64 else 512
    n = 2 if f32 and units <= 8 and kib >= worth else 1
    while n < most and kib >= 2 * worth * n:
        n *= 2
    return n


@pytest.mark.parametrize("dtype,units,G,budgets,retrievals,steps", [
    ("f16", 3, 4, (300, 1030, 2060, 4200, 1 << 20), [1, 2, 4, 8, 8], [1, 2, 4, 8, 8]),
    ("bf16", 40, 7, (300, 1030, 2060, 3100, 1 << 20), [1, 2, 4, 4, 4], [1, 1, 1, 2, 4]),
    ("bf16", 100, 3, (300, 2060, 3100), [1, 2, 2], [1, 1, 2]),
    ("f32", 2, 5, (200, 300, 1030, 2060, 1 << 20), [1, 2, 4, 8, 8], [1, 2, 4, 8, 8]),
    ("f32", 20, 4, (300, 600, 1030, 2060), [1, 2, 4, 8], [1, 2, 4, 8])])
@pytest.mark.parametrize("buffer_max", [0, 6])
def test_units_shared_by_several_workgroups(dtype, units, G, budgets, retrievals, steps, buffer_max):
    """Budgets at which the single kernel takes one, two, four and eight workgroups per unit, in retrievals and whole steps in turn
    (its arrival counters go on from launch to launch), with more than four splits due in one step, whose later rounds want the
    pages that the first has freed, and (buffer_max > 0) a forced split after the delayed ones."""
    sizes = [[9, 12, 30, 4, 8, 20, 3, 60, 100] + [1 + (j * 5 + u) % 47 for j in range(262)] for u in range(units)]
    flagged = [9] * units
    cap = max(sum(x) for x in sizes) + 2 * len(budgets)
    for want, step in ((retrievals, False), (steps, True)):
        assert [workgroups_per_unit(dtype, units, b, cap, step) for b in budgets] == want
    gen = torch.Generator(device=DEV).manual_seed(3)
    s = WorkloadSpec("share", dtype, units, G, cap, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=buffer_max, seed=5)
    ix, o = make_pair(s, units, max_tokens=cap, max_clusters=400)
    st = snapshot(dtype, sizes, flagged, 400, cap, gen, 0.0, 9.0)
    ix.dynakv_import_state(st)
    tally = Tally()
    parity.resync(ix, o, None, set(range(units)), tally)
    keys, dt = st["keys"].float(), st["keys"].dtype
    out, lse = torch.empty(units, G, D, device=DEV), torch.empty(units, G, device=DEV)
    for t, budget in enumerate(b for b in budgets for _ in range(3)):
        Q = (keys[:, 11 * t + 3, None] + 0.5 * torch.randn(units, G, D, generator=gen, device=DEV)).to(dt).contiguous()
        k = (keys[:, 7 * t + 1] + 0.2 * torch.randn(units, D, generator=gen, device=DEV)).to(dt).contiguous()
        v = torch.randn(units, D, generator=gen, device=DEV).to(dt)
        Qn, what = Q.float().cpu().numpy(), "call %d, budget %d" % (t, budget)
        oo, ol = o.retrieve_attend(Qn, budget)
        if t % 3 == 1:
            ix.dynakv_retrieve_attend(Q, budget, out, lse)
            assert not parity.compare_retrieval(ix, o, tally, what, Q=Qn, budget=budget)
        else:
            ix.dynakv_decode_step(Q, budget, out, lse, k, v)
            o.append(k.float().cpu().numpy(), v.float().cpu().numpy())
            o.split()
            assert not compare_state(ix, o, tally, what)
        parity.check_attention(out.cpu().numpy(), lse.cpu().numpy(), oo, ol, what)
    forced = int(ix.dynakv_export_state(["counters"])["counters"][:, 2].sum())
    print("shared units", dtype, units, buffer_max, forced, dict(tally), flush=True)
    assert (forced > 0) == (buffer_max > 0)


@pytest.mark.parametrize("dtype,G", [("f16", 4), ("bf16", 7), ("f32", 5)])
def test_a_given_number_of_workgroups_per_unit_is_kept(dtype, G):
    """launch_shape(1) is one workgroup per unit in the single kernel too: retrievals of 8 units add up in the order, and give the
    bits, of the same units among 136, which never share; left to the library, the 8 units are shared and the order is another."""
    few = 8
    sizes = [[1 + (j * 5 + u % few) % 23 for j in range(200)] for u in range(136)]
    cap = max(sum(x) for x in sizes)
    gen = torch.Generator(device=DEV).manual_seed(51)
    st = snapshot(dtype, sizes[:few], [0] * few, 300, cap, gen, 0.0, 9.0)
    Q = (st["keys"][:, 7:8].float() + 0.5 * torch.randn(few, G, D, generator=gen, device=DEV)).to(st["keys"].dtype)
    outs, room = {}, {}
    for name, U, launch in (("one", few, launch_shape(1)), ("many", 136, 0), ("free", few, 0)):
        s = WorkloadSpec("kept", dtype, U, G, cap, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=0, seed=51)
        ix = make_pair(s, U, max_tokens=cap, max_clusters=300, launch=launch, oracle_units=1)[0]
        reps = U // few
        ix.dynakv_import_state({k: x.repeat(reps, *[1] * (x.dim() - 1)).contiguous() for k, x in st.items()})
        out, lse = torch.empty(U, G, D, device=DEV), torch.empty(U, G, device=DEV)
        ix.dynakv_retrieve_attend(Q.repeat(reps, 1, 1).contiguous(), 2200, out, lse)
        outs[name], room[name] = (out[:few].cpu(), lse[:few].cpu()), ix.workspace.numel()
    assert all(torch.equal(a, b) for a, b in zip(outs["one"], outs["many"]))
    assert not torch.equal(outs["one"][0], outs["free"][0])
    assert torch.allclose(outs["one"][0], outs["free"][0], rtol=1e-4, atol=1e-5) and room["one"] < room["free"]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_decisions_retaken_are_counted_once_per_unit(dtype):
    """Counter 7 of the exported state where every new entry lies as far from one cluster as from its copy: the same number of
    decisions with one workgroup per unit, several, and separate kernels."""
    sizes = [[1 + (j * 5) % 23 for j in range(200)]] * 3
    cap = sum(sizes[0]) + 8
    gen = torch.Generator(device=DEV).manual_seed(61)
    st = snapshot(dtype, sizes, [0] * 3, 300, cap, gen, 0.0, 1e9)
    off, mem = st["offsets"], st["members"].long()
    st["centroids"][:, 1:200:2] = st["centroids"][:, 0:200:2]
    counts = {}
    for launch in (launch_shape(1), 0, LAUNCH_SEPARATE):
        s = WorkloadSpec("counted", dtype, 3, 2, cap, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=0, seed=61)
        ix = make_pair(s, 3, max_tokens=cap, max_clusters=300, launch=launch)[0]
        ix.dynakv_import_state(st)
        out, lse = torch.empty(3, 2, D, device=DEV), torch.empty(3, 2, device=DEV)
        for t in range(8):
            k = torch.stack([st["keys"][u, mem[u, int(off[u, 20 * t + 4])]] for u in range(3)]).contiguous()
            Q = (k[:, None].float() + 0.5 * torch.randn(3, 2, D, generator=torch.Generator(device=DEV).manual_seed(t), device=DEV)).to(k.dtype)
            ix.dynakv_decode_step(Q.contiguous(), 2200, out, lse, k, k)
        counts[launch] = ix.dynakv_export_state(["counters"])["counters"][:, 4:].tolist()
    print("retaken", dtype, counts, flush=True)
    assert counts[0] == counts[launch_shape(1)] == counts[LAUNCH_SEPARATE]
    assert all(c[3] >= 8 for c in counts[0])

@pytest.mark.parametrize("units,budget", [(1, 256), (1, 2100), (5, 600), (40, 700), (130, 300)])
def test_float32_steps_repeat_bit_for_bit(units, budget):
    """Whole steps of float32 storage add up in the same order every time, however many workgroups share a unit, whichever of them has the
    append, and with splits due or not."""
    sizes = [[9, 12, 30, 4, 8, 20, 3, 60, 40] + [1 + (j * 5 + u) % 23 for j in range(180)] for u in range(units)]
    flagged = [u % 7 for u in range(units)]
    cap = max(sum(x) for x in sizes) + 8
    gen = torch.Generator(device=DEV).manual_seed(81)
    st = snapshot("f32", sizes, flagged, 400, cap, gen, 0.0, 9.0)
    Q = [(st["keys"][:, 7 * t + 3, None] + 0.5 * torch.randn(units, 4, D, generator=gen, device=DEV)).contiguous() for t in range(8)]
    k = [(st["keys"][:, 5 * t + 1] + 0.2 * torch.randn(units, D, generator=gen, device=DEV)).contiguous() for t in range(8)]
    s = WorkloadSpec("repeat", "f32", units, 4, cap, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=0, seed=81)
    ix = make_pair(s, units, max_tokens=cap, max_clusters=400, oracle_units=1)[0]
    first = None
    for _ in range(6):
        ix.dynakv_import_state(st)
        out, lse = torch.empty(8, units, 4, D, device=DEV), torch.empty(8, units, 4, device=DEV)
        for t in range(8):
            ix.dynakv_decode_step(Q[t], budget, out[t], lse[t], k[t], k[t])
        e = ix.dynakv_export_state(["n_clusters", "members", "offsets", "centroids", "m2", "error"])
        got = (out.cpu(), lse.cpu(), *e.values())
        assert not e["error"].any()
        first = first or got
        assert all(torch.equal(a, b) for a, b in zip(first, got))


def test_extension_decides_ties_between_coinciding_clusters():
    """Every entry lies near two clusters of the same entries, and the splits that follow one another raise the norms that the
    error bounds are made of: the lowest id wins each tie, in every lane."""
    gen = torch.Generator(device=DEV).manual_seed(9)
    sizes, n = [[4, 4, 3, 3, 2, 2, 5, 5]] * 2, 48
    s = WorkloadSpec("ties", "f16", 2, 2, 28, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, buffer_max=0, seed=9)
    ix, o = make_pair(s, 2, max_tokens=28 + n, max_clusters=120)
    st = snapshot("f16", sizes, [0, 0], 120, 28 + n, gen, 0.0, 6.0)
    for u in range(2):                                  # clusters 2k + 1 are copies of clusters 2k
        off, mem = st["offsets"][u], st["members"][u].long()
        for j in range(0, 8, 2):
            a, b = mem[off[j]:off[j + 1]], mem[off[j + 1]:off[j + 2]]
            st["keys"][u, b] = st["keys"][u, a]
            st["centroids"][u, j + 1] = st["centroids"][u, j]
            st["m2"][u, j + 1] = st["m2"][u, j]
    ix.dynakv_import_state(st)
    tally = Tally()
    parity.resync(ix, o, None, {0, 1}, tally)
    grow = 1.0 + 0.04 * torch.arange(n, device=DEV)[None, :, None]
    K = (st["keys"][:, torch.arange(n, device=DEV) % 28].float() * grow + 0.1 * torch.randn(2, n, D, generator=gen, device=DEV)).half()
    V = torch.randn(2, n, D, generator=gen, device=DEV).half()
    ix.dynakv_extend_index(K.contiguous(), V)
    o.extend(K.float().cpu().numpy(), V.float().cpu().numpy())
    assert not compare_state(ix, o, tally, "ties", assign=False)
    assert int(ix.dynakv_export_state(["n_clusters"])["n_clusters"].min()) > 12


@pytest.mark.parametrize("clusters,copies", [(700, 0), (700, 2), (20, 20), (17000, 0)])
def test_snapshot_lists_a_long_selection_by_score(clusters, copies):
    """Where more than 16384 clusters are possible a snapshot lists the last selection by descending score, the lowest id first
    among equals, and the entries in that order, whichever order the retrieval has attended them in (copies of a cluster have
    equal scores: a cut among them is left to the selection on the scores in memory)."""
    gen = torch.Generator(device=DEV).manual_seed(clusters + copies)
    sizes = [[1 + (7 * j) % 3 if clusters < 5000 else 1 for j in range(clusters)]] * 2
    N = sum(sizes[0])
    s = WorkloadSpec("listing", "f16", 2, 2, N, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, seed=9)
    ix, o = make_pair(s, 2, max_tokens=N, max_clusters=17100)
    st = snapshot("f16", sizes, [0, 0], 17100, N, gen, 0.0, 6.0)
    for j in range(1, copies):
        st["centroids"][:, j] = st["centroids"][:, 0]
    ix.dynakv_import_state(st)
    out, lse = torch.empty(2, 2, D, device=DEV), torch.empty(2, 2, device=DEV)
    Q = (st["centroids"][:, :1] + 0.5 * torch.randn(2, 2, D, generator=gen, device=DEV)).half().contiguous()
    for budget in (1, 2, 30, 333, min(N // 2, 4000)):
        ix.dynakv_retrieve_attend(Q, budget, out, lse)
        e = ix.dynakv_export_state(["n_selected", "selected", "n_gathered", "gathered", "scores", "offsets", "members", "error"])
        assert not e["error"].any()
        for u in range(2):
            ids, score = e["selected"][u, :e["n_selected"][u]].long(), e["scores"][u]
            assert ids.tolist() == sorted(ids.tolist(), key=lambda j: (-float(score[j]), j)), budget
            off, mem = e["offsets"][u].tolist(), e["members"][u]
            want = torch.cat([mem[off[j]:off[j + 1]] for j in ids.tolist()])[:budget]
            assert int(e["n_gathered"][u]) == len(want) and torch.equal(e["gathered"][u, :len(want)], want), budget


def test_a_refused_import_leaves_the_listing_as_it_was():
    """A unit that an import refuses keeps its state, the list of its last retrieval among it."""
    gen = torch.Generator(device=DEV).manual_seed(91)
    sizes = [[1 + (7 * j + u) % 5 for j in range(500)] for u in range(2)]
    N = max(sum(x) for x in sizes)
    s = WorkloadSpec("kept", "f16", 2, 2, N, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, seed=91)
    ix = make_pair(s, 2, max_tokens=N, max_clusters=17100)[0]
    st = snapshot("f16", sizes, [0, 0], 17100, N, gen, 0.0, 6.0)
    ix.dynakv_import_state(st)
    out, lse = torch.empty(2, 2, D, device=DEV), torch.empty(2, 2, device=DEV)
    Q = (st["centroids"][:, :1] + 0.5 * torch.randn(2, 2, D, generator=gen, device=DEV)).half().contiguous()
    ix.dynakv_retrieve_attend(Q, 700, out, lse)
    fields = ["n_selected", "selected", "n_gathered", "gathered", "size", "members", "centroids"]
    before = ix.dynakv_export_state(fields)
    bad = {k: x.clone() for k, x in st.items()}
    bad["size"][:, 499] += 1                             # the last cluster says one entry more than it has
    ix.dynakv_import_state(bad)
    after = ix.dynakv_export_state(fields + ["error"])
    assert after["error"].tolist() == [binding.ERR_IMPORT] * 2 and int(before["n_gathered"].min()) > 600
    for u in range(2):
        g = int(before["n_gathered"][u])
        assert torch.equal(before["gathered"][u, :g], after["gathered"][u, :g])
    for k in fields:
        if k != "gathered":
            assert torch.equal(before[k], after[k]), k


@pytest.mark.parametrize("budget", [4096, 4097, 6000, 9000])
def test_a_selection_of_more_than_4096_clusters_is_cut_short(budget):
    """Where more than 16384 clusters are possible at most 4096 can be selected: clusters of one entry each, all of them within the budget by score,
    and the error word where there would have been more."""
    gen = torch.Generator(device=DEV).manual_seed(budget)
    M = 17000
    s = WorkloadSpec("cut", "f16", 2, 2, M, 1, 1, 64, 6, 0.05, var_alpha=1.5, size_factor=0.0, seed=9)
    ix = make_pair(s, 2, max_tokens=M, max_clusters=17100, oracle_units=1)[0]
    st = snapshot("f16", [[1] * M] * 2, [0, 0], 17100, M, gen, 0.0, 6.0)
    ix.dynakv_import_state(st)
    out, lse = torch.empty(2, 2, D, device=DEV), torch.empty(2, 2, device=DEV)
    Q = (st["centroids"][:, :1] + 0.5 * torch.randn(2, 2, D, generator=gen, device=DEV)).half().contiguous()
    ix.dynakv_retrieve_attend(Q, budget, out, lse)
    e = ix.dynakv_export_state(["n_selected", "selected", "n_gathered", "gathered", "scores", "offsets", "members", "error"])
    assert e["error"].tolist() == [binding.ERR_SELECT if budget > 4096 else 0] * 2 and bool(torch.isfinite(out).all())
    for u in range(2):
        ids, score = e["selected"][u, :4096].long(), e["scores"][u, :M]
        assert e["n_selected"][u] == 4096 and e["n_gathered"][u] == 4096 and len(set(ids.tolist())) == 4096
        assert ids.tolist() == sorted(ids.tolist(), key=lambda j: (-float(score[j]), j))
        assert bool((score[ids] >= score.sort(descending=True).values[budget - 1] - 1e-4).all())
        mem, off = e["members"][u], e["offsets"][u].long()
        assert torch.equal(e["gathered"][u, :4096], mem[off[ids]])
