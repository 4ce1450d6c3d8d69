"""GPU parity of splits over every way a cluster can be split and of the chunked prefill across its batches, from snapshots that
put each size at the edge where the next way begins."""
import os
import sys

import numpy as np
import pytest
import torch

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))

import parity  # noqa: E402
from parity import DEV, Tally, compare_state, make_pair  # noqa: E402
from paper_2511_07427_amd import binding  # noqa: E402
from paper_2511_07427_amd.workload import WorkloadSpec  # noqa: E402

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


SIZES = [2, 3, 5, 15, 16, 17, 32, 33, 63, 64, 65, 96, 97, 128, 129, 191, 192, 193, 255, 256, 257, 300]


@pytest.mark.parametrize("dtype", ["f16", "bf16", "f32"])
@pytest.mark.parametrize("offset", [0.0, 30.0])
def test_splits_at_the_edges_of_every_path(dtype, offset):
    """One flagged cluster per unit of every size at which another path begins (16, 32, 64, 128, 192 and 256 entries), also with
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
    ("f16", 10218, 8, 10300), ("f16", 10221, 8, 10300), ("f32", 70, 20, 200), ("f16", 3, 70, 90), ("bf16", 600, 90, 900)])
def test_extension_across_batches(dtype, M, n, Mcap):
    """dynakv_extend_index against the oracle where its batches change size (640, 1280, .. clusters) or end: one entry, one batch,
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
