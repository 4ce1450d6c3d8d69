"""The calls that users of this package make, as cases to be timed.

A case is one pass of one of six kinds, on the drifting Gaussian mixture of paper_2511_07427_amd/workload.py drawn on
the GPU:

  prefill   dynakv_build_index on a prompt: the latency before the first token
  request   dynakv_build_index, then `steps` whole decode steps: one batch of requests from its prompt to its answer
  resume    dynakv_import_state of a session's snapshot, then `steps` whole decode steps: the next turn of a long session
            whose `tokens` entries drift has cut into many clusters
  chunked   dynakv_build_index on the first `tokens` entries of a prompt, dynakv_extend_index with the next `steps`
  retrieve  dynakv_retrieve_attend alone on a standing index: a query that adds nothing to the cache
  calls     dynakv_import_state, then `steps` times dynakv_retrieve_attend, dynakv_append and dynakv_split one by one: a
            program that puts work of its own between them

Every pass begins from the same prompt or snapshot and can be repeated.  Passes that change the index end with
dynakv_export_state: that is where the library reports a unit's error word, and it returns what the pass has made of the
index.
"""
import math

import torch

from paper_2511_07427_amd import binding

D = 128                                  # head_dim, the one the library takes
COMP_STD, QUERY_NOISE, OUTLIERS, OUTLIER_SCALE = 0.3, 0.5, 4, 8.0
KMEANS_ITERS, BUFFER_MAX, VAR_ALPHA = 10, 16, 1.5


def _case(name, kind, dtype, units, group, tokens, clusters, budget, steps, drift=0.02, max_clusters=0, size_factor=0.0):
    return dict(name=name, kind=kind, dtype=dtype, units=units, group=group, tokens=tokens, clusters=clusters, budget=budget,
                steps=steps, drift=drift, max_clusters=max_clusters or 16 * clusters, size_factor=size_factor)


def listed():
    return [
        # the smallest call: one retrieval over the smallest configuration's cache (float32, one unit)
        _case("retrieve_tiny_f32", "retrieve", "f32", 1, 4, 2048, 32, 256, 0, max_clusters=128, size_factor=2.0),
        # that configuration from prompt to answer: everything waits on launches and on dependent steps
        _case("request_tiny_f32", "request", "f32", 1, 4, 2048, 32, 256, 256, max_clusters=128, size_factor=2.0),
        # a small ragged batch driven call by call
        _case("calls_ragged_bf16", "calls", "bf16", 13, 5, 3001, 211, 777, 32, max_clusters=1024),
        # the prompt of the benchmark's workload: 32 layers x 8 KV heads
        _case("prefill_llama3", "prefill", "f16", 256, 4, 4096, 256, 1024, 0),
        # the same prompt and the first 256 tokens of its answer
        _case("request_llama3", "request", "f16", 256, 4, 4096, 256, 1024, 256),
        # and a turn late in the same session, when drift has made about eight times the clusters
        _case("resume_llama3", "resume", "f16", 256, 4, 12000, 1900, 1024, 128, max_clusters=4096),
        # 28 layers x 4 KV heads, seven query heads each, twice the budget: fewer units than compute units
        _case("request_qwen25_bf16", "request", "bf16", 112, 7, 2048, 128, 2048, 256, drift=0.05),
        # batched serving: long prompts
        _case("prefill_batched16", "prefill", "f16", 128, 4, 8192, 512, 2048, 0, max_clusters=4096),
        # and late in their sessions, with more clusters than one kernel launch per step takes
        _case("resume_batched16", "resume", "f16", 128, 4, 32000, 7300, 2048, 64, max_clusters=10240),
        # the longest context: few units with very many clusters
        _case("resume_long131k_bf16", "resume", "bf16", 8, 8, 131000, 50000, 4096, 64, drift=0.1, max_clusters=65536),
        # the longest prompt that is clustered at once, on as few units
        _case("prefill_long_bf16", "prefill", "bf16", 8, 8, 16384, 2048, 4096, 0, max_clusters=8192),
        # a prompt that arrives in chunks
        _case("chunked_llama3", "chunked", "f16", 256, 4, 2048, 256, 1024, 1024),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["prefill", "request", "resume", "resume", "chunked", "retrieve", "calls"])
    dtype = rng.choice(["f16", "f16", "bf16"])
    units = rng.choice([_log(rng, 1, 256), rng.randint(96, 256)])
    group = rng.randint(1, 8)
    if kind in ("resume", "calls", "retrieve"):
        # about four to sixteen entries per cluster, as long sessions end up; bounded by the largest listed snapshot
        tokens = _log(rng, 1500, min(131000, 4096000 // units))
        clusters = max(16, int(tokens / rng.uniform(4, 16)))
        max_clusters = clusters + int(0.3 * clusters) + rng.randint(512, 1280)
    else:
        tokens = _log(rng, 700, min(16384, 1048576 // units) if units < 256 else 4096)
        clusters = max(8, int(tokens / rng.uniform(8, 32)))
        max_clusters = 8 * clusters
    budget = min(tokens, _log(rng, 128, 4096))
    steps = {"prefill": 0, "retrieve": 0, "calls": rng.randint(8, 48), "chunked": _log(rng, 64, 1024)}.get(kind) if kind not in (
        "request", "resume") else rng.randint(24, 160 if kind == "request" else 64)
    if kind in ("request", "retrieve", "prefill") and rng.random() < 0.2:
        # float32 storage: small caches
        dtype, units, tokens = "f32", rng.randint(1, 4), _log(rng, 512, 2048)
        clusters = max(8, int(tokens / rng.uniform(32, 64)))
        max_clusters, budget = 8 * clusters + 32, min(budget, tokens)
    case = _case("", kind, dtype, units, group, tokens, clusters, budget, steps, drift=rng.choice([0.02, 0.05]), max_clusters=max_clusters)
    del case["name"]
    return case


# ---------------------------------------------------------------------------------------------- inputs
def _components(case):
    return max(4, min(64, case["clusters"] // 2))


def _mixture(case, gen, n0, n1):
    """Keys and values [U, n0 + n1, D] (float32) of a mixture whose component means stand still for the first n0 entries
    and then walk, a few key channels scaled up; the component of every entry [U, n0 + n1]."""
    dev, U, n = "cuda", case["units"], n0 + n1
    rnd = lambda *s: torch.randn(*s, generator=gen, device=dev)  # noqa: E731
    P = _components(case)
    mu, nu = rnd(U, P, D), rnd(U, P, D)
    chan = torch.ones(U, D, device=dev)
    chan.scatter_(1, torch.rand(U, D, generator=gen, device=dev).topk(OUTLIERS, 1).indices, OUTLIER_SCALE)
    comp = torch.randint(0, P, (U, n), generator=gen, device=dev)
    K = torch.empty(U, n, D, device=dev)
    V = torch.empty(U, n, D, device=dev)
    for u0 in range(0, U, 16):                         # some units at a time: the walk's scratch stays small
        s = slice(u0, min(U, u0 + 16))
        c = comp[s]
        mean = torch.gather(mu[s], 1, c[:, :, None].expand(-1, -1, D))
        if n1:
            # a component's mean is needed only where it is used: between two uses dt entries apart it moves by
            # drift * sqrt(dt) * N(0, I)
            order = torch.argsort(c[:, n0:], dim=1, stable=True)
            cs, t = torch.gather(c[:, n0:], 1, order), order.float() + 1.0
            first = torch.ones_like(cs, dtype=torch.bool)
            first[:, 1:] = cs[:, 1:] != cs[:, :-1]
            prev = torch.where(first, torch.zeros_like(t), torch.nn.functional.pad(t[:, :-1], (1, 0)))
            inc = (case["drift"] * (t - prev).sqrt())[:, :, None] * rnd(c.shape[0], n1, D)
            walk = inc.cumsum(1)
            start = torch.where(first, torch.arange(n1, device=dev)[None, :], torch.zeros_like(order)).cummax(1).values
            ix = start[:, :, None].expand(-1, -1, D)
            walk = walk - torch.gather(walk, 1, ix) + torch.gather(inc, 1, ix)
            mean[:, n0:].scatter_add_(1, order[:, :, None].expand(-1, -1, D), walk)
        K[s] = (mean + COMP_STD * rnd(*mean.shape)) * chan[s][:, None, :]
        V[s] = torch.gather(nu[s], 1, c[:, :, None].expand(-1, -1, D)) + COMP_STD * rnd(*mean.shape)
    return K, V, comp


def _queries(case, gen, K, n, steps):
    """[steps, U, G, D]: each a stored key (of the n + t that step t finds) plus noise per head, float32."""
    U = case["units"]
    t = torch.arange(steps, device="cuda")[:, None]
    pick = (torch.rand(steps, U, generator=gen, device="cuda") * (n + t)).long().clamp_max(K.shape[1] - 1)
    base = K[torch.arange(U, device="cuda")[None, :], pick]
    return base[:, :, None, :] + QUERY_NOISE * torch.randn(steps, U, case["group"], D, generator=gen, device="cuda")


def _snapshot(case, gen, K, V, comp, n, capacity):
    """A session's state after n entries, as dynakv_import_state takes it: the clusters are runs of entries of one
    component, neighbours in time, cut at random (what splitting leaves of a drifting component)."""
    U, M, Mcap, dev = case["units"], case["clusters"], case["max_clusters"], "cuda"
    n_clusters = torch.empty(U, dtype=torch.int32, device=dev)
    st = dict(n_clusters=n_clusters, n_tokens=torch.full((U,), n, dtype=torch.int32, device=dev),
              tau=torch.zeros(U, dtype=torch.float64, device=dev),
              centroids=torch.zeros(U, Mcap, D, device=dev), size=torch.zeros(U, Mcap, dtype=torch.int32, device=dev),
              buffered=torch.zeros(U, Mcap, dtype=torch.int32, device=dev), flag=torch.zeros(U, Mcap, dtype=torch.int32, device=dev),
              m2=torch.zeros(U, Mcap, dtype=torch.float64, device=dev),
              offsets=torch.full((U, Mcap + 1), n, dtype=torch.int32, device=dev),
              members=torch.zeros(U, capacity, dtype=torch.int32, device=dev),
              keys=torch.zeros(U, capacity, D, dtype=K.dtype, device=dev), values=torch.zeros(U, capacity, D, dtype=V.dtype, device=dev))
    st["keys"][:, :n], st["values"][:, :n] = K[:, :n], V[:, :n]
    for u in range(U):
        order = torch.argsort(comp[u, :n], stable=True)
        cs = comp[u, :n][order]
        cut = torch.zeros(n, dtype=torch.bool, device=dev)
        cut[0] = True
        cut[1:] = cs[1:] != cs[:-1]
        cut |= torch.rand(n, generator=gen, device=dev) < (M - _components(case)) / n
        label = (cut.cumsum(0) - 1).clamp_max(Mcap - Mcap // 8 - 1)       # about M clusters; room for a turn's splits
        count = int(label[-1]) + 1
        label = torch.randperm(count, generator=gen, device=dev)[label]   # ids carry no order of their own in a long session
        by = torch.argsort(label, stable=True)
        order, label = order[by], label[by]
        sz = torch.zeros(Mcap, dtype=torch.int64, device=dev).scatter_add_(0, label, torch.ones_like(label))
        keys = K[u, :n].double()[order]
        mean = torch.zeros(Mcap, D, dtype=torch.float64, device=dev).index_add_(0, label, keys) / sz.clamp_min(1)[:, None]
        mean32 = mean.float()
        st["centroids"][u] = mean32
        st["size"][u] = sz.int()
        m2 = torch.zeros(Mcap, dtype=torch.float64, device=dev).index_add_(0, label, (keys - mean32.double()[label]).square().sum(1))
        st["m2"][u] = m2.float()                         # the same number whatever the order of the sum
        st["offsets"][u, 0] = 0
        st["offsets"][u, 1:] = sz.cumsum(0).int()
        st["members"][u, :n] = order.int()
        st["tau"][u] = VAR_ALPHA * (st["m2"][u].sum() / n).float().double()
        n_clusters[u] = count
    return st


def _config(case, capacity):
    # a session's prompt had about an eighth of the clusters
    M0 = max(1, case["clusters"] // 8) if case["kind"] in ("resume", "calls", "retrieve") else case["clusters"]
    return binding.Config(case["units"], case["group"], case["dtype"], M0, case["max_clusters"], capacity,
                          KMEANS_ITERS, BUFFER_MAX, 0, 0.0 if case["size_factor"] else VAR_ALPHA, case["size_factor"])


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    kind, U, G, n, T = case["kind"], case["units"], case["group"], case["tokens"], case["steps"]
    dt = binding.TORCH_DTYPES[case["dtype"]]
    session = kind in ("resume", "calls", "retrieve")
    # in a session most entries come after the prompt and have drifted
    K, V, comp = _mixture(case, gen, n // 3 if session else n, n - n // 3 + T if session else T)
    K, V = K.to(dt), V.to(dt)
    Q = _queries(case, gen, K, n, max(1, T) if kind != "chunked" else 1).to(dt)
    s = dict(case=case, index=binding.Index(_config(case, n + T)), Q=Q,
             out=torch.empty(Q.shape, dtype=torch.float32, device="cuda"),
             lse=torch.empty(Q.shape[:3], dtype=torch.float32, device="cuda"))
    if kind in ("resume", "calls"):
        s["snapshot"] = _snapshot(case, gen, K, V, comp, n, n + T)
    elif kind == "retrieve":                            # the standing index
        s["index"].dynakv_import_state(_snapshot(case, gen, K, V, comp, n, n + T))
        torch.cuda.synchronize()
    else:
        s["K0"], s["V0"] = K[:, :n].contiguous(), V[:, :n].contiguous()
        s["init"] = torch.rand(U, n, generator=gen, device="cuda").topk(case["clusters"], 1).indices.int().contiguous()
        if kind == "chunked":
            s["K1"], s["V1"] = K[:, n:].contiguous(), V[:, n:].contiguous()
    if T and kind != "chunked":
        s["Kn"], s["Vn"] = K[:, n:].transpose(0, 1).contiguous(), V[:, n:].transpose(0, 1).contiguous()
    return s


# ---------------------------------------------------------------------------------------------- one pass
# the partition, its statistics and the error words: the index as Algorithm 1 knows it, without keys and values
_STATE = ["n_clusters", "n_tokens", "error", "tau", "centroids", "size", "buffered", "flag", "m2", "offsets", "members"]


def run(s):
    case, ix, kind = s["case"], s["index"], s["case"]["kind"]
    budget, Q, out, lse = case["budget"], s["Q"], s["out"], s["lse"]
    if kind == "retrieve":
        ix.dynakv_retrieve_attend(Q[0], budget, out[0], lse[0])
        return {"out": out, "lse": lse}
    if kind in ("prefill", "chunked", "request"):
        ix.dynakv_build_index(s["K0"], s["V0"], s["init"])
    else:
        ix.dynakv_import_state(s["snapshot"])
    if kind == "chunked":
        ix.dynakv_extend_index(s["K1"], s["V1"])
    if kind in ("prefill", "chunked"):
        return ix.dynakv_export_state(_STATE, to_cpu=False)
    if kind == "calls":
        for t in range(case["steps"]):
            ix.dynakv_retrieve_attend(Q[t], budget, out[t], lse[t])
            ix.dynakv_append(s["Kn"][t], s["Vn"][t])
            ix.dynakv_split()
    else:
        # the loop of bench.py: raw addresses, the tensors were checked when they were made
        es, stream, step = Q.element_size(), torch.cuda.current_stream().cuda_stream, ix.decode_step_ptrs
        dq, dk, dl = Q.stride(0), s["Kn"].stride(0), lse.stride(0)
        q, o, l, k, v = (x.data_ptr() for x in (Q, out, lse, s["Kn"], s["Vn"]))
        for t in range(case["steps"]):
            step(q + t * dq * es, budget, o + t * dq * 4, l + t * dl * 4, k + t * dk * es, v + t * dk * es, stream)
    return {"out": out, "lse": lse, **ix.dynakv_export_state(_STATE + ["last_assign"], to_cpu=False)}


def work(case):
    """Each input read once and each output written once: a build reads the prompt and writes its pages (and evaluates every
    entry against every cluster in each iteration); a step reads the clusters' representatives and the entries that the
    budget admits; an import moves the snapshot's entries into pages."""
    U, G, n, M, T, B = (case[k] for k in ("units", "group", "tokens", "clusters", "steps", "budget"))
    e = 4 if case["dtype"] == "f32" else 2
    row = D * e
    b = f = 0.0
    if case["kind"] in ("prefill", "chunked", "request"):
        b += U * (2 * 2 * n * row + M * D * 4)
        f += 2.0 * U * n * M * D * KMEANS_ITERS
    elif case["kind"] in ("resume", "calls"):
        b += U * (2 * 2 * n * row + 2 * M * D * 4)
    if case["kind"] == "chunked":                       # an entry is compared with every cluster; representatives stay at hand
        b += U * T * 2 * 2 * row
        f += 2.0 * U * T * M * D
    elif case["kind"] != "prefill":
        steps = max(1, T)
        took = min(B, n)
        b += steps * U * (M * row + 2 * took * row + G * row + G * D * 4 + G * 4)
        f += steps * U * (2.0 * G * M * D + 4.0 * G * took * D)
        if T:
            b += T * U * 4 * row
            f += 2.0 * T * U * M * D
    return {"bytes": b, "flops": f}


def tolerance(case):
    """Partitions are decided in float64 and are whole numbers that do not change.  Attention (float32 sums over up to a few
    thousand entries of weights whose exponents reach 150): against a float64 attention over the same entries the
    relative error is 4e-7 to 7e-7 and the largest difference 2e-6 to 5e-6 of the root mean square, and two runs, whose
    tiles fall to other wavefronts, differ by up to 1.6e-7 and 5e-6; means, M2 and tau lie closer."""
    return {"rel": 3e-6, "max": 2e-5}
