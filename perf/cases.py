"""Performance cases of the expert-map matching path, through the public calls.

Five kinds of call make up a serving program of this framework:

* ``traj``  trajectory match and prefetch selection of a batch (one call);
* ``sem``   semantic match and prefetch selection of a batch (one call);
* ``step``  one incremental re-search pass, a call per observed layer;
* ``dedup`` insertion of a batch of finished iterations into a full store,
            then the prefetch sets of the entries as they now stand;
* ``plan``  selection, prefetch order and miss count of resident matches.

Stores and queries are drawn on the GPU the way ``synth`` draws them on the
host: expert maps are row softmaxes of clustered logits in the shapes of
Mixtral-8x7B (32 x 8), Qwen1.5-MoE (24 x 60) and Phi-3.5-MoE (32 x 16),
trajectory queries are perturbed stored maps, embeddings are unit vectors
around cluster centroids.
"""
from __future__ import annotations

import math

import torch

import paper_2502_05370_amd as fm

# model -> layers, experts, map clusters, logit noise, experts activated per
# token, fixed threshold, largest prefetch set
MODELS = {
    "mixtral": (32, 8, 16, 0.5, 2, 0.9, 4),
    "qwen": (24, 60, 256, 0.7, 4, 0.8, 8),
    "phi": (32, 16, 1024, 0.6, 2, 0.85, 4),
}
EMB_CLUSTERS = 512
EMB_NOISE = 0.3
DISTANCE = 3          # prefetch distance of the deduplicating insert (layers)
STEP_DISTANCE = 6     # an incremental pass searches after layers 0 .. L - 7
GEOMETRIC_P = 0.15
DEDUP_BATCHES = 4     # batches of finished iterations a dedup state cycles through
CHUNK = 65536


def _case(kind, model, n, B, dtype="f32", d=0, k=1, law="uniform", blend=False, dynamic=False, name=None):
    c = {"kind": kind, "model": model, "n": n, "B": B, "dtype": dtype, "d": d, "k": k, "law": law, "blend": blend,
         "dynamic": dynamic}
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # a young store early in serving, one small batch: launches and latency
        _case("traj", "mixtral", 1000, 8, name="traj_mixtral_n1k_b8"),
        _case("sem", "mixtral", 1000, 8, d=4096, name="sem_d4096_n1k_b8"),
        # one decode iteration of 64 requests against a float32 store
        _case("traj", "qwen", 50000, 64, name="traj_qwen_n50k_b64"),
        # decode of many short prefixes, the best four maps blended
        _case("traj", "phi", 200000, 512, k=4, law="geometric", blend=True, name="traj_phi_top4_n200k_b512"),
        # a bfloat16 store of odd size and a batch below the large-batch scan
        _case("traj", "qwen", 200003, 100, dtype="bf16", name="traj_qwen_bf16_n200k_b100"),
        # the two halves of the largest mixed batch (the benchmark's step)
        _case("traj", "qwen", 1000000, 512, dtype="bf16", name="traj_qwen_bf16_n1m_b512"),
        _case("sem", "qwen", 1000000, 512, dtype="bf16", d=2048, name="sem_d2048_n1m_b512"),
        # prefill: a batch of new prompts by embedding
        _case("sem", "mixtral", 100000, 256, d=4096, name="sem_d4096_n100k_b256"),
        # the same with eight matches blended under the similarity threshold, ragged sizes
        _case("sem", "mixtral", 32749, 100, d=4096, k=8, blend=True, dynamic=True, name="sem_top8_d4096_n32k_b100"),
        # re-search after every layer of one forward pass
        _case("step", "qwen", 50000, 64, name="step_qwen_n50k_b64"),
        # a full store taking in a batch of finished iterations
        _case("dedup", "mixtral", 100000, 256, d=4096, name="dedup_d4096_n100k_b256"),
        # what the expert cache asks for between search and prefetch
        _case("plan", "qwen", 50000, 512, k=4, blend=True, dynamic=True, name="plan_qwen_n50k_b512"),
    ]


def _log(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["traj", "traj", "traj", "sem", "sem", "sem", "step", "dedup", "plan"])
    model = rng.choice(sorted(MODELS))
    dtype = rng.choice(["f32", "bf16"])
    L, E = MODELS[model][:2]
    if kind == "traj":
        # bounded so that no draw costs more than the largest listed cases
        n = _log(rng, 1000, 1000000 if dtype == "bf16" else 300000)
        B = _log(rng, 1, min(1024, max(8, 250000000 // n)))
        k = rng.choice([1, 1, 1, 4, 8])
        return _case(kind, model, n, B, dtype, 0, k, rng.choice(["uniform", "geometric"]), k > 1, rng.random() < 0.3)
    if kind == "sem":
        d = rng.choice([1024, 2048, 4096])
        k = rng.choice([1, 1, 1, 4, 8])
        n = _log(rng, 1000, 1000000 // (d // 1024))
        B = _log(rng, 1, min(1024, max(8, (1000000000 if k == 1 else 300000000) // (n * (d // 1024)))))
        return _case(kind, model, n, B, dtype, d, k, "uniform", k > 1, rng.random() < 0.3)
    if kind == "step":
        return _case(kind, model, _log(rng, 1000, 60000), _log(rng, 1, 128), dtype, 0, rng.choice([1, 1, 4]))
    if kind == "dedup":
        return _case(kind, model, _log(rng, 2000, 100000), _log(rng, 4, 256), dtype, rng.choice([1024, 2048, 4096]))
    k = rng.choice([1, 4])
    return _case(kind, model, _log(rng, 1000, 200000), _log(rng, 8, 1024), dtype, 0, k, "uniform", k > 1,
                 rng.random() < 0.5)


# ---------------------------------------------------------------- inputs

def _gen(seed, stream):
    g = torch.Generator(device="cuda")
    g.manual_seed((int(seed) * 1000003 + stream) & 0x7FFFFFFFFFFF)
    return g


def _randn(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda")


def _torch_dtype(c):
    return torch.bfloat16 if c["dtype"] == "bf16" else torch.float32


def _maps_like(c, clusters, centroids, g):
    sigma = MODELS[c["model"]][3]
    return torch.softmax(centroids[clusters] + sigma * _randn(g, len(clusters), *centroids.shape[1:]), dim=-1).to(
        _torch_dtype(c))


def _embs_like(clusters, centroids, g):
    x = centroids[clusters] + EMB_NOISE * _randn(g, len(clusters), centroids.shape[1])
    return (x / x.norm(dim=1, keepdim=True)).to(torch.bfloat16)


def _drawn(c, seed):
    """The clusters, the stored arrays and the batch's queries of a case."""
    L, E, n_map, sigma = MODELS[c["model"]][:4]
    n, d, B = c["n"], c["d"], c["B"]
    g = _gen(seed, 1)
    z = _randn(g, n_map, L, E)
    mu = _randn(g, EMB_CLUSTERS, d) if d else None
    ec = torch.randint(0, EMB_CLUSTERS, (n,), generator=g, device="cuda") if d else None
    mc = ec % n_map if d else torch.randint(0, n_map, (n,), generator=g, device="cuda")
    maps = torch.empty(n, L, E, dtype=_torch_dtype(c), device="cuda")
    embs = torch.empty(n, d, dtype=torch.bfloat16, device="cuda") if d else None
    for a in range(0, n, CHUNK):
        maps[a:a + CHUNK] = _maps_like(c, mc[a:a + CHUNK], z, g)
        if d:
            embs[a:a + CHUNK] = _embs_like(ec[a:a + CHUNK], mu, g)
    out = {"z": z, "mu": mu, "maps": maps, "embs": embs, "g": _gen(seed, 2)}
    g = out["g"]
    if c["kind"] == "sem":
        out["q"] = _embs_like(torch.randint(0, EMB_CLUSTERS, (B,), generator=g, device="cuda"), mu, g)
    elif c["kind"] in ("traj", "step", "plan"):
        src = torch.randint(0, n, (B,), generator=g, device="cuda")
        logits = torch.log(maps[src].float().clamp_min(1e-30))
        out["src"] = src
        out["q"] = torch.softmax(logits + sigma / 2 * _randn(g, B, L, E), dim=-1).to(_torch_dtype(c))
    if c["kind"] == "traj":
        u = torch.rand(B, generator=g, device="cuda", dtype=torch.float64)
        if c["law"] == "geometric":
            depth = 1 + torch.floor(torch.log1p(-u) / math.log1p(-GEOMETRIC_P))
        else:
            depth = 1 + torch.floor(u * (L - 1))
        out["depth"] = depth.clamp(1, L - 1).to(torch.int32)
    return out


def _new_iterations(c, a):
    """A batch of finished iterations: one in eight repeats a stored prompt."""
    B, g = c["B"], a["g"]
    ec = torch.randint(0, EMB_CLUSTERS, (B,), generator=g, device="cuda")
    maps, embs = _maps_like(c, ec % len(a["z"]), a["z"], g), _embs_like(ec, a["mu"], g)
    again = torch.rand(B, generator=g, device="cuda") < 0.125
    src = torch.randint(0, c["n"], (B,), generator=g, device="cuda")
    maps = torch.where(again[:, None, None], a["maps"][src], maps)
    embs = torch.where(again[:, None], a["embs"][src], embs)
    return maps.contiguous(), embs.contiguous()


def _selection(c):
    _, E, _, _, K, tau, k_max = MODELS[c["model"]]
    dyn = c["dynamic"]
    return {"tau": tau, "k_min": K if dyn else 1, "k_max": k_max, "mode": fm.FM_TAU_DYNAMIC if dyn else fm.FM_TAU_FIXED,
            "blend": fm.FM_BLEND_SCORE if c["blend"] else fm.FM_BLEND_NONE}


def prepare(case, seed):
    """A resident store with its workspace, one batch of queries and the
    output tensors that a serving loop keeps between iterations."""
    c = case
    L, E = MODELS[c["model"]][:2]
    B, k = c["B"], c["k"]
    a = _drawn(c, seed)
    store = fm.Store(c["n"], L, E, c["d"], c["dtype"])
    store.insert(a["maps"], a["embs"])
    s = {"case": c, "store": store, "ws": fm.Workspace(store), "sel": _selection(c)}

    def empty(dtype, *shape):
        return torch.empty(*shape, dtype=dtype, device="cuda")

    s["out"] = (empty(torch.int32, B, k), empty(torch.float32, B, k), empty(torch.int64, B, L),
                empty(torch.uint8, B, L))
    s["lb"] = torch.zeros(B, dtype=torch.int32, device="cuda")
    s["le"] = torch.full((B,), L, dtype=torch.int32, device="cuda")
    if c["kind"] == "traj":
        s["q"], s["depth"], s["lb"] = a["q"], a["depth"], a["depth"].clone()
    elif c["kind"] == "sem":
        s["q"] = a["q"]
    elif c["kind"] == "step":
        n_steps = L - STEP_DISTANCE
        s["pass"] = fm.TrajPass(store, B)
        s["q"] = [a["q"][:, l].contiguous() for l in range(n_steps)]
        s["out"] = (empty(torch.int32, n_steps, B, k), empty(torch.float32, n_steps, B, k))
    elif c["kind"] == "dedup":
        s["new"] = [_new_iterations(c, a) for _ in range(DEDUP_BATCHES)]
        s["turn"] = 0
        s["ones"] = torch.ones(B, 1, device="cuda")
        s["scratch"] = torch.empty(fm.dedup_scratch_bytes(c["n"], B) // 256 * 256 + 512, dtype=torch.uint8,
                                   device="cuda")
        s["scratch"] = s["scratch"][-s["scratch"].data_ptr() % 256:]
    else:
        idx, score = _matches(c, a)
        s["idx"], s["score"], s["q"] = idx, score, a["q"]
        s["l_now"] = torch.randint(0, L // 2, (B,), generator=a["g"], device="cuda").to(torch.int32)
        s["lb"] = s["l_now"] + 1
        s["order"] = (empty(torch.int32, B, L * E), empty(torch.float32, B, L * E), empty(torch.int32, B))
        s["miss"] = empty(torch.uint8, B, L)
    return s


def _matches(c, a):
    """Matches of a plan case: the query's source map first, then others,
    with the falling similarities of a top-k list."""
    B, k, g = c["B"], c["k"], a["g"]
    idx = torch.randint(0, c["n"], (B, k), generator=g, device="cuda").to(torch.int32)
    idx[:, 0] = a["src"].to(torch.int32)
    score = 0.95 - 0.3 * torch.rand(B, k, generator=g, device="cuda")
    return idx, score.sort(dim=1, descending=True).values.contiguous()


# ---------------------------------------------------------------- one pass

def run(s):
    c, store, ws, sel = s["case"], s["store"], s["ws"], s["sel"]
    if c["kind"] == "traj":
        return fm.match_trajectory_select(store, s["q"], s["depth"], s["lb"], s["le"], k=c["k"], out=s["out"],
                                          workspace=ws, **sel)
    if c["kind"] == "sem":
        return fm.match_semantic_select(store, s["q"], s["lb"], s["le"], k=c["k"], out=s["out"], workspace=ws, **sel)
    if c["kind"] == "step":
        idx, score = s["out"]
        for l, q in enumerate(s["q"]):
            s["pass"].step(q, l, c["k"], out=(idx[l], score[l]), workspace=ws)
        return idx, score
    if c["kind"] == "dedup":
        maps, embs = s["new"][s["turn"] % DEDUP_BATCHES]
        s["turn"] += 1
        slots = store.insert_dedup(maps, embs, DISTANCE, workspace=ws, scratch=s["scratch"])
        mask, count = fm.select_prefetch(store, slots[:, None], s["ones"], s["lb"], s["le"], out=s["out"][2:], **sel)
        return slots, mask, count
    mask, count = fm.select_prefetch(store, s["idx"], s["score"], s["lb"], s["le"], out=s["out"][2:], **sel)
    order, pri, n_pri = fm.priority_order(store, s["idx"], s["score"], mask, l_now=s["l_now"], blend=sel["blend"],
                                          out=s["order"])
    miss = fm.miss_count(store, s["q"], mask, MODELS[c["model"]][4], s["lb"], s["le"], out=s["miss"])
    return mask, count, order, pri, n_pri, miss


# ---------------------------------------------------------------- work, tolerance, exact results

def _mean_depth(c):
    L = MODELS[c["model"]][0]
    if c["law"] == "geometric":
        return sum((1 - GEOMETRIC_P) ** j for j in range(L - 1))
    return L / 2


def _max_depth(c):
    """Expected deepest prefix of the batch (the layers that must be read)."""
    L, B = MODELS[c["model"]][0], c["B"]
    if c["law"] == "geometric":
        return sum(1 - (1 - (1 - GEOMETRIC_P) ** j) ** B for j in range(L - 1))
    return sum(1 - (j / (L - 1)) ** B for j in range(L - 1))


def work(case):
    c = case
    L, E = MODELS[c["model"]][:2]
    n, B, k, d, es = c["n"], c["B"], c["k"], c["d"], 2 if c["dtype"] == "bf16" else 4
    rows = B * k * (L * E * es + 8) + B * L * 9   # matched rows read, matches and sets written
    if c["kind"] == "traj":
        return {"bytes": n * _max_depth(c) * E * es + B * _mean_depth(c) * E * es + rows,
                "flops": 2.0 * n * E * B * _mean_depth(c)}
    if c["kind"] == "sem":
        return {"bytes": n * d * 2 + B * d * 2 + rows, "flops": 2.0 * n * d * B}
    if c["kind"] == "step":
        steps = L - STEP_DISTANCE
        # a layer of the store, the running sums read and written
        return {"bytes": steps * (n * E * es + 8.0 * n * B + B * E * es + 8 * B * k), "flops": 2.0 * n * E * B * steps}
    if c["kind"] == "dedup":
        return {"bytes": n * (L * E * es + 2.0 * d) + 2 * B * (L * E * es + 2 * d) + rows,
                "flops": 2.0 * B * n * (L * E + d)}
    # the matched rows, the query rows and the outputs, each once
    return {"bytes": B * k * L * E * es + B * L * E * es + B * L * E * 8 + B * L * 10, "flops": 4.0 * B * k * L * E}


def tolerance(case):
    # float32 sums over up to 1,440 or 4,096 products; an index, and with it a
    # query's sets, may differ where two stored maps score alike
    if case["kind"] == "plan":
        return "exact"
    return {"rel": 2e-6, "max": 1e-5, "differ": 0.01}


def _top(scores, best, k):
    best = scores if best is None else torch.cat([best, scores], dim=1)
    return best.topk(min(k, best.shape[1]), dim=1).values


def _exact_trajectory(maps, q, depth, k):
    """[B][k] best cosines over the first depth[b] layers."""
    B, L, E = q.shape
    seen = torch.arange(L, device="cuda")[None, :] < depth[:, None]
    q = (q.double() * seen[:, :, None]).reshape(B, L * E)
    q = q / q.norm(dim=1, keepdim=True)
    best = None
    for a in range(0, len(maps), CHUNK):
        x = maps[a:a + CHUNK].double()
        norm = x.square().sum(dim=2).cumsum(dim=1).sqrt()[:, depth.long() - 1]
        best = _top((q @ x.reshape(len(x), L * E).t()) / norm.t(), best, k)
    return best


def exact(case, seed):
    c = case
    L, E = MODELS[c["model"]][:2]
    if c["kind"] == "dedup":
        return None   # slots and sets only
    a = _drawn(c, seed)
    if c["kind"] == "traj":
        return None, _exact_trajectory(a["maps"], a["q"], a["depth"], c["k"]), None, None
    if c["kind"] == "step":
        full = [torch.full((c["B"],), l + 1, dtype=torch.int32, device="cuda") for l in range(L - STEP_DISTANCE)]
        return None, torch.stack([_exact_trajectory(a["maps"], a["q"], f, c["k"]) for f in full])
    if c["kind"] == "sem":
        q = a["q"].double()
        q = q / q.norm(dim=1, keepdim=True)
        best = None
        for b in range(0, c["n"], CHUNK):
            x = a["embs"][b:b + CHUNK].double()
            best = _top((q @ x.t()) / x.norm(dim=1)[None, :], best, c["k"])
        return None, best, None, None
    # plan: the guiding probabilities, the sets and the ordered priorities
    idx, score = _matches(c, a)
    l_now = torch.randint(0, L // 2, (c["B"],), generator=a["g"], device="cuda")
    if c["blend"]:
        w = score.double().clamp_min(0)
        p = (a["maps"][idx.long()].double() * (w / w.sum(dim=1, keepdim=True))[:, :, None, None]).sum(dim=1)
    else:
        p = a["maps"][idx[:, 0].long()].double()
    sel = _selection(c)
    limit = (1 - score[:, 0].double()).clamp(0, 1) if c["dynamic"] else torch.full(
        (c["B"],), float(torch.tensor(sel["tau"], dtype=torch.float32)), dtype=torch.float64, device="cuda")
    value, rank = p.sort(dim=2, descending=True, stable=True)
    before = value.cumsum(dim=2) - value
    size = (before < limit[:, None, None]).sum(dim=2).clamp(sel["k_min"], sel["k_max"])
    kept = torch.zeros_like(p, dtype=torch.bool).scatter(2, rank, torch.arange(E, device="cuda") < size[:, :, None])
    ahead = torch.arange(L, device="cuda")[None, :] - l_now[:, None]
    pri = torch.where(kept & (ahead > 0)[:, :, None], p / ahead.clamp_min(1)[:, :, None], -math.inf)
    return None, None, None, pri.reshape(c["B"], L * E).sort(dim=1, descending=True).values, None, None
