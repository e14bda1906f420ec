"""Workloads of the MoE-layer path: the calls a serving program makes of this
package, with their inputs, their necessary work and a 64-bit reference.

A case is a dict of plain values. Its "kind" says which calls one pass makes:

  layer    one MoE layer on one batch: route, permute, expert_ffn, combine,
           with the always-on shared experts where the model has them
  stack    one batch through several residual layers (stack_forward)
  plan     what precedes a unit of batches: schedule_multi over predicted
           routes, kv_gather where the tokens carry KV rows, kv_reindex
  predict  the routing path predictor and the binarised routes (rpp_forward,
           route_binarize)

Shapes are those of synth.WORKLOADS: a Mixtral-8x7B layer, a Qwen1.5-MoE layer,
a DeepSeek-V2-Lite layer and the tiny float32 layer. Inputs follow the same
recipe (hidden states N(0,1), weights N(0,0.02), Zipf-skewed routers, Markov
routes) drawn on the GPU. Workspaces and outputs are allocated beforehand, as
a serving loop keeps them.
"""
import math

import numpy as np
import torch

from paper_2410_17954_amd import ops

DEV = "cuda:0"

# One layer of each workload. A case adds T (tokens of the batch), S (experts
# the cache holds) and unit (the batch is 1/unit of the hidden states at hand,
# picked by token ids, as the scheduler's batches are).
FAMILIES = {
    "mixtral": dict(dtype="bf16", H=4096, E=8, F=14336, k=2, shared=0, zipf=0.0, renorm=True),
    "qwen": dict(dtype="bf16", H=2048, E=60, F=1408, k=4, shared=4, zipf=1.2, renorm=False),
    "deepseek": dict(dtype="bf16", H=2048, E=64, F=1408, k=6, shared=2, zipf=1.0, renorm=False),
    "tiny": dict(dtype="f32", H=128, E=8, F=256, k=2, shared=0, zipf=0.0, renorm=True),
}


def _layer(family, T, resident=None, unit=1, name=None, **over):
    c = dict(FAMILIES[family], kind="layer", T=T, unit=unit, **over)
    c["S"] = c["E"] if resident is None else resident
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the tiny float32 layer: the shape a user checks a change of their own
        # program with; nothing but launches
        _layer("tiny", 64, name="tiny_f32_t64"),
        # one token of one sequence: the smallest decode step
        _layer("qwen", 1, name="qwen_decode_t1"),
        # decode batch of an odd number of sequences over many small experts
        _layer("qwen", 53, name="qwen_decode_t53"),
        # decode batch over few large experts: the weight stream
        _layer("mixtral", 16, name="mixtral_decode_t16"),
        # a ragged chunk of chunked prefill: experts of some 200 rows
        _layer("mixtral", 777, name="mixtral_chunk_t777"),
        # prefill batch, every expert resident
        _layer("mixtral", 4096, name="mixtral_prefill_t4096"),
        # prefill batch, 32 of 60 experts resident, skewed router, shared experts
        _layer("qwen", 8192, resident=32, name="qwen_prefill_t8192"),
        # half of a 32768-token unit, 48 of 64 experts resident, shared experts
        _layer("deepseek", 16384, resident=48, unit=2, name="deepseek_half_t16384"),
        # decode batch through consecutive layers: the gaps between launches
        dict(kind="stack", name="qwen_stack_t24_l8", T=24, L=8, H=2048, E=60, F=1408, k=4),
        # a prefill unit split into two batches by predicted routes
        dict(kind="plan", name="plan_n8192_b2", N=8192, L=32, E=8, k=2, B=2, kv_bytes=0),
        # decode sequences regrouped into small batches, their KV rows moved
        dict(kind="plan", name="plan_n256_b8_kv", N=256, L=24, E=60, k=4, B=8, kv_bytes=1024),
        # the predictor over a prefill unit's token ids
        dict(kind="predict", name="predict_b16_s512", B=16, S=512, L=32, E=8, k=2),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["mixtral", "qwen", "qwen_cache", "deepseek", "generic", "tiny", "stack",
                       "plan", "plan_kv", "predict"])
    if kind == "mixtral":
        return _layer("mixtral", _log_int(rng, 1, 4096), resident=rng.choice([8, 8, 4]))
    if kind == "qwen":
        return _layer("qwen", _log_int(rng, 1, 4096))
    if kind == "qwen_cache":
        return _layer("qwen", _log_int(rng, 64, 8192), resident=rng.randint(16, 48))
    if kind == "deepseek":
        return _layer("deepseek", _log_int(rng, 16, 12288), resident=rng.randint(32, 64), unit=2)
    if kind == "generic":
        E, step = rng.choice([4, 8, 16, 32]), rng.choice([64, 64, 8])
        return _layer("mixtral", _log_int(rng, 4, 2048), H=step * rng.randint(512 // step, 2560 // step),
                      F=step * rng.randint(768 // step, 4096 // step), E=E,
                      k=rng.choice([1, 2, 4]), resident=E)
    if kind == "tiny":
        E = rng.choice([4, 8, 16])
        return _layer("tiny", _log_int(rng, 8, 512), H=4 * _log_int(rng, 16, 128),
                      F=4 * _log_int(rng, 32, 256), E=E, k=rng.choice([1, 2]), resident=E)
    if kind == "stack":
        return dict(kind="stack", T=_log_int(rng, 1, 64), L=rng.randint(2, 8), H=2048, E=60,
                    F=1408, k=4)
    if kind == "plan":
        L, E, k = rng.choice([(32, 8, 2), (24, 60, 4), (26, 64, 6)])
        return dict(kind="plan", N=_log_int(rng, 512, 32768), L=L, E=E, k=k, B=2, kv_bytes=0)
    if kind == "plan_kv":
        L, E, k = rng.choice([(32, 8, 2), (24, 60, 4), (26, 64, 6)])
        return dict(kind="plan", N=_log_int(rng, 16, 2048), L=L, E=E, k=k,
                    B=rng.choice([2, 3, 4, 8, 16]), kv_bytes=rng.choice([512, 1000, 1024, 2048]))
    L, E, k = rng.choice([(32, 8, 2), (24, 60, 4)])
    return dict(kind="predict", B=_log_int(rng, 1, 16), S=rng.randint(24, 512), L=L, E=E, k=k)


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _normal(g, shape, std, dtype):
    out = torch.empty(shape, dtype=dtype, device=DEV)
    return out.normal_(0.0, std, generator=g)


def _zipf_bias(g, E, s):
    """ln of the Zipf(s) mass over a drawn popularity order, float32 [E]."""
    mass = torch.arange(1, E + 1, dtype=torch.float64, device=DEV) ** -s
    b = torch.empty(E, dtype=torch.float64, device=DEV)
    b[torch.randperm(E, generator=g, device=DEV)] = torch.log(mass / mass.sum())
    return b.float()


def _routes(g, N, L, E, k, keep=0.7, s=1.1):
    """Predicted routes uint8 [N, L, k]: a choice keeps its expert of the layer
    before with probability `keep` where that is free, else draws by Zipf(s)
    over the layer's own popularity order among the free experts."""
    out = torch.empty((N, L, k), dtype=torch.uint8, device=DEV)
    mass = torch.arange(1, E + 1, dtype=torch.float32, device=DEV) ** -s
    prev = None
    for l in range(L):
        w = torch.empty(E, device=DEV)
        w[torch.randperm(E, generator=g, device=DEV)] = mass
        free = torch.ones((N, E), device=DEV)
        cur = []
        for j in range(k):
            pick = torch.multinomial(free * w, 1, generator=g)
            if prev is not None:
                stay = (torch.rand((N, 1), generator=g, device=DEV) < keep) \
                    & (free.gather(1, prev[j]) > 0)
                pick = torch.where(stay, prev[j], pick)
            free.scatter_(1, pick, 0.0)
            cur.append(pick)
            out[:, l, j] = pick[:, 0].to(torch.uint8)
        prev = cur
    return out


def _predictor_dims(case):
    return dict(vocab=32000, d_model=32, n_heads=4, d_ff=2048, n_enc=3, n_dec=3, L=case["L"],
                E=case["E"], num_buckets=32, max_distance=128, eps=1e-6)


def _prepare_layer(case, seed):
    g = _gen(seed)
    H, E, F, k, T, S = (case[n] for n in ("H", "E", "F", "k", "T", "S"))
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    code = ops.MOE_F32 if case["dtype"] == "f32" else ops.MOE_BF16
    n = T * case["unit"]
    s = dict(case=case)
    s["x"] = _normal(g, (n, H), 1.0, dt)
    s["w_router"] = _normal(g, (E, H), 0.02, dt)
    s["bias"] = _zipf_bias(g, E, case["zipf"]) if case["zipf"] else None
    s["w_gate"] = _normal(g, (S, F, H), 0.02, dt)
    s["w_up"] = _normal(g, (S, F, H), 0.02, dt)
    s["w_down"] = _normal(g, (S, H, F), 0.02, dt)
    s["tok"] = None
    if case["unit"] > 1:       # the scheduler's batches hold their ids ascending
        s["tok"] = torch.randperm(n, generator=g, device=DEV)[:T].sort().values.int()
    s["slot"] = None
    if S < E:                  # the S experts with the largest demand, ids ascending
        z = s["x"].float() @ s["w_router"].float().T
        z = z if s["bias"] is None else z + s["bias"]
        idx = z.topk(k, dim=1).indices
        idx = idx if s["tok"] is None else idx[s["tok"].long()]
        demand = torch.bincount(idx.reshape(-1), minlength=E)
        held = demand.sort(descending=True, stable=True).indices[:S].sort().values
        slot = torch.full((E,), -1, dtype=torch.int32, device=DEV)
        slot[held] = torch.arange(S, dtype=torch.int32, device=DEV)
        s["slot"] = slot
    R = T * k
    s["idx"] = torch.empty((n, k), dtype=torch.int32, device=DEV)
    s["gates"] = torch.empty((n, k), dtype=torch.float32, device=DEV)
    s["offs"] = torch.empty(E + 1, dtype=torch.int32, device=DEV)
    s["rop"] = torch.empty(R, dtype=torch.int32, device=DEV)
    s["por"] = torch.empty(R, dtype=torch.int32, device=DEV)
    s["xp"] = torch.empty((R, H), dtype=dt, device=DEV)
    s["yp"] = torch.empty((R, H), dtype=dt, device=DEV)
    s["y"] = torch.zeros((n, H), dtype=dt, device=DEV)
    s["inc"] = torch.empty(T, dtype=torch.int32, device=DEV)
    s["ws_p"] = ops.workspace_tensor(ops.permute_workspace(T, k, E), DEV)
    s["ws_f"] = ops.workspace_tensor(ops.expert_ffn_workspace(R, H, F, E, code), DEV)
    if case["shared"]:
        Fs = case["shared"] * F
        s["sh_gate"] = _normal(g, (1, Fs, H), 0.02, dt)
        s["sh_up"] = _normal(g, (1, Fs, H), 0.02, dt)
        s["sh_down"] = _normal(g, (1, H, Fs), 0.02, dt)
        s["sh_offs"] = torch.tensor([0, T], dtype=torch.int32, device=DEV)
        s["xs"] = torch.empty((T, H), dtype=dt, device=DEV) if case["unit"] > 1 else None
        s["ys"] = torch.empty((T, H), dtype=dt, device=DEV)
        s["ws_s"] = ops.workspace_tensor(ops.expert_ffn_workspace(T, H, Fs, 1, code), DEV)
    return s


def _prepare_stack(case, seed):
    """Layers of different routers; a token's hidden state points towards the
    k experts per layer that it is routed to, as trained routers have it (so
    that a rounding does not decide the route of a token)."""
    g = _gen(seed)
    T, L, H, E, F, k = (case[n] for n in ("T", "L", "H", "E", "F", "k"))
    bf = torch.bfloat16
    layers, norms = [], []
    h = torch.empty((T, H), device=DEV).normal_(0.0, 1.0, generator=g)
    for _ in range(L):
        wr = _normal(g, (E, H), 0.02, bf)
        layers.append((wr, _normal(g, (E, F, H), 0.02, bf), _normal(g, (E, F, H), 0.02, bf),
                       _normal(g, (E, H, F), 0.02, bf)))
        norms.append(_normal(g, (H,), 0.1, bf) + 1.0)
        to = torch.rand((T, E), generator=g, device=DEV).topk(k, dim=1).indices
        unit = torch.nn.functional.normalize(wr.float(), dim=1)
        for j in range(k):
            h += (5.0 + 0.6 * j) * unit[to[:, j]]
    return dict(case=case, h0=h.to(bf), h=torch.empty((T, H), dtype=bf, device=DEV),
                layers=layers, norms=norms,
                err=torch.zeros(1, dtype=torch.int32, device=DEV),
                ws=ops.workspace_tensor(ops.stack_workspace(T, H, F, E, k), DEV))


def _prepare_plan(case, seed):
    g = _gen(seed)
    N, L, E, k, B, kv = (case[n] for n in ("N", "L", "E", "k", "B", "kv_bytes"))
    s = dict(case=case, routes=_routes(g, N, L, E, k))
    s["perm"] = torch.empty(N, dtype=torch.int32, device=DEV)
    s["offs"] = torch.empty(B + 1, dtype=torch.int32, device=DEV)
    s["demand"] = torch.empty((B, L, E), dtype=torch.int32, device=DEV)
    s["info"] = torch.empty((B - 1, 8), dtype=torch.int64, device=DEV)
    s["err"] = torch.zeros(1, dtype=torch.int32, device=DEV)
    s["batch_of"] = torch.empty(N, dtype=torch.int32, device=DEV)
    s["pos_of"] = torch.empty(N, dtype=torch.int32, device=DEV)
    s["ws"] = ops.workspace_tensor(ops.schedule_multi_workspace(N, L, E, k, B), DEV)
    if kv:                     # the caches of the B original batches
        cuts = [N * b // B for b in range(B + 1)]
        s["kv"] = [torch.randint(0, 256, (L, hi - lo, kv), dtype=torch.uint8, device=DEV,
                                 generator=g) for lo, hi in zip(cuts, cuts[1:])]
        s["kv_new"] = torch.empty((L, N, kv), dtype=torch.uint8, device=DEV)
    return s


def _prepare_predict(case, seed):
    g = _gen(seed)
    dims = _predictor_dims(case)
    B, S = case["B"], case["S"]
    shape = (B, S, dims["L"], dims["E"])
    return dict(case=case, dims=dims,
                ids=torch.randint(0, dims["vocab"], (B, S), generator=g, device=DEV,
                                  dtype=torch.int32),
                weights=torch.randn(ops.rpp_weights_count(dims), generator=g, device=DEV) * 0.1,
                probs=torch.empty(shape, dtype=torch.float32, device=DEV),
                logits=torch.empty(shape, dtype=torch.float32, device=DEV),
                routes=torch.empty(shape[:3] + (case["k"],), dtype=torch.uint8, device=DEV),
                err=torch.zeros(1, dtype=torch.int32, device=DEV),
                ws=ops.workspace_tensor(ops.load_library().moe_rpp_workspace(
                    B, S, ops.ctypes.byref(ops.rpp_dims(dims))), DEV))


_PREPARE = dict(layer=_prepare_layer, stack=_prepare_stack, plan=_prepare_plan,
                predict=_prepare_predict)


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, seed)


# ------------------------------------------------------------------ pass
def _run_layer(s):
    c = s["case"]
    E, k = c["E"], c["k"]
    ops.route(s["x"], s["w_router"], k, bias=s["bias"], renormalize=c["renorm"],
              topk_idx=s["idx"], topk_w=s["gates"])
    ops.permute(s["x"], s["idx"], E, token_ids=s["tok"], expert_offsets=s["offs"],
                row_of_pair=s["rop"], pair_of_row=s["por"], x_perm=s["xp"], workspace=s["ws_p"])
    ops.expert_ffn(s["xp"], s["offs"], s["w_gate"], s["w_up"], s["w_down"],
                   slot_of_expert=s["slot"], y_perm=s["yp"], workspace=s["ws_f"])
    ys = None
    if c["shared"]:
        xs = s["x"]
        if s["tok"] is not None:
            xs = torch.index_select(s["x"], 0, s["tok"], out=s["xs"])
        ys = ops.expert_ffn(xs, s["sh_offs"], s["sh_gate"], s["sh_up"], s["sh_down"],
                            y_perm=s["ys"], workspace=s["ws_s"])
    ops.combine(s["yp"], s["idx"], s["gates"], s["rop"], token_ids=s["tok"],
                slot_of_expert=s["slot"], y_shared=ys, y=s["y"], incomplete=s["inc"])
    return dict(y=s["y"], idx=s["idx"], gates=s["gates"], incomplete=s["inc"])


def _run_stack(s):
    s["h"].copy_(s["h0"])      # the layers update the hidden states in place
    ops.stack_forward(s["h"], s["layers"], s["case"]["k"], pre_norm=True,
                      norm_weights=s["norms"], err=s["err"], workspace=s["ws"])
    return dict(h=s["h"], err=s["err"])


def _run_plan(s):
    c = s["case"]
    ops.schedule_multi(s["routes"], c["E"], c["B"], perm=s["perm"], batch_offsets=s["offs"],
                       demand=s["demand"], info=s["info"], workspace=s["ws"], err=s["err"])
    out = dict(perm=s["perm"], offs=s["offs"], demand=s["demand"], info=s["info"], err=s["err"],
               batch_of=s["batch_of"], pos_of=s["pos_of"])
    if c["kv_bytes"]:
        ops.kv_gather(s["kv"], index=s["perm"], out=s["kv_new"], err=s["err"])
        out["kv"] = s["kv_new"]
    ops.kv_reindex(s["perm"], s["offs"], batch_of=s["batch_of"], pos_of=s["pos_of"],
                   err=s["err"])
    return out


def _run_predict(s):
    ops.rpp_forward(s["ids"], s["weights"], s["dims"], probs=s["probs"], logits=s["logits"],
                    err=s["err"], workspace=s["ws"])
    ops.route_binarize(s["logits"], s["case"]["k"], routes=s["routes"])
    return dict(probs=s["probs"], logits=s["logits"], routes=s["routes"], err=s["err"])


_RUN = dict(layer=_run_layer, stack=_run_stack, plan=_run_plan, predict=_run_predict)


def run(state):
    return _RUN[state["case"]["kind"]](state)


# ------------------------------------------------------- necessary work
def _expert_loads(case, T):
    """Expected share of a batch's tokens each expert gets, by a draw of router
    logits, float64 [E], and the expected number of experts with any token."""
    r = np.random.default_rng(1)
    z = r.normal(0.0, 0.02 * math.sqrt(case["H"]), (20000, case["E"]))
    if case["zipf"]:
        z += np.log(np.arange(1, case["E"] + 1) ** -case["zipf"])
    top = np.argpartition(-z, case["k"] - 1, axis=1)[:, :case["k"]]
    p = np.bincount(top.reshape(-1), minlength=case["E"]) / z.shape[0]
    return p, 1.0 - (1.0 - np.minimum(p, 1.0)) ** T


def _work_layer(case):
    H, E, F, k, T, S = (case[n] for n in ("H", "E", "F", "k", "T", "S"))
    es = 4 if case["dtype"] == "f32" else 2
    n = T * case["unit"]
    p, used = _expert_loads(case, T)
    held = np.argsort(-p, kind="stable")[:S]
    pairs = T * float(p[held].sum())
    Fs = case["shared"] * F
    b = es * (n * H + E * H)                                   # hidden states, router
    b += es * 3 * H * F * float(used[held].sum()) + es * 3 * H * Fs   # weights
    b += es * T * H + n * k * 8 + T * 4                        # y, top-k, flags
    return {"bytes": b, "flops": 2.0 * n * H * E + 6.0 * H * F * pairs + 6.0 * H * Fs * T}


def _work_stack(case):
    T, L, H, E, F, k = (case[n] for n in ("T", "L", "H", "E", "F", "k"))
    used = E * (1.0 - (1.0 - k / E) ** T)
    return {"bytes": 2.0 * L * (3 * H * F * used + E * H + H) + 2.0 * 2 * T * H,
            "flops": L * (2.0 * T * H * E + 6.0 * H * F * T * k)}


def _work_plan(case):
    N, L, E, k, B, kv = (case[n] for n in ("N", "L", "E", "k", "B", "kv_bytes"))
    # routes read once, perm, maps and demand written once, KV rows moved once;
    # one similarity of a token's k*L choices to two centroids per split level
    return {"bytes": N * L * k + 4.0 * (3 * N + B + 1) + 4.0 * B * L * E + 64.0 * (B - 1)
            + 2.0 * L * N * kv,
            "flops": 2.0 * N * L * k * max(1, math.ceil(math.log2(B)))}


def _work_predict(case):
    d = _predictor_dims(case)
    D, dff, LE, S = d["d_model"], d["d_ff"], d["L"] * d["E"], case["S"]
    M = case["B"] * S
    enc = d["n_enc"] * M * (8.0 * D * D + 4 * D * dff + 4 * S * D)
    dec = d["n_dec"] * M * (16.0 * D * D + 4 * D * dff + 4 * S * D + 2 * (S + 1) * D)
    weights = ops.rpp_weights_count(d) - d["vocab"] * D + min(M, d["vocab"]) * D
    return {"bytes": 4.0 * (M + weights + 2 * M * LE) + M * d["L"] * case["k"],
            "flops": enc + dec + 2.0 * M * D * LE}


_WORK = dict(layer=_work_layer, stack=_work_stack, plan=_work_plan, predict=_work_predict)


def work(case):
    return _WORK[case["kind"]](case)


def tolerance(case):
    """Whole numbers (top-k ids, flags, plans, KV bytes) are exact. bf16 values:
    about four times what a pass differs from the 64-bit reference by (0.0029 a
    layer, 0.0054 eight layers); float32 sums: what another order may show."""
    if case["kind"] == "plan":
        return "exact"
    if case["kind"] == "predict":
        # float32 sums through six blocks; a near tie may swap a route
        return {"rel": 1e-5, "differ": 1e-3}
    if case["kind"] == "stack":
        # bf16 states, one rounding per layer
        return {"rel": 2e-2}
    if case["dtype"] == "f32":
        return {"rel": 1e-5}
    # bf16 activations, expert outputs and layer outputs, each rounded once
    return {"rel": 1e-2}


# ------------------------------------------------------ 64-bit reference
def _ffn64(x, wg, wu, wd):
    g = x @ wg.double().T
    return (g * torch.sigmoid(g) * (x @ wu.double().T)) @ wd.double().T


def _gate64(x, w, bias, k, renorm):
    z = x @ w.double().T
    z = z if bias is None else z + bias.double()
    top = z.sort(dim=1, descending=True, stable=True)
    idx = top.indices[:, :k]
    gates = torch.softmax(z, dim=1).gather(1, idx)
    return idx, gates / gates.sum(1, keepdim=True) if renorm else gates


def _experts64(x, idx, gates, slot, wg, wu, wd):
    y = torch.zeros_like(x)
    for e in range(slot.shape[0]):
        s = int(slot[e])
        if s < 0:
            continue
        t, j = (idx == e).nonzero(as_tuple=True)
        if t.numel():
            y.index_add_(0, t, gates[t, j, None] * _ffn64(x[t], wg[s], wu[s], wd[s]))
    return y


def _exact_layer(case, seed):
    s = _prepare_layer(case, seed)
    E = case["E"]
    x = s["x"].double()
    idx, gates = _gate64(x, s["w_router"], s["bias"], case["k"], case["renorm"])
    slot = s["slot"] if s["slot"] is not None else torch.arange(E, device=DEV)
    tok = s["tok"].long() if s["tok"] is not None else torch.arange(x.shape[0], device=DEV)
    xb = x[tok]
    yb = _experts64(xb, idx[tok], gates[tok], slot.cpu(), s["w_gate"], s["w_up"], s["w_down"])
    if case["shared"]:
        yb += _ffn64(xb, s["sh_gate"][0], s["sh_up"][0], s["sh_down"][0])
    y = torch.zeros_like(x)
    y[tok] = yb
    inc = (slot[idx[tok]] < 0).any(1)
    return dict(y=y, idx=idx.int(), gates=gates, incomplete=inc.int())


def _exact_stack(case, seed):
    s = _prepare_stack(case, seed)
    h = s["h0"].double()
    slot = torch.arange(case["E"])
    for (wr, wg, wu, wd), nw in zip(s["layers"], s["norms"]):
        x = h / torch.sqrt((h * h).mean(1, keepdim=True) + 1e-5) * nw.double()
        idx, gates = _gate64(x, wr, None, case["k"], True)
        h = h + _experts64(x, idx, gates, slot, wg, wu, wd)
    return dict(h=h, err=torch.zeros_like(s["err"]))


def _bucket(n, bidirectional, nb=32, far=128):
    """T5 relative-position bucket of distance n = query - key, in integers."""
    base = 0
    if bidirectional:
        nb //= 2
        base, n = (nb, -n) if n < 0 else (0, n)
    n = max(n, 0)
    m = nb // 2
    if n < m:
        return base + n
    if n >= far:
        return base + nb - 1
    a, c = nb - m, (far // m).bit_length() - 1
    return base + min(nb - 1, m + ((n ** a).bit_length() - 1 - a * (m.bit_length() - 1)) // c)


def _exact_predict(case, seed):
    s = _prepare_predict(case, seed)
    d = s["dims"]
    D, nh, dff, nb, eps = d["d_model"], d["n_heads"], d["d_ff"], d["num_buckets"], d["eps"]
    w, at = s["weights"].double(), [0]

    def take(*shape):
        n = math.prod(shape)
        at[0] += n
        return w[at[0] - n:at[0]].view(shape)

    def rms(v, scale):
        return v / torch.sqrt((v * v).mean(-1, keepdim=True) + eps) * scale

    B, S = case["B"], case["S"]
    dk = D // nh

    def heads(t):
        return t.view(B, S, nh, dk).transpose(1, 2)

    def attend(xq, xkv, q, k, v, o, bias):
        p = heads(xq @ q.T) @ heads(xkv @ k.T).transpose(2, 3)
        p = torch.softmax(p if bias is None else p + bias, dim=-1)
        return (p @ heads(xkv @ v.T)).transpose(1, 2).reshape(B, S, D) @ o.T

    def position(rel, bidirectional):
        r = range(-(S - 1), S)
        t = rel[torch.tensor([_bucket(n, bidirectional) for n in r], device=DEV)]
        i = torch.arange(S, device=DEV)
        dist = i[:, None] - i[None, :]
        b = t[dist + S - 1].permute(2, 0, 1)
        return b if bidirectional else b.masked_fill(dist < 0, -math.inf)

    emb = take(d["vocab"], D)
    x = emb[s["ids"].long()]
    y = x
    bias = position(take(nb, nh), True)
    for _ in range(d["n_enc"]):
        n = rms(x, take(D))
        x = x + attend(n, n, take(D, D), take(D, D), take(D, D), take(D, D), bias)
        n = rms(x, take(D))
        x = x + torch.relu(n @ take(dff, D).T) @ take(D, dff).T
    enc = rms(x, take(D))
    bias = position(take(nb, nh), False)
    for _ in range(d["n_dec"]):
        n = rms(y, take(D))
        y = y + attend(n, n, take(D, D), take(D, D), take(D, D), take(D, D), bias)
        n = rms(y, take(D))
        y = y + attend(n, enc, take(D, D), take(D, D), take(D, D), take(D, D), None)
        n = rms(y, take(D))
        y = y + torch.relu(n @ take(dff, D).T) @ take(D, dff).T
    y = rms(y, take(D))
    logits = (y @ take(d["L"] * d["E"], D).T).view(B, S, d["L"], d["E"])
    return dict(probs=torch.sigmoid(logits), logits=logits, routes=None,
                err=torch.zeros_like(s["err"]))


def exact(case, seed):
    if case["kind"] == "layer":
        return _exact_layer(case, seed)
    if case["kind"] == "stack":
        return _exact_stack(case, seed)
    if case["kind"] == "predict":
        return _exact_predict(case, seed)
    return None
