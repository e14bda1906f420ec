"""GPU parity of moe_route against the oracle's gating (Sec. 2.1)."""
import numpy as np
import pytest

import oracle
from paper_2410_17954_amd import ops, synth
from gpu_helpers import to_dev, to_host, check_topk_against_bound, logit_bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,E,k,levels,renorm", [
    (1, 1, 1, None, True), (37, 8, 2, None, True), (37, 8, 2, 3, False), (1000, 60, 4, 5, True),
    (513, 64, 6, None, True), (300, 64, 6, 2, False), (64, 5, 5, 2, True), (200, 256, 8, 4, True),
    (7, 16, 1, None, True)])
def test_logits_in_mode_is_exact(T, E, k, levels, renorm):
    z = synth.random_logits(T, E, seed=T + E + k, levels=levels)
    idx, w, _ = ops.route(k=k, logits=to_dev(z), renormalize=renorm)
    idx, w = to_host(idx), to_host(w)
    z64 = z.astype(np.float64)
    ref_idx = oracle.topk_select(z64, k)
    assert np.array_equal(idx, ref_idx)
    ref_w = oracle.gate_weights(z64, ref_idx, renorm)
    assert np.max(np.abs(w - ref_w)) <= 1e-6


def test_signed_zero_and_equal_logits():
    z = np.array([[-0.0, 0.0, -0.0, -1.0, 0.0, -0.0, 0.0, -2.0],
                  [1.0] * 8, [2.0, 1.0, 2.0, 1.0, 3.0, 3.0, 0.0, 0.0]], dtype=np.float32)
    idx, w, _ = ops.route(k=3, logits=to_dev(z))
    assert to_host(idx).tolist() == oracle.topk_select(z.astype(np.float64), 3).tolist()


def _x_mode_case(name, T, seed, bias_kind=None, renorm=True):
    cfg = synth.workload(name)
    inp = synth.layer_inputs(cfg, seed, T=T, parts=("x", "router"))
    E, k = cfg["E"], cfg["k"]
    bias = None
    if bias_kind == "expert":
        bias = synth.zipf_bias(E, 1.2, synth.popularity_order(seed, E, 1)[0])
    elif bias_kind == "token":
        routes = synth.predicted_routes(T, 2, E, k, 0.7, 1.0, seed)
        bias = synth.route_boost_bias(routes, 0, E, 3.0,
                                      synth.zipf_bias(E, 1.0, synth.popularity_order(seed, E, 1)[0]))
    idx, w, z = ops.route(to_dev(inp["x"]), to_dev(inp["w_router"]), k,
                          bias=None if bias is None else to_dev(bias), renormalize=renorm,
                          want_logits=True)
    idx, w, z = to_host(idx), to_host(w), to_host(z)
    x, wr = synth.values(inp["x"]), synth.values(inp["w_router"])
    z_ref = oracle.router_logits(x, wr, bias)
    bound = logit_bound(x, wr, z_ref, bias)
    assert (np.abs(z - z_ref) <= bound).all(), np.max(np.abs(z - z_ref) / bound)
    near = check_topk_against_bound(idx, z_ref, bound, k)
    # decisions are taken on float64 logits on both sides: exact on every token
    assert np.array_equal(idx, oracle.topk_select(z_ref, k))
    ref_w = oracle.gate_weights(z_ref, idx, renorm)
    assert np.max(np.abs(w - ref_w)) <= bound.max() + 1e-6
    return near


def test_x_mode_tiny_fp32():
    _x_mode_case("tiny_fp32", 64, 1)


@pytest.mark.parametrize("T", [1, 17, 300])
def test_x_mode_ragged_token_counts(T):
    _x_mode_case("mixtral8x7b_layer", T, 7)


def test_x_mode_mixtral_full_size():
    near = _x_mode_case("mixtral8x7b_layer", 8192, 2)
    # a sizeable share of tokens is not decided by the float32 error bound
    # alone; those go through the float64 refinement
    assert near > 0


def test_x_mode_qwen_expert_bias():
    _x_mode_case("qwen15_moe_layer", 2048, 4, bias_kind="expert")


def test_x_mode_deepseek_token_bias_no_renorm():
    _x_mode_case("deepseek_v2_lite_layer", 4096, 5, bias_kind="token", renorm=False)


@pytest.mark.parametrize("T", [17, 8209, 20001, 40003])
def test_x_mode_token_tiles_ragged(T):
    # 33..64 experts run in tiles of 16, 32 or 64 tokens (the largest that
    # still gives two blocks per compute unit: 16 up to ~16K tokens, 32 up to
    # ~32K, then 64 on 256 CUs): one partial tile, and many tiles with a
    # ragged last one, for each tile size
    _x_mode_case("deepseek_v2_lite_layer", T, 11, bias_kind="expert")


def test_x_mode_48_experts():
    cfg = dict(synth.workload("qwen15_moe_layer"), E=40, k=5)
    inp = synth.layer_inputs(cfg, 12, T=300, parts=("x", "router"))
    idx, w, z = ops.route(to_dev(inp["x"]), to_dev(inp["w_router"]), 5, want_logits=True)
    x, wr = synth.values(inp["x"]), synth.values(inp["w_router"])
    z_ref = oracle.router_logits(x, wr)
    assert (np.abs(to_host(z) - z_ref) <= logit_bound(x, wr, z_ref)).all()
    assert np.array_equal(to_host(idx), oracle.topk_select(z_ref, 5))
    assert np.max(np.abs(to_host(w) - oracle.gate_weights(z_ref, to_host(idx), True))) <= 1e-5


def test_x_mode_wide_expert_count():
    cfg = dict(synth.workload("qwen15_moe_layer"), E=256, k=8)
    inp = synth.layer_inputs(cfg, 9, T=100, parts=("x", "router"))
    idx, w, z = ops.route(to_dev(inp["x"]), to_dev(inp["w_router"]), 8, want_logits=True)
    x, wr = synth.values(inp["x"]), synth.values(inp["w_router"])
    z_ref = oracle.router_logits(x, wr)
    bound = logit_bound(x, wr, z_ref)
    assert (np.abs(to_host(z) - z_ref) <= bound).all()
    check_topk_against_bound(to_host(idx), z_ref, bound, 8)


def test_x_mode_crafted_exact_and_near_ties():
    """Router rows that tie exactly, or differ by one bf16 ulp in one
    element, so float32 cannot separate them: the decision must still match
    the float64 oracle, exact ties going to the lower expert id."""
    g = np.random.default_rng(17)
    H, E, T, k = 512, 8, 64, 3
    w = synth.bf16_bits((g.standard_normal((E, H)) * 0.02).astype(np.float32))
    w[3] = w[1]                               # exact tie
    w[5] = w[1]
    w[5, 7] ^= 1                              # one ulp apart in one element
    w[6] = w[2]
    w[6, 100] += 1
    x = synth.bf16_bits(g.standard_normal((T, H)).astype(np.float32))
    x[:, 7] = synth.bf16_bits(np.full(T, 3.0, np.float32))
    idx, _, _ = ops.route(to_dev(x), to_dev(w), k)
    z_ref = oracle.router_logits(synth.values(x), synth.values(w))
    assert np.array_equal(to_host(idx), oracle.topk_select(z_ref, k))


@pytest.mark.parametrize("T", [64, 40000])
def test_x_mode_crafted_ties_60_experts(T):
    """The 33-64-expert kernel (float32 chains of one K-step in 16-token
    tiles, of four in 64-token tiles): strong router rows that tie exactly or
    differ by one bf16 ulp in one element sit in most tokens' top-4, so the
    certificate fails and the float64 recomputation decides; the result must
    match the float64 oracle, exact ties going to the lower expert id."""
    g = np.random.default_rng(23)
    H, E, k = 512, 60, 4
    wf = (g.standard_normal((E, H)) * 0.02).astype(np.float32)
    wf[[1, 9, 33], 7] = 0.5                   # with x[:, 7] = 3: usually selected
    w = synth.bf16_bits(wf)
    w[12] = w[1]                              # exact tie with expert 1
    w[40] = w[9]
    w[40, 3] ^= 1                             # one ulp from expert 9 in one element
    w[59] = w[33]                             # exact tie, the higher id last
    w[20] = w[33]
    w[20, 200] += 1
    x = synth.bf16_bits(g.standard_normal((T, H)).astype(np.float32))
    x[:, 7] = synth.bf16_bits(np.full(T, 3.0, np.float32))
    idx, _, _ = ops.route(to_dev(x), to_dev(w), k)
    z_ref = oracle.router_logits(synth.values(x), synth.values(w))
    got = to_host(idx)
    assert np.array_equal(got, oracle.topk_select(z_ref, k))
    # seven strong experts compete for four places: the crafted pairs are
    # decided in a large share of the tokens
    assert (got == 12).any(axis=1).mean() > 0.4 and (got == 59).any(axis=1).mean() > 0.4


def test_x_mode_crafted_ties_16_token_tiles():
    # more 16-token blocks than compute units: the tile kernel with 16-token
    # tiles (fewer take the K-split kernel, the 64-token case above)
    test_x_mode_crafted_ties_60_experts(5000)


@pytest.mark.parametrize("T,H,E,k,bias_kind", [
    (5, 100, 200, 70, None), (3, 64, 256, 256, "token"), (9, 7, 5, 5, "expert"), (2, 130, 65, 1, None),
])
def test_f32_router(T, H, E, k, bias_kind):
    """float32 inputs are decided in float64: exact ties (equal router rows)
    go to the lower id at any rank; gates within float32 rounding."""
    g = np.random.default_rng(31 + E)
    x = g.standard_normal((T, H)).astype(np.float32)
    w = (g.standard_normal((E, H)) * 0.2).astype(np.float32)
    w[E // 2] = w[1]
    w[E - 1] = w[1]
    bias = None if bias_kind is None else \
        g.standard_normal((T, E) if bias_kind == "token" else E).astype(np.float32)
    z = x.astype(np.float64) @ w.astype(np.float64).T + (0.0 if bias is None else bias)
    for renorm in (True, False):
        idx, gate, lg = ops.route(to_dev(x), to_dev(w), k, want_logits=True, renormalize=renorm,
                                  bias=None if bias is None else to_dev(bias))
        ref = oracle.topk_select(z, k)
        assert np.array_equal(to_host(idx), ref)
        # a float32 exponential of a float32 difference, summed over E
        assert np.max(np.abs(to_host(gate) - oracle.gate_weights(z, ref, renorm))) <= 1e-5
        assert np.max(np.abs(to_host(lg) - z)) <= 2.0 ** -23 * np.max(np.abs(z))


@pytest.mark.parametrize("renorm", [True, False])
def test_f32_router_nan_and_infinities(renorm):
    # NaN logits are never chosen and hide no other expert (6 shares a lane with
    # 70, 134 and 198), -inf ones only after all others; a token whose hidden
    # state is NaN gets no expert
    T, H, E, k = 6, 40, 200, 6
    g = np.random.default_rng(77)
    x = g.standard_normal((T, H)).astype(np.float32)
    w = (g.standard_normal((E, H)) * 0.2).astype(np.float32)
    w[[6, 64, 199]] = np.nan
    bias = g.standard_normal(E).astype(np.float32)
    bias[[70, 134, 0]] = 20, 21, 19
    bias[9:60] = -np.inf
    x[4, 3] = np.nan
    with np.errstate(invalid="ignore"):
        z = x.astype(np.float64) @ w.astype(np.float64).T + bias
    idx, gate, _ = ops.route(to_dev(x), to_dev(w), k, bias=to_dev(bias), renormalize=renorm)
    idx, gate = to_host(idx), to_host(gate)
    key = np.where(np.isnan(z), -np.inf, z)
    for t in range(T):
        if t == 4:
            assert (idx[t] == -1).all() and np.isnan(gate[t]).all()
            continue
        ref = np.argsort(-key[t], kind="stable")[:k]
        assert np.array_equal(idx[t], ref)
        if renorm:
            e = np.exp(z[t, ref] - z[t, ref].max())
            assert np.max(np.abs(gate[t] - e / e.sum())) <= 1e-5
        else:
            assert np.isnan(gate[t]).all()        # the softmax runs over a NaN
    # fewer numbers than k
    idx, gate, _ = ops.route(to_dev(x[:1]), to_dev(w[5:8]), 3, renormalize=True)
    z = x[:1].astype(np.float64) @ w[[5, 7]].astype(np.float64).T
    a, b = (5, 7) if z[0, 0] >= z[0, 1] else (7, 5)
    assert to_host(idx)[0].tolist() == [a - 5, b - 5, -1] and to_host(gate)[0, 2] == 0
