"""GPU parity of moe_expert_ffn against the oracle's SwiGLU experts."""
import numpy as np
import pytest
import torch

import oracle
from paper_2410_17954_amd import ops, synth
from gpu_helpers import to_dev, to_host, vals, rel_max_err

pytestmark = pytest.mark.gpu


def _weights(S, F, H, seed, dtype="bf16", std=0.02):
    g = np.random.default_rng(seed)
    ws = [g.standard_normal(s).astype(np.float32) * np.float32(std)
          for s in ((S, F, H), (S, F, H), (S, H, F))]
    return [synth.bf16_bits(w) for w in ws] if dtype == "bf16" else ws


def _rows(R, H, seed, dtype="bf16"):
    x = np.random.default_rng(seed + 1).standard_normal((R, H)).astype(np.float32)
    return synth.bf16_bits(x) if dtype == "bf16" else x


def _run(counts, H, F, slot, S, seed, dtype="bf16", tol=1e-2, extra_rows=0):
    counts = np.asarray(counts)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offsets[-1]) + extra_rows
    x = _rows(max(R, 1), H, seed, dtype)
    wg, wu, wd = _weights(S, F, H, seed, dtype)
    sentinel = 3.0
    tdt = torch.bfloat16 if dtype == "bf16" else torch.float32
    y = torch.full((max(R, 1), H), sentinel, dtype=tdt, device="cuda:0")
    ops.expert_ffn(to_dev(x), to_dev(offsets), to_dev(wg), to_dev(wu), to_dev(wd),
                   slot_of_expert=None if slot is None else to_dev(np.asarray(slot, np.int32)),
                   y_perm=y)
    torch.cuda.synchronize()
    got = vals(y)
    sl = np.arange(len(counts)) if slot is None else np.asarray(slot)
    ref, computed = oracle.expert_ffn(synth.values(x)[:offsets[-1]], offsets, sl,
                                      synth.values(wg), synth.values(wu), synth.values(wd))
    if computed.any():
        assert rel_max_err(got[:offsets[-1]][computed], ref[computed]) <= tol
    assert (got[:offsets[-1]][~computed] == sentinel).all()
    assert (got[offsets[-1]:] == sentinel).all()
    return got, ref, computed


def test_tiny_fp32_config():
    cfg = synth.workload("tiny_fp32")
    counts = np.bincount(synth.random_topk_idx(64, 8, 2, 1).ravel(), minlength=8)
    _run(counts, cfg["H"], cfg["F"], None, 8, seed=1, dtype="f32", tol=1e-4)


@pytest.mark.parametrize("counts,H,F", [
    ([0, 300, 17, 513], 256, 512),        # ragged, several row tiles, an empty expert
    ([900, 2, 20, 30], 256, 512),          # large batch: its few-row experts take the large tiles
    ([1], 64, 64),                         # one row
    ([256, 256], 128, 192),                # exact tiles, F not a multiple of 64
    ([700, 3, 0, 1029, 64], 512, 1408),    # Qwen-like F
    ([300, 5, 260], 136, 200),             # H, F not multiples of 32: general path
    ([40, 300], 264, 96),                  # general path, K tail inside a 64-deep step
    ([263, 544, 300, 1025, 0, 287], 256, 512),   # small last row tiles (7, 32, 44, 1, 31 rows)
    ([257, 7, 288], 512, 1408),            # small last row tiles next to a lone 7-row expert
    ([356, 326, 320, 321, 128, 96, 288], 256, 512),  # last tiles of 100, 70, 64, 65 rows stay in place, 32 goes last
    ([1400, 300, 2100], 256, 512),         # experts of 6 and 9 full-cost row tiles
])
def test_bf16_ragged_groups(counts, H, F):
    _run(counts, H, F, None, len(counts), seed=sum(counts) + H)


@pytest.mark.parametrize("counts,H,F", [
    ([300, 40, 200], 4096, 4096),      # both GEMMs split their only, partial round along K (2 pieces)
    ([300, 40, 200], 1024, 8192),      # the down projection in 4 pieces
    ([9, 1100, 257, 31], 512, 4096),   # split down projection over ragged tiles of every size
    ([280, 530], 1024, 4096),          # the down projection's split round holds small last row tiles (24, 18 rows)
])
def test_bf16_split_k_tail(counts, H, F):
    # Fewer tiles than compute units: the last round is split into K-pieces
    # whose fp32 partials are summed in a fixed order, so a second call gives
    # identical bits.
    got, _, _ = _run(counts, H, F, None, len(counts), seed=sum(counts) + F)
    again, _, _ = _run(counts, H, F, None, len(counts), seed=sum(counts) + F)
    np.testing.assert_array_equal(got, again)


@pytest.mark.parametrize("H,F", [
    (32, 64), (64, 96), (96, 32), (128, 160),      # 1 to 5 K-steps: prologue and tail only
    (416, 448), (480, 512), (544, 576),            # 13 to 18: around the first steady round
    (768, 800), (1120, 832),                       # 24 to 26 and 35: around the second
])
def test_bf16_k_loop_edges(H, F):
    # every remainder of the K loop's pairs and rounds in each row mode (full
    # tile, 128, 64 and 32 rows left); bound of the other bf16 cases
    _run([290, 129, 70, 20, 256], H, F, None, 5, seed=H + F)


@pytest.mark.parametrize("counts,H,F,slot", [
    ([200, 97, 96, 5, 0, 1, 33, 17, 64, 80], 256, 512, None),   # experts of 3, 2 and 1 items
    ([193, 0, 288, 2, 95, 1], 96, 160, None),        # K ends in 32 in both projections; 3 whole items
    ([1, 0, 0, 2], 32, 2080, None),                  # K of one half block; more waves than K blocks
    ([150, 7, 20, 100], 704, 96, [1, -1, 0, 2]),     # a split expert beside a missed one
    ([1] * 256, 64, 64, None),                       # the longest list
    ([40], 2048, 5632, None), ([2], 5632, 64, None),   # one expert: narrow units
    ([3] * 60, 256, 1408, None),                     # narrow down, wide up
])
def test_bf16_few_row_items(counts, H, F, slot):
    # decode-sized batches: no expert takes the large tiles, an expert of more
    # than 96 rows is cut into items; bound of the other bf16 cases
    S = len(counts) if slot is None else max(slot) + 1
    _run(counts, H, F, slot, S, seed=sum(counts) + H, extra_rows=7)


@pytest.mark.parametrize("counts,H,F,slot", [
    ([1, 0, 64, 65, 130], 128, 256, None),           # row groups of 64: whole, one over, several
    ([20, 3, 17], 4, 20, [1, -1, 0]),                # the shortest K, a part of a column block, a miss
    ([70, 33], 68, 36, None),                        # K ends inside a 16-wide step
    ([5, 40], 30, 50, None),                         # rows not 16-byte aligned: one thread per output
    ([1] * 130, 16, 16, None),                       # experts past the first 64 and 128
])
def test_f32_groups(counts, H, F, slot):
    S = len(counts) if slot is None else max(slot) + 1
    _run(counts, H, F, slot, S, seed=sum(counts) + H, dtype="f32", tol=1e-4, extra_rows=3)


@pytest.mark.parametrize("counts,H,F", [
    ([129, 192, 193, 224, 225], 256, 512),     # edges of the one-tile modes
    ([160, 512, 200, 416], 512, 416),          # beside experts of two tiles, one of 160 rows
    ([140, 210], 4096, 4096),                  # split along K
])
def test_bf16_one_row_tile_experts(counts, H, F):
    _run(counts, H, F, None, len(counts), seed=sum(counts) + H)


def test_bf16_resident_subset_and_slot_order():
    counts = [100, 200, 50, 300, 10, 0]
    slot = [2, -1, 0, -1, 1, 3]
    _run(counts, 256, 384, slot, 4, seed=21, extra_rows=33)


def test_bf16_nothing_resident():
    _run([10, 20], 64, 64, [-1, -1], 2, seed=22)


def test_shared_experts_as_one_dense_group():
    # two shared experts of width F concatenated along F == one expert of width 2F
    T, H, F = 333, 256, 256
    g = np.random.default_rng(5)
    x = synth.bf16_bits(g.standard_normal((T, H)).astype(np.float32))
    wg, wu, wd = _weights(1, 2 * F, H, seed=5)
    y = ops.expert_ffn(to_dev(x), to_dev(np.array([0, T], np.int32)), to_dev(wg), to_dev(wu),
                       to_dev(wd))
    xs, G, Uw, D = synth.values(x), synth.values(wg)[0], synth.values(wu)[0], synth.values(wd)[0]
    ref = sum(oracle.swiglu(xs, G[s * F:(s + 1) * F], Uw[s * F:(s + 1) * F], D[:, s * F:(s + 1) * F])
              for s in range(2))
    assert rel_max_err(vals(y), ref) <= 1e-2


@pytest.mark.parametrize("name", ["mixtral8x7b_layer", "qwen15_moe_layer"])
def test_full_shape_every_row(name):
    """Full expert shapes (Mixtral: 8192 rows of 4096 over F 14336; Qwen: 32768
    rows over 60 experts of F 1408): every row of y_perm against the oracle,
    which evaluates each expert's rows as one batch."""
    cfg = synth.workload(name)
    seed = cfg["seed"]
    E, H, F, k = cfg["E"], cfg["H"], cfg["F"], cfg["k"]
    T = cfg["T"]
    idx = synth.random_topk_idx(T, E, k, seed=seed, skew=cfg["zipf_bias"])
    counts = np.bincount(idx.ravel(), minlength=E)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offsets[-1])
    inp = synth.layer_inputs(cfg, seed, T=R, parts=("x", "experts"))
    x = inp["x"]
    y = ops.expert_ffn(to_dev(x), to_dev(offsets), to_dev(inp["w_gate"]), to_dev(inp["w_up"]),
                       to_dev(inp["w_down"]))
    got = vals(y)
    ref = np.empty((R, H))
    for e in range(E):
        lo, hi = int(offsets[e]), int(offsets[e + 1])
        if hi > lo:
            ref[lo:hi] = oracle.swiglu(synth.values(x[lo:hi]), synth.values(inp["w_gate"][e]),
                                       synth.values(inp["w_up"][e]),
                                       synth.values(inp["w_down"][e]))
    assert rel_max_err(got, ref) <= 1e-2


@pytest.mark.parametrize("counts,H,F", [
    ([1], 64, 64),                          # one row, one K batch
    ([1, 3, 16, 0, 17, 2], 512, 1408),      # few-row experts beside one with 17 rows
    ([16, 16, 16, 16], 256, 512),           # every expert at the few-row limit
    ([2, 7, 0, 5], 192, 320),               # K = 6 and 10 steps of 32: partial batches
    ([17, 32, 16, 33, 24], 256, 416),       # two-tile experts (17..32 rows) beside the others
    ([31, 1, 29], 160, 96),                 # K = 5 and 3 steps: every wave's range is short
    ([33, 48, 49, 64, 1, 17], 256, 416),    # three and four row tiles beside one and two
    ([65, 80, 96, 40, 3], 192, 320),        # five and six row tiles; K = 6 and 10 steps
    ([70, 2, 50], 160, 96),                 # down projection 160 wide: a half-empty last unit
    ([96, 96], 512, 1408),                  # every expert at the few-row limit (96 rows)
    ([81, 0, 0, 35], 128, 64),              # K = 4 and 2 steps with six and three row tiles
])
def test_bf16_few_rows_per_expert(counts, H, F):
    # in decode-sized batches experts with at most 96 rows take the
    # weight-streaming kernel
    _run(counts, H, F, None, len(counts), seed=sum(counts) + H + F)


@pytest.mark.parametrize("counts,slot,S,extra", [
    ([3, 0, 16, 1, 120, 9], [1, 0, -1, 3, 2, -1], 4, 5),
    ([97, 5, 60, 33], [2, 0, 1, -1], 3, 0),     # 97 rows: one row past the few-row limit
])
def test_bf16_few_rows_resident_subset(counts, slot, S, extra):
    # decode-sized batch (at most 64 rows per expert on average) with one
    # expert of more than one item, all of it for the few-row kernel
    _run(counts, 256, 384, slot, S, seed=23 + sum(counts), extra_rows=extra)


def test_bf16_few_rows_many_experts_subset():
    # decode-sized batch over 256 experts (the list of items built from all of
    # them, sorted by row tiles), a fifth of them not resident, many empty, one
    # of two items
    g = np.random.default_rng(5)
    E = 256
    counts = np.where(g.random(E) < 0.4, 0, g.integers(1, 80, size=E))
    counts[17] = 97
    slot = np.full(E, -1, np.int32)
    res = np.flatnonzero(g.random(E) < 0.8)
    slot[res] = np.arange(len(res), dtype=np.int32)
    assert counts.sum() <= 64 * E
    _run(counts, 64, 96, slot, len(res), seed=5, extra_rows=3)


@pytest.mark.parametrize("counts,slot,H,F", [
    ([130, 5, 60, 33], None, 2048, 2304),
    ([130, 5, 60, 33], [1, -1, 2, 0], 2048, 2304),
    ([5, 97, 0, 60], [-1, 0, 1, -1], 3072, 3072),         # the listed experts hold no rows or no slot
    ([20, 260, 96, 1, 0, 33, 17], None, 1536, 1536),      # a last row tile of 4 rows
    ([260, 20, 96, 1, 5, 33, 288], [0, 1, 2, -1, 3, 4, 5], 1536, 1536),   # of 4 and of 32 rows
])
def test_bf16_few_rows_beside_large_tiles(counts, slot, H, F):
    # decode-sized batch whose weights are too large to be read once more per
    # 96 rows: experts up to 96 rows are listed for the few-row kernel, the
    # others take the large tiles of the same call
    rows = sum(counts)
    counts = counts + [0] * max(0, -(-rows // 64) - len(counts))
    slot = None if slot is None else slot + [-1] * (len(counts) - len(slot))
    assert 96 < rows <= 64 * len(counts) and (rows - 1) // 96 * 6 * H * F > 54e6
    _run(counts, H, F, slot, len(counts) if slot is None else max(slot) + 1, seed=rows + H)


def test_bf16_few_rows_nothing_to_do():
    # decode-sized batch whose experts are all empty or not resident: the
    # launches find no work and the output keeps its sentinel
    _run([0, 5, 0, 9], 128, 256, [0, -1, 1, -1], 2, seed=8, extra_rows=4)


@pytest.mark.parametrize("T,lo,hi", [(24, 1, 16), (100, 17, 32), (160, 33, 64), (256, 49, 96)])
def test_full_shape_decode_batch(T, lo, hi):
    """Decode-sized batch at the full 8-expert shape (H 4096, F 14336): 24,
    100, 160 or 256 tokens with top-2 give at most one, two, four or six
    16-row tiles per expert; every row is checked."""
    cfg = synth.workload("mixtral8x7b_layer")
    E, H, F, k = cfg["E"], cfg["H"], cfg["F"], cfg["k"]
    idx = synth.random_topk_idx(T, E, k, seed=77)
    counts = np.bincount(idx.ravel(), minlength=E)
    assert lo <= counts.max() <= hi
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    R = int(offsets[-1])
    inp = synth.layer_inputs(cfg, 2, T=R, parts=("x", "experts"))
    x = inp["x"]
    y = ops.expert_ffn(to_dev(x), to_dev(offsets), to_dev(inp["w_gate"]), to_dev(inp["w_up"]),
                       to_dev(inp["w_down"]))
    got = vals(y)
    ref = np.empty((R, H))
    for e in range(E):
        lo, hi = int(offsets[e]), int(offsets[e + 1])
        if hi > lo:
            ref[lo:hi] = oracle.swiglu(synth.values(x[lo:hi]), synth.values(inp["w_gate"][e]),
                                       synth.values(inp["w_up"][e]), synth.values(inp["w_down"][e]))
    assert rel_max_err(got, ref) <= 1e-2


def test_bf16_many_experts_large_tiles():
    # 256 experts, a third of them empty and some non-resident, the rest from 1
    # to 700 rows: too many rows for the few-row kernels, so every tile's
    # expert is found among long flat stretches of the row-tile prefix
    g = np.random.default_rng(91)
    E = 256
    counts = np.where(g.random(E) < 0.35, 0, g.integers(1, 700, size=E))
    slot = np.full(E, -1, np.int32)
    res = np.flatnonzero(g.random(E) < 0.8)
    slot[res] = np.arange(len(res), dtype=np.int32)
    assert counts.sum() > 32 * E
    _run(counts, 64, 96, slot, len(res), seed=91)


def _quarter_sum(a):
    """a [..., K] summed as the few-row kernel sums it: four contiguous quarters
    of 32-wide steps, each a float32 chain of whole steps in ascending K, added
    in order."""
    ks = a.shape[-1] // 32
    steps = a.reshape(a.shape[:-1] + (ks, 32)).astype(np.float64).sum(-1)
    per, total = -(-ks // 4), None
    for q in range(4):
        s = np.zeros(a.shape[:-1], np.float32)
        for i in range(q * per, min(ks, (q + 1) * per)):
            s = (s + steps[..., i]).astype(np.float32)
        total = s if total is None else (total + s).astype(np.float32)
    return total


def _order_rows(K, n):
    """n rows [n, K] whose sum depends on the order it is taken in: 2^26 at one
    step, 3 at each of the next two (lost beside it, 8 without it), -2^26 in the
    last quarter; for every step of the first two quarters and a bit beyond, then
    such a pair within one step beside a 3 at another chunk of it."""
    ks = K // 32
    rows = np.zeros((n, K), np.float32)
    last = 32 * (3 * -(-ks // 4))
    for i in range(n):
        s = i // 2 % max(1, min(ks // 2 + 2, last // 32 - 3))
        if i % 2 == 0:
            rows[i, 32 * s] = 2.0 ** 26
            rows[i, 32 * (s + 1) + 9] = rows[i, 32 * (s + 2) + 23] = 3
            rows[i, last] = -2.0 ** 26
        else:
            rows[i, 32 * s] = 2.0 ** 26
            rows[i, 32 * s + 8] = 3
            rows[i, 32 * (s + 1)] = -2.0 ** 26
    return rows


@pytest.mark.parametrize("K", [1408, 1024, 2080, 480])    # quarters of 11, 8, 17 and 4 steps
@pytest.mark.parametrize("counts,N", [
    ([3], 128), ([40], 128),                              # 16-column units
    ([1] * 39 + [18], 128),                               # wide units of eight waves
    ([1, 17, 33, 49, 65, 81] + [1] * 134, 128),           # wide units of four waves
])
def test_bf16_few_row_sum_order(counts, N, K):
    # the sum's order is the same whichever units compute it, exactly: up
    # projection (x of ones), then down projection (activations of ones)
    E, rows = len(counts), _order_rows(K, N)
    want = _quarter_sum(rows)
    assert (want == 0).any() and (want != 0).any()
    offsets = to_dev(np.concatenate([[0], np.cumsum(counts)]).astype(np.int32))
    R = sum(counts)
    slot = to_dev(np.zeros(E, np.int32))                  # every expert: the same weights
    bf = lambda a: to_dev(synth.bf16_bits(np.asarray(a, np.float32)))[None]
    one = np.zeros((N, K), np.float32)
    one[:, 0] = 1
    pick = np.zeros((K, N), np.float32)
    pick[np.arange(N), np.arange(N)] = 1
    y = vals(ops.expert_ffn(bf(np.ones((R, K)))[0], offsets, bf(rows), bf(one), bf(pick),
                            slot_of_expert=slot))
    act = np.where(want > 80, want, want / (1 + np.exp(-np.minimum(want, 80))))
    ref = synth.values(synth.bf16_bits(act.astype(np.float32)))
    np.testing.assert_allclose(y[:, :N], np.broadcast_to(ref, (R, N)), rtol=2.0 ** -7, atol=0)
    gate, up, x = np.zeros((K, N)), np.zeros((K, N)), np.zeros((R, N))
    gate[:, 0] = 64                                       # silu(64) / 64 = 1
    up[:, 0] = 2.0 ** -6
    x[:, 0] = 1
    y = vals(ops.expert_ffn(bf(x)[0], offsets, bf(gate), bf(up), bf(rows), slot_of_expert=slot))
    ref = synth.values(synth.bf16_bits(want))
    np.testing.assert_array_equal(y, np.broadcast_to(ref, (R, N)))


@pytest.mark.parametrize("counts", [[3, 40, 1], [300, 20, 513]])     # few rows; large tiles
@pytest.mark.parametrize("which", ["x", "w_gate", "w_down"])
def test_bf16_operands_off_16_bytes(which, counts):
    # an operand that starts 8 bytes past a 16-byte boundary takes the general
    # kernels; bound of the other bf16 cases
    H, F, S = 128, 192, len(counts)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    x = _rows(offsets[-1], H, 3)
    ws = dict(zip(("w_gate", "w_up", "w_down"), _weights(S, F, H, 3)))
    dev = dict({n: to_dev(w) for n, w in ws.items()}, x=to_dev(x))
    buf = torch.zeros(dev[which].numel() + 4, dtype=torch.bfloat16, device="cuda:0")
    buf[4:] = dev[which].reshape(-1)
    dev[which] = buf[4:].view(dev[which].shape)
    assert dev[which].data_ptr() % 16 == 8
    y = ops.expert_ffn(dev["x"], to_dev(offsets), dev["w_gate"], dev["w_up"], dev["w_down"])
    ref, _ = oracle.expert_ffn(synth.values(x), offsets, np.arange(S),
                               *(synth.values(ws[n]) for n in ("w_gate", "w_up", "w_down")))
    assert rel_max_err(vals(y), ref) <= 1e-2
