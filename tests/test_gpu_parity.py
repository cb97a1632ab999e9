"""GPU parity: the HIP library, called through its C ABI, against the CPU oracle on the
same seeded inputs.  Integer outputs (selected experts, slots, histogram, offsets,
permutation, gathered rows) must match bit for bit; floating-point outputs within

    bf16 storage:  |got - ref| <= 1e-2 + 2e-2 |ref|
    fp32 storage:  |got - ref| <= 1e-4 |ref| + 1e-4 rms(ref)

Small cases compare every element; the full benchmark shapes compare every integer output,
every row of the smallest and the largest slot, and 512 seeded tokens.
"""
import ctypes

import numpy as np
import pytest
import torch

from paper_2505_06481_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mm():
    from paper_2505_06481_amd import mmoe
    mmoe.lib()
    assert torch.cuda.is_available()
    return mmoe


@pytest.fixture(scope="module")
def gc():
    import gpu_common
    return gpu_common


def staged_vs_oracle(mm, gc, oracle, cfg, inp=None, tile_rows=0):
    """Run the four stages one by one through the C ABI and compare each with the oracle."""
    print(f"case {cfg.name} T={cfg.T} d={cfg.d_model} f={cfg.d_ff} V={cfg.V} E={cfg.E} k={cfg.top_k} "
          f"{cfg.dtype} {cfg.act} seed={cfg.seed}", flush=True)
    case = gc.DeviceCase(cfg, inp, tile_rows=tile_rows)
    inp, sh, dt = case.inp, case.shape, cfg.dtype
    ref = oracle.layer_forward(inp, cfg.top_k, dt, cfg.act, gate=cfg.gate)

    idx, w = mm.route(sh, case.X, case.vid, case.Wr, case.br)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), ref["topk_idx"]), "selected experts differ"
    np.testing.assert_allclose(w.cpu().numpy(), ref["topk_w"], rtol=2e-6, atol=1e-7)

    slot, counts, offsets, perm, inv, Xg = mm.remap_permute(sh, case.X, case.vid, idx, case.M, case.ws)
    torch.cuda.synchronize()
    for name, t in (("slot", slot), ("counts", counts), ("offsets", offsets), ("perm", perm), ("inv_perm", inv)):
        assert np.array_equal(t.cpu().numpy(), ref[name]), name
    assert np.array_equal(gc.bits(Xg), ref["Xg"]), "gathered rows differ"

    Yg = mm.expert_ffn(sh, Xg, offsets, case.W1p, case.W3p, case.W2p, case.ws)
    torch.cuda.synchronize()
    gc.assert_close(gc.to_np64(Yg), ref["Yg"], dt, "Yg")

    Y = mm.combine(sh, Yg, inv, w)
    torch.cuda.synchronize()
    gc.assert_close(gc.to_np64(Y), ref["Y"], dt, "Y (staged)")

    Y2 = case.forward()
    torch.cuda.synchronize()
    assert torch.equal(Y2, Y), "fused entry point differs from the staged path"
    Y3 = case.forward()
    torch.cuda.synchronize()
    assert torch.equal(Y3, Y2), "two runs differ: the path is not deterministic"
    return case, ref


SMALL = [
    # weight-streaming kernels (few rows per slot; the two fp32 cases with more have matrix-core tiles), ragged
    # row counts, several 16-row blocks
    synth.Config("s_bf16_swiglu", 45, 512, 768, 3, 4, 2, "bf16", "swiglu", seed=1),
    synth.Config("s_bf16_relu", 70, 256, 512, 2, 8, 1, "bf16", "relu", seed=2),
    synth.Config("s_f32_relu", 33, 256, 512, 2, 4, 1, "f32", "relu", seed=3),
    synth.Config("s_f32_swiglu", 50, 512, 256, 2, 4, 2, "f32", "swiglu", seed=4, bias_alpha=0.5),
    synth.Config("s_f32_many_rows", 300, 256, 256, 1, 2, 1, "f32", "relu", seed=5),     # fp32 matrix-core tiles
    # few rows per slot on average, but a biased router fills one slot beyond a 32-row pass
    synth.Config("s_bf16_skewed_passes", 100, 512, 256, 1, 8, 1, "bf16", "swiglu", seed=26, bias_alpha=3.0),
    # matrix-core tiled kernels (many rows per slot), ragged tails, several tiles per slot
    synth.Config("t_bf16_swiglu", 700, 512, 768, 2, 4, 2, "bf16", "swiglu", seed=6),
    synth.Config("t_bf16_relu", 900, 256, 512, 3, 4, 1, "bf16", "relu", seed=7),
    synth.Config("t_bf16_skew", 1500, 256, 256, 4, 8, 2, "bf16", "swiglu", seed=8, vid_mode="zipf",
                 bias_alpha=1.0),
    synth.Config("t_bf16_topk_all", 400, 256, 256, 1, 3, 3, "bf16", "swiglu", seed=9),   # top_k = E
    # batches large enough for the wavefront-per-token router, odd expert counts, fp32 and bf16
    synth.Config("r_f32_odd_e", 2100, 512, 256, 2, 5, 2, "f32", "swiglu", seed=17, bias_alpha=0.7),
    synth.Config("r_bf16_odd_e", 2060, 1536, 256, 3, 7, 2, "bf16", "relu", seed=18, bias_alpha=0.3),
    # one pick per token (the down product writes the layer's output rows itself) on the matrix-core kernels, fp32
    # and, with many slots, bf16; both tile heights are t_bf16_relu.  (Streaming after the grouping: STREAMED.)
    synth.Config("k1_f32_grouped", 1500, 256, 512, 2, 6, 1, "f32", "gelu", seed=27),
    synth.Config("k1_bf16_grouped_stream", 1300, 512, 256, 8, 16, 1, "bf16", "relu", seed=28, share_prob=0.1),
    synth.Config("k1_bf16_long_k", 1100, 2048, 256, 2, 4, 1, "bf16", "relu", seed=29),     # tall-tile shape rule
]


STREAMED = [
    # more pairs than the expert kernels group themselves: the grouping kernel, then the streaming kernels through perm
    # (experts of over 4 Mi elements, many slots; fp32 with many slots), one and two picks per token
    synth.Config("stream_grouped_bf16_k1", 1060, 256, 16640, 2, 64, 1, "bf16", "relu", seed=70, share_prob=0.9),
    synth.Config("stream_grouped_bf16_k2", 530, 2048, 2304, 2, 64, 2, "bf16", "swiglu", seed=71, share_prob=0.9),
    synth.Config("stream_grouped_f32_k1", 1300, 256, 512, 8, 16, 1, "f32", "gelu", seed=72, share_prob=0.1),
    synth.Config("stream_grouped_f32_k2_two_chunks", 1200, 256, 256, 64, 16, 2, "f32", "relu", seed=73, share_prob=0.1),
    # few slots: more rows per slot than elsewhere, up to the line
    synth.Config("stream_few_slots_k1", 128, 256, 512, 1, 4, 1, "bf16", "gelu", seed=77, gate="all"),
    synth.Config("stream_few_slots_k2", 92, 512, 768, 1, 8, 2, "bf16", "swiglu", seed=78),
    # fp32: a biased router fills one slot beyond a 32-row pass
    synth.Config("stream_f32_skewed_passes", 90, 512, 256, 1, 8, 1, "f32", "swiglu", seed=74, bias_alpha=3.0),
    # several hundred slots, most of them empty, on the kernels that group the pairs themselves
    synth.Config("stream_many_slots", 250, 256, 256, 64, 16, 2, "bf16", "swiglu", seed=75, share_prob=0.1),
]


@pytest.mark.parametrize("cfg", STREAMED, ids=lambda c: c.name)
def test_streaming_kernels(mm, gc, oracle, cfg):
    """Every stage and the fused call where the dispatch streams: the plan is asserted, so that a dispatch line that
    moves does not take the case to the other kernels unseen."""
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg)
    assert mm.expert_plan(case.shape) == (True, 32)
    if "grouped" in cfg.name:
        assert cfg.P > 1024
    if "passes" in cfg.name:
        assert ref["counts"].max() > 32


@pytest.mark.parametrize("cfg", SMALL, ids=lambda c: c.name)
def test_small_cases_every_stage(mm, gc, oracle, cfg):
    staged_vs_oracle(mm, gc, oracle, cfg)


@pytest.mark.parametrize("rows", [256, 128])
@pytest.mark.parametrize("cfg", [c for c in SMALL if c.name.startswith("t_")], ids=lambda c: c.name)
def test_both_tile_heights(mm, gc, oracle, cfg, rows):
    """The matrix-core kernels at a forced tile height (by shape these small batches would only
    ever get the 128-row tiles): every stage against the oracle, ragged last tiles of 1..8 sub-tiles."""
    staged_vs_oracle(mm, gc, oracle, cfg, tile_rows=rows)


@pytest.mark.parametrize("rows", [256, 128])
@pytest.mark.parametrize("act,k", [("swiglu", 1), ("relu", 1), ("gelu", 2)])
def test_tiled_row_remainders(mm, gc, oracle, act, k, rows):
    """Every number of 16-row fragments a tile can end in, full and one-row remainders, one and two
    tiles in the slot: a single slot (two when k = 2) that holds T rows.  A cut at a wrong row or lane
    shows as a whole wrong row, so the tolerance is the storage type's."""
    for T in (33, 47, 48, 49, 65, 97, 112, 128, 129, 161, 193, 225, 241, 255, 256, 257, 300):
        staged_vs_oracle(mm, gc, oracle, synth.Config(f"rem_{act}_{T}", T, 256, 256, 1, k, k, "bf16", act, seed=400 + T),
                         tile_rows=rows)


@pytest.mark.parametrize("act,k,d,f", [("swiglu", 1, 256, 512), ("relu", 1, 768, 256), ("gelu", 2, 512, 1280)])
def test_tiled_f32_row_remainders(mm, gc, oracle, act, k, d, f):
    """Every number of 16-row fragments of the fp32 tiles, full and one-row remainders, one to three tiles in
    a slot, one and several chains of the reduction: a single slot (two when k = 2) that holds T rows."""
    for T in (25, 32, 33, 48, 49, 64, 65, 80, 81, 96, 97, 128, 129, 192, 193, 200, 300):
        cfg = synth.Config(f"rem32_{act}_{T}", T, d, f, 1, k, k, "f32", act, seed=800 + T)
        case, _ = staged_vs_oracle(mm, gc, oracle, cfg)
        assert mm.expert_plan(case.shape) == (False, 96)


def _parts_case(mm, oracle, act, d, f, seed, counts=None):
    """A grouped batch in fp32 whose slots hold every number of rows at which a tile's fragments change; products of 512
    outputs and more and the gated one run on bf16 parts, those of 256 on the fp32 instruction."""
    counts = counts or [1, 15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 81, 95, 96, 97, 0, 129, 191, 193, 289]
    rng = np.random.default_rng(seed)
    S, P = len(counts), sum(counts)
    assert P >= 40 * S
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    Xg = rng.standard_normal((P, d)).astype(np.float32)
    W1, W2 = (0.05 * rng.standard_normal((S, a, b)).astype(np.float32) for a, b in ((d, f), (f, d)))
    W3 = 0.05 * rng.standard_normal((S, d, f)).astype(np.float32) if act == "swiglu" else None
    shape = mm.make_shape(P, d, f, 1, S, S, 1, "f32", act)
    assert mm.expert_plan(shape) == (False, 96)
    return shape, offsets, Xg, W1, W3, W2


# few slots, so that both products of 2048 x 2048 are little enough for eight wavefronts to a tile
AHEAD_ROWS = [1, 33, 49, 95, 112, 161, 193]


def _ahead(dispatch_rule, shape):
    return dispatch_rule("f32_ahead", shape, shape.d_ff, True), dispatch_rule("f32_ahead", shape, shape.d_model, False)


def _parts_run(mm, shape, offsets, Xg, W1, W3, W2):
    dev = lambda a: None if a is None else torch.from_numpy(a).cuda()
    packed = mm.pack_weights(shape, dev(W1), dev(W3), dev(W2))
    Y = mm.expert_ffn(shape, dev(Xg), dev(offsets), *packed, mm.alloc_workspace(shape))
    torch.cuda.synchronize()
    return Y.cpu().numpy()


@pytest.mark.parametrize("act,d,f,counts,ahead", [
    ("relu", 256, 768, None, (False, False)), ("gelu", 768, 256, None, (False, False)), ("swiglu", 512, 768, None, (False, False)),
    ("swiglu", 768, 1024, None, (False, False)), ("relu", 768, 2560, None, (False, False)),
    ("gelu", 512, 1024, None, (False, True)), ("swiglu", 512, 1280, None, (False, True)),      # eight wavefronts to a tile
    ("relu", 2048, 2048, AHEAD_ROWS, (True, True)), ("gelu", 1024, 2048, AHEAD_ROWS, (True, False))])
def test_f32_products_on_bf16_parts(mm, gc, oracle, dispatch_rule, act, d, f, counts, ahead):
    """Rows at the edges of the tiles, one and several chains of the reduction, either product on either kernel.
    The tolerance on the 2-norm is what the fp32 instruction gives (measured: 2.2e-7 to 2.9e-7 here, 3.5e-7 to 5.2e-7
    there), so that parts of too few bits, or a missing one (2^-16), do not pass."""
    shape, offsets, Xg, W1, W3, W2 = _parts_case(mm, oracle, act, d, f, seed=d + f, counts=counts)
    assert _ahead(dispatch_rule, shape) == ahead
    assert dispatch_rule("f32_in_parts", shape, f, act == "swiglu") == (f > 256 or act == "swiglu")
    assert dispatch_rule("f32_in_parts", shape, d, False) == (d > 256 and (counts is None or d == 2048))
    got = _parts_run(mm, shape, offsets, Xg, W1, W3, W2).astype(np.float64)
    ref = oracle.expert_ffn(Xg, offsets, W1, W3, W2, "f32", act)
    gc.assert_close(got, ref, "f32", "Yg")
    assert np.linalg.norm(got - ref) <= 6e-7 * np.linalg.norm(ref)


@pytest.mark.parametrize("d,f,counts", [(768, 768, None), (2048, 2048, AHEAD_ROWS)])
def test_f32_parts_of_numbers_that_are_not_finite(mm, gc, oracle, dispatch_rule, d, f, counts):
    """Infinities, NaN and numbers that round to an infinity in bf16 give what fp32 gives, and only in their own
    rows and features, with four wavefronts to a tile and with eight."""
    shape, offsets, Xg, W1, _, W2 = _parts_case(mm, oracle, "gelu", d, f, seed=5, counts=counts)
    assert _ahead(dispatch_rule, shape) == (counts is not None,) * 2
    W1[:, 700, :] = np.abs(W1[:, 700, :]) * 1e-3 + 1e-6  # the large entry's products: finite, of one sign
    rows = [3, 40, 200, len(Xg) - 1]
    others = ~np.isin(np.arange(len(Xg)), rows)
    clean = np.where(others[:, None], Xg, np.float32(0))
    Xg[rows, 700] = np.inf, -np.inf, np.nan, np.finfo(np.float32).max
    got = _parts_run(mm, shape, offsets, Xg, W1, None, W2)
    assert np.array_equal(got[others], _parts_run(mm, shape, offsets, clean, W1, None, W2)[others])
    with np.errstate(over="ignore", invalid="ignore"):
        want = oracle.expert_ffn(Xg, offsets, W1, None, W2, "f32", "gelu").astype(np.float32)
    for r in rows:
        nan, fin = np.isnan(want[r]), np.isfinite(want[r])
        assert np.array_equal(np.isnan(got[r]), nan), r
        assert np.array_equal(got[r][~nan & ~fin], want[r][~nan & ~fin]), r
        # the error of a sum of both signs goes with its terms: of 2048 sums the least may be 2000 times smaller than the largest, with
        # an error of 5e-7 of that
        least = 0.0 if counts is None else 1e-6 * np.abs(want[r][fin]).max(initial=0.0)
        assert np.allclose(got[r][fin], want[r][fin], rtol=1e-4, atol=max(1e-8, least)), r
    W2[5, 10, 100] = np.inf  # one feature of one slot, on the other operand
    got = _parts_run(mm, shape, offsets, clean, W1, None, W2)
    hit = np.zeros(got.shape, bool)
    hit[offsets[5]:offsets[6], 100] = True
    assert np.isfinite(got[~hit]).all() and not np.isfinite(got[hit]).any()


PARTS_LAYERS = [
    # one pick per token (the down product on parts writes the layer's rows), either gate; several picks; token rows read
    # through the permutation by every up product
    synth.Config("parts_k1_relu", 900, 768, 1024, 2, 8, 1, "f32", "relu", seed=95, share_prob=0.0),
    synth.Config("parts_k1_gelu_all", 1001, 1024, 768, 2, 8, 1, "f32", "gelu", seed=96, share_prob=0.0, gate="all"),
    synth.Config("parts_k1_swiglu", 1500, 768, 512, 2, 6, 1, "f32", "swiglu", seed=97, share_prob=0.0, bias_alpha=0.5),
    synth.Config("parts_k2_relu", 620, 1024, 1280, 2, 8, 2, "f32", "relu", seed=98, share_prob=0.0),
    # eight wavefronts to a tile in both products
    synth.Config("parts_ahead_gelu_all", 640, 2048, 2048, 1, 7, 1, "f32", "gelu", seed=99, gate="all"),
]


@pytest.mark.parametrize("cfg", PARTS_LAYERS, ids=lambda c: c.name)
def test_f32_layers_on_bf16_parts(mm, gc, oracle, dispatch_rule, cfg):
    """Every stage and the fused call; both products on parts."""
    case, _ = staged_vs_oracle(mm, gc, oracle, cfg)
    assert dispatch_rule("f32_in_parts", case.shape, cfg.d_ff, cfg.act == "swiglu")
    assert dispatch_rule("f32_in_parts", case.shape, cfg.d_model, False)
    assert ("ahead" in cfg.name) == (_ahead(dispatch_rule, case.shape) == (True, True))


@pytest.mark.parametrize("cfg", PARTS_LAYERS[1:3] + PARTS_LAYERS[4:], ids=lambda c: c.name)
def test_f32_layers_on_bf16_parts_with_weights_that_are_not_finite(mm, gc, oracle, dispatch_rule, cfg):
    """Infinite weights, and large ones that are finite in fp32 only, in the plain factor of the gated product and in the
    down product that writes the layer's rows: what fp32 gives, and only in the tokens and features they reach."""
    inp = synth.make_inputs(cfg)
    clean = gc.DeviceCase(cfg, inp).forward()
    torch.cuda.synchronize()
    inp = dict(inp, W2=inp["W2"].copy())
    inp["W2"][5, 10, 100] = np.inf
    inp["W2"][6, 20, 200] = -np.finfo(np.float32).max
    if cfg.act == "swiglu":
        inp["W3"] = inp["W3"].copy()
        inp["W3"][4, 30, 300] = -np.inf
    case = gc.DeviceCase(cfg, inp)
    assert _ahead(dispatch_rule, case.shape)[1] == ("ahead" in cfg.name)
    got = case.forward()
    torch.cuda.synchronize()
    got, clean = got.cpu().numpy(), clean.cpu().numpy()
    with np.errstate(over="ignore", invalid="ignore"):
        ref = oracle.layer_forward(inp, 1, "f32", cfg.act, gate=cfg.gate)
        want = (ref["Yg"].astype(np.float32)[ref["inv_perm"]] * ref["topk_w"]).astype(np.float32)  # Yg is fp32
    slot = ref["slot"]
    hit = np.zeros(got.shape, bool)
    hit[slot == 5, 100] = hit[slot == 6, 200] = True
    if cfg.act == "swiglu":
        hit[slot == 4] = True
    assert hit.any() and np.array_equal(got[~hit], clean[~hit])
    assert np.array_equal(np.isnan(got), np.isnan(want))
    inf = np.isinf(want)
    assert inf.any() and np.array_equal(got[inf], want[inf])
    fin = hit & np.isfinite(want)
    assert fin.any()
    gc.assert_close_f32(got[fin].astype(np.float64), want[fin].astype(np.float64), "features of the large weight")


@pytest.mark.parametrize("act,d,f,x_exp,w1_exp,w2_exp", [
    ("relu", 2048, 2048, -118, 0, 0), ("gelu", 2048, 2048, 0, 0, -118), ("relu", 2048, 2048, 0, -60, -55),   # eight wavefronts to a tile
    ("relu", 2048, 2048, -118, 110, 0), ("relu", 2048, 2048, 106, -100, 0),
    ("relu", 768, 768, -110, 0, 0), ("gelu", 768, 768, -118, 0, 0), ("relu", 768, 768, 0, -118, 0),
    ("relu", 768, 768, 0, 0, -118), ("relu", 768, 768, -58, -55, 0), ("relu", 768, 768, 0, -60, -55),
    ("relu", 768, 768, -118, 110, 0), ("swiglu", 512, 768, -58, -4, 0), ("swiglu", 512, 768, 0, 0, -118),
    ("relu", 768, 768, 106, -100, 0), ("relu", 768, 768, 60, 40, -90)])
def test_f32_parts_keep_the_range_of_fp32(mm, gc, oracle, dispatch_rule, act, d, f, x_exp, w1_exp, w2_exp):
    """Operands and products of any size that fp32 holds with all its bits, in either operand of either product, keep
    the accuracy of ordinary ones: the bound is test_f32_products_on_bf16_parts's.  (The last two, and the fifth: operands and sums beyond
    what the scaled parts hold, on the fp32 instruction, whose relative error does not depend on the scale.  It adds 64 products
    one by one and then the chains, about 3e-8 (sqrt(64 / 2) + sqrt(chains / 2)) of the sum: with 32 chains for 12 a fifth more.)"""
    shape, offsets, Xg, W1, W3, W2 = _parts_case(mm, oracle, act, d, f, seed=31, counts=AHEAD_ROWS if d == 2048 else None)
    assert _ahead(dispatch_rule, shape) == (d == 2048,) * 2
    Xg, W1, W2 = (a * np.float32(2.0 ** e) for a, e in ((Xg, x_exp), (W1, w1_exp), (W2, w2_exp)))
    W3 = None if W3 is None else W3 * np.float32(2.0 ** w1_exp)
    got = _parts_run(mm, shape, offsets, Xg, W1, W3, W2).astype(np.float64)
    ref = oracle.expert_ffn(Xg, offsets, W1, W3, W2, "f32", act)
    scale = 1.0 / np.abs(ref).max()
    bound = 7.2e-7 if d == 2048 and x_exp == 106 else 6e-7
    assert np.linalg.norm((got - ref) * scale) <= bound * np.linalg.norm(ref * scale)


@pytest.mark.parametrize("dtype,act,k,T,d,f", [("bf16", "relu", 1, 100, 2048, 2048), ("bf16", "swiglu", 2, 60, 2048, 1536),
                                               ("f32", "gelu", 1, 95, 1024, 2304), ("f32", "swiglu", 2, 47, 1536, 1024)])
def test_streaming_slots_of_several_passes_in_large_pools(mm, gc, oracle, dispatch_rule, dtype, act, k, T, d, f):
    """Where weights are read past the caches, beside slots of one pass: slots of two passes and more, read through them."""
    cfg = synth.Config(f"passes_{dtype}_{act}", T, d, f, 1, 8, k, dtype, act, seed=90, bias_alpha=2.0)
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg)
    assert mm.expert_plan(case.shape) == (True, 32) and dispatch_rule("past_the_caches", case.shape)
    assert ref["counts"].max() > 32 and (ref["counts"] > 0).sum() > (ref["counts"] > 32).sum()


PER_TOKEN, TOKENS, GROUPS, TILES = range(4)  # router kernels: a workgroup per token, a wavefront per token, a workgroup per four, tiles


@pytest.fixture(scope="module")
def router_kernel(dispatch_rule):
    return lambda shape: dispatch_rule("route_kernel_for", shape, restype=ctypes.c_int)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_router_with_every_remainder_of_experts(mm, gc, oracle, router_kernel, dtype):
    """Numbers of experts around the four whose sums share a butterfly and around a wavefront's lanes, on each router
    kernel (a workgroup per token, a wavefront per token, a workgroup per four): the oracle's picks, and its coefficients to rounding.
    (Nine variants: too many for tiles.)"""
    for T, d, kernel in ((70, 512, PER_TOKEN), (2050, 256, TOKENS), (2051, 768, TOKENS), (771, 4096, GROUPS), (2100, 2304, GROUPS)):
        for E in (1, 2, 3, 4, 5, 8, 9, 17, 33, 64, 67):
            cfg = synth.Config(f"route_{dtype}_{T}_{d}_{E}", T, d, 256, 9, E, min(E, 4), dtype, "relu", seed=1500 + T + E, bias_alpha=0.5, gate="all")
            inp = synth.make_inputs(cfg, weights=False)
            shape = mm.make_shape(T, d, 256, 9, E, E, cfg.top_k, dtype, "relu", gate="all")
            few = dtype == "f32" and d == 4096 and E < 5  # long rows of fp32 and little to score
            assert router_kernel(shape) == (PER_TOKEN if few else kernel), (T, d, E)
            idx, w = mm.route(shape, gc.to_dev(inp["X"], dtype), torch.from_numpy(inp["vid"]).cuda(), gc.to_dev(inp["Wr"], dtype),
                              torch.from_numpy(inp["br"]).cuda())
            torch.cuda.synchronize()
            idx_ref, w_ref, _ = oracle.route(inp["X"], inp["vid"], inp["Wr"], inp["br"], cfg.top_k, dtype, gate="all")
            assert np.array_equal(idx.cpu().numpy(), idx_ref), (T, d, E)
            np.testing.assert_allclose(w.cpu().numpy(), w_ref, rtol=2e-6, atol=1e-7)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_router_kernels_agree_bit_for_bit(mm, gc, router_kernel, dtype):
    """Batches on a wavefront per token (rows of the router in registers four and two at a time) and on groups of four, and their
    parts on a workgroup per token: the same picks and the same bits of every coefficient.  (Nine variants: too many for tiles.)"""
    for T, d, groups in ((2050, 256, False), (2049, 768, False), (2049, 2048, False), (2050, 3072, False), (2050, 4096, False),
                         (771, 4096, True), (2053, 2304, True), (2051, 3072, True)):
        for E in ((1, 2, 3, 5, 6, 7, 9) if not groups else (17, 66) if d == 3072 else (6, 7, 33)):
            cfg = synth.Config(f"bits_{dtype}_{T}_{d}_{E}", T, d, 256, 9, E, min(E, 4), dtype, "relu", seed=1700 + T + E, bias_alpha=0.5, gate="all")
            inp = synth.make_inputs(cfg, weights=False)
            X, Wr, br = gc.to_dev(inp["X"], dtype), gc.to_dev(inp["Wr"], dtype), torch.from_numpy(inp["br"]).cuda()
            vid = torch.from_numpy(inp["vid"]).cuda()
            make = lambda n: mm.make_shape(n, d, 256, 9, E, E, cfg.top_k, dtype, "relu", gate="all")
            assert router_kernel(make(T)) == (GROUPS if groups else TOKENS), (T, d, E)
            idx, w = mm.route(make(T), X, vid, Wr, br)
            for t0 in range(0, T, 700):
                n = min(700, T - t0)
                assert router_kernel(make(n)) == PER_TOKEN, (n, d, E)
                part_idx, part_w = mm.route(make(n), X[t0:t0 + n], vid[t0:t0 + n], Wr, br)
                assert torch.equal(part_idx, idx[t0:t0 + n]) and torch.equal(part_w, w[t0:t0 + n]), (T, d, E, t0)


@pytest.mark.parametrize("rows", [256, 128])
def test_down_tiles_in_runs(mm, gc, oracle, dispatch_rule, rows):
    """Down products whose tiles may go to the XCDs in runs (128-row tiles: do): fewer tiles than XCDs, numbers that do not
    divide among them, few and many slots, equally and unequally used, and as many panels as XCDs or more."""
    for T, V, E, k, d, f, alpha in ((65, 1, 1, 1, 256, 256, 0.0), (300, 1, 3, 1, 256, 512, 0.0), (1100, 3, 16, 1, 768, 256, 3.0),
                                    (800, 1, 40, 2, 512, 256, 2.0), (1300, 2, 6, 2, 2304, 256, 0.5), (1100, 1, 5, 1, 2048, 256, 0.0)):
        cfg = synth.Config(f"runs_{T}_{d}", T, d, f, V, E, k, "bf16", "relu" if k == 1 else "swiglu", seed=1400 + T, bias_alpha=alpha)
        case, _ = staged_vs_oracle(mm, gc, oracle, cfg, tile_rows=rows)
        assert mm.expert_plan(case.shape) == (False, rows)
        if rows == 128:
            assert dispatch_rule("xcd_runs", case.shape, 1, restype=ctypes.c_int) == 1


@pytest.mark.parametrize("T,d,V,E,k,gate", [
    (2307, 4096, 1, 8, 2, "selected"), (2369, 4096, 3, 7, 7, "all"), (2500, 2816, 8, 8, 1, "all"),   # a group to a wavefront
    (2700, 2048, 8, 9, 2, "selected"), (2570, 3072, 2, 16, 4, "all"),                                # to a workgroup, with every number of wavefronts
    (1999, 2048, 3, 17, 8, "selected"), (644, 2560, 5, 32, 2, "all"), (641, 3072, 3, 33, 4, "all"), (650, 1280, 2, 67, 3, "selected"),
    (3649, 512, 3, 66, 4, "all"), (3586, 256, 2, 255, 8, "selected")])
def test_router_tiles_agree_bit_for_bit(mm, gc, router_kernel, T, d, V, E, k, gate):
    """Groups of four tokens of a variant, the last ones of a chunk of 64 not full, against the parts of the batch on the kernels
    for fewer tokens: the same picks, the same bits of every coefficient, and in the layer the same slots."""
    cfg = synth.Config(f"tiles_{T}_{d}_{E}", T, d, 256, V, E, k, "bf16", "relu", seed=1900 + T + E, bias_alpha=0.5, gate=gate)
    inp = synth.make_inputs(cfg, weights=False)
    X, Wr, br = gc.to_dev(inp["X"], "bf16"), gc.to_dev(inp["Wr"], "bf16"), torch.from_numpy(inp["br"]).cuda()
    vid = torch.from_numpy(inp["vid"]).cuda()
    make = lambda n: mm.make_shape(n, d, 256, V, E, E, k, "bf16", "relu", gate=gate)
    assert router_kernel(make(T)) == TILES
    idx, w = mm.route(make(T), X, vid, Wr, br)
    none, _ = mm.route(make(T), X, vid, Wr)
    for t0 in range(0, T, 300):
        n = min(300, T - t0)
        assert router_kernel(make(n)) == PER_TOKEN
        part_idx, part_w = mm.route(make(n), X[t0:t0 + n], vid[t0:t0 + n], Wr, br)
        assert torch.equal(part_idx, idx[t0:t0 + n]) and torch.equal(part_w, w[t0:t0 + n]), t0
        assert torch.equal(mm.route(make(n), X[t0:t0 + n], vid[t0:t0 + n], Wr)[0], none[t0:t0 + n]), t0


@pytest.mark.parametrize("T,E,k,d", [(2400, 8, 1, 3072), (2600, 16, 2, 2304), (650, 32, 2, 2304), (650, 64, 3, 1280), (4200, 48, 1, 1024)])
def test_layer_behind_router_tiles(mm, gc, oracle, router_kernel, T, E, k, d):
    """Every launch of the tile kernel looks the slots up: a group to a wavefront, and to a workgroup with four and eight wavefronts of
    four and of eight experts."""
    cfg = synth.Config(f"tiles_layer_{T}_{E}", T, d, 256, 3, E, k, "bf16", "relu", seed=2000 + T, bias_alpha=0.5)
    case, _ = staged_vs_oracle(mm, gc, oracle, cfg)
    assert router_kernel(case.shape) == TILES


def expert_lists(mm, gc, oracle, d, f, act, counts, tile_rows=0):
    """The expert stage on slots of `counts` rows, against the oracle; its shape and the tile lists it has left in the
    workspace behind H (int32)."""
    rng = np.random.default_rng(sum(counts) + d)
    S, P = len(counts), sum(counts)
    offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
    draw = lambda sigma, *shape: synth.f32_to_bf16_bits(sigma * rng.standard_normal(shape, dtype=np.float32))
    Xg, W1, W2 = draw(1.0, P, d), draw(0.02, S, d, f), draw(0.02, S, f, d)
    shape = mm.make_shape(P, d, f, 1, S, S, 1, "bf16", act, tile_rows=tile_rows)
    dev = lambda a: gc.to_dev(a, "bf16")
    ws = mm.alloc_workspace(shape)
    Yg = mm.expert_ffn(shape, dev(Xg), torch.from_numpy(offsets).cuda(), *mm.pack_weights(shape, dev(W1), None, dev(W2)), ws)
    torch.cuda.synchronize()
    gc.assert_close(gc.to_np64(Yg), oracle.expert_ffn(Xg, offsets, W1, None, W2, "bf16", act), "bf16", "Yg")
    at = -(-P * f * 2 // 256) * 256
    return shape, ws[at:at + (ws.numel() - at) // 4 * 4].view(torch.int32).cpu().numpy()


def rounds(tiles, conc):
    """Rounds that an XCD takes for its tiles, so many at a time (32 of 256 rows, 64 of 128)."""
    return -(-int(tiles) // conc)


def in_runs(per_xcd):
    share = -(-int(per_xcd.sum()) // 8)
    return list(per_xcd) == [min(share, max(int(per_xcd.sum()) - x * share, 0)) for x in range(8)]


@pytest.mark.parametrize("d,counts", [
    (256, [65]), (256, [0, 0, 40, 0, 200, 1, 0]),                                   # fewer tiles than XCDs; empty slots at either end
    (768, [0, 1500, 3, 0, 40, 260, 90, 1, 33, 0, 0]), (1280, [5, 0, 700, 129, 64]),  # six and ten panels, very unequal slots
    (1024, [300, 20, 0, 500, 31]), (2048, [0, 128, 400, 257, 90, 0]),                # panels that divide among the XCDs
    (256, [9000, 17000, 300, 12500, 0])])                                            # one panel a slot
def test_128_row_down_tiles_in_runs(mm, gc, oracle, dispatch_rule, d, counts):
    """Every XCD's list is a run of as many tiles, but for the last ones that hold any."""
    shape, tab = expert_lists(mm, gc, oracle, d, 256, "relu", counts, tile_rows=128)
    assert mm.expert_plan(shape) == (False, 128) and dispatch_rule("xcd_runs", shape, 1, restype=ctypes.c_int) == 1
    assert in_runs(tab[8:16])


@pytest.mark.parametrize("d,counts,runs", [
    # nine panels a slot, unequal slots: panels in turn would give one XCD 34 tiles, 33 and 35 of 243
    (2304, [76, 110, 90, 496, 70, 331, 62, 82, 993, 99, 198, 124, 141, 66, 165, 248], True),
    (2304, [587, 223, 168, 115, 126, 182, 139, 111, 303, 200, 147, 255, 387, 132, 120, 157], True),
    (2304, [165, 124, 198, 248, 99, 76, 141, 331, 496, 90, 993, 66, 82, 70, 110, 62], True),
    # ten panels: 33 of 250
    (2560, [159, 150, 241, 216, 328, 182, 169, 276, 197, 418, 634, 142], True),
    # panels in turn take one round as well: nobody else reads a panel; empty slots at both ends
    (2304, [211, 157, 362, 202, 260, 161, 223, 164, 194, 239, 294, 187, 168, 172, 176, 181], False),
    (2560, [0, 0, 335, 1005, 111, 125, 502, 143, 251, 100, 167, 83, 91, 201, 0], False)])
def test_256_row_down_tiles_in_the_fewest_rounds(mm, gc, oracle, dispatch_rule, d, counts, runs):
    shape, tab = expert_lists(mm, gc, oracle, d, 1792, "relu", counts)
    assert mm.expert_plan(shape) == (False, 256) and dispatch_rule("xcd_runs", shape, 1, restype=ctypes.c_int) == 2
    down = tab[8:16]
    assert in_runs(down) == runs and rounds(down.max(), 32) == rounds(-(-down.sum() // 8), 32) == 1


@pytest.mark.parametrize("d,counts,rule", [
    (2304, [211, 157, 362, 202, 260, 161, 223, 164, 194, 239, 294, 187], 1), (2048, [0, 157, 362, 1202, 33, 161, 2, 164, 194, 239, 294, 0], 1),
    (2560, [0, 335, 1005, 1, 125, 502, 143, 0], 2), (2048, [300, 900, 64, 280], 0)])    # narrow tiles
def test_256_row_down_tiles_of_short_reductions(mm, gc, oracle, dispatch_rule, d, counts, rule):
    shape, tab = expert_lists(mm, gc, oracle, d, 256, "relu", counts, tile_rows=256)
    assert dispatch_rule("few_wide_tiles", shape, d) == (rule != 1) and dispatch_rule("xcd_runs", shape, 1, restype=ctypes.c_int) == rule
    assert in_runs(tab[8:16]) or rule != 1


@pytest.mark.parametrize("act,f,counts,runs", [
    # twelve panels a slot, unequal slots: panels in turn would give four XCDs 71 tiles, 69 of 504
    ("relu", 3072, [176, 201, 706, 353, 471, 282, 1413, 157, 235], True), ("gelu", 3072, [176, 201, 706, 353, 471, 282, 1413, 157, 235], True),
    ("relu", 3072, [208, 195, 296, 185, 403, 167, 514, 175, 779, 339, 223, 242, 266], True),
    # six: 66 and 68 of 456
    ("relu", 1536, [733, 2201, 550, 220, 183, 200, 1100, 314, 275, 440, 169, 244, 366], True),
    ("gelu", 1536, [366, 550, 169, 275, 733, 244, 220, 314, 440, 1100, 200, 2201, 183], True),
    # panels in turn take one round as well; empty slots at both ends
    ("relu", 3072, [492, 296, 414, 273, 628, 952, 254, 362, 325], False),
    ("gelu", 1536, [0, 550, 169, 244, 314, 275, 2201, 440, 1100, 183, 200, 733, 366, 220, 0], False)])
def test_128_row_up_tiles_in_the_fewest_rounds(mm, gc, oracle, dispatch_rule, act, f, counts, runs):
    shape, tab = expert_lists(mm, gc, oracle, 256, f, act, counts)
    assert mm.expert_plan(shape) == (False, 128) and dispatch_rule("xcd_runs", shape, 0, restype=ctypes.c_int) == 2
    up = tab[:8]
    assert in_runs(up) == runs and rounds(up.max(), 64) == rounds(-(-up.sum() // 8), 64) == 1


@pytest.mark.parametrize("T,V,E,k,d,f,act,alpha,lone", [
    (700, 3, 6, 1, 512, 768, "relu", 0.4, False), (1300, 1, 3, 1, 1024, 256, "gelu", 1.0, False), (900, 2, 5, 2, 256, 512, "gelu", 0.3, False),
    (1500, 1, 16, 1, 256, 2048, "relu", 1.0, False), (1100, 1, 16, 2, 2048, 256, "gelu", 1.0, False),
    (1700, 1, 16, 1, 1792, 2560, "relu", 0.5, True), (900, 1, 16, 2, 1792, 2560, "swiglu", 0.5, True)])
def test_256_row_tiles_of_128_features(mm, gc, oracle, dispatch_rule, T, V, E, k, d, f, act, alpha, lone):
    """Products of few tiles beside ones of many (the larger sizes), tiles of every height, each activation and both outputs."""
    cfg = synth.Config(f"narrow_{T}_{d}", T, d, f, V, E, k, "bf16", act, seed=1600 + T, bias_alpha=alpha)
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg, tile_rows=256)
    assert mm.expert_plan(case.shape) == (False, 256) and dispatch_rule("lone_tiles", case.shape) == lone
    assert dispatch_rule("few_wide_tiles", case.shape, d) == (d < 2048) and dispatch_rule("few_wide_tiles", case.shape, f) == (f < 2048)
    assert len({-(-int(c) // 32) for c in ref["counts"]}) >= min(3, E - 2)


@pytest.mark.parametrize("d,f,rows,want", [
    # slots of 4 MiB (128-row tiles) and of 9 MiB (256-row ones), 73 and 34 of them in the pool: at 96 MiB used, and one slot more
    (1024, 1024, [40] * 24, False), (1024, 1024, [40] * 25, True), (1024, 1024, [300] + [40] * 24, True),
    (2304, 1024, [160] * 10, False), (2304, 1024, [160] * 11, True)])
def test_few_used_slots_of_large_pools_stay_cached(mm, gc, oracle, dispatch_rule, d, f, rows, want):
    """Tiles are marked as the only ones of their slots only where the batch uses more of the pool than 96 MiB."""
    counts = rows + [0] * ((73 if d == 1024 else 34) - len(rows))
    shape, tab = expert_lists(mm, gc, oracle, d, f, "relu", counts, tile_rows=128 if d == 1024 else 256)
    assert not mm.expert_plan(shape)[0] and dispatch_rule("lone_tiles", shape)
    entries = tab[64:64 + 4 * int(tab[0])].reshape(-1, 4)     # the up product's, of the first XCD
    only = {int(s): bool(marked) for s, marked in zip(entries[:, 0] & 0xFFFF, entries[:, 0] >> 16)}
    assert only == {s: want and rows[s] <= 256 for s in only} and len(only) > 4


@pytest.mark.parametrize("T,V,E,k,d,f,act,alpha,up,down", [
    # a round that 128 rows to a tile do not fill evenly, tiles of every height up to 256 rows; either product, each output
    (3500, 2, 14, 1, 768, 2048, "relu", 0.5, 0, 2), (1800, 1, 16, 2, 768, 2048, "swiglu", 0.6, 0, 2), (2600, 1, 9, 1, 1280, 2048, "relu", 2.5, 1, 2),
    (3500, 2, 14, 1, 768, 256, "relu", 0.5, 0, 1), (3300, 2, 12, 1, 256, 1024, "gelu", 1.0, 1, 1), (1800, 1, 16, 2, 768, 512, "swiglu", 0.6, 0, 1),
    (700, 2, 8, 1, 1024, 1280, "relu", 2.0, 0, 1), (70, 1, 1, 1, 256, 256, "gelu", 0.0, 1, 1),     # rows that a round has room for
    (600, 2, 6, 1, 512, 768, "relu", 0.5, 1, 1), (700, 1, 16, 1, 1280, 256, "gelu", 0.5, 1, 1), (450, 1, 15, 1, 1280, 768, "relu", 1.0, 1, 0),
    (2900, 1, 40, 1, 1280, 256, "relu", 1.0, 1, 0), (900, 1, 30, 1, 1280, 768, "relu", 1.0, 0, 0),
    (700, 1, 40, 1, 1024, 2048, "relu", 2.0, 0, 1)])  # more than a round, few rows per slot
def test_row_tiles_that_fill_whole_rounds(mm, gc, oracle, dispatch_rule, T, V, E, k, d, f, act, alpha, up, down):
    """Row tiles of a height that gives every compute unit one (1), of up to 256 rows where 128 do not do (2), and plain ones."""
    cfg = synth.Config(f"fill_{T}_{d}", T, d, f, V, E, k, "bf16", act, seed=1700 + T, bias_alpha=alpha)
    case, _ = staged_vs_oracle(mm, gc, oracle, cfg)
    assert mm.expert_plan(case.shape) == (False, 128)
    share = lambda n, is_up: dispatch_rule("tile_share", case.shape, n, is_up, restype=ctypes.c_int)
    assert (share(f, True), share(d, False)) == (up, down)


@pytest.mark.parametrize("T,V,E,k,d,f,act,alpha,ahead", [
    (1900, 2, 5, 1, 768, 1024, "relu", 1.0, (False, True)), (650, 1, 5, 1, 2048, 2048, "gelu", 0.5, (True, True)),    # tiles of every height
    (800, 1, 5, 1, 1536, 1536, "gelu", 0.5, (False, True)), (480, 1, 9, 1, 1536, 1536, "relu", 1.0, (True, True)),
    (1700, 1, 4, 2, 768, 1024, "swiglu", 2.5, (False, False)), (1000, 2, 8, 2, 768, 1280, "swiglu", 1.0, (False, True)),
    (1700, 1, 5, 1, 1280, 1024, "relu", 0.3, (True, False)), (3400, 1, 4, 1, 512, 1024, "gelu", 2.0, (False, True))])
def test_fp32_tiles_of_eight_wavefronts(mm, gc, oracle, dispatch_rule, T, V, E, k, d, f, act, alpha, ahead):
    cfg = synth.Config(f"ahead_{T}_{d}", T, d, f, V, E, k, "f32", act, seed=2200 + T, bias_alpha=alpha)
    case, _ = staged_vs_oracle(mm, gc, oracle, cfg)
    assert mm.expert_plan(case.shape) == (False, 96)
    assert (dispatch_rule("f32_ahead", case.shape, f, True), dispatch_rule("f32_ahead", case.shape, d, False)) == ahead, case.shape.S


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_large_combinations_agree_bit_for_bit(mm, dispatch_rule, dtype):
    """Expert outputs read past the caches, the last token's rows too, against the parts of the batch, through the caches and with a row
    shared out to several workgroups."""
    T, d, k = 897, 8192, 8
    make = lambda n: mm.make_shape(n, d, 256, 1, k, k, k, dtype, "relu")
    gen = torch.Generator("cuda").manual_seed(23)
    Yg = torch.randn((T * k, d), generator=gen, device="cuda")
    inv = torch.randperm(T * k, generator=gen, device="cuda").to(torch.int32)
    w = torch.rand((T, k), generator=gen, device="cuda")
    assert dispatch_rule("combine_past_the_caches", make(T)) and not dispatch_rule("combine_past_the_caches", make(600))
    Y = mm.combine(make(T), Yg, inv, w)
    for t0, t1 in ((0, 600), (600, T)):
        part = mm.combine(make(t1 - t0), Yg, inv[t0 * k:t1 * k].contiguous(), w[t0:t1].contiguous())
        assert torch.equal(part, Y[t0:t1]), t0
    want = (Yg[inv.long()].view(T, k, d) * w[:, :, None]).sum(1)
    # sums of eight products below 5 in size, in another order: 8 * 2^-24 * 40; bf16 rounds the result, 2^-9 of it
    assert torch.allclose(Y.float(), want, rtol=2.0 ** -8 if dtype == "bf16" else 0.0, atol=2e-5)


@pytest.mark.parametrize("T,V,E,k,d,f,act,alpha,runs", [
    (900, 2, 6, 1, 768, 512, "relu", 1.0, True), (1300, 1, 5, 1, 256, 768, "gelu", 0.5, True),         # six panels a slot, two or four
    (700, 2, 8, 2, 1280, 256, "swiglu", 2.0, True), (500, 1, 3, 2, 2304, 256, "swiglu", 0.5, True),    # more panels than XCDs, as many
    (700, 2, 8, 2, 1024, 256, "swiglu", 2.0, False),
    (60, 1, 1, 1, 256, 256, "relu", 0.0, True), (330, 1, 24, 1, 2048, 256, "relu", 0.3, False)])
def test_fp32_down_tiles_in_runs(mm, gc, oracle, dispatch_rule, T, V, E, k, d, f, act, alpha, runs):
    cfg = synth.Config(f"runs_f32_{T}_{d}", T, d, f, V, E, k, "f32", act, seed=2100 + T, bias_alpha=alpha)
    case, _ = staged_vs_oracle(mm, gc, oracle, cfg)
    assert mm.expert_plan(case.shape) == (False, 96) and dispatch_rule("f32_down_in_runs", case.shape) is runs


@pytest.mark.parametrize("d,f,counts,share", [
    (768, 256, [512, 540, 490, 515, 520, 500, 530, 489], 1),                           # 128 rows: 43 row tiles, 258 tiles, in full height
    (768, 2048, [350, 128, 360, 140, 330, 90, 129, 340, 100, 380, 128, 160, 350, 120, 345, 355, 110, 141], 2), (256, 256, [3000, 1, 0, 900], 1)])
def test_one_tile_to_a_compute_unit(mm, gc, oracle, dispatch_rule, d, f, counts, share):
    shape, tab = expert_lists(mm, gc, oracle, d, f, "relu", counts)
    assert mm.expert_plan(shape) == (False, 128) and dispatch_rule("tile_share", shape, d, False, restype=ctypes.c_int) == share
    assert in_runs(tab[8:16]) and 24 < tab[8:16].max() <= 32


@pytest.mark.parametrize("act,k,E,d,f", [("gelu", 1, 16, 1024, 1536), ("swiglu", 2, 12, 1280, 1024)])
def test_tiles_of_128_rows_in_large_pools(mm, gc, oracle, dispatch_rule, act, k, E, d, f):
    """Slots of one tile, whose weights are read past the caches, of every height, beside slots of several tiles."""
    cfg = synth.Config(f"lone128_{act}", 2600 // k, d, f, 3, E, k, "bf16", act, seed=91, share_prob=0.0, bias_alpha=0.6)
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg)
    assert mm.expert_plan(case.shape) == (False, 128) and dispatch_rule("lone_tiles", case.shape)
    heights = {-(-int(c) // 32) for c in ref["counts"]}
    assert {1, 2, 3, 4} <= heights and max(heights) > 4


@pytest.mark.parametrize("act,k", [("relu", 1), ("swiglu", 2)])
def test_f32_streaming_split_over_eight_wavefronts(mm, gc, oracle, act, k):
    """Reductions of one run, of an uneven number of runs and of several chains per wavefront, grids at both sides of
    the line (256 workgroups), slots of one 16-row block and of two."""
    for T, V, E, d, f, alpha in ((1, 2, 8, 512, 256, 0.0), (3, 2, 8, 768, 512, 0.0), (1, 2, 8, 1280, 4096, 0.0), (1, 2, 8, 512, 4352, 0.0),
                                 (20, 1, 4, 768, 1024, 0.0), (45, 1, 4, 2304, 512, 2.5), (24, 1, 2, 512, 768, 0.0)):
        cfg = synth.Config(f"eight_{act}_{T}_{d}", T // k or 1, d, f, V, E, k, "f32", act, seed=1300 + T + d, bias_alpha=alpha)
        case, ref = staged_vs_oracle(mm, gc, oracle, cfg)
        assert mm.expert_plan(case.shape) == (True, 32)
        if alpha:
            assert ref["counts"].max() > 16


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_streaming_grid_by_pair(mm, gc, oracle, dtype):
    """Batches of fewer pairs than slots (a row of workgroups per pair), as many and one more, with slots picked by
    several pairs; and numbers of pairs around the rounds in which a slot's list is made."""
    for T, V, E, k, d, f in ((1, 4, 8, 1, 256, 1280), (2, 1, 4, 2, 512, 256), (7, 4, 4, 2, 256, 512), (31, 4, 8, 1, 1280, 256),
                             (32, 4, 8, 1, 256, 512), (33, 4, 8, 1, 256, 512), (16, 1, 33, 2, 256, 512), (64, 8, 9, 1, 256, 256),
                             (65, 8, 9, 1, 256, 256), (255, 4, 8, 1, 256, 256), (128, 4, 8, 2, 256, 256), (257, 4, 8, 1, 256, 256)):
        cfg = synth.Config(f"by_pair_{dtype}_{T}", T, d, f, V, E, k, dtype, "gelu" if k == 1 else "swiglu", seed=1200 + T,
                           share_prob=0.0, bias_alpha=1.0)
        case, _ = staged_vs_oracle(mm, gc, oracle, cfg)
        assert mm.expert_plan(case.shape) == (True, 32)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d", [256, 768, 1024, 1280, 2048, 2304, 4096, 4352])
def test_router_row_lengths(mm, gc, oracle, dtype, d):
    """Rows that fill, end inside and exceed the chunks the router holds in registers, expert counts on both
    sides of the reductions' powers of two, both gates: picks equal, coefficients to fp32."""
    import torch
    rng = np.random.default_rng(d)
    for E, k, gate in ((1, 1, "selected"), (2, 2, "all"), (3, 1, "all"), (5, 4, "selected"), (8, 2, "selected"),
                       (9, 8, "all"), (64, 4, "selected"), (65, 2, "all")):
        T, V = 7, 3
        def stored(a):
            t = torch.from_numpy(a.astype(np.float32))
            return t if dtype == "f32" else t.bfloat16()
        X, Wr = stored(rng.standard_normal((T, d))), stored(0.05 * rng.standard_normal((V, E, d)))
        vid = torch.from_numpy(rng.integers(0, V, T).astype(np.int32))
        br = torch.from_numpy(rng.standard_normal((V, E)).astype(np.float32))
        shape = mm.make_shape(T, d, 256, V, E, E, k, dtype, "relu", gate=gate)
        idx, w = mm.route(shape, X.cuda(), vid.cuda(), Wr.cuda(), br.cuda())
        ref_idx, ref_w, _ = oracle.route(gc.bits(X), vid.numpy(), gc.bits(Wr), br.numpy(), k, dtype, gate=gate)
        assert np.array_equal(idx.cpu().numpy(), ref_idx), (E, k, gate)
        np.testing.assert_allclose(w.cpu().numpy(), ref_w, rtol=2e-6, atol=1e-7)


@pytest.mark.parametrize("T,d,E,k,dtype", [(911, 2304, 3, 1, "bf16"), (2053, 1280, 17, 4, "f32"), (770, 2816, 130, 8, "bf16"),
                                           (1031, 2304, 16, 2, "f32"), (2049, 3072, 16, 2, "bf16"), (2050, 1536, 64, 4, "f32"),
                                           (2051, 3328, 8, 2, "bf16"), (2052, 6144, 1, 1, "bf16")])
def test_router_token_groups(mm, gc, oracle, router_kernel, T, d, E, k, dtype):
    """Four tokens to a workgroup: variants (too many for tiles) mixed inside the groups, a last group of one to four tokens, experts
    that do and do not divide among the wavefronts.  Picks equal, coefficients to fp32."""
    rng = np.random.default_rng(T)
    def stored(a):
        t = torch.from_numpy(a.astype(np.float32))
        return t if dtype == "f32" else t.bfloat16()
    V = 9
    X, Wr = stored(rng.standard_normal((T, d))), stored(0.02 * rng.standard_normal((V, E, d)))
    vid = torch.from_numpy(rng.integers(0, V, T).astype(np.int32))
    br = torch.from_numpy(rng.standard_normal((V, E)).astype(np.float32))
    for gate in ("selected", "all"):
        shape = mm.make_shape(T, d, 256, V, E, E, k, dtype, "relu", gate=gate)
        assert router_kernel(shape) == GROUPS
        idx, w = mm.route(shape, X.cuda(), vid.cuda(), Wr.cuda(), br.cuda())
        ref_idx, ref_w, _ = oracle.route(gc.bits(X), vid.numpy(), gc.bits(Wr), br.numpy(), k, dtype, gate=gate)
        assert np.array_equal(idx.cpu().numpy(), ref_idx), gate
        np.testing.assert_allclose(w.cpu().numpy(), ref_w, rtol=2e-6, atol=1e-7)


def test_router_token_groups_look_up_slots(mm, gc, oracle, router_kernel):
    """The layer on a batch whose router takes four tokens to a workgroup: every stage and the fused call."""
    case, _ = staged_vs_oracle(mm, gc, oracle, synth.Config("route_groups", 915, 2304, 256, 3, 8, 2, "bf16", "swiglu", seed=901))
    assert router_kernel(case.shape) == GROUPS


@pytest.mark.parametrize("S", [1, 2, 63, 64, 65, 1024])
def test_grouping_sizes(mm, S):
    """Integer outputs of the grouping at the edges of its steps and of its two forms, against a stable sort:
    slots in use at random, all in one slot, some empty."""
    import torch
    for P, k in ((1, 1), (63, 1), (64, 2), (1023, 1), (1024, 4), (1025, 1), (4096, 2), (4097, 1), (8200, 4), (16384, 2),
                 (16385, 1), (40000, 1)):
        for spread in (S, max(1, S // 3)):
            g = torch.Generator().manual_seed(P * 7 + S)
            T, E = (P + k - 1) // k, 8
            V = (S + E - 1) // E
            shape = mm.make_shape(T, 256, 256, V, E, S, k, "bf16", "relu")
            vid = torch.randint(0, V, (T,), generator=g, dtype=torch.int32)
            idx = torch.randint(0, E, (T, k), generator=g, dtype=torch.int32)
            M = torch.randint(0, spread, (V, E), generator=g, dtype=torch.int32)
            out = mm.remap_permute(shape, torch.zeros((T, 256), dtype=torch.bfloat16, device="cuda"), vid.cuda(),
                                   idx.cuda(), M.cuda(), mm.alloc_workspace(shape))
            slot = M[vid.long().repeat_interleave(k), idx.flatten().long()]
            perm = torch.argsort(slot, stable=True)
            counts = torch.bincount(slot, minlength=S)
            inv = torch.empty_like(perm)
            inv[perm] = torch.arange(T * k)
            offsets = torch.cat([torch.zeros(1, dtype=torch.long), counts.cumsum(0)])
            for name, got, want in zip(("slot", "counts", "offsets", "perm", "inv_perm"), out,
                                       (slot, counts, offsets, perm, inv)):
                assert torch.equal(got.cpu().long(), want.long()), (P, S, spread, name)


UNEVEN_TILES = [
    # feature tiles that do not divide among the XCDs, one list of tiles per XCD: fewer tiles than XCDs, one
    # slot, many slots (some empty), one slot with most of the rows, an even up product beside an uneven down
    synth.Config("uneven_one_tile", 200, 256, 256, 1, 1, 1, "bf16", "relu", seed=700),
    synth.Config("uneven_d768_f1280", 900, 768, 1280, 2, 8, 2, "bf16", "swiglu", seed=701),
    synth.Config("uneven_skew", 2100, 768, 1536, 3, 16, 2, "bf16", "gelu", seed=702, bias_alpha=2.5, vid_mode="zipf"),
    synth.Config("uneven_empty_slots", 1500, 1280, 256, 4, 16, 1, "bf16", "relu", seed=703, bias_alpha=6.0),
    synth.Config("uneven_down_only", 700, 768, 1024, 2, 4, 4, "bf16", "swiglu", seed=704),
]


@pytest.mark.parametrize("rows", [256, 128])
@pytest.mark.parametrize("cfg", UNEVEN_TILES, ids=lambda c: c.name)
def test_uneven_feature_tiles(mm, gc, oracle, cfg, rows):
    staged_vs_oracle(mm, gc, oracle, cfg, tile_rows=rows)


GATES_AND_ACTS = [
    # Switch-style gate (probability over all experts, not renormalised), top-1, ReLU and GELU experts,
    # three variants; streaming kernels and matrix-core kernels, fp32 and bf16
    synth.Config("g_switch_f32_gelu", 60, 256, 512, 3, 8, 1, "f32", "gelu", seed=41, gate="all"),
    synth.Config("g_switch_bf16_relu_tiled", 1200, 256, 512, 3, 8, 1, "bf16", "relu", seed=42, gate="all"),
    synth.Config("g_switch_bf16_gelu_tiled", 1000, 512, 768, 3, 8, 1, "bf16", "gelu", seed=43, gate="all"),
    synth.Config("g_switch_bf16_gelu_stream", 90, 512, 256, 3, 8, 1, "bf16", "gelu", seed=44, gate="all"),
    # k = 2 and 4 with either gate, up to 64 experts per variant, gated and plain experts
    synth.Config("g_all_k2_e64", 500, 256, 256, 2, 64, 2, "bf16", "swiglu", seed=45, gate="all"),
    synth.Config("g_all_k4_e64", 300, 256, 256, 3, 64, 4, "bf16", "gelu", seed=46, gate="all", bias_alpha=0.5),
    synth.Config("g_sel_k4_e16", 2100, 256, 256, 3, 16, 4, "bf16", "gelu", seed=47),
    synth.Config("g_all_k4_f32", 2060, 512, 256, 3, 16, 4, "f32", "swiglu", seed=48, gate="all"),
    synth.Config("g_all_k_equals_e", 70, 256, 256, 2, 4, 4, "f32", "relu", seed=49, gate="all"),   # sums to 1 again
]


@pytest.mark.parametrize("cfg", GATES_AND_ACTS, ids=lambda c: c.name)
def test_gate_modes_and_activations(mm, gc, oracle, cfg):
    """Section 3.2's coefficients "for each expert" read the Switch way (section 4.3's family), and the
    GELU expert: every stage against the oracle, both router kernels, both expert-stage kernels."""
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg)
    if cfg.gate == "all" and cfg.top_k < cfg.E:
        assert (ref["topk_w"].sum(1) < 1.0).all()        # not renormalised


def test_edge_cases(mm, gc, oracle):
    # a single token
    staged_vs_oracle(mm, gc, oracle, synth.Config("one_token", 1, 256, 256, 2, 4, 2, "bf16", "swiglu", seed=10))
    # every pick lands in one slot, all other slots are empty; two picks of a token share a slot
    cfg = synth.Config("one_slot", 130, 256, 256, 2, 4, 2, "bf16", "swiglu", seed=11)
    inp = synth.make_inputs(cfg)
    inp["M"][:] = 2
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg, inp)
    assert ref["counts"][2] == 260 and ref["counts"].sum() == 260
    # exact ties in the router: duplicated router rows and an all-zero token
    cfg = synth.Config("ties", 64, 256, 256, 1, 6, 3, "f32", "relu", seed=12)
    inp = synth.make_inputs(cfg)
    inp["Wr"][0, 4] = inp["Wr"][0, 1]
    inp["Wr"][0, 5] = inp["Wr"][0, 2]
    inp["X"][7] = 0.0
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg, inp)
    assert list(ref["topk_idx"][7]) == [0, 1, 2]
    # E above one wavefront's width, k = 8
    staged_vs_oracle(mm, gc, oracle, synth.Config("wide_e", 40, 256, 256, 1, 130, 8, "bf16", "relu", seed=13))
    staged_vs_oracle(mm, gc, oracle, synth.Config("wide_e_many", 2050, 256, 256, 1, 130, 8, "bf16", "relu", seed=19))


def test_validate_inputs(mm, gc):
    cfg = synth.Config("val", 16, 256, 256, 2, 4, 1, "f32", "relu", seed=14)
    case = gc.DeviceCase(cfg)
    assert mm.validate_inputs(case.shape, case.vid, case.M, case.ws)
    bad = case.vid.clone()
    bad[3] = 2
    assert not mm.validate_inputs(case.shape, bad, case.M, case.ws)
    badM = case.M.clone()
    badM[1, 1] = case.S
    assert not mm.validate_inputs(case.shape, case.vid, badM, case.ws)


def packed_layout_bf16(W):
    """Plain [S, K, N] ("in x out") bf16 bit patterns -> the documented fragment layout, by the
    index formula of include/mmoe.h (written with numpy index arithmetic, no kernel code)."""
    S, K, N = W.shape
    n = np.arange(N)[None, :]
    k = np.arange(K)[:, None]
    m, h, kk = k // 64, (k % 64) // 32, (k % 32) // 8
    ks = 4 * m + kk
    off = ((((n // 32) * (K // 16) + ks) * 64 + 32 * h + n % 32) * 8 + k % 8)        # [K, N], within a slot
    out = np.empty((S, K * N), W.dtype)
    for s in range(S):
        out[s, off.reshape(-1)] = W[s].reshape(-1)
    return out


def test_pack_round_trip(mm, gc):
    cfg = synth.Config("pack", 4, 256, 512, 1, 3, 1, "bf16", "swiglu", seed=15)
    inp = synth.make_inputs(cfg)
    case = gc.DeviceCase(cfg, inp)
    for packed, plain in ((case.W1p, inp["W1"]), (case.W3p, inp["W3"]), (case.W2p, inp["W2"])):
        got = gc.bits(packed).reshape(plain.shape[0], -1)
        assert np.array_equal(got, packed_layout_bf16(plain))
    cfg = synth.Config("pack32", 4, 256, 512, 1, 2, 1, "f32", "relu", seed=16)
    inp = synth.make_inputs(cfg)
    case = gc.DeviceCase(cfg, inp)
    assert np.array_equal(gc.bits(case.W1p), inp["W1"].transpose(0, 2, 1))      # fp32: the transpose
    assert np.array_equal(gc.bits(case.W2p), inp["W2"].transpose(0, 2, 1))


FULL_SMALL = ["switch8_fp32_v2_t128", "switch8_bf16_v4_t4096", "mixtral_decode_bf16_v2_t64"]


@pytest.mark.parametrize("name", FULL_SMALL)
def test_benchmark_shapes_full_parity(mm, gc, oracle, name):
    staged_vs_oracle(mm, gc, oracle, synth.CONFIGS[name])


@pytest.mark.parametrize("name,seed", [("mixtral_prefill_bf16_v2_t8192", 0), ("mixtral_skew_bf16_v4_t16384", 0),
                                       ("mixtral_prefill_bf16_v2_t8192", 1)])
def test_benchmark_shapes_sampled_parity(mm, gc, oracle, name, seed):
    """Full-size layers in the benchmark's launch configuration: integer outputs on every
    token; expert outputs on every row of the smallest and of the largest slot; layer outputs
    on 512 seeded tokens that the oracle evaluates one by one."""
    cfg = synth.CONFIGS[name].replace(seed=seed)
    print(f"case {name} seed {seed}: generating", flush=True)
    case = gc.DeviceCase(cfg)
    inp, sh = case.inp, case.shape
    print("routing oracle", flush=True)
    idx_ref, w_ref, _ = oracle.route(inp["X"], inp["vid"], inp["Wr"], inp["br"], cfg.top_k, cfg.dtype)
    slot_ref, counts_ref, offsets_ref, perm_ref, inv_ref = oracle.remap_group(inp["vid"], idx_ref, inp["M"], case.S)

    idx, w = mm.route(sh, case.X, case.vid, case.Wr, case.br)
    slot, counts, offsets, perm, inv, Xg = mm.remap_permute(sh, case.X, case.vid, idx, case.M, case.ws)
    torch.cuda.synchronize()
    assert np.array_equal(idx.cpu().numpy(), idx_ref)
    np.testing.assert_allclose(w.cpu().numpy(), w_ref, rtol=2e-6, atol=1e-7)
    for got, ref in ((slot, slot_ref), (counts, counts_ref), (offsets, offsets_ref), (perm, perm_ref), (inv, inv_ref)):
        assert np.array_equal(got.cpu().numpy(), ref)
    assert np.array_equal(gc.bits(Xg), inp["X"][perm_ref // cfg.top_k])
    print("slot counts min/median/max:", counts_ref.min(), int(np.median(counts_ref)), counts_ref.max(), flush=True)

    # staged expert stage and combination, then the fused entry point: bit-equal to each other
    Yg = mm.expert_ffn(sh, Xg, offsets, case.W1p, case.W3p, case.W2p, case.ws)
    Ys = mm.combine(sh, Yg, inv, w)
    Y = case.forward()
    torch.cuda.synchronize()
    assert torch.isfinite(Y.float()).all()
    assert torch.equal(Y, Ys), "fused entry point differs from the staged path"

    # every row of the smallest and of the largest slot, one expert evaluation each
    smallest, largest = int(np.argmin(np.where(counts_ref > 0, counts_ref, 1 << 30))), int(np.argmax(counts_ref))
    for s in (smallest, largest):
        r0, r1 = int(offsets_ref[s]), int(offsets_ref[s + 1])
        print(f"expert oracle on all {r1 - r0} rows of slot {s}", flush=True)
        rows = np.arange(r0, r1)
        Yg_ref = oracle.ffn_rows(inp["X"], (perm_ref[rows] // cfg.top_k).astype(np.int32),
                                 np.full(r1 - r0, s, np.int32), inp["W1"], inp["W3"], inp["W2"], cfg.dtype, cfg.act)
        gc.assert_close(gc.to_np64(Yg[r0:r1]), Yg_ref, cfg.dtype, f"Yg (all rows of slot {s})")
    # a seeded sample of tokens through the whole layer
    toks = np.sort(np.random.default_rng(7).choice(cfg.T, 512, replace=False))
    print(f"layer oracle on {len(toks)} sampled tokens", flush=True)
    Y_ref = oracle.layer_tokens(inp, cfg.top_k, cfg.dtype, cfg.act, toks, routed=(idx_ref, w_ref, slot_ref))
    gc.assert_close(gc.to_np64(Y[torch.from_numpy(toks).cuda()]), Y_ref, cfg.dtype, "Y (sampled)")


def test_decode_sizes_one_to_sixty_four_tokens(mm, gc, oracle):
    """Single-request decode is the paper's own workload (section 4).  The Mixtral-shaped layer at
    1, 2, 4, ... 64 tokens on one pool: the fused entry point (four launches, the expert kernels
    group the pairs themselves) against the oracle on every token, bit-equal to the staged calls
    and to itself on a second run."""
    cfg64 = synth.CONFIGS["mixtral_decode_bf16_v2_t64"]
    case = gc.DeviceCase(cfg64)
    for T in (1, 2, 4, 8, 16, 32, 64):
        print(f"decode T={T}", flush=True)
        cfg = cfg64.replace(T=T)
        sh = mm.make_shape(T, cfg.d_model, cfg.d_ff, cfg.V, cfg.E, case.S, cfg.top_k, cfg.dtype, cfg.act)
        inp = dict(case.inp, X=case.inp["X"][:T], vid=case.inp["vid"][:T])
        X, vid = case.X[:T].contiguous(), case.vid[:T].contiguous()
        ref = oracle.layer_forward(inp, cfg.top_k, cfg.dtype, cfg.act)
        Y = mm.layer_forward(sh, X, vid, case.Wr, case.br, case.M, case.W1p, case.W3p, case.W2p, case.ws)
        torch.cuda.synchronize()
        gc.assert_close(gc.to_np64(Y), ref["Y"], cfg.dtype, f"Y at T={T}")
        idx, w = mm.route(sh, X, vid, case.Wr, case.br)
        slot, counts, offsets, perm, inv, Xg = mm.remap_permute(sh, X, vid, idx, case.M, case.ws)
        assert np.array_equal(idx.cpu().numpy(), ref["topk_idx"]) and np.array_equal(perm.cpu().numpy(), ref["perm"])
        Ys = mm.combine(sh, mm.expert_ffn(sh, Xg, offsets, case.W1p, case.W3p, case.W2p, case.ws), inv, w)
        Y2 = mm.layer_forward(sh, X, vid, case.Wr, case.br, case.M, case.W1p, case.W3p, case.W2p, case.ws)
        torch.cuda.synchronize()
        assert torch.equal(Y, Ys), f"T={T}: fused entry point differs from the staged path"
        assert torch.equal(Y, Y2), f"T={T}: two runs differ"


def test_limits_many_slots_and_widest_router(mm, gc, oracle):
    """Close to the documented limits: a pool of several hundred slots (most of them empty or
    nearly empty for a small batch), and E = 256 experts with k = 8."""
    cfg = synth.Config("many_slots", 300, 256, 256, 64, 16, 2, "bf16", "swiglu", seed=20, share_prob=0.1)
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg)
    assert 800 < case.S <= 1024 and (ref["counts"] == 0).any()
    cfg = synth.Config("many_slots_f32", 90, 256, 256, 40, 16, 1, "f32", "relu", seed=21, share_prob=0.2)
    staged_vs_oracle(mm, gc, oracle, cfg)
    staged_vs_oracle(mm, gc, oracle, synth.Config("widest_e", 70, 512, 256, 1, 256, 8, "bf16", "relu", seed=22))
    # many slots and enough rows for the matrix-core kernels (hundreds of short tile lists)
    cfg = synth.Config("many_slots_tiled", 6000, 256, 256, 8, 16, 2, "bf16", "swiglu", seed=23, share_prob=0.3)
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg)
    assert case.S > 80
    # several hundred slots and enough pairs for the matrix-core kernels at two or three rows per slot
    cfg = synth.Config("many_slots_two_chunks", 1200, 256, 256, 64, 16, 2, "bf16", "swiglu", seed=30, share_prob=0.1)
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg)
    assert 800 < case.S <= 1024
    # the same pool with enough rows per slot for the matrix-core kernels: nine hundred short tile lists,
    # a target height chosen over all of them
    cfg = synth.Config("many_slots_tiled_wide", 20000, 256, 256, 64, 16, 2, "bf16", "relu", seed=31, share_prob=0.1)
    case, ref = staged_vs_oracle(mm, gc, oracle, cfg)
    assert 800 < case.S <= 1024 and mm.expert_plan(case.shape)[0] is False


@pytest.mark.parametrize("name", ["switch8_fp32_v2_t128", "switch8_bf16_v4_t4096", "mixtral_decode_bf16_v2_t64"])
def test_benchmark_shapes_second_seed(mm, gc, oracle, name):
    """Robustness row: the same shapes with another seed (another table, other counts)."""
    staged_vs_oracle(mm, gc, oracle, synth.CONFIGS[name].replace(seed=1))


def test_layer_forward_in_a_captured_graph(mm, gc, oracle):
    """The fused entry point allocates nothing and never synchronises, so a caller can record
    it into a HIP graph.  Every replay, with new tokens written into the same buffers in
    between and eager work around it, must reproduce the eager result bit for bit."""
    for cfg in (synth.Config("graph_stream", 48, 512, 768, 2, 4, 2, "bf16", "swiglu", seed=24),
                synth.Config("graph_tiled", 800, 256, 512, 2, 4, 2, "bf16", "swiglu", seed=25),
                # one pick per token: three launches (stream) or five (tiled), the down product writes Y
                synth.Config("graph_stream_top1", 40, 256, 512, 3, 8, 1, "f32", "gelu", seed=32, gate="all"),
                synth.Config("graph_tiled_top1", 2500, 256, 512, 3, 8, 1, "bf16", "relu", seed=33, gate="all")):
        case = gc.DeviceCase(cfg)
        sh = case.shape
        Y = torch.empty((cfg.T, cfg.d_model), dtype=case.X.dtype, device="cuda")
        side = torch.cuda.Stream()
        side.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(side):    # warm-up on the capture stream, as graph capture requires
            mm.layer_forward(sh, case.X, case.vid, case.Wr, case.br, case.M, case.W1p, case.W3p, case.W2p,
                             case.ws, Y=Y)
        torch.cuda.current_stream().wait_stream(side)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            mm.layer_forward(sh, case.X, case.vid, case.Wr, case.br, case.M, case.W1p, case.W3p, case.W2p,
                             case.ws, Y=Y)
        for rep in range(3):
            inp = synth.make_inputs(cfg.replace(seed=100 + rep), weights=False)
            case.X.copy_(gc.to_dev(inp["X"], cfg.dtype))
            case.vid.copy_(torch.from_numpy(inp["vid"]).cuda())
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
            got = Y.clone()
            eager = case.forward()
            torch.cuda.synchronize()
            assert torch.equal(got, eager), f"{cfg.name}: replay {rep} differs from the eager result"
        # and against the oracle once, for the last batch (same pool and table, new tokens)
        last = dict(case.inp, X=inp["X"], vid=inp["vid"])
        ref = oracle.layer_forward(last, cfg.top_k, cfg.dtype, cfg.act, gate=cfg.gate)
        gc.assert_close(gc.to_np64(got), ref["Y"], cfg.dtype, "Y (graph replay)")


def _random_configs(n, seed):
    """Seeded sweep over shapes: both dtypes and activations, every k up to E, token counts on
    both sides of every dispatch threshold (router variants, streaming vs tiled expert
    kernels, one or several grouping workgroups), with and without a router bias."""
    rng = np.random.default_rng(seed)
    out = []
    for i in range(n):
        dtype = "f32" if i % 4 == 3 else "bf16"
        act = "relu" if i % 3 == 2 else "swiglu"
        d = int(rng.choice([256, 512, 768, 1024]))
        f = int(rng.choice([256, 512, 1280]))
        V = int(rng.integers(1, 5))
        E = int(rng.integers(1, 10))
        k = int(rng.integers(1, min(E, 4) + 1))
        T = int(rng.choice([1, 7, 64, 200, 511, 512, 700, 1100, 2047, 2048, 2300]))
        if dtype == "f32":
            T = min(T, 300) if i % 2 else T  # half the cases stay small (the oracle's time)
        out.append(synth.Config(f"rnd{i}_{dtype}_{act}_T{T}_d{d}_f{f}_V{V}_E{E}_k{k}", T, d, f, V, E, k, dtype, act,
                                seed=1000 + i, bias_alpha=float(rng.choice([0.0, 0.5])),
                                vid_mode=str(rng.choice(["uniform", "zipf", "interleave"])),
                                share_prob=float(rng.choice([0.0, 0.5, 1.0]))))
    return out


@pytest.mark.parametrize("cfg", _random_configs(24, seed=2024), ids=lambda c: c.name)
def test_random_shapes(mm, gc, oracle, cfg):
    staged_vs_oracle(mm, gc, oracle, cfg)


def test_calls_run_on_the_current_stream(mm):
    """The raw handle that the binding passes on is torch's current stream: the default one, a stream of a context, of a
    nested one, and the default one again."""
    torch.zeros(1, device="cuda")
    a, b = torch.cuda.Stream(), torch.cuda.Stream()

    def same(stream):
        return mm._stream() == torch.cuda.current_stream().cuda_stream == stream.cuda_stream

    assert same(torch.cuda.default_stream())
    with torch.cuda.stream(a):
        assert same(a)
        with torch.cuda.stream(b):
            assert same(b)
        assert same(a)
    assert same(torch.cuda.default_stream()) and a.cuda_stream != b.cuda_stream


def test_ceiling_probe_reports_plausible_rates(mm):
    gbs, tflops = mm.probe_ceilings(gib=1)
    assert 2000.0 < gbs < 8000.0, gbs          # below the 8 TB/s data-sheet peak, above a third of it
    assert 500.0 < tflops < 2500.0, tflops     # below the 2.5 PFLOP/s data-sheet peak
