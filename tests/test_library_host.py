"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every symbol
the header declares, sizes the workspace, and turns bad arguments into error codes."""
import ctypes
import os
import random
import re

import pytest

from paper_2505_06481_amd import build as mbuild

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def mm():
    if mbuild.is_stale():
        mbuild.build()
    from paper_2505_06481_amd import mmoe
    mmoe.lib()
    return mmoe


def test_every_declared_symbol_is_exported(mm):
    header = open(os.path.join(ROOT, "include", "mmoe.h")).read()
    header = re.sub(r"/\*.*?\*/", "", header, flags=re.S)
    declared = set(re.findall(r"\b(mmoe_[a-z_0-9]+)\s*\(", header))
    assert declared == set(mm.EXPORTS)
    L = ctypes.CDLL(os.path.join(ROOT, "paper_2505_06481_amd", "libmmoe.so"))
    for name in declared:
        assert hasattr(L, name), name


def test_workspace_size_accounts_for_every_intermediate(mm):
    sh = mm.make_shape(8192, 4096, 14336, 2, 8, 12, 2, "bf16", "swiglu")
    P = 8192 * 2
    need = P * 14336 * 2 + P * 4096 * 4     # H + Yg (the fused layer keeps no gathered copy of the tokens)
    got = mm.workspace_bytes(sh)
    assert need <= got <= need + (1 << 20)
    assert mm.workspace_bytes(mm.make_shape(8, 100, 256, 1, 1, 1, 1, "f32", "relu")) == 0


def test_bad_arguments_become_error_codes(mm):
    L = mm.lib()
    ok = mm.make_shape(4, 256, 256, 1, 2, 2, 1, "f32", "relu")
    p = ctypes.c_void_p(4096)          # never dereferenced: checks fail before any launch
    none = None

    def route(shape, X=p, vid=p, Wr=p):
        return L.mmoe_route(ctypes.byref(shape), X, vid, Wr, none, p, p, none)

    assert route(ok, X=none) == -1                                                       # NULL
    assert route(mm.make_shape(0, 256, 256, 1, 2, 2, 1, "f32", "relu")) == -2            # dimension
    assert route(mm.make_shape(4, 256, 256, 1, 2, 2, 3, "f32", "relu")) == -3            # top_k > E
    assert route(mm.make_shape(4, 256, 256, 1, 16, 2, 9, "f32", "relu")) == -3           # top_k > 8
    assert route(mm.make_shape(4, 256, 256, 1, 2, 2, 1, 7, "relu")) == -4                # dtype
    assert route(mm.make_shape(4, 256, 256, 1, 2, 2, 1, "f32", 5)) == -4                 # activation
    assert route(mm.make_shape(4, 256, 256, 1, 2, 2, 1, "f32", "gelu", gate=2)) == -4     # gate mode
    assert route(mm.make_shape(4, 256, 256, 1, 2, 2, 1, "f32", "gelu", gate="all"), X=none) == -1
    assert route(mm.make_shape(4, 200, 256, 1, 2, 2, 1, "f32", "relu")) == -8            # multiple of 256
    assert route(mm.make_shape(4, 256, 256, 1, 300, 2, 1, "f32", "relu")) == -9          # E limit
    assert route(mm.make_shape(4, 256, 256, 1, 2, 5000, 1, "f32", "relu")) == -9         # S limit
    assert route(ok, X=ctypes.c_void_p(4100)) == -7                                      # alignment
    # the 2^31 limit of the matrix-core expert path is a property of the shape: refused by every entry
    # point before anything is launched, and the workspace size of such a shape is 0
    huge = mm.make_shape(100000, 4096, 14336, 2, 8, 12, 2, "bf16", "swiglu")
    assert route(huge) == -9 and mm.workspace_bytes(huge) == 0
    # expert stage: W3 must match the activation; workspace must be large enough
    gated = mm.make_shape(4, 256, 256, 1, 2, 2, 1, "bf16", "swiglu")
    assert L.mmoe_expert_ffn(ctypes.byref(gated), p, p, p, none, p, p, p, 1 << 30, none) == -5
    assert L.mmoe_expert_ffn(ctypes.byref(ok), p, p, p, p, p, p, p, 1 << 30, none) == -5
    gelu = mm.make_shape(4, 256, 256, 1, 2, 2, 1, "bf16", "gelu")
    assert L.mmoe_expert_ffn(ctypes.byref(gelu), p, p, p, p, p, p, p, 1 << 30, none) == -5   # GELU takes no W3
    assert L.mmoe_expert_ffn(ctypes.byref(ok), p, p, p, none, p, p, p, 16, none) == -6
    assert L.mmoe_expert_ffn(ctypes.byref(ok), p, p, p, none, p, p, none, 1 << 30, none) == -6
    assert L.mmoe_layer_forward(ctypes.byref(ok), p, p, p, none, p, p, none, p, p, ctypes.c_void_p(4352), 8,
                                none) == -6
    assert L.mmoe_layer_forward(ctypes.byref(ok), p, p, p, none, p, p, none, p, p, ctypes.c_void_p(4100),
                                1 << 30, none) == -7
    assert L.mmoe_pack_weights(ctypes.byref(gated), p, none, p, p, p, p, none) == -5
    assert L.mmoe_combine(ctypes.byref(ok), none, p, p, p, none) == -1
    assert L.mmoe_remap_permute(ctypes.byref(ok), p, p, p, p, p, p, p, p, p, p, none, 0, none) == -6
    # the entry point without a workspace refuses, before any GPU call, what its fixed array cannot hold
    big = mm.make_shape(8192, 4096, 14336, 2, 8, 12, 2, "bf16", "swiglu")
    assert mm.workspace_bytes(big) > mm.STATIC_WORKSPACE_BYTES
    assert L.mmoe_layer_forward_static(ctypes.byref(big), p, p, p, none, p, p, p, p, p, none) == -11
    assert L.mmoe_layer_forward_static(ctypes.byref(mm.make_shape(0, 256, 256, 1, 2, 2, 1, "f32", "relu")),
                                       p, p, p, none, p, p, none, p, p, none) == -2
    for code in range(0, -12, -1):
        assert mm.strerror(code) != "unknown status"
    assert mm.strerror(-99) == "unknown status"


def test_paged_layer_argument_checks(mm):
    L = mm.lib()
    p = ctypes.c_void_p(4096)
    q = ctypes.c_void_p(8192)
    sh = mm.make_shape(4, 256, 256, 1, 2, 2, 1, "f32", "relu")
    res = (ctypes.c_uint8 * 2)(1, 0)
    hp = (ctypes.c_void_p * 2)(None, 4096)
    none_hp = (ctypes.c_void_p * 2)(None, None)
    big = ctypes.c_size_t(1 << 30)

    def call(resident=res, h1=hp, h2=hp, h3=None, W3=None, stream=p, copy=q, ws=p, ws_bytes=big):
        return L.mmoe_layer_forward_paged(ctypes.byref(sh), p, p, p, None, p, p, W3, p, resident, h1, h3, h2, p, ws,
                                          ws_bytes, stream, copy, None)

    assert call(resident=None) == -1
    assert call(h1=none_hp) == -1                      # a non-resident slot without a host copy
    assert call(copy=p) == -1                          # the copies need a stream of their own
    assert call(copy=None) == -1
    assert call(W3=p) == -5                            # RELU takes no W3
    assert call(ws_bytes=ctypes.c_size_t(8)) == -6


def test_expert_map_builder_argument_checks(mm):
    L = mm.lib()
    p = ctypes.c_void_p(4096)
    ok = mm.make_loader_shape(2, 3, 4, [256 * 512] * 2, "bf16", 5)
    ptrs = (ctypes.c_void_p * 4)(4096, 4096, 4096, 4096)
    need = L.mmoe_loader_workspace_bytes(ctypes.byref(ok))
    assert need >= 3 * 4 * 2 * 8                               # a partial sum per location and chunk
    assert L.mmoe_expert_distance(ctypes.byref(ok), ptrs, p, p, 16, None) == -6          # workspace too small
    assert L.mmoe_expert_distance(ctypes.byref(ok), None, p, p, need, None) == -1
    bad = (ctypes.c_void_p * 4)(4096, 4100, 4096, 4096)
    assert L.mmoe_expert_distance(ctypes.byref(ok), bad, p, p, need, None) == -7          # misaligned matrix
    for shape, code in ((mm.make_loader_shape(9, 3, 4, [256], "bf16", 1), -9),           # more than 8 variants
                        (mm.make_loader_shape(2, 100, 100, [256], "bf16", 1), -9),       # more than 4096 locations
                        (mm.make_loader_shape(2, 3, 4, [100], "bf16", 1), -8),           # not a multiple of 256
                        (mm.make_loader_shape(2, 3, 4, [256], "bf16", -1), -2),          # negative capacity
                        (mm.make_loader_shape(2, 0, 4, [256], "bf16", 1), -2),
                        (mm.make_loader_shape(2, 3, 4, [256], 7, 1), -4)):
        assert L.mmoe_loader_workspace_bytes(ctypes.byref(shape)) == 0
        assert L.mmoe_build_expert_map(ctypes.byref(shape), p, p, p, p, p, p, None) == code
    assert L.mmoe_build_expert_map(ctypes.byref(ok), p, p, None, p, p, p, None) == -1
    pool = (ctypes.c_void_p * 2)(4096, 4096)
    assert L.mmoe_assemble_pool(ctypes.byref(ok), ptrs, p, 3, 4, pool, None) == -2      # layer out of range
    assert L.mmoe_assemble_pool(ctypes.byref(ok), ptrs, p, 0, 9, pool, None) == -2      # more slots than V*E
    assert L.mmoe_assemble_pool(ctypes.byref(ok), ptrs, None, 0, 4, pool, None) == -1
    assert L.mmoe_assemble_pool(ctypes.byref(ok), ptrs, p, 0, 4, (ctypes.c_void_p * 2)(4096, 4100), None) == -7


def test_binding_refuses_host_tensors(mm):
    import torch
    sh = mm.make_shape(4, 256, 256, 1, 2, 2, 1, "f32", "relu")
    with pytest.raises(ValueError):
        mm.route(sh, torch.zeros(4, 256), torch.zeros(4, dtype=torch.int32), torch.zeros(1, 2, 256))


def test_tile_rows_field_accepts_only_its_three_values(mm):
    for good in (128, 256, 0):
        assert mm.workspace_bytes(mm.make_shape(512, 256, 256, 1, 2, 2, 1, "bf16", "relu", tile_rows=good)) > 0
    p = ctypes.c_void_p(4096)
    for bad in (64, 512, -1, 100):
        sh = mm.make_shape(512, 256, 256, 1, 2, 2, 1, "bf16", "relu", tile_rows=bad)
        assert mm.workspace_bytes(sh) == 0
        assert mm.lib().mmoe_route(ctypes.byref(sh), p, p, p, None, p, p, None) == -2


def test_probe_rejects_bad_arguments_before_touching_the_gpu(mm):
    L = mm.lib()
    out = (ctypes.c_float * 2)()
    p = ctypes.c_void_p(4096)
    assert L.mmoe_probe_ceilings(None, ctypes.c_size_t(1 << 30), out, None) == -1
    assert L.mmoe_probe_ceilings(p, ctypes.c_size_t(1 << 30), None, None) == -1
    assert L.mmoe_probe_ceilings(p, ctypes.c_size_t(1 << 20), out, None) == -6     # buffer too small
    assert L.mmoe_probe_ceilings(ctypes.c_void_p(4097), ctypes.c_size_t(1 << 30), out, None) == -7


def test_expert_plan_follows_the_documented_dispatch(mm):
    from paper_2505_06481_amd import synth

    def plan(name_or_cfg, S, tile_rows=0):
        c = synth.CONFIGS[name_or_cfg] if isinstance(name_or_cfg, str) else name_or_cfg
        return mm.expert_plan(mm.make_shape(c.T, c.d_model, c.d_ff, c.V, c.E, S, c.top_k, c.dtype, c.act,
                                            tile_rows=tile_rows))

    assert plan("switch8_fp32_v2_t128", 12) == (True, 32)            # fp32, 11 rows per slot
    assert plan("mixtral_decode_bf16_v2_t64", 13) == (True, 32)      # 10 rows per slot
    assert plan("switch8_bf16_v4_t4096", 20) == (False, 128)         # short reduction: 128-row tiles
    assert plan("mixtral_prefill_bf16_v2_t8192", 13) == (False, 256)
    assert plan("mixtral_skew_bf16_v4_t16384", 20) == (False, 256)
    mix = synth.CONFIGS["mixtral_decode_bf16_v2_t64"]
    assert plan(mix.replace(T=104), 13) == (True, 32)                # 16 rows per slot: still streaming
    assert plan(mix.replace(T=105), 13) == (False, 128)              # beyond: matrix-core kernels, small tiles
    assert plan(mix.replace(T=415), 13) == (False, 128)              # under 64 rows per slot
    assert plan(mix.replace(T=416), 13) == (False, 256)
    # the tuning field overrides the tile height only, and only for the call it is passed to
    assert plan("mixtral_prefill_bf16_v2_t8192", 13, tile_rows=128) == (False, 128)
    assert plan("mixtral_decode_bf16_v2_t64", 13, tile_rows=128) == (True, 32)
    assert plan("mixtral_prefill_bf16_v2_t8192", 13) == (False, 256)


@pytest.mark.parametrize("d,f,S,P,want", [
    (2048, 2048, 12, 240, (True, 32)), (2048, 2048, 12, 241, (False, 128)),     # small experts: 20 rows per slot
    (512, 1024, 64, 512, (True, 32)), (512, 1024, 64, 513, (False, 128)),       # and at most 512 pairs
    (768, 3072, 4, 128, (True, 32)), (768, 3072, 4, 129, (False, 128)),         # 4 to 11 slots: 14 rows and 72 pairs more
    (2048, 2048, 8, 184, (True, 32)), (2048, 2048, 8, 185, (False, 128)),
    (768, 3072, 3, 60, (True, 32)), (768, 3072, 3, 61, (False, 128)),
    (1536, 3072, 8, 16000, (False, 128)), (1792, 3072, 8, 799, (False, 128)), (1792, 3072, 8, 800, (False, 256)),
    (2304, 3072, 8, 511, (False, 128)), (2304, 3072, 8, 512, (False, 256)),     # tall tiles by rows per slot
])
def test_expert_plan_at_its_lines(mm, d, f, S, P, want):
    assert mm.expert_plan(mm.make_shape(P, d, f, 1, S, S, 1, "bf16", "relu")) == want


def test_expert_plan_says_where_down_tiles_may_be_taller(mm, dispatch_rule):
    """256-row tiles of the down product where the plan says 128: with the shape's tile_rows 0 only, never of the up product, and the
    header and the binding say so."""
    taller = 0
    for T in range(1000, 9000, 37):
        for d, S in ((768, 18), (768, 24), (1280, 12)):
            for rows in (0, 128, 256):
                shape = mm.make_shape(T, d, 3072, 4, 8, S, 1, "bf16", "relu", tile_rows=rows)
                if dispatch_rule("tile_share", shape, d, False, restype=ctypes.c_int) == 2:
                    taller += 1
                    assert rows == 0 and mm.expert_plan(shape) == (False, 128)
                assert dispatch_rule("tile_share", shape, 3072, True, restype=ctypes.c_int) != 2
    assert taller
    header = re.sub(r"[\s*]+", " ", open(os.path.join(ROOT, "include", "mmoe.h")).read())
    assert "Where that is 128 and the shape's tile_rows is 0, tiles of the down product may have up to 256" in header
    assert "tiles of the down product may have up to 256" in re.sub(r"\s+", " ", mm.expert_plan.__doc__)


@pytest.mark.parametrize("P,want", [(96, (True, 32)), (97, (False, 96))])
def test_expert_plan_f32(mm, P, want):
    assert mm.expert_plan(mm.make_shape(P, 768, 3072, 1, 8, 8, 1, "f32", "relu")) == want


def static_refuses(mm, shape):
    """Does mmoe_layer_forward_static refuse the shape's size?  Null pointers: nothing can be launched."""
    return mm.lib().mmoe_layer_forward_static(ctypes.byref(shape), *([None] * 10)) == -11


@pytest.mark.parametrize("d,f,S,E,k,dtype,act,T0", [
    (768, 3072, 18, 8, 1, "bf16", "relu", 7262), (4096, 14336, 128, 8, 2, "bf16", "swiglu", 744),
    (768, 3072, 1024, 8, 1, "f32", "relu", 4356), (768, 3072, 13, 8, 1, "f32", "gelu", 4400),
    (2048, 1280, 90, 64, 4, "bf16", "swiglu", 1500), (256, 256, 4, 4, 2, "bf16", "relu", 21500)])
def test_static_entry_point_takes_what_the_workspace_size_says(mm, d, f, S, E, k, dtype, act, T0):
    """A program that asks for the workspace size first is never refused: every batch whose workspace is within
    MMOE_STATIC_WORKSPACE_BYTES is accepted, token by token across the limit."""
    below = above = 0
    for T in range(T0 - 600, T0 + 600):
        sh = mm.make_shape(T, d, f, 2, E, S, k, dtype, act)
        if mm.workspace_bytes(sh) <= mm.STATIC_WORKSPACE_BYTES:
            below += 1
            assert not static_refuses(mm, sh), (T, mm.workspace_bytes(sh))
        else:
            above += 1
    assert below and above


@pytest.mark.parametrize("d,f,S,E,k,dtype,act,tile_rows", [
    (256, 8448, 503, 4, 1, "bf16", "relu", 256), (1792, 256, 459, 64, 4, "bf16", "swiglu", 0),
    (768, 5376, 13, 13, 1, "bf16", "gelu", 256), (1280, 2816, 556, 8, 4, "bf16", "gelu", 128),
    (768, 3072, 18, 8, 1, "bf16", "relu", 0), (4096, 14336, 18, 8, 2, "bf16", "swiglu", 0),
    (1024, 2048, 90, 4, 1, "f32", "swiglu", 0), (256, 16128, 1024, 8, 1, "bf16", "swiglu", 0)])
def test_workspace_of_the_largest_batch_holds_every_smaller_one(mm, d, f, S, E, k, dtype, act, tile_rows):
    """The workspace size never shrinks as T grows (kernels and list layouts change with T, and a program makes one
    workspace for its largest batch), and the tile height that a call asks for does not change it."""
    last = 0
    for T in range(1, 5000):
        size = mm.workspace_bytes(mm.make_shape(T, d, f, 2, E, S, k, dtype, act, tile_rows=tile_rows))
        assert size >= last, (T, size, last)
        last = size
    for T in (700, 1920, 4000):
        assert len({mm.workspace_bytes(mm.make_shape(T, d, f, 2, E, S, k, dtype, act, tile_rows=r))
                    for r in (0, 128, 256)}) == 1


STATIC_LARGEST = [
    # d, f, S, E, k, dtype, activation, largest accepted batch.  Many slots, feature tiles that do not divide among
    # the XCDs: the lists take more than they are counted at
    (256, 14080, 1024, 8, 1, "bf16", "swiglu", 2276),
    (256, 8448, 1024, 8, 2, "bf16", "swiglu", 1858),
    (256, 14592, 1024, 64, 2, "bf16", "swiglu", 1099),
    (256, 14080, 821, 4, 4, "bf16", "relu", 570),
    (256, 16128, 1024, 8, 1, "bf16", "gelu", 1994),
    # and ordinary shapes
    (2048, 1280, 90, 64, 4, "bf16", "swiglu", 1556),
    (768, 3072, 18, 8, 1, "bf16", "relu", 7261),
    (4096, 14336, 128, 8, 2, "bf16", "swiglu", 743),
    (768, 3072, 1024, 8, 1, "f32", "relu", 4350),
    (256, 5376, 300, 8, 1, "f32", "swiglu", 2971),
]


@pytest.mark.parametrize("d,f,S,E,k,dtype,act,largest", STATIC_LARGEST)
def test_static_entry_point_size_limit(mm, d, f, S, E, k, dtype, act, largest):
    """Which batches fit is a plain sum over the intermediates with the tile lists counted at a fixed rate: the
    largest accepted batch of shapes whose lists need more room than that, and of shapes whose lists need less."""
    def shape(T):
        return mm.make_shape(T, d, f, 2, E, S, k, dtype, act)
    for T in range(max(1, largest - 300), largest + 1):
        assert not static_refuses(mm, shape(T)), T
    for T in range(largest + 1, largest + 300):
        assert static_refuses(mm, shape(T)), T


def test_few_picks_of_large_experts_leave_the_caches(mm, dispatch_rule):
    """One pick touches one slot of S, or nearly: an expert of hundreds of MB streams past the caches for it."""
    for T, k, d, f, S, act, dtype, want in ((1, 1, 4096, 14336, 8, "relu", "bf16", True), (1, 1, 4096, 14336, 9, "swiglu", "bf16", True),
                                            (1, 1, 4096, 4096, 8, "swiglu", "bf16", False), (2, 1, 4096, 4096, 8, "swiglu", "bf16", True),
                                            (1, 2, 4096, 4096, 13, "swiglu", "bf16", True), (1, 1, 4096, 8192, 9, "relu", "f32", True),
                                            (3, 1, 768, 3072, 16, "gelu", "bf16", False), (40, 1, 768, 3072, 16, "gelu", "bf16", True)):
        shape = mm.make_shape(T, d, f, 2, 8, S, k, dtype, act)
        assert dispatch_rule("past_the_caches", shape) is want, (T, k, d, f, S)


def test_one_tile_slots_leave_the_caches_only_with_large_pools(mm, dispatch_rule):
    """A pool that the last-level cache (256 MB) holds is read through it, whatever the rows per slot."""
    for T, d, f, S, act, want in ((540, 2304, 768, 6, "swiglu", False), (450, 4096, 512, 5, "relu", False),
                                  (440, 4096, 1024, 8, "swiglu", False), (1100, 2560, 2560, 20, "gelu", True),
                                  (715, 4096, 2048, 13, "swiglu", True), (777, 4096, 14336, 18, "swiglu", True),
                                  (8192, 4096, 14336, 13, "swiglu", False)):
        shape = mm.make_shape(T, d, f, 4, 8, S, 2, "bf16", act)
        assert mm.expert_plan(shape) == (False, 256)
        assert dispatch_rule("lone_tiles", shape) is want, (d, f, S)


def test_down_products_take_runs_of_tiles(mm, dispatch_rule):
    """256-row tiles do (1) in short reductions with fewer than 16 panels; in long ones never where panels divide among the XCDs, else
    only where that takes fewer rounds (2).  128-row tiles do where token rows are a quarter of the traffic, or half where panels divide."""
    for T, k, d, f, S, want in ((1170, 2, 4096, 14336, 18, 0), (2250, 2, 4096, 14336, 18, 0), (4050, 2, 4096, 14336, 18, 0),
                                (2520, 2, 2048, 3072, 12, 0), (840, 2, 4096, 7680, 12, 0), (1600, 2, 2560, 7680, 12, 2),
                                (2520, 2, 2304, 7680, 12, 2), (1440, 2, 2304, 1536, 12, 1),
                                (1440, 2, 2304, 1792, 12, 2), (2520, 2, 2048, 1024, 12, 1), (1440, 2, 4096, 1024, 12, 0), (840, 2, 2304, 1024, 12, 2), (3600, 2, 2560, 7680, 12, 0), (500, 2, 2560, 7680, 16, 0),
                                (4096, 1, 768, 3072, 18, 1), (200, 2, 768, 3072, 18, 0), (520, 2, 1024, 4096, 13, 1),
                                (330, 2, 1024, 4096, 13, 0), (520, 2, 2048, 3072, 13, 0), (960, 2, 2048, 3072, 24, 0), (300, 2, 1280, 2560, 13, 1)):
        shape = mm.make_shape(T, d, f, 4, 8, S, k, "bf16", "swiglu")
        assert dispatch_rule("xcd_runs", shape, 1, restype=ctypes.c_int) == want, (T, d, f, S)
        assert dispatch_rule("xcd_runs", mm.make_shape(T, d, f, 4, 8, S, k, "f32", "swiglu"), 1, restype=ctypes.c_int) == 0


def test_up_products_of_less_than_a_round(mm, dispatch_rule):
    """Wide 128-row tiles below a round of the chip, with GELU only where another half tile per slot leaves them one; and there
    the XCDs may take runs (2) unless panels divide among them."""
    for T, d, f, S, act, want, runs in ((4096, 768, 3072, 18, "relu", True, 2), (4096, 768, 3072, 13, "gelu", True, 2),
                                        (4096, 768, 3072, 24, "gelu", False, 0), (4096, 768, 3072, 24, "relu", True, 2),
                                        (5000, 768, 3072, 18, "relu", True, 2), (5000, 768, 3072, 18, "gelu", False, 0),
                                        (5000, 768, 3072, 9, "gelu", False, 0), (4500, 768, 3072, 9, "gelu", True, 2),
                                        (6000, 512, 2048, 13, "relu", True, 0), (6000, 512, 2048, 13, "gelu", True, 0),
                                        (4096, 768, 3072, 30, "relu", False, 0), (3000, 768, 3072, 13, "relu", False, 0),
                                        (5500, 768, 3072, 13, "relu", False, 0), (8000, 1536, 1536, 13, "relu", True, 2)):
        shape = mm.make_shape(T, d, f, 4, 8, S, 1, "bf16", act)
        assert mm.expert_plan(shape) == (False, 128)
        assert dispatch_rule("wide_below_a_round", shape, f, True) is want, (T, d, f, S, act)
        assert dispatch_rule("xcd_runs", shape, 0, restype=ctypes.c_int) == runs, (T, d, f, S, act)
    assert dispatch_rule("wide_below_a_round", mm.make_shape(8000, 1536, 3072, 4, 8, 24, 1, "bf16", "gelu"), 1536, False)
    assert dispatch_rule("xcd_runs", mm.make_shape(4096, 768, 3072, 4, 8, 18, 1, "bf16", "swiglu"), 0, restype=ctypes.c_int) == 0


def test_routers_of_few_scores_take_no_groups_of_long_rows(mm, dispatch_rule):
    """fp32 rows of over 3072 elements go to groups of four tokens only with 3500 (token, expert) pairs to score; shorter
    rows and bf16 as their own lines say."""
    for T, d, E, dtype, want in ((768, 4096, 1, "f32", False), (768, 3584, 4, "f32", False), (768, 3328, 8, "f32", True),
                                 (1024, 4096, 3, "f32", False), (1024, 4096, 4, "f32", True), (1536, 3840, 2, "f32", False),
                                 (1536, 3840, 3, "f32", True), (2000, 4096, 1, "f32", False), (2000, 4096, 2, "f32", True), (2047, 3584, 64, "f32", True),
                                 (767, 4096, 64, "f32", False), (2500, 4096, 64, "f32", True), (2500, 4096, 8, "f32", False),
                                 (768, 3072, 1, "f32", True), (768, 4096, 1, "bf16", True), (768, 4352, 64, "f32", False)):
        shape = mm.make_shape(T, d, 256, 2, E, E, 1, dtype, "relu")
        assert dispatch_rule("route_in_groups", shape) is want, (T, d, E, dtype)


def test_routers_in_tiles_only_where_groups_of_a_variant_fill(mm, dispatch_rule):
    """bf16 batches with much to score go to tiles (four tokens of a variant to a wavefront) with up to eight variants, up to four
    if rows are short; of one variant, or with few experts, not in the first rounds of the groups of any four tokens if the rounds are full; and not
    where wavefronts would have few experts each.  (T, d, V, E, tiles)"""
    for T, d, V, E, want in ((8192, 4096, 8, 8, True), (8192, 4096, 9, 8, False), (8000, 1024, 64, 32, False), (8388600, 256, 64, 32, False),
                             (4096, 1024, 4, 12, True), (4096, 1024, 5, 12, False), (4096, 1024, 8, 48, True),
                             (2303, 3072, 2, 8, False), (2304, 3072, 2, 8, True), (3000, 2048, 2, 8, False), (4096, 2048, 2, 8, True),
                             (1024, 4096, 4, 12, False), (2048, 4096, 4, 12, False), (2049, 4096, 4, 12, False), (6144, 4096, 4, 12, True), (2049, 3072, 4, 12, True),
                             (1024, 4096, 1, 32, False), (1025, 4096, 1, 32, True), (1408, 4096, 1, 32, True), (1409, 4096, 1, 32, False), (1024, 4096, 2, 32, True), (1733, 2816, 3, 32, True),
                             (3184, 3584, 4, 32, True), (4275, 3840, 2, 16, True), (4275, 3840, 1, 16, False), (2048, 3584, 2, 16, False), (2049, 3584, 2, 16, True), (2048, 3328, 2, 16, True), (2049, 4096, 2, 15, False),
                             (900, 4096, 1, 64, True), (960, 4096, 1, 64, True), (961, 4096, 1, 64, False), (961, 2048, 1, 64, True), (1024, 4096, 1, 64, False), (1024, 4096, 2, 64, True), (1025, 4096, 1, 64, True),
                             (1984, 4096, 1, 64, True), (1985, 4096, 1, 64, False), (1985, 4096, 2, 64, True), (3072, 4096, 1, 64, False), (3073, 4096, 1, 64, True), (4096, 4096, 2, 64, True),
                             (1037, 2048, 2, 64, True), (640, 3072, 2, 32, True), (639, 3072, 2, 32, False),
                             (12000, 512, 4, 16, False), (12000, 768, 4, 16, True), (12000, 768, 4, 17, False), (3583, 512, 1, 64, False), (2100, 512, 2, 64, True), (3088, 256, 2, 64, False), (3584, 512, 2, 64, True),
                             (12000, 256, 2, 48, False), (12000, 256, 2, 64, True), (8191, 2048, 2, 33, False), (8192, 2048, 2, 33, True), (5000, 2048, 2, 48, True)):
        shape = mm.make_shape(T, d, 256, V, E, E, 1, "bf16", "relu")
        assert dispatch_rule("route_in_tiles", shape) is want, (T, d, V, E)
        assert not dispatch_rule("route_in_tiles", mm.make_shape(min(T, 20000), d, 256, V, E, E, 1, "f32", "relu"))


def test_router_launches_fit_a_grid(mm, dispatch_rule):
    """A launch has fewer than 2^32 work-items: the groups of the largest batches in tiles, 512 work-items each at most."""
    for V in (1, 2, 5, 8, 9, 64, 1000):
        for E in (8, 16, 32, 64, 256):
            shape = mm.make_shape((1 << 23) - 1, 256, 256, V, E, E, 1, "bf16", "relu")
            chunks, groups = -(-shape.T // 64), min(64, 16 + (3 * V + 3) // 4)
            if dispatch_rule("route_in_tiles", shape):
                assert chunks * groups * 512 < 1 << 32, (V, E)


def test_few_wide_tiles_are_cut_in_two(mm, dispatch_rule):
    """Down products of 256-row tiles: fewer wide tiles than half of the compute units, and a little over one round of them up to
    100 rows per slot."""
    for T, k, d, S, want in ((400, 2, 4096, 4, True), (1000, 2, 2304, 12, True), (720, 4, 2048, 9, True), (820, 4, 2048, 9, False),
                             (1070, 2, 2560, 8, True), (1200, 2, 2560, 8, False), (777, 2, 4096, 18, True), (1170, 2, 4096, 18, False),
                             (777, 2, 4096, 24, False)):
        shape = mm.make_shape(T, d, 4096, 4, 8, S, k, "bf16", "swiglu")
        assert mm.expert_plan(shape) == (False, 256)
        assert dispatch_rule("few_wide_tiles", shape, d) is want, (T, k, d, S)


def test_row_tiles_fill_rounds_of_few_tiles(mm, dispatch_rule):
    """Ungated products of narrow 128-row tiles.  Down: heights that fill a round (1) up to 512 tiles, counted with one more for every
    slot, from 32 rows per slot on, or up to 32 full tiles in a round, or where panels of a reduction from 2048 on divide among the XCDs; 256-row tiles (2) where those may be more than a round of 256 and these are not,
    in reductions from 2048 and with 64 rows per slot on; neither beyond, nor with a forced height of 256.  Up: 1, where panels divide
    among the XCDs, or with up to 32 full tiles in a round, or tiles are half a round and slots have up to 128 rows."""
    for T, d, f, S, rows, want in ((4096, 768, 3072, 18, 0, 2), (4096, 768, 3072, 18, 128, 1), (4096, 768, 3072, 18, 256, 0), (4096, 768, 3072, 8, 0, 1),
                                   (3072, 768, 3072, 18, 0, 1), (3073, 768, 3072, 18, 0, 2), (8063, 768, 3072, 18, 0, 2), (8064, 768, 3072, 18, 0, 1),
                                   (8576, 768, 3072, 18, 0, 1), (8577, 768, 3072, 18, 0, 0), (5000, 1024, 3072, 30, 0, 0), (600, 1536, 3072, 18, 0, 1), (575, 1536, 3072, 18, 0, 0),
                                   (500, 1536, 3072, 16, 0, 0), (768, 1536, 3072, 16, 0, 1), (767, 1536, 3072, 16, 0, 1), (600, 1792, 3072, 8, 0, 1), (1000, 1792, 3072, 8, 0, 0),
                                   (4096, 768, 1792, 18, 0, 1), (4096, 768, 2048, 18, 0, 2), (1216, 1280, 3072, 19, 0, 2), (1215, 1280, 3072, 19, 0, 1),
                                   (900, 1280, 3072, 19, 0, 1), (330, 512, 2048, 28, 0, 1), (513, 512, 3072, 28, 0, 1), (682, 768, 3072, 36, 0, 1), (683, 768, 3072, 36, 0, 0),
                                   (682, 768, 3072, 37, 0, 0), (800, 768, 3072, 25, 0, 1), (799, 768, 3072, 25, 0, 0),
                                   (248, 4096, 14336, 9, 0, 1), (700, 1024, 2048, 40, 0, 1), (700, 1024, 1792, 40, 0, 0)):
        shape = mm.make_shape(T, d, f, 4, 8, S, 1, "bf16", "relu", tile_rows=rows)
        assert dispatch_rule("tile_share", shape, d, False, restype=ctypes.c_int) == want, (T, d, f, S, rows)
        assert dispatch_rule("tile_share", mm.make_shape(T, d, f, 4, 8, S, 1, "f32", "relu"), d, False, restype=ctypes.c_int) == 0
    for T, f, S, want in ((1024, 1024, 8, 1), (4096, 1024, 8, 1), (7168, 1024, 8, 1), (7169, 1024, 8, 0), (2304, 768, 3, 0), (384, 768, 3, 1), (682, 768, 3, 1), (683, 768, 3, 0),
                          (2048, 768, 16, 0), (600, 768, 16, 1), (682, 768, 16, 1), (683, 768, 16, 0), (682, 768, 37, 0), (2600, 1280, 14, 0), (3500, 2048, 1, 1)):
        for act in ("relu", "gelu"):
            shape = mm.make_shape(T, 768, f, 4, 8, S, 1, "bf16", act)
            assert dispatch_rule("tile_share", shape, f, True, restype=ctypes.c_int) == want, (T, f, S)
        assert dispatch_rule("tile_share", mm.make_shape(T, 768, f, 4, 8, S, 2, "bf16", "swiglu"), f, True, restype=ctypes.c_int) == 0


def test_fp32_tiles_of_eight_wavefronts_where_they_are_one_round(mm, dispatch_rule):
    """Tiles of 64 rows, counted with three quarters of one more for every slot, in up to 256, reductions from 1024 on; up products
    only where panels divide among the XCDs, or with four panels and more and up to 56 rows per slot.  (T, d, f, S, up, down)"""
    for T, d, f, S, up, down in ((2000, 768, 3072, 13, False, True), (2346, 768, 3072, 8, False, True), (2347, 768, 3072, 8, False, False),
                                 (2500, 768, 3072, 8, False, False), (4020, 512, 2816, 5, False, False), (1900, 768, 768, 8, False, False),
                                 (700, 2048, 1024, 12, True, False), (1472, 2048, 1024, 12, True, False), (1473, 2048, 1024, 12, False, False),
                                 (1084, 3072, 768, 16, False, False), (608, 2560, 1280, 9, False, False), (2653, 1280, 512, 12, False, False),
                                 (560, 1792, 1280, 10, True, True), (561, 1792, 1280, 10, False, True)):
        shape = mm.make_shape(T, d, f, 4, min(S, 8), S, 1, "f32", "relu")
        assert (dispatch_rule("f32_ahead", shape, f, True), dispatch_rule("f32_ahead", shape, d, False)) == (up, down), (T, d, f, S)
        assert not dispatch_rule("f32_ahead", mm.make_shape(T, d, f, 4, min(S, 8), S, 1, "f32", "swiglu"), f, True)
        assert not dispatch_rule("f32_ahead", mm.make_shape(T, d, f, 4, min(S, 8), S, 1, "bf16", "relu"), d, False)


def test_fp32_down_products_in_runs_only_of_few_uneven_panels(mm, dispatch_rule):
    """Fewer panels than XCDs; more that do not divide among them up to 700 tiles; from a quarter of the traffic in token rows on."""
    for T, d, S, want in ((2000, 768, 13, True), (4096, 768, 32, True), (700, 768, 29, True), (700, 768, 30, False), (2600, 1024, 13, False), (900, 512, 24, False),
                          (2000, 1024, 8, False), (2944, 1280, 24, True), (2945, 1280, 24, False), (1024, 1280, 48, False), (1344, 2304, 17, True), (1345, 2304, 17, False), (3000, 2304, 12, False), (330, 2048, 24, False),
                          (500, 2304, 6, True)):
        shape = mm.make_shape(T, d, 3072, 4, 6, S, 1, "f32", "relu")
        assert not mm.expert_plan(shape)[0] and dispatch_rule("f32_down_in_runs", shape) is want, (T, d, S)


def test_combination_reads_past_the_caches_only_what_they_cannot_hold(mm, dispatch_rule):
    for T, d, k, want in ((4800, 4096, 2, False), (7168, 4096, 2, False), (7169, 4096, 2, True), (8192, 4096, 2, True), (673, 7424, 8, False), (3500, 4096, 4, False)):
        for dtype in ("bf16", "f32"):
            assert dispatch_rule("combine_past_the_caches", mm.make_shape(T, d, 256, 1, 8, 8, k, dtype, "relu")) is want, (T, d, k)


def test_lists_of_every_plan_fit_the_scratch_that_is_asked_for(mm, dispatch_rule):
    """What mmoe_expert_ffn asks for behind H is never less than the lists of the plan it then launches: whatever height the call asks
    for, 256-row tiles of the down product beside a height of 128 among them, and heights that fill a round."""
    rng, tall, filled = random.Random(7), 0, 0
    size = lambda name, shape: dispatch_rule(name, shape, restype=ctypes.c_size_t)
    for _ in range(20000):
        d, f, S, k = 256 * rng.randint(1, 8), 256 * rng.randint(1, 16), rng.randint(1, 40), rng.choice([1, 1, 2])
        T, dtype, act = int(100 * 120 ** rng.random()), rng.choice(["bf16", "bf16", "bf16", "f32"]), rng.choice(["relu", "gelu", "swiglu"])
        asked = set()
        for rows in (0, 128, 256):
            shape = mm.make_shape(T, d, f, 2, min(S, 8), S, min(k, S), dtype, act, tile_rows=rows)
            if mm.expert_plan(shape)[0]:
                continue
            asked.add(size("tiled_table_bytes", shape))
            assert size("planned_table_bytes", shape) <= min(asked), (T, d, f, S, k, dtype, act, rows)
            share = dispatch_rule("tile_share", shape, d, False, restype=ctypes.c_int)
            tall, filled = tall + (share == 2), filled + (share == 1)
        assert len(asked) <= 1
    assert tall > 100 and filled > 1000


def test_static_entry_point_has_room_for_what_it_accepts(mm):
    """The lists are counted at a plain rate against the limit; what they take beyond it fits the 4 MB of slack, tile heights that
    fill a round among them."""
    rng, accepted, beyond = random.Random(8), 0, 0
    for _ in range(60000):
        S, dtype = int(1024 ** rng.random()), rng.choice(["bf16", "bf16", "f32"])
        k, act = rng.choice([1, 1, 2, 4]), rng.choice(["relu", "gelu", "swiglu"])
        shape = mm.make_shape(int(30000 ** rng.random()), 256 * int(64 ** rng.random()), 256 * int(64 ** rng.random()), 2, max(k, min(S, 8)), S, k, dtype, act)
        if static_refuses(mm, shape) or mm.workspace_bytes(shape) == 0:
            continue
        accepted += 1
        beyond = max(beyond, mm.workspace_bytes(shape) - mm.STATIC_WORKSPACE_BYTES)
        assert beyond <= 4 << 20, (shape.T, shape.d_model, shape.d_ff, S, k, dtype, act)
    assert accepted > 10000 and beyond > 0


def test_lists_of_every_batch_fit_the_room_of_the_largest(mm, dispatch_rule):
    for d, f, S, k, dtype, act in ((768, 3072, 18, 1, "bf16", "relu"), (256, 1024, 300, 1, "bf16", "gelu"), (1280, 2560, 16, 2, "bf16", "swiglu"),
                                   (1536, 768, 5, 1, "bf16", "relu"), (2304, 1024, 12, 2, "bf16", "gelu"), (768, 3072, 13, 1, "f32", "relu")):
        last = 0
        for T in range(200, 12000, 37):
            shape = mm.make_shape(T, d, f, 2, 8, S, k, dtype, act)
            most = dispatch_rule("tiled_table_most", shape, restype=ctypes.c_size_t)
            assert dispatch_rule("tiled_table_bytes", shape, restype=ctypes.c_size_t) <= most and last <= most, (T, d, f)
            last = most
