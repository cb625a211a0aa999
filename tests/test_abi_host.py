"""CPU-only checks of the C ABI: the library loads, exports every symbol the header declares,
and rejects bad arguments on the host before anything is launched (no GPU needed)."""
import ctypes as C
import os
import re

import numpy as np
import pytest

from paper_2408_10746_amd import binding as pb

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def header_functions():
    names = set()
    for h in sorted(os.listdir(os.path.join(ROOT, "include"))):
        if not h.endswith(".h"):
            continue
        src = open(os.path.join(ROOT, "include", h)).read()
        src = re.sub(r"/\*.*?\*/", "", src, flags=re.S)
        names |= set(re.findall(r"\b(pac_[a-z0-9_]+)\s*\(", src))
    return sorted(names)


def test_library_exports_every_declared_symbol():
    names = header_functions()
    assert len(names) >= 11
    lib = pb.lib()
    for n in names:
        assert hasattr(lib, n), f"{n} is declared in include/pac.h but not exported"
    assert sorted(pb.EXPORTS) == names, "the Python binding must mirror the header one to one"


def test_create_validation_and_sizes():
    with pytest.raises(pb.PacError) as e:
        pb.pac_create(0, 768, 128, 96, 3, 32, 16, pb.PAC_BF16)
    assert e.value.status == pb.PAC_ERR_SHAPE
    for bad in [dict(d=770), dict(r=100), dict(C=17), dict(B_max=65)]:
        kw = dict(L=2, d=768, n_max=128, r=96, C=3, B_max=32, N=16)
        kw.update(bad)
        with pytest.raises(pb.PacError) as e:
            pb.pac_create(kw["L"], kw["d"], kw["n_max"], kw["r"], kw["C"], kw["B_max"], kw["N"], pb.PAC_BF16)
        assert e.value.status == pb.PAC_ERR_UNSUPPORTED
    with pytest.raises(pb.PacError) as e:
        pb.pac_create(2, 768, 128, 96, 3, 32, 16, 7)
    assert e.value.status == pb.PAC_ERR_SHAPE
    assert pb.lib().pac_create(None, None) == pb.PAC_ERR_NULL

    ctx = pb.pac_create(12, 768, 128, 96, 3, 32, 4096, pb.PAC_BF16)
    try:
        P = 12 * (2 * 768 * 96 + 96 + 768 + 1) + 768 * 3 + 3
        assert pb.pac_param_count(ctx) == P == 1782159
        assert pb.pac_param_offsets(ctx, 0) == [0, 768 * 96, 768 * 96 + 96, 2 * 768 * 96 + 96, 2 * 768 * 96 + 96 + 768]
        assert pb.pac_param_offsets(ctx, -1)[:2] == [P - 768 * 3 - 3, P - 3]
        with pytest.raises(pb.PacError):
            pb.pac_param_offsets(ctx, 12)
        # storage: tokens x hidden x layers elements per sequence (paper Sec. 5.2), 2 bytes each
        assert pb.pac_cache_bytes(ctx, None, 4096) == 4096 * 128 * 768 * 12 * 2
        assert pb.pac_cache_bytes(ctx, [5, 128, 1], 3) == (5 + 128 + 1) * 768 * 12 * 2
        assert pb.pac_cache_bytes(ctx, [0], 1) == -1 and pb.pac_cache_bytes(ctx, [129], 1) == -1
        assert pb.pac_workspace_bytes(ctx) > 0 and pb.pac_workspace_bytes(ctx) % 256 == 0
    finally:
        pb.pac_destroy(ctx)
    # the paper's storage example: T5-Base, 500 samples of 30 tokens, fp32, below 1 GB
    ctx = pb.pac_create(12, 768, 30, 96, 3, 32, 500, pb.PAC_F32)
    assert pb.pac_cache_bytes(ctx, None, 500) == 552_960_000 < 10 ** 9
    pb.pac_destroy(ctx)
    pb.pac_destroy(None)


def test_formulation_chosen_per_configuration():
    """Host logic: which formulation a configuration runs on (0 per-layer, 1 Gram with single-launch chains,
    2 Gram with layer-by-layer chains)."""
    def path(L, d, n, r, C, B, dtype=pb.PAC_BF16, flags=0):
        ctx = pb.pac_create(L, d, n, r, C, B, 64, dtype, flags)
        try:
            return pb.pac_step_path(ctx)
        finally:
            pb.pac_destroy(ctx)

    assert path(12, 768, 128, 96, 3, 32) == 1            # T5-Base-shaped
    assert path(24, 1024, 128, 128, 2, 32) == 1          # Large-shaped: the chain kernels' LDS just fits
    assert path(32, 4096, 256, 256, 4, 16) == 2          # LLaMA-7B-shaped: r > 128
    assert path(12, 768, 128, 160, 3, 32) == 2
    assert path(40, 1024, 128, 128, 2, 32) == 2          # too many layers for the LDS-resident chains
    assert path(12, 768, 128, 96, 3, 32, pb.PAC_F32) == 0
    assert path(12, 768, 128, 96, 3, 32, flags=pb.PAC_FLAG_PER_LAYER) == 0
    assert path(12, 768, 128, 96, 3, 32, flags=pb.PAC_FLAG_LAYER_CHAIN) == 2
    assert path(32, 4096, 1024, 512, 2, 8) == 2          # long-sequence configuration
    assert path(12, 768, 128, 320, 3, 32) == 2
    assert path(12, 768, 128, 288, 3, 32) == 0           # above 256 only in multiples of 64
    assert path(12, 768, 128, 544, 3, 32) == 0           # wider than the Gram path takes
    assert path(40, 1024, 128, 384, 2, 32) == 0          # above 256 only up to 32 layers
    assert path(80, 4096, 64, 256, 3, 8) == 0            # more layers than the wide path's vector part deals with
    assert pb.lib().pac_step_path(None) == -1


def step_tiles(L, d, n, r, B, lens=None, dtype=pb.PAC_BF16):
    ctx = pb.pac_create(L, d, n, r, 3, B, 64, dtype)
    try:
        return pb.pac_step_tiles(ctx, lens, B)
    finally:
        pb.pac_destroy(ctx)


def test_tiles_chosen_per_batch():
    """Host logic: which tiles the launches of a step take."""
    assert step_tiles(12, 768, 128, 96, 32) == dict(proj=128, tokens=128, grads=64, rows=0, se=4, sg=4)   # T5-Base-shaped
    assert step_tiles(32, 4096, 256, 256, 16) == dict(proj=256, tokens=256, grads=256, rows=1, se=1, sg=1)  # LLaMA-7B-shaped
    assert step_tiles(32, 4096, 1024, 512, 8, [640] * 8)["proj"] == 256                                     # long sequences
    assert step_tiles(12, 768, 128, 96, 32, dtype=pb.PAC_F32) == dict(proj=16, tokens=0, grads=0, rows=0, se=0, sg=0)
    # wide K-contiguous contractions: 256 x 256 tiles where there are many long ones, not for short or few ones
    assert step_tiles(3, 512, 768, 512, 8)["proj"] == 128       # (46 us against 30)
    assert step_tiles(11, 448, 224, 320, 1)["proj"] == 128      # (65 / 46)
    assert step_tiles(3, 1280, 648, 512, 8)["proj"] == 128      # (58 / 45)
    assert step_tiles(48, 256, 768, 160, 8)["proj"] == 256      # (150 / 179)
    assert step_tiles(17, 2560, 892, 448, 4)["proj"] == 256     # (368 / 414)
    assert step_tiles(20, 896, 197, 256, 3)["grads"] == 128     # (147 / 119)
    assert step_tiles(8, 1632, 178, 448, 8)["grads"] == 128     # (119 / 98)
    assert step_tiles(31, 672, 50, 512, 2)["grads"] == 256      # (492 / 561)
    assert step_tiles(22, 2080, 50, 256, 8)["grads"] == 256     # (222 / 251)
    # contractions over the tokens: the large tiles where both kinds of tile walk over many tokens
    assert step_tiles(24, 512, 128, 160, 8)["tokens"] == 128    # (54 / 43)
    assert step_tiles(16, 832, 300, 320, 2)["tokens"] == 128    # (71 / 51)
    assert step_tiles(4, 256, 803, 512, 8)["tokens"] == 128     # (133 / 118)
    assert step_tiles(16, 2048, 768, 224, 8)["tokens"] == 128   # (272 / 225)
    assert step_tiles(24, 1280, 768, 160, 8)["tokens"] == 128   # (279 / 213)
    assert step_tiles(18, 640, 189, 160, 16)["tokens"] == 128   # (101 / 77)
    assert step_tiles(4, 1024, 768, 192, 8)["tokens"] == 256    # (36 / 44)
    assert step_tiles(16, 2048, 768, 256, 8)["tokens"] == 256
    assert step_tiles(27, 768, 327, 320, 16)["tokens"] == 256   # (503 / 658)
    assert step_tiles(12, 1024, 256, 256, 16)["tokens"] == 256  # (92 / 111)
    t = step_tiles(4, 2048, 768, 256, 8)
    assert t["tokens"] == 256 and t["se"] == 3 and t["sg"] == 4  # (54 / 70)
    # vector gradients as whole rows
    assert step_tiles(8, 1024, 768, 256, 8)["rows"] == 0        # 2 M elements of a stacked copy: 62 us against 51
    assert step_tiles(4, 2048, 768, 256, 8)["rows"] == 0        # 2 M: 43 / 35
    assert step_tiles(8, 1024, 256, 384, 8)["rows"] == 1        # 3 M: 73 / 78
    assert step_tiles(16, 1024, 256, 192, 16)["rows"] == 1      # 3 M: 77 / 81
    # fp32 contractions: 16-row tiles where 64 x 64 ones leave compute units idle, the latter where they fill the chip
    fp32 = {(768, 96, 4096): 16, (768, 96, 8192): 16, (2048, 32, 16384): 16, (1024, 128, 4096): 16, (4096, 512, 1024): 16,
            (1024, 128, 8192): 64, (1024, 256, 4096): 64, (4096, 256, 8192): 64, (2048, 512, 2048): 64, (4096, 512, 8192): 64,
            (2048, 32, 32768): 64, (2080, 128, 8192): 16, (2080, 512, 2048): 16, (2080, 512, 4096): 64}
    for (d, r, rows), tile in fp32.items():
        assert step_tiles(3, d, rows // 32, r, 32, dtype=pb.PAC_F32)["proj"] == tile, (d, r, rows)
    with pytest.raises(pb.PacError) as e:
        step_tiles(12, 768, 128, 96, 2, [128, 129])
    assert e.value.status == pb.PAC_ERR_RANGE
    assert pb.lib().pac_step_tiles(None, None, 1, (C.c_int32 * 6)()) == pb.PAC_ERR_NULL


def test_fp32_formulation_per_batch():
    """Host logic: which formulation an fp32 call takes, on both sides of the line (us in the Gram-matrix formulation / in the
    per-layer kernels), and what is reserved for it."""
    def ask(L, d, r, n, B, lens=None, grads=True, C=3, n_max=None, dtype=pb.PAC_F32, flags=0):
        ctx = pb.pac_create(L, d, n_max or n, r, C, B, 64, dtype, flags)
        try:
            return pb.pac_f32_plan(ctx, lens, B if lens is None else len(lens), grads), pb.pac_workspace_bytes(ctx)
        finally:
            pb.pac_destroy(ctx)

    def gram(*a, **kw):
        return ask(*a, **kw)[0]["gram"]

    assert ask(12, 768, 96, 128, 32)[0] == dict(gram=1, proj=32, splits=1, wc=1)   # T5-Base-shaped
    assert ask(2, 64, 32, 400, 8)[0] == dict(gram=1, proj=16, splits=8, wc=1)
    for grads in (True, False):
        assert gram(12, 768, 96, 128, 32, grads=grads) and gram(4, 256, 32, 64, 8, grads=grads)
        assert not gram(12, 768, 96, 128, 32, grads=grads, flags=pb.PAC_FLAG_PER_LAYER)
        assert not gram(12, 768, 96, 128, 32, grads=grads, dtype=pb.PAC_BF16)
        assert not gram(12, 768, 160, 128, 32, grads=grads)       # a width without kernels
        assert not gram(17, 768, 96, 128, 32, grads=grads)        # too many layers for a compute unit's LDS
        assert not gram(1, 768, 96, 128, 32, grads=grads)
        assert not gram(14, 256, 128, 512, 32, grads=grads)       # 64 x 64 tiles fill the chip (1981 / 1459, 827 / 518)
        assert not gram(31, 128, 64, 256, 32, grads=grads)        # (1297 / 1173, 502 / 425)
        assert not gram(8, 384, 192, 1, 1, grads=grads)           # (271 / 242, 129 / 114)
        assert not gram(5, 512, 256, 16, 1, grads=grads)          # (201 / 192, 100 / 91)
        assert gram(14, 512, 128, 128, 8, grads=grads)
    # steps one way, forward-only calls the other (2576 / 2650, 925 / 704)
    # and by the batch, whatever the largest is
    big = dict(n_max=1024, B=4)
    assert gram(8, 1024, 192, 1024, 4) and not gram(8, 1024, 192, lens=[16], n=16, **big)
    # reserved: one formulation where every batch takes it, the larger of both otherwise
    _, every = ask(12, 768, 96, 128, 32)
    _, per_layer = ask(12, 768, 96, 128, 32, flags=pb.PAC_FLAG_PER_LAYER)
    assert every < per_layer
    _, both = ask(8, 1024, 192, 1024, 4)
    _, per_layer = ask(8, 1024, 192, 1024, 4, flags=pb.PAC_FLAG_PER_LAYER)
    assert both >= per_layer
    # within the static entry's workspace alone: the Gram-matrix formulation for every batch
    plan, ws = ask(5, 1952, 256, 16, 32, grads=False)
    assert plan["gram"] and ws <= pb.PAC_STATIC_WORKSPACE_BYTES < ask(5, 1952, 256, 16, 32, flags=pb.PAC_FLAG_PER_LAYER)[1]
    with pytest.raises(pb.PacError) as e:
        ask(12, 768, 96, 128, 2, [128, 129])
    assert e.value.status == pb.PAC_ERR_RANGE
    assert pb.lib().pac_f32_plan(None, None, 1, 1, (C.c_int32 * 4)()) == pb.PAC_ERR_NULL


@pytest.mark.parametrize("shape", [(31, 128, 32, 26, 1), (13, 256, 128, 64, 4), (12, 768, 96, 16, 2)])
def test_fp32_calls_take_the_workspace_of_either_formulation(shape):
    """A workspace that holds the per-layer kernels alone, or the Gram-matrix formulation alone, is no error; a byte less is."""
    L, d, r, n, B = shape
    need = []
    for flags in (0, pb.PAC_FLAG_PER_LAYER):
        ctx = pb.pac_create(L, d, n, r, 3, B, 8, pb.PAC_F32, flags)
        need.append(pb.pac_workspace_bytes(ctx))
        pb.pac_destroy(ctx)
    ctx = pb.pac_create(L, d, n, r, 3, B, 8, pb.PAC_F32)
    dev, idp = 0x7000_0000_0000, np.zeros(1, dtype=np.int64).ctypes.data_as(C.c_void_p)
    call = lambda ws_bytes: pb.lib().pac_adapter_loss_grad(ctx, dev, idp, 1, dev, dev, dev, ws_bytes, dev, None, None, None)
    try:  # (sample 0 was never filled: where the workspace is accepted, the state is the next thing found wrong)
        assert call(need[0]) == call(min(need)) == pb.PAC_ERR_STATE
        assert call(min(need) - 1) == pb.PAC_ERR_WORKSPACE
    finally:
        pb.pac_destroy(ctx)


def test_per_layer_workspace_holds_the_splits_that_run():
    """bf16 weight gradients walk 128 token rows a step: 128 rows are one split and reserve one set of partial sums."""
    def ws(n):
        ctx = pb.pac_create(1, 512, n, 512, 2, 1, 1, pb.PAC_BF16, flags=pb.PAC_FLAG_PER_LAYER)
        try:
            return pb.pac_workspace_bytes(ctx)
        finally:
            pb.pac_destroy(ctx)
    partials = 4 * (2 * 512 * 512 + 512 + 512 + 1)
    assert ws(128) - ws(64) < partials       # the 64 rows more need a quarter of that
    assert ws(129) - ws(128) > partials


def test_ladder_tiles_by_the_work_there_is():
    """Host logic: tiles of the ladder's contractions over the tokens, at most 64 columns where the chip is not filled twice."""
    def ask(L, d, w, n, B, heads):
        ctx = pb.pac_create(L, d, n, w, 3, B, 64, pb.PAC_BF16)
        try:
            return pb.pac_ladder_tiles(ctx, heads)
        finally:
            pb.pac_destroy(ctx)
    assert ask(12, 768, 96, 128, 32, 12) == ([(64, 96), (48, 96), (48, 96), (48, 128), (64, 96)], 4)   # T5-Base-shaped
    assert ask(6, 448, 64, 36, 27, 8) == ([(64, 64)] * 5, 4)                                           # 384 workgroups
    assert ask(3, 416, 64, 256, 17, 4)[0] == [(64, 64)] * 5
    with pytest.raises(pb.PacError) as e:
        ask(2, 64, 32, 16, 4, 3)
    assert e.value.status == pb.PAC_ERR_UNSUPPORTED
    assert pb.lib().pac_ladder_tiles(None, 4, (C.c_int32 * 11)()) == pb.PAC_ERR_NULL


def test_linear_layer_kernel_and_tiles():
    """Host logic: both kernels and all tiles of the quantised linear layer, at the lines between them."""
    t = lambda *a: tuple(pb.pac_dequant_linear_tiles(*a).values())
    assert t(4096, 4096, 4096, 64, 8) == t(4096, 4096, 4096, 32, 4, True) == (1, 256, 128)
    assert t(4096, 4096, 4096, 128, 8) == (0, 128, 128)
    assert t(1664, 4096, 1920, 64, 8) == (1, 128, 128) and t(1536, 4096, 2048, 64, 8) == (1, 128, 64)  # 195 and 192 tiles
    assert t(2441, 416, 2794, 32, 8) == (1, 128, 128) and t(2441, 448, 2794, 32, 8) == (1, 256, 128)   # short K
    assert t(2546, 352, 1558, 32, 8) == (0, 64, 64)                                                    # (16.6 us / 14.1)
    assert t(2048, 4096, 2048, 128, 8) == (0, 64, 64) and t(2048, 4096, 2049, 128, 8) == (0, 128, 128)
    assert t(2048, 1920, 2560, 96, 8) == (0, 64, 64) and t(2048, 1920, 2561, 96, 8) == (0, 128, 128)
    assert t(128, 4096, 4096, 64, 8) == (1, 128, 64) and t(156, 1600, 197, 64, 4) == (0, 64, 64)
    assert t(527, 1536, 1500, 64, 4) == (1, 128, 64) and t(527, 1536, 1500, 64, 4, True) == (0, 64, 64)
    assert t(22, 928, 3067, 32, 8) == (1, 128, 64) and t(312, 576, 211, 32, 4) == (0, 64, 64)
    assert t(47, 1216, 178, 32, 4) == (0, 64, 64) and t(47, 2304, 178, 32, 4) == (1, 128, 64)          # a handful of tiles
    for bad, status in (((0, 64, 8, 32, 8), pb.PAC_ERR_SHAPE), ((4, 100, 8, 32, 8), pb.PAC_ERR_SHAPE),
                        ((4, 64, 8, 32, 5), pb.PAC_ERR_SHAPE), ((4, 64, 8, 48, 8), pb.PAC_ERR_RANGE)):
        with pytest.raises(pb.PacError) as e:
            t(*bad)
        assert e.value.status == status
    assert pb.lib().pac_dequant_linear_tiles(4, 64, 8, 32, 8, 0, None) == pb.PAC_ERR_NULL


def test_chain_plan_per_batch():
    """Host logic: how the layer-by-layer chains are cut, and the tiles of the widest contraction."""
    def plan(L, d, n, r, B, lens=None, **kw):
        ctx = pb.pac_create(L, d, n, r, 3, B, 64, pb.PAC_BF16, **kw)
        try:
            return tuple(pb.pac_chain_plan(ctx, lens, B).values())
        finally:
            pb.pac_destroy(ctx)
    assert plan(32, 4096, 256, 256, 16) == (8, 4, 1, 4, 256, 256)              # LLaMA-7B-shaped: halves
    assert plan(32, 4096, 1024, 512, 8, [640] * 8) == (16, 2, 1, 13, 256, 256)  # long sequences
    assert plan(14, 32, 4200, 160, 2) == (3, 6, 0, 2, 128, 128)                # many tokens on few weights: no room for ranges
    assert plan(8, 576, 627, 224, 8) == (2, 4, 1, 1, 128, 128)                 # K steps of 32: no rounds (20.9 us / 23.8)
    assert plan(4, 512, 64, 224, 8) == (1, 4, 1, 0, 0, 0)                      # one group
    assert plan(12, 768, 128, 96, 32) == (0, 0, 0, 0, 0, 0)                    # single-launch chains
    assert plan(12, 768, 128, 96, 32, flags=pb.PAC_FLAG_LAYER_CHAIN)[:3] == (2, 8, 1)
    with pytest.raises(pb.PacError) as e:
        plan(32, 4096, 256, 256, 2, [256, 0])
    assert e.value.status == pb.PAC_ERR_RANGE
    assert pb.lib().pac_chain_plan(None, None, 1, (C.c_int32 * 6)()) == pb.PAC_ERR_NULL


def test_argument_errors_are_caught_before_any_launch():
    """Fake (never dereferenced) device addresses: every call below must fail on the host."""
    ctx = pb.pac_create(2, 64, 16, 32, 3, 4, 8, pb.PAC_BF16)
    lib = pb.lib()
    dev = 0x7000_0000_0000          # aligned, never touched
    ids = np.array([0, 1], dtype=np.int64)
    idp = ids.ctypes.data_as(C.c_void_p)
    big = 1 << 30
    try:
        assert lib.pac_cache_fill(ctx, None, big, idp, 2, dev, pb.PAC_F32, None, None) == pb.PAC_ERR_NULL
        assert lib.pac_cache_fill(ctx, dev + 8, big, idp, 2, dev, pb.PAC_F32, None, None) == pb.PAC_ERR_ALIGN
        assert lib.pac_cache_fill(ctx, dev, big, idp, -1, dev, pb.PAC_F32, None, None) == pb.PAC_ERR_RANGE
        assert lib.pac_cache_fill(ctx, dev, big, idp, 2, dev, 9, None, None) == pb.PAC_ERR_SHAPE
        assert lib.pac_cache_fill(ctx, dev, 100, idp, 2, dev, pb.PAC_F32, None, None) == pb.PAC_ERR_WORKSPACE
        bad_ids = np.array([0, 8], dtype=np.int64)
        assert lib.pac_cache_fill(ctx, dev, big, bad_ids.ctypes.data_as(C.c_void_p), 2, dev, pb.PAC_F32, None,
                                  None) == pb.PAC_ERR_RANGE
        dup = np.array([3, 3], dtype=np.int64)
        assert lib.pac_cache_fill(ctx, dev, big, dup.ctypes.data_as(C.c_void_p), 2, dev, pb.PAC_F32, None,
                                  None) == pb.PAC_ERR_RANGE
        lens = np.array([4, 17], dtype=np.int32)
        assert lib.pac_cache_fill(ctx, dev, big, idp, 2, dev, pb.PAC_F32, lens.ctypes.data_as(C.c_void_p),
                                  None) == pb.PAC_ERR_RANGE
        assert lib.pac_cache_fill(ctx, dev, big, idp, 0, dev, pb.PAC_F32, None, None) == pb.PAC_OK
        with pytest.raises(pb.PacError) as e:
            pb.pac_cache_lookup(ctx, 0)
        assert e.value.status == pb.PAC_ERR_STATE

        ws = pb.pac_workspace_bytes(ctx)
        call = lambda **k: lib.pac_adapter_loss_grad(
            ctx, k.get("cache", dev), k.get("ids", idp), k.get("B", 2), k.get("labels", dev),
            k.get("params", dev), k.get("ws", dev), k.get("ws_bytes", ws), k.get("loss", dev), None, None, None)
        assert call(cache=None) == pb.PAC_ERR_NULL
        assert call(loss=None) == pb.PAC_ERR_NULL
        assert call(ws=dev + 16) == pb.PAC_ERR_ALIGN
        assert call(ws_bytes=ws - 1) == pb.PAC_ERR_WORKSPACE
        assert call(B=0) == pb.PAC_ERR_RANGE and call(B=5) == pb.PAC_ERR_RANGE
        assert call() == pb.PAC_ERR_STATE            # samples 0 and 1 were never filled
        hp = pb.pac_adamw(1e-3, 0.9, 0.999, 1e-8, 0.01)
        st = C.c_int64(0)
        stepcall = lambda hp_, st_: lib.pac_adapter_step(ctx, dev, idp, 2, dev, dev, dev, dev, st_, hp_, dev, ws,
                                                         dev, None, None)
        assert stepcall(None, C.byref(st)) == pb.PAC_ERR_NULL
        assert stepcall(C.byref(pb.pac_adamw(1e-3, 1.0, 0.999, 1e-8, 0.0)), C.byref(st)) == pb.PAC_ERR_RANGE
        assert stepcall(C.byref(hp), C.byref(C.c_int64(-1))) == pb.PAC_ERR_RANGE
        assert stepcall(C.byref(hp), C.byref(st)) == pb.PAC_ERR_STATE and st.value == 0
        # measurement probes: argument errors before any launch
        assert lib.pac_probe_hbm_read(None, 1024, dev, None) == pb.PAC_ERR_NULL
        assert lib.pac_probe_hbm_read(dev, 0, dev, None) == pb.PAC_ERR_RANGE
        assert lib.pac_probe_hbm_read(dev, 1000, dev, None) == pb.PAC_ERR_RANGE
        assert lib.pac_probe_hbm_read(dev + 8, 1024, dev, None) == pb.PAC_ERR_ALIGN
        assert lib.pac_probe_mfma_bf16(0, dev, None) == pb.PAC_ERR_RANGE
        assert lib.pac_probe_mfma_bf16(10, None, None) == pb.PAC_ERR_NULL
        assert pb.pac_probe_mfma_flops(1) == 4 * 2 * 32 * 32 * 16 * 4 * 1024
        assert lib.pac_profile_end(ctx, 32, None, None, None) == pb.PAC_ERR_NULL
        for s in range(9):
            assert isinstance(pb.status_str(s), str) and pb.status_str(s)
    finally:
        pb.pac_destroy(ctx)


def test_ladder_argument_errors_are_caught_before_any_launch():
    """The ladder's calls (include/pac_ladder.h) on fake device addresses: every call must fail on the host."""
    ctx = pb.pac_create(2, 64, 16, 32, 3, 4, 8, pb.PAC_BF16)
    lib = pb.lib()
    dev = 0x7000_0000_0000
    ids = np.array([0, 1], dtype=np.int64)
    idp = ids.ctypes.data_as(C.c_void_p)
    try:
        w, d, f, L, Cc = 32, 64, 128, 2, 3
        per_layer = d * w + w + 2 * w + 3 * w * w + 3 * w + w * w + w + 2 * w + w * f + f + f * w + w + 4
        assert pb.pac_ladder_param_count(ctx) == L * per_layer + w * d + d + d * Cc + Cc
        assert lib.pac_ladder_param_count(None) == -1
        assert pb.pac_ladder_workspace_bytes(ctx, 3) == -1        # 32 / 3 is not a whole head width
        assert pb.pac_ladder_workspace_bytes(ctx, 16) == -1       # head width 2 is not supported
        ws = pb.pac_ladder_workspace_bytes(ctx, 4)
        assert ws > 0 and ws % 256 == 0
        call = lambda **k: lib.pac_ladder_loss_grad(
            ctx, k.get("cache", dev), k.get("ids", idp), k.get("B", 2), k.get("labels", dev), k.get("heads", 4),
            k.get("params", dev), k.get("ws", dev), k.get("ws_bytes", ws), k.get("loss", dev), None, None, None)
        assert call(cache=None) == pb.PAC_ERR_NULL and call(loss=None) == pb.PAC_ERR_NULL
        assert call(params=dev + 4) == pb.PAC_ERR_ALIGN and call(ws=dev + 16) == pb.PAC_ERR_ALIGN
        assert call(heads=3) == pb.PAC_ERR_UNSUPPORTED
        assert call(ws_bytes=ws - 1) == pb.PAC_ERR_WORKSPACE
        assert call(B=0) == pb.PAC_ERR_RANGE and call(B=5) == pb.PAC_ERR_RANGE
        assert call() == pb.PAC_ERR_STATE                         # samples 0 and 1 were never filled
        hp = pb.pac_adamw(1e-3, 0.9, 0.999, 1e-8, 0.01)
        st = C.c_int64(0)
        step = lambda hp_, st_, m_=dev: lib.pac_ladder_step(ctx, dev, idp, 2, dev, 4, dev, m_, dev, st_, hp_, dev, ws, dev,
                                                            None, None)
        assert step(None, C.byref(st)) == pb.PAC_ERR_NULL and step(C.byref(hp), C.byref(st), None) == pb.PAC_ERR_NULL
        assert step(C.byref(pb.pac_adamw(1e-3, 0.9, 1.0, 1e-8, 0.0)), C.byref(st)) == pb.PAC_ERR_RANGE
        assert step(C.byref(hp), C.byref(C.c_int64(-1))) == pb.PAC_ERR_RANGE
        assert step(C.byref(hp), C.byref(st)) == pb.PAC_ERR_STATE and st.value == 0
        assert lib.pac_probe_hbm_update(dev, dev, dev, None, 1024, None) == pb.PAC_ERR_NULL
        assert lib.pac_probe_hbm_update(dev, dev, dev, dev, 1022, None) == pb.PAC_ERR_RANGE
        assert lib.pac_probe_hbm_update(dev, dev + 8, dev, dev, 1024, None) == pb.PAC_ERR_ALIGN
    finally:
        pb.pac_destroy(ctx)
