"""GPU parity of the first epoch's storage side (block-wise quantisation, its inverse, the mixed-precision linear
layer with and without the fused cache fill) against oracle/quant_oracle.c, through the C ABI.

Bars: integer codes and quantisation constants bit-exact (both sides decide the integer in 32-bit arithmetic);
dequantised values bit-exact (one 32-bit division); the linear layer within 1e-5 relative L2 of the double-precision
oracle (fp32 accumulation of exact products is all that differs); values written to a bf16 cache within one bf16
rounding step of the oracle's value."""
import numpy as np
import pytest
import torch

from oracle import oracle as orc
from oracle import quant_oracle as qo
from paper_2408_10746_amd import binding as pb
from paper_2408_10746_amd import inputs
from paper_2408_10746_amd.inputs import Workload

pytestmark = pytest.mark.gpu


def weights(rng, N, K, outliers=True):
    """Weights with the heavy-tailed structure that motivates block-wise constants: N(0, 1/K) plus a few large entries."""
    W = (rng.standard_normal((N, K)) / np.sqrt(K)).astype(np.float32)
    if outliers:
        idx = rng.integers(0, N * K, size=max(1, N * K // 500))
        W.ravel()[idx] *= 20.0
    return W


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("n,block", [(64 * 300 + 40, 64), (5000, 128), (7, 64), (4096 * 33, 4096), (1000, 2),
                                     # blocks that tile the tensor exactly: the four-values-per-lane form
                                     (64 * 1001, 64), (256 * 37, 256), (8 * 1001, 8), (4 * 999, 4), (128 * 513, 128),
                                     (32 * 70001, 32)])
def test_quant_and_dequant_bit_exact(n, block, bits):
    rng = np.random.default_rng(n + bits)
    x = (rng.standard_normal(n) * np.exp(rng.uniform(-4, 4, size=n))).astype(np.float32)
    x[:: max(1, n // 7)] = 0.0
    if n > 200:
        x[128:192] = 0.0                       # an all-zero block
        x[200] = np.float32(2.0) ** -130       # a denormal
    codes_ref, consts_ref = qo.quant(x, block, bits)
    xd = torch.from_numpy(x).cuda()
    codes = torch.zeros(codes_ref.size, dtype=torch.int8, device="cuda")
    consts = torch.zeros(consts_ref.size, dtype=torch.float32, device="cuda")
    pb.pac_quant_blockwise(xd.data_ptr(), n, block, bits, codes.data_ptr(), consts.data_ptr())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(consts.cpu().numpy().view(np.uint32), consts_ref.view(np.uint32))
    np.testing.assert_array_equal(codes.cpu().numpy(), codes_ref)
    out = torch.zeros(n, dtype=torch.float32, device="cuda")
    pb.pac_dequant_blockwise(codes.data_ptr(), consts.data_ptr(), n, block, bits, out.data_ptr())
    torch.cuda.synchronize()
    np.testing.assert_array_equal(out.cpu().numpy().view(np.uint32), qo.dequant(codes_ref, consts_ref, n, block, bits).view(np.uint32))


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,block", [(70, 128, 96, 64), (5, 64, 33, 32), (257, 768, 200, 128), (64, 1024, 64, 1024)])
def test_linear_layer_against_oracle(M, K, N, block, bits):
    check_linear_layer(M, K, N, block, bits)


# ragged at both edges on 272 and 289 tiles of 128 x 128 (or four times as many of 64 x 64), blocks of one to four K steps
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,block", [(2049, 64, 2001, 32), (2100, 192, 2033, 96), (2047, 192, 2100, 64), (2048, 256, 2048, 128)])
def test_linear_layer_on_wide_and_narrow_tiles(M, K, N, block, bits):
    check_linear_layer(M, K, N, block, bits)


# blocks that are an odd multiple of 32 take the large tiles from 321 on (361 here), up to 64 rows never do
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,block", [(2401, 64, 2200, 32), (2310, 192, 2311, 96), (2400, 96, 2001, 32), (40, 128, 33000, 64)])
def test_linear_layer_tiles_by_block_and_rows(M, K, N, block, bits):
    check_linear_layer(M, K, N, block, bits)


# blocks of 32 and 64, ragged at both edges: two and three K steps of 64, a last one of a single block of 32, long K on few
# tiles, a tile of a few rows and columns (the forms of k_dq_short by name: below)
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,block", [(2100, 160, 2100, 32), (2050, 128, 2111, 32), (1700, 192, 1799, 64), (129, 64, 24650, 64),
                                         (70, 96, 33000, 32), (300, 1536, 200, 64), (131, 1568, 70, 32), (5, 1184, 3, 32), (300, 512, 129, 32)])
def test_linear_layer_short_blocks(M, K, N, block, bits):
    check_linear_layer(M, K, N, block, bits)


# blocks longer than 64 with K steps of 64 on 128 x 128 tiles, ragged at both edges: one and two steps a block more than two
@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,block", [(2100, 384, 2111, 128), (2100, 512, 2111, 256)])
def test_linear_layer_long_blocks_on_wide_tiles(M, K, N, block, bits):
    assert pb.pac_dequant_linear_tiles(M, K, N, block, bits) == dict(short=0, rows=128, cols=128)
    check_linear_layer(M, K, N, block, bits)


def stored_layer(rng, N, K, block, bits):
    W = torch.from_numpy(weights(rng, N, K)).cuda()
    codes = torch.zeros((N, K * bits // 8), dtype=torch.int8, device="cuda")
    consts = torch.zeros((N, K // block), dtype=torch.float32, device="cuda")
    pb.pac_quant_blockwise(W.data_ptr(), N * K, block, bits, codes.data_ptr(), consts.data_ptr())
    return codes, consts


def linear(x, codes, consts, block, bits):
    M, K, N = *x.shape, codes.shape[0]
    y = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    pb.pac_dequant_linear(x.data_ptr(), M, K, codes.data_ptr(), consts.data_ptr(), N, block, bits, y.data_ptr())
    return y


# The kernel for short blocks on each of its tiles, ragged at both edges: last tiles of 12 and 20 rows, last steps of one block
# of 32.
DENSE = [(300, 2048, 2000, 64, (1, 128, 64)), (300, 1184, 200, 32, (1, 128, 64)), (20, 1184, 700, 32, (1, 128, 64)),
         (1700, 320, 1799, 64, (1, 128, 128)), (1700, 512, 1799, 64, (1, 128, 128)), (2100, 416, 2111, 32, (1, 128, 128)),
         (2060, 448, 2111, 64, (1, 256, 128)), (2060, 480, 2111, 32, (1, 256, 128))]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,block,form", DENSE)
def test_linear_layer_short_blocks_on_each_tile(M, K, N, block, form, bits):
    assert tuple(pb.pac_dequant_linear_tiles(M, K, N, block, bits).values()) == form
    check_linear_layer(M, K, N, block, bits)


# tiles of 128 x 64, 128 x 128 and 256 x 128 of the kernel for short blocks, 128 x 128 and 64 x 64 of the other one; ragged
# samples whose rows lie across the tiles' edges
FORMS = [(5, 37, 8192, 1760, 64, (1, 128, 64)), (5, 37, 3040, 448, 32, (1, 128, 64)), (20, 85, 960, 1824, 64, (1, 128, 128)),
         (20, 103, 480, 3712, 32, (1, 128, 128)), (20, 103, 768, 2144, 64, (1, 256, 128)), (20, 103, 672, 2144, 32, (1, 256, 128)),
         (20, 103, 256, 2144, 128, (0, 128, 128)), (20, 103, 96, 2144, 32, (0, 64, 64))]


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("B,n_max,K,N,block,form", FORMS)
def test_linear_layer_to_cache_has_the_dense_call_s_bits(B, n_max, K, N, block, form, bits):
    """Every epilogue that writes the cache, in both cache dtypes, against the dense output (rounded to nearest even)."""
    from paper_2408_10746_amd.runtime import Session
    assert tuple(pb.pac_dequant_linear_tiles(B * n_max, K, N, block, bits, to_cache=True).values()) == form
    rng = np.random.default_rng(B + K + bits)
    codes, consts = stored_layer(rng, N, K, block, bits)
    x = torch.from_numpy(rng.standard_normal((B * n_max, K)).astype(np.float32)).to(torch.bfloat16).cuda()
    y = linear(x, codes, consts, block, bits).view(B, n_max, N)
    assert torch.isfinite(y).all()
    ids, lens = rng.permutation(B), rng.integers(1, n_max + 1, size=B).astype(np.int32)
    lens[:2] = 1, n_max
    for dtype in ("bf16", "f32"):
        w = Workload("qf", L=2, d=N, n_max=n_max, B=B, r=32, C=2, N=B, cache_dtype=dtype)
        by_id = np.empty_like(lens)
        by_id[ids] = lens
        sess = Session(w, lens=by_id)
        sess.cache.fill_(0x55)
        pb.pac_dequant_linear_to_cache(sess.ctx, sess.cache.data_ptr(), sess.cache_bytes, ids, lens, 1, x.data_ptr(), K,
                                       codes.data_ptr(), consts.data_ptr(), block, bits)
        torch.cuda.synchronize()
        for b, sid in enumerate(ids):
            got, want = sess.cache_block(int(sid)), y[b, :lens[b]]
            want = want.cpu().numpy() if dtype == "f32" else want.to(torch.bfloat16).view(torch.int16).cpu().numpy().view(np.uint16)
            assert np.array_equal(got[1], want)
            assert (np.ascontiguousarray(got[0]).view(np.uint8) == 0x55).all()  # the other layer's rows stay as they were


@pytest.mark.parametrize("bits", [8, 4])
@pytest.mark.parametrize("M,K,N,block,form", [c for c in DENSE if c[0] > 60])
def test_linear_layer_forms_give_the_same_bits(M, K, N, block, form, bits):
    """Rows and columns of a large call alone, where the kernel for short blocks is not taken."""
    assert tuple(pb.pac_dequant_linear_tiles(M, K, N, block, bits).values()) == form
    assert tuple(pb.pac_dequant_linear_tiles(60, K, 90, block, bits).values()) == (0, 64, 64)
    rng = np.random.default_rng(M + K + bits)
    codes, consts = stored_layer(rng, N, K, block, bits)
    x = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).to(torch.bfloat16).cuda()
    y = linear(x, codes, consts, block, bits)
    for m, n in ((0, 0), (M - 60, N - 90), (M // 3, N // 2)):
        part = linear(x[m:m + 60].clone(), codes[n:n + 90].clone(), consts[n:n + 90].clone(), block, bits)
        assert torch.equal(part, y[m:m + 60, n:n + 90])


def check_linear_layer(M, K, N, block, bits):
    rng = np.random.default_rng(M + K + bits)
    W = weights(rng, N, K)
    x16 = torch.from_numpy(rng.standard_normal((M, K)).astype(np.float32)).to(torch.bfloat16)
    codes_ref, consts_ref = qo.quant(W, block, bits)
    ref = qo.dequant_linear(x16.float().numpy(), codes_ref, consts_ref, N, block, bits)
    # the stored form is produced on the device as well (bit-equal to the oracle's, checked above)
    Wd = torch.from_numpy(W).cuda()
    codes = torch.zeros(codes_ref.size, dtype=torch.int8, device="cuda")
    consts = torch.zeros(consts_ref.size, dtype=torch.float32, device="cuda")
    pb.pac_quant_blockwise(Wd.data_ptr(), N * K, block, bits, codes.data_ptr(), consts.data_ptr())
    xd = x16.cuda()
    y = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    pb.pac_dequant_linear(xd.data_ptr(), M, K, codes.data_ptr(), consts.data_ptr(), N, block, bits, y.data_ptr())
    torch.cuda.synchronize()
    assert np.array_equal(codes.cpu().numpy(), codes_ref)
    got = y.cpu().numpy().astype(np.float64)
    assert np.isfinite(got).all()
    err = np.linalg.norm(got - ref) / np.linalg.norm(ref)
    assert err <= 1e-5, err
    # element-wise: fp32 accumulation of K exact products, against the sum of their magnitudes
    mag = np.abs(x16.float().numpy().astype(np.float64)) @ np.abs(
        qo.dequant(codes_ref, consts_ref, N * K, block, bits).reshape(N, K).astype(np.float64)).T
    assert np.max(np.abs(got - ref) / mag) <= 1e-5


@pytest.mark.parametrize("dtype,bits", [("bf16", 8), ("bf16", 4), ("f32", 8)])
def test_linear_layer_with_fused_cache_fill(dtype, bits):
    """Layer by layer, the quantised projection's output goes straight into the cache (ragged samples, two calls,
    a sample registered by an ordinary fill first); the cache then holds what filling it with the oracle's outputs
    would hold, to one rounding step of the cache dtype."""
    w = Workload("qc", L=3, d=96, n_max=21, B=4, r=32, C=2, N=6, cache_dtype=dtype)
    K, block = 128, 64
    rng = np.random.default_rng(17)
    lens = np.array([21, 1, 13, 8, 21, 5], dtype=np.int32)
    from paper_2408_10746_amd.runtime import Session
    sess = Session(w, lens=lens)
    Ws = [weights(rng, w.d, K) for _ in range(w.L)]
    x16 = torch.from_numpy(rng.standard_normal((w.N, w.L, w.n_max, K)).astype(np.float32)).to(torch.bfloat16)
    # sample 3 is known before (an ordinary fill of zeros): its block must be reused, not appended again
    sess.cache_fill([3], np.zeros((1, w.L, w.n_max, w.d), dtype=np.float32), lens[[3]])
    order = [np.array([0, 3, 5]), np.array([4, 1, 2])]
    stored = []
    for l in range(w.L):
        codes_ref, consts_ref = qo.quant(Ws[l], block, bits)
        stored.append((codes_ref, consts_ref))
        codes = torch.from_numpy(codes_ref).cuda()
        consts = torch.from_numpy(consts_ref).cuda()
        for ids in order:
            xd = x16[ids, l].contiguous().cuda()
            pb.pac_dequant_linear_to_cache(sess.ctx, sess.cache.data_ptr(), sess.cache_bytes, ids, lens[ids], l,
                                           xd.data_ptr(), K, codes.data_ptr(), consts.data_ptr(), block, bits)
    torch.cuda.synchronize()
    # layout: fill order 3, then 0, 5, 4, 1, 2
    expect_off, pos = {}, 0
    for sid in [3, 0, 5, 4, 1, 2]:
        expect_off[sid] = pos
        pos += w.L * int(lens[sid]) * w.d
    for sid in range(w.N):
        off, ln = pb.pac_cache_lookup(sess.ctx, sid)
        assert off == expect_off[sid] and ln == lens[sid]
        got = sess.cache_block(sid)
        for l in range(w.L):
            ref = qo.dequant_linear(x16[sid, l, :ln].float().numpy(), stored[l][0], stored[l][1], w.d, block, bits)
            if dtype == "f32":
                np.testing.assert_allclose(got[l], ref, rtol=0, atol=1e-5 * np.abs(ref).max())
            else:
                val = orc.widen(got[l].ravel()).reshape(ln, w.d).astype(np.float64)
                # one bf16 rounding step: half a unit in the last place of an 8-bit significand, plus the fp32 sum's error
                assert np.all(np.abs(val - ref) <= np.abs(ref) * 2.0 ** -8 + 1e-5 * np.abs(ref).max())
                # and most values are the correctly rounded ones
                exact = np.array([orc.f32_to_bf16_bits(float(v)) for v in ref.ravel()[:500]], dtype=np.uint16)
                assert np.mean(exact == got[l].ravel()[:500]) > 0.98


def test_argument_errors_before_any_launch():
    lib = pb.lib()
    dev = 0x7000_0000_0000
    assert lib.pac_quant_blockwise(None, 10, 64, 8, dev, dev, None) == pb.PAC_ERR_NULL
    assert lib.pac_quant_blockwise(dev, 10, 64, 5, dev, dev, None) == pb.PAC_ERR_SHAPE
    assert lib.pac_quant_blockwise(dev, 10, 3, 4, dev, dev, None) == pb.PAC_ERR_RANGE
    assert lib.pac_quant_blockwise(dev, -1, 64, 8, dev, dev, None) == pb.PAC_ERR_RANGE
    assert lib.pac_dequant_linear(dev, 4, 100, dev, dev, 8, 32, 8, dev, None) == pb.PAC_ERR_SHAPE
    assert lib.pac_dequant_linear(dev, 4, 128, dev, dev, 8, 48, 8, dev, None) == pb.PAC_ERR_RANGE
    assert lib.pac_dequant_linear(dev + 2, 4, 128, dev, dev, 8, 64, 8, dev, None) == pb.PAC_ERR_ALIGN
    assert lib.pac_dequant_linear(dev, 4, 128, dev, dev, 8, 64, 8, None, None) == pb.PAC_ERR_NULL
