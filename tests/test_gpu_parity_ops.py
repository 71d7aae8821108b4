"""GPU parity of every operator against the fp64 oracle, at sizes the oracle
evaluates in full: the tiny fp32 decoder layer (tolerance 1e-5) and bf16 shapes
that span several kernel tiles with ragged tails in every dimension
(tolerance 2e-2), plus the degenerate cases (single row, single key, empty
prompts, zero-length contexts, invalid page ids).  All calls go through the C
ABI via the ctypes binding."""
import math

import numpy as np
import pytest

import oracle
import workloads as wl
from parity_util import assert_close, cuda, f64, gen, linear_plan, say, torch_dtype

pytestmark = pytest.mark.gpu


TILES = {"256x256": 0, "192x256": 1, "256x128": 2, "256x256w8": 3}  # opscale_tune GEMM_TILE values
SCHEDULES = {"grid": 0, "list": 1}                   # opscale_tune PREFILL_SCHEDULE values


@pytest.fixture(scope="module")
def ops():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_13499_amd as ops
    ops.load()
    return ops


# ------------------------------------------------------------------ RMSNorm --
@pytest.mark.parametrize("dtype,M,H", [
    ("f32", 128, 256), ("f32", 5, 4), ("bf16", 37, 4096), ("bf16", 3, 8192),
    ("bf16", 9, 24), ("bf16", 2, 24576), ("bf16", 1, 4096), ("f32", 7, 16384 + 4),
])
def test_rmsnorm(ops, dtype, M, H):
    import torch
    say(f"rmsnorm {dtype} M={M} H={H}")
    x = gen(11, "x", (M, H), dtype)
    w = gen(11, "w_norm", (H,), dtype, std=0.02, mean=1.0)
    y = ops.opscale_rmsnorm(cuda(x), cuda(w), eps=1e-5)
    torch.cuda.synchronize()
    assert_close(f64(y.cpu()), oracle.rmsnorm(f64(x), f64(w), 1e-5), dtype, "rmsnorm")


def test_rmsnorm_inplace_and_unit_gain(ops):
    import torch
    x = gen(12, "x", (64, 4096), "bf16")
    xd = cuda(x)
    ops.opscale_rmsnorm(xd, cuda(torch.ones(4096, dtype=torch.bfloat16)), y=xd, eps=0.0)
    torch.cuda.synchronize()
    y = f64(xd.cpu())
    # unit gain, eps 0: every row has RMS 1 up to bf16 output rounding
    rms = np.sqrt(np.mean(y * y, axis=1))
    assert np.abs(rms - 1).max() < 4e-3
    assert_close(y, oracle.rmsnorm(f64(x), np.ones(4096), 0.0), "bf16", "in-place rmsnorm")


# ------------------------------------------------------------------- linear --
@pytest.mark.parametrize("dtype,M,N,K,bias", [
    ("f32", 128, 768, 256, False), ("f32", 128, 256, 256, False), ("f32", 128, 1376, 256, False),
    ("f32", 128, 256, 688, False), ("f32", 3, 12, 20, True),
    ("bf16", 300, 264, 200, False), ("bf16", 513, 1024, 4096, False), ("bf16", 1, 256, 64, False),
    ("bf16", 257, 520, 136, True), ("bf16", 64, 6144, 4096, False), ("bf16", 40, 256, 14336, False),
    ("bf16", 1000, 768, 8, False),
])
def test_linear(ops, dtype, M, N, K, bias):
    import torch
    say(f"linear {dtype} M={M} N={N} K={K} bias={bias}")
    x = gen(21, "x", (M, K), dtype)
    W = gen(21, "w_qkv", (N, K), dtype, std=0.02)
    b = gen(21, "bias", (N,), dtype) if bias else None
    y = ops.opscale_linear(cuda(x), cuda(W), None if b is None else cuda(b))
    torch.cuda.synchronize()
    assert_close(f64(y.cpu()), oracle.linear(f64(x), f64(W), None if b is None else f64(b)), dtype, "linear")


@pytest.mark.parametrize("M,N,K,bias", [(33, 36, 4, True), (1, 4, 28, False), (31, 100, 36, True), (65, 64, 132, False),
                                        (64, 32, 260, True), (1500, 1532, 100, True), (1536, 2048, 64, False),
                                        (1537, 2048, 132, False), (2000, 1540, 32, True)])
def test_linear_f32_tiles(ops, M, N, K, bias):
    """Both fp32 kernels: the 32x32 tile (K split over its waves in blocks of
    32: fewer blocks than waves, partial blocks, ragged M and N), and from 192
    tiles of 128x128 the large one (the last three shapes; 144 tiles before
    them)."""
    import torch
    say(f"linear f32 tiles M={M} N={N} K={K} bias={bias}")
    x = gen(31, "x", (M, K), "f32")
    W = gen(31, "w_qkv", (N, K), "f32", std=0.02)
    b = gen(31, "bias", (N,), "f32") if bias else None
    args = (cuda(x), cuda(W), None if b is None else cuda(b))
    y, y2 = ops.opscale_linear(*args), ops.opscale_linear(*args)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    assert_close(f64(y.cpu()), oracle.linear(f64(x), f64(W), None if b is None else f64(b)), "f32", "linear f32")


@pytest.mark.parametrize("tile", ["256x256", "192x256", "256x128", "256x256w8"])
@pytest.mark.parametrize("M,N,K,bias", [(300, 264, 200, True), (513, 1024, 4096, False), (1, 256, 64, False),
                                        (700, 520, 136, False)])
def test_linear_each_tile(ops, tune, tile, M, N, K, bias):
    """Every bf16 tile that the tile knob names, with ragged M, N and K."""
    import torch
    say(f"linear bf16 tile={tile} M={M} N={N} K={K} bias={bias}")
    tune(gemm_tile=TILES[tile])
    x = gen(23, "x", (M, K), "bf16")
    W = gen(23, "w_qkv", (N, K), "bf16", std=0.02)
    b = gen(23, "bias", (N,), "bf16") if bias else None
    y = ops.opscale_linear(cuda(x), cuda(W), None if b is None else cuda(b))
    torch.cuda.synchronize()
    assert_close(f64(y.cpu()), oracle.linear(f64(x), f64(W), None if b is None else f64(b)), "bf16", "linear")


@pytest.mark.parametrize("M,N,K,bias", [
    (1, 256, 64, False), (3, 40, 96, True), (16, 6144, 4096, False), (17, 520, 128, True), (33, 8, 32, False),
    (64, 4096, 14336, False), (100, 1000, 4096, True), (129, 264, 256, False), (256, 6144, 4096, False),
    (256, 4104, 32, True),
])
@pytest.mark.parametrize("ng", [1, 2])
def test_linear_small_m(ops, tune, ng, M, N, K, bias):
    """The decode-batch path (M <= 256, K % 32 == 0), forced on, with 16 and
    32 columns per workgroup: every row-group count, N tails shorter than one
    column group, K of one k-step per wave and fewer k-steps than waves."""
    import torch
    tune(gemm_skinny=1, skinny_ng=ng)
    say(f"linear bf16 small-M NG={ng} M={M} N={N} K={K} bias={bias}")
    x = gen(24, "x", (M, K), "bf16")
    W = gen(24, "w_qkv", (N, K), "bf16", std=0.02)
    b = gen(24, "bias", (N,), "bf16") if bias else None
    y = ops.opscale_linear(cuda(x), cuda(W), None if b is None else cuda(b))
    y2 = ops.opscale_linear(cuda(x), cuda(W), None if b is None else cuda(b))
    torch.cuda.synchronize()
    assert torch.equal(y, y2)  # fixed reduction order
    assert_close(f64(y.cpu()), oracle.linear(f64(x), f64(W), None if b is None else f64(b)), "bf16", "linear")


@pytest.mark.parametrize("M,N,K,bias", [
    (256, 6144, 4096, False), (100, 520, 1032, True), (17, 4096, 14336, False), (200, 1000, 2048, True),
    (64, 8, 1024, False), (700, 4096, 4096, True), (64, 6144, 4096, True), (65, 1000, 2048, False),
    (96, 4096, 4096, False), (128, 28672, 1024, True), (256, 4096, 14336, False),
    (200, 16648, 1024, True), (256, 28672, 4096, False),
])
def test_linear_split_k(ops, tune, M, N, K, bias):
    """Decode-sized M with K split over workgroups (fp32 partials summed in
    split order), on each tile the path picks (64 or 128 rows up to 256, 256
    rows with 256 or 128 columns above): ragged M, N and K, a K range that
    does not divide evenly, bias; 129-256 rows whose 128-row tiles fill the
    GPU without a split (the last two cases); bitwise equal across calls.
    The partials live in the caller's workspace (poisoned before the call:
    its contents on entry must not matter); without one the same shapes take
    an unsplit path."""
    import torch
    tune(gemm_skinny=0, gemm_decode=0)
    say(f"linear bf16 split-K M={M} N={N} K={K} bias={bias}")
    x = gen(25, "x", (M, K), "bf16")
    W = gen(25, "w_qkv", (N, K), "bf16", std=0.02)
    b = gen(25, "bias", (N,), "bf16") if bias else None
    args = (cuda(x), cuda(W), None if b is None else cuda(b))
    need = ops.opscale_linear_workspace_size(M, N, K)
    ws = torch.full((max(need, 16),), 0x7f, dtype=torch.uint8, device="cuda")  # fp32 3.4e38 if read
    y = ops.opscale_linear(*args, workspace=ws)
    y2 = ops.opscale_linear(*args, workspace=ws)
    y0 = ops.opscale_linear(*args, workspace=False)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    ref = oracle.linear(f64(x), f64(W), None if b is None else f64(b))
    assert_close(f64(y.cpu()), ref, "bf16", "linear")
    assert_close(f64(y0.cpu()), ref, "bf16", "linear without a workspace")


@pytest.mark.parametrize("M,N,K,bias", [
    (256, 6144, 4096, False), (256, 4096, 4096, True), (256, 4096, 14336, False), (256, 28672, 4096, False),
    (200, 1000, 2048, True), (129, 264, 256, False), (100, 520, 1088, True), (65, 136, 64, True),
    (33, 8, 512, False), (1, 256, 64, False), (64, 6144, 4096, True), (256, 4104, 576, True),
    (256, 256, 16384, False), (128, 1304, 832, False),
])
def test_linear_decode_batch(ops, tune, M, N, K, bias):
    """The decode-batch kernel (weights streamed into registers, 128 columns
    and all M rows per workgroup), forced on: every row-block count (M up to
    64, 128, 256 and ragged between), N tails down to 8 columns and waves
    with no weight rows, K of one slice, ranges that are not a multiple of the
    8-slice round and uneven K ranges, K split over workgroups through the
    caller's workspace (poisoned: its contents on entry must not matter) or
    not at all; bitwise equal across calls.  Without a workspace a shape that
    would split takes another path."""
    import torch
    tune(gemm_decode=1)
    say(f"linear bf16 decode-batch M={M} N={N} K={K} bias={bias}")
    x = gen(28, "x", (M, K), "bf16")
    W = gen(28, "w_qkv", (N, K), "bf16", std=0.02)
    b = gen(28, "bias", (N,), "bf16") if bias else None
    args = (cuda(x), cuda(W), None if b is None else cuda(b))
    need = ops.opscale_linear_workspace_size(M, N, K)
    ws = torch.full((max(need, 16),), 0x7f, dtype=torch.uint8, device="cuda")
    y = ops.opscale_linear(*args, workspace=ws)
    y2 = ops.opscale_linear(*args, workspace=ws)
    y0 = ops.opscale_linear(*args, workspace=False)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    ref = oracle.linear(f64(x), f64(W), None if b is None else f64(b))
    assert_close(f64(y.cpu()), ref, "bf16", "linear")
    assert_close(f64(y0.cpu()), ref, "bf16", "linear without a workspace")


@pytest.mark.parametrize("M,N,K,bias", [
    (16, 10232, 1024, True), (17, 24584, 128, False), (32, 24576, 512, True), (33, 4096, 4096, False),
    (64, 6136, 1536, True), (65, 28672, 192, True), (128, 200, 4672, False), (100, 8, 1152, True), (2, 28664, 64, False),
    (48, 28664, 4096, True), (20, 57336, 1984, False),
])
def test_linear_decode_batch_shapes(ops, tune, M, N, K, bias):
    """The weight-streaming kernel at its edges: the most and fewest rows of
    each row-block count (16, 32, 64, 128), five to eight waves of 16 columns
    with a ragged last workgroup, one to nine K ranges of one to nine slices
    (each workgroup starting at another one), fewer slices than the ring
    holds and a partial last round of it; the last two shapes keep K whole: 64
    and 31 slices, eight and four rounds of the ring, which wraps in the middle."""
    import torch
    tune(gemm_decode=1)
    say(f"linear bf16 decode-batch shapes M={M} N={N} K={K} bias={bias}")
    x = gen(30, "x", (M, K), "bf16")
    W = gen(30, "w_qkv", (N, K), "bf16", std=0.02)
    b = gen(30, "bias", (N,), "bf16") if bias else None
    args = (cuda(x), cuda(W), None if b is None else cuda(b))
    need = ops.opscale_linear_workspace_size(M, N, K)
    ws = torch.full((max(need, 16),), 0x7f, dtype=torch.uint8, device="cuda")
    y, y2 = ops.opscale_linear(*args, workspace=ws), ops.opscale_linear(*args, workspace=ws)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    ref = oracle.linear(f64(x), f64(W), None if b is None else f64(b))
    assert_close(f64(y.cpu()), ref, "bf16", "linear")


@pytest.mark.parametrize("M", [8, 16, 32])
def test_linear_small_m_workspace_too_small(ops, M):
    """Rows that the small-M kernel takes without a workspace still run with
    one too small for the weight-streaming kernel's K ranges, on the path that
    takes none; more rows than that are refused."""
    import torch
    N, K = 6144, 4096
    assert ops.opscale_linear_workspace_size(M, N, K) > 16
    say(f"linear bf16 small-M with a small workspace M={M}")
    x, W = cuda(gen(34, "x", (64, K), "bf16")), cuda(gen(34, "w_qkv", (N, K), "bf16", std=0.02))
    ws = torch.zeros(16, dtype=torch.uint8, device="cuda")
    y = ops.opscale_linear(x[:M], W, workspace=ws)
    assert torch.equal(y, ops.opscale_linear(x[:M], W, workspace=False))
    big = torch.zeros(ops.opscale_linear_workspace_size(M, N, K) + 16, dtype=torch.uint8, device="cuda")
    assert torch.equal(y, ops.opscale_linear(x[:M], W, workspace=big[4:])), "a misaligned one"
    with pytest.raises(ops.OpscaleError) as e:
        ops.opscale_linear(x, W, workspace=ws)
    assert e.value.status == ops.OPSCALE_ERR_WORKSPACE


@pytest.mark.parametrize("M,N,K,bias", [
    (129, 264, 64, True), (130, 8, 200, False), (256, 520, 128, True), (385, 1032, 192, False), (257, 2056, 1000, True),
    (140, 5000, 1096, False), (256, 4096, 2048, True), (300, 776, 3080, True), (512, 4104, 4096, False),
    (1224, 1856, 8920, True), (1079, 13256, 584, True),
])
def test_linear_128_row_tiles(ops, tune, M, N, K, bias):
    """Past 128 rows and few 256x256 tiles: the 128x256 tile, whole (each
    column tile starting at another slice of K, one to 16 slices, the last a
    part of one) and split over K (ranges of 8 slices and more, the last one
    ragged), ragged M and N, through a poisoned workspace and without one; the
    last two shapes have nine and ten rows of tiles (a whole group of eight and a
    part of one), K past 8192, and 468 tiles (more than a round)."""
    import torch
    TILED, H4 = 2, 6
    plan = linear_plan(M, N, K)
    assert (plan.path, plan.cfg) == (TILED, H4), "not the 128x256 tile any more: take other sizes"
    say(f"linear bf16 128-row tiles M={M} N={N} K={K} bias={bias}")
    x = gen(32, "x", (M, K), "bf16")
    W = gen(32, "w_qkv", (N, K), "bf16", std=0.02)
    b = gen(32, "bias", (N,), "bf16") if bias else None
    args = (cuda(x), cuda(W), None if b is None else cuda(b))
    ws = torch.full((max(ops.opscale_linear_workspace_size(M, N, K), 16),), 0x7f, dtype=torch.uint8, device="cuda")
    y, y2 = ops.opscale_linear(*args, workspace=ws), ops.opscale_linear(*args, workspace=ws)
    y0 = ops.opscale_linear(*args, workspace=False)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    ref = oracle.linear(f64(x), f64(W), None if b is None else f64(b))
    assert_close(f64(y.cpu()), ref, "bf16", "linear 128-row tiles")
    assert_close(f64(y0.cpu()), ref, "bf16", "linear 128-row tiles without a workspace")


@pytest.mark.parametrize("M,N,K,bias", [(777, 1304, 2120, True), (2048, 6144, 4096, False), (256, 512, 64, True),
                                        (1300, 1000, 2056, True), (520, 384, 8256, False)])
def test_linear_four_and_eight_waves_agree(ops, tune, M, N, K, bias):
    """The 256x256 tile as four waves of 128x128 (accumulators in AGPRs) and
    as eight waves of 128x64 accumulate every output over the same k-steps
    with the same MFMA, so their results are bitwise equal; both match the
    oracle.  The four-wave ring gives the two-slice lead to x on the first,
    third and fifth shapes (tile groups of at most four tile-rows) and to W
    on the second and fourth (groups of more rows); the ragged K of the first
    and fourth ends in a partial slice, the fifth runs 129 slices and the
    third a single one."""
    import torch
    say(f"linear bf16 four vs eight waves M={M} N={N} K={K} bias={bias}")
    x = gen(27, "x", (M, K), "bf16")
    W = gen(27, "w_qkv", (N, K), "bf16", std=0.02)
    b = gen(27, "bias", (N,), "bf16") if bias else None
    args = (cuda(x), cuda(W), None if b is None else cuda(b))
    tune(gemm_tile=TILES["256x256"])
    y4 = ops.opscale_linear(*args)
    tune(gemm_tile=TILES["256x256w8"])
    y8 = ops.opscale_linear(*args)
    torch.cuda.synchronize()
    assert torch.equal(y4.view(torch.int16), y8.view(torch.int16))
    assert_close(f64(y4.cpu()), oracle.linear(f64(x), f64(W), None if b is None else f64(b)), "bf16", "linear")


@pytest.mark.parametrize("M,N,K,bias,tail", [
    (4300, 8200, 192, True, 0), (4300, 8200, 136, False, 0), (9000, 22000, 128, True, 0), (9000, 8456, 320, True, 0),
    (5200, 5000, 1032, True, 0), (4300, 4104, 2056, True, 4), (9000, 22000, 192, True, 0), (9200, 11000, 136, False, 0),
    (9000, 11000, 1032, True, 2), (16900, 5000, 8200, True, 4), (20736, 4096, 8256, False, 4),
])
def test_linear_chained_tiles(ops, tune, M, N, K, bias, tail):
    """More 256x256 tiles than one round of the CUs: from six rounds on a
    workgroup of the four-wave kernel runs a chain of them, the next tile's first
    slices loading while the previous one ends.  289 to 1224 tiles in two to five
    rounds (each tile a workgroup); 1344 to 1560 in six or seven (chains of two
    to single items); 3096 in 13 (chains of four to one).  K of three slices (the
    fewest chained), of two and a part, of two (never chained), of five, of
    sixteen and a part, past 8192 and ragged (x in the lead); a last round split
    over K in front of which chains end; ragged M and N.  Bitwise equal to the
    eight-wave kernel, which runs one tile per workgroup."""
    import torch
    say(f"linear bf16 chained tiles M={M} N={N} K={K} bias={bias} tail={tail}")
    tune(gemm_tile=TILES["256x256"])
    assert linear_plan(M, N, K).tail_splits == tail
    g = torch.Generator(device="cuda").manual_seed(29)
    normal = lambda *s, std=1.0: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    x, W = normal(M, K), normal(N, K, std=0.02)
    b = normal(N) if bias else None
    args = (x, W, b)
    got = []
    for tile in ("256x256", "256x256", "256x256w8"):
        tune(gemm_tile=TILES[tile])
        got.append(ops.opscale_linear(*args))
    torch.cuda.synchronize()
    assert torch.equal(got[0].view(torch.int16), got[1].view(torch.int16))
    assert torch.equal(got[0].view(torch.int16), got[2].view(torch.int16))
    rows = torch.from_numpy(np.unique(np.r_[0:M:397, 255:M:512, M - 1])).cuda()
    ref = x[rows].double() @ W.double().t()
    if b is not None:
        ref += b.double()
    assert_close(got[0][rows].double().cpu().numpy(), ref.cpu().numpy(), "bf16", "linear chained")


@pytest.mark.parametrize("tile,M,N,K,bias", [("256x256", 4352, 4096, 1024, True), ("256x256", 4300, 4104, 2056, False),
                                             ("192x256", 4352, 4096, 1024, False),
                                             ("256x256w8", 4300, 4104, 2056, True)])
def test_linear_split_tail(ops, tune, tile, M, N, K, bias):
    """More tiles than CUs with the last round at most half full: those tiles
    run as 2-4 K ranges (fp32 partials summed in split order) in the same
    launch as the others.  Ragged M, N and K, bias; bitwise equal across
    calls; the same result with the split tail turned off and with no
    workspace (which also plans no split)."""
    import torch
    say(f"linear bf16 split tail tile={tile} M={M} N={N} K={K} bias={bias}")
    tune(gemm_tile=TILES[tile])
    assert ops.opscale_linear_workspace_size(M, N, K) > 0
    x = gen(26, "x", (M, K), "bf16")
    W = gen(26, "w_qkv", (N, K), "bf16", std=0.02)
    b = gen(26, "bias", (N,), "bf16") if bias else None
    args = (cuda(x), cuda(W), None if b is None else cuda(b))
    y = ops.opscale_linear(*args)
    y2 = ops.opscale_linear(*args)
    yn = ops.opscale_linear(*args, workspace=False)
    tune(gemm_tail=0)
    y0 = ops.opscale_linear(*args)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    ref = oracle.linear(f64(x), f64(W), None if b is None else f64(b))
    assert_close(f64(y.cpu()), ref, "bf16", "linear split tail")
    assert_close(f64(y0.cpu()), ref, "bf16", "linear without split tail")
    assert torch.equal(y0, yn)  # both unsplit


def test_linear_identity_weight(ops):
    """W = I (bf16-exact) returns x exactly: no accumulation rounding occurs."""
    import torch
    x = gen(22, "x", (300, 512), "bf16")
    W = torch.eye(512, dtype=torch.bfloat16)
    y = ops.opscale_linear(cuda(x), cuda(W))
    torch.cuda.synchronize()
    assert torch.equal(y.cpu(), x)


# ------------------------------------------------------------------- SwiGLU --
@pytest.mark.parametrize("dtype,M,F", [("f32", 128, 688), ("bf16", 33, 1000), ("bf16", 1, 14336),
                                       ("bf16", 700, 8), ("f32", 3, 4)])
def test_swiglu(ops, dtype, M, F):
    import torch
    say(f"swiglu {dtype} M={M} F={F}")
    u = gen(31, "gate_up", (M, 2 * F), dtype, std=3.0)
    out = ops.opscale_swiglu(cuda(u))
    torch.cuda.synchronize()
    assert_close(f64(out.cpu()), oracle.swiglu(f64(u)), dtype, "swiglu")


@pytest.mark.parametrize("dtype,M,F", [("bf16", 256, 40), ("bf16", 257, 40), ("bf16", 257, 8184), ("bf16", 2, 8192),
                                       ("bf16", 2048, 8192), ("bf16", 2049, 8192), ("f32", 5, 8196)])
def test_swiglu_small_and_streaming(ops, dtype, M, F):
    """Both forms (cached, one vector a thread; nontemporal, two) at the line
    between them: 256 rows of narrow outputs, 2^24 outputs of wide ones."""
    import torch
    say(f"swiglu forms {dtype} M={M} F={F}")
    u = gen(37, "gate_up", (M, 2 * F), dtype, std=3.0)
    out = ops.opscale_swiglu(cuda(u))
    torch.cuda.synchronize()
    assert_close(f64(out.cpu()), oracle.swiglu(f64(u)), dtype, "swiglu")


# -------------------------------------------------------- prefill attention --
def _prefill_case(ops, dtype, lens, Hq, Hkv, D, causal, packed, seed=41):
    import torch
    lens = np.asarray(lens, np.int64)
    cu = wl.cu_seqlens(lens)
    T = int(cu[-1])
    if packed:  # views into one [T, (Hq + 2 Hkv) D] tensor, as after the QKV linear
        qkv = gen(seed, "q", (T, (Hq + 2 * Hkv) * D), dtype)
        qd = cuda(qkv)
        q = qd[:, : Hq * D].view(T, Hq, D)
        k = qd[:, Hq * D:(Hq + Hkv) * D].view(T, Hkv, D)
        v = qd[:, (Hq + Hkv) * D:].view(T, Hkv, D)
        qh = f64(qkv[:, : Hq * D]).reshape(T, Hq, D)
        kh = f64(qkv[:, Hq * D:(Hq + Hkv) * D]).reshape(T, Hkv, D)
        vh = f64(qkv[:, (Hq + Hkv) * D:]).reshape(T, Hkv, D)
    else:
        qc, kc, vc = (gen(seed, "q", (T, Hq, D), dtype), gen(seed, "k", (T, Hkv, D), dtype),
                      gen(seed, "v", (T, Hkv, D), dtype))
        q, k, v = cuda(qc), cuda(kc), cuda(vc)
        qh, kh, vh = f64(qc), f64(kc), f64(vc)
    scale = 1.0 / math.sqrt(D)
    out = ops.opscale_attn_prefill(q, k, v, cuda(torch.from_numpy(cu)), int(max(1, lens.max())), scale,
                                   causal)
    torch.cuda.synchronize()
    ref = oracle.attn_prefill(qh, kh, vh, cu, scale, causal)
    return f64(out.cpu()), ref


@pytest.mark.parametrize("dtype,lens,Hq,Hkv,D,causal,packed", [
    ("f32", [128], 4, 4, 64, True, False),
    ("f32", [5, 70, 0, 1], 4, 2, 128, True, True),
    ("f32", [33, 7], 2, 1, 64, False, False),
    ("bf16", [1, 17, 64, 65, 130, 0, 300], 8, 2, 128, True, False),
    ("bf16", [128, 40, 1], 4, 4, 64, True, False),
    ("bf16", [200, 31, 97], 16, 2, 128, True, True),
    ("bf16", [77, 3, 150], 6, 2, 128, True, False),
    ("bf16", [100, 1, 64], 8, 2, 128, False, False),
    ("bf16", [513], 2, 2, 64, True, True),
])
def test_attn_prefill(ops, dtype, lens, Hq, Hkv, D, causal, packed):
    say(f"attn_prefill {dtype} lens={lens} Hq={Hq} Hkv={Hkv} D={D} causal={causal} packed={packed}")
    got, ref = _prefill_case(ops, dtype, lens, Hq, Hkv, D, causal, packed)
    assert_close(got, ref, dtype, "attn_prefill")


@pytest.mark.parametrize("lens,Hq,Hkv,D,causal", [([31, 32, 33, 0, 129, 300, 1], 6, 2, 64, True),
                                                  ([31, 0, 32, 33, 160, 257], 3, 1, 128, True),
                                                  ([97, 65, 2], 4, 4, 128, False), ([300, 64], 2, 2, 64, False)])
def test_attn_prefill_f32_tiles(ops, lens, Hq, Hkv, D, causal):
    """The fp32 kernel's edges: prompts around one 32-query tile, fewer key
    tiles than waves and more, a last tile of one key, both head widths."""
    say(f"attn_prefill f32 tiles lens={lens} Hq={Hq} Hkv={Hkv} D={D} causal={causal}")
    got, ref = _prefill_case(ops, "f32", lens, Hq, Hkv, D, causal, True)
    assert_close(got, ref, "f32", "attn_prefill f32")


@pytest.mark.parametrize("lens,bound,Hq,Hkv,D,causal", [
    ([64], None, 4, 2, 64, True), ([40, 3, 64], None, 4, 4, 128, True),          # a wave per token: few tokens
    ([10] * 30 + [0, 1], None, 8, 2, 64, True), ([16] * 40, None, 6, 2, 128, False),  # ... or short prompts
    ([33] * 70, None, 2, 1, 64, True), ([70, 64, 65], None, 8, 8, 128, False),   # tiles, as many for every prompt
    ([40] * 3, 8192, 12, 4, 64, True), ([90] + [17] * 40, None, 4, 2, 128, False),   # a list of tiles
    ([20] * 63 + [0, 200, 0, 33] + [20] * 70 + [100], None, 4, 4, 64, True),     # ... over three blocks of prompts
    ([0] * 64 + [500], None, 3, 1, 128, True), ([100, 90, 130, 97], 40, 4, 2, 128, True),  # (a bound that is none)
    ([1] * 150 + [300, 33, 32, 31] + [2] * 60 + [34], None, 8, 2, 64, True),     # both: up to 32 tokens a wave each
    ([0, 32, 65] + [3] * 100, 4096, 4, 4, 128, True), ([5] * 300, 2048, 4, 2, 64, False),
])
def test_attn_prefill_f32_plans(ops, lens, bound, Hq, Hkv, D, causal):
    """The fp32 kernels and their work lists, each on batches that take it:
    tight and loose bounds, empty prompts, skewed lengths."""
    import torch
    say(f"attn_prefill f32 plans lens={lens[:4]}... B={len(lens)} bound={bound} Hq={Hq} Hkv={Hkv} D={D} causal={causal}")
    cu = wl.cu_seqlens(lens)
    T = int(cu[-1])
    q, k, v = gen(38, "q", (T, Hq, D), "f32"), gen(38, "k", (T, Hkv, D), "f32"), gen(38, "v", (T, Hkv, D), "f32")
    out = torch.full((T, Hq, D), float("nan"), device="cuda")
    ops.opscale_attn_prefill(cuda(q), cuda(k), cuda(v), cuda(torch.from_numpy(cu)), bound or max(lens), D ** -0.5, causal,
                             out=out)
    torch.cuda.synchronize()
    assert_close(f64(out.cpu()), oracle.attn_prefill(f64(q), f64(k), f64(v), cu, D ** -0.5, causal), "f32", "attn f32 plans")


def test_attn_prefill_f32_loose_bound_of_many_prompts(ops):
    """1024 prompts of 20 tokens, 32 heads, under a bound of 16384: as many tiles
    for every prompt as the bound allows are 2^24 workgroups, more than a grid."""
    import torch
    B, L, Hq, Hkv, D = 1024, 20, 32, 1, 64
    say("attn_prefill f32 loose bound")
    cu = wl.cu_seqlens([L] * B)
    g = torch.Generator(device="cuda").manual_seed(3)
    q, k, v = (torch.empty(B * L, h, D, device="cuda").normal_(generator=g) for h in (Hq, Hkv, Hkv))
    out = ops.opscale_attn_prefill(q, k, v, cuda(torch.from_numpy(cu)), 16384, D ** -0.5)
    torch.cuda.synchronize()
    heads = [0, 13, 31]
    ref = oracle.attn_prefill(f64(q[:, heads].cpu()), f64(k.cpu()), f64(v.cpu()), cu, D ** -0.5, True)
    assert_close(f64(out[:, heads].cpu()), ref, "f32", "attn f32 loose bound")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_attn_prefill_f32_future_is_not_read(ops, bad, D):
    """An infinity or NaN in the keys and values of later tokens of the prompt,
    or of the next prompt, leaves the queries before them unchanged (prompts long
    enough for the tiles)."""
    import torch
    say(f"attn_prefill f32 future {bad} D={D}")
    lens, H = [75, 40], 2
    T = sum(lens)
    q, k, v = (gen(33, t, (T, H, D), "f32") for t in ("q", "k", "v"))
    ref = oracle.attn_prefill(f64(q), f64(k), f64(v), wl.cu_seqlens(lens), D ** -0.5, True)
    k[70:75], v[70:75], k[80:], v[80:] = bad, bad, bad, bad
    out = ops.opscale_attn_prefill(cuda(q), cuda(k), cuda(v), cuda(torch.from_numpy(wl.cu_seqlens(lens))), max(lens),
                                   D ** -0.5)
    torch.cuda.synchronize()
    keep = np.r_[0:70, 75:80]
    assert_close(f64(out.cpu())[keep], ref[keep], "f32", "queries before the bad keys")
    assert not np.isfinite(f64(out.cpu())[np.r_[70:75, 80:T]]).any()


@pytest.mark.parametrize("lens,Hq,Hkv,D", [
    ([1, 17, 64, 65, 130, 0, 300, 33], 8, 2, 128),   # ragged, G = 4 (32-query tiles)
    ([96, 96, 96], 4, 2, 64),                        # uniform, G = 2 (64-query tiles)
    ([900, 5, 1, 260], 3, 3, 128),                   # G = 1 (128-query tiles)
    ([1, 2, 3, 17] * 20 + [700], 8, 1, 64),          # 81 prompts: more than one wave of 64
    # a long prompt before a short one, two equal prompts, one tile and a key:
    # the K/V loads in these tiles must land where their stage says (a missing
    # wait state before a load once wrote some of them to the previous load's
    # place, in the grid schedule only)
    ([300, 1], 4, 1, 128),
    ([130, 130], 4, 1, 128),
    ([65], 4, 1, 128),
])
def test_attn_prefill_schedules(ops, tune, lens, Hq, Hkv, D):
    """Both schedules (grid; level-major work list) against the oracle, and
    bitwise equal to each other (each tile is computed the same way)."""
    outs = {}
    for sched in ("grid", "list"):
        tune(prefill_schedule=SCHEDULES[sched])
        say(f"attn_prefill bf16 schedule={sched} lens={lens} Hq={Hq} Hkv={Hkv} D={D}")
        got, ref = _prefill_case(ops, "bf16", lens, Hq, Hkv, D, True, True)
        assert_close(got, ref, "bf16", f"attn_prefill ({sched})")
        outs[sched] = got
    assert np.array_equal(outs["grid"], outs["list"])


def test_attn_prefill_many_prompts(ops, tune):
    """More prompts than the work list holds in LDS: the launcher takes the grid
    even when the list is asked for."""
    tune(prefill_schedule=SCHEDULES["list"])
    say("attn_prefill bf16 1101 prompts")
    lens = ([1, 2, 3, 17] * 276)[:1101]
    got, ref = _prefill_case(ops, "bf16", lens, 8, 2, 128, True, True)
    assert_close(got, ref, "bf16", "attn_prefill 1101 prompts")


def test_attn_prefill_1024_prompts_list(ops, tune):
    """The largest batch the work list takes (1024 prompts, 16 waves of 64)."""
    tune(prefill_schedule=SCHEDULES["list"])
    say("attn_prefill bf16 1024 prompts (work list)")
    lens = ([1, 40, 3, 97, 0, 64] * 171)[:1024]
    got, ref = _prefill_case(ops, "bf16", lens, 8, 2, 64, True, True)
    assert_close(got, ref, "bf16", "attn_prefill 1024 prompts")


def test_attn_prefill_single_key_returns_v(ops):
    """Prompts of length 1: softmax over one key is exactly 1, output == v."""
    import torch
    lens = [1] * 9
    cu = wl.cu_seqlens(lens)
    q = gen(42, "q", (9, 8, 128), "bf16")
    k = gen(42, "k", (9, 2, 128), "bf16")
    v = gen(42, "v", (9, 2, 128), "bf16")
    out = ops.opscale_attn_prefill(cuda(q), cuda(k), cuda(v), cuda(torch.from_numpy(cu)), 1, 0.088)
    torch.cuda.synchronize()
    exp = v.repeat_interleave(4, dim=1)
    assert torch.equal(out.cpu(), exp)


# --------------------------------------------------------- decode attention --
def _decode_case(ops, dtype, ctx, Hq, Hkv, D, bs, seed=51, bad_block=False, max_context_len=None):
    import torch
    ctx = np.asarray(ctx, np.int64)
    rng = wl.rng_for(seed, "block_table")
    table, nb = wl.paged_cache_layout(ctx, bs, rng, extra_blocks=3)
    if bad_block:
        table = table.copy()
        table[0, 0] = nb + 5  # out of range: the keys of this page are skipped
    kc = gen(seed, "k_cache", (nb, bs, Hkv, D), dtype)
    vc = gen(seed, "v_cache", (nb, bs, Hkv, D), dtype)
    q = gen(seed, "q", (len(ctx), Hq, D), dtype)
    scale = 1.0 / math.sqrt(D)
    maxc = int(max(1, ctx.max())) if max_context_len is None else max_context_len
    out = ops.opscale_attn_decode(cuda(q), cuda(kc), cuda(vc), cuda(torch.from_numpy(table)),
                                  cuda(torch.from_numpy(ctx.astype(np.int32))), maxc, scale)
    torch.cuda.synchronize()
    kh, vh = f64(kc), f64(vc)
    if bad_block:
        # expected: the same sequence without the keys of its first page
        ref = oracle.attn_decode(f64(q), kh, vh, np.concatenate([table[:, 1:], table[:, :1]], 1),
                                 np.concatenate([[ctx[0] - bs], ctx[1:]]), scale)
        ref[1:] = oracle.attn_decode(f64(q)[1:], kh, vh, table[1:], ctx[1:], scale)
    else:
        ref = oracle.attn_decode(f64(q), kh, vh, table, ctx, scale)
    return f64(out.cpu()), ref


@pytest.mark.parametrize("dtype,ctx,Hq,Hkv,D,bs", [
    ("f32", [1, 16, 17, 600, 0], 8, 2, 128, 16),
    ("f32", [37, 5], 4, 4, 64, 8),
    ("bf16", [1, 16, 17, 600, 0], 8, 2, 128, 16),
    ("bf16", [1030, 2, 513, 9], 32, 8, 128, 16),
    ("bf16", [40, 300], 4, 4, 64, 16),
    ("bf16", [129, 2049, 31], 16, 2, 128, 32),
    ("bf16", [100, 7], 4, 2, 128, 1),
    ("bf16", [4000, 64], 16, 8, 64, 256),
])
def test_attn_decode(ops, dtype, ctx, Hq, Hkv, D, bs):
    say(f"attn_decode {dtype} ctx={ctx} Hq={Hq} Hkv={Hkv} D={D} bs={bs}")
    got, ref = _decode_case(ops, dtype, ctx, Hq, Hkv, D, bs)
    assert_close(got, ref, dtype, "attn_decode")


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("ctx", [[1], [33, 0], [512, 32 * 16 + 1], [32 * 63, 40], [32 * 65 + 5, 31, 1],
                                 [9000, 0, 70, 5, 17, 300, 64, 33]])
def test_attn_decode_many_segments(ops, ctx, D):
    """Few sequences over more than 16 workgroups each (launches for contexts of
    2048 and more): the merge by four waves of 16 segments, at one segment, one
    wave's 16 and one more, 63 to 66 (a second block of 64), and with most of a
    batch's segments in one sequence; and over the workgroups that the contexts
    themselves give, at most 16 a sequence (one wave) for the short ones."""
    say(f"attn_decode many segments ctx={ctx} D={D}")
    for maxc in (max(2048, max(ctx)), None):
        got, ref = _decode_case(ops, "bf16", ctx, 8, 2, D, 16, max_context_len=maxc)
        assert_close(got, ref, "bf16", f"attn_decode many segments, max_context_len={maxc}")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_attn_decode_invalid_block_is_skipped(ops, dtype):
    say(f"attn_decode invalid block id {dtype}")
    got, ref = _decode_case(ops, dtype, [40, 20], 8, 2, 128, 16, bad_block=True)
    assert_close(got, ref, dtype, "attn_decode bad block")


@pytest.mark.parametrize("name,ctx,maxc", [
    # far fewer 32-key tiles than workgroups: most workgroups have no keys
    ("sparse", [0, 5, 0, 33, 1, 0, 64, 2], 4096),
    ("one long, many short", [9000] + [3] * 39, None),
    # about 1.5 tiles a workgroup: ranges straddle sequence boundaries
    ("straddling", list(np.random.default_rng(8).integers(1, 2000, 100)), None),
    # one workgroup a sequence, each over several 512-key page windows
    ("few workgroups", [3000, 1, 1500, 0, 2047], 1),
    ("all empty", [0, 0, 0], 64),
    # above 512 sequences the plan comes from its own kernel
    ("large batch", list(np.random.default_rng(9).integers(0, 300, 700)), None),
    ("large batch, sparse", [0] * 600 + [40] + [0] * 100 + [1], 2048),
])
def test_attn_decode_balanced_ranges(ops, name, ctx, maxc):
    """Every workgroup takes an equal range of the batch's 32-key tiles; the
    ranges and the merge must cover each sequence's keys exactly once."""
    say(f"attn_decode balanced ranges: {name} (B={len(ctx)})")
    got, ref = _decode_case(ops, "bf16", ctx, 8, 2, 128, 16, seed=len(ctx), max_context_len=maxc)
    assert_close(got, ref, "bf16", f"attn_decode {name}")
    if max(ctx) == 0:
        assert np.all(got == 0)


@pytest.mark.parametrize("bs", [16, 1])
def test_attn_decode_context_beyond_launch_bound(ops, bs):
    """max_context_len only sizes the launch: a longer context is processed in
    several key windows by one split and the result is unchanged."""
    say(f"attn_decode context beyond max_context_len, bs={bs}")
    got, ref = _decode_case(ops, "bf16", [2000, 700, 3], 8, 2, 128, bs, max_context_len=100)
    assert_close(got, ref, "bf16", "attn_decode long context")


# ------------------------------------------------------- temporary workspaces --
@pytest.mark.parametrize("op", ["linear", "attn_decode", "fused_moe"])
def test_temporary_workspace_on_another_stream(ops, op):
    """A workspace that the binding allocates for a call on another stream is
    not handed on while that stream still has the call before it."""
    import torch
    bf = torch.bfloat16
    if op == "linear":
        x, W, y = torch.randn(16, 4096, device="cuda").to(bf), torch.randn(6144, 4096, device="cuda").to(bf), None
        y = torch.empty(16, 6144, device="cuda", dtype=bf)
        need = ops.opscale_linear_workspace_size(16, 6144, 4096)
        call = lambda s: ops.opscale_linear(x, W, y=y, stream=s)
    elif op == "attn_decode":
        q, out = torch.randn(2, 8, 64, device="cuda").to(bf), torch.empty(2, 8, 64, device="cuda", dtype=bf)
        kc = torch.randn(64, 16, 2, 64, device="cuda").to(bf)
        table = torch.arange(64, device="cuda", dtype=torch.int32).view(2, 32)
        ctx = torch.tensor([512, 500], device="cuda", dtype=torch.int32)
        need = ops.opscale_attn_decode_workspace_size(2, 8, 64, 512)
        call = lambda s: ops.opscale_attn_decode(q, kc, kc, table, ctx, 512, 0.125, out=out, stream=s)
    else:
        x, out = torch.randn(32, 64, device="cuda").to(bf), torch.empty(32, 64, device="cuda", dtype=bf)
        w1, w2 = torch.randn(4, 256, 64, device="cuda").to(bf), torch.randn(4, 64, 128, device="cuda").to(bf)
        ids = torch.zeros(32, 2, device="cuda", dtype=torch.int32)
        wts = torch.ones(32, 2, device="cuda")
        need = ops.opscale_fused_moe_workspace_size(32, 64, 128, 4, 2)
        call = lambda s: ops.opscale_fused_moe(x, w1, w2, ids, wts, out=out, stream=s)
    assert need > 0
    say(f"temporary workspace on another stream: {op}, {need} bytes")
    call(None)
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for stream in (side, side.cuda_stream):  # a torch stream, and its handle
        spot = torch.empty(need, dtype=torch.uint8, device="cuda")
        p = spot.data_ptr()
        del spot  # the block that the next allocation of this size gets
        with torch.cuda.stream(side):
            torch.cuda._sleep(20_000_000)  # (bounded: about 10 ms)
        call(stream)
        again = torch.empty(need, dtype=torch.uint8, device="cuda")
        assert not side.query(), "the other stream was done too early to tell"
        assert again.data_ptr() != p, "the workspace was handed on while in use"
        del again
        torch.cuda.synchronize()
    # on the current stream it may be: work there is in order
    spot = torch.empty(need, dtype=torch.uint8, device="cuda")
    p = spot.data_ptr()
    del spot
    call(torch.cuda.current_stream())
    assert torch.empty(need, dtype=torch.uint8, device="cuda").data_ptr() == p
    torch.cuda.synchronize()
