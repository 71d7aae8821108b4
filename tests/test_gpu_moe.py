"""The mixture-of-experts path on the GPU against the oracle: top-k routing
(ids exact, the decision taken on the same fp32 logits; weights to fp32
rounding) and the fused expert MLPs (bf16 tolerance), on ragged problems
(experts without tokens, one expert with every token, invalid ids, duplicate
routes, one token), at Mixtral-8x7B widths on sampled tokens, and bitwise
repeatability."""
import numpy as np
import pytest

from oracle import moe as om
from parity_util import assert_close, say

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ops():
    import torch
    assert torch.cuda.is_available()
    import paper_2608_13499_amd as P
    P.load()
    return P


def _t(a, dtype):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to(dtype).cuda()


@pytest.mark.parametrize("T,E,k,ren,ties", [(300, 64, 8, True, False), (300, 64, 8, False, True),
                                             (129, 8, 2, True, True), (5, 3, 1, False, False),
                                             (70, 1000, 16, True, False)])
def test_topk_routing(ops, T, E, k, ren, ties):
    import torch
    say(f"moe_topk T={T} E={E} k={k} renormalize={ren} ties={ties}")
    rng = np.random.default_rng(T + E + k)
    lg = rng.normal(size=(T, E)).astype(np.float32)
    if ties:
        lg = np.round(lg * 2) / 2  # many equal logits
    ids, w = ops.opscale_moe_topk(_t(lg, torch.float32), k, ren)
    torch.cuda.synchronize()
    rid, rw = om.topk_route(lg, k, ren)
    assert np.array_equal(ids.cpu().numpy(), rid)
    assert np.allclose(w.cpu().numpy(), rw, rtol=2e-6, atol=1e-7)


def _moe_case(ops, T, H, F, E, k, seed, ids=None, wts=None):
    import torch
    rng = np.random.default_rng(seed)
    x = rng.normal(size=(T, H)).astype(np.float32)
    w1 = (rng.normal(size=(E, 2 * F, H)) / np.sqrt(H)).astype(np.float32)
    w2 = (rng.normal(size=(E, H, F)) / np.sqrt(F)).astype(np.float32)
    if ids is None:
        ids = np.stack([rng.permutation(E)[:k] for _ in range(T)]) if k <= E else rng.integers(0, E, (T, k))
    if wts is None:
        wts = rng.uniform(0.1, 1.0, size=(T, k)).astype(np.float32)
    xb, w1b, w2b = (_t(a, torch.bfloat16) for a in (x, w1, w2))
    out = ops.opscale_fused_moe(xb, w1b, w2b, _t(np.asarray(ids, np.int32), torch.int32),
                                _t(np.asarray(wts, np.float32), torch.float32))
    out2 = ops.opscale_fused_moe(xb, w1b, w2b, _t(np.asarray(ids, np.int32), torch.int32),
                                 _t(np.asarray(wts, np.float32), torch.float32))
    torch.cuda.synchronize()
    assert torch.equal(out, out2)  # ordered sort and sums: bitwise repeatable
    f64 = lambda t_: t_.float().cpu().numpy().astype(np.float64)
    ref = om.fused_moe(f64(xb), f64(w1b), f64(w2b), ids, np.asarray(wts, np.float32))
    return f64(out), ref


@pytest.mark.parametrize("fuse", [-1, 0])
@pytest.mark.parametrize("T,H,F,E,k", [(37, 64, 96, 8, 2), (300, 128, 256, 64, 8), (1, 64, 64, 4, 1),
                                        (600, 256, 512, 3, 2), (257, 96, 40, 16, 4)])
def test_fused_moe(ops, tune, fuse, T, H, F, E, k):
    """Both paths: the SwiGLU fused into the gate-up GEMM's epilogue (gate
    and up rows interleaved), and the separate gate-up output plus SwiGLU."""
    tune(moe_fuse=fuse)  # -1: automatic (fused at these sizes); 0: unfused
    say(f"fused_moe T={T} H={H} F={F} E={E} topk={k} fuse={fuse}")
    got, ref = _moe_case(ops, T, H, F, E, k, seed=T * 7 + E)
    assert_close(got, ref, "bf16", "fused_moe")


@pytest.mark.parametrize("T,E,k", [(512, 8, 2), (513, 256, 2), (31, 1, 1), (90, 257, 4), (4096, 5, 2), (4097, 5, 2)])
def test_fused_moe_sort_sizes(ops, T, E, k):
    """The sort at its edges: lists of exactly and just past a whole wave of
    entries for each of its 16 waves, the most experts and entries of the
    one-workgroup form (256; 8192) and one more of each (three kernels), one
    expert; invalid ids among them."""
    say(f"fused_moe sort T={T} E={E} topk={k}")
    rng = np.random.default_rng(T + E)
    ids = rng.integers(0, E, size=(T, k))
    ids[::97, 0] = -1
    ids[5::131, k - 1] = E
    got, ref = _moe_case(ops, T, 32, 16, E, k, seed=T + E, ids=ids)
    assert_close(got, ref, "bf16", "fused_moe sort sizes")


@pytest.mark.parametrize("fuse", [-1, 0])
@pytest.mark.parametrize("T,H,F,E,k", [(1500, 264, 4096, 4, 2), (700, 192, 8200, 2, 2), (1200, 136, 1032, 9, 1)])
def test_fused_moe_chained_tiles(ops, tune, fuse, T, H, F, E, k):
    """Batches of more than 64 rows an expert run on the four-wave kernel: a
    partial last K slice on either side, K of three slices, K past 8192 (x in the
    lead), rows of no expert, ragged tile-rows.  (Fewer tiles than it chains: the
    test after this one.)"""
    tune(moe_fuse=fuse)
    say(f"fused_moe four-wave tiles T={T} H={H} F={F} E={E} topk={k} fuse={fuse}")
    ids = np.random.default_rng(T).integers(0, E, size=(T, k))
    ids[::53, 0] = -1
    got, ref = _moe_case(ops, T, H, F, E, k, seed=T + F, ids=ids)
    assert_close(got, ref, "bf16", "fused_moe four-wave tiles")


@pytest.mark.parametrize("fuse", [-1, 0])
@pytest.mark.parametrize("T,H,F,E,k,chained", [
    (2500, 136, 12808, 9, 1, "gate_up"),   # ragged K of two slices and a part, in chains
    (2500, 192, 12808, 9, 1, "gate_up"),   # K of three slices
    (11000, 4096, 8200, 6, 2, "both"),     # gate-up in 22 rounds; down with x in the lead, ragged
    (11000, 4096, 8192, 6, 2, "both"),
])
def test_fused_moe_chains_over_experts(ops, tune, fuse, T, H, F, E, k, chained):
    """Six rounds of the CUs' 256x256 tiles and more: the four-wave kernel's
    workgroups run chains of tiles, which cross from an expert's rows and weights
    to another's; experts of uneven and of no rows, entries of no expert."""
    import torch
    tune(moe_fuse=fuse)
    say(f"fused_moe chains T={T} H={H} F={F} E={E} topk={k} fuse={fuse}")
    rng = np.random.default_rng(T + F)
    p = np.arange(1.0, E + 1)
    p[E // 2] = 0  # an expert without rows
    ids = rng.choice(E, size=(T, k), p=p / p.sum())
    ids[::53, 0] = -1
    tile_rows = int((-(-np.bincount(ids[ids >= 0], minlength=E) // 256)).sum())
    assert T * k > 64 * E and tile_rows * -(-2 * F // 256) > 5 * 256
    assert chained == "gate_up" or tile_rows * -(-H // 256) > 5 * 256
    g = torch.Generator(device="cuda").manual_seed(T)
    normal = lambda *s, std=1.0: torch.empty(s, dtype=torch.bfloat16, device="cuda").normal_(0, std, generator=g)
    x, w1, w2 = normal(T, H), normal(E, 2 * F, H, std=H ** -0.5), normal(E, H, F, std=F ** -0.5)
    idd = torch.from_numpy(ids.astype(np.int32)).cuda()
    wts = torch.empty(T, k, device="cuda").uniform_(0.1, 1.0, generator=g)
    out = ops.opscale_fused_moe(x, w1, w2, idd, wts)
    assert torch.equal(out, ops.opscale_fused_moe(x, w1, w2, idd, wts))
    ref = torch.zeros(T, H, device="cuda")
    for e in range(E):
        rows, slot = torch.nonzero(idd == e, as_tuple=True)
        if len(rows):
            gu = x[rows].float() @ w1[e].float().t()
            act = torch.nn.functional.silu(gu[:, :F]) * gu[:, F:]
            ref.index_put_((rows,), wts[rows, slot][:, None] * (act @ w2[e].float().t()), accumulate=True)
    torch.cuda.synchronize()
    # (a token whose entries are all of no expert is zero on both sides)
    live = (idd >= 0).any(1).cpu().numpy()
    got, ref = out.float().cpu().numpy(), ref.cpu().numpy()
    assert not got[~live].any()
    assert_close(got[live], ref[live], "bf16", "fused_moe chains")


def test_fused_moe_one_hot_expert(ops):
    """Every token to expert 2 (600 rows: three 256-row tiles), the others empty."""
    say("fused_moe all tokens to one expert")
    T = 600
    got, ref = _moe_case(ops, T, 128, 128, 6, 1, seed=5, ids=np.full((T, 1), 2))
    assert_close(got, ref, "bf16", "fused_moe one expert")


def test_fused_moe_invalid_and_duplicate_routes(ops):
    """Ids outside [0, E) contribute nothing; two slots may name one expert."""
    say("fused_moe invalid and duplicate ids")
    T, E = 50, 5
    rng = np.random.default_rng(9)
    ids = rng.integers(0, E, size=(T, 3))
    ids[::7, 0] = -1
    ids[3::11, 2] = E + 3
    ids[::5, 1] = ids[::5, 0]
    got, ref = _moe_case(ops, T, 64, 64, E, 3, seed=9, ids=ids)
    assert_close(got, ref, "bf16", "fused_moe invalid ids")
    dead = np.all((ids < 0) | (ids >= E), axis=1)
    assert np.all(got[dead] == 0)


def test_fused_moe_mixtral_width_sampled(ops):
    """Mixtral-8x7B expert widths (H 4096, F 14336), two experts, top-2, 256
    tokens; the oracle on 6 sampled tokens (rows are independent)."""
    import torch
    say("fused_moe Mixtral widths, 256 tokens, sampled rows")
    T, H, F, E, k = 256, 4096, 14336, 2, 2
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn(T, H, device="cuda", generator=g).to(torch.bfloat16)
    w1 = (torch.randn(E, 2 * F, H, device="cuda", generator=g) / 64).to(torch.bfloat16)
    w2 = (torch.randn(E, H, F, device="cuda", generator=g) / 120).to(torch.bfloat16)
    rng = np.random.default_rng(3)
    ids = np.stack([rng.permutation(E) for _ in range(T)]).astype(np.int32)
    wts = rng.uniform(0.2, 1.0, (T, k)).astype(np.float32)
    out = ops.opscale_fused_moe(x, w1, w2, _t(ids, torch.int32), _t(wts, torch.float32))
    torch.cuda.synchronize()
    rows = [0, 1, 77, 128, 200, 255]
    f64 = lambda t_: t_.float().cpu().numpy().astype(np.float64)
    ref = om.fused_moe(f64(x[rows]), f64(w1), f64(w2), ids[rows], wts[rows])
    assert_close(f64(out[rows]), ref, "bf16", "fused_moe Mixtral rows")


def test_fused_moe_rejects(ops):
    import torch
    x = torch.zeros(4, 64, dtype=torch.float32, device="cuda")
    w1 = torch.zeros(2, 128, 64, dtype=torch.float32, device="cuda")
    w2 = torch.zeros(2, 64, 64, dtype=torch.float32, device="cuda")
    ids = torch.zeros(4, 1, dtype=torch.int32, device="cuda")
    wts = torch.ones(4, 1, dtype=torch.float32, device="cuda")
    with pytest.raises(ops.OpscaleError):
        ops.opscale_fused_moe(x, w1, w2, ids, wts)  # fp32: bf16 only
