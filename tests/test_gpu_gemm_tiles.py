"""GPU parity of the GEMM tiles at the sizes where they can go wrong: token
counts one past or one short of a tile, key ranges of few 64-deep k-tiles (fewer
than or just past the ring), split ranges whose last part is short, and the
low-rank term read from the down-projection kernel's partials.  Each case names
the plan it is for, and the plan and the kernel that ran are checked.  The
reference is the fp64 product of the same bf16 operands; the bar is the one of a
bf16-stored step (tests/_tol.py)."""

import math

import pytest
import torch

from tests._plan import F32, kernel_of, plain_plan, qproj_plan
from tests._tol import assert_intermediate_close

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2609_36722_amd.api import Context, ModelCfg


def _normal(gen, *shape, std=1.0):
    return torch.randn(*shape, generator=gen, device="cuda").mul_(std).to(torch.bfloat16)


def _assert_ran(times, plan, down=False):
    """The launches of one product: its plan's kernel, the split's reduction and
    the down-projection where there are any, and no other GEMM kernel."""
    want = {"gemv_mfma_kernel"} if plan == "gemv" else {kernel_of(plan)}
    if plan != "gemv" and not plan.endswith("/1") and "/" in plan:
        want.add("splitk_reduce_kernel")
    if down:
        want.add("lora_down_kernel")
    assert set(times) == want, (plan, sorted(times))


@pytest.mark.parametrize("T,K,N,res,plan", [
    (2049, 1024, 4096, True, "256x256a/1"),    # one token past eight tiles
    (2500, 192, 5120, False, "256x256a/1"),    # three k-tiles in a ring of two
    (2049, 4864, 2048, True, "256x256a/3"),    # 26, 26 and 24 k-tiles
    (1000, 2048, 9216, False, "256x192a/1"),   # ragged last token tile
    (769, 64, 7104, True, "256x192a/1"),       # one k-tile, fewer than the ring
    (1025, 5120, 2880, False, "256x192a/3"),   # 27, 27 and 26 k-tiles
    (1025, 512, 4096, True, "128x256a/1"),     # eight k-tiles in a ring of three
    (385, 64, 8448, False, "128x256a/1"),      # one k-tile
    (769, 4096, 2560, True, "128x256a/3"),     # 22, 22 and 20 k-tiles
    (257, 4096, 9216, False, "128x128a/1"),    # one token past two tiles
    (65, 64, 8320, True, "128x128a/1"),        # one k-tile
    (769, 2048, 1280, True, "128x128a/3"),     # 11, 11 and 10 k-tiles
    (2049, 512, 512, True, "128x64a/1"),       # eight k-tiles in a ring of six
    (385, 64, 2368, False, "128x64a/1"),       # one k-tile
    (769, 2816, 640, True, "128x64a/3"),       # 15, 15 and 14 k-tiles
    (257, 64, 8256, True, "128x192k/1"), (1025, 7104, 960, True, "128x192k/4"),
    (129, 320, 8640, True, "128x96k/1"), (256, 4096, 6144, False, "128x96k/2"), (769, 4160, 960, True, "128x96k/3"),
    (769, 320, 1344, True, "64x96/1"), (33, 2240, 8256, True, "64x96/2"), (257, 2752, 1152, False, "64x96/4"), (65, 64, 8448, False, "64x96/1"),
    (190, 2560, 2048, True, "64x64/2"), (1500, 2752, 256, True, "64x64/2"), (33, 832, 64, True, "64x64/3"),
    # few tokens: the GEMV, the 64-token tiles, and the 32-token ones (fewest
    # tokens, 16, one past the GEMV's, one short of a tile, a full one)
    (9, 2560, 8192, True, "gemv"), (12, 512, 40960, False, "gemv"),
    (16, 9728, 2560, True, "64x64/6"), (17, 4096, 4096, True, "64x64/4"), (32, 2560, 2560, False, "32x64a/4"),
    (31, 1088, 640, True, "32x64a/3"), (17, 64, 64, True, "32x64a/1"), (17, 2240, 5760, False, "64x96/4"),
    (9, 12288, 4096, True, "32x128a/8"), (32, 12288, 4096, False, "64x64/4"), (31, 6720, 2752, True, "32x64a/4"),
    (24, 1792, 8384, True, "32x64a/1"), (16, 3584, 12672, False, "32x128a/2"),
    (17, 1600, 8320, True, "32x64a/1"), (15, 3968, 8576, False, "32x128a/3"),
])
def test_read_ahead_tiles(T, K, N, res, plan):
    print(f"[case] linear T={T} K={K} N={N} residual={res} plan={plan}", flush=True)
    assert plain_plan(T, N, K) == plan
    g = torch.Generator(device="cuda").manual_seed(T + K + N)
    x, w = _normal(g, T, K), _normal(g, N, K, std=1 / math.sqrt(K))
    r = _normal(g, T, N) if res else None
    out = torch.empty(T, N, dtype=torch.bfloat16, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=256), pool_pages=0) as ctx:
        ctx.trace_begin()
        ctx.linear(x, w, out, residual=r)
        _assert_ran(ctx.trace_end(), plan)
    ref = x.double() @ w.double().t() + (r.double() if res else 0)
    assert_intermediate_close(out.double().cpu().numpy(), ref.cpu().numpy(), "linear")


@pytest.mark.parametrize("T,K,inter,plan", [
    (16, 4096, 12288, "32x128a/1"), (9, 2560, 9728, "32x128a/1"), (32, 2560, 9728, "32x128a/1"),  # stored by the tile
    (17, 1600, 4160, "32x64a/1"), (31, 8192, 4352, "32x128a/3"), (31, 6720, 1376, "32x64a/4"),   # the last two through the reduction
    (1000, 4096, 12288, "256x192a/1"), (192, 4096, 12288, "128x192k/1"), (17, 512, 1024, "32x64a/1"), (33, 512, 1024, "64x64/1"),
])
def test_swiglu_tiles(T, K, inter, plan):
    print(f"[case] gate_up_swiglu T={T} K={K} inter={inter} plan={plan}", flush=True)
    assert plain_plan(T, 2 * inter, K) == plan
    g = torch.Generator(device="cuda").manual_seed(T + K + inter)
    x, w = _normal(g, T, K), _normal(g, 2 * inter, K, std=1 / math.sqrt(K))
    out = torch.empty(T, inter, dtype=torch.bfloat16, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=256), pool_pages=0) as ctx:
        ctx.trace_begin()
        ctx.gate_up_swiglu(x, w, out)
        _assert_ran(ctx.trace_end(), plan)
    ref = x.double() @ w.double().t()
    ref = torch.nn.functional.silu(ref[:, 0::2]) * ref[:, 1::2]
    assert_intermediate_close(out.double().cpu().numpy(), ref.cpu().numpy(), "swiglu")


@pytest.mark.parametrize("n,H,V,plan", [
    (12, 2560, 151936, "32x128a/1"), (32, 2560, 151936, "32x128a/1"), (16, 8192, 8192, "32x128a/4"), (16, 4096, 6144, "32x128a/4"),
    (9, 8192, 6144, "32x128a/4"), (31, 2240, 5504, "32x64a/2"), (32, 512, 4096, "32x64a/1"), (128, 4096, 4096, "64x64/2"),
])
def test_lm_head_tiles(n, H, V, plan):
    # fp32 stores of the tile and of the split's reduction.  An fp32 sum of H
    # products is off by at most H roundings of 2^-24 of the sum of their
    # absolute values.
    print(f"[case] lm_head n={n} H={H} V={V} plan={plan}", flush=True)
    assert plain_plan(n, V, H, mode=F32) == plan
    g = torch.Generator(device="cuda").manual_seed(n + H + V)
    x, w = _normal(g, n, H), _normal(g, V, H, std=1 / math.sqrt(H))
    ids = torch.empty(n, dtype=torch.int32, device="cuda")
    top = torch.empty(n, dtype=torch.float32, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=H), pool_pages=0) as ctx:
        ctx.trace_begin()
        ctx.lm_head_argmax(x, w, ids, top)
        times = ctx.trace_end()
    assert kernel_of(plan) in times and ("splitk_reduce_kernel" in times) == (not plan.endswith("/1")), sorted(times)
    best = torch.full((n,), -math.inf, dtype=torch.float64, device="cuda")
    for v in range(0, V, 32768):
        best = torch.maximum(best, (x.double() @ w[v:v + 32768].double().t()).max(-1).values)
    picked = (x.double() * w[ids.long()].double())
    bound = H * 2.0 ** -24 * picked.abs().sum(-1)
    assert bool(((top.double() - picked.sum(-1)).abs() <= bound).all())
    assert bool((picked.sum(-1) >= best - 2 * bound).all())


@pytest.mark.parametrize("T,H,rank,tile,down", [
    (1100, 2560, 33, "128x256a", True), (2500, 4096, 0, "256x256a", False), (2500, 4096, 16, "256x256a", True),
    (1500, 4096, 64, "256x192a", True),    # its 96-wide waves straddle the last adapted column
    (1152, 2560, 16, "128x256", False), (1025, 2560, 32, "128x256", False), (1152, 4096, 16, "128x256a", True), (3500, 2560, 32, "256x192a", True),
    (300, 4096, 64, "128x96k", True), (257, 2560, 0, "128x96k", False), (600, 2560, 16, "128x128", False),
    (900, 2560, 32, "128x192k", False), (150, 2560, 8, "64x96", False), (40, 4096, 64, "64x64", True),
])
def test_projection_tiles(T, H, rank, tile, down):
    # down: t from the separate kernel (ranks above the fused limit, and tiles
    # that do not compute it).  B ~ N(0, 1): the low-rank term is no rounding error
    print(f"[case] qproj T={T} H={H} rank={rank} tile={tile}", flush=True)
    nq, n, scale = 4096, 6144, 0.5
    assert qproj_plan(T, n, H, rank) == tile
    g = torch.Generator(device="cuda").manual_seed(T + H + rank)
    x, w = _normal(g, T, H), _normal(g, n, H, std=1 / math.sqrt(H))
    a = _normal(g, rank, H, std=1 / math.sqrt(H)) if rank else None
    b = _normal(g, nq, rank) if rank else None
    out = torch.empty(T, n, dtype=torch.bfloat16, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=H), pool_pages=0) as ctx:
        ctx.trace_begin()
        ctx.qproj_lora(x, w, a, b, rank, scale, nq, out)
        _assert_ran(ctx.trace_end(), tile, down)
    ref = x.double() @ w.double().t()
    if rank:
        ref[:, :nq] += scale * (x.double() @ a.double().t()) @ b.double().t()
    assert_intermediate_close(out.double().cpu().numpy(), ref.cpu().numpy(), "qkv")


def test_few_tokens_capture_without_a_workspace():
    # 16 tokens x 9728 -> 2560 runs as key splits; on a captured stream whose
    # context has no split workspace it runs unsplit, and replays
    print("[case] linear captured, 16 tokens, nothing reserved", flush=True)
    T, K, N = 16, 9728, 2560
    g = torch.Generator(device="cuda").manual_seed(5)
    w = _normal(g, N, K, std=1 / math.sqrt(K))
    x, out = torch.zeros(T, K, dtype=torch.bfloat16, device="cuda"), torch.empty(T, N, dtype=torch.bfloat16, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=256), pool_pages=0) as ctx:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            ctx.linear(x, w, out)
        for _ in range(3):
            x.copy_(_normal(g, T, K))
            graph.replay()
            torch.cuda.synchronize()
            ref = x.double() @ w.double().t()
            assert_intermediate_close(out.double().cpu().numpy(), ref.cpu().numpy(), "linear")


@pytest.mark.parametrize("call,T,K,N,rank", [
    # key splits when eager; captured with nothing reserved they run unsplit
    ("linear", 24, 12288, 4096, 0), ("linear", 65, 2560, 2560, 0), ("linear", 256, 4096, 4096, 0),
    ("linear", 1100, 9728, 2560, 0), ("gate_up", 60, 2560, 19456, 0),
    # t from the separate kernel when eager; captured, a tile that computes t
    ("qproj", 1152, 4096, 6144, 16), ("qproj", 2500, 4096, 6144, 32),
])
def test_capture_with_nothing_reserved(call, T, K, N, rank):
    print(f"[case] {call} captured, nothing reserved: T={T} K={K} N={N} rank={rank}", flush=True)
    nq = 4096
    g = torch.Generator(device="cuda").manual_seed(T + K + N)
    w = _normal(g, N, K, std=1 / math.sqrt(K))
    a = _normal(g, rank, K, std=1 / math.sqrt(K)) if rank else None
    b = _normal(g, nq, rank) if rank else None
    x = torch.zeros(T, K, dtype=torch.bfloat16, device="cuda")
    out = torch.empty(T, N // 2 if call == "gate_up" else N, dtype=torch.bfloat16, device="cuda")

    def run(ctx, o):
        if call == "linear":
            ctx.linear(x, w, o)
        elif call == "gate_up":
            ctx.gate_up_swiglu(x, w, o)
        else:
            ctx.qproj_lora(x, w, a, b, rank, 0.5, nq, o)

    cfg = ModelCfg(n_layers=1, hidden=K if call == "qproj" else 256)
    with Context(cfg, pool_pages=0) as ctx, Context(cfg, pool_pages=0) as eager:
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            run(ctx, out)
        for _ in range(3):
            x.copy_(_normal(g, T, K))
            graph.replay()
            plain = torch.empty_like(out)
            run(eager, plain)
            torch.cuda.synchronize()
            ref = x.double() @ w.double().t()
            if rank:
                ref[:, :nq] += 0.5 * (x.double() @ a.double().t()) @ b.double().t()
            if call == "gate_up":
                ref = torch.nn.functional.silu(ref[:, 0::2]) * ref[:, 1::2]
            for got, what in ((out, "captured"), (plain, "eager")):
                assert_intermediate_close(got.double().cpu().numpy(), ref.cpu().numpy(), what)


@pytest.mark.parametrize("n,H,V", [(16, 8192, 8192), (128, 4096, 4096)])
def test_reserved_lm_head_allocates_nothing(n, H, V):
    # limits that name the LM head alone cover its key-split partials too (1 and
    # 4 MiB here): the first call takes no device memory
    print(f"[case] lm_head reserved by its own limits, n={n} H={H} V={V}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(n + H + V)
    x, w = _normal(g, n, H), _normal(g, V, H, std=1 / math.sqrt(H))
    ids = torch.empty(n, dtype=torch.int32, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=H), pool_pages=0) as ctx, \
            Context(ModelCfg(n_layers=1, hidden=H), pool_pages=0) as other:
        other.lm_head_argmax(x, w, ids)  # kernels loaded, another context's workspaces grown
        ctx.reserve(max_lm_rows=n, max_vocab=V)
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        ctx.lm_head_argmax(x, w, ids)
        torch.cuda.synchronize()
        assert torch.cuda.mem_get_info()[0] == before


def _picked(n, H, V, seed):
    """Rows x and a vocabulary whose rows i and j are both the copy of x[r] that
    wins row r (logit sqrt(H) = 22 or more against unit normals)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    x, w = _normal(g, n, H), _normal(g, V, H, std=1 / math.sqrt(H))
    at = torch.randperm(V, generator=g, device="cuda")[:2 * n].view(2, n)
    w[at] = (x.float() / math.sqrt(H)).to(torch.bfloat16)
    return x, w, at


@pytest.mark.parametrize("n,H,V,plan", [
    (9, 2560, 9728, "32x128a/3"), (16, 512, 47104, "32x128a/1"), (12, 4096, 6144, "32x128a/4"),  # past the GEMV
    (31, 8192, 1536, "32x64a/8"), (32, 8192, 5632, "32x128a/4"), (32, 2560, 10240, "32x64a/1"),
    (17, 512, 4096, "32x64a/1"), (17, 64, 640, "32x64a/1"), (20, 192, 1280, "32x64a/1"),        # eight, one and three k-tiles
    (8, 2560, 4096, "gemv"), (32, 2560, 16384, "64x64/1"), (24, 1088, 19200, "64x96/1"), (33, 2560, 16384, "64x64/1"),
])
def test_lm_head_equal_rows_tie(n, H, V, plan):
    # equal vocabulary rows give the same fp32 logit wherever they stand, so
    # the smaller index wins
    print(f"[case] lm_head tie n={n} H={H} V={V} plan={plan}", flush=True)
    assert plain_plan(n, V, H, mode=F32) == plan
    x, w, at = _picked(n, H, V, n + H + V)
    ids = torch.empty(n, dtype=torch.int32, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=H), pool_pages=0) as ctx:
        ctx.lm_head_argmax(x, w, ids)
        torch.cuda.synchronize()
    assert ids.tolist() == at.min(0).values.tolist()


@pytest.mark.parametrize("n,H,V", [(9, 4096, 6144), (16, 4096, 6144), (32, 4096, 6144), (32, 8192, 5632), (16, 2560, 9728)])
def test_lm_head_logit_precision(n, H, V):
    # The winning logit's products have one sign, so a partial sum of j of m
    # terms is j / m of it and each fp32 addition of the sum adds a rounding of
    # 2^-24 / sqrt(3) of the partial sum (rms).  Eight parts of H / 128 matrix
    # steps, summed pairwise: sqrt(1 + 2/4 + 4/16 + (H / 128) / 24) roundings,
    # 1.75 at 4096; the bar is twice that.  One chain of H / 16 steps:
    # sqrt(H / 48), 9.2 at 4096.
    print(f"[case] lm_head precision n={n} H={H} V={V}", flush=True)
    err = []
    with Context(ModelCfg(n_layers=1, hidden=H), pool_pages=0) as ctx:
        for seed in range(4):
            x, w, at = _picked(n, H, V, 1000 * seed + n + H)
            ids = torch.empty(n, dtype=torch.int32, device="cuda")
            top = torch.empty(n, dtype=torch.float32, device="cuda")
            ctx.lm_head_argmax(x, w, ids, top)
            torch.cuda.synchronize()
            ref = (x.double() * w[at[0]].double()).sum(-1)
            err.append((top.double() / ref - 1).cpu())
    rms = torch.cat(err).square().mean().sqrt().item()
    bar = 2 * math.sqrt(1.75 + H / 128 / 24) * 2.0 ** -24 / math.sqrt(3)
    assert rms <= bar, f"rms relative error {rms:.2e} > {bar:.2e}"
