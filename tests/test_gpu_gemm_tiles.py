"""GPU parity of the read-ahead GEMM tiles at the sizes where they can go
wrong: token counts one past or one short of a tile, key ranges of few
64-deep k-tiles (fewer than or just past the ring), split ranges whose last
part is short, and the low-rank term read from the down-projection kernel's
partials.  The reference is the fp64 product of the same bf16 operands; the
bar is the one of a bf16-stored step (tests/_tol.py)."""

import math

import pytest
import torch

from tests._tol import assert_intermediate_close

pytestmark = pytest.mark.gpu

if torch.cuda.is_available():
    from paper_2609_36722_amd.api import Context, ModelCfg


def _normal(gen, *shape, std=1.0):
    return torch.randn(*shape, generator=gen, device="cuda").mul_(std).to(torch.bfloat16)


@pytest.mark.parametrize("T,K,N,res", [
    (2049, 1024, 4096, True),    # 256 x 256, one token past eight tiles
    (1000, 2048, 9216, False),   # 256 x 192, ragged last token tile
    (1025, 512, 4096, True),     # 128 x 256, eight k-tiles in a ring of three
    (769, 4096, 2560, True),     # 128 x 256 in 3 splits of 22, 22 and 20 k-tiles
    (257, 4096, 9216, False),    # 128 x 128, one token past two tiles
    (2049, 512, 512, True),      # 128 x 64, eight k-tiles in a ring of six
    (190, 2560, 2048, True),     # 128 x 64 in 4 splits of 10 k-tiles
    (1500, 2752, 256, True),     # 128 x 64 in 4 splits, the last one short (43 k-tiles)
    # 32-token tiles: the fewest tokens, 16, one past the GEMV's, a full tile
    (9, 2560, 8192, True), (16, 9728, 2560, True), (17, 4096, 4096, True), (32, 2560, 2560, False),
    (31, 1088, 640, True), (12, 512, 40960, False), (17, 64, 64, True),
])
def test_read_ahead_tiles(T, K, N, res):
    print(f"[case] linear T={T} K={K} N={N} residual={res}", flush=True)
    g = torch.Generator(device="cuda").manual_seed(T + K + N)
    x, w = _normal(g, T, K), _normal(g, N, K, std=1 / math.sqrt(K))
    r = _normal(g, T, N) if res else None
    out = torch.empty(T, N, dtype=torch.bfloat16, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=256), pool_pages=0) as ctx:
        ctx.linear(x, w, out, residual=r)
        torch.cuda.synchronize()
    ref = x.double() @ w.double().t() + (r.double() if res else 0)
    assert_intermediate_close(out.double().cpu().numpy(), ref.cpu().numpy(), "linear")


@pytest.mark.parametrize("T,H,rank", [(1100, 2560, 33), (2500, 4096, 0), (2500, 4096, 16), (300, 4096, 64), (257, 2560, 0)])
def test_read_ahead_projection(T, H, rank):
    # rank 0 and ranks above the fused limit take the read-ahead tiles; at
    # 2500 tokens the small ranks do too, with t from the separate kernel
    print(f"[case] qproj T={T} H={H} rank={rank}", flush=True)
    nq, n, scale = 4096, 6144, 0.5
    g = torch.Generator(device="cuda").manual_seed(T + H + rank)
    x, w = _normal(g, T, H), _normal(g, n, H, std=1 / math.sqrt(H))
    a = _normal(g, rank, H, std=1 / math.sqrt(H)) if rank else None
    b = _normal(g, nq, rank) if rank else None
    out = torch.empty(T, n, dtype=torch.bfloat16, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=H), pool_pages=0) as ctx:
        ctx.qproj_lora(x, w, a, b, rank, scale, nq, out)
        torch.cuda.synchronize()
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
    ("qproj", 1152, 2560, 6144, 16), ("qproj", 2500, 4096, 6144, 32),
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


@pytest.mark.parametrize("n,H,V", [
    (9, 2560, 9728), (16, 512, 47104), (12, 4096, 6144),     # past the GEMV: 24M weights and more
    (17, 512, 4096), (32, 2560, 16384), (24, 1088, 19200),   # in key splits; unsplit; k-tiles no multiple of eight
    (17, 64, 640), (20, 192, 1280),                          # one and three k-tiles
    (8, 2560, 4096), (33, 2560, 16384),                      # either side: the GEMV and the larger tiles
])
def test_lm_head_equal_rows_tie(n, H, V):
    # equal vocabulary rows give the same fp32 logit wherever they stand, so
    # the smaller index wins
    print(f"[case] lm_head tie n={n} H={H} V={V}", flush=True)
    x, w, at = _picked(n, H, V, n + H + V)
    ids = torch.empty(n, dtype=torch.int32, device="cuda")
    with Context(ModelCfg(n_layers=1, hidden=H), pool_pages=0) as ctx:
        ctx.lm_head_argmax(x, w, ids)
        torch.cuda.synchronize()
    assert ids.tolist() == at.min(0).values.tolist()


@pytest.mark.parametrize("n,H,V", [(9, 4096, 6144), (16, 4096, 6144), (32, 4096, 6144), (16, 2560, 9728)])
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
