"""GEMM kernels at the edges of their tiles: row counts around the rows per
block of the weight-streaming kernel, W on both sides of the size that
decides them, K ranges that end inside a stage (for 8-bit W inside a 16-code
chunk), and the tiles of the 256 x 256 kernel.

The bound per element: the result is one bf16 rounding (half an ulp, 2^-9
relative) of a sum whose fp32 additions each round by at most 2^-24 of the
partial sums, themselves at most S = |A| |W|^T; K additions in any order stay
within K 2^-24 S (taken twice, and the bf16 part twice)."""
import numpy as np
import pytest
import torch

from paper_2606_00516_amd import binding as B
from paper_2606_00516_amd import inputs as gen
from tests._cases import make_case
from tests._gpu import DevCase, maxrel, to_f32

pytestmark = pytest.mark.gpu


def _check(M, N, K, epi, w8, seed=0):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed + M + N + K)
    A = torch.randn(M, K, generator=g, device="cuda").to(torch.bfloat16)
    R = torch.randn(M, N, generator=g, device="cuda").to(torch.bfloat16)
    if w8:
        W, s = gen.make_fp8_matrix(N, K, seed + 1, device="cuda", proj_std=0.05)
        w64 = W.view(torch.float8_e4m3fn).float().double() * s.double()[:, None]
        got = B.eb_op_gemm_w8(A, W, s, epi, residual=R if epi == "residual" else None)
    else:
        W = (torch.randn(N, K, generator=g, device="cuda") * 0.05).to(torch.bfloat16)
        w64 = W.double()
        got = B.eb_op_gemm(A, W, epi, residual=R if epi == "residual" else None)
    p = A.double() @ w64.t()
    acc = 2 * K * 2.0 ** -24 * (A.double().abs() @ w64.abs().t())
    if epi == "silu_mul":
        F = N // 2
        gate, up = p[:, :F], p[:, F:]
        ref = gate * torch.sigmoid(gate) * up
        # |d silu / dx| <= 1.1; the exponential and reciprocal add a few ulps of fp32
        acc = 1.1 * acc[:, :F] * up.abs() + acc[:, F:] * gate.abs() + 2.0 ** -20 * ref.abs()
    else:
        ref = p + (R.double() if epi == "residual" else 0)
    err = (got.double() - ref).abs()
    worst = (err - (2.0 ** -8 * ref.abs() + acc + 1e-30)).max().item()
    assert worst <= 0, (worst, err.max().item())


# 4104 x 1032: W of 8.5 MB (rows per block follow the batch; K ends 8 values into a stage and, for codes, into a
# chunk); 264 x 520: W inside one L2 (blocks of 64 rows)
@pytest.mark.parametrize("w8", [False, True], ids=["bf16", "w8"])
@pytest.mark.parametrize("N,K", [(4104, 1032), (8208, 1048), (264, 520)])
@pytest.mark.parametrize("M", [1, 15, 64, 65, 128, 129, 192, 193, 255])
def test_stream_rows(M, N, K, w8):
    _check(M, N, K, "store" if M % 2 else "residual", w8)


@pytest.mark.parametrize("M,N,K", [(1, 4104, 1032), (64, 264, 520), (65, 4104, 1032), (128, 8208, 1048),
                                   (300, 1032, 2056), (37, 28688, 264)])
def test_nan_codes_stay_in_their_row(M, N, K):
    """NaN codes (0x7F, 0xFF) in the first 8 columns of some weight rows, with a K that ends 8 codes into a 16-code
    chunk, whose other half is the next row's start: exactly those rows' output columns are NaN, the others keep the
    bits of a matrix without them."""
    A = torch.randn(M, K, device="cuda").to(torch.bfloat16)
    W, s = gen.make_fp8_matrix(N, K, 3, device="cuda", proj_std=0.05)
    clean = B.eb_op_gemm_w8(A, W, s)
    rows = torch.tensor([1, 2, 17, 130, N - 1], device="cuda")
    W = W.clone()
    W[rows, torch.tensor([0, 7, 3, 5, 6], device="cuda")] = torch.tensor([0x7F, 0xFF, 0x7F, 0xFF, 0x7F],
                                                                         dtype=torch.uint8, device="cuda")
    got = B.eb_op_gemm_w8(A, W, s)
    bad = torch.zeros(N, dtype=torch.bool, device="cuda")
    bad[rows] = True
    assert torch.isnan(got[:, bad]).all()
    assert torch.equal(got[:, ~bad], clean[:, ~bad])


@pytest.mark.parametrize("M,N,K,w8", [(32, 4104, 1032, False), (33, 4104, 1032, False), (32, 8208, 1032, True),
                                      (64, 24584, 2056, False), (65, 24584, 2056, False), (130, 24584, 2056, False),
                                      (200, 24584, 2056, False), (64, 49160, 2056, True), (65, 49160, 2056, True)])
def test_stream_once(M, N, K, w8):
    """Both sides of the sizes from which W is loaded past the caches (4 MiB to 32 rows, 96 MiB above)."""
    _check(M, N, K, "residual", w8)


@pytest.mark.parametrize("w8", [False, True], ids=["bf16", "w8"])
@pytest.mark.parametrize("M,N,K", [(33, 28688, 512), (100, 28688, 512), (180, 28688, 264), (240, 28688, 1152),
                                   (64, 25600, 136), (130, 1376, 256)])
def test_stream_silu(M, N, K, w8):
    """Unsplit gate/up products (each column tile starts its K walk elsewhere)."""
    _check(M, N, K, "silu_mul", w8)


@pytest.mark.parametrize("w8", [False, True], ids=["bf16", "w8"])
@pytest.mark.parametrize("M,N,K,epi", [
    (255, 2056, 2048, "residual"), (130, 2056, 2048, "store"),   # four and three block rows of 64, split
    (96, 28672, 512, "silu_mul"), (160, 6144, 4096, "residual"), (135, 24584, 1024, "store"),     # 128, 192 rows
    (224, 28672, 1024, "silu_mul"), (250, 6144, 4096, "store"), (250, 12296, 4096, "residual"),   # 256 rows; 2 x 128
    (200, 57344, 512, "silu_mul"), (130, 8200, 8192, "residual"), (180, 8200, 16384, "store"),    # part of a 256 x 256
    (150, 4104, 16384, "residual"),                              # tile, unsplit and split
    (256, 264, 520, "store"), (700, 264, 520, "residual"), (3000, 264, 264, "silu_mul")])         # a W inside one L2
def test_plans_by_time(M, N, K, epi, w8):
    """One shape or more for each kernel and block size that the estimated times choose between."""
    _check(M, N, K, epi, w8)


@pytest.mark.parametrize("w8", [False, True], ids=["bf16", "w8"])
@pytest.mark.parametrize("M", [40, 100, 300])
def test_silu_at_the_end_of_its_range(M, w8):
    """Gates from -88.5 to -80 (silu down to 3e-37, a normal bf16) times 1: every M takes another kernel.  __expf of
    arguments to 88.5 is good to 2 ulps + 88.5 2^-23 relative from its scaled argument's rounding; with bf16's 2^-9 taken
    twice 2^-7 covers both."""
    N, K = 512, 128
    A = torch.zeros(M, K, device="cuda", dtype=torch.bfloat16)
    gate = -80 - torch.arange(M, device="cuda") % 18 * 0.5    # a bf16 each
    A[:, 0] = gate.to(torch.bfloat16)
    A[:, 1] = 1
    W = torch.zeros(N, K, device="cuda", dtype=torch.bfloat16)
    W[:N // 2, 0] = 1
    W[N // 2:, 1] = 1
    if w8:
        got = B.eb_op_gemm_w8(A, W.float().to(torch.float8_e4m3fn).view(torch.uint8), torch.ones(N, device="cuda"),
                              "silu_mul")
    else:
        got = B.eb_op_gemm(A, W, "silu_mul")
    g = A[:, :1].double()
    ref = (g * torch.sigmoid(g)).expand(M, N // 2)
    assert ((got.double() - ref).abs() <= 2.0 ** -7 * ref.abs()).all()


@pytest.mark.parametrize("w8", [False, True], ids=["bf16", "w8"])
@pytest.mark.parametrize("epi", ["store", "residual", "silu_mul"])
@pytest.mark.parametrize("M,N,K", [(256, 528, 64), (257, 4112, 128), (511, 264, 192), (700, 2064, 4160)])
def test_big_tiles(M, N, K, epi, w8):
    _check(M, N, K, epi, w8)


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "w8"])
@pytest.mark.parametrize("T", [64, 65, 130, 200])
def test_layer_rows(T, fp8):
    """Decode layers around 64 rows, to which the split QKV projection takes the first RMSNorm with it, and of more,
    where the norm is a launch of its own, against the oracle."""
    shape = gen.LayerShape("mid", 2048, 16, 4, 128, 2064, 1e4)
    rng = np.random.default_rng(T)
    case = make_case(shape, gen.batch_decode(T, 1, 40, rng),
                     weights=gen.make_weights_fp8(shape) if fp8 else None)
    if fp8:
        dense = {k: v for k, v in case.weights.items() if not k.startswith("s_")}
        for k in ("qkv", "o", "gate_up", "down"):
            w = case.weights["w_" + k].view(torch.float8_e4m3fn).float() * case.weights["s_" + k][:, None]
            dense["w_" + k] = w.to(torch.bfloat16)
    ref = make_case(shape, case.batch, weights=dense if fp8 else case.weights).run_oracle()[0]
    dc = DevCase(case)
    h = B.Handle(shape, T, T)
    y = B.eb_layer_step_decode(h, dc.w, dc.k, dc.v, dc.bt, case.batch.context_lens, case.batch.chunk_lens, dc.x)
    # 8-bit weights: the oracle's are rounded to bf16 once (2^-9 each), the kernel's codes and scales are not
    assert maxrel(to_f32(y), ref) < 2e-2


@pytest.mark.parametrize("T", [3, 70])
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "w8"])
def test_infinite_gain_stays_in_its_k_range(T, fp8):
    """An infinite first-norm gain at every multiple of 32, so at the first column of each K split too, where the split
    before may end inside a stage: the v rows are infinite (one infinite term each), never NaN."""
    shape = gen.LayerShape("wide-qkv", 2048, 64, 8, 128, 256, 1e4)
    batch = gen.batch_decode(T, 1, 40, np.random.default_rng(T))
    case = make_case(shape, batch, weights=gen.make_weights_fp8(shape) if fp8 else None)
    if not fp8:   # (a zero would make the term NaN by itself)
        case.weights["w_qkv"][case.weights["w_qkv"] == 0] = 2.0 ** -10
    case.x[case.x == 0] = 2.0 ** -10
    dc = DevCase(case)
    h = B.Handle(shape, T, T)
    pos = torch.as_tensor(batch.context_lens, device="cuda").long()
    page = dc.bt[torch.arange(T, device="cuda"), pos // 16].long()
    gain = dc.w["attn_norm"].clone()
    for k in range(0, shape.hidden, 32):
        dc.w["attn_norm"].copy_(gain)
        dc.w["attn_norm"][k] = float("inf")
        B.eb_layer_step_decode(h, dc.w, dc.k, dc.v, dc.bt, batch.context_lens, batch.chunk_lens, dc.x)
        new = dc.v[page, :, pos % 16].float()
        assert torch.isinf(new).all(), (k, torch.isnan(new).sum().item())


@pytest.mark.parametrize("shape,T,ctx", [(gen.L8B, 129, 500), (gen.L8B, 252, 100), (gen.L8B, 252, 500),
                                         (gen.L8B, 252, 900), (gen.L70B, 200, 200), (gen.L70B, 252, 600)],
                         ids=lambda v: getattr(v, "name", v))
def test_wide_decode_batch_fits_the_fixed_scratch(shape, T, ctx):
    """Batches of 129 to 255 rows split K further than their 64-row blocks would, but never out of the scratch of the
    entry point without a workspace (the 70B shape's are cut to it): what fits it without partials still does, with the
    bits of the regular step."""
    rng = np.random.default_rng(T + ctx)
    batch = gen.batch_decode(T, ctx - 50, ctx, rng)
    w = gen.make_weights(shape, device="cuda")
    pool = gen.make_kv_pool(shape, batch, device="cuda")
    x = gen.make_x(shape, T, device="cuda")
    h = B.Handle(shape, T, T)
    assert B.eb_workspace_bytes(h, batch.context_lens, batch.chunk_lens, "mixed") <= B.eb_noalloc_scratch_bytes()
    args = (h, w, pool.k_cache, pool.v_cache, pool.block_tables, batch.context_lens, batch.chunk_lens, x)
    y = B.eb_layer_step_mixed(*args).clone()
    assert torch.equal(y, B.eb_layer_step_mixed_noalloc(*args))
    # the narrower plan's rows against the batch cut to 64 (its own splits)
    n = 64
    y64 = B.eb_layer_step_mixed(h, w, pool.k_cache, pool.v_cache, pool.block_tables[:n].contiguous(),
                                batch.context_lens[:n], batch.chunk_lens[:n], x[:n].contiguous())
    assert maxrel(to_f32(y[:n]), to_f32(y64)) < 1e-2


@pytest.mark.parametrize("shape", [gen.L8B, gen.L70B, gen.Q30B], ids=lambda s: s.name)
@pytest.mark.parametrize("T", [1, 64, 65, 100, 128, 160, 192, 252, 256, 300])
def test_workspace_never_falls_with_contexts(shape, T):
    """A workspace sized for a batch's longest contexts serves every shorter one of as many rows (host planning alone).
    Among the contexts: those around 64 keys, from which on a request is split, and around whole 512-key splits."""
    h = B.Handle(shape, T, T)
    one = np.ones(T, np.int32)
    ctx = sorted({*range(0, 16400, 300), *(s - 1 + d for s in (64, *range(512, 16385, 512)) for d in (-1, 0, 1))})
    sizes = [B.eb_workspace_bytes(h, np.full(T, c, np.int32), one, "decode") for c in ctx]
    assert sizes == sorted(sizes), [(a, b) for a, b in zip(sizes, sizes[1:]) if b < a]


@pytest.mark.parametrize("T,lo,hi", [(160, 3500, 9800), (128, 200, 13000)])
def test_rows_do_not_depend_on_their_neighbours_contexts(T, lo, hi):
    """The first 8 requests of two batches of T rows, whose other requests have short and long contexts: the projections'
    K splits follow from the rows, so these requests' outputs are the same bits."""
    shape, n = gen.L8B, 8
    w = gen.make_weights(shape, device="cuda")
    x = gen.make_x(shape, T, device="cuda")
    h = B.Handle(shape, T, T)
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    first = torch.randn(2, n * 4, shape.n_kv_heads, 16, shape.head_dim, generator=g, device="cuda").to(torch.bfloat16)
    ys = []
    for ctx in (lo, hi):
        per = ctx // 16 + 1      # pages of each of the others, behind the first n requests' four each
        k = torch.zeros(n * 4 + (T - n) * per, shape.n_kv_heads, 16, shape.head_dim, dtype=torch.bfloat16, device="cuda")
        v = k.clone()
        k[:n * 4], v[:n * 4] = first
        bt = torch.arange(-n, T - n, device="cuda")[:, None] * per + torch.arange(per, device="cuda") + n * 4
        bt[:n, :4] = torch.arange(n * 4, device="cuda").view(n, 4)
        bt[:n, 4:] = -1
        lens = np.full(T, ctx, np.int32)
        lens[:n] = 50
        ys.append(B.eb_layer_step_decode(h, w, k, v, bt.int().contiguous(), lens, np.ones(T, np.int32), x)[:n])
    assert torch.equal(ys[0], ys[1])
