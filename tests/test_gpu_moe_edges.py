"""The mixture-of-experts block where its kernels change: the sorted order by
one block and by several (from 4096 assignments), logits by wavefronts and by
the weight-streaming GEMM (above 2^18 token-expert pairs), expert products in
64-row tiles and in 256-row ones, hidden sizes and widths that end inside a
stage.

Reference in float64 under the routing the block reports, which must be a
valid top k.  The bound per element: the result and each m are rounded to bf16
once (2^-9 relative, taken twice), m's error enters through |Wd|; fp32 sums of
n terms stay within n 2^-24 of their absolute terms."""
import pytest
import torch

from paper_2606_00516_amd import binding as B
from paper_2606_00516_amd import inputs as gen

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,E,k,F,T", [
    (256, 16, 4, 128, 1), (256, 16, 4, 128, 1023), (256, 16, 4, 128, 1024), (256, 16, 4, 128, 2049),
    (96, 256, 6, 40, 2100),      # two logits column tiles, K ends inside a stage, 64-row tiles
    (96, 256, 6, 40, 700),       # the plan on several blocks, few rows per expert
    (128, 32, 3, 64, 1500),      # many rows per expert, too little work for 256-row tiles
    (512, 16, 4, 576, 1000), (512, 16, 4, 512, 1023), (512, 16, 4, 512, 1024),   # 256-row tiles; both sides of 2^30
    (4096, 16, 8, 64, 520),      # 256-row tiles of a single K tile down
    (160, 256, 2, 24, 1024), (160, 256, 2, 24, 1025), (96, 16, 1, 8, 16384), (96, 16, 1, 8, 16385),   # logits, both sides
    (2080, 48, 5, 24, 70), (64, 16, 16, 8, 300)])
def test_moe_edges(d, E, k, F, T):
    shape = gen.MoeShape("edge", d, E, k, F)
    w = gen.make_moe_weights(shape, seed=d + T, device="cuda", proj_std=0.1)
    g = torch.Generator(device="cuda")
    g.manual_seed(T)
    b = torch.randn(T, d, generator=g, device="cuda").to(torch.bfloat16)
    res = torch.randn(T, d, generator=g, device="cuda").to(torch.bfloat16)
    out, ids, wts = B.eb_op_moe_ffn(b, w["w_router"], w["w_gate_up"], w["w_down"], k, residual=res,
                                    return_routing=True)
    x, ids = b.double(), ids.long()
    logits = x @ w["w_router"].double().t()
    slack = d * 2.0 ** -23 * (x.abs() @ w["w_router"].double().abs().t()).max()
    chosen = logits.gather(1, ids)
    assert (ids.sort(1).values.diff(dim=1) > 0).all() if k > 1 else True
    assert (chosen.min(1).values >= logits.topk(k, 1).values[:, -1] - slack).all()
    rw = torch.softmax(chosen, 1)
    assert (wts.double() - rw).abs().max() < 1e-5 + 4 * slack
    ref, bound = res.double(), torch.zeros(T, d, dtype=torch.float64, device="cuda")
    for e in range(E):
        t, j = (ids == e).nonzero(as_tuple=True)
        if not t.numel():
            continue
        gw, uw, dw = w["w_gate_up"][e, :F].double(), w["w_gate_up"][e, F:].double(), w["w_down"][e].double()
        gt, up = x[t] @ gw.t(), x[t] @ uw.t()
        m = gt * torch.sigmoid(gt) * up
        # m: its rounding, and the sums behind it (|d silu| <= 1.1)
        me = 2.0 ** -8 * m.abs() + d * 2.0 ** -23 * (1.1 * (x[t].abs() @ gw.abs().t()) * up.abs()
                                                     + (x[t].abs() @ uw.abs().t()) * gt.abs())
        wt = wts[t, j].double()[:, None]
        ref.index_add_(0, t, wt * (m @ dw.t()))
        bound.index_add_(0, t, wt * (me @ dw.abs().t() + (F + k) * 2.0 ** -23 * (m.abs() @ dw.abs().t())))
    err = (out.double() - ref).abs()
    assert (err <= 2.0 ** -8 * ref.abs() + bound + 1e-6).all(), (err - bound).max().item()


def test_rows_wider_than_a_tiles_buffer_range():
    """256 rows of one expert, 2^21 + 64 fp32 outputs each: more than the 2^31 bytes that one buffer range of the 256-row
    tiles could address (columns outside the matrix, dropped by that range, landed inside it)."""
    T, d, E, k, F = 256, (1 << 21) + 64, 16, 5, 64
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    bf = dict(dtype=torch.bfloat16, device="cuda")
    b = torch.empty(T, d, **bf).normal_(generator=g)
    b[:, 0] = 1
    router = torch.zeros(E, d, **bf)
    router[:k, 0] = torch.arange(k, 0, -1) * 0.25   # every token: experts 0 .. 4
    gu = torch.empty(E, 2 * F, d, **bf).normal_(std=d ** -0.5, generator=g)
    dw = torch.empty(E, d, F, **bf).normal_(generator=g)
    out, ids, wts = B.eb_op_moe_ffn(b, router, gu, dw, k, return_routing=True)
    assert (ids == torch.arange(k, device="cuda")).all()
    at = (1 << 29) - 255 * d      # the column of the 256th row that lies 2^31 bytes into the tile
    cols = torch.cat([torch.arange(256), torch.arange(at - 128, at + 128), torch.arange(d - 256, d)]).cuda()
    ref, x = torch.zeros(T, cols.numel(), dtype=torch.float64, device="cuda"), b.double()
    for e in range(k):
        gt, up = x @ gu[e, :F].double().t(), x @ gu[e, F:].double().t()
        ref += wts[:, e, None].double() * ((gt * torch.sigmoid(gt) * up) @ dw[e, cols].double().t())
    # m is rounded to bf16 (2^-9 of each of the 64 terms), the sums behind it to 1e-4 of values near 1
    err = (out[:, cols].double() - ref).abs().max() / ref.abs().max()
    assert err < 1e-2, err.item()
