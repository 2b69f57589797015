"""The GEMMs behind laga_reconstruct_kv, laga_attn_bwd's dc_kv / dW and laga_out_proj_*
at the edges of their tile shapes and of the rules that choose them: partial row tiles,
contractions that end inside a 32-index stage (odd token counts; d_model and F at 16 mod 32),
single rows, and both sides of each rule. The reference is the product in float64 of the
same bf16 operands; the bounds follow from the arithmetic: fp32 accumulation of K bf16
products (relative 2^-24 per addition, a few ulp over sqrt(K) terms at these sizes: 2e-6 of
sum |a b|), then one rounding to the output type (bf16: half an ulp, 2^-9 relative)."""
import pytest

pytestmark = pytest.mark.gpu


def check(got, a, b, where):
    """got ~ a @ b (float64 device tensors), elementwise."""
    import torch
    ref, mag = a @ b, a.abs() @ b.abs()
    bound = 2e-6 * mag + (2.0 ** -8 if got.dtype == torch.bfloat16 else 0.0) * ref.abs() + 1e-30
    d = (got.double().reshape(ref.shape) - ref).abs()
    assert torch.isfinite(got).all(), where
    assert (d <= bound).all(), (where, float((d / bound).max()))


def randn(gen, *shape):
    import torch
    return torch.randn(shape, generator=gen, device="cuda").to(torch.bfloat16)


# fp32: 16-wide contraction steps loaded four ahead (2, 4, 6, 64 of them) and partial row tiles;
# fp32 accumulation of K products, 2^-24 relative per addition in the worst case (and one more
# for the sum of split ranges)
@pytest.mark.parametrize("T,H,d_c", [(1, 1, 32), (63, 2, 64), (65, 1, 96), (130, 3, 1024)])
def test_reconstruct_fp32(T, H, d_c):
    import torch
    import paper_2607_17644_amd as L
    gen = torch.Generator(device="cuda").manual_seed(T)
    c = torch.randn(1, T, d_c, generator=gen, device="cuda")
    w = torch.randn(d_c, H * 256, generator=gen, device="cuda")
    kv = L.laga_reconstruct_kv(L.Problem(1, T, H, d_c, 128, 64, 128, 0.07, dtype=L.DTYPE_FP32), c, w)
    a, b = c[0].double(), w.double()
    assert ((kv.double().reshape(T, -1) - a @ b).abs() <= (d_c + 1) * 2.0 ** -24 * (a.abs() @ b.abs())).all()


# fp32 weight gradient of W_o: the contraction over the tokens ends inside a step and inside
# the four steps in flight (1, 15, 17, 65 and 600 tokens, the last in two ranges)
@pytest.mark.parametrize("T", [1, 15, 17, 65, 600])
def test_out_proj_fp32(T):
    import torch
    import paper_2607_17644_amd as L
    gen = torch.Generator(device="cuda").manual_seed(T)
    p = L.OutProj(T, 5, 16, 144, dtype=L.DTYPE_FP32)
    out, w, dy = (torch.randn(s, generator=gen, device="cuda") for s in ((T, 5, 16), (80, 144), (T, 144)))
    y = L.laga_out_proj_fwd(p, out, w)
    d_out, dw = L.laga_out_proj_bwd(p, out, w, dy)
    o = out.reshape(T, 80).double()
    for got, a, b in ((y, o, w.double()), (d_out.reshape(T, 80), dy.double(), w.double().t()), (dw, o.t(), dy.double())):
        assert ((got.double() - a @ b).abs() <= (a.shape[1] + 1) * 2.0 ** -24 * (a.abs() @ b.abs())).all()


# N = 16 * 256: 256 x 128 tiles up to 2048 rows, 256 x 256 above (2049, 2304), partial row
# tiles in the persistent kernel (3841: one row in the last tile; 8000: uneven rounds), and
# 5001 rows (the second round of the persistent kernel would be mostly idle); d_c 480, 96:
# contractions too short for it
@pytest.mark.parametrize("T,H,d_c", [(1, 1, 512), (127, 16, 512), (129, 16, 96), (2049, 16, 512), (3841, 16, 512),
                                     (5001, 16, 512), (8000, 16, 512), (4097, 16, 480), (16383, 16, 512),
                                     (2047, 16, 512), (2304, 16, 512)])
def test_reconstruct(T, H, d_c):
    import torch
    import paper_2607_17644_amd as L
    gen = torch.Generator(device="cuda").manual_seed(T)
    c, w = randn(gen, 1, T, d_c), randn(gen, d_c, H * 256)
    kv = L.laga_reconstruct_kv(L.Problem(1, T, H, d_c, 128, 64, 128, 0.07), c, w)
    check(kv, c[0].double(), w.double(), (T, H, d_c))


@pytest.mark.parametrize("T,nh,dv,D", [(1, 2, 16, 48), (17, 3, 48, 80), (31, 1, 16, 7168), (33, 16, 128, 1040),
                                       (1000, 5, 16, 2064), (2047, 128, 128, 144), (300, 64, 128, 4112),
                                       (1001, 128, 128, 2000), (4097, 16, 128, 256)])
def test_out_proj(T, nh, dv, D):
    import torch
    import paper_2607_17644_amd as L
    gen = torch.Generator(device="cuda").manual_seed(D)
    F = nh * dv
    out, w, dy = randn(gen, T, nh, dv), randn(gen, F, D), randn(gen, T, D)
    p = L.OutProj(T, nh, dv, D)
    y = L.laga_out_proj_fwd(p, out, w)
    d_out, dw = L.laga_out_proj_bwd(p, out, w, dy)
    o = out.reshape(T, F).double()
    check(y, o, w.double(), "y")
    check(d_out, dy.double(), w.double().t(), "d_out")
    check(dw, o.t(), dy.double(), "dw_o")


# dc_kv / dW: 128 x 128 tiles with the contraction split (8, 4, 2, 1 ways), 128 x 512 tiles
# beyond 288 of them (9217 tokens), d_c <= 256; token counts at 1, 15, 16, 17, 31 mod 32 and
# token splits whose last range is short (1025 = 1024 + 1, 2563)
@pytest.mark.parametrize("S,H,d_c", [(1, 1, 32), (15, 1, 512), (17, 16, 512), (31, 3, 256), (1025, 16, 512),
                                     (2563, 16, 512), (4097, 2, 224), (9217, 16, 512)])
def test_up_projection_backward(S, H, d_c):
    """dc_kv and dW against float64 products of the dKV pair that the attention backward left
    in its workspace (hi + lo, read back from there)."""
    import torch
    import paper_2607_17644_amd as L
    gen = torch.Generator(device="cuda").manual_seed(S)
    p = L.Problem(1, S, H, d_c, 128, 64, 128, 192 ** -0.5, dq_mode=L.DQ_RECOMPUTE)
    c, kpe, q = randn(gen, 1, S, d_c), randn(gen, 1, S, 64), randn(gen, 1, S, H, 192)
    w = (randn(gen, d_c, H * 256).float() * d_c ** -0.5).to(torch.bfloat16)
    dout = randn(gen, 1, S, H, 128)
    kv = L.laga_reconstruct_kv(p, c, w)
    out, lse = L.laga_attn_fwd(p, q, c, kpe, w, kv)
    ws = torch.empty(L.laga_workspace_bytes(p, L.OP_BWD), dtype=torch.uint8, device="cuda")
    dq, dc, dkpe, dw = L.laga_attn_bwd(p, q, c, kpe, w, kv, out, lse, dout, workspace=ws)
    # workspace: delta and lse2 (fp32 [H, S rounded to 64]), then dKV hi and lo, each at a
    # multiple of 256 bytes
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    o1 = 2 * up(4 * H * ((S + 63) // 64 * 64))
    nb = 2 * S * H * 256
    dkv = sum(ws[o:o + nb].view(torch.bfloat16).double() for o in (o1, o1 + up(nb))).reshape(S, H * 256)
    check(dc, dkv, w.double().t(), "dc_kv")
    check(dw, c[0].double().t(), dkv, "dw_kv_b")


# splits of dc_kv's contraction that do not divide it (31 of 16384 indices, 21 of 11776, 51 of
# 34304): the ranges launched are no more than the partials that the workspace holds
@pytest.mark.parametrize("dtype,S,H,d_c", [("fp32", 1000, 64, 64), ("fp32", 300, 46, 512), ("bf16", 100, 134, 544)])
def test_dc_partials_stay_in_the_workspace(dtype, S, H, d_c):
    import torch
    import paper_2607_17644_amd as L
    gen = torch.Generator(device="cuda").manual_seed(S)
    bf = dtype == "bf16"
    p = L.Problem(1, S, H, d_c, 128, 64, 128, 192 ** -0.5, dtype=L.DTYPE_BF16 if bf else L.DTYPE_FP32,
                  dq_mode=L.DQ_RECOMPUTE)
    c, kpe, q, dout = (torch.randn(s, generator=gen, device="cuda").to(p.torch_dtype)
                       for s in ((1, S, d_c), (1, S, 64), (1, S, H, 192), (1, S, H, 128)))
    w = (torch.randn(d_c, H * 256, generator=gen, device="cuda") * d_c ** -0.5).to(p.torch_dtype)
    kv = L.laga_reconstruct_kv(p, c, w)
    out, lse = L.laga_attn_fwd(p, q, c, kpe, w, kv)
    need, guard = L.laga_workspace_bytes(p, L.OP_BWD), 4 * S * d_c + 4096
    buf = torch.full((need + guard,), 0x5A, dtype=torch.uint8, device="cuda")
    dq, dc, dkpe, dw = L.laga_attn_bwd(p, q, c, kpe, w, kv, out, lse, dout, workspace=buf[:need])
    torch.cuda.synchronize()
    assert bool((buf[need:] == 0x5A).all())
    up = lambda n: (n + 255) // 256 * 256  # noqa: E731
    o1, nb = 2 * up(4 * H * ((S + 63) // 64 * 64)), S * H * 256 * (2 if bf else 4)
    dkv = sum(buf[o:o + nb].view(p.torch_dtype).double() for o in ((o1, o1 + up(nb)) if bf else (o1,))).reshape(S, -1)
    for got, a, b in ((dc[0], dkv, w.double().t()), (dw, c[0].double().t(), dkv)):
        assert ((got.double() - a @ b).abs() <= (a.shape[1] + 1) * 2.0 ** -24 * (a.abs() @ b.abs())).all()


def test_tail_rows_do_not_leak():
    """Values far beyond the data's scale in the last token's row stay in that token's products:
    rows copied in the place of missing ones never reach a sum (33 tokens: one index in the
    second stage; infinities would turn 0 * inf into NaN everywhere)."""
    import torch
    import paper_2607_17644_amd as L
    gen = torch.Generator(device="cuda").manual_seed(5)
    T, D = 33, 64
    out, w, dy = randn(gen, T, 2, 32), randn(gen, 64, D), randn(gen, T, D)
    out[-1, 0, 0] = float("inf")
    dw = L.laga_out_proj_bwd(L.OutProj(T, 2, 32, D), out, w, dy)[1]
    ref = out.reshape(T, 64).double().t() @ dy.double()
    assert torch.equal(torch.isfinite(dw), torch.isfinite(ref))
    assert torch.equal(dw[0].isinf(), ref[0].isinf()) and bool(dw[0].isinf().all())


# kv and dW columns of a head, whatever the number of heads: 2048 tokens take small tiles (4
# heads), middle (16), large (18) and the persistent kernel (32); 2200 the last of them ragged;
# 300 share dc's and dW's launch at 16 heads and not at 64; 1100 split dW's tokens
@pytest.mark.parametrize("T,heads", [(2048, (4, 16, 18, 32)), (2200, (4, 16, 32)), (300, (1, 16, 64)),
                                     (1100, (2, 16, 40))])
def test_columns_do_not_depend_on_the_heads(T, heads):
    import torch
    import paper_2607_17644_amd as L
    gen = torch.Generator(device="cuda").manual_seed(T)
    H = max(heads)
    c, kpe, q, dout = randn(gen, 1, T, 512), randn(gen, 1, T, 64), randn(gen, 1, T, H, 192), randn(gen, 1, T, H, 128)
    w = (randn(gen, 512, H * 256).float() * 512 ** -0.5).to(torch.bfloat16)
    res = {}
    for h in heads:
        p = L.Problem(1, T, h, 512, 128, 64, 128, 192 ** -0.5, dq_mode=L.DQ_RECOMPUTE)
        qh, dh, wh = q[:, :, :h].contiguous(), dout[:, :, :h].contiguous(), w[:, :h * 256].contiguous()
        kv = L.laga_reconstruct_kv(p, c, wh)
        out, lse = L.laga_attn_fwd(p, qh, c, kpe, wh, kv)
        res[h] = kv, L.laga_attn_bwd(p, qh, c, kpe, wh, kv, out, lse, dh)[3]
    for h in heads:
        n = min(heads)
        assert torch.equal(res[h][0][:, :, :n], res[n][0]), h
        assert torch.equal(res[h][1][:, :n * 256], res[n][1]), h
