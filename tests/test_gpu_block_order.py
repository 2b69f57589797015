"""Attention workgroups over several groups of heads (see block_order in common.hpp), the last
group partial: every head's results equal, bit for bit, those of the same heads computed alone
in one group. Every attention kernel, with and without the mask."""
import pytest

pytestmark = pytest.mark.gpu

WIDTHS = {"v3": (128, 64, 128), "half": (64, 32, 64), "small": (32, 16, 32)}


# blocks per head: 4096 / 256 (forward, dQ: groups of 64 heads without the mask, 128 with it),
# 4096 / 128 (dK/dV, half-width heads: 32, 64), 4096 / 64 (generic dK/dV and dQ: 16, 32)
@pytest.mark.parametrize("widths,dtype,H,causal,fused,recompute,d_c", [
    ("v3", "bf16", 66, 0, 0, 0, 64), ("v3", "bf16", 132, 1, 0, 0, 64), ("v3", "bf16", 66, 0, 0, 1, 64),
    ("v3", "bf16", 66, 0, 1, 0, 512), ("v3", "bf16", 66, 0, 1, 0, 128), ("half", "bf16", 68, 1, 0, 0, 64),
    ("small", "bf16", 36, 1, 0, 0, 32), ("small", "fp32", 20, 0, 0, 0, 32), ("small", "fp32", 66, 1, 1, 0, 32)])
def test_heads_of_every_group(widths, dtype, H, causal, fused, recompute, d_c):
    import torch
    import paper_2607_17644_amd as L
    S, (dn, dr, dv) = 4096, WIDTHS[widths]
    gen = torch.Generator(device="cuda").manual_seed(H)

    def problem(h):
        return L.Problem(1, S, h, d_c, dn, dr, dv, (dn + dr) ** -0.5, causal=causal,
                         dtype=L.DTYPE_FP32 if dtype == "fp32" else L.DTYPE_BF16,
                         kv_mode=L.KV_FUSED if fused else L.KV_MATERIALIZED,
                         dq_mode=L.DQ_RECOMPUTE if recompute else L.DQ_FROM_STORE)

    p = problem(H)
    sh = p.shapes()
    c, kpe, q, dout = (torch.randn(sh[n], generator=gen, device="cuda").to(p.torch_dtype)
                       for n in ("c_kv", "k_pe", "q", "dout"))
    w = (torch.randn(sh["w_kv_b"], generator=gen, device="cuda") * d_c ** -0.5).to(p.torch_dtype)

    def step(p, q, dout, w):
        kv = None if fused else L.laga_reconstruct_kv(p, c, w)
        out, lse = L.laga_attn_fwd(p, q, c, kpe, w, kv)
        dq, _, _, dw = L.laga_attn_bwd(p, q, c, kpe, w, kv, out, lse, dout)
        return out, lse, dq, dw

    full = step(p, q, dout, w)
    for h0 in (0, 14, H - 4):
        hs, cols = slice(h0, h0 + 4), slice(h0 * (dn + dv), (h0 + 4) * (dn + dv))
        alone = step(problem(4), q[:, :, hs].contiguous(), dout[:, :, hs].contiguous(), w[:, cols].contiguous())
        for n, a, f in zip(("out", "lse", "dq", "dw_kv_b"), alone,
                           (full[0][:, :, hs], full[1][:, hs], full[2][:, :, hs], full[3][:, cols])):
            assert torch.equal(a, f), (n, h0)
    assert all(bool(torch.isfinite(t).all()) for t in full)
