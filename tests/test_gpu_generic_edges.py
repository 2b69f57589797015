"""The generic backward kernels (fp32 at every head width, bf16 at 32/16/32) against the oracle
where their work is divided: one row, one past a 32-row tile and a 64-row workgroup, an odd and
an even number of tiles (the two pairs of waves take the even and the odd ones), a last tile
without rows for one pair, with and without the mask. The usual bar: 1e-4 in fp32, 2e-2 in
bf16."""
import pytest

import laga_inputs as LI
from oracle import laga as O
from _util import check_tol, dev_inputs, f64, problem_for

pytestmark = pytest.mark.gpu

WIDTHS = {"v3": (128, 64, 128), "half": (64, 32, 64), "small": (32, 16, 32)}


@pytest.mark.parametrize("dtype,width,S,H,B,causal", [
    ("fp32", "v3", 1, 1, 1, True), ("fp32", "v3", 33, 2, 1, True), ("fp32", "v3", 97, 8, 1, False),
    ("fp32", "half", 64, 3, 2, True), ("fp32", "half", 65, 1, 1, False), ("fp32", "half", 161, 4, 1, True),
    ("fp32", "small", 31, 8, 1, False), ("fp32", "small", 96, 5, 2, True), ("fp32", "small", 513, 2, 1, True),
    ("bf16", "small", 32, 1, 1, True), ("bf16", "small", 63, 8, 1, False), ("bf16", "small", 129, 3, 2, True)])
def test_edges(dtype, width, S, H, B, causal):
    import torch
    import paper_2607_17644_amd as L
    dn, dr, dv = WIDTHS[width]
    w = LI.WORKLOADS["v3_train_s16384"].replace(seq_len=S, n_heads=H, batch=B, causal=causal, dtype=dtype, d_c=64,
                                                d_nope=dn, d_rope=dr, d_v=dv, seed=S)
    x = LI.make_inputs(w)
    d = dev_inputs(w, x)
    p = problem_for(w)
    kv = L.laga_reconstruct_kv(p, d["c_kv"], d["w_kv_b"])
    out, lse = L.laga_attn_fwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"], kv=kv)
    g = L.laga_attn_bwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"], kv, out, lse, d["dout"])
    torch.cuda.synchronize()
    ref = O.attn_bwd(x["q"], x["c_kv"], x["k_pe"], x["w_kv_b"], x["dout"], n_heads=H, d_nope=dn, d_v=dv, scale=w.scale,
                     causal=causal)
    for n, a in zip(("dq", "dc_kv", "dk_pe", "dw_kv_b"), g):
        check_tol(n, f64(a), ref[n], dtype, (width, S, n))
