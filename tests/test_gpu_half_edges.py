"""bf16 at 64/32/64-wide heads (the ring forward, dkdv_half_kernel and the recomputing dQ pass)
against the oracle where their tiles end: one key, one past a 32-row tile, a 64-key tile, a
128-row workgroup and a four-slot ring, with and without the mask, and more heads than one per
XCD or a head count that is no multiple of 8. Same bar as everywhere (2e-2 of unit scale)."""
import pytest

import laga_inputs as LI
from oracle import laga as O
from _util import check_tol, dev_inputs, f64, problem_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("S,H,B,causal", [(1, 1, 1, True), (31, 3, 1, False), (33, 5, 2, True), (64, 8, 1, True),
                                          (65, 2, 1, False), (127, 8, 2, True), (129, 4, 1, True),
                                          (257, 16, 1, False), (1153, 8, 1, True)])
def test_half_width_edges(S, H, B, causal):
    import torch
    import paper_2607_17644_amd as L
    w = LI.WORKLOADS["v3_train_s16384"].replace(seq_len=S, n_heads=H, batch=B, causal=causal, d_c=128, d_nope=64,
                                                d_rope=32, d_v=64, seed=S)
    x = LI.make_inputs(w)
    d = dev_inputs(w, x)
    p = problem_for(w)
    kv = L.laga_reconstruct_kv(p, d["c_kv"], d["w_kv_b"])
    out, lse = L.laga_attn_fwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"], kv=kv)
    g = L.laga_attn_bwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"], kv, out, lse, d["dout"])
    torch.cuda.synchronize()
    kw = dict(n_heads=H, d_nope=64, d_v=64, scale=w.scale, causal=causal)
    ro, rl = O.attn_fwd(x["q"], x["c_kv"], x["k_pe"], x["w_kv_b"], **kw)
    ref = O.attn_bwd(x["q"], x["c_kv"], x["k_pe"], x["w_kv_b"], x["dout"], **kw)
    check_tol("out", f64(out), ro, "bf16", S)
    check_tol("lse", f64(lse), rl, "bf16", S)
    for n, a in zip(("dq", "dc_kv", "dk_pe", "dw_kv_b"), g):
        check_tol(n, f64(a), ref[n], "bf16", S)
