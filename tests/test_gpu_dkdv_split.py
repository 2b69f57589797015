"""bf16 at 192/128-wide heads: dK/dV with the queries split over pairs of waves (causal below
2304 tokens, no mask below 1280) and without, against the oracle where their tiles end: a
single key, a last step with one of its two query tiles empty (33 = 32 + 1 rows; 96), partial
tiles, one key past a 64-key workgroup, both sides of each line of the rule. Same bar as
everywhere (2e-2 of unit scale). And a head's results do not depend on the heads and batch
elements beside it on either side of the line."""
import pytest

import laga_inputs as LI
from oracle import laga as O
from _util import check_tol, dev_inputs, f64, problem_for

pytestmark = pytest.mark.gpu

NAMES = ("dq", "dc_kv", "dk_pe", "dw_kv_b")


def step(w, d, **kw):
    import torch
    import paper_2607_17644_amd as L
    p = problem_for(w, **kw)
    kv = L.laga_reconstruct_kv(p, d["c_kv"], d["w_kv_b"])
    out, lse = L.laga_attn_fwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"], kv=kv)
    g = L.laga_attn_bwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"], kv, out, lse, d["dout"])
    torch.cuda.synchronize()
    return dict(zip(NAMES, g))


@pytest.mark.parametrize("S,H,causal", [(1, 1, True), (33, 2, True), (96, 3, False), (65, 8, False), (129, 1, True),
                                        (1279, 1, False), (1280, 1, False), (2303, 1, True), (2304, 1, True)])
def test_edges(S, H, causal):
    import paper_2607_17644_amd as L
    w = LI.WORKLOADS["v3_train_s16384"].replace(seq_len=S, n_heads=H, causal=causal, seed=S)
    x = LI.make_inputs(w)
    d = dev_inputs(w, x)
    ref = O.attn_bwd(x["q"], x["c_kv"], x["k_pe"], x["w_kv_b"], x["dout"], n_heads=H, d_nope=w.d_nope, d_v=w.d_v,
                     scale=w.scale, causal=causal)
    store, rec = step(w, d), step(w, d, dq_mode=L.DQ_RECOMPUTE)
    for n in NAMES:
        check_tol(n, f64(store[n]), ref[n], "bf16", (S, n))
        assert bool((store[n] == rec[n]).all()), n


# no mask and an odd number of 32-query tiles, at four steps or more: the last workgroup's second
# key half lies past every stored key, so its waves issue no dS^T store between the copies of
# the rows that the first half reads and the wait for them
@pytest.mark.parametrize("S", [200, 260, 515, 900, 1247])
def test_last_workgroup_without_stores(S):
    import torch
    import paper_2607_17644_amd as L
    w = LI.WORKLOADS["v3_train_s16384"].replace(seq_len=S, n_heads=2, causal=False, seed=S)
    x = LI.make_inputs(w)
    d = dev_inputs(w, x)
    ref = O.attn_bwd(x["q"], x["c_kv"], x["k_pe"], x["w_kv_b"], x["dout"], n_heads=2, d_nope=w.d_nope, d_v=w.d_v,
                     scale=w.scale, causal=False)
    store, rec = step(w, d), step(w, d, dq_mode=L.DQ_RECOMPUTE)
    p = problem_for(w, kv_mode=L.KV_FUSED)
    out, lse = L.laga_attn_fwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"])
    fused = dict(zip(NAMES, L.laga_attn_bwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"], None, out, lse, d["dout"])))
    for n in NAMES:
        check_tol(n, f64(store[n]), ref[n], "bf16", (S, n))
        assert torch.equal(store[n], rec[n]), n  # the recomputing form has no store and waits for everything
        assert torch.equal(store[n], fused[n]), n


# K/V rebuilt on chip, half of the columns in each of the two waves of the same keys: equal bit
# for bit to K/V from memory, for contractions of one to four groups of steps
@pytest.mark.parametrize("S,H,d_c,causal", [(1, 2, 128, True), (33, 1, 256, True), (65, 3, 384, False),
                                            (300, 2, 128, False), (1000, 2, 384, True), (2303, 1, 512, True)])
def test_rebuilt_kv(S, H, d_c, causal):
    import torch
    import paper_2607_17644_amd as L
    w = LI.WORKLOADS["v3_train_s16384"].replace(seq_len=S, n_heads=H, d_c=d_c, causal=causal, seed=S)
    d = dev_inputs(w, LI.make_inputs(w))
    mat = step(w, d)
    p = problem_for(w, kv_mode=L.KV_FUSED)
    out, lse = L.laga_attn_fwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"])
    fused = dict(zip(NAMES, L.laga_attn_bwd(p, d["q"], d["c_kv"], d["k_pe"], d["w_kv_b"], None, out, lse, d["dout"])))
    for n in NAMES:
        assert torch.equal(mat[n], fused[n]), n


@pytest.mark.parametrize("S", [300, 2100])
def test_heads_and_batch_beside_do_not_matter(S):
    import torch
    w = LI.WORKLOADS["v3_train_s16384"].replace(seq_len=S, n_heads=4, batch=2)
    d = dev_inputs(w, LI.make_inputs(w))
    full = step(w, d)
    ws = w.replace(n_heads=1, batch=1)
    ds = {"q": d["q"][1:2, :, 2:3].contiguous(), "c_kv": d["c_kv"][1:2].contiguous(),
          "k_pe": d["k_pe"][1:2].contiguous(), "w_kv_b": d["w_kv_b"][:, 512:768].contiguous(),
          "dout": d["dout"][1:2, :, 2:3].contiguous()}
    assert torch.equal(step(ws, ds)["dq"], full["dq"][1:2, :, 2:3])
    wb = w.replace(batch=1)
    db = {k: (v if k == "w_kv_b" else v[1:2].contiguous()) for k, v in d.items()}
    assert torch.equal(step(wb, db)["dk_pe"], full["dk_pe"][1:2])
    wh = w.replace(n_heads=2)
    dh = {"q": d["q"][:, :, 2:].contiguous(), "c_kv": d["c_kv"], "k_pe": d["k_pe"],
          "w_kv_b": d["w_kv_b"][:, 512:].contiguous(), "dout": d["dout"][:, :, 2:].contiguous()}
    assert torch.equal(step(wh, dh)["dw_kv_b"], full["dw_kv_b"][:, 512:])
