"""One workspace, prepared once, for calls of several row counts: what a step returns does not depend on
what other sizes have run on the workspace before, and no call finds counters that are not zero."""
import numpy as np
import pytest
import torch

from oracle import fp8_weights as f8
from oracle import int4_weights as i4
from oracle import verify_oracle as vo
from paper_2507_22424_amd import binding as sv
from paper_2507_22424_amd import workload as wl
from paper_2507_22424_amd.runner import VerifyPass

from parity_utils import bf16_store, f64, row_rel_err, say, worst_row
from test_gpu_products import TOL_WIDE as TOL

pytestmark = pytest.mark.gpu

SMALL = dict(hidden=512, n_heads=4, head_dim=128, mlp_dim=1536, vocab=1024, n_bins=256)


def _prepared_for(vp):
    """A workspace full of ones, then initialised for the sizes of `vp`."""
    ws = torch.empty_like(vp.workspace).fill_(0xFF)
    sv.sv_workspace_init(vp.cfg, vp.B, vp.T, vp.n_scored, ws)
    return ws


def _status(vp):
    torch.cuda.synchronize()
    return vp.placement_status()


@pytest.mark.parametrize("dtype,model,sizes", [
    ("bf16", {}, [(1, 60), (1, 26), (1, 1), (1, 60)]),
    ("bf16", {}, [(10, 64), (8, 65), (10, 64)]),
    ("bf16", {}, [(16, 60), (1, 60), (16, 60)]),
    ("bf16_w8", SMALL, [(3, 64), (2, 50), (1, 128), (3, 64)]),
    ("bf16_w4", SMALL, [(3, 50), (1, 60), (3, 50)]),
])
def test_one_workspace_serves_several_row_counts(dtype, model, sizes):
    """One layer and the packed head, `sizes` (episodes, nodes) in turn on a workspace prepared for the first.
    Every result equals, bit for bit, that of the same call on a workspace of its own, and (first and last
    episode) the oracle's."""
    base = wl.C2.scaled(**dict(dict(name="ws", index=70, dtype=dtype, vocab=32000, n_layers=1, prefix_lo=560, prefix_hi=600,
                                    max_children=6, spine_lo=0), **model))
    raw = {"bf16": wl.layer_weights, "bf16_w8": wl.layer_weights_w8, "bf16_w4": wl.layer_weights_w4}[dtype](base, 0)
    dequantise = {"bf16": lambda n: f64(raw[n]), "bf16_w8": lambda n: f8.dequantise(raw[n].numpy(), raw[n + "_scale"].numpy()),
                  "bf16_w4": lambda n: i4.dequantise(raw[n].numpy(), raw[n + "_scale"].numpy())}[dtype]
    w64 = {n: f64(raw[n]) if n.startswith("g") else dequantise(n) for n in wl.LAYER_TENSORS}
    head = wl.head_weights(base)
    passes, packed, first = {}, None, {}
    for B, T in dict.fromkeys(sizes):
        cfg = base.scaled(n_episodes=B, tree_nodes=T)
        parents = [wl.episode_tree(cfg, b) for b in range(B)]
        vp = VerifyPass(cfg, wl.prefix_lengths(cfg), np.concatenate(parents))
        if packed is None:
            vp.load_layer(0, raw)
            packed = vp.packed[0]
        vp.packed[0] = packed
        for b, P in enumerate(wl.prefix_lengths(cfg)):
            vp.load_prefix(0, b, *wl.prefix_kv(cfg, b, 0, int(P)))
        vp.load_head(head["g_final"], head["w_lm"])
        vp.set_hidden(torch.cat([wl.hidden_rows(cfg, b) for b in range(B)]))
        vp.workspace = _prepared_for(vp)
        vp.forward()
        assert _status(vp) == 0
        first[B, T] = [t.clone() for t in (vp.x, vp.logits, vp.token)]
        passes[B, T] = vp
        for b in {0, B - 1}:
            P = int(wl.prefix_lengths(cfg)[b])
            kp, vpf = wl.prefix_kv(cfg, b, 0, P)
            ref = vo.verify_layer(f64(wl.hidden_rows(cfg, b)), w64, f64(kp), f64(vpf), parents[b], cfg.n_heads, cfg.rms_eps,
                                  cfg.rope_theta, bf16_store)["x"]
            logits, _ = vo.action_head(ref, f64(head["g_final"]), f64(head["w_lm"]), cfg.action_lo, cfg.rms_eps)
            rows = slice(b * T, (b + 1) * T)
            ex = worst_row(row_rel_err(vp.x[rows].cpu().numpy(), ref))
            el = worst_row(row_rel_err(vp.logits[rows].cpu().numpy(), logits))
            say(f"[workspace {dtype} {B}x{T}] episode {b}: x err {ex:.2e}, logit err {el:.2e}")
            assert ex <= TOL and el <= TOL
    shared = _prepared_for(passes[sizes[0]])
    for B, T in sizes:
        vp = passes[B, T]
        vp.workspace = shared
        vp.forward()
        assert _status(vp) == 0
        assert all(torch.equal(a, b) for a, b in zip((vp.x, vp.logits, vp.token), first[B, T])), (B, T)


def test_packed_head_of_fewer_rows_behind_a_pass_that_splits_its_attention():
    """A 60-node step over a long prefix fills its scratch, then the head alone on 1 and 26 rows."""
    cfg = wl.C2.scaled(name="ws-head", index=71, vocab=32000, tree_nodes=60, prefix_lo=1100, prefix_hi=1100, spine_lo=0)
    vp = VerifyPass(cfg, wl.prefix_lengths(cfg), wl.episode_tree(cfg, 0))
    vp.load_layer(0, wl.layer_weights(cfg, 0))
    vp.load_prefix(0, 0, *wl.prefix_kv(cfg, 0, 0, 1100))
    head = wl.head_weights(cfg)
    vp.load_head(head["g_final"], head["w_lm"])
    x = torch.randn(60, cfg.hidden, generator=torch.Generator().manual_seed(3))
    vp.set_hidden(x)
    vp.workspace = _prepared_for(vp)
    ref, _ = vo.action_head(f64(x), f64(head["g_final"]), f64(head["w_lm"]), cfg.action_lo, cfg.rms_eps)
    xd = x.cuda()
    for n in (26, 1, 60, 26):
        vp.forward()
        token = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        logits = torch.zeros(n, vp.n_scored, dtype=torch.float32, device="cuda")
        sv.sv_action_head_argmax_packed(vp.cfg, vp.packed_head, xd, n, vp.vocab_lo, vp.vocab_hi, token, logits, vp.workspace)
        assert _status(vp) == 0
        assert worst_row(row_rel_err(logits.cpu().numpy(), ref[:n])) <= TOL
        assert np.array_equal(token.cpu().numpy(), vp.vocab_lo + np.argmax(logits.cpu().numpy(), axis=-1))
