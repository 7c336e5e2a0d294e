"""The layer's products where their split over the chip changes: row counts around the 32-row blocks and
the kernels' limits (1, 64, 128 rows), ragged numbers of weight tiles per workgroup and of K steps per
wave, every weight format, against the float64 oracle: small layer stacks, and one layer of the 7B shape in
every form that the planner gives it."""
import numpy as np
import pytest
import torch

from paper_2507_22424_amd import binding as sv
from paper_2507_22424_amd import workload as wl

from oracle import verify_oracle as vo
from parity_utils import SideBySide, bf16_store, f64, row_rel_err, say, worst_row
from test_gpu_parity import check_forward

pytestmark = pytest.mark.gpu

# Residual stream and logits, against an oracle whose cache holds bf16 values too.  An activation is two bf16
# parts, which loses 2^-17 of it, sums are float32, rotary angles hold 2e-5 at these positions; with that, a few
# appended K/V values round to the neighbour of the oracle's.  An emulation of all of it on these cases leaves at
# most 2e-5 of a row, one that drops the low parts at least 2.4e-3 of the logits (and 3.5e-4 .. 3.7e-3 of x).
TOL = 2e-4
# Attention output: a value that rounds to its neighbour moves by up to 2^-7, and the 20 keys and more of these
# rows, drawn small, share the weight.  Emulated as above: up to 1e-3.
TOL_ATTN = 2e-3


@pytest.mark.parametrize("dtype,T,B,H,F", [
    ("bf16", 1, 1, 512, 768), ("bf16", 32, 1, 1024, 2816), ("bf16", 33, 1, 512, 1280), ("bf16", 32, 2, 1024, 2816),
    ("bf16", 65, 1, 1024, 2816), ("bf16", 96, 1, 512, 768), ("bf16", 97, 1, 1024, 2816), ("bf16", 64, 2, 512, 1280),
    ("bf16", 43, 3, 1024, 2816), ("bf16", 80, 2, 512, 768), ("bf16", 23, 7, 1024, 2816), ("bf16", 64, 5, 512, 1280),
    ("bf16_w8", 1, 1, 512, 768), ("bf16_w8", 64, 1, 1024, 2816), ("bf16_w8", 97, 1, 512, 1280), ("bf16_w8", 43, 3, 1024, 2816),
    # two chunks of 64 k-values in a slice
    ("bf16_w8", 64, 5, 512, 1280), ("bf16_w8", 64, 4, 1024, 2816),
    # gate/up groups of 2.25 weight tiles: they end at half tiles (not at 33 rows)
    ("bf16", 1, 1, 1024, 2304), ("bf16", 32, 1, 1024, 2304), ("bf16", 8, 3, 1024, 2304), ("bf16", 33, 1, 1024, 2304),
    ("bf16_w4", 1, 1, 512, 768), ("bf16_w4", 64, 1, 1024, 2816), ("bf16_w4", 97, 1, 512, 1280), ("bf16_w4", 43, 3, 1024, 2816),
])
def test_products_at_the_edges_of_their_split(dtype, T, B, H, F):
    cfg = wl.C2.scaled(name=f"edge-{dtype}-{B}x{T}-{H}-{F}", index=80 + B, dtype=dtype, n_layers=2, hidden=H,
                       n_heads=H // 128, head_dim=128, mlp_dim=F, vocab=1024, n_bins=256, tree_nodes=T,
                       n_episodes=B, prefix_lo=20, prefix_hi=30, max_children=6, spine_lo=min(3, T - 1), r_values=(0, 4))
    check_forward(SideBySide(cfg, store=bf16_store, stack_tol=TOL), TOL, TOL_ATTN)


@pytest.mark.parametrize("T,B", [(20, 1), (65, 2)])
def test_every_finite_e4m3_code(T, B, monkeypatch):
    """Codes drawn evenly from all 254 finite ones, subnormals and 448 among them (drawn weights use the middle of
    the range only), on both product kernels."""
    drawn = wl.layer_weights_w8

    def all_codes(cfg, layer):
        w, rng = drawn(cfg, layer), np.random.default_rng(layer)
        codes = np.array([c for c in range(256) if c & 0x7f != 0x7f], dtype=np.uint8)
        for n in ("wq", "wk", "wv", "wo", "wg", "wu", "wd"):
            w[n] = torch.from_numpy(rng.choice(codes, size=tuple(w[n].shape)))
            w[n + "_scale"] = w[n + "_scale"] * 0 + 2e-4       # (the codes' root mean square is 100)
        return w

    monkeypatch.setattr(wl, "layer_weights_w8", all_codes)
    cfg = wl.C2.scaled(name=f"codes-{B}x{T}", index=79, dtype="bf16_w8", n_layers=2, hidden=512, n_heads=4, head_dim=128, mlp_dim=768,
                       vocab=1024, n_bins=256, tree_nodes=T, n_episodes=B, prefix_lo=20, prefix_hi=30, max_children=6, spine_lo=3,
                       r_values=(0, 4))
    check_forward(SideBySide(cfg, store=bf16_store, stack_tol=TOL), TOL, TOL_ATTN)


# One layer of the 7B shape.  Episodes and nodes for which the planner gives each product, up to 960 rows of bf16
# weights and 640 of the others, every form it has (tests/test_plan_coverage.py holds the lists to that).
# Here the softmax often picks one key, and 4096 terms make large keys: appended values that round to the
# neighbour of the oracle's (0.1 - 1 % of them, after 1e-6 .. 1e-5 of error) move x by up to 3.5e-4 and the logits
# by 3.7e-4 in an emulation; dropping the low parts 3.3e-3 and 4.3e-3.
TOL_WIDE = 8e-4
TOL_WIDE_ATTN = 2.0 ** -7        # a picked value passes whole: one unit in its last place
WIDE_LAYERS = {"bf16": [(1, 65), (3, 50), (7, 23), (4, 60), (5, 60), (3, 107), (5, 77), (13, 37), (9, 57), (6, 107), (10, 77)],
               "bf16_w8": [(1, 65), (1, 128), (3, 50), (7, 23), (4, 60), (3, 93), (3, 107), (5, 77), (13, 37), (9, 57)],
               "bf16_w4": [(1, 65), (1, 128), (3, 50), (7, 23), (4, 60), (3, 93), (3, 107), (5, 77), (13, 37), (9, 57)]}
UP_TO_16 = {"bf16": [1, 16], "bf16_w8": [16], "bf16_w4": [1, 16]}    # nodes of one episode, likewise
WIDE_ELSEWHERE = {"bf16": [26, 60, 128, 960], "bf16_w8": [26, 60], "bf16_w4": [26, 60]}   # rows, in test_gpu_parity.py


@pytest.mark.parametrize("dtype,B,T", [(dtype, B, T) for dtype, sizes in WIDE_LAYERS.items() for B, T in sizes])
def test_one_7b_layer_in_every_form_of_its_products(dtype, B, T):
    cfg = wl.C2.scaled(name=f"wide-{dtype}-{B}x{T}", index=90 + B, dtype=dtype, vocab=32000, tree_nodes=T, n_episodes=B,
                       prefix_lo=190, prefix_hi=210, max_children=6, spine_lo=3, r_values=(0, 4))
    check_forward(SideBySide(cfg, store=bf16_store, stack_tol=TOL_WIDE), TOL_WIDE, TOL_WIDE_ATTN)


# rows of the packed head over the whole vocabulary, likewise
WIDE_HEAD = [1, 26, 60, 65, 97, 150, 161, 240, 300, 400, 780]


def test_full_vocabulary_head_in_every_form_of_its_product():
    H, V = 4096, 32000
    cfg = sv.model_cfg("bf16", H, 32, 128, 11008, V)
    gen = torch.Generator().manual_seed(23)
    x = torch.randn(max(WIDE_HEAD), H, generator=gen)
    g = (1.0 + 0.1 * torch.randn(H, generator=gen)).to(torch.bfloat16)
    w = (0.02 * torch.randn(V, H, generator=gen)).to(torch.bfloat16)
    ref, _ = vo.action_head(f64(x), f64(g), f64(w), 0, 1e-5)
    xd = x.cuda()
    packed = torch.empty(sv.sv_packed_head_bytes(cfg, 0, V), dtype=torch.uint8, device="cuda")
    sv.sv_pack_head(cfg, g.cuda(), w.cuda(), 0, V, packed)
    ws = torch.empty(sv.sv_workspace_bytes(cfg, 13, 60, V), dtype=torch.uint8, device="cuda").fill_(0xFF)
    sv.sv_workspace_init(cfg, 13, 60, V, ws)
    off, _ = sv.sv_workspace_region(cfg, 13, 60, V, sv.SV_WS_STATUS)
    for n in WIDE_HEAD:
        token = torch.full((n,), -1, dtype=torch.int32, device="cuda")
        logits = torch.full((n, V), float("nan"), dtype=torch.float32, device="cuda")
        sv.sv_action_head_argmax_packed(cfg, packed, xd, n, 0, V, token, logits, ws)
        assert int(ws[off:off + 4].view(torch.int32).item()) == 0
        got = logits.cpu().numpy()
        err = worst_row(row_rel_err(got, ref[:n]))
        say(f"[wide head] {n} rows: logit err {err:.2e}")
        assert err <= TOL
        assert np.array_equal(token.cpu().numpy(), np.argmax(got, axis=1))


@pytest.mark.parametrize("H", [512, 4096])
def test_head_of_few_columns_on_blocks_of_rows(H):
    """Up to two weight tiles per XCD and more than 64 rows: one to four 32-row blocks per workgroup, the last block
    of rows full, ragged or partly beyond the rows; one column tile, one and two per XCD."""
    V, rows = 512, [65, 96, 128, 129, 225, 257, 289, 400, 481, 673, 960]
    cfg = sv.model_cfg("bf16", H, H // 128, 128, 256, V)
    gen = torch.Generator().manual_seed(29)
    x = torch.randn(max(rows), H, generator=gen)
    g = (1.0 + 0.1 * torch.randn(H, generator=gen)).to(torch.bfloat16)
    w = (0.02 * torch.randn(V, H, generator=gen)).to(torch.bfloat16)
    ref, _ = vo.action_head(f64(x), f64(g), f64(w), 0, 1e-5)
    xd, gd, wd = x.cuda(), g.cuda(), w.cuda()
    for n in (32, 256, 512):
        packed = torch.empty(sv.sv_packed_head_bytes(cfg, V - n, V), dtype=torch.uint8, device="cuda")
        sv.sv_pack_head(cfg, gd, wd, V - n, V, packed)
        ws = torch.empty(sv.sv_workspace_bytes(cfg, 16, 60, n), dtype=torch.uint8, device="cuda").fill_(0xFF)
        sv.sv_workspace_init(cfg, 16, 60, n, ws)
        off, _ = sv.sv_workspace_region(cfg, 16, 60, n, sv.SV_WS_STATUS)
        for M in rows:
            token = torch.full((M + 1,), -7, dtype=torch.int32, device="cuda")
            logits = torch.full((M + 1, n), -7.0, dtype=torch.float32, device="cuda")
            sv.sv_action_head_argmax_packed(cfg, packed, xd, M, V - n, V, token, logits, ws)
            assert int(ws[off:off + 4].view(torch.int32).item()) == 0
            got = logits.cpu().numpy()
            assert worst_row(row_rel_err(got[:M], ref[:M, V - n:])) <= TOL, (n, M)
            assert np.array_equal(token[:M].cpu().numpy(), V - n + np.argmax(got[:M], axis=1))
            assert (got[M] == -7.0).all() and int(token[M]) == -7


# float32: sums of at most 8192 products in another order than the oracle's float64, 2^-24 each and random in
# sign: below 1e-6 of a row; the parity tests' bound for float32 models leaves room for the softmax.
TOL_F32 = 1e-5


@pytest.mark.parametrize("T,B,P,H,nh,d,F,V", [
    (1, 1, 5, 256, 4, 64, 688, 512),          # one row in a tile of 16
    (17, 2, 40, 254, 3, 10, 77, 300),         # K no multiple of 4, odd half heads, ragged tiles everywhere
    (33, 1, 250, 132, 2, 36, 90, 512),        # ragged K of 16-byte rows; keys beyond one pass of 256
    (128, 1, 600, 64, 2, 128, 64, 512),       # two mask words, three passes, columns dealt in two key groups a wave
    (128, 2, 20, 64, 32, 128, 8192, 8192),    # 64 x 64 blocks: q/k/v, gate/up, head
    (100, 3, 20, 8192, 1, 64, 64, 512),       # 64 x 64 blocks: output, down; rows ragged
])
def test_float32_products_and_attention_at_their_edges(T, B, P, H, nh, d, F, V):
    cfg = wl.C1.scaled(name=f"f32-{B}x{T}-{H}-{nh}x{d}-{F}", index=60 + B, n_layers=1, hidden=H, n_heads=nh, head_dim=d, mlp_dim=F,
                       vocab=V, n_bins=256, tree_nodes=T, n_episodes=B, prefix_lo=max(1, P - 9), prefix_hi=P, max_children=6,
                       spine_lo=min(3, T - 1), r_values=(0, 4))
    check_forward(SideBySide(cfg, full_vocab=V > 4096), TOL_F32)


@pytest.mark.parametrize("dtype,d,shift", [("f32", 64, 0), ("f32", 6, 0), ("f32", 64, 1), ("bf16", 128, 0), ("bf16", 128, 1)])
def test_commit_of_deep_paths_and_unaligned_caches(dtype, d, shift):
    """Paths of up to 31 nodes (several passes of the copy), a moved row that is itself the target of a deeper
    node, caches whose rows are not aligned to 16 bytes (shift: elements): rows move as one after the other."""
    B, T, d_cap, nh, cap = 3, 128, 31, 2, 192
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    cfg = sv.ModelCfg(sv.SV_F32 if dtype == "f32" else sv.SV_BF16, 256, nh, d, 256, 512, 1e-5, 1e4)
    prefix, n = [7, 0, 33], B * nh * cap * d
    gen = torch.Generator().manual_seed(5)
    k0, v0 = (torch.randn(n, generator=gen).to(tdt) for _ in "kv")
    buf = [torch.zeros(n + 8, dtype=tdt, device="cuda") for _ in "kv"]
    for t, src in zip(buf, (k0, v0)):
        t[shift:shift + n] = src.cuda()
    path = np.full((B, d_cap + 1), -1, dtype=np.int32)
    path[0] = np.arange(32) * 4                             # 0, 4, 8, ...: node 4 moves to row 1, node 16 to row 4, ...
    path[1, :9] = [0, 2, 3, 4, 5, 6, 7, 8, 100]             # every source row but one is a target as well
    path[2, :4] = [0, 1, 2, 127]
    alen = np.array([31, 8, 3], dtype=np.int32)
    plen = torch.tensor(prefix, dtype=torch.int32, device="cuda")
    size = k0.element_size()
    view = sv.KvView(buf[0].data_ptr() + shift * size, buf[1].data_ptr() + shift * size, plen.data_ptr(), max(prefix), cap)
    sv.sv_commit_path(cfg, view, T, torch.from_numpy(path).cuda(), torch.from_numpy(alen).cuda(), B, d_cap)
    torch.cuda.synchronize()
    for t, src in zip(buf, (k0, v0)):
        want = src.clone().reshape(B, nh, cap, d)
        for b in range(B):
            for i in range(1, alen[b] + 1):
                want[b, :, prefix[b] + i] = want[b, :, prefix[b] + path[b, i]].clone()
        assert torch.equal(t[shift:shift + n].cpu().reshape(B, nh, cap, d), want)
        assert not t[:shift].any() and not t[shift + n:].any()


@pytest.mark.parametrize("dtype", ["bf16", "bf16_w8", "bf16_w4"])
@pytest.mark.parametrize("T,B,H,F", [(16, 1, 1024, 2816), (15, 1, 512, 768), (4, 4, 1024, 2304), (17, 1, 1024, 2304), (1, 1, 512, 1280)])
def test_up_to_16_rows(dtype, T, B, H, F):
    """Both sides of the row count up to which half of the rows is left out; K slices shorter than the rings (512), odd
    numbers of steps per wave, groups that end at half tiles (2304)."""
    cfg = wl.C2.scaled(name=f"thin-{dtype}-{B}x{T}-{H}-{F}", index=60 + B, dtype=dtype, n_layers=2, hidden=H, n_heads=H // 128,
                       head_dim=128, mlp_dim=F, vocab=1024, n_bins=256, tree_nodes=T, n_episodes=B, prefix_lo=20, prefix_hi=30,
                       max_children=6, spine_lo=min(3, T - 1), r_values=(0, 4))
    check_forward(SideBySide(cfg, store=bf16_store, stack_tol=TOL), TOL, TOL_ATTN)


@pytest.mark.parametrize("dtype,T", [(dtype, T) for dtype, nodes in UP_TO_16.items() for T in nodes])
def test_one_7b_layer_of_up_to_16_rows(dtype, T):
    test_one_7b_layer_in_every_form_of_its_products(dtype, 1, T)


@pytest.mark.parametrize("T,H,heads,F", [(16, 4096, 2, 256), (9, 4096, 10, 2048), (16, 512, 4, 4096)])
def test_4_bit_weights_of_few_tiles_up_to_16_rows(T, H, heads, F):
    """gemm_thin takes 4-bit weights from two steps a wave on: its forms of two and four tiles, with exactly two."""
    cfg = wl.C2.scaled(name=f"thin-w4-{T}-{H}-{heads}-{F}", index=70, dtype="bf16_w4", n_layers=1, hidden=H, n_heads=heads,
                       head_dim=128, mlp_dim=F, vocab=1024, n_bins=256, tree_nodes=T, n_episodes=1, prefix_lo=20, prefix_hi=30,
                       max_children=6, spine_lo=3, r_values=(0, 4))
    check_forward(SideBySide(cfg, store=bf16_store, stack_tol=TOL_WIDE), TOL_WIDE, TOL_WIDE_ATTN)
