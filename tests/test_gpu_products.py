"""The layer's products where their split over the chip changes: row counts around the 32-row blocks and
the kernels' limits (1, 64, 128 rows), ragged numbers of weight tiles per workgroup and of K steps per
wave, every weight format.  One small layer stack against the float64 oracle."""
import pytest

from paper_2507_22424_amd import workload as wl

from parity_utils import SideBySide
from test_gpu_parity import check_forward

pytestmark = pytest.mark.gpu

# The products themselves are within K * 2^-24 + 2^-16 < 2e-4 of exact (float32 sums of hi + lo bf16 parts);
# what remains is the rounding of the appended K/V rows to bf16 (2^-9 each): about 4e-3 of a row's largest
# value after a softmax over a few dozen of them, with a margin of 2.5.
TOL = 1e-2


@pytest.mark.parametrize("dtype,T,B,H,F", [
    ("bf16", 1, 1, 512, 768), ("bf16", 32, 1, 1024, 2816), ("bf16", 33, 1, 512, 1280), ("bf16", 32, 2, 1024, 2816),
    ("bf16", 65, 1, 1024, 2816), ("bf16", 96, 1, 512, 768), ("bf16", 97, 1, 1024, 2816), ("bf16", 64, 2, 512, 1280),
    ("bf16", 43, 3, 1024, 2816), ("bf16", 80, 2, 512, 768), ("bf16", 23, 7, 1024, 2816), ("bf16", 64, 5, 512, 1280),
    ("bf16_w8", 1, 1, 512, 768), ("bf16_w8", 64, 1, 1024, 2816), ("bf16_w8", 97, 1, 512, 1280), ("bf16_w8", 43, 3, 1024, 2816),
    ("bf16_w4", 1, 1, 512, 768), ("bf16_w4", 64, 1, 1024, 2816), ("bf16_w4", 97, 1, 512, 1280), ("bf16_w4", 43, 3, 1024, 2816),
])
def test_products_at_the_edges_of_their_split(dtype, T, B, H, F):
    cfg = wl.C2.scaled(name=f"edge-{dtype}-{B}x{T}-{H}-{F}", index=80 + B, dtype=dtype, n_layers=2, hidden=H,
                       n_heads=H // 128, head_dim=128, mlp_dim=F, vocab=1024, n_bins=256, tree_nodes=T,
                       n_episodes=B, prefix_lo=20, prefix_hi=30, max_children=6, spine_lo=min(3, T - 1), r_values=(0, 4))
    check_forward(SideBySide(cfg), TOL)
