"""Every form in which the planner splits a product of the 7B shape - kernel, row blocks, weight tiles, K slices,
weight format - is held to the oracle by a GPU test: the listed sizes reach all forms of the declared range."""
import pytest

import bench
from paper_2507_22424_amd import binding as sv
from perf import cases
from test_gpu_products import UP_TO_16, WIDE_ELSEWHERE, WIDE_HEAD, WIDE_LAYERS

LAYER = (sv.SV_PLAN_QKV, sv.SV_PLAN_OUT, sv.SV_PLAN_GATE_UP, sv.SV_PLAN_DOWN)


def _cfg(dtype):
    return sv.model_cfg(dtype, *cases.MODELS["7b"])


def _forms(dtype, rows):
    return {(which,) + sv.sv_product_plan(_cfg(dtype), rows, which)[:4] for which in LAYER}


def _layer_rows(dtype):
    return [B * T for B, T in WIDE_LAYERS[dtype]] + UP_TO_16[dtype] + WIDE_ELSEWHERE[dtype]


def _head_form(rows, n):
    return sv.sv_product_plan(_cfg("bf16"), rows, sv.SV_PLAN_HEAD, n)[:4]


@pytest.mark.parametrize("dtype,most", [("bf16", 960), ("bf16_w8", 640), ("bf16_w4", 640)])
def test_every_form_of_a_layers_products_has_a_test(dtype, most):
    tested = set().union(*(_forms(dtype, M) for M in _layer_rows(dtype)))
    missing = {M: _forms(dtype, M) - tested for M in range(1, most + 1)}
    assert not {M: f for M, f in missing.items() if f}


def test_every_form_of_the_heads_product_has_a_test():
    layers = _layer_rows("bf16")                     # (their logits: 256 action rows)
    assert {_head_form(M, 256) for M in range(1, 961)} <= {_head_form(M, 256) for M in layers}
    assert {_head_form(M, 32000) for M in range(1, 961)} <= {_head_form(M, 32000) for M in WIDE_HEAD}


@pytest.mark.parametrize("H,F", [(512, 1536), (1024, 2816)])
def test_8_bit_weights_split_along_k_as_far_as_bf16_weights(H, F):
    cfgs = [sv.model_cfg(dtype, H, H // 128, 128, F, 1024) for dtype in ("bf16", "bf16_w8")]
    for rows in range(129, 961):
        for which in LAYER:
            bf16, w8 = (sv.sv_product_plan(c, rows, which)[3] for c in cfgs)
            assert w8 >= bf16, (rows, which)


def test_half_of_the_rows_is_left_out_up_to_16_rows():
    """... and the query tells that kernel from gemm_skinny: without a test of its own, its forms have none."""
    for dtype in ("bf16", "bf16_w8", "bf16_w4"):
        for which in LAYER:
            kernels = [sv.sv_product_plan(_cfg(dtype), rows, which)[0] for rows in (1, 16, 17, 64)]
            assert kernels == [sv.SV_KERNEL_THIN] * 2 + [sv.SV_KERNEL_SKINNY] * 2, (dtype, which)
    assert _head_form(16, 256)[0] == _head_form(16, 32000)[0] == sv.SV_KERNEL_THIN


def test_heads_leave_rows_out_where_a_wave_has_four_steps():
    for H in (512, 1024, 2048, 4096):
        cfg = sv.model_cfg("bf16", H, H // 128, 128, 2816, 32000)
        for n in (256, 1024, 32000):
            kernel, _, _, slices, _, _ = sv.sv_product_plan(cfg, 16, sv.SV_PLAN_HEAD, n)
            assert (kernel == sv.SV_KERNEL_THIN) == (H // slices >= 4 * 4 * 32), (H, n)


def test_4_bit_weights_leave_rows_out_where_a_wave_has_two_steps():
    for H, F in ((512, 1536), (1024, 2816), (2048, 5632), (4096, 11008), (5120, 13824)):
        cfg = sv.model_cfg("bf16_w4", H, H // 128, 128, F, 1024)
        for which, K in zip(LAYER, (H, H, H, F)):
            kernel, _, _, slices, _, _ = sv.sv_product_plan(cfg, 16, which)
            assert (kernel == sv.SV_KERNEL_THIN) == (K // slices >= 2 * 4 * 64), (H, which)


@pytest.mark.parametrize("H,F,mid", [(512, 1536, ()), (2048, 5632, ()), (3072, 8192, (sv.SV_PLAN_GATE_UP,)),
                                     (4096, 11008, (sv.SV_PLAN_GATE_UP, sv.SV_PLAN_DOWN)), (5120, 13824, (sv.SV_PLAN_QKV, sv.SV_PLAN_GATE_UP)),
                                     (6144, 16384, (sv.SV_PLAN_QKV, sv.SV_PLAN_GATE_UP)), (8192, 28672, LAYER)])
def test_products_of_65_to_128_rows_on_the_kernel_that_was_faster(H, F, mid):
    cfg = sv.model_cfg("bf16", H, H // 128, 128, F, 1024)
    for rows in (65, 80, 96, 97, 112, 128):
        assert tuple(which for which in LAYER if sv.sv_product_plan(cfg, rows, which)[0] == sv.SV_KERNEL_MID) == mid, rows


def test_the_timed_cases_lie_in_the_range_that_is_tested():
    for case in cases.listed():
        rows = case["episodes"] * case["nodes"]
        assert case["model"] != "7b" or rows <= (960 if case["dtype"] == "bf16" else 640), case["name"]


@pytest.mark.parametrize("H,F", [(256, 65536), (512, 65536), (4096, 11008), (8192, 28672)])
def test_groups_that_share_sums_fit_the_counters(H, F):
    """A workspace holds counters of 4096 groups, an equal share for every XCD, whatever the sizes: no plan that
    splits along K has more."""
    cfg = sv.model_cfg("bf16", H, H // 128, 128, F, 32000)
    for n_xcd in range(1, 9):
        for rows in list(range(1, 1025, 31)) + list(range(1025, 32769, 401)):
            for which in LAYER + (sv.SV_PLAN_HEAD,):
                _, _, _, slices, groups, blocks = sv.sv_product_plan(cfg, rows, which, 32000, n_xcd)
                assert slices == 1 or groups * blocks <= 4096 // n_xcd, (n_xcd, rows, which)


@pytest.mark.parametrize("dtype,rows,label,mfma_bound", [
    ("bf16", 1, "gemm_thin (4 launches per layer: q/k/v, o, gate/up, down)", False), ("bf16", 60, "gemm_skinny (4 launches per layer: q/k/v, o, gate/up, down)", False),
    ("bf16", 128, "gemm_skinny, gemm_mid (4 launches per layer: q/k/v, o; gate/up, down)", False), ("bf16", 960, "gemm_mid (4 launches per layer: q/k/v, o, gate/up, down)", True)])
def test_the_benchmark_names_the_kernels_that_run(dtype, rows, label, mfma_bound):
    plans = {n: sv.sv_product_plan(_cfg(dtype), rows, which) for n, which in zip(("qkv", "o", "gate_up", "down"), LAYER)}
    assert bench.product_kernels(sv, plans) == (label, mfma_bound)


def test_plan_queries_check_their_arguments():
    bf, f32 = _cfg("bf16"), sv.model_cfg("f32", 256, 4, 64, 688, 512)
    assert sv.lib().sv_product_plan(bf, 60, 0, 0, 8, None) == sv.SV_ERR_NULL
    for args, status in (((f32, 60, 0), sv.SV_ERR_DTYPE), ((bf, 0, 0), sv.SV_ERR_SHAPE), ((bf, 1 << 16, 0), sv.SV_ERR_SHAPE),
                         ((bf, 60, 5), sv.SV_ERR_SHAPE), ((bf, 60, 4, 100), sv.SV_ERR_SHAPE), ((bf, 60, 0, 0, 9), sv.SV_ERR_SHAPE)):
        with pytest.raises(sv.SvError) as e:
            sv.sv_product_plan(*args)
        assert e.value.status == status, args
