"""CPU: how the benchmark and the counter probe read the library's launches."""
import bench
from paper_2507_09029_amd.traffic_probe import kernel_site


def test_attention_core_backward_as_one_launch_or_two():
    kern = {"attn_qkv": 9.0, "attn_core_fwd": 1.0, "attn_dout": 5.0}
    assert bench.attention_core_ms({**kern, "attn_core_bwd_dq": 2.0, "attn_core_bwd_dkv": 3.0}) == (1.0, 5.0)
    assert bench.attention_core_ms({**kern, "attn_core_bwd": 4.0}) == (1.0, 4.0)


def test_transposes_are_told_of_only_where_a_launch_carries_them():
    big = {"mlp_gate_up": "256x256", "mlp_down": "256x256", "mlp_dact": "128x256", "mlp_dx": "256x256", "mlp_dw": "128x256"}
    assert bench.carries("mlp_gate_up", big) == "mlp_wt_fwd" and bench.carries("mlp_dact", big).startswith("mlp_tr_bwd")
    assert bench.carries("mlp_gate_up", {**big, "mlp_wt_fwd": None}) is None and bench.carries("mlp_dw", big) is None
    small = {"mlp_gate_up": "64x64", "mlp_down": "64x64", "mlp_dact": "64x64", "mlp_dx_dw": None}  # both read the weights as stored
    assert bench.carries("mlp_gate_up", small) is None and bench.carries("mlp_dact", small) is None


def test_counter_probe_knows_the_launches():
    assert kernel_site("void (anonymous namespace)::sdp_gemm_kernel<256, 256, 2, 4, 2, 0, 0>(Dev, SideArg)") == "mlp_gate_up"
    assert kernel_site("void (anonymous namespace)::sdp_gemm_pair_kernel<64, 128, 1, 6, 3>(Dev, Dev, int)") == "mlp_dx_dw"
    assert kernel_site("void (anonymous namespace)::sdp_gemm_pair_kernel<64, 64, 0, 6, 3>(Dev, Dev, int)") is None  # an attention's
    assert kernel_site("void (anonymous namespace)::avg_groups_kernel<1, 0, 0>(GradPtrs)") == "coverage_grad_avg"
    assert kernel_site("void (anonymous namespace)::avg_groups_kernel<1, 2, 0>(GradPtrs)") is None
