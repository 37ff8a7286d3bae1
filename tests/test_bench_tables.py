"""CPU: how the benchmark and the counter probe read the library's launches."""
import bench


def test_attention_core_backward_as_one_launch_or_two():
    kern = {"attn_qkv": 9.0, "attn_core_fwd": 1.0, "attn_dout": 5.0}
    assert bench.attention_core_ms({**kern, "attn_core_bwd_dq": 2.0, "attn_core_bwd_dkv": 3.0}) == (1.0, 5.0)
    assert bench.attention_core_ms({**kern, "attn_core_bwd": 4.0}) == (1.0, 4.0)
