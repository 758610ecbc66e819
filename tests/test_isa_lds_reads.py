"""CPU-only: in the code built for gfx950, no LDS buffer is handed over while a wave may still be reading it."""
import pytest

import isa_util


# The rings refill a stage after the one barrier that follows its reads: every read has to be waited for before it.  The
# ping-pong kernel reads before the swap that opens its products and has to wait before the one that closes them: the
# buffer may be requested again from the second barrier after that on, by a wave that is half a phase ahead.
@pytest.mark.parametrize("family,allowed", [("gemm_bf16_pingpong_kernel", 1), ("gemm_bf16_w48", 0),
                                            ("gemm_bf16_spec_kernel", 0), ("gemm_bf16_pipe_kernel", 0),
                                            ("gemm_f32_", 0)])
def test_lds_reads_return_before_their_buffer_is_handed_over(tmp_path, family, allowed):
    found = isa_util.kernels(tmp_path, family)
    assert found, family
    for name, code in found.items():
        assert isa_util.barriers_crossed_by_lds_reads(code) <= allowed, name
