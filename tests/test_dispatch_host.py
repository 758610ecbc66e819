"""CPU-only: which kernel a product goes to (launches.py)."""
from launches import launches


def test_negative_leading_dimensions_stay_off_the_pingpong_kernel(tmp_path):
    # its offsets within an operand panel are unsigned: rows stored backwards lie outside what they can reach
    big = dict(prec=1, M=4096, N=4096, K=1024)
    plain, back_a, back_b, zero = launches(tmp_path, [["gemm", big], ["gemm", dict(big, lda=-1024)],
                                                      ["gemm", dict(big, ldb=-1024)], ["gemm", dict(big, lda=0, ldb=0)]])
    for status, _ in (plain, back_a, back_b, zero):
        assert status == 0
    assert plain[1][0][0] == zero[1][0][0] == "gemm_bf16_pingpong_kernel"
    assert back_a[1][0][0] == back_b[1][0][0] == "gemm_bf16_w48s_kernel"
