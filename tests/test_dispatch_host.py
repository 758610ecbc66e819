"""CPU-only: which kernel a product goes to (launches.py)."""
import pytest

from gemm_shapes import F32_GROUPS, PP, SHAPES
from launches import launches


def layer_cfg(heads, ffn, precision=0):
    return dict(batch=1, seq=32, hidden=64 * heads, heads=heads, ffn=ffn, pre_ln=0, causal=0, gelu_tanh=0,
                precision=precision, ln_eps=1e-5, dropout_p=0.1, seed=1, layer_id=0)


@pytest.mark.parametrize("epilogue", [1, 4, 5, 6])
def test_shapes_reach_the_kernels_they_are_listed_for(tmp_path, epilogue):
    got = launches(tmp_path, [["gemm", dict(prec=1, M=M, N=N, K=K, epi=epilogue)] for M, N, K, _, _ in SHAPES])
    for (M, N, K, kernel, args), (status, found) in zip(SHAPES, got):
        assert status == 0 and [f[0] for f in found] == [kernel] and found[0][1][:len(args)] == args, (M, N, K, found)
        assert found[0][1][-1] == (1 if K % 64 else 0), (M, N, K, found)   # last argument: half a k-step at the end


def test_every_gemm_kernel_of_the_library_is_listed(tmp_path):
    import isa_util
    listed = {(k, a, bool(K % 64)) for _, _, K, k, a in SHAPES}
    for family, length in ((SHAPES[0][3], 2), ("gemm_bf16_w48s_kernel", 3), ("gemm_bf16_w48_kernel", 2), (PP, 4)):
        built = isa_util.kernels(tmp_path, family)
        assert len(built) == len([x for x in listed if x[0] == family]), (family, sorted(built))


def test_float32_layers_reach_the_group_tiles_they_are_listed_for(tmp_path):
    got = launches(tmp_path, [["layer_bwd", layer_cfg(h, f)] for h, f, _ in F32_GROUPS])
    for (heads, ffn, tile), (status, found) in zip(F32_GROUPS, got):
        group = [f[1] for f in found if f[0] == "gemm_f32_group_kernel"]
        assert status == 0 and len(group) == 1, (heads, ffn, found)
        wgm, wgn, mb, nb = group[0][:4]
        assert (16 * wgm * mb, 16 * wgn * nb) == tile, (heads, ffn, group)


def test_f32_shapes_of_the_value_tests_take_every_tile(tmp_path):
    shapes = [(992, 3040), (992, 2272), (992, 1504), (992, 992), (992, 736), (32, 64)]
    got = launches(tmp_path, [["gemm", dict(prec=0, M=M, N=N, K=96, f32=1)] for M, N in shapes])
    tiles = [(16 * k[0][1][0] * k[0][1][2], 16 * k[0][1][1] * k[0][1][3]) for _, k in got]
    assert tiles == [(64, 192), (64, 144), (64, 96), (64, 64), (64, 48), (32, 32)]


def test_negative_leading_dimensions_stay_off_the_pingpong_kernel(tmp_path):
    # its offsets within an operand panel are unsigned: rows stored backwards lie outside what they can reach
    big = dict(prec=1, M=4096, N=4096, K=1024)
    plain, back_a, back_b, zero = launches(tmp_path, [["gemm", big], ["gemm", dict(big, lda=-1024)],
                                                      ["gemm", dict(big, ldb=-1024)], ["gemm", dict(big, lda=0, ldb=0)]])
    for status, _ in (plain, back_a, back_b, zero):
        assert status == 0
    assert plain[1][0][0] == zero[1][0][0] == "gemm_bf16_pingpong_kernel"
    assert back_a[1][0][0] == back_b[1][0][0] == "gemm_bf16_w48s_kernel"


def test_rows_far_apart_stay_on_the_ring(tmp_path):
    got = launches(tmp_path, [["gemm", dict(prec=1, M=224, N=49152, K=K, lda=(1 << 20) + 8)] for K in (32, 96, 192)])
    assert [k[0][0] for _, k in got] == ["gemm_bf16_w48_kernel"] * 3


def test_products_run_where_the_lds_limit_cannot_be_raised(tmp_path):
    # as before the kernels with more than 64 KiB: no product is refused, each goes to a kernel that needs no raised limit
    f32 = [dict(prec=0, M=M, N=N, K=96, ak=ak, bk=bk, f32=1) for M, N in ((992, 3040), (992, 2272), (992, 1504), (32, 64))
           for ak, bk in ((1, 1), (1, 0), (0, 0), (0, 1))]
    bf16 = [dict(prec=1, M=4096, N=3072, K=768), dict(prec=1, M=64, N=768, K=3072), dict(prec=1, M=1824, N=768, K=3072),
            dict(prec=1, M=4096, N=3072, K=32), dict(prec=1, M=768, N=3072, K=4096, ak=0, bk=0, f32=1)]
    layers = [layer_cfg(h, f) for h, f in ((2, 512), (8, 2048), (8, 1504), (4, 3616))]
    calls = [["gemm", g] for g in f32 + bf16] + [["layer_bwd", c] for c in layers]
    raised, unraised = launches(tmp_path, calls), launches(tmp_path, calls, lds_limit_fails=True)
    for call, (status, kernels) in zip(calls, unraised):
        assert status == 0 and kernels, call
    for family in ("gemm_f32_kernel", "gemm_f32_group_kernel"):   # both tiles of more than 64 KiB are among the calls
        assert {k[1][:6] for _, ks in raised for k in ks if k[0] == family} >= {(2, 2, 2, 6, 2, 3), (2, 1, 2, 9, 4, 2)}
    assert {k[1][:6] for _, ks in unraised for k in ks if k[0] in ("gemm_f32_kernel", "gemm_f32_group_kernel")} <= {
        (2, 2, 2, 3, 2, 3), (2, 2, 2, 2, 2, 3), (2, 1, 2, 3, 4, 2), (1, 1, 2, 2, 8, 2)}
    assert {k[0] for _, ks in unraised[len(f32):len(f32) + len(bf16)] for k in ks} <= {"gemm_bf16_kernel", "gemm_bf16_split_kernel"}


def test_short_single_weight_gradients_take_the_staged_kernel(tmp_path):
    shapes = [(576, 768, 128), (4352, 352, 512), (128, 128, 32), (4352, 352, 544), (5248, 832, 384)]
    got = launches(tmp_path, [["gemm", dict(prec=1, M=M, N=N, K=K, ak=0, bk=0, f32=1)] for M, N, K in shapes])
    assert [(s, len(k), k[0][0]) for s, k in got] == [(0, 1, "gemm_bf16_kernel")] * 3 + [(0, 1, "gemm_bf16_spec_kernel")] * 2


def test_64_columns_of_a_short_contraction_take_the_three_stage_ring(tmp_path):
    ring = [dict(prec=1, M=M, N=64, K=K, ak=0, bk=0) for M in (128, 65536) for K in (64, 128)]
    staged = [dict(prec=1, M=160, N=64, K=64, ak=0, bk=0), dict(prec=1, M=128, N=64, K=96, ak=0, bk=0),
              dict(prec=1, M=128, N=64, K=192, ak=0, bk=0), dict(prec=1, M=128, N=64, K=64, ak=1, bk=0)]
    got = launches(tmp_path, [["gemm", g] for g in ring + staged])
    assert [k[0][0] for _, k in got] == ["gemm_bf16_pipe_kernel"] * 4 + ["gemm_bf16_kernel"] * 4


def test_products_of_one_wide_round_or_more_stay_on_the_staged_kernel_where_it_wins(tmp_path):
    split, ring, pp, staged = "gemm_bf16_split_kernel", "gemm_bf16_w48s_kernel", "gemm_bf16_pingpong_kernel", "gemm_bf16_kernel"
    want = [((32, 16384, 128, 1), split), ((16384, 32, 128, 1), split),                 # one round of split tiles
            ((32, 16480, 128, 1), staged), ((20480, 32, 192, 1), staged), ((32, 32768, 256, 1), ring),
            ((45056, 32, 512, 1), staged), ((36000, 32, 1024, 1), pp), ((32, 131072, 2048, 1), staged),
            ((64, 24576, 64, 1), ring), ((64, 24576, 64, 0), staged), ((64, 24576, 192, 0), ring),
            ((57344, 64, 64, 1), staged), ((57344, 64, 128, 1), pp), ((98304, 64, 256, 1), staged),
            ((64, 131072, 128, 1), staged), ((64, 50272, 512, 0), staged), ((64, 50272, 512, 1), ring),
            ((96, 65536, 32, 1), staged), ((96, 65536, 128, 4), pp),
            ((39616, 3840, 32, 0), staged), ((39616, 3840, 32, 4), ring), ((39616, 3840, 64, 0), ring), ((2016, 1952, 32, 1), ring)]
    got = launches(tmp_path, [["gemm", dict(prec=1, M=M, N=N, K=K, epi=e)] for (M, N, K, e), _ in want])
    for (shape, kernel), (status, found) in zip(want, got):
        assert status == 0 and found[0][0] == kernel, (shape, found)
