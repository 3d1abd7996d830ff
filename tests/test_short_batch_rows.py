"""Row tiles per workgroup of short batches: 2 or 4 while an eighth of the 256 CUs would have no workgroup, 8 from there on; with
one or two segments the line is at 48 workgroups of 8."""
import pytest

import paper_2306_16601_amd as sp
import workloads as wl

# (N, K, M, rows per workgroup): 16-token tiles; last token count on one side of a line, first one on the other
LINES = [
    (512, 1100, 224, 32), (512, 1100, 225, 64), (512, 1100, 448, 64), (512, 1100, 449, 128),        # 3 segments: 224 workgroups
    (1023, 1100, 224, 64), (1023, 1100, 225, 128),
    (512, 1024, 176, 32), (512, 1024, 177, 128),                                                     # 2
    (640, 2048, 160, 32), (640, 2048, 161, 64),                                                      # 4
    (512, 512, 176, 32), (512, 512, 177, 128),                                                       # 1
]


def _case(N, K, M, out_type="s8", postop="none"):
    return wl.Case("rows", N, K, M, 0.7, wl.N4K1, out_type, postop, keys=(120, N, K, M))


@pytest.mark.parametrize("N,K,M,rows", LINES)
def test_rows_per_workgroup_on_both_sides_of_the_lines(N, K, M, rows):
    h = sp.spmm_pack_host(wl.make(_case(N, K, M))["W"])
    try:
        for out_type in ("s8", "f32"):
            token_tile, here, workgroups = sp.spmm_plan(h, M, out_type)
            assert (token_tile, here) == (16, rows)
            if rows < 128:
                assert workgroups <= 224
    finally:
        sp.spmm_destroy(h)


@pytest.mark.gpu
@pytest.mark.parametrize("out_type,postop", [("s32", "none"), ("f32", "gelu"), ("u8", "gelu")])
@pytest.mark.parametrize("N,K,M,rows", LINES)
def test_both_sides_of_the_lines_match_the_oracle(N, K, M, rows, out_type, postop):
    from test_gpu_parity import check_case
    check_case(_case(N, K, M, out_type, postop))
