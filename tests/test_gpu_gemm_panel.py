"""The weight-gradient kernel that keeps a panel of B in registers, at the edges of its k-steps, tiles and panels, against the
CPU oracle; tolerance as in test_gpu_gemm_kernels.py."""
import pytest

from kernel_choice import choice
from test_gpu_gemm_edges import run_rows
from test_gpu_gemm_kernels import spread


def longest(E, C, M, N):
    """Row tiles of a launch's longest workgroup"""
    mt, run = -(-M // 128), choice().gemm_panel_run(E, M, N, C)
    return -(-mt // -(-mt // run))


def stages(rows):
    """Tiles in the ring of an expert with so many rows"""
    return min(4, 16 // max(1, -(-rows // 32)))


@pytest.mark.gpu
@pytest.mark.parametrize("E,rows,h,f,reused", [
    # reused: row counts whose workgroups take more tiles than the ring has stages, in one of the gradients, so that the wait
    # that counts stores is reached and a stage is filled twice (at most 64 rows in the launch: at most four tiles)
    (32, (32, 31, 0, 1, 17), 1088, 1216, ()),                               # one k-step; ragged row tile and panel
    (32, (64, 33, 0, 1, 63), 1088, 1216, ()),                               # two, panel beside the ring
    (16, (64, 33, 0, 1, 63, 32, 31, 16), 4096, 1024, ()),                   # four tiles: the last one's wait counts stores
    (32, (160, 129, 97, 96, 65, 64, 33, 128, 0), 1088, 1216, ()),           # one to five k-steps in one launch, two tiles
    (40, (160, 129, 97, 96, 65, 64, 33, 128, 0), 1088, 1216, (160, 128, 96, 64, 1)),             # the same, five tiles
    (32, (256, 225, 224, 193, 192, 161, 160, 97, 0), 1024, 1536, (256, 224, 192, 160)),          # six to eight: panel loaded in two parts
    (17, (160, 130, 0, 7), 1088, 2624, (160,)),                             # workgroups that do not divide by eight
    (20, (160, 128, 97, 96, 65, 64, 33, 129, 0, 1, 31, 32), 1088, 2624, (160, 128, 96, 64, 32)),
])
def test_panel_kernel(orc, E, rows, h, f, reused):
    k = choice().layer_gemms(E, max(rows), h, f)
    assert k["dw1"][0] == "panel" and k["dw2"][0] == "panel", k
    tiles = max(longest(E, max(rows), h, f), longest(E, max(rows), f, h))
    assert all(tiles > stages(n) for n in reused) and (reused or tiles <= 4), tiles
    if h == 4096:
        assert tiles == 4
    run_rows(orc, spread(E, rows) if max(rows) > 40 else rows + tuple(n % 32 for n in range(E - len(rows))), h, f, per_expert=True)


def test_rule_of_the_panel_kernel():
    r = choice()
    assert r.gemm_panel_chosen(16, 2048, 8192, 256) and not r.gemm_panel_chosen(16, 2048, 8192, 257)
    assert r.gemm_panel_chosen(8, 2048, 2048, 100) and not r.gemm_panel_chosen(7, 2048, 2048, 100)
    assert not r.gemm_panel_chosen(256, 2048, 1016, 100)
    for E in (1, 3, 16, 256):
        for M in (1024, 1032, 5144, 8192):
            for N in (1024, 1088, 8192):
                for K in (1, 64, 65, 160, 161, 256):
                    assert 1 <= r.gemm_panel_run(E, M, N, K) <= (4 if K <= 64 else 8 if K <= 160 else 16)
    assert r.gemm_panel_fills(16, 2048, 8192, 160) and not r.gemm_panel_fills(16, 2560, 5120, 125)


@pytest.mark.parametrize("E,M,N,slower,faster", [
    # the panel would be loaded for every tile
    (4, 2880, 5248, (16, 40, 64), (100, 144)), (4, 3136, 4864, (16, 40, 64), (100, 144)), (16, 2688, 1088, (40, 64), (100,)),
    # the other gradient's rows are parts of lines: few experts and results, many
    (16, 2256, 1280, (16, 64, 144), (161, 200)), (4, 1616, 5440, (16, 40, 64, 144), (200,)),
    (32, 1200, 1984, (), (16, 64, 144)), (32, 920, 1216, (), (16, 64, 130)), (16, 3000, 1600, (), (6, 64, 160)),
    # 65 to 160 rows of few experts: few results, many, and a whole round
    (8, 1536, 2752, (100, 144), (16, 64, 161)), (4, 2624, 3904, (100, 130, 150), (64, 200)), (2, 4544, 4928, (100, 150), ()),
    (8, 2816, 2112, (), (100, 150)), (16, 1472, 1472, (), (100, 150)), (4, 2048, 4096, (), (100, 160)),
    (8, 2048, 2048, (), (6, 64, 160)), (64, 1024, 1024, (), (6, 64, 128))])
def test_sizes_at_which_the_panel_kernel_was_measured(E, M, N, slower, faster):
    """Row counts at which it was slower and faster than the kernel that serves otherwise"""
    assert not any(choice().gemm_panel_chosen(E, M, N, k) for k in slower)
    assert all(choice().gemm_panel_chosen(E, M, N, k) for k in faster)
