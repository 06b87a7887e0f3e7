"""The weight-gradient kernel that keeps a panel of B in registers, at the edges of its k-steps, tiles and panels, against the
CPU oracle; tolerance as in test_gpu_gemm_kernels.py."""
import pytest

from kernel_choice import choice
from test_gpu_gemm_edges import run_rows
from test_gpu_gemm_kernels import spread


@pytest.mark.gpu
@pytest.mark.parametrize("E,rows,h,f", [
    (32, (32, 31, 0, 1, 17), 1088, 1216),                                   # one k-step; ragged row tile and panel
    (32, (64, 33, 0, 1, 63), 1088, 1216),                                   # two, panel beside the ring
    (32, (160, 129, 97, 96, 65, 64, 33, 128, 0), 1088, 1216),               # one to five k-steps in one launch
    (32, (256, 225, 224, 193, 192, 161, 160, 97, 0), 1024, 1536),           # six to eight: panel loaded in two parts
    (17, (160, 130, 0, 7), 1088, 2624),                                     # workgroups that do not divide by eight
])
def test_panel_kernel(orc, E, rows, h, f):
    k = choice().layer_gemms(E, max(rows), h, f)
    assert k["dw1"][0] == "panel" and k["dw2"][0] == "panel", k
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
