"""The large grouped GEMM where few experts hold rows, so that its plan cuts them into low tiles: against the CPU oracle, tolerance
as in test_gpu_gemm_kernels.py, and the folded permutations bit for bit against the separate ones."""
import numpy as np
import pytest
import torch

from kernel_choice import choice
from gpu_util import DevInputs, host, make_layer
from paper_2303_06318_amd import synth
from test_gpu_gemm_edges import W, route_rows, run_rows

pytestmark = pytest.mark.gpu

CASES = [
    # experts; rows of the first; widths
    (64, (300, 288, 256, 161, 129, 128, 7), 264, 1032),       # heavy, light and tall ones by the usual plan
    (64, (0, 0, 257, 0, 31, 256), 520, 1288),                 # one block more than two low tiles
    (40, (0,) * 39 + (520,), 328, 1600),                      # one expert, the last, in five low tiles
    (100, (300, 0, 161, 96) + (0,) * 90 + (257, 33, 288, 0, 129, 1), 264, 1032),       # more than a wave of experts
]


@pytest.mark.parametrize("E,rows,h,f", CASES)
def test_low_tiles(orc, E, rows, h, f):
    k = choice().layer_gemms(E, max(rows), h, f)
    assert all(k[g] == "large" for g in ("fwd1", "fwd2", "dh", "dd")), k
    rows = rows + (0,) * (E - len(rows))
    assert choice().low_tiles(rows, h) and choice().low_tiles(rows, f)
    run_rows(orc, rows, h, f, per_expert=True)


def test_a_list_that_an_xcd_would_not_finish_in_one_round(orc):
    """245 low tiles and 10 light ones are fewer than the compute units, but one XCD would have 31 and 2 of them for its 32: the
    first GEMM keeps the usual tiles, the second (98 and 4) does not."""
    rows = (300,) + (161,) * 23 + (7, 128) + (0,) * 38
    k = choice().layer_gemms(64, 300, 264, 1032)
    assert all(k[g] == "large" for g in ("fwd1", "fwd2", "dh", "dd")), k
    assert not choice().low_tiles(rows, 1032) and choice().low_tiles(rows, 264)
    run_rows(orc, rows, 264, 1032, per_expert=True)


@pytest.mark.parametrize("E,rows,h,f", [CASES[0], CASES[3]])
def test_folded_permutations_on_low_tiles(E, rows, h, f):
    rows = rows + (0,) * (E - len(rows))
    T = sum(rows)
    wl = synth.scaled(W, T=T, h=h, f=f, E=E, capacity_factor=max(rows) * E / T, seed=5)
    dev = DevInputs(synth.make_inputs(wl))
    a, b = make_layer(wl, backward=False), make_layer(wl, backward=False)
    logits = torch.from_numpy(route_rows(a, rows, 7)).cuda()
    a.forward(dev.x, dev.wg, dev.w1, dev.w2, logits_in=logits)
    b.forward(dev.x, dev.wg, dev.w1, dev.w2, logits_in=logits, fused=True)
    torch.cuda.synchronize()
    assert choice().low_tiles(rows, h) and choice().low_tiles(rows, f)
    assert np.array_equal(host(a.out).view(np.uint32), host(b.out).view(np.uint32))
