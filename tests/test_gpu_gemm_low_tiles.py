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
    # 64 experts; column tiles of GEMM1 and GEMM2; blocks of 32 rows per expert
    (64, (300, 288, 256, 161, 129, 128, 7), 264, 1032),       # heavy, light and tall ones by the usual plan
    (64, (0, 0, 257, 0, 31, 256), 520, 1288),                 # one block more than two low tiles
    (40, (0,) * 39 + (520,), 328, 1600),                      # one expert, the last, in five low tiles
]


@pytest.mark.parametrize("E,rows,h,f", CASES)
def test_low_tiles(orc, E, rows, h, f):
    k = choice().layer_gemms(E, max(rows), h, f)
    assert all(k[g] == "large" for g in ("fwd1", "fwd2", "dh", "dd")), k
    run_rows(orc, rows + (0,) * (E - len(rows)), h, f, per_expert=True)


@pytest.mark.parametrize("E,rows,h,f", CASES[:1])
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
    assert np.array_equal(host(a.out).view(np.uint32), host(b.out).view(np.uint32))
