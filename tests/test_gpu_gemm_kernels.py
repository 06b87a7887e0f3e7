"""Every grouped bf16 GEMM kernel at the edges of its tiles, against the CPU oracle.  Each case names the kernel that its
GEMMs are meant to reach and checks that against the host rules, so that a change of a rule cannot empty it.  Tolerance as in
test_gpu_gemm_edges.py: 2e-2 per row and tile plus the element bound, the weight gradients expert by expert."""
import numpy as np
import pytest
import torch

from paper_2303_06318_amd import moe, synth
from paper_2303_06318_amd.layer import MoeLayer
from gpu_util import DevInputs, host, make_layer
from kernel_choice import choice
from test_gpu_gemm_edges import W, route_rows, run_rows

pytestmark = pytest.mark.gpu


def spread(E, rows):
    """E row counts: the given ones first, then a repetition of handfuls (cheap for the oracle)."""
    few = (3, 0, 17, 1, 40, 8, 0, 33)
    return tuple(rows) + tuple(few[i % len(few)] for i in range(E - len(rows)))


LARGE = [
    # E, rows of the first experts, h, f.  256 experts of one column tile: the large kernel from 161 rows on
    (256, (161, 192, 224, 225, 256, 128, 160, 129), 8, 72),            # five to eight blocks, light tiles; one short k-tile, two
    (256, (257, 288, 256, 283, 96, 161, 130), 64, 128),                # tall tiles, the second one full; whole k-tiles
    (256, (289, 320, 300, 352, 384, 400, 161), 72, 136),               # two tiles: five and five blocks to seven and six
    (256, (545, 576, 512, 513, 450, 31), 136, 192),                    # two tall tiles; eight and nine blocks; odd and even k-tiles
    (256, (800, 161, 177), 200, 264),                                  # nine, eight and eight blocks; a second column tile of 8
    (64, (170, 161, 190, 64, 150), 520, 776),                          # ragged column tiles, many k-tiles; low tiles in GEMM2 and dD; weight gradients too
    (128, (170, 161, 190, 64, 150), 520, 776),                         # the same without low tiles
]


@pytest.mark.parametrize("act", [moe.MOE_GELU_ERF, moe.MOE_GELU_TANH])
@pytest.mark.parametrize("E,rows,h,f", LARGE)
def test_large_kernel(orc, E, rows, h, f, act):
    k = choice().layer_gemms(E, max(rows), h, f)
    assert all(k[g] == "large" for g in ("fwd1", "fwd2", "dh", "dd")), k
    if E <= 128:
        assert k["dw1"] == "large" and k["dw2"] == "large", k
    rows = spread(E, rows)
    assert not choice().low_tiles(rows, f) and choice().low_tiles(rows, h) == (E == 64)
    run_rows(orc, rows, h, f, act, per_expert=True)


@pytest.mark.parametrize("E,rows,h,f,kernels", [
    # five 32-row blocks, two workgroups per compute unit (more than 256 tiles); one workgroup
    (64, (145, 160, 0, 7, 129, 33, 96, 128), 648, 712, {"fwd1": ("rows", 5, False), "dh": ("rows", 5, False), "fwd2": ("rows", 5, False)}),
    (16, (145, 160, 0, 7, 129, 33, 96, 128), 136, 648, {"fwd1": ("rows", 5, True), "dd": ("rows", 5, True)}),
    # one block: paced ring (one k-tile, fewer and more than the ring, odd), full ring, backward
    (64, (32, 17, 1, 0, 16, 31), 40, 512, {"fwd1": ("rows", 1, True), "fwd2": ("rows", 1, False), "dh": ("rows", 1, False)}),
    (56, (32, 17, 1, 0, 16, 31), 456, 504, {"fwd1": ("rows", 1, True), "fwd2": ("rows", 1, True), "dd": ("rows", 1, False)}),
    (32, (30, 17, 1, 0, 16, 31), 136, 1032, {"fwd1": ("rows", 1, False), "fwd2": ("rows", 1, False)}),
    # two and four blocks, both forms
    (64, (64, 33, 0, 17), 136, 648, {"fwd1": ("rows", 2, False), "fwd2": ("rows", 2, True)}),
    (64, (128, 65, 0, 17, 97), 136, 648, {"fwd1": ("rows", 4, False), "fwd2": ("rows", 4, True)}),
    # weight gradients in runs of tiles: whole lines, runs of four and one, and of two; one k-tile and two, and none
    (256, (64, 33, 0, 100, 128, 1, 65), 256, 640, {"dw1": ("wgrad", True, 4, 1), "dw2": ("wgrad", True, 2, 2)}),
    (256, (160, 33, 0, 100, 128, 129, 65), 256, 640, {"dw1": ("wgrad", True, 4, 1), "dw2": ("wgrad", True, 2, 2)}),
    # parts of lines, runs of two whose last tile is ragged; three k-tiles and more
    (256, (161, 33, 0, 100, 400, 129, 65), 248, 504, {"dw1": ("wgrad", False, 2, 2), "dw2": ("wgrad", False, 2, 2)}),
])
def test_few_row_kernels(orc, E, rows, h, f, kernels):
    k = choice().layer_gemms(E, max(rows), h, f)
    assert {g: k[g] for g in kernels} == kernels, k
    few = tuple(r if r <= max(rows) else 1 for r in spread(E, rows))
    run_rows(orc, few, h, f, per_expert=True)


@pytest.mark.parametrize("E,rows,h,f", [
    (256, (161, 288, 0, 300, 256, 130), 136, 72), (64, (170, 161, 190, 64, 0, 150), 520, 776), (128, (170, 161, 190, 64, 0, 150), 520, 776)])
def test_folded_permutations_on_the_large_kernel(E, rows, h, f):
    """Dispatch read through the index by the first GEMM and combine written by the second, on the large kernel's light,
    partial, full and tall tiles: the same bits as the separate passes."""
    rows = spread(E, rows)
    k = choice().layer_gemms(E, max(rows), h, f)
    assert k["fwd1"] == "large" and k["fwd2"] == "large", k
    T = sum(rows)
    wl = synth.scaled(W, T=T, h=h, f=f, E=E, capacity_factor=max(rows) * E / T, seed=5)
    dev = DevInputs(synth.make_inputs(wl))
    for backward in (False, True):             # rows gathered from x; dispatched rows, y written as well
        a, b = make_layer(wl, backward=backward), make_layer(wl, backward=backward)
        logits = torch.from_numpy(route_rows(a, rows, 7)).cuda()
        a.forward(dev.x, dev.wg, dev.w1, dev.w2, logits_in=logits)
        b.forward(dev.x, dev.wg, dev.w1, dev.w2, logits_in=logits, fused=True)
        torch.cuda.synchronize()
        assert host(a.kept).tolist() == list(rows)
        assert np.array_equal(host(a.out).view(np.uint32), host(b.out).view(np.uint32))
        ha, hb = host(a.hact), host(b.hact)
        for e, n in enumerate(rows):
            assert np.array_equal(ha[e, :n].view(np.uint32), hb[e, :n].view(np.uint32)), e
