"""The grouped bf16 GEMMs of small layers at the edges of their tiles, against the CPU oracle: reduction lengths around the
64-deep k-tile (h and f for the forward and data gradients, the kept rows for the weight gradients), row counts
around the 32-row block and its multiples, output widths around 128 and 256 columns.  Layers as small as these run
on the few-row kernels (the last case's weight gradients on the large one); test_gpu_gemm_kernels.py names the kernel
that each of its cases reaches.  Tolerance: bf16 storage with fp32
accumulation, 2e-2 per row and tile like every other parity test, plus the element bound of gpu_util."""
import numpy as np
import pytest
import torch

from paper_2303_06318_amd import moe, synth
from gpu_util import DevInputs, assert_close_everywhere, host, make_layer, tol
from kernel_choice import choice

pytestmark = pytest.mark.gpu

W = synth.WORKLOADS["cfg5_6p7b_tp4_fwdbwd"]


def route_rows(layer, rows, seed):
    """Routing of exactly rows[e] tokens to expert e, in a shuffled order, through moe_gate on given logits."""
    e = np.repeat(np.arange(len(rows)), rows)
    np.random.default_rng(seed).shuffle(e)
    logits = np.zeros((len(e), len(rows)), np.float32)
    logits[np.arange(len(e)), e] = 1.5
    layer.gate(None, None, logits_in=torch.from_numpy(logits).cuda())
    return logits


def run_rows(orc, rows, h, f, act=moe.MOE_GELU_ERF, seed=11, dtype="bf16", per_expert=False, few=False):
    """per_expert: the weight gradients are compared expert by expert.  The element bound is a share of the compared
    array's rms; an expert's gradient sums over its own n rows, so its values and its rounding errors grow with the root of
    n, and beside 288 rows the rms of a tensor of mostly 3-row experts is four times too small a measure.  For few rows the
    share has a term of its own: an element's error is at most 2^-8 of its terms (both factors are rounded to bf16), the
    largest of 10^5 products of two normal factors is 25 times a term's rms, and the gradient's rms is sqrt(n) times that,
    so one large term moves its element by up to 25 x 2^-8 / sqrt(n), a tenth of the rms over sqrt(n).
    few: some experts hold so few rows that a row of d_w2, hact's column times d_y, may be next to zero where a single hact is,
    and its own norm measures nothing: d_w2 is compared expert by expert, a row's error against the expert's rms row norm."""
    T, E = int(sum(rows)), len(rows)
    wl = synth.scaled(W, T=T, h=h, f=f, E=E, capacity_factor=max(rows) * E / T, seed=seed, dtype=dtype)
    inp = synth.make_inputs(wl)
    dev = DevInputs(inp)
    layer = make_layer(wl, backward=True, act=act)
    logits = route_rows(layer, rows, seed)
    moe.moe_dispatch(layer.shape, dev.x, layer.token_of_slot, layer.buf)
    moe.moe_expert_ffn_fwd(layer.shape, layer.buf, dev.w1, dev.w2, layer.kept, layer.z_save, layer.hact, layer.y, layer.ws)
    moe.moe_combine(layer.shape, layer.y, layer.expert, layer.slot, layer.gate_p, layer.out)
    layer.backward(dev.d_out, dev.x, dev.wg, dev.w1, dev.w2)
    torch.cuda.synchronize()
    assert host(layer.kept).tolist() == list(rows)
    fw = orc.layer_forward(inp.x, inp.wg, inp.w1, inp.w2, wl.C, mode=act, logits=logits)
    bw = orc.layer_backward(fw, inp.d_out, inp.x, inp.wg, inp.w1, inp.w2, mode=act)
    t = tol(wl)
    hact, y, d_buf = host(layer.hact), host(layer.y), host(layer.d_buf)
    for e, k in enumerate(rows):
        if k:
            assert_close_everywhere("hact", hact[e, :k], fw["H"][e, :k], t)
            assert_close_everywhere("y", y[e, :k], fw["Y"][e, :k], t)
            assert_close_everywhere("d_buf", d_buf[e, :k], bw["dD"][e, :k], t)
    d_w1, d_w2 = host(layer.d_w1), host(layer.d_w2)
    if per_expert:
        for e, k in enumerate(rows):
            if k:
                assert_close_everywhere("d_w1", d_w1[e], bw["dW1"][e], t, elem_rms=0.03 + 0.1 / k ** 0.5)
                assert_close_everywhere("d_w2", d_w2[e], bw["dW2"][e], t, elem_rms=0.03 + 0.1 / k ** 0.5)
    else:
        assert_close_everywhere("d_w1", d_w1, bw["dW1"], t)
        if few:
            for e, k in enumerate(rows):
                if k:
                    assert_close_everywhere("d_w2", d_w2[e], bw["dW2"][e], t, rows_relative=False)
        else:
            assert_close_everywhere("d_w2", d_w2, bw["dW2"], t)
    for e, k in enumerate(rows):
        if k == 0:
            assert not d_w1[e].any() and not d_w2[e].any()


@pytest.mark.parametrize("rows,h,f", [
    ((1, 0, 33), 8, 8),                 # one short k-tile everywhere
    ((63, 65), 56, 72),                 # just below and above one k-tile
    ((64, 128), 64, 128),               # whole k-tiles, odd and even counts
    ((129, 191, 0), 120, 200),          # five and six 32-row blocks
    ((193, 256), 136, 264),             # seven and eight blocks; eight columns more than two tiles
    ((257, 288), 248, 256),             # nine blocks in tiles of three
    ((289, 576, 5), 264, 520),          # ten and eighteen blocks, a handful of rows
    ((16, 3, 17, 32), 136, 264),        # few rows: one 32-row block, half of it empty or full
    ((33, 64, 0, 48), 192, 128),        # two blocks; three k-tiles for a ring of three
    ((145, 160, 160, 7), 264, 200),     # five blocks
    ((161, 240, 225, 31), 72, 520),     # six to eight blocks
    ((9, 0, 65, 20, 1, 64, 33, 2), 2056, 2064),  # weight gradients of parts of lines and many tiles: the large kernel
])
@pytest.mark.parametrize("act", [moe.MOE_GELU_ERF, moe.MOE_GELU_TANH])
def test_tile_edges(orc, rows, h, f, act):
    run_rows(orc, rows, h, f, act)


@pytest.mark.parametrize("rows,h,f", [
    ((1, 0, 5), 4, 4),                  # narrow tiles (32 x 32, k-tiles of 128): a few values of one tile
    ((31, 33, 127), 124, 132),          # around the tile and the k-tile
    ((128, 129, 2), 128, 260),          # whole k-tiles and one row more
    ((63, 65, 0, 97) * 8, 260, 252),    # wide tiles (64 x 64, k-tiles of 32) in the weight gradients, narrow ones before
    ((64, 96) * 16, 256, 324),          # the same; the block form in GEMM2 and dD
])
def test_tile_edges_f32(orc, rows, h, f):
    """fp32 storage: 1e-5 per row and tile, as in the other parity tests (fp32 products and sums on both sides)."""
    r, R = choice(), min(-(-sum(rows) // len(rows)), max(rows))
    wide = len(rows) == 32
    assert r.f32_wgrad_form(len(rows), h, f, R) == (1 if wide else 0)
    assert [r.f32_row_plan(len(rows), max(rows), R, n, k, True) >> 2 for n, k in ((f, h), (h, f))] == [0, 2 if h == 256 else 0]
    run_rows(orc, rows, h, f, dtype="f32")
