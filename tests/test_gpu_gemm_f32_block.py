"""The block form of the fp32 grouped GEMM (tiles of up to 160 x 64 on 16 x 16 x 4 MFMAs) at the edges of its tiles, against
the CPU oracle; tolerance as for every fp32 parity test (1e-5 per row and tile).  In the first test experts hold no rows or at least
six: a row of d_w2 is a sum over the expert's rows of hact times d_y, and where a single hact is next to zero (its z is a sum of 512
products with a rounding error of 1e-7, whatever computes it) that row's own norm measures nothing."""
import pytest
import torch

from paper_2303_06318_amd import moe
from kernel_choice import choice
from test_gpu_gemm_edges import run_rows

NARROW, WIDE, BLOCK = range(3)


def forms(E, rows, h, f):
    """(row blocks of a tile, alone on its unit) of GEMM1 and of GEMM2 (from 24 rows on of dH and of dD too), form of the weight
    gradients"""
    r, C = choice(), max(rows)
    R = min(-(-sum(rows) // E), C)
    a, b = ([r.f32_row_plan(E, C, R, n, k, xc) for n, k in ((f, h), (h, f))] for xc in (True, False))
    assert a == b or R < 24
    return [(p >> 2, bool(p & 1)) for p in a], r.f32_wgrad_form(E, h, f, R)


def fill(E, rows, rest):
    return tuple(rows) + tuple(rest[i % len(rest)] for i in range(E - len(rows)))


@pytest.mark.gpu
@pytest.mark.parametrize("E,rows,h,f,want,wgrad", [
    # one tile per unit, five blocks: ragged columns and k-tiles; 8 to 10 and 16 to 20 row blocks
    (8, (320, 272, 257, 256, 241, 240, 160, 161), 1024, 1020, [(5, True), (5, True)], BLOCK),
    # two workgroups per unit; experts without rows, with a handful, with partial blocks
    (64, fill(64, (160, 161, 320, 0, 6, 15, 16, 17, 33, 0), (130, 128, 97)), 512, 516, [(3, False), (5, False)], WIDE),
    # three and two blocks
    (8, (140, 128, 129, 127, 112, 96, 150, 142), 1024, 1024, [(3, True), (3, True)], WIDE),
    (4, (100, 97, 96, 112), 1984, 2044, [(3, True), (3, True)], WIDE),
    (4, (256, 193, 240, 241), 1000, 1000, [(2, True), (2, True)], BLOCK),
    (66, fill(66, (65, 64, 0, 33, 32), (60, 61)), 260, 260, [(2, False), (2, False)], WIDE),
    # more than 64 experts are counted in pieces; few rows
    (100, fill(100, (125, 0, 0, 96, 97), (100, 111, 64, 90)), 256, 256, [(5, False), (5, False)], WIDE),
    (70, fill(70, (7, 0, 64, 65), (50, 49, 6)), 388, 324, [(5, False), (5, False)], WIDE),
    # tokens far from even: tiles of fewer blocks, as long as each has a unit
    (8, (700, 320, 6, 0, 7, 16, 17, 6), 1024, 1024, [(3, True), (3, True)], WIDE),
    (8, (320, 0, 0, 0, 1100, 320, 0, 0), 512, 512, [(2, True), (2, True)], BLOCK),
])
def test_block_form(orc, E, rows, h, f, want, wgrad):
    assert forms(E, rows, h, f) == (want, wgrad)
    run_rows(orc, rows, h, f, dtype="f32")


@pytest.mark.gpu
@pytest.mark.parametrize("E,rows,h,f,want,wgrad", [
    (32, fill(32, (1, 2, 3, 4, 5, 0), (1, 5, 2)), 1024, 1020, [(5, False), (0, False)], WIDE),
    (128, fill(128, (5, 4, 0, 1), (3, 2)), 220, 292, [(0, False), (5, False)], WIDE),
    # weight gradients whose only k-tile holds one to five rows, beside long ones
    (8, (900, 1, 2, 5, 0, 3, 700, 4), 516, 516, [(3, True), (3, True)], BLOCK),
])
def test_block_form_of_handfuls(orc, E, rows, h, f, want, wgrad):
    assert forms(E, rows, h, f) == (want, wgrad)
    run_rows(orc, rows, h, f, dtype="f32", few=True)


def test_estimates_never_ask_for_a_second_round_alone():
    """A tile alone on its compute unit is only planned where an average layer has no more tiles than units."""
    r = choice()
    for E in (1, 2, 8, 64, 256):
        for R in (1, 16, 100, 255, 256, 1000, 5000):
            for N in (4, 64, 260, 1024, 8192):
                for K in (4, 32, 1000, 4096):
                    mb, lone = divmod(r.f32_plan(E, R, N, K), 2)
                    assert mb in (0, 2, 3, 5)
                    if lone:
                        assert E * -(-N // 64) * -(-(R // 16 + 1) // (2 * mb)) <= 256


def row_form(E, M, R, N, K, b_xc=True):
    v = choice().f32_row_plan(E, M, R, N, K, b_xc)
    return "block" if v >> 2 else "wide" if v & 2 else "narrow"


def test_every_capacity_has_a_launch():
    """Whatever an expert holds on average and may hold at most, the form that is chosen has a grid for it: fewer than 2^32 threads,
    and at most 65535 workgroups in the second dimension (64-row tiles; beyond 4,194,240 rows only the block form, whose grid has one
    dimension, has one)."""
    for E in (1, 2, 8, 128, 256):
        for M in (1, 2097120, 2097121, 2200000, 3000000, 4194240):
            for R in (1, 50, 1000, M):
                for N, K in ((4, 4), (64, 64), (128, 64), (64, 128)):
                    form, tiles = row_form(E, M, min(R, M), N, K), E * -(-N // 64) * -(-M // 64)
                    if form == "narrow":
                        assert -(-M // 32) <= 65535, (E, M, R, N, K)
                    elif form == "wide":
                        assert -(-M // 64) <= 65535
                    else:
                        assert tiles < 1 << 22
    assert row_form(128, 2200000, 2200000, 64, 64) == "wide" and row_form(1, 3000000, 100, 64, 64) == "wide"
    assert row_form(1, 2097120, 100, 64, 64) == "narrow" and row_form(1, 2097121, 100, 64, 64) == "wide"


@pytest.mark.parametrize("E,R,K,N,forward,backward", [
    (16, 20, 2048, 2048, "narrow", "narrow"), (64, 16, 1024, 1024, "narrow", "narrow"), (128, 5, 84, 3404, "narrow", "narrow"),
    (64, 4, 2620, 540, "narrow", "narrow"), (32, 2, 1024, 1020, "block", "narrow"), (64, 6, 1924, 472, "block", "narrow"),
    (8, 19, 832, 3140, "block", "narrow"), (4, 30, 4096, 4096, "block", "block"), (32, 40, 440, 1912, "block", "block")])
def test_form_of_few_rows(E, R, K, N, forward, backward):
    """The faster form of a forward and of a data-gradient GEMM, as measured"""
    assert (row_form(E, 2 * R, R, N, K), row_form(E, 2 * R, R, N, K, False)) == (forward, backward)


@pytest.mark.gpu
def test_wide_rows_beyond_the_grid_of_narrow_ones():
    """A capacity that only the wide form's grid covers: the first rows of an expert with few, and every row of one that is full,
    against the same pass in 64 bits; a relative error per row of 1e-5 as for every fp32 test."""
    E, C, h, f = 2, 2097120 + 33, 8, 12
    shape = moe.make_shape(200, h, E, f, C, moe.MOE_F32)
    assert row_form(E, C, 100, f, h) == row_form(E, C, 100, h, f) == "wide"
    g = torch.Generator(device="cuda").manual_seed(4)
    buf, w1, w2 = (torch.randn(s, generator=g, device="cuda") for s in ((E, C, h), (E, h, f), (E, f, h)))
    kept = torch.tensor([37, C], dtype=torch.int32, device="cuda")
    hact, y = torch.full((E, C, f), float("nan"), device="cuda"), torch.full((E, C, h), float("nan"), device="cuda")
    ws = torch.empty(moe.moe_workspace_bytes(shape, 0), dtype=torch.uint8, device="cuda")
    moe.moe_expert_ffn_fwd(shape, buf, w1, w2, kept, None, hact, y, ws)
    for e, k in enumerate((37, C)):
        ref = torch.nn.functional.gelu(buf[e, :k].double() @ w1[e].double())
        for got, want in ((hact[e, :k], ref), (y[e, :k], ref @ w2[e].double())):
            assert bool(((got - want).norm(dim=1) <= 1e-5 * want.norm(dim=1).clamp_min(1e-3)).all())
    assert bool(y[0, 37:].isnan().all())
