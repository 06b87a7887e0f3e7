"""The host rules that choose kernels and cut launches (csrc/kernel_choice.h, plain C++), built alone with g++: no GPU."""
import pytest

from kernel_choice import choice


@pytest.fixture(scope="module")
def rules():
    return choice()


@pytest.mark.parametrize("n", [1, 3, 4, 1023, 1 << 20, (1 << 33) - 1, 1 << 33, (1 << 33) + 5, (1 << 34) - 1, 1 << 34, (1 << 34) + 3,
                               3 * (1 << 33) + 1, (1 << 40) - 1])
def test_adamw_launches_cover_the_group_and_fit_a_grid(rules, n):
    """Every launch has fewer than 2^32 threads (the runtime's limit), starts on a 16-byte boundary of every array
    (8 elements of the 2-byte ones), and the launches cover the n parameters that the entry point accepts."""
    i0 = 0
    while i0 < n:
        ln = rules.adamw_launch_len(n - i0)
        blocks = rules.adamw_blocks(ln)
        assert 1 <= ln <= n - i0 and i0 % 8 == 0
        assert blocks * rules.adamw_threads() < 1 << 32
        assert blocks * rules.adamw_threads() * 4 >= ln
        i0 += ln
    assert i0 == n


@pytest.mark.parametrize("T,E,direct", [(1, 1, True), (1024, 16, True), (1025, 16, False), (128, 17, True), (129, 17, False),
                                        (128, 64, True), (129, 64, False), (16, 65, False), (1, 128, False), (16, 256, False)])
def test_gate_weight_gradient_kernel(rules, T, E, direct):
    """bf16: the fp32-instruction kernel reads x once per 16 experts, which with many experts costs more than the
    other kernel's launches, however few tokens there are; fp32 tokens have no other kernel."""
    assert rules.gate_dwg_direct(False, T, E) == direct
    assert rules.gate_dwg_direct(True, T, E)


@pytest.mark.parametrize("T,h,E,rows_ok,direct", [
    (1024, 2048, 16, True, True), (1025, 2048, 16, True, False), (2048, 2048, 16, True, False),
    (512, 2048, 17, True, True), (513, 2048, 17, True, False), (2048, 2048, 32, True, False), (512, 2048, 64, True, True),
    (1024, 2048, 64, True, False), (1024, 2048, 65, False, True), (1025, 2048, 65, False, False), (1024, 2048, 32, False, True)])
def test_gate_token_gradient_kernel(rules, T, h, E, rows_ok, direct):
    """bf16: where the row kernel serves, the fp32-instruction kernel only takes token tensors that give it one workgroup
    per compute unit (two for one 16-expert tile); fp32 tokens have no other kernel."""
    assert rules.gate_dx_direct(False, T, h, E, rows_ok) == direct
    assert rules.gate_dx_direct(True, T, h, E, rows_ok)


@pytest.mark.parametrize("tiles,blocks,forward,lone", [(256, 1, True, True), (257, 1, True, False), (192, 1, True, True),
                                                       (191, 1, True, False), (256, 1, False, False), (8, 2, True, True),
                                                       (256, 5, False, True), (257, 4, True, False)])
def test_form_of_the_row_kernel(rules, tiles, blocks, forward, lone):
    assert rules.gemm_rows_lone(tiles, blocks, forward) == lone


@pytest.mark.parametrize("usual,low,light,room,fits", [
    (128, 256, 0, 256, True), (129, 257, 0, 512, False), (160, 192, 64, 256, True), (161, 192, 64, 256, False), (128, 252, 4, 256, False),
    (128, 248, 8, 256, True), (128, 248, 9, 512, False), (130, 245, 10, 256, False), (28, 40, 8, 48, True), (28, 40, 8, 47, False)])
def test_low_tiles_fit_one_round_of_every_xcd(rules, usual, low, light, room, fits):
    """An XCD works off its eighths of the two lists by itself: what fits 256 units need not fit the 32 of each."""
    assert rules.gemm_low_tiles(usual, low, light, 32, room) == fits
    if fits:
        assert max(((x + 1) * low >> 3) - (x * low >> 3) + ((x + 1) * light >> 3) - (x * light >> 3) for x in range(8)) <= 32


def test_kernels_of_layers_at_the_lines(rules):
    """Which kernel serves a layer's GEMMs on both sides of each line"""
    assert rules.row_gemm(64, 160, 2048, True) == ("rows", 5, False) and rules.row_gemm(64, 161, 2048, True) == "large"
    assert rules.row_gemm(255, 256, 128, True) == ("rows", 4, False) and rules.row_gemm(256, 256, 128, True) == "large"
    assert rules.row_gemm(64, 256, 512, True) == ("rows", 4, False) and rules.row_gemm(64, 257, 512, True) == "large"
    assert rules.weight_gemm(16, 160, 2048, 8192) == ("wgrad", True, 8, 8)
    assert rules.weight_gemm(16, 161, 2048, 8192) == "large"
    assert rules.weight_gemm(16, 160, 2048, 8192, aligned=False) == "large" and rules.weight_gemm(64, 32, 2048, 2056) == "large"
    assert rules.weight_gemm(8, 512, 2048, 2048)[0] == "wgrad" and rules.weight_gemm(8, 513, 2048, 2048) == "large"
    assert rules.weight_gemm(4, 1024, 2048, 2048)[0] == "wgrad" and rules.weight_gemm(4, 1025, 2048, 2048) == "large"
    assert rules.weight_gemm(2, 100000, 2048, 2048)[0] == "wgrad"
    assert rules.gate_direct(False, 4096) and not rules.gate_direct(False, 4097) and rules.gate_direct(True, 1 << 20)
    assert [rules.gate_dx_chunk(T, 4096, 16) for T in (6048, 6144, 12096, 12288)] == [48, 96, 96, 192]
    assert rules.adamw_streams(57_600_000, True) and not rules.adamw_streams(57_500_000, True)
