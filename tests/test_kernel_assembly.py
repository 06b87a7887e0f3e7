"""What the compiler made of the kernels' explicit ordering, read from the assembly of their sources (hipcc for gfx950,
no GPU): properties that results on a GPU show late or not at all."""
import os
import re
import subprocess

import pytest

from paper_2303_06318_amd import build


@pytest.fixture(scope="module")
def kernels(tmp_path_factory):
    """source file -> {kernel symbol: lines of its assembly}"""
    tmp = tmp_path_factory.mktemp("asm")
    cache = {}

    def get(src):
        if src not in cache:
            out = str(tmp / (src + ".s"))
            subprocess.run([build._hipcc(), *build.FLAGS, "--offload-device-only", "-S", os.path.join(build.CSRC, src), "-o", out],
                           check=True, capture_output=True, timeout=300)
            fns, name = {}, None
            for line in open(out):
                m = re.match(r"(_ZN3moe\w+):", line)
                if m:
                    name = m[1]
                    fns[name] = []
                elif line.startswith(".Lfunc_end"):
                    name = None
                elif name:
                    fns[name].append(line.strip())
            cache[src] = fns
        return cache[src]

    return get


def test_wgrad_staging_is_ordered_across_lanes(kernels):
    """gemm_wgrad_kernel hands its results from lane to lane through LDS that only one wave uses.  A wave-level
    barrier separates the writes (8 bytes a lane) from the reads (16 bytes a lane) of other lanes' values, and these
    reads from the next writes; without it nothing but the compiler's habit keeps them in order."""
    found = 0
    for name, lines in kernels("gemm_wgrad.hip").items():
        if "gemm_wgrad_kernel" not in name:
            continue
        found += 1
        ev = []
        for l in lines:
            if l.startswith("ds_write_b64"):
                ev.append("W")
            elif l.startswith("ds_read_b128"):
                ev.append("R")
            elif "wave barrier" in l:
                ev.append("B")
        assert "W" in ev and "R" in ev, name
        for a, b in zip(ev, ev[1:]):
            assert a == b or "B" in (a, b), (name, "".join(ev))
    assert found == 2


def test_row_kernel_keeps_its_ring_in_flight(kernels):
    """gemm_rows_kernel waits in every k-tile for the oldest of its S - 1 requested k-tiles and leaves the S - 2 newer ones
    outstanding: (S - 2) x (loads of a wave per k-tile), 2 of B and its share of the 4 MB chunks of A.  In the paced form
    the waves with a chunk of A leave 2.  The hardware's count has six bits in two places; a value that runs out of its
    field waits for something else."""
    seen = set()
    for name, lines in kernels("gemm_rows.hip").items():
        m = re.search(r"gemm_rows_kernelILb([01])ELi\d+ELi(\d+)ELb([01])E", name)
        if not m:
            continue
        bxc, mb, lone = m[1] == "1", int(m[2]), m[3] == "1"
        stages = {1: 4, 2: 6 if lone else 3}.get(mb, 4 if lone else 2)
        per_wave = {2 + len(range(w, 4 * mb, 8)) for w in range(8)}                 # chunk q of A: wave q % 8
        want = {(stages - 2) * n for n in per_wave}
        if mb == 1 and lone:
            want = {2, (stages - 2) * 2}
        main = lines[:max(i for i, l in enumerate(lines) if l.startswith("v_mfma"))]
        got = {int(n) for l in main for n in re.findall(r"^s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)$", l)}
        assert got == want, (name, want, got)
        seen.add((bxc, mb, lone))
    assert seen == {(b, mb, d) for b in (False, True) for mb in (1, 2, 4, 5) for d in (False, True)} - {(False, 1, True)}


def test_large_gemm_loops_do_not_spill(kernels):
    """No register of gemm_bf16_kernel is spilled inside a main loop, and the loops wait for loads by count only: a
    scratch access, or a wait for everything that one of them makes the compiler put in, drains the loop's pipeline (the
    tall loop once cost a fifth of a forward pass that way)."""
    found = 0
    for name, lines in kernels("gemm_bf16.hip").items():
        if "gemm_bf16_kernel" not in name:
            continue
        found += 1
        inner, mfma = False, 0
        for l in lines:
            if l.startswith(".LBB"):
                inner = "Depth=2" in l
            elif l.startswith(";") and "Depth=2" in l:
                inner = True
            if inner:
                mfma += l.startswith("v_mfma")
                assert not l.startswith("scratch_"), (name, l)
                assert not re.match(r"s_waitcnt vmcnt\(0\)", l), (name, l)
        assert mfma >= 128, name          # the loops were found
    assert found == 5


def waits(lines):
    """Counts of the explicit waits: outstanding global accesses, no LDS access"""
    return {int(n) for l in lines for n in re.findall(r"^s_waitcnt vmcnt\((\d+)\) lgkmcnt\(0\)$", l)}


def test_panel_kernel_counts_loads_and_stores(kernels):
    """gemm_panel_kernel waits for a tile with the loads of S - 2 newer tiles (NKS each) and, once that many have been written,
    the 16 stores of S - 1 older ones outstanding; B's panel is waited for behind the first tiles' loads where it lies beside
    the ring.  Every tile issues its 16 stores (8 in the code of a half tile), nothing is spilled, and the private staging is
    ordered as in gemm_wgrad_kernel."""
    found = 0
    for name, lines in kernels("gemm_panel.hip").items():
        m = re.search(r"gemm_panel_kernelILi(\d+)E", name)
        if not m:
            continue
        found += 1
        want = {0}
        for nks in range(1, int(m[1]) + 1):
            s = min(4, 16 // nks)
            want |= {(s - 2) * nks, (s - 2) * nks + (s - 1) * 16, (s - 1) * nks if (s + 4) * nks <= 20 else 0}
        assert waits(lines) == want, (name, want, waits(lines))
        assert sum(l.startswith("buffer_store_dwordx4") for l in lines) == 8 * int(m[1]), name
        assert not any(l.startswith("scratch_") for l in lines), name
        ev = ["W" if l.startswith("ds_write") else "R" if l.startswith("ds_read_b128") else "B" for l in lines
              if l.startswith(("ds_write", "ds_read_b128")) or "wave barrier" in l]
        assert "W" in ev and "R" in ev, name
        for a, b in zip(ev, ev[1:]):
            assert a == b or "B" in (a, b), (name, "".join(ev))
    assert found == 2


def test_f32_block_kernel_keeps_its_ring_in_flight(kernels):
    """gemm_f32_block_kernel waits for a k-tile with S - 2 newer ones outstanding: one load of B per wave and its share of the 4 MB
    chunks of A; nothing is spilled."""
    seen = set()
    for name, lines in kernels("gemm_f32.hip").items():
        m = re.search(r"gemm_f32_block_kernelILi\d+ELb([01])ELb[01]ELi(\d+)ELb([01])E", name)
        if not m:
            continue
        axc, mb, lone = m[1] == "1", int(m[2]), m[3] == "1"
        stages = {5: 4, 3: 5, 2: 6}[mb] if lone else 2
        per_wave = {1 + len(range(w, 4 * mb, 8)) for w in range(8)}
        assert waits(lines) == {0} | {(stages - 2) * n for n in per_wave}, (name, waits(lines))
        assert not any(l.startswith("scratch_") for l in lines), name
        seen.add((axc, mb, lone))
    assert seen == {(False, mb, d) for mb in (2, 3, 5) for d in (False, True)} | {(True, 2, False)}
