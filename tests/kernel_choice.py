"""The host rules of csrc/kernel_choice.h through a small C shim, compiled once per process with g++ (no GPU), and the
kernels that a layer's GEMMs reach by them."""
import ctypes as C
import os
import subprocess
import tempfile

from paper_2303_06318_amd import build

SHIM = r"""
#include "%s"
using namespace moe;
extern "C" {
int64_t adamw_launch_len_(int64_t rest) { return adamw_launch_len(rest); }
int64_t adamw_blocks_(int64_t len) { return adamw_blocks(len); }
int adamw_threads_() { return OPT_THREADS; }
bool adamw_streams_(int64_t n, bool bf16) { return adamw_streams(n, bf16); }
bool gemm_rows_chosen_(int64_t E, int64_t M, int64_t N) { return gemm_rows_chosen(E, M, N); }
int gemm_rows_blocks_(int64_t M) { return gemm_rows_blocks(M); }
int64_t gemm_rows_tiles_(int64_t E, int64_t M, int64_t N, int blocks) { return gemm_rows_tiles(E, M, N, blocks); }
bool gemm_rows_lone_(int64_t tiles, int blocks, bool b_xc) { return gemm_rows_lone(tiles, blocks, b_xc); }
bool gemm_low_tiles_(int usual, int low, int light, int units, int room) { return gemm_low_tiles(usual, low, light, units, room); }
bool gemm_wgrad_chosen_(int64_t E, int64_t M, int64_t N, int64_t K, bool whole) { return gemm_wgrad_chosen(E, M, N, K, whole); }
int gemm_wgrad_run_(int64_t E, int64_t M, int64_t N) { return gemm_wgrad_run(E, M, N); }
bool gemm_panel_chosen_(int64_t E, int64_t M, int64_t N, int64_t K) { return gemm_panel_chosen(E, M, N, K); }
int gemm_panel_run_(int64_t E, int64_t M, int64_t N, int64_t K) { return gemm_panel_run(E, M, N, K); }
bool gemm_panel_fills_(int64_t E, int64_t M, int64_t N, int64_t K) { return gemm_panel_fills(E, M, N, K); }
int f32_plan_(int64_t E, int64_t R, int64_t N, int64_t K) { const F32Plan p = f32_plan(E, R, N, K); return p.mb * 2 + p.lone; }
int f32_row_plan_(int64_t E, int64_t M, int64_t R, int64_t N, int64_t K, bool b_xc) { const F32Plan p = f32_row_plan(E, M, R, N, K, b_xc); return p.mb * 4 + p.wide * 2 + p.lone; }
int f32_wgrad_form_(int64_t E, int64_t M, int64_t N, int64_t R) { return f32_wgrad_form(E, M, N, R); }
bool gate_direct_(bool f32, int64_t T) { return gate_direct(f32, T); }
bool gate_dwg_direct_(bool f32, int64_t T, int E) { return gate_dwg_direct(f32, T, E); }
bool gate_dx_direct_(bool f32, int64_t T, int64_t h, int E, bool rows_ok) { return gate_dx_direct(f32, T, h, E, rows_ok); }
int gate_dx_chunk_(int64_t T, int64_t h, int E) { return gate_dx_chunk(T, h, E); }
}
"""

I64, INT, BOOL = C.c_int64, C.c_int, C.c_bool
SIGNATURES = {
    "adamw_launch_len": (I64, [I64]), "adamw_blocks": (I64, [I64]), "adamw_threads": (INT, []),
    "adamw_streams": (BOOL, [I64, BOOL]), "gemm_rows_chosen": (BOOL, [I64, I64, I64]), "gemm_rows_blocks": (INT, [I64]),
    "gemm_rows_tiles": (I64, [I64, I64, I64, INT]), "gemm_rows_lone": (BOOL, [I64, INT, BOOL]),
    "gemm_low_tiles": (BOOL, [INT, INT, INT, INT, INT]),
    "gemm_wgrad_chosen": (BOOL, [I64, I64, I64, I64, BOOL]), "gemm_wgrad_run": (INT, [I64, I64, I64]),
    "gemm_panel_chosen": (BOOL, [I64, I64, I64, I64]), "gemm_panel_run": (INT, [I64, I64, I64, I64]),
    "gemm_panel_fills": (BOOL, [I64, I64, I64, I64]), "f32_plan": (INT, [I64, I64, I64, I64]),
    "f32_row_plan": (INT, [I64, I64, I64, I64, I64, BOOL]),
    "f32_wgrad_form": (INT, [I64, I64, I64, I64]), "gate_direct": (BOOL, [BOOL, I64]), "gate_dwg_direct": (BOOL, [BOOL, I64, INT]),
    "gate_dx_direct": (BOOL, [BOOL, I64, I64, INT, BOOL]), "gate_dx_chunk": (INT, [I64, I64, INT]),
}

_lib = None


class Rules:
    def __init__(self, L):
        for name, (res, args) in SIGNATURES.items():
            fn = getattr(L, name + "_")
            fn.restype, fn.argtypes = res, args
            setattr(self, name, fn)

    def row_gemm(self, E, C, N, forward):
        """Kernel of a forward or data-gradient GEMM: 'large', or ('rows', 32-row blocks per tile, one workgroup per unit)"""
        if not self.gemm_rows_chosen(E, C, N):
            return "large"
        b = self.gemm_rows_blocks(C)
        return ("rows", b, bool(self.gemm_rows_lone(self.gemm_rows_tiles(E, C, N, b), b, forward)))

    def low_tiles(self, rows, N):
        """Whether the large kernel's plan cuts these experts' rows into low tiles (256 compute units in 8 XCDs)"""
        nt, nb = -(-N // 256), [-(-n // 32) for n in rows]
        low, light = sum(-(-b // 4) for b in nb if b > 4), sum(0 < b <= 4 for b in nb)
        usual = sum(1 if b <= 4 else -(-b // 9) for b in nb if b)
        return low > 0 and bool(self.gemm_low_tiles(usual * nt, low * nt, light * nt, 32, min(len(rows) * -(-max(rows) // 256) * nt, 256)))

    def weight_gemm(self, E, C, M, N, aligned=True):
        """Kernel of a weight gradient [M, N] over C rows where the panel kernel does not come first: 'large', or ('wgrad', whole
        lines, tiles of the longest and of the last run).  aligned: the result array starts on a cache line."""
        whole = aligned and N % 64 == 0
        if not self.gemm_wgrad_chosen(E, M, N, C, whole):
            return "large"
        nt, run = -(-N // 128), self.gemm_wgrad_run(E, M, N)
        return ("wgrad", whole, min(run, nt), (nt - 1) % run + 1)

    def gradient_gemm(self, E, C, M, N):
        """Kernel of a weight gradient into an aligned array: ('panel', row tiles of a run), or as above"""
        if N % 64 == 0 and self.gemm_panel_chosen(E, M, N, C):
            return ("panel", self.gemm_panel_run(E, M, N, C))
        return self.weight_gemm(E, C, M, N)

    def layer_gemms(self, E, C, h, f):
        """Kernels of a bf16 layer's GEMMs"""
        return {"fwd1": self.row_gemm(E, C, f, True), "fwd2": self.row_gemm(E, C, h, True),
                "dh": self.row_gemm(E, C, f, False), "dd": self.row_gemm(E, C, h, False),
                "dw2": self.gradient_gemm(E, C, f, h), "dw1": self.gradient_gemm(E, C, h, f)}


def choice() -> Rules:
    global _lib
    if _lib is None:
        with tempfile.TemporaryDirectory() as d:
            src, so = os.path.join(d, "shim.cpp"), os.path.join(d, "shim.so")
            with open(src, "w") as f:
                f.write(SHIM % os.path.join(build.CSRC, "kernel_choice.h"))
            subprocess.run(["g++", "-std=c++17", "-O1", "-Wall", "-shared", "-fPIC", src, "-o", so], check=True, timeout=120)
            _lib = Rules(C.CDLL(so))
    return _lib
