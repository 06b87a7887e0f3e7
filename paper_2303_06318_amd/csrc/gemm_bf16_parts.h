// Device code shared by the matrix kernels: activations of the bf16 epilogues, operand loads from global memory straight
// into LDS, fragment reads.  The bf16 grouped GEMMs (large, few-row, weight gradients, panel) run 512 threads and the same
// MFMA with the same operand order over k ascending, so for the same inputs they add up in the same order and give the same
// bits; the gate of long token tensors and the fp32 block form use the loaders and the fragment reads.
#pragma once
#include "moe_common.h"

namespace moe {

constexpr int BK = 64, GEMM_THREADS = 512;
constexpr int KS = BK / 32;                    // MFMA k-steps per k-tile
constexpr int KC_ROW = BK * 2;                 // bytes of one KC row in LDS
typedef __attribute__((address_space(3))) s16x4 lds_s16x4;
typedef __attribute__((address_space(3))) void lds_void;

// GeLU for the bf16 epilogues: erf by the Abramowitz-Stegun 7.1.26 rational form (absolute error
// 1.5e-7, far below bf16 resolution) with hardware exp and reciprocal; no branches.
__device__ __forceinline__ float erf_exp_fast(float u, float &ex) {   // u >= 0; ex = exp(-u*u)
    const float t = __builtin_amdgcn_rcpf(fmaf(0.3275911f, u, 1.0f));
    ex = __expf(-u * u);
    float p = fmaf(t, 1.061405429f, -1.453152027f);
    p = fmaf(t, p, 1.421413741f);
    p = fmaf(t, p, -0.284496736f);
    p = fmaf(t, p, 0.254829592f);
    return 1.0f - p * t * ex;
}
__device__ __forceinline__ float tanh_fast(float u) {
    const float e2 = __expf(2.0f * u);
    return 1.0f - 2.0f * __builtin_amdgcn_rcpf(e2 + 1.0f);
}
__device__ __forceinline__ float gelu_fast(float x, int act) {
    if (act == MOE_GELU_TANH) {
        const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
        return 0.5f * x * (1.0f + tanh_fast(u));
    }
    float ex;
    const float er = erf_exp_fast(fabsf(x) * 0.7071067811865476f, ex);
    return 0.5f * x * (1.0f + copysignf(er, x));
}
// GeLU and its derivative together (they share the erf / tanh and the exponential).
__device__ __forceinline__ void gelu_both_fast(float x, int act, float &h, float &g) {
    if (act == MOE_GELU_TANH) {
        const float u = 0.7978845608028654f * (x + 0.044715f * x * x * x);
        const float th = tanh_fast(u);
        const float du = 0.7978845608028654f * (1.0f + 0.134145f * x * x);
        const float phi = 0.5f * (1.0f + th);
        h = x * phi;
        g = phi + 0.5f * x * (1.0f - th * th) * du;
        return;
    }
    float ex;
    const float er = erf_exp_fast(fabsf(x) * 0.7071067811865476f, ex);
    const float phi = 0.5f * (1.0f + copysignf(er, x));
    h = x * phi;
    g = phi + x * ex * 0.3989422804014327f;
}

// Buffer resource (raw, stride 0) over one expert's operand: lanes whose byte offset is not below
// `bytes` -- including offsets forced to OOB -- deliver zero without a branch.
typedef __attribute__((ext_vector_type(4))) int i32x4;
__device__ __forceinline__ i32x4 make_rsrc(const void *p, uint32_t bytes) {
    const uint64_t a = (uint64_t)p;
    i32x4 r;
    r[0] = __builtin_amdgcn_readfirstlane((int)(uint32_t)a);
    r[1] = __builtin_amdgcn_readfirstlane((int)((uint32_t)(a >> 32) & 0xffffu));
    r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
    r[3] = 0x00020000;
    return r;
}
constexpr uint32_t OOB = 0x80000000u;

// One direct global -> LDS load: lane L's 16 bytes land at LDS byte address lds_addr + 16 L, taken from
// voff (per lane) + soff (same for all lanes).
// Written as inline assembly so that the compiler does not order later LDS reads of the *other*
// stage behind it; completion is awaited explicitly (s_waitcnt vmcnt) before the stage is read.
__device__ __forceinline__ void load_to_lds(const i32x4 &rsrc, uint32_t lds_addr, uint32_t voff, uint32_t soff) {
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, %3 offen lds"
                 :
                 : "s"(lds_addr), "v"(voff), "s"(rsrc), "s"(soff)
                 : "memory", "m0");
}

// Wait until at most LOADS of this wave's global memory accesses are outstanding (loads retire in the order of issue) and,
// with LDS, none of its LDS accesses.  The count has six bits, in bits 3:0 and 15:14 of the operand.
template <int LOADS, bool LDS = true>
__device__ __forceinline__ void wait_outstanding() {
    static_assert(LOADS >= 0 && LOADS < 64, "the count is six bits wide");
    __builtin_amdgcn_s_waitcnt((LDS ? 0x0070 : 0x0F70) | (LOADS & 15) | (LOADS >> 4) << 14);
}

// LDS that only one wave uses: what its lanes wrote before is there for its other lanes afterwards (and what they read
// before is not overwritten).  The LDS serves a wave's accesses in order, so this only keeps the compiler from
// moving them; it costs no instruction.
__device__ __forceinline__ void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Where row gx of a KC operand lives in the array its resource covers, when that is not row gx itself:
// through an index array (negative entry: no such row), or in the row shares of duplicate token dropping
// (share gx % G, row base + gx / G of that share).
struct RowMap {
    const int32_t *index;
    int32_t G, share_rows, base;          // G > 0: shares of share_rows rows each; base = first row of this expert in a share
    __device__ __forceinline__ bool mapped() const { return index != nullptr || G > 0; }
    __device__ __forceinline__ int row(int gx) const {
        return index != nullptr ? index[gx] : (gx % G) * share_rows + base + gx / G;
    }
};

// Global -> LDS copy of one operand.  A part of a tile (a half of A, the whole of B) is filled by 1 KB
// chunks, chunk wave + WAVES q by wave `wave`; lane L fills granule L of the chunk:
//   KC chunk:   8 rows of 128 bytes,    lane L -> row L / 8,    position L % 8
//   XC A chunk: 4 k-rows of 256 bytes,  lane L -> k-row L / 16, position L % 16
//   XC B chunk: 2 k-rows of 512 bytes,  lane L -> k-row L / 32, position L % 32
// Chunks of a wave are 8 (or, in workgroups of 4 waves, 4) apart, so the swizzle of a lane is the same in all of them,
// and in an XC operand they differ by a whole number of k-rows, which goes into the load's scalar offset: one offset
// register per part, whereas the rows of a KC operand are bounds-checked (or gathered) one by one.
template <bool XC, int NQ, int XC_COLS, int WAVES = 8>
struct Loader {
    static_assert(WAVES == 8 || (WAVES == 4 && (!XC || XC_COLS == 128)), "chunks of a wave share one swizzle");
    static constexpr int KROWS = 1024 / (XC_COLS * 2);      // XC: k-rows per chunk
    uint32_t off[XC ? 1 : NQ];           // byte offset of this lane's granule at k = 0 (OOB: outside the operand in x)
    int32_t kthr;                        // the granule of chunk q is below klim iff k0 (XC: + q * WAVES * KROWS) < kthr
    __device__ __forceinline__ void init_k(int klim, int wave, int lane) {
        if (XC) kthr = klim - (wave * KROWS + lane / (64 / KROWS));
        else kthr = klim - (((lane & 7) ^ ((wave * 4 + (lane >> 4)) & 7)) << 3);
    }
    __device__ __forceinline__ void init(int ld, int x0, int xlim, int wave, int lane,
                                         const RowMap &map = RowMap{nullptr, 0, 0, 0}) {
        if (XC) {
            const int krow = wave * KROWS + lane / (64 / KROWS);
            const int gx = x0 + (((lane % (64 / KROWS)) ^ ((krow & 3) << 2) ^ ((krow >> 3 & 1) << 1)) << 3);
            off[0] = gx < xlim ? ((uint32_t)krow * ld + gx) * 2u : OOB;
        } else {
#pragma unroll
            for (int q = 0; q < (XC ? 1 : NQ); ++q) {
                const int row = (wave + WAVES * q) * 8 + (lane >> 3);
                const int g = (lane & 7) ^ ((row >> 1) & 7);
                const int gx = x0 + row;
                if (map.mapped()) {
                    const int src = gx < xlim ? map.row(gx) : -1;
                    off[q] = src >= 0 ? ((uint32_t)src * ld + g * 8) * 2u : OOB;
                } else {
                    off[q] = gx < xlim ? ((uint32_t)gx * ld + g * 8) * 2u : OOB;
                }
            }
        }
    }
    // request chunk q of the part's k-tile at origin k0 (it lands at lds + q * WAVES KB); past the end of K: zeros
    __device__ __forceinline__ void request(const i32x4 &rsrc, uint32_t lds, int k0, int ld, int q) const {
        const int k = XC ? k0 + q * WAVES * KROWS : k0;
        const uint32_t voff = k < kthr ? off[XC ? 0 : q] : OOB;
        load_to_lds(rsrc, lds + q * WAVES * 1024, voff, XC ? (uint32_t)k * ld * 2u : (uint32_t)k * 2u);
    }
};

// Byte offsets (inside an operand part) from which lane `lane` reads its MFMA fragments: lane l supplies row or
// column l % 16 of a 16-wide block and k = 8 (l / 16) .. + 7 of a 32-deep k-step.
//   KC: one offset per k-step, blocks of 16 rows add 16 * KC_ROW bytes.
//   XC: one offset per 16-column block, k-steps add 32 k-rows, the second half 4 k-rows (of XC_COLS columns).
template <bool XC, int XC_COLS>
struct FragAddr {
    int32_t a[XC ? 4 : KS];
    // XC: fragment b is the 16-column block b ^ swap (swap 0 or 2)
    __device__ __forceinline__ void init(int xbase, int lane, int swap = 0) {
        if (XC) {
            const int kr = 8 * (lane >> 4) + ((lane & 15) >> 2);
            const int swz = ((kr & 3) << 2) ^ ((kr >> 3 & 1) << 1);
#pragma unroll
            for (int b = 0; b < (XC ? 4 : 0); ++b)
                a[b] = kr * (XC_COLS * 2) + (((((xbase + (b ^ swap) * 16) >> 3) + ((lane & 3) >> 1)) ^ swz) << 4) + (lane & 1) * 8;
        } else {
            // swizzle term of row = xbase + lane%16 (xbase is a multiple of 16, which the term ignores)
            const int s = ((lane & 15) >> 1) & 7;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks)
                a[ks] = (xbase + (lane & 15)) * KC_ROW + (((ks * 4 + (lane >> 4)) ^ s) << 4);
        }
    }
    __device__ __forceinline__ bf16x8 read(const char *tile, int blk, int ks) const {
        if (XC) {
            const char *p = tile + a[blk] + ks * 32 * (XC_COLS * 2);
            s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p));
            s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4 *)(p + 4 * (XC_COLS * 2)));
            typedef __attribute__((ext_vector_type(8))) short s16x8;
            s16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            return __builtin_bit_cast(bf16x8, both);
        } else {
            return *(const bf16x8 *)(tile + a[ks] + blk * 16 * KC_ROW);
        }
    }
};

}  // namespace moe
