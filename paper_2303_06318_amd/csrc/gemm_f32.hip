// Grouped fp32 GEMM for the fp32 storage type on the fp32 matrix instruction (v_mfma_f32_32x32x2_f32: fp32
// products and fp32 sums, no reduced-precision inputs; twice the rate of vector FMAs).
//
// A workgroup of 4 waves owns one output tile of one expert; global data goes through registers (the loads of
// the next k-tile are in flight during the MFMAs of the current one) into LDS.  Two tile forms:
//   wide:   64 x 64, each wave one 32 x 32 quarter, k-tiles of 32, two LDS stages;
//   narrow: 32 x 32, k-tiles of 128 of which each wave takes 32, partial sums added through LDS at the end.
// Narrow tiles serve GEMMs whose 64 x 64 tiles leave compute units idle: there a k-tile costs a memory latency
// and not MFMAs, and a narrow tile needs a quarter of the k-tiles.
#include "moe_common.h"

namespace moe {

constexpr int F32_THREADS = 256;

// One operand's k-tile in LDS.  KC (k contiguous in memory): [X][BK + 4], so that a lane reads four consecutive
// k of its row in one 16-byte read; XC (output index contiguous): [BK][X + 8], one 4-byte read per k.  Both
// paddings keep the reads of a wave free of bank conflicts (row strides of an odd number of 16-byte slots; rows
// 4 apart differ by 32 banks).
template <bool XC, int X, int BK>
struct F32Tile {
    static constexpr int LD = XC ? X + 8 : BK + 4;
    static constexpr int FLOATS = XC ? BK * LD : X * LD;
    static constexpr int NV = X * BK / 4 / F32_THREADS;        // 16-byte loads per thread and k-tile
    static constexpr int PER = XC ? X / 4 : BK / 4;            // 16-byte granules per row
    f32x4 v[NV];
    // x and k extents are checked; contiguous extents are multiples of 4, so a granule is in or out as a whole
    __device__ __forceinline__ void load(const float *p, int ld, int x0, int xlim, int k0, int klim, int tid) {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + F32_THREADS * q, r = idx / PER, c = (idx % PER) * 4;
            const int x = x0 + (XC ? c : r), k = k0 + (XC ? r : c);
            v[q] = x < xlim && k < klim ? *(const f32x4 *)(p + (XC ? (int64_t)k * ld + x : (int64_t)x * ld + k))
                                        : f32x4{0.f, 0.f, 0.f, 0.f};
        }
    }
    __device__ __forceinline__ void store(float *lds, int tid) const {
#pragma unroll
        for (int q = 0; q < NV; ++q) {
            const int idx = tid + F32_THREADS * q;
            *(f32x4 *)(lds + (idx / PER) * LD + (idx % PER) * 4) = v[q];
        }
    }
    // the four values k .. k + 3 of row (column) x
    static __device__ __forceinline__ f32x4 read(const float *lds, int x, int k) {
        if (!XC) return *(const f32x4 *)(lds + x * LD + k);
        f32x4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = lds[(k + j) * LD + x];
        return o;
    }
};

template <int EPI, bool AXC, bool BXC, bool WIDE>
__global__ __launch_bounds__(F32_THREADS) void gemm_f32_kernel(GemmDesc d) {
    constexpr int T = WIDE ? 64 : 32, BK = WIDE ? 32 : 128, STAGES = WIDE ? 2 : 1;
    typedef F32Tile<AXC, T, BK> TA;
    typedef F32Tile<BXC, T, BK> TB;
    constexpr int STAGE = TA::FLOATS + TB::FLOATS;
    constexpr int RED = WIDE ? 0 : 4 * 16 * 64;              // narrow: every wave's 16 partial sums per lane
    __shared__ __attribute__((aligned(16))) float smem[STAGES * STAGE > RED ? STAGES * STAGE : RED];
    const int e = blockIdx.z;
    const int kept = d.kept[e];
    const int Me = d.rows_from_kept ? kept : d.M;
    const int Ke = d.rows_from_kept ? d.K : kept;
    const int m0 = blockIdx.y * T, n0 = blockIdx.x * T;
    if (m0 >= Me) return;
    const float *A = (const float *)d.A + (int64_t)e * d.strideA;
    const float *B = (const float *)d.B + (int64_t)e * d.strideB;
    float *C = (float *)d.C + (int64_t)e * d.strideC;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = WIDE ? (wave >> 1) * 32 : 0, wn = WIDE ? (wave & 1) * 32 : 0;
    const int kw = (WIDE ? 0 : wave * 32) + (lane >> 5) * 4; // this lane's first k of a k-tile
    const int xa = wm + (lane & 31), xb = wn + (lane & 31);

    TA a;
    TB b;
    f32x16 acc;
#pragma unroll
    for (int i = 0; i < 16; ++i) acc[i] = 0.f;
    a.load(A, d.lda, m0, Me, 0, Ke, tid);
    b.load(B, d.ldb, n0, d.N, 0, Ke, tid);
    int stage = 0;
    for (int k0 = 0; k0 < Ke; k0 += BK) {
        float *la = smem + stage * STAGE, *lb = la + TA::FLOATS;
        if (STAGES == 1) __syncthreads();                    // the previous k-tile has been read
        a.store(la, tid);
        b.store(lb, tid);
        __syncthreads();
        if (k0 + BK < Ke) {
            a.load(A, d.lda, m0, Me, k0 + BK, Ke, tid);
            b.load(B, d.ldb, n0, d.N, k0 + BK, Ke, tid);
        }
        // lanes 0-31 supply k = 8 s + j, lanes 32-63 k = 8 s + 4 + j, to both operands
#pragma unroll
        for (int s = 0; s < 4; ++s) {
            const f32x4 av = TA::read(la, xa, kw + 8 * s), bv = TB::read(lb, xb, kw + 8 * s);
#pragma unroll
            for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(av[j], bv[j], acc, 0, 0, 0);
        }
        if (STAGES == 2) stage ^= 1;
    }
    // lane l holds column l % 32 and rows 8 (i / 4) + 4 (l / 32) + i % 4 of its 32 x 32 block
    auto put = [&](int row, int col, float v) {
        const int gm = m0 + row, gn = n0 + col;
        if (gm >= Me || gn >= d.N) return;
        const int64_t o = (int64_t)gm * d.ldc + gn;
        if (EPI == EPI_GELU) {
            if (d.C2) ((float *)d.C2 + (int64_t)e * d.strideC)[o] = act_grad(v, d.act);
            C[o] = act_fwd(v, d.act);
        } else if (EPI == EPI_DGELU) {
            C[o] = v * ((const float *)d.Zin + (int64_t)e * d.strideC)[o];
        } else {
            C[o] = v;
        }
    };
    if (WIDE) {
#pragma unroll
        for (int i = 0; i < 16; ++i) put(wm + 8 * (i >> 2) + 4 * (lane >> 5) + (i & 3), wn + (lane & 31), acc[i]);
        return;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 16; ++i) smem[(wave * 16 + i) * 64 + lane] = acc[i];
    __syncthreads();
#pragma unroll
    for (int q = 0; q < 4; ++q) {                            // wave w adds and writes registers 4 w .. 4 w + 3
        const int i = wave * 4 + q;
        float v = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) v += smem[(w * 16 + i) * 64 + lane];
        put(8 * (i >> 2) + 4 * (lane >> 5) + (i & 3), lane & 31, v);
    }
}

template <int EPI, bool AXC, bool BXC>
static void launch_f32(const GemmDesc &d, hipStream_t s) {
    // Wide tiles from four per compute unit on.  Forward pair of GEMMs, wide / narrow: 32 tiles 17.5 / 11.8 us,
    // 192 tiles 37 / 26, 384 tiles 93 / 69, 640 tiles 129 / 111; with weight gradients of 2048 tiles the backward
    // takes 144 / 155.  Weight gradients, whose reduction is short, from one per compute unit on (whole backward with
    // 256 tiles 34.4 / 37.3, with 512 tiles 49.5 / 55.1).
    const bool w = (int64_t)((d.N + 63) / 64) * ((d.M + 63) / 64) * d.E >= (AXC ? 256 : 1024);
    const int t = w ? 64 : 32;
    const dim3 grid((d.N + t - 1) / t, (d.M + t - 1) / t, d.E);
    if (w) hipLaunchKernelGGL((gemm_f32_kernel<EPI, AXC, BXC, true>), grid, dim3(F32_THREADS), 0, s, d);
    else hipLaunchKernelGGL((gemm_f32_kernel<EPI, AXC, BXC, false>), grid, dim3(F32_THREADS), 0, s, d);
}

moe_status_t launch_gemm_f32(const GemmDesc &d, hipStream_t s) {
    if (!d.a_xc && d.b_xc && d.epi == EPI_GELU) launch_f32<EPI_GELU, false, true>(d, s);           // forward: A [M,K], B [K,N]
    else if (!d.a_xc && d.b_xc && d.epi == EPI_STORE) launch_f32<EPI_STORE, false, true>(d, s);
    else if (!d.a_xc && !d.b_xc && d.epi == EPI_DGELU) launch_f32<EPI_DGELU, false, false>(d, s);  // data gradient: A [M,K], B [N,K]
    else if (!d.a_xc && !d.b_xc && d.epi == EPI_STORE) launch_f32<EPI_STORE, false, false>(d, s);
    else if (d.a_xc && d.b_xc && d.epi == EPI_STORE) launch_f32<EPI_STORE, true, true>(d, s);      // weight gradient: A [K,M], B [K,N]
    else {
        set_error("gemm_f32: combination of operand layouts and epilogue not built");
        return MOE_ERR_UNSUPPORTED;
    }
    return check_launch("gemm_f32");
}

}  // namespace moe
