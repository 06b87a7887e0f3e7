// Grouped fp32 GEMM for the fp32 storage type on the fp32 matrix instructions (fp32 products and fp32 sums, no
// reduced-precision inputs; twice the rate of vector FMAs).  Three forms:
//   block:  up to 32 MB rows (MB = 5, 3, 2) x 64 columns per workgroup of 8 waves, operands straight into LDS;
//   wide:   64 x 64, 4 waves, each one 32 x 32 quarter, k-tiles of 32, two LDS stages (weight gradients, and the largest capacities);
//   narrow: 32 x 32, 4 waves, k-tiles of 128 of which each wave takes 32, partial sums added through LDS at the end.
// In the latter two global data goes through registers (the loads of the next k-tile are in flight during the MFMAs of the
// current one).  Small tiles are bound by the path from L2 into the compute units: 8 experts x 256 rows of 1024 x 1024 in
// narrow tiles load 570 MB, 55 us at 10 TB/s, where the MFMAs take 31.  The block form loads a third of that (one tile per
// compute unit at that size, 45 us: MFMAs 34, the first loads, the epilogue and the launch the rest).  Where tiles are too
// few for the chip a k-tile costs a memory latency and not MFMAs, and a narrow tile needs a quarter of the k-tiles.
// Forward pair / backward of that layer: 111 -> 90 us, 208 -> 177.
#include <type_traits>
#include "gemm_bf16_parts.h"
#include "kernel_choice.h"

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

// Block form: a workgroup of 8 waves (2 x 4), a wave every second 16-row block and 16 columns, on
// v_mfma_f32_16x16x4_f32.  Operands go straight into LDS through a ring of S k-tiles of 32; alone on a compute unit (LONE: at
// most one tile for each) the ring is deeper, else two to four workgroups of two stages share a unit.  Four chains of sums
// per element, as many as the narrow form has: two made the error against 64 bits 1.4 times as large (hact 4.5e-7 for
// 3.1e-7), four leave it as it was there and lower it in the weight gradients (4.5e-7 -> 3.7e-7).
constexpr int FB_THREADS = 512, FB_BK = 32, FB_N = 64;
constexpr int LONE_TILES = 256;                              // compute units
constexpr int FB_B_BYTES = FB_BK * FB_N * 4;                 // B's k-tile (8 KB)

// An XC operand in LDS: [32 k][X], 16-byte granule g of k-row k at position g ^ (k / 4 % 4) * 4: the four k-rows that a
// read takes, 4 apart, lie in different quarters of the banks.
template <int X>
struct F32XC {
    static constexpr int ROW = X * 4, KROWS = 1024 / ROW, NQ = FB_BK / (8 * KROWS);   // k-rows per 1 KB chunk, chunks per wave
    uint32_t off;
    int32_t kthr;
    __device__ __forceinline__ void init(int ld, int x0, int xlim, int klim, int wave, int lane) {
        const int krow = wave * KROWS + lane / (64 / KROWS), g = (lane % (64 / KROWS)) ^ ((krow >> 2 & 3) << 2), gx = x0 + g * 4;
        off = gx < xlim ? ((uint32_t)krow * ld + gx) * 4u : OOB;
        kthr = klim - krow;
    }
    __device__ __forceinline__ void request(const i32x4 &rsrc, uint32_t lds, int k0, int ld) const {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int k = k0 + q * 8 * KROWS;
            load_to_lds(rsrc, lds + q * 8192, k < kthr ? off : OOB, (uint32_t)k * ld * 4u);
        }
    }
    // byte address of lane's value of k-row 4 (lane / 16) and column x + lane % 16
    static __device__ __forceinline__ int addr(int x, int lane) {
        const int c = x + (lane & 15);
        return 4 * (lane >> 4) * ROW + (((c >> 2) ^ ((lane >> 4) << 2)) << 4) + (c & 3) * 4;
    }
    static __device__ __forceinline__ f32x4 read(const char *p, int ks) {
        f32x4 o;
#pragma unroll
        for (int j = 0; j < 4; ++j) o[j] = *(const float *)(p + (16 * ks + j) * ROW);
        return o;
    }
};

template <int EPI, bool AXC, bool BXC, int MB, bool LONE>
__global__ __launch_bounds__(FB_THREADS) void gemm_f32_block_kernel(GemmDesc d, int nt) {
    constexpr int S = f32_stages(MB, LONE);
    static_assert(!AXC || MB == 2, "k-rows of A are a power of two long");
    constexpr int A_BYTES = MB * 32 * FB_BK * 4, STAGE = A_BYTES + FB_B_BYTES;
    constexpr int XA = AXC ? 32 * MB : 128, QA = AXC ? F32XC<XA>::NQ : (4 * MB + 7) / 8;   // 1 KB chunks of A per wave
    __shared__ __attribute__((aligned(1024))) char smem[S * STAGE];
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(lds_void *)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int e = 0, kept = 0, r = 0, bm = 2 * MB;                 // the expert, its rows, the tile among its tiles, most blocks of a tile
    if constexpr (AXC) {
        // All experts have the same tiles, but reductions of different length: each XCD takes an eighth of every expert's.
        const int n = nt * ((d.M + 32 * MB - 1) / (32 * MB)), share = (n + 7) >> 3, i = blockIdx.x >> 3;
        e = i / share;
        r = (blockIdx.x & 7) * share + i - e * share;
        if (r >= n) return;
        kept = __builtin_amdgcn_readfirstlane(d.kept[e]);
    } else {
        // The launch has a workgroup for every tile that the capacity allows.  The tiles that exist, an expert's 16-row blocks in
        // m-tiles of nearly equal size, are numbered here, and each XCD takes a contiguous eighth of them: by the capacity's
        // numbers the absent tiles would leave one XCD with more tiles than compute units.
        const int last = d.E < 64 ? d.E - 1 : 63;
        auto rows_of = [&](int at) { return at + lane < d.E ? d.kept[at + lane] : 0; };
        auto count = [&](int rows) {                         // inclusive count of m-tiles up to this lane's expert
            int n = (((rows + 15) >> 4) + bm - 1) / bm;
            for (int o = 1; o < 64 && o < d.E; o <<= 1) {
                const int up = __shfl_up(n, o);
                n += lane >= o ? up : 0;
            }
            return n;
        };
        int e0 = 0, first = 0, rows0 = rows_of(0), upto = count(rows0), tiles = __builtin_amdgcn_readlane(upto, last);
        for (int at = 64; at < d.E; at += 64) tiles += __builtin_amdgcn_readlane(count(rows_of(at)), 63);
        if (LONE && d.E <= 64) {                             // smaller tiles while every one still has a compute unit of its own
            while (bm > 2) {
                const int was = bm;
                bm -= bm > 6 ? 3 : bm > 4 ? 2 : 1;
                const int fewer = count(rows0), n = __builtin_amdgcn_readlane(fewer, last);
                if (n * nt > LONE_TILES) {
                    bm = was;
                    break;
                }
                upto = fewer;
                tiles = n;
            }
        }
        tiles *= nt;
        const int per = (tiles + 7) >> 3, t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
        if ((int)(blockIdx.x >> 3) >= per || t >= tiles) return;
        uint64_t past;
        while ((past = __ballot(upto * nt > t - first)) == 0) {
            first += __builtin_amdgcn_readlane(upto, last) * nt;
            e0 += 64;
            rows0 = rows_of(e0);
            upto = count(rows0);
        }
        const int l = __builtin_ctzll(past);
        e = e0 + l;
        kept = __builtin_amdgcn_readlane(rows0, l);
        r = t - first - (l > 0 ? __builtin_amdgcn_readlane(upto, l - 1) * nt : 0);
    }
    const int Me = d.rows_from_kept ? kept : d.M, Ke = d.rows_from_kept ? d.K : kept;
    const int nb = (Me + 15) >> 4, mts = (nb + bm - 1) / bm;
    const int nti = r / mts, mti = r - nti * mts, n0 = nti * FB_N;
    const int bb = nb / mts, bx = nb - bb * mts;
    const int m0 = (mti * bb + (mti < bx ? mti : bx)) * 16, mend = m0 + (bb + (mti < bx ? 1 : 0)) * 16;
    const int mlim = Me < mend ? Me : mend;
    const int wr = wave >> 2, wc = (wave & 3) * 16;
    const bool has_last = AXC || MB % 2 == 0 || wave < 4;    // this wave loads QA chunks of A, otherwise QA - 1

    const i32x4 A = make_rsrc((const float *)d.A + (int64_t)e * d.strideA, (uint32_t)(AXC ? Ke : Me) * (uint32_t)d.lda * 4u);
    const i32x4 B = make_rsrc((const float *)d.B + (int64_t)e * d.strideB, (uint32_t)(BXC ? Ke : d.N) * (uint32_t)d.ldb * 4u);
    // KC operands: the bf16 loader on rows of twice as many 2-byte elements
    Loader<false, QA, 128> lak;
    Loader<false, 1, 128> lbk;
    F32XC<XA> lax;
    F32XC<FB_N> lbx;
    FragAddr<false, 128> fa, fb;
    int ax[MB], bxa = 0;
    if constexpr (AXC) {
        lax.init(d.lda, m0, mlim, Ke, wave, lane);
#pragma unroll
        for (int i = 0; i < MB; ++i) ax[i] = F32XC<XA>::addr((2 * i + wr) * 16, lane);
    } else {
        lak.init(2 * d.lda, m0, mlim, wave, lane);
        lak.init_k(2 * Ke, wave, lane);
        fa.init(wr * 16, lane);
    }
    if constexpr (BXC) {
        lbx.init(d.ldb, n0, d.N, Ke, wave, lane);
        bxa = F32XC<FB_N>::addr(wc, lane);
    } else {
        lbk.init(2 * d.ldb, n0, d.N, wave, lane);
        lbk.init_k(2 * Ke, wave, lane);
        fb.init(wc, lane);
    }
    auto request = [&](int kt, int stage) {                  // past the end of K: zeros, without memory traffic
        const uint32_t base = smem_addr + stage * STAGE + wave * 1024;
        if constexpr (AXC) lax.request(A, base, kt * FB_BK, d.lda);
        else {
#pragma unroll
            for (int q = 0; q < QA; ++q)
                if (q < QA - 1 || has_last) lak.request(A, base, kt * 2 * FB_BK, 2 * d.lda, q);
        }
        if constexpr (BXC) lbx.request(B, base + A_BYTES, kt * FB_BK, d.ldb);
        else lbk.request(B, base + A_BYTES, kt * 2 * FB_BK, 2 * d.ldb, 0);
    };
    // four chains of sums per block
    f32x4 acc[4][MB];
#pragma unroll
    for (int c = 0; c < 4; ++c)
#pragma unroll
        for (int i = 0; i < MB; ++i) acc[c][i] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nk = (Ke + FB_BK - 1) / FB_BK;
    const int ni = (((mlim - m0 + 15) >> 4) - wr + 1) >> 1;  // 16-row blocks 2 i + wr, i < ni, of this wave hold rows
    auto main_loop = [&](auto nic) {
        constexpr int NI = decltype(nic)::value;
#pragma unroll
        for (int s = 0; s < S - 1; ++s) request(s, s);
        int stage = 0;
        for (int kt = 0; kt < nk; ++kt) {
            // k-tile kt has landed (S - 2 newer ones may be outstanding), and every wave has read k-tile kt - 1, whose
            // stage the next request overwrites
            __builtin_amdgcn_sched_barrier(0);
            if (has_last) wait_outstanding<(S - 2) * (QA + 1)>();
            else wait_outstanding<(S - 2) * QA>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            request(kt + S - 1, stage == 0 ? S - 1 : stage - 1);
            const char *ta = smem + stage * STAGE, *tb = ta + A_BYTES;
#pragma unroll
            for (int ks = 0; ks < 2; ++ks) {
                f32x4 bf, af[MB];
                if constexpr (BXC) bf = F32XC<FB_N>::read(tb + bxa, ks);
                else bf = __builtin_bit_cast(f32x4, fb.read(tb, 0, ks));
#pragma unroll
                for (int i = 0; i < NI; ++i) {
                    if constexpr (AXC) af[i] = F32XC<XA>::read(ta + ax[i], ks);
                    else af[i] = __builtin_bit_cast(f32x4, fa.read(ta, 2 * i, ks));
                }
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int i = 0; i < NI; ++i)
                        acc[2 * ks + (j & 1)][i] = __builtin_amdgcn_mfma_f32_16x16x4f32(bf[j], af[i][j], acc[2 * ks + (j & 1)][i], 0, 0, 0);
            }
            stage = stage == S - 1 ? 0 : stage + 1;
        }
    };
    // a loop for every number of blocks: a branch around a block's reads would wait for each of them
    switch (ni) {
        case 0: main_loop(std::integral_constant<int, 0>{}); break;
        case 1: main_loop(std::integral_constant<int, 1>{}); break;
        case 2: main_loop(std::integral_constant<int, MB < 2 ? MB : 2>{}); break;
        case 3: main_loop(std::integral_constant<int, MB < 3 ? MB : 3>{}); break;
        case 4: main_loop(std::integral_constant<int, MB < 4 ? MB : 4>{}); break;
        default: main_loop(std::integral_constant<int, MB>{});
    }
    wait_outstanding<0>();                                   // no request may outlive the workgroup's LDS
    // lane holds row lane % 16 and columns 4 (lane / 16) .. + 3 of every block
    const int gn = n0 + wc + 4 * (lane >> 4);
    if (gn >= d.N) return;
#pragma unroll
    for (int i = 0; i < MB; ++i) {
        const int gm = m0 + (2 * i + wr) * 16 + (lane & 15);
        if (gm >= mlim) continue;
        f32x4 v = (acc[0][i] + acc[1][i]) + (acc[2][i] + acc[3][i]);
        const int64_t o = (int64_t)e * d.strideC + (int64_t)gm * d.ldc + gn;
        if (EPI == EPI_GELU) {
            f32x4 g;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (d.C2) g[q] = act_grad(v[q], d.act);
                v[q] = act_fwd(v[q], d.act);
            }
            if (d.C2) *(f32x4 *)((float *)d.C2 + o) = g;
        } else if (EPI == EPI_DGELU) {
            v *= *(const f32x4 *)((const float *)d.Zin + o);
        }
        *(f32x4 *)((float *)d.C + o) = v;
    }
}

template <int EPI, bool AXC, bool BXC, int MB>
static void launch_f32_block(const GemmDesc &d, hipStream_t s, bool lone) {
    const int nt = (d.N + FB_N - 1) / FB_N, mt = (d.M + 32 * MB - 1) / (32 * MB), total = AXC ? d.E * ((nt * mt + 7) / 8) : (d.E * nt * mt + 7) / 8;
    const dim3 grid((unsigned)(lone && total * 8 < LONE_TILES ? LONE_TILES : total * 8));
    if constexpr (!AXC) {
        if (lone) {
            hipLaunchKernelGGL((gemm_f32_block_kernel<EPI, AXC, BXC, MB, true>), grid, dim3(FB_THREADS), 0, s, d, nt);
            return;
        }
    }
    hipLaunchKernelGGL((gemm_f32_block_kernel<EPI, AXC, BXC, MB, false>), grid, dim3(FB_THREADS), 0, s, d, nt);
}

template <int EPI, bool AXC, bool BXC, bool WIDE>
static void launch_f32_tiles(const GemmDesc &d, hipStream_t s) {
    constexpr int t = WIDE ? 64 : 32;
    const dim3 grid((d.N + t - 1) / t, (d.M + t - 1) / t, d.E);
    hipLaunchKernelGGL((gemm_f32_kernel<EPI, AXC, BXC, WIDE>), grid, dim3(F32_THREADS), 0, s, d);
}

template <int EPI, bool AXC, bool BXC>
static void launch_f32(const GemmDesc &d, hipStream_t s) {
    if constexpr (AXC) {
        switch (f32_wgrad_form(d.E, d.M, d.N, d.rows)) {
            case F32_BLOCK: return launch_f32_block<EPI, AXC, BXC, 2>(d, s, false);
            case F32_WIDE: return launch_f32_tiles<EPI, AXC, BXC, true>(d, s);
            default: return launch_f32_tiles<EPI, AXC, BXC, false>(d, s);
        }
    } else {
        const F32Plan p = f32_row_plan(d.E, d.M, d.rows, d.N, d.K, BXC);
        if (p.mb == 5) launch_f32_block<EPI, AXC, BXC, 5>(d, s, p.lone);
        else if (p.mb == 3) launch_f32_block<EPI, AXC, BXC, 3>(d, s, p.lone);
        else if (p.mb == 2) launch_f32_block<EPI, AXC, BXC, 2>(d, s, p.lone);
        else if (p.wide) launch_f32_tiles<EPI, AXC, BXC, true>(d, s);
        else launch_f32_tiles<EPI, AXC, BXC, false>(d, s);
    }
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
