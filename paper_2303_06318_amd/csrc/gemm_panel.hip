// Grouped bf16 weight gradient for experts with few rows and large matrices:  C[M, N] = A^T B over kept[e] rows,
// A [rows, M], B [rows, N].
//
// With a short reduction the GEMM is a stream of results (16 experts of 2048 x 8192 write 537 MB however few rows they
// hold), and memory traffic is at its least (counted: 537 MB written, 21 MB read).  What bounds it is that stream and,
// beside it, the path from L2 into the compute units, which loads and stores share.  So
//  - a workgroup (8 waves, one per compute unit) keeps B's fragments of 512 columns in registers for a run of 128-row tiles,
//    a wave's 64 columns x all k, and only A is loaded per tile: by whole tiles (all k), through a ring of S stages in LDS,
//    requested S - 1 tiles ahead.  One barrier per tile; its wait leaves the newer requests and the stores of S - 1 tiles
//    outstanding.  (Panels of 256 columns, which load A twice as often: 120-134 us against 105-118 for 16 experts x 128 rows of
//    2048 x 8192 or 4096 x 4096; without the loads of A that kernel took 90, without its stores 76.)
//  - the workgroups of an expert walk down its rows side by side, so that what is being written at a time is a block of
//    whole rows (walking along the columns instead, 6 rows per expert: 118 us, now 85 for 537 MB), and their tiles
//    alternate.  Every wave writes its part through a private 4 KB of LDS as whole 128-byte lines, past the caches: nothing
//    reads them soon, and written through the L2 they cost 20 % more.
// Weight gradient of 16 experts x 128 rows: 2048 x 8192 168 -> 110 us, 4096 x 4096 163 -> 109 (gemm_wgrad.hip before).
// Operand layouts, swizzles and the order of the sums are those of gemm_bf16.hip.
#include <type_traits>
#include "gemm_bf16_parts.h"
#include "kernel_choice.h"

namespace moe {

constexpr int P_M = PANEL_ROWS, P_N = PANEL_COLS;
constexpr int P_STEP = 32 * P_M * 2;                         // 32 k-rows of a tile (8 KB)
constexpr int P_RING = 128 * 1024;
constexpr int P_OUT = 32 * 128;                              // a wave's staging area: 32 rows of 64 columns
constexpr int P_LDS = P_RING + 8 * P_OUT;
constexpr int P_STORES = 16;                                 // 1 KB stores of a wave per tile
constexpr int STREAM = 18;                                   // nt, sc1: 2-5 % faster than nt alone
constexpr int panel_stages(int nks) { return P_RING / (P_STEP * nks) < 4 ? P_RING / (P_STEP * nks) : 4; }

template <int KMAX>
__global__ __launch_bounds__(GEMM_THREADS, 2) void gemm_panel_kernel(GemmDesc d, int np, int mt, int runs, int total) {
    __shared__ __attribute__((aligned(1024))) char smem[P_LDS];
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(lds_void *)smem;
    // each XCD takes a contiguous eighth of the list: the panels of one expert read the same A from one L2
    const int per = (total + 7) >> 3, t = (blockIdx.x & 7) * per + (blockIdx.x >> 3);
    if (t >= total) return;
    const int at = t / (np * runs), r = t - at * np * runs, ri = r / np, n0 = (r - ri * np) * P_N;
    // Every eighth expert goes to one XCD: an uneven router may favour a stretch of the experts (64 experts of 2048 x 4096, capacity
    // 256, the first nine full: whole backward 544 us by contiguous eighths, now 507).
    const int e = d.E % 8 == 0 ? at % (d.E / 8) * 8 + at / (d.E / 8) : at;
    const int ntiles = (mt - ri + runs - 1) / runs;           // row tiles ri, ri + runs, ...
    const int Ke = __builtin_amdgcn_readfirstlane(d.kept[e]);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int wn = wave * 64;
    const i32x4 A = make_rsrc((const bf16_t *)d.A + (int64_t)e * d.strideA, (uint32_t)Ke * (uint32_t)d.lda * 2u);
    const i32x4 B = make_rsrc((const bf16_t *)d.B + (int64_t)e * d.strideB, (uint32_t)Ke * (uint32_t)d.ldb * 2u);
    // Results go out through a buffer resource (a matrix is shorter than 2 GiB): rows past M lie past its end, columns past
    // N get an offset past it, and every tile issues the same number of stores, which the waits count.
    const __amdgpu_buffer_rsrc_t C =
        __builtin_amdgcn_make_buffer_rsrc((bf16_t *)d.C + (int64_t)e * d.strideC, 0, (int)((uint32_t)d.M * (uint32_t)d.ldc * 2u), 0x00020000);
    const int gn = n0 + wn + (lane & 7) * 8;

    auto body = [&](auto nksc) __attribute__((always_inline)) {
        constexpr int NKS = decltype(nksc)::value, S = panel_stages(NKS), STAGE = NKS * P_STEP;
        static_assert(S >= 2 && (S - 2) * NKS + (S - 1) * P_STORES < 64, "the waits count up to 63 accesses");
        Loader<true, NKS, P_M> ld;
        FragAddr<true, P_M> fr;
        ld.init_k(Ke, wave, lane);
        auto request = [&](const i32x4 &rsrc, int row_len, int at) {
#pragma unroll
            for (int q = 0; q < NKS; ++q) ld.request(rsrc, smem_addr + at + wave * 1024, 0, row_len, q);
        };
        int nreq = 0;                                        // next tile of the run to request
        auto request_a = [&](int stage) {                    // past the end of the run: zeros, without memory traffic
            ld.init(d.lda, (ri + nreq * runs) * P_M, nreq < ntiles ? d.M : 0, wave, lane);
            request(A, d.lda, stage * STAGE);
            ++nreq;
        };
        // B's panel in quarters of 128 columns, two waves to each.  Short reductions: beside the ring, whose first tiles are
        // requested at once; else through the ring's memory, all four together or two at a time.
        constexpr bool BESIDE = (S + 4) * STAGE <= P_LDS;
        constexpr int Q = BESIDE || 4 * STAGE <= P_LDS ? 4 : 2, FIRST = BESIDE ? S - 1 : 0, B_AT = BESIDE ? S * STAGE : 0;
        bf16x8 bf[4][NKS];
        fr.init((wave & 1) * 64, lane);
#pragma unroll
        for (int q0 = 0; q0 < 4; q0 += Q) {
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                ld.init(d.ldb, n0 + (q0 + q) * P_M, d.N, wave, lane);
                request(B, d.ldb, B_AT + q * STAGE);
            }
#pragma unroll
            for (int s = 0; s < FIRST; ++s) request_a(s);
            wait_outstanding<FIRST * NKS>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            if (Q == 4 || (wave >> 2) * 2 == q0) {
                const char *tb = smem + B_AT + (wave / 2 - q0) * STAGE;
#pragma unroll
                for (int j = 0; j < 4; ++j)
#pragma unroll
                    for (int ks = 0; ks < NKS; ++ks) bf[j][ks] = fr.read(tb, j, ks);
            }
            __builtin_amdgcn_sched_barrier(0);
            wait_outstanding<FIRST * NKS>();                 // the reads are done before the memory is used again
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int s = FIRST; s < S - 1; ++s) request_a(s);
        char *out = smem + P_RING + wave * P_OUT;
        int stage = 0;
        for (int n = 0; n < ntiles; ++n) {
            // tile n has landed (S - 2 newer ones and the stores of up to S - 1 older ones may be outstanding), and every
            // wave has read tile n - 1, whose stage the next request overwrites
            __builtin_amdgcn_sched_barrier(0);
            if (n < S - 1) wait_outstanding<(S - 2) * NKS>();
            else wait_outstanding<(S - 2) * NKS + (S - 1) * P_STORES>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            request_a(stage == 0 ? S - 1 : stage - 1);
#pragma unroll 1
            for (int half = 0; half < 2; ++half) {
                fr.init(half * 64, lane);
                const char *ta = smem + stage * STAGE;
                f32x4 acc[4][4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
#pragma unroll
                    for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int ks = 0; ks < NKS; ++ks) {
                    bf16x8 af[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) af[i] = fr.read(ta, i, ks);
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[j][ks], af[i], acc[i][j], 0, 0, 0);
                }
                // lane holds row lane % 16 and columns (lane / 16) * 4 .. + 3 of every 16 x 16 block; 16-byte granule g of
                // staging row r sits at position g ^ (r & 7)
                const uint32_t base = gn < d.N ? ((uint32_t)((ri + n * runs) * P_M + half * 64 + (lane >> 3)) * (uint32_t)d.ldc + gn) * 2u : OOB;
#pragma unroll
                for (int hf = 0; hf < 2; ++hf) {
                    const int sr = lane & 15;
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const f32x4 v = acc[2 * hf + i][j];
                            bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
                            *(bf16x4 *)(out + (i * 16 + sr) * 128 + (((j * 2 + (lane >> 5)) ^ (sr & 7)) << 4) + ((lane >> 4) & 1) * 8) = o;
                        }
                    wave_lds_fence();
#pragma unroll
                    for (int p = 0; p < 4; ++p) {
                        const int row = p * 8 + (lane >> 3);
                        const u32x4 v = *(const u32x4 *)(out + row * 128 + (((lane & 7) ^ (row & 7)) << 4));
                        const uint32_t off = base == OOB ? OOB : base + (uint32_t)(hf * 32 + p * 8) * (uint32_t)d.ldc * 2u;
                        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned int, v), C, off, 0, STREAM);
                    }
                    wave_lds_fence();                            // the next rows overwrite what was just read
                }
            }
            stage = stage == S - 1 ? 0 : stage + 1;
        }
        wait_outstanding<0>();                               // no request may outlive the workgroup's LDS
    };
    const int nks = (Ke + 31) >> 5;                          // no rows: one k-step of zeros
    switch (nks) {
        case 0:
        case 1: body(std::integral_constant<int, 1>{}); break;
        case 2: body(std::integral_constant<int, 2>{}); break;
        case 3: body(std::integral_constant<int, 3>{}); break;
        case 4: body(std::integral_constant<int, 4>{}); break;
        case 5: body(std::integral_constant<int, 5>{}); break;
        default:
            if constexpr (KMAX > 5) {
                if (nks == 6) body(std::integral_constant<int, 6>{});
                else if (nks == 7) body(std::integral_constant<int, 7>{});
                else body(std::integral_constant<int, 8>{});
            }
    }
}

bool gemm_panel_fits(const GemmDesc &d) {
    return !d.rows_from_kept && ((uintptr_t)d.C & 127) == 0 && d.ldc % 64 == 0 && gemm_panel_chosen(d.E, d.M, d.N, d.K);
}

moe_status_t launch_gemm_panel(const GemmDesc &d, hipStream_t s) {
    if (!gemm_panel_fits(d) || !d.a_xc || !d.b_xc || d.epi != EPI_STORE) {
        set_error("gemm_panel: sizes or operand layouts of another kernel");
        return MOE_ERR_UNSUPPORTED;
    }
    const int np = (d.N + P_N - 1) / P_N, mt = (d.M + P_M - 1) / P_M;
    const int run = gemm_panel_run(d.E, d.M, d.N, d.K), runs = (mt + run - 1) / run, total = d.E * np * runs;
    const dim3 grid((unsigned)((total + 7) / 8 * 8)), block(GEMM_THREADS);
    if (d.K <= 160) hipLaunchKernelGGL(gemm_panel_kernel<5>, grid, block, 0, s, d, np, mt, runs, total);
    else hipLaunchKernelGGL(gemm_panel_kernel<8>, grid, block, 0, s, d, np, mt, runs, total);
    return check_launch("gemm_panel");
}

}  // namespace moe
