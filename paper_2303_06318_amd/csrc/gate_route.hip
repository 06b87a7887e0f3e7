// Gate (routing function: linear map, softmax, top-1) and capacity-limited slot assignment.
//
// bf16 tokens: logits = X Wg on the matrix cores in one pass over X.  Wg stays fp32-accurate
// by splitting every weight into three bf16 pieces (hi + mid + lo == w to ~2^-24) and issuing
// three bf16 MFMAs into one fp32 accumulator; bf16 x bf16 products are exact in fp32, so the
// result has fp32 dot-product accuracy while X is streamed once at HBM speed.
// fp32 tokens, and short bf16 token tensors: fp32 matrix instructions on the operands as they are.
//
// Routing: per-token-block histograms of the chosen experts (integer LDS atomics: the result does not
// depend on their order), written by the gate kernel itself (a block = the 64 or 16 tokens of a
// workgroup) and by a small kernel when the logits are given (blocks of 1024 tokens); then one kernel in
// which every block of 1024 tokens adds up the histograms of the tokens before it (all threads in
// parallel, integer atomics again), ranks its own tokens with wave ballots (token order inside a wave
// = lane order) and writes slot / token_of_slot; the last block writes counts and kept.
#include <type_traits>
#include "gemm_bf16_parts.h"
#include "kernel_choice.h"

namespace moe {

// ------------------------------------------------------------------ weight split
// ws layout: 3 planes [Epad][h] bf16 (k contiguous), rows >= E are zero.
__global__ void gate_split_wg_kernel(const float *wg, bf16_t *planes, int h, int E, int Epad) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    int64_t n = (int64_t)Epad * h;
    if (i >= n) return;
    int e = (int)(i / h), k = (int)(i % h);
    float w = e < E ? wg[(int64_t)k * E + e] : 0.f;
    bf16_t hi = f32_to_bf16(w);
    float r1 = w - bf16_to_f32(hi);
    bf16_t mid = f32_to_bf16(r1);
    float r2 = r1 - bf16_to_f32(mid);
    bf16_t lo = f32_to_bf16(r2);
    planes[i] = hi;
    planes[n + i] = mid;
    planes[2 * n + i] = lo;
}

// ------------------------------------------------------------------ choice of the expert, from the logits in LDS
// (all threads of the workgroup of TM tokens; the logits are complete before the call; TPT lanes per token, whose sums
// fix the last bits of the probabilities)
template <int EP, int TM, int THREADS, int TPT = THREADS / TM>
__device__ __forceinline__ void gate_choose(const float (*lg)[EP + 1], int32_t *hist_s, float *probs, int32_t *expert,
                                            float *gate_p, int64_t T, int E, int32_t *hist, int32_t *token_of_slot,
                                            int64_t EC) {
    const int tid = threadIdx.x;
    const int64_t t0 = (int64_t)blockIdx.x * TM;
    if (tid < EP) hist_s[tid] = 0;
    __syncthreads();
    // Softmax and top-1 with TPT adjacent lanes per token: lane `sub` looks at experts sub, sub + TPT, ...;
    // the lanes' candidates are merged by butterfly exchanges (larger logit wins, the lower index among
    // equal ones: the same choice as a left-to-right scan with a strict comparison).
    static_assert(TPT >= 1 && (TPT & (TPT - 1)) == 0 && TPT <= 64 && TM * TPT <= THREADS && (TM * TPT == THREADS || TM * TPT % 64 == 0),
                  "lanes per token, in whole waves");
    const int tt = tid / TPT, sub = TM * TPT == THREADS || tt < TM ? tid % TPT : E;      // waves without tokens look at no expert
    const float *row = &lg[tt][0];
    float best = -__builtin_inff();
    int bi = 0x7fffffff;
    for (int j = sub; j < E; j += TPT) {
        const float v = row[j];
        if (v > best || bi == 0x7fffffff) { best = v; bi = j; }      // strict: the first of equal values stays
    }
#pragma unroll
    for (int o = 1; o < TPT; o <<= 1) {
        const float ov = __shfl_xor(best, o);
        const int oi = __shfl_xor(bi, o);
        if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
    }
    float denom = 0.f;
    for (int j = sub; j < E; j += TPT) denom += expf(row[j] - best);
#pragma unroll
    for (int o = 1; o < TPT; o <<= 1) denom += __shfl_xor(denom, o);
    const float inv = 1.0f / denom;
    const int64_t t = t0 + tt;
    if (t < T) {
        if (probs)
            for (int j = sub; j < E; j += TPT) probs[t * E + j] = expf(row[j] - best) * inv;
        if (sub == 0) {
            expert[t] = bi;
            gate_p[t] = inv;
            atomicAdd(&hist_s[bi], 1);
        }
    }
    __syncthreads();
    // the routing kernel's inputs: this block's histogram, and its share of the inverse map cleared
    if (tid < E) hist[(int64_t)blockIdx.x * E + tid] = hist_s[tid];
    const int64_t per = (EC + gridDim.x - 1) / gridDim.x, i0 = (int64_t)blockIdx.x * per;
    for (int64_t i = i0 + tid; i < i0 + per && i < EC; i += THREADS) token_of_slot[i] = -1;
}

// ------------------------------------------------------------------ fused gate, bf16 tokens, up to 64 experts
// A workgroup of W waves takes 64 tokens; x and the planes of Wg go straight into LDS in k-tiles of 64 through a ring
// of S stages (the loaders of the grouped GEMMs); a wave multiplies RW blocks of 16 tokens with one of the NT expert tiles.
// From two expert tiles on there are eight waves, two per SIMD, so that one reads fragments while the other multiplies (with
// four, LDS reads, MFMAs and the barrier follow each other).  Whole moe_gate call, us, four waves / eight, tokens after 1 GB of
// writes and in cache: 16384 x 2048, E = 64: 59.9 and 48.8 / 58.7 and 42.4; 5000 x 4096, E = 64: 68.8 and 61.6 / 66.4 and 49.5;
// 65536 x 1024, E = 64: 122 and 107 / 115 and 90; 16384 x 2560, E = 32: 55.0 and 37.0 / 54.8 and 35.2.  Not bound by what is in
// flight: a ring of 6 to 16 k-tiles of x costs 0 to 4 us.  One expert tile is four blocks, one for each of four waves:
// 16384 x 4096, E = 16: 69.4 and 35.5.
// MFMA fragments loaded from memory directly are requests of 64 bytes out of 16 rows each, half a cache line (h = 4096,
// E = 16: 38.5 us for the call where the ring takes 32.9).
// The sums of the high planes run in four chains (k-step parity x k-tile parity), those of the other planes in a
// chain of their own that is added last, so that fewer roundings at the size of the result follow each other than with one
// chain.  (Eight waves of which four take either k-step read a third fewer fragments and take 1 to 3 us less with 64 experts,
// but each then adds its low sum to its half of the high one: one more rounding, error against 64 bits at h = 40 4.5e-8 for 4.2e-8.)
template <int NT, int S, int W>
__global__ __launch_bounds__(64 * W) void gate_stream_kernel(const bf16_t *x, const bf16_t *planes, const float *bias,
                                                             float *logits, float *probs, int32_t *expert, float *gate_p,
                                                             int64_t T, int h, int E, int32_t *hist, int32_t *token_of_slot,
                                                             int64_t EC) {
    constexpr int EP = NT * 16, TM = 64, RW = 4 * NT / W;                        // a wave's blocks of 16 tokens
    constexpr int XQ = 8 / W, PQ = (6 * NT + W - 1) / W, L = XQ + PQ;            // 1 KB requests of a wave per k-tile: of x, of the planes
    constexpr int X_BYTES = TM * KC_ROW, STAGE = X_BYTES + PQ * W * 1024;
    static_assert(RW >= 1, "every wave has a block");
    static_assert(TM * (EP + 1) * 4 <= S * STAGE, "the logits are staged in the operand stages");
    __shared__ __attribute__((aligned(1024))) char smem[S * STAGE];
    __shared__ int32_t hist_s[EP];
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(lds_void *)smem;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t t0 = (int64_t)blockIdx.x * TM;
    const int rows = (int)(T - t0 < TM ? T - t0 : TM);
    const i32x4 X = make_rsrc(x + t0 * h, (uint32_t)rows * (uint32_t)h * 2u);
    const i32x4 P = make_rsrc(planes, (uint32_t)(3 * EP) * (uint32_t)h * 2u);
    Loader<false, XQ, 128, W> lx;
    Loader<false, PQ, 128, W> lp;
    lx.init(h, 0, rows, wave, lane);
    lp.init(h, 0, 3 * EP, wave, lane);
    lx.init_k(h, wave, lane);
    lp.kthr = lx.kthr;
    FragAddr<false, 128> fx, fp;
    const int wn = wave % NT, wm = wave / NT * RW;               // the wave's expert tile and first block of 16 tokens (of RW)
    fx.init(wm * 16, lane);
    fp.init(wn * 16, lane);
    auto request = [&](int kt, int stage) {                      // past the end of h: zeros, without memory traffic
        const uint32_t base = smem_addr + stage * STAGE + wave * 1024;
#pragma unroll
        for (int q = 0; q < XQ; ++q) lx.request(X, base, kt * BK, h, q);
#pragma unroll
        for (int q = 0; q < PQ; ++q) lp.request(P, base + X_BYTES, kt * BK, h, q);
    };
    f32x4 hi[4][RW], low[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        low[r] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < 4; ++c) hi[c][r] = low[r];
    }
    const int nk = (h + BK - 1) / BK;
#pragma unroll
    for (int s = 0; s < S - 1; ++s) request(s, s);
    int stage = 0;
    auto k_tile = [&](int kt, auto parity) {
        // k-tile kt has landed (S - 2 newer ones may be outstanding), and every wave has read k-tile kt - 1, whose
        // stage the next request overwrites
        __builtin_amdgcn_sched_barrier(0);
        wait_outstanding<(S - 2) * L>();
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_sched_barrier(0);
        request(kt + S - 1, stage == 0 ? S - 1 : stage - 1);
        const char *tx = smem + stage * STAGE, *tp = tx + X_BYTES;
        bf16x8 a[KS][RW], b[KS][3];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int p = 0; p < 3; ++p) b[ks][p] = fp.read(tp, p * NT, ks);
#pragma unroll
            for (int r = 0; r < RW; ++r) a[ks][r] = fx.read(tx, r, ks);
        }
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
#pragma unroll
            for (int r = 0; r < RW; ++r) low[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][r], b[ks][1], low[r], 0, 0, 0);
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                f32x4 &c = hi[2 * decltype(parity)::value + ks][r];
                c = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][r], b[ks][0], c, 0, 0, 0);
            }
#pragma unroll
            for (int r = 0; r < RW; ++r) low[r] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[ks][r], b[ks][2], low[r], 0, 0, 0);
        }
        stage = stage == S - 1 ? 0 : stage + 1;
    };
    for (int kt = 0; kt < nk; kt += 2) {
        k_tile(kt, std::integral_constant<int, 0>{});
        if (kt + 1 < nk) k_tile(kt + 1, std::integral_constant<int, 1>{});
    }
    __builtin_amdgcn_sched_barrier(0);
    wait_outstanding<0>();                          // nothing may still be writing LDS when it is reused
    __syncthreads();
    // 16x16 result: lane holds column (expert) lane%16, rows (tokens) 4*(lane/16) + v
    float(*lg)[EP + 1] = (float(*)[EP + 1])smem;
#pragma unroll
    for (int r = 0; r < RW; ++r)
#pragma unroll
        for (int v = 0; v < 4; ++v)
            lg[(wm + r) * 16 + (lane >> 4) * 4 + v][wn * 16 + (lane & 15)] = ((hi[0][r][v] + hi[1][r][v]) + (hi[2][r][v] + hi[3][r][v])) + low[r][v];
    __syncthreads();
    for (int idx = tid; idx < TM * E; idx += 64 * W) {
        const int tt = idx / E, j = idx - tt * E;
        float v = lg[tt][j];
        if (bias) v += bias[j];
        lg[tt][j] = v;
        if (t0 + tt < T) logits[(t0 + tt) * E + j] = v;
    }
    gate_choose<EP, TM, 64 * W, 4>(lg, hist_s, probs, expert, gate_p, T, E, hist, token_of_slot, EC);
}

// ------------------------------------------------------------------ fused gate, bf16 tokens, more experts
// (their planes do not fit a ring of k-tiles in LDS)
// Workgroup: NW waves, 16*R tokens.  Wave w takes k-steps w, w+NW, ... (32 k each); the NW partial
// [16R x Epad] tiles are summed through LDS in a fixed order.  The three planes of Wg are read from
// L2 once per workgroup, so R is chosen large enough that this traffic stays below that of X.
template <int NT, int R, int NW, int U>
__global__ __launch_bounds__(64 * NW) void gate_bf16_kernel(const bf16_t *x, const bf16_t *planes, const float *bias,
                                                         float *logits, float *probs, int32_t *expert,
                                                         float *gate_p, int64_t T, int h, int E, int32_t *hist,
                                                         int32_t *token_of_slot, int64_t EC) {
    constexpr int EP = NT * 16;
    constexpr int TM = 16 * R;
    __shared__ float part[NW][TM][EP + 1];
    __shared__ int32_t hist_s[EP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t t0 = (int64_t)blockIdx.x * TM;
    const int i16 = lane & 15, g = lane >> 4;
    const int64_t plane = (int64_t)EP * h;

    f32x4 acc[R][NT];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int n = 0; n < NT; ++n) acc[r][n] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Buffer resources: rows beyond the last token and k beyond h read as zero, so the loop has no
    // branches and U k-steps of loads are in flight per wave before their MFMAs issue.
    constexpr uint32_t OOB = 0x80000000u;
    const int64_t rows = T - t0 < TM ? T - t0 : TM;
    const __amdgpu_buffer_rsrc_t xr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(x + t0 * h), 0, (int)(rows * h * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t pr =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t *>(planes), 0, (int)(3 * plane * 2), 0x00020000);
    const int nsteps = (h + 31) / 32;
    // A batch = U k-steps of this wave: all its requests (R token fragments and 3 NT plane fragments per
    // k-step) are issued together, and the arithmetic of a batch runs while the requests of the next one
    // are in flight: two register sets alternate.  The scheduling barriers keep the compiler from
    // trickling the loads out between the MFMAs (which it does to save registers, leaving a few KB in
    // flight per wave: the kernel is bound by memory latency).  Batches past the end read zeros.
    auto issue = [&](int s, bf16x8(&a)[U][R], bf16x8(&b)[U][NT][3]) {
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (s + NW * u) * 32 + g * 8;
            const uint32_t koff = k < h ? (uint32_t)k * 2u : OOB;
#pragma unroll
            for (int r = 0; r < R; ++r)
                a[u][r] = __builtin_bit_cast(
                    bf16x8, __builtin_amdgcn_raw_buffer_load_b128(xr, (uint32_t)(r * 16 + i16) * h * 2u + koff, 0, 0));
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int p = 0; p < 3; ++p)
                    b[u][n][p] = __builtin_bit_cast(
                        bf16x8, __builtin_amdgcn_raw_buffer_load_b128(
                                    pr, (uint32_t)(p * plane + (int64_t)(n * 16 + i16) * h) * 2u + koff, 0, 0));
        }
    };
    auto multiply = [&](const bf16x8(&a)[U][R], const bf16x8(&b)[U][NT][3]) {
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int n = 0; n < NT; ++n)
#pragma unroll
                for (int p = 0; p < 3; ++p)
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        acc[r][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[u][r], b[u][n][p], acc[r][n], 0, 0, 0);
    };
    // All workgroups read the same Wg planes.  Walking k in the same order, the workgroups of an XCD would ask
    // its L2 for the same few lines at the same time (one or two of its 16 channels serving everybody), so each
    // workgroup starts at a different batch and wraps around.
    constexpr int BS = NW * U;                                   // k-steps per batch of the workgroup
    const int nbatch = (nsteps + BS - 1) / BS;
    const int nbatch2 = (nbatch + 1) & ~1;                       // the loop body holds two batches
    const int rot = (int)((blockIdx.x >> 3) % (unsigned)nbatch2);        // blockIdx / 8: index inside the XCD
    auto first_step = [&](int i) {                               // batch i of this workgroup, rotated; past the end: zeros
        int bi = i + rot;
        bi = bi >= nbatch2 ? bi - nbatch2 : bi;
        return i < nbatch2 ? bi * BS + wave : nsteps;
    };
    constexpr bool TWO_SETS = 2 * U * (R + 3 * NT) * 4 <= 200;   // registers of two batches of fragments
    if constexpr (TWO_SETS) {
        bf16x8 aA[U][R], bA[U][NT][3], aB[U][R], bB[U][NT][3];
        issue(first_step(0), aA, bA);
        for (int i = 0; i < nbatch2; i += 2) {
            issue(first_step(i + 1), aB, bB);
            __builtin_amdgcn_sched_barrier(0);
            multiply(aA, bA);
            __builtin_amdgcn_sched_barrier(0);
            issue(first_step(i + 2), aA, bA);
            __builtin_amdgcn_sched_barrier(0);
            multiply(aB, bB);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {                                                     // many experts: one batch at a time
        bf16x8 aA[U][R], bA[U][NT][3];
        for (int i = 0; i < nbatch2; ++i) {
            issue(first_step(i), aA, bA);
            __builtin_amdgcn_sched_barrier(0);
            multiply(aA, bA);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    // 16x16 result: lane holds column (expert) lane%16, rows (tokens) 4*(lane/16) + v
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int n = 0; n < NT; ++n)
#pragma unroll
            for (int v = 0; v < 4; ++v) part[wave][r * 16 + g * 4 + v][n * 16 + i16] = acc[r][n][v];
    __syncthreads();
    for (int idx = tid; idx < TM * E; idx += 64 * NW) {
        int tt = idx / E, j = idx - tt * E;
        float v = part[0][tt][j];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += part[w][tt][j];
        if (bias) v += bias[j];
        part[0][tt][j] = v;
        if (t0 + tt < T) logits[(t0 + tt) * E + j] = v;
    }
    gate_choose<EP, TM, 64 * NW>(part[0], hist_s, probs, expert, gate_p, T, E, hist, token_of_slot, EC);
}

// ------------------------------------------------------------------ fp32 matrix instruction
// The whole gate of 16 tokens per workgroup on v_mfma_f32_16x16x4_f32, for fp32 tokens, and for bf16 tokens while
// there are few of them: Wg is used as it is stored, without planes and the launch that makes them, and 16 tokens
// per workgroup spread a short token tensor over four times as many compute units as 64 do.
// The 8 waves split the reduction (16 k per step, U consecutive steps in flight: whole cache lines of x); lane l supplies token l % 16 and expert l % 16
// with k = 4 (l / 16) + j to the j-th of four instructions.  A launch-latency kernel: fp32, 2048 tokens, h = 1024, E = 8:
// 42 us for the whole moe_gate call with vector FMAs, a softmax kernel and a histogram kernel, now 11.7.
template <typename XT, int NT, int U>
__global__ __launch_bounds__(512) void gate_direct_kernel(const XT *x, const float *wg, const float *bias, float *logits,
                                                          float *probs, int32_t *expert, float *gate_p, int64_t T, int h,
                                                          int E, int32_t *hist, int32_t *token_of_slot, int64_t EC) {
    constexpr int EP = NT * 16, TM = 16, NW = 8;
    __shared__ float part[NW][TM][EP + 1];
    __shared__ int32_t hist_s[EP];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, i16 = lane & 15, g = lane >> 4;
    const int64_t t0 = (int64_t)blockIdx.x * TM, t = t0 + i16 < T ? t0 + i16 : T - 1;
    const XT *row = x + t * h;
    f32x4 acc[NT];
#pragma unroll
    for (int n = 0; n < NT; ++n) acc[n] = f32x4{0.f, 0.f, 0.f, 0.f};
    const int nsteps = (h + 15) / 16;
    for (int s0 = wave * U; s0 < nsteps; s0 += NW * U) {
        f32x4 a[U];
        float b[U][NT][4];
        // loads from clamped addresses, zeros selected afterwards: no branches between them
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = (s0 + u) * 16 + 4 * g;
            const bool in = k < h;
            const int kc = in ? k : 0;
            a[u] = load4(row + kc);
#pragma unroll
            for (int n = 0; n < NT; ++n) {
                const int e = n * 16 + i16;
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const float w = wg[(int64_t)(kc + j) * E + (e < E ? e : 0)];
                    b[u][n][j] = (in & (e < E)) ? w : 0.f;
                }
            }
            if (!in) a[u] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int n = 0; n < NT; ++n) acc[n] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[u][j], b[u][n][j], acc[n], 0, 0, 0);
    }
#pragma unroll
    for (int n = 0; n < NT; ++n)
#pragma unroll
        for (int v = 0; v < 4; ++v) part[wave][g * 4 + v][n * 16 + i16] = acc[n][v];
    __syncthreads();
    for (int idx = tid; idx < TM * E; idx += 64 * NW) {
        const int tt = idx / E, j = idx - tt * E;
        float v = part[0][tt][j];
#pragma unroll
        for (int w = 1; w < NW; ++w) v += part[w][tt][j];
        if (bias) v += bias[j];
        part[0][tt][j] = v;
        if (t0 + tt < T) logits[(t0 + tt) * E + j] = v;
    }
    gate_choose<EP, TM, 64 * NW>(part[0], hist_s, probs, expert, gate_p, T, E, hist, token_of_slot, EC);
}

// softmax + top-1 from stored logits: 16 adjacent lanes per token, lane `sub` looks at experts sub, sub + 16, ...
// (consecutive lanes read consecutive logits); candidates merged by butterfly exchanges, lower index among equals
constexpr int SM_TPT = 16;
__global__ __launch_bounds__(256) void gate_softmax_top1_kernel(const float *logits, float *probs, int32_t *expert,
                                                                 float *gate_p, int64_t T, int E) {
    const int64_t t = ((int64_t)blockIdx.x * 256 + threadIdx.x) / SM_TPT;
    const int sub = threadIdx.x % SM_TPT;
    const float *row = logits + (t < T ? t : 0) * E;         // lanes past the end work on row 0 and write nothing
    float best = -__builtin_inff();
    int bi = 0x7fffffff;
    for (int j = sub; j < E; j += SM_TPT) {
        const float v = row[j];
        if (v > best || bi == 0x7fffffff) { best = v; bi = j; }
    }
#pragma unroll
    for (int o = 1; o < SM_TPT; o <<= 1) {
        const float ov = __shfl_xor(best, o);
        const int oi = __shfl_xor(bi, o);
        if (ov > best || (ov == best && oi < bi)) { best = ov; bi = oi; }
    }
    float denom = 0.f;
    for (int j = sub; j < E; j += SM_TPT) denom += expf(row[j] - best);
#pragma unroll
    for (int o = 1; o < SM_TPT; o <<= 1) denom += __shfl_xor(denom, o);
    const float inv = 1.0f / denom;
    if (t >= T) return;
    if (probs)
        for (int j = sub; j < E; j += SM_TPT) probs[t * E + j] = expf(row[j] - best) * inv;
    if (sub == 0) {
        expert[t] = bi;
        gate_p[t] = inv;
    }
}

// ------------------------------------------------------------------ routing
constexpr int RB = 1024;   // tokens per routing block
constexpr unsigned ROUTE_DIRECT_BLOCKS = 64;   // up to this many routing blocks, each sums the histograms in front of it itself

__global__ __launch_bounds__(RB) void route_hist_kernel(const int32_t *expert, int32_t *hist, int32_t *token_of_slot,
                                                         int64_t T, int E, int64_t EC) {
    __shared__ int32_t h[256];
    const int tid = threadIdx.x;
    if (tid < E) h[tid] = 0;
    __syncthreads();
    int64_t t = (int64_t)blockIdx.x * RB + tid;
    if (t < T) atomicAdd(&h[expert[t]], 1);
    __syncthreads();
    if (tid < E) hist[(int64_t)blockIdx.x * E + tid] = h[tid];
    for (int64_t i = (int64_t)blockIdx.x * RB + tid; i < EC; i += (int64_t)gridDim.x * RB) token_of_slot[i] = -1;
}

// Many routing blocks (long token tensors): the tokens in front of every routing block, per expert, by one
// pass over the histogram rows instead of every block summing all rows in front of it.  Workgroup e walks the
// routing blocks 1024 at a time: a thread adds up the rows of one block, the workgroup scans the totals
// (wave shuffles, then the 16 wave totals), and the running sum carries over to the next 1024 blocks.
// block_base[b * E + e] = tokens of expert e in routing blocks 0 .. b-1.
__global__ __launch_bounds__(1024) void route_block_base_kernel(const int32_t *hist, int32_t *block_base, int64_t n_rows,
                                                                 int64_t n_blocks, int E, int rows_per_block) {
    __shared__ int32_t wsum[16];
    __shared__ int32_t carry_s;
    const int e = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    if (tid == 0) carry_s = 0;
    __syncthreads();
    for (int64_t b0 = 0; b0 < n_blocks; b0 += 1024) {
        const int64_t b = b0 + tid;
        int32_t tot = 0;
        if (b < n_blocks) {
            const int64_t r0 = b * rows_per_block;
            for (int r = 0; r < rows_per_block && r0 + r < n_rows; ++r) tot += hist[(r0 + r) * E + e];
        }
        int32_t inc = tot;                           // inclusive scan inside the wave
#pragma unroll
        for (int o = 1; o < 64; o <<= 1) {
            const int32_t v = __shfl_up(inc, o);
            if (lane >= o) inc += v;
        }
        if (lane == 63) wsum[wave] = inc;
        __syncthreads();
        int32_t before = carry_s;                    // the carry and the waves in front of this one
        for (int w = 0; w < wave; ++w) before += wsum[w];
        if (b < n_blocks) block_base[b * E + e] = before + inc - tot;
        __syncthreads();
        if (tid == 1023) carry_s = before + inc;
        __syncthreads();
    }
}

// hist holds one row of E counts per `hist_block` tokens (RB is a multiple of hist_block).  block_base: the
// result of route_block_base_kernel, or null (few routing blocks: every block sums the rows in front of it).
__global__ __launch_bounds__(RB) void route_slot_kernel(const int32_t *expert, const int32_t *hist, int32_t *slot,
                                                         int32_t *counts, int32_t *kept, int32_t *token_of_slot,
                                                         int64_t T, int E, int64_t C, int hist_block,
                                                         const int32_t *block_base) {
    __shared__ int32_t base[256];
    __shared__ int32_t wcnt[RB / 64][256];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int b = blockIdx.x;
    for (int i = tid; i < (RB / 64) * 256; i += RB) (&wcnt[0][0])[i] = 0;
    if (tid < 256) base[tid] = 0;
    __syncthreads();
    // tokens before this block: all histogram rows in front of it, summed by all threads at once
    // (consecutive threads read consecutive counts; integer atomics, so the order does not matter)
    if (block_base != nullptr) {
        if (tid < E) base[tid] = block_base[(int64_t)b * E + tid];
    } else {
        const int64_t n_before = (int64_t)b * (RB / hist_block) * E;
        for (int64_t i = tid; i < n_before; i += RB) {
            const int32_t v = hist[i];
            if (v) atomicAdd(&base[(int)(i % E)], v);
        }
    }
    __syncthreads();
    const int64_t t = (int64_t)b * RB + tid;
    const int e = t < T ? expert[t] : -1;
    int rank = 0;
    unsigned long long remaining = __ballot(e >= 0);
    while (remaining) {
        const int leader = __ffsll((long long)remaining) - 1;
        const int e0 = __shfl(e, leader);
        const unsigned long long m = __ballot(e == e0);
        if (e == e0) {
            rank = __popcll(m & ((1ull << lane) - 1ull));
            if (lane == leader) wcnt[wave][e0] = __popcll(m);
        }
        remaining &= ~m;
    }
    __syncthreads();
    if (tid < E) {       // exclusive prefix over the block's waves, in wave order
        int32_t s = base[tid];
        for (int w = 0; w < RB / 64; ++w) {
            int32_t c = wcnt[w][tid];
            wcnt[w][tid] = s;
            s += c;
        }
        if (b == (int)gridDim.x - 1) {
            counts[tid] = s;
            kept[tid] = s < C ? s : (int32_t)C;
        }
    }
    __syncthreads();
    if (e >= 0) {
        const int64_t s = (int64_t)wcnt[wave][e] + rank;
        if (s < C) {
            slot[t] = (int32_t)s;
            token_of_slot[(int64_t)e * C + s] = (int32_t)t;
        } else {
            slot[t] = -1;
        }
    }
}

// ------------------------------------------------------------------ host side
size_t gate_ws_bytes(const moe_shape_t *sh) {
    int NT = 1;
    while (NT * 16 < sh->E) NT *= 2;
    size_t planes = (size_t)3 * NT * 16 * sh->h * 2;
    size_t hist = (size_t)((sh->T + 15) / 16) * sh->E * 4;        // one row per 16 tokens at most (see run_gate)
    size_t bases = (size_t)((sh->T + RB - 1) / RB) * sh->E * 4;   // tokens in front of every routing block
    return ((planes + 255) / 256) * 256 + ((hist + 255) / 256) * 256 + ((bases + 255) / 256) * 256;
}

template <int NT, int R, int NW, int U>
static void launch_gate_bf16(const moe_shape_t *sh, const void *x, const bf16_t *planes, const float *bias,
                             float *logits, float *probs, int32_t *expert, float *gate_p, int32_t *hist,
                             int32_t *token_of_slot, hipStream_t s) {
    const int TM = 16 * R;
    dim3 grid((unsigned)((sh->T + TM - 1) / TM));
    hipLaunchKernelGGL((gate_bf16_kernel<NT, R, NW, U>), grid, dim3(64 * NW), 0, s, (const bf16_t *)x, planes, bias, logits,
                       probs, expert, gate_p, sh->T, sh->h, sh->E, hist, token_of_slot, (int64_t)sh->E * sh->C);
}

template <typename XT>
static void launch_gate_direct(const moe_shape_t *sh, int NT, const void *x, const float *wg, const float *bias,
                               float *logits, float *probs, int32_t *expert, float *gate_p, int32_t *hist,
                               int32_t *token_of_slot, hipStream_t s) {
    const dim3 grid((unsigned)((sh->T + 15) / 16)), block(512);
#define MOE_GATE_DIRECT(NT_, U_)                                                                                         \
    hipLaunchKernelGGL((gate_direct_kernel<XT, NT_, U_>), grid, block, 0, s, (const XT *)x, wg, bias, logits, probs, expert, \
                       gate_p, sh->T, sh->h, sh->E, hist, token_of_slot, (int64_t)sh->E * sh->C)
    switch (NT) {
        case 1: MOE_GATE_DIRECT(1, 8); break;
        case 2: MOE_GATE_DIRECT(2, 4); break;
        case 4: MOE_GATE_DIRECT(4, 4); break;
        case 8: MOE_GATE_DIRECT(8, 1); break;
        default: MOE_GATE_DIRECT(16, 1); break;
    }
#undef MOE_GATE_DIRECT
}

moe_status_t run_gate(const moe_shape_t *sh, const void *x, const float *w_gate, const float *bias, float *logits,
                      float *probs, int32_t *expert, float *gate_p, int32_t *slot, int32_t *counts, int32_t *kept,
                      int32_t *token_of_slot, void *ws, hipStream_t s) {
    int NT = 1;
    while (NT * 16 < sh->E) NT *= 2;
    const size_t planes_bytes = (((size_t)3 * NT * 16 * sh->h * 2 + 255) / 256) * 256;
    bf16_t *planes = (bf16_t *)ws;
    int32_t *hist = (int32_t *)((char *)ws + planes_bytes);
    const int64_t T = sh->T;
    const bool f32 = sh->dtype == MOE_F32;
    if (x == nullptr) {
        hipLaunchKernelGGL(gate_softmax_top1_kernel, dim3((unsigned)((T * SM_TPT + 255) / 256)), dim3(256), 0, s, logits,
                           probs, expert, gate_p, T, sh->E);
    } else if (f32) {
        launch_gate_direct<float>(sh, NT, x, w_gate, bias, logits, probs, expert, gate_p, hist, token_of_slot, s);
    } else if (gate_direct(f32, T)) {
        launch_gate_direct<bf16_t>(sh, NT, x, w_gate, bias, logits, probs, expert, gate_p, hist, token_of_slot, s);
    } else {
        const int64_t n = (int64_t)NT * 16 * sh->h;
        hipLaunchKernelGGL(gate_split_wg_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, w_gate, planes,
                           sh->h, sh->E, NT * 16);
#define MOE_GATE_STREAM(NT_, S_, W_)                                                                                          \
    hipLaunchKernelGGL((gate_stream_kernel<NT_, S_, W_>), dim3((unsigned)((T + 63) / 64)), dim3(64 * W_), 0, s, (const bf16_t *)x, planes, \
                       bias, logits, probs, expert, gate_p, T, sh->h, sh->E, hist, token_of_slot, (int64_t)sh->E * sh->C)
        // launch_gate_bf16: 16-expert tiles, tokens per workgroup / 16, waves, k-steps per batch
        switch (NT) {
            case 1: MOE_GATE_STREAM(1, 4, 4); break;
            case 2: MOE_GATE_STREAM(2, 4, 8); break;
            case 4: MOE_GATE_STREAM(4, 4, 8); break;
            case 8: launch_gate_bf16<8, 1, 4, 1>(sh, x, planes, bias, logits, probs, expert, gate_p, hist, token_of_slot, s); break;
            default: launch_gate_bf16<16, 1, 4, 1>(sh, x, planes, bias, logits, probs, expert, gate_p, hist, token_of_slot, s); break;
        }
#undef MOE_GATE_STREAM
    }
    moe_status_t st = check_launch("gate");
    if (st != MOE_OK) return st;
    const unsigned nb = (unsigned)((T + RB - 1) / RB);
    int hist_block = RB;
    if (x != nullptr) {                          // the gate kernel has written a histogram per workgroup (16 R tokens)
        hist_block = gate_direct(f32, T) || NT >= 8 ? 16 : 64;
    } else {
        hipLaunchKernelGGL(route_hist_kernel, dim3(nb), dim3(RB), 0, s, expert, hist, token_of_slot, T, sh->E,
                           (int64_t)sh->E * sh->C);
    }
    // beyond ROUTE_DIRECT_BLOCKS routing blocks one more small kernel sums the histograms once for all
    int32_t *block_base = nullptr;
    if (nb > ROUTE_DIRECT_BLOCKS) {
        const size_t hist_bytes = (((size_t)((T + 15) / 16) * sh->E * 4 + 255) / 256) * 256;
        block_base = (int32_t *)((char *)hist + hist_bytes);
        hipLaunchKernelGGL(route_block_base_kernel, dim3((unsigned)sh->E), dim3(1024), 0, s, hist, block_base,
                           (T + hist_block - 1) / hist_block, (int64_t)nb, sh->E, RB / hist_block);
    }
    hipLaunchKernelGGL(route_slot_kernel, dim3(nb), dim3(RB), 0, s, expert, hist, slot, counts, kept, token_of_slot,
                       T, sh->E, sh->C, hist_block, block_base);
    return check_launch("route");
}

}  // namespace moe
