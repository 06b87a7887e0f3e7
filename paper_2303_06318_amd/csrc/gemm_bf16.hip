// Grouped bf16 GEMM on gfx950 matrix cores (v_mfma_f32_16x16x32_bf16, fp32 accumulation) for the
// expert FFN: forward (Z = D W1 with fused GeLU and GeLU', Y = H W2), data gradients (dH = dY W2^T
// times the saved GeLU', dD = dZ W1^T) and weight gradients (dW = A^T B over the kept rows).
//
// One workgroup of 512 threads (8 waves, 2 x 4) owns a 256 x 256 output tile of one expert and
// walks K in 64-deep tiles through two to three LDS stages (156 KB).  Each wave owns 64 columns, and 64 rows
// in either 128-row half of the tile: 8 x 4 MFMA blocks of 16 x 16.  Global data goes straight into
// LDS (buffer_load ... lds, 16 bytes per lane, no register staging); out-of-range lanes deliver
// zeros, so ragged row counts and K tails need no branches.  The two waves of a SIMD alternate
// between a memory phase and an MFMA phase, half an iteration apart (see the main loop).
//
// The kernel runs into the chip's power limit (the shader clock sinks from 2.4 to 1.7-1.9 GHz), so what
// counts is energy per flop.  Registers-only loops on random operands sustain 2.11 PFLOP/s with the
// 16 x 16 x 32 instruction and 1.87 with 32 x 32 x 16: per multiply-add it reads and writes half as many
// accumulators.
//
// Operands are taken in the layout the layer stores them in, so no transposed copy is ever made:
//   "KC" operand: the reduction index is contiguous in memory  -> LDS tile [256 x][64 k], 16-byte
//                 LDS reads deliver 8 consecutive k to a lane directly;
//   "XC" operand: the output index is contiguous in memory     -> LDS tile [64 k][x], read with
//                 the LDS transpose load (ds_read_b64_tr_b16), which hands lane i of a 16-lane
//                 group the i-th column of a 4 x 16 block.
// The k-tile is 64 deep because 64 k are 128 bytes of a KC row, one cache line: with 32-deep tiles
// every line was brought from L2 into the CU twice, once for each half (counted, 16384 rows, h = f = 4096: 67 M line
// reads per launch with two KC operands and 50 M with one; now 33.6 M in every layout).
//
// A direct-to-LDS load writes lane L's 16 bytes at base + 16 L, so tiles cannot be padded; bank
// conflicts are avoided by XOR-swizzling the 16-byte granules inside each row instead:
//   KC: granule g of row r sits at position g ^ ((r >> 1) & 7)   (rows are 128 bytes)
//   XC: granule g of k-row k sits at position g ^ ((k & 3) << 2) ^ ((k >> 3 & 1) << 1) (k-rows are 256 bytes
//       for A, whose two 128-column halves are separate, and 512 bytes for B)
// Rows beyond kept[e] are never read (loaded as zero) and never written.
#include <type_traits>
#include "gemm_bf16_parts.h"
#include "kernel_choice.h"

namespace moe {

constexpr int BM = 256, BN = 256;
constexpr int LIGHT_BLOCKS = 4;                // an expert with at most this many 32-row blocks is one "light" tile
constexpr int MAXB = 9;                        // 32-row blocks of a tile when A is a KC operand: 8, or 9 in a "tall" tile
enum { FULL, TALL, PARTIAL };                  // forms of the main loop
// In tiles of up to this many blocks half of the waves have no rows in the tile's upper half and leave its MFMAs out.
// Forward pair, 300 rows per expert (tiles of five blocks), without / with: 16 experts, 4096 x 4096 452 / 412 us, 64 experts,
// 2048 x 2048 504 / 463.  (Leaving out single 16-row blocks instead, a branch each, made that pair 540 us.)
constexpr int PARTIAL_BLOCKS = 6;
constexpr int A_ROWS = MAXB * 32;              // rows of the epilogue staging tile
constexpr int HALF_BYTES = 128 * BK * 2;       // one 128-row (or 128-column) half of A's k-tile (16 KB)
constexpr int X_BYTES = 32 * BK * 2;           // the ninth block of a tall tile (4 KB)
constexpr int B_BYTES = 256 * BK * 2;          // B's k-tile (32 KB)
// LDS map: A's lower half (three stages), upper half (two), ninth block (three), B (two); the stages of a part
// lie next to each other, so that a read's stage is an immediate offset where it is known at compile time
constexpr int A_HI = 0, A_LO = 2 * HALF_BYTES, A_X = A_LO + 3 * HALF_BYTES, B_AT = A_X + 3 * X_BYTES;
constexpr int CLD = BN + 8;                    // epilogue staging row (elements)
constexpr int SMEM_BYTES = A_ROWS * CLD * 2 > B_AT + 2 * B_BYTES ? A_ROWS * CLD * 2 : B_AT + 2 * B_BYTES;

// Tile plan.  An expert's rows are cut into 32-row MFMA blocks, and its nb blocks into
// ceil(nb / maxb) m-tiles of nearly equal block counts (maxb = 9 for a KC A operand, else 8): an
// expert with a few rows more than a multiple of 256 gets "tall" tiles of 9 blocks instead of an
// extra tile that would stream a whole weight panel for a handful of rows.  An expert with at most
// LIGHT_BLOCKS blocks is one "light" tile per column of n-tiles.
// The heavy tiles form one list (expert -- in an order that alternates light and heavy experts --, then
// n-tile, then m-tile, so that the m-tiles of one weight panel are neighbours).  The list is cut into 8 contiguous shares of equal work (tile cost x
// k-tiles: experts differ in size), one per XCD, so that tiles which share a weight panel share an
// L2; each share is followed by an eighth of the light tiles.  kept[] lives on the device, so a
// small kernel writes the plan before every GEMM launch:
//   plan[0..7]   per-share fetch counters (zeroed here, advanced by the GEMM workgroups)
//   plan[8..16]  start of each share in the tile array (plan[16] = number of tiles)
//   plan[32 + 4 t ..]  tile t: {expert | blocks << 8 | light << 12, n-tile, first block, kept[expert]}
// The GEMM kernel is persistent: one workgroup per compute unit takes tiles from the share of its
// own XCD (workgroup ids go round-robin over the XCDs) until that share is empty.
constexpr int PLAN_HDR_INTS = 32;
constexpr int PLAN_THREADS = 1024;
constexpr int MAX_PLANS = 4;
constexpr int PLAN_SLICES = 8;                 // blocks per plan: each recomputes the header and fills a slice of the tiles

// Measured cost of a heavy tile, in half blocks of a full tile's main loop: tiles of seven and eight blocks run through
// the full loop (blocks without rows multiply zeros), nine through the tall loop; up to six save half of the upper
// half's MFMAs (16 experts, 4096 x 4096, forward pair, a tile of the two of 300 rows / of the four of 1024: 103 / 117 us).
__device__ __forceinline__ int tile_cost(int nblk) { return nblk >= 9 ? 19 : nblk > PARTIAL_BLOCKS ? 16 : 14; }

struct PlanDesc {
    const int32_t *kept;
    int32_t *plan;
    int E, M, K, nt, rows_from_kept, maxb, cus_per_xcd, low_tiles;
    uint32_t per_maxb;                            // 2^32 / maxb, rounded up
};
struct PlanArgs {
    PlanDesc p[MAX_PLANS];
};

__global__ __launch_bounds__(PLAN_THREADS) void gemm_plan_kernel(PlanArgs args) {
    const PlanDesc &p = args.p[blockIdx.x];
    __shared__ int s_kept[256], s_nb[256], s_hv[256], s_nk[256], s_eid[256];   // by list position, not by expert
    __shared__ int s_preH[257], s_preL[257];      // tiles of the experts before e (heavy, light)
    __shared__ long long s_preW[257], s_w[256];   // work of the heavy tiles of the experts before e, and of expert e
    __shared__ long long s_w0[256];               // work by expert index, for the ordering
    __shared__ int s_ts[9], s_sl[9];              // split points of the heavy and of the light list
    __shared__ int2 s_cnt[256];                   // m-tiles by expert index: {usual, low | light << 20}; 1023 for more, which never fit
    const int tid = threadIdx.x, nt = p.nt;
    int kx = 0, nb = 0, nkf = 1, hv = 0;
    long long w = 0;
    if (tid < p.E) {
        kx = p.kept[tid];
        const int Mx = p.rows_from_kept ? kx : p.M;
        nb = (Mx + 31) >> 5;
        const int nk = p.rows_from_kept ? 1 : (kx + BK - 1) / BK;
        nkf = nk > 0 ? nk : 1;                    // never 0: every heavy tile must fall into some share
        if (nb > LIGHT_BLOCKS) {  // one column of the expert's tiles: bx tiles of bb + 1 blocks, the others of bb
            hv = (int)__umulhi((uint32_t)(nb + p.maxb - 1), p.per_maxb);      // ceil(nb / maxb), exact up to 2^29
            const int bb = nb / hv, bx = nb - bb * hv;
            w = (long long)(bx * tile_cost(bb + 1) + (hv - bx) * tile_cost(bb)) * nkf * nt;
        }
        s_w0[tid] = w;
        const int low = (nb + LIGHT_BLOCKS - 1) / LIGHT_BLOCKS;
        s_cnt[tid] = hv > 0 ? make_int2(hv < 1023 ? hv : 1023, low < 1023 ? low : 1023) : make_int2(low, low << 20);
    }
    __syncthreads();
    if (tid < p.E) {
        // Order of the experts in the list: lightest, heaviest, second lightest, second heaviest, ...  A share
        // mostly holds whole experts (their tiles share weight panels), and with few experts per share the
        // shares of a plain 0, 1, 2, ... order differ by the spread of the experts' sizes; pairing the extremes
        // evens them out.  Any order gives the same results: tiles are independent.
        int r = 0, usual = 0, rest = 0;
        for (int e = 0; e < p.E; ++e) {
            r += (s_w0[e] < w || (s_w0[e] == w && e < tid)) ? 1 : 0;
            usual += s_cnt[e].x;
            rest += s_cnt[e].y;
        }
        // Few tiles (the host counts them by capacity; with an uneven router most experts may hold next to nothing): tiles of at
        // most LIGHT_BLOCKS blocks, twice as many and half as much MFMA work in each, by the rule of kernel_choice.h.  The usual
        // tiles' work still orders the experts, and one round's shares are equal in tile count.
        if (hv > 0 && gemm_low_tiles(usual * nt, (rest & 0xfffff) * nt, (rest >> 20) * nt, p.cus_per_xcd, p.low_tiles))
            hv = (nb + LIGHT_BLOCKS - 1) / LIGHT_BLOCKS;
        const int pos = r < (p.E + 1) / 2 ? 2 * r : 2 * (p.E - 1 - r) + 1;
        s_eid[pos] = tid;
        s_kept[pos] = kx;
        s_nb[pos] = nb;
        s_hv[pos] = hv;
        s_nk[pos] = nkf;
        s_w[pos] = w;
    }
    __syncthreads();
    if (tid < p.E) {              // exclusive prefix sums, every thread for itself (E <= 256: no dependent chain)
        int h = 0, l = 0;
        long long wp = 0;
        for (int e = 0; e < tid; ++e) {
            h += s_hv[e] * nt;
            l += (s_nb[e] > 0 && s_nb[e] <= LIGHT_BLOCKS) ? nt : 0;
            wp += s_w[e];
        }
        s_preH[tid] = h; s_preL[tid] = l; s_preW[tid] = wp;
        if (tid == p.E - 1) {
            s_preH[p.E] = h + s_hv[tid] * nt;
            s_preL[p.E] = l + ((s_nb[tid] > 0 && s_nb[tid] <= LIGHT_BLOCKS) ? nt : 0);
            s_preW[p.E] = wp + s_w[tid];
        }
    }
    __syncthreads();
    const int nH = s_preH[p.E], nL = s_preL[p.E];
    const long long WH = s_preW[p.E];
    if (tid <= 8) {
        // heavy tiles whose preceding work is below th = tid WH / 8
        const long long th = (tid * WH) >> 3;
        int res = 0;
        if (tid == 8) res = nH;
        else if (th > 0) {
            int e = 0;
            while (s_preW[e + 1] < th) ++e;       // s_preW[e] < th <= s_preW[e + 1], so expert e is heavy
            const int mts = s_hv[e], bb = s_nb[e] / mts, bx = s_nb[e] - bb * mts;
            const int c1 = tile_cost(bb + 1), c0t = tile_cost(bb);
            const long long wc = (long long)(bx * c1 + (mts - bx) * c0t) * s_nk[e];   // work of one column of its tiles
            const long long r = th - s_preW[e];                      // 1 .. wc nt
            const int c0 = (int)((r - 1) / wc);                       // whole columns of n-tiles before
            const int rem = (int)(((r - 1) - c0 * wc) / s_nk[e]);     // cost inside the column, 0 .. wc / nk - 1
            // tiles of the column whose preceding cost is at most rem
            int cm = rem < bx * c1 ? rem / c1 + 1 : bx + (rem - bx * c1) / c0t + 1;
            cm = cm < mts ? cm : mts;
            res = s_preH[e] + c0 * mts + cm;
        }
        // A share is worked off by the cus_per_xcd compute units of one XCD, a tile at a time: a few
        // tiles beyond a multiple of that number cost a whole extra round, so the split points are
        // moved to the nearest multiple (this matters when there are only a few rounds).  With no more
        // tiles than compute units there is one round if no share holds more tiles than its XCD has
        // units: the shares are then equal in tile count, which also uses the memory paths of all XCDs
        // instead of filling two or three of them.
        if (tid > 0 && tid < 8) {
            const int c = p.cus_per_xcd;
            if (nH <= 8 * c) {
                res = (tid * nH) >> 3;
            } else {
                res = (res + c / 2) / c * c;
                res = res < nH ? res : nH;
            }
        }
        s_ts[tid] = res;
        s_sl[tid] = (int)(((long long)tid * nL) >> 3);
    }
    __syncthreads();
    if (blockIdx.y == 0) {
        if (tid < 8) p.plan[tid] = 0;
        if (tid <= 8) p.plan[8 + tid] = s_ts[tid] + s_sl[tid];
    }
    int4 *tiles = (int4 *)(p.plan + PLAN_HDR_INTS);
    for (int t = blockIdx.y * PLAN_THREADS + tid; t < nH + nL; t += PLAN_THREADS * PLAN_SLICES) {
        const bool light = t >= nH;
        const int q = light ? t - nH : t;
        const int *pre = light ? s_preL : s_preH;
        int lo = 0, hi = p.E;                     // largest e with pre[e] <= q (experts without tiles are skipped)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (pre[mid] <= q) lo = mid; else hi = mid;
        }
        const int e = lo, r = q - pre[e];
        const int *split = light ? s_sl : s_ts;
        int x = 0;
        while (split[x + 1] <= q) ++x;
        int4 ent;
        int pos;
        if (light) {
            ent = make_int4(s_eid[e] | (s_nb[e] << 8) | (1 << 12), r, 0, s_kept[e]);
            pos = s_ts[x + 1] + s_sl[x] + (q - s_sl[x]);
        } else {
            const int mts = s_hv[e];
            // the first nb % mts tiles of a column hold one block more than the others
            const int bb = s_nb[e] / mts, bx = s_nb[e] - bb * mts;
            int nti = r / mts, mti = r - nti * mts;                        // m fastest
            if (bx == 0 && mts > 4) {
                // many equal m-tiles (the weight gradients): n fastest inside groups of 8 n-tiles, so that
                // the 32 tiles an XCD works on together are 4 m-tiles x 8 n-tiles (12 operand panels)
                // rather than 16 x 2 (18 panels)
                const int ng = r / (mts * 8), rr = r - ng * (mts * 8);
                const int gw = nt - ng * 8 < 8 ? nt - ng * 8 : 8;
                mti = rr / gw;
                nti = ng * 8 + (rr - mti * gw);
            }
            const int nblk = bb + (mti < bx ? 1 : 0), blk0 = mti * bb + (mti < bx ? mti : bx);
            ent = make_int4(s_eid[e] | (nblk << 8), nti, blk0, s_kept[e]);
            pos = s_ts[x] + s_sl[x] + (q - s_ts[x]);
        }
        tiles[pos] = ent;
    }
}

template <bool AXC, bool BXC, int EPI>
__global__ __launch_bounds__(GEMM_THREADS) void gemm_bf16_kernel(GemmDesc d) {
    __shared__ __attribute__((aligned(1024))) char smem[SMEM_BYTES];
    __shared__ int s_next[8];                    // the tile fetched by thread 0: its plan entry, its index; thread 0's state
    __shared__ int s_ctok[A_ROWS];               // scattered result: target row of each tile row (-1: none) ...
    __shared__ float s_cscl[A_ROWS];             // ... and its scale
    const uint32_t smem_addr = (uint32_t)(uintptr_t)(lds_void *)smem;
    const int tid0 = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid0 >> 6);
    const int wr = wave >> 2, wn = (wave & 3) * 64;   // the wave's rows: wr * 64 .. + 63 of either 128-row half
    FragAddr<AXC, 128> fa;
    FragAddr<BXC, 256> fb;
    fa.init(wr * 64, tid0 & 63);
    // Column block of B fragment j: j ^ swap.  With B n-contiguous the blocks are numbered so that fragments 0 and 1 are
    // the ninth row block's columns in either wave row: a choice between fragments inside the loop made the compiler hold
    // that block's accumulators twice, and spill (forward pair, 16 experts x 288 rows, 4096 x 4096: 390 us, now 320).
    const int swap = BXC ? 2 * wr : 0;
    fb.init(wn, tid0 & 63, swap);
    int32_t *plan = (int32_t *)d.plan;
    const int4 *tiles = (const int4 *)(plan + PLAN_HDR_INTS);
    const int myx = blockIdx.x & 7;
    // Tile fetch (thread 0): the workgroup draws tiles from the share of its own XCD until the
    // share's counter passes its size.  (Taking tiles from other shares at the end was tried and
    // lost: such a tile finds nothing of its panels in the local L2 and runs at half speed.)
    // Thread 0's own state, the next tile and its share's first tile and size, rests in s_next[5 .. 7]: in registers
    // it would take three vector registers of every lane through the main loop.
    auto fetch_blocking = [&](int cur_first, int cur_cnt) {
        const int t = atomicAdd(plan + myx, 1);
        return t < cur_cnt ? cur_first + t : -1;
    };
    auto publish = [&](int idx, const int4 &ent) {
        s_next[0] = ent.x; s_next[1] = ent.y; s_next[2] = ent.z; s_next[3] = ent.w; s_next[4] = idx;
    };
    // Fetches run two tiles ahead and only during epilogues: the number of the tile after next is
    // requested and the plan entry of the next tile is loaded while this tile's result is written,
    // so that no such request is outstanding during a main loop (whose explicit vmcnt waits count
    // only the loop's own loads).
    if (tid0 == 0) {
        const int cur_first = plan[8 + myx], cur_cnt = plan[9 + myx] - cur_first;
        const int idx = fetch_blocking(cur_first, cur_cnt);
        publish(idx, idx >= 0 ? tiles[idx] : make_int4(0, 0, 0, 0));
        s_next[5] = idx >= 0 ? fetch_blocking(cur_first, cur_cnt) : -1;
        s_next[6] = cur_first;
        s_next[7] = cur_cnt;
    }
    __syncthreads();

  for (;;) {
    // The thread index is made opaque per tile: otherwise the compiler hoists the lane-dependent
    // address arithmetic of the loaders and of the epilogue out of this loop and keeps it in
    // registers through the main loop, which has none to spare.
    int tid = tid0;
    asm volatile("" : "+v"(tid));
    const int lane = tid & 63;
    const int tile_idx = __builtin_amdgcn_readfirstlane(s_next[4]);
    if (tile_idx < 0) break;
    const int ent0 = __builtin_amdgcn_readfirstlane(s_next[0]);
    const int e = ent0 & 255, nblk = (ent0 >> 8) & 15;
    const int nti = __builtin_amdgcn_readfirstlane(s_next[1]);
    const int blk0 = __builtin_amdgcn_readfirstlane(s_next[2]);
    const int kept = __builtin_amdgcn_readfirstlane(s_next[3]);
    const bool tall = !AXC && nblk == MAXB;

    const int Me = d.rows_from_kept ? kept : d.M;
    const int Ke = d.rows_from_kept ? d.K : kept;
    const int m0 = blk0 * 32, n0 = nti * BN;
    const int mlim = Me < m0 + nblk * 32 ? Me : m0 + nblk * 32;     // rows [m0, mlim) are this tile's

    // gathered A (dispatch folded in, or the row shares of duplicate token dropping): one array for all
    // experts, rows through this expert's index slice or the share arithmetic
    RowMap amap = {nullptr, 0, 0, 0};
    if (!AXC && d.a_index != nullptr) amap.index = d.a_index + (int64_t)e * d.M;
    else if (!AXC && d.a_dtd_g > 1) { amap.G = d.a_dtd_g; amap.share_rows = d.E * d.a_dtd_cg; amap.base = e * d.a_dtd_cg; }
    const bool a_index = amap.mapped();
    const bf16_t *Ap = a_index ? (const bf16_t *)d.A : (const bf16_t *)d.A + (int64_t)e * d.strideA;
    const bf16_t *Bp = (const bf16_t *)d.B + (int64_t)e * d.strideB;
    // extent of this expert's operands in bytes (rows x row length)
    const uint32_t a_bytes = a_index ? (uint32_t)d.a_rows * (uint32_t)d.lda * 2u
                                     : (uint32_t)(AXC ? Ke : Me) * (uint32_t)d.lda * 2u;
    // scattered result (combine folded in): target row and scale of each of the tile's rows, through LDS
    const bool scatter = EPI == EPI_STORE && d.c_index != nullptr;
    if (scatter && tid < A_ROWS) {
        const int gm = m0 + tid;
        const bool ok = gm < mlim;
        s_ctok[tid] = ok ? d.c_index[(int64_t)e * d.M + gm] : -1;
        s_cscl[tid] = ok ? d.c_scale[(int64_t)e * d.M + gm] : 0.f;
    }
    const uint32_t b_bytes = (uint32_t)(BXC ? Ke : d.N) * (uint32_t)d.ldb * 2u;
    const i32x4 A = make_rsrc(Ap, a_bytes), B = make_rsrc(Bp, b_bytes);

    f32x4 acc[8][4];                                 // rows: 4 blocks of the lower half, 4 of the upper one
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
    // Ninth 32-row block of a tall tile (rows 256..287): its 8 column blocks of 32 go one to each wave, wave
    // (wr, wn) taking the columns wn + 32 wr .. + 31, which it holds B fragments for.
    f32x4 accx[2][2];                                // set by the loop of tall tiles only

    const int nk = (Ke + BK - 1) / BK;
    // Fragments of one k-tile: all of B (kept through both MFMA phases), one half of A at a time, and one
    // k-step of the ninth block.
    bf16x8 af[4][KS], bf[4][KS], ax[2];
    Loader<AXC, 2, 128> lo, hi;
    Loader<BXC, 4, 256> lb;
    lo.init(d.lda, m0, mlim, wave, lane, amap);
    hi.init(d.lda, m0 + 128, mlim, wave, lane, amap);
    lb.init(d.ldb, n0, d.N, wave, lane);
    lo.init_k(Ke, wave, lane);
    hi.kthr = lo.kthr;
    lb.init_k(Ke, wave, lane);
    // tall tile: the four 1 KB chunks of rows 256..287 are loaded by waves 0, 5, 2 and 7 (one on each SIMD,
    // two of each ping-pong group)
    const int xw = ((wave >> 2) ^ (wave & 1)) == 0 ? (wave & 3) : -1;
    const bool has_x = !AXC && tall && xw >= 0;
    uint32_t offx = OOB;
    if (has_x) {
        const int row = 256 + 8 * xw + (lane >> 3);
        const int g = (lane & 7) ^ ((row >> 1) & 7);
        const int gx = m0 + row;
        if (a_index) {
            const int src = gx < mlim ? amap.row(gx) : -1;
            offx = src >= 0 ? ((uint32_t)src * d.lda + g * 8) * 2u : OOB;
        } else {
            offx = gx < mlim ? ((uint32_t)gx * d.lda + g * 8) * 2u : OOB;
        }
    }
    auto read_b = [&](int stage) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int j = 0; j < 4; ++j) bf[j][ks] = fb.read(smem + B_AT + stage * B_BYTES, j, ks);
    };
    auto read_a = [&](const char *half) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks)
#pragma unroll
            for (int i = 0; i < 4; ++i) af[i][ks] = fa.read(half, i, ks);
    };
    // the 4 MFMAs of one block row and k-step; nothing is moved across (loads are placed between them)
    auto mma_row = [&](int half, int ks, int i) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            acc[4 * half + i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[j][ks], af[i][ks], acc[4 * half + i][j], 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    // ninth block: k-step ks of the k-tile in stage s3
    auto read_x = [&](int ks, int s3) {
        const char *t = smem + A_X + s3 * X_BYTES - wr * 64 * KC_ROW;
        ax[0] = fa.read(t, 0, ks);
        ax[1] = fa.read(t, 1, ks);
    };
    auto mma_x = [&](int ks) {
        auto cols = [&](auto first) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    accx[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(bf[decltype(first)::value + j][ks], ax[i], accx[i][j], 0, 0, 0);
        };
        if (BXC || wr == 0) cols(std::integral_constant<int, 0>{});          // (see swap)
        else cols(std::integral_constant<int, 2>{});
    };
    // one of this wave's 1 KB requests (2 for either half of A, 4 for B, per k-tile)
    auto request_lo = [&](int kt, int s3, int q) {
        lo.request(A, smem_addr + A_LO + s3 * HALF_BYTES + wave * 1024, kt * BK, d.lda, q);
    };
    auto request_hi = [&](int kt, int stage, int q) {
        hi.request(A, smem_addr + A_HI + stage * HALF_BYTES + wave * 1024, kt * BK, d.lda, q);
    };
    auto request_b = [&](int kt, int stage, int q) {
        lb.request(B, smem_addr + B_AT + stage * B_BYTES + wave * 1024, kt * BK, d.ldb, q);
    };
    auto request_x = [&](int kt, int s3) {            // tall tiles, waves 0, 5, 2 and 7 only
        const int k0 = kt * BK;
        // (xw = wave % 4: the same swizzle, and so the same bound, as in the wave's other chunks)
        load_to_lds(A, smem_addr + A_X + s3 * X_BYTES + xw * 1024, k0 < lo.kthr ? offx : OOB, (uint32_t)k0 * 2u);
    };
    // Main loop, "ping-pong" form.  Waves w and w+4 share a SIMD.  For every k-tile each wave goes through
    // two memory phases M and two compute phases C, every phase ending in a workgroup barrier:
    //   M1(kt): read all of B and A's lower half of tile kt
    //   C1(kt): 32 MFMAs, rows of the lower half;  between them, request A's upper half of tile kt+1 and its
    //           lower half of tile kt+2
    //   M2(kt): read A's upper half of tile kt
    //   C2(kt): 32 MFMAs, rows of the upper half;  between them, request B of tile kt+2 (a wave without rows there,
    //           in a partial tile: the requests only)
    // Waves 4-7 run one phase behind waves 0-3 (one extra barrier up front, matched by one extra barrier of
    // waves 0-3 at the end), so on every SIMD one wave feeds the matrix pipe while the other waits on the LDS.
    // The requests sit between the MFMAs, 4 per compute phase, because the path from L2 into LDS takes about
    // 29 cycles per KB: in bursts at the start of the memory phases they outlasted the 512 cycles of MFMAs
    // beside them.  With this placement and the 16 x 16 x 32 instruction, 16 experts x 1024 rows, h = f = 4096:
    // GEMM2 442 -> 409 us, dD 434 -> 398, dW 509 -> 470.
    //  - A part is overwritten only after every wave has read it.  Upper half of tile kt+1, over tile kt-1: read
    //    in M2(kt-1), which waves 4-7 leave (lgkmcnt(0), barrier) before waves 0-3 enter M1(kt).  Lower half of
    //    tile kt+2, over tile kt-1 (three stages): read in M1(kt-1).  B of tile kt+2, over tile kt: read in
    //    M1(kt), which waves 4-7 leave before waves 0-3 enter M2(kt).
    //  - A part is complete before any wave reads it: every wave waits for its own loads at the end of each
    //    phase, leaving outstanding the newest ones, which the two phases to come do not read.  Request order
    //    per k-tile: C1: [ninth block of kt+2,] upper half of kt+1 (2), lower half of kt+2 (2); C2: B of kt+2 (4).
    //      M1(kt+1) reads B of kt+1 (C2(kt-1)) and the lower half (older): at the end of C2(kt) 8 newer loads
    //      exist, at the end of M2(kt) (the late group's place when the early one enters M1(kt+1)) 4.
    //      M2(kt) reads the upper half of kt (C1(kt-1)): 2 + 4 newer loads at the end of M1(kt), 10 at C1(kt).
    //  - The ninth block of a tall tile is read in both memory phases (one k-step each) and has three stages like
    //    the lower half; the four waves that load it have one load more between the others in C1.
    const bool late_group = wave >= 4;
    const bool upper = mlim - m0 > 128 + wr * 64;        // this wave has rows in the upper half
    auto main_loop = [&](auto formc) {
        constexpr bool TALLV = decltype(formc)::value == TALL;
        // With B n-contiguous a third copy of the loop makes the others spill: there the full loop serves partial tiles too.
        constexpr bool CHECK = decltype(formc)::value == PARTIAL || (BXC && !AXC && !TALLV);
        const bool five = TALLV && has_x;                // this wave issues 5 loads in C1 (the ninth block's first)
        auto end_M = [&](auto nc, auto more) {           // at most nc loads outstanding (+ 1 with five), and lgkmcnt(0)
            __builtin_amdgcn_sched_barrier(0);
            if (decltype(more)::value && five) wait_outstanding<decltype(nc)::value + 1>();
            else wait_outstanding<decltype(nc)::value>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            __builtin_amdgcn_s_setprio(1);
        };
        auto end_C = [&](auto nc) {
            __builtin_amdgcn_s_setprio(0);
            __builtin_amdgcn_sched_barrier(0);
            if (five) wait_outstanding<decltype(nc)::value + 1, false>();
            else wait_outstanding<decltype(nc)::value, false>();
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
        };
        if (TALLV) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j) accx[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        }
        if (nk == 0) return;
        // prologue: the requests of the k-tiles -2 and -1 in the loop's order
        if (five) request_x(0, 0);
        request_lo(0, 0, 0); request_lo(0, 0, 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) request_b(0, 0, q);
        if (five) request_x(1, 1);
        request_hi(0, 0, 0); request_hi(0, 0, 1);
        request_lo(1, 1, 0); request_lo(1, 1, 1);
#pragma unroll
        for (int q = 0; q < 4; ++q) request_b(1, 1, q);
        wait_outstanding<8, false>();          // lower half and B of tile 0 (and its ninth block) have landed
        __builtin_amdgcn_s_barrier();
        if (late_group) __builtin_amdgcn_s_barrier();
        int s3 = 0;                                      // kt % 3
        auto k_tile = [&](int kt, auto stagec) {
            constexpr int stage = decltype(stagec)::value;
            const int s3_next2 = s3 == 0 ? 2 : s3 - 1;   // (kt + 2) % 3
            read_b(stage);
            read_a(smem + A_LO + s3 * HALF_BYTES);
            if (TALLV) read_x(0, s3);
            end_M(std::integral_constant<int, 6>{}, std::false_type{});
            mma_row(0, 0, 0);
            if (TALLV) {
                if (five) request_x(kt + 2, s3_next2);
            }
            mma_row(0, 0, 1);
            request_hi(kt + 1, stage ^ 1, 0);
            mma_row(0, 0, 2); mma_row(0, 0, 3);
            request_hi(kt + 1, stage ^ 1, 1);
            mma_row(0, 1, 0); mma_row(0, 1, 1);
            request_lo(kt + 2, s3_next2, 0);
            mma_row(0, 1, 2);
            request_lo(kt + 2, s3_next2, 1);
            mma_row(0, 1, 3);
            if (TALLV) mma_x(0);
            end_C(std::integral_constant<int, 10>{});
            // a wave without rows in the upper half has no MFMAs in C2; the branch lies in the memory phase, where the
            // wave waits anyway (at the start of C2 it cost full tiles 1 %)
            if (!CHECK || __builtin_expect(upper, true)) {
                read_a(smem + A_HI + stage * HALF_BYTES);
                if (TALLV) read_x(1, s3);
                end_M(std::integral_constant<int, 4>{}, std::true_type{});
                mma_row(1, 0, 0); mma_row(1, 0, 1);
                request_b(kt + 2, stage, 0);
                mma_row(1, 0, 2); mma_row(1, 0, 3);
                request_b(kt + 2, stage, 1);
                mma_row(1, 1, 0); mma_row(1, 1, 1);
                request_b(kt + 2, stage, 2);
                mma_row(1, 1, 2);
                request_b(kt + 2, stage, 3);
                mma_row(1, 1, 3);
            } else {
                end_M(std::integral_constant<int, 4>{}, std::true_type{});
#pragma unroll
                for (int q = 0; q < 4; ++q) request_b(kt + 2, stage, q);
            }
            if (TALLV) mma_x(1);
            end_C(std::integral_constant<int, 8>{});
            s3 = s3 == 2 ? 0 : s3 + 1;
        };
        int kt = 0;
        for (; kt + 1 < nk; kt += 2) {
            k_tile(kt, std::integral_constant<int, 0>{});
            k_tile(kt + 1, std::integral_constant<int, 1>{});
        }
        if (kt < nk) k_tile(kt, std::integral_constant<int, 0>{});
        if (!late_group) __builtin_amdgcn_s_barrier();
    };
    if constexpr (AXC) main_loop(std::integral_constant<int, FULL>{});
    else if (tall) main_loop(std::integral_constant<int, TALL>{});
    else if (!BXC && nblk <= PARTIAL_BLOCKS) main_loop(std::integral_constant<int, PARTIAL>{});
    else main_loop(std::integral_constant<int, FULL>{});          // blocks without rows multiply zeros
    wait_outstanding<0>();              // nothing may still be writing LDS when it is reused
    __syncthreads();
    int4 ent_next = make_int4(0, 0, 0, 0);
    int t_after = 0, idx_n = -1;
    if (tid == 0) {                                  // both arrive during the epilogue
        idx_n = s_next[5];
        if (idx_n >= 0) {
            ent_next = tiles[idx_n];
            t_after = atomicAdd(plan + myx, 1);
        }
    }

    // Epilogue.  The MFMAs were issued with the operands swapped (B fragment first), so the
    // accumulators hold the transposed block: lane owns output row m = lane%16 and four consecutive
    // columns n = (lane/16)*4 + v of every 16 x 16 block.  The tile is
    // converted to bf16, staged in LDS (the operand stages are free now; reads still in flight
    // from the loop's last prefetch are never used) and written out as full 512-byte rows.
    bf16_t *C = (bf16_t *)d.C + (int64_t)e * d.strideC;
    bf16_t *st = (bf16_t *)smem;
    const int act = d.act;
    auto col_of = [&](int j) { return j < 2 ? wn + swap * 16 + j * 16 : wn - swap * 16 + j * 16; };   // wn + (j ^ swap) * 16
    auto for_each_quad = [&](auto fn) {
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int j = 0; j < 4; ++j)
                fn(st + ((i >> 2) * 128 + wr * 64 + (i & 3) * 16 + (lane & 15)) * CLD + col_of(j) + (lane >> 4) * 4, acc[i][j]);
        if (tall) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    fn(st + (256 + i * 16 + (lane & 15)) * CLD + wn + wr * 32 + j * 16 + (lane >> 4) * 4, accx[i][j]);
        }
    };
    auto put4 = [](bf16_t *pos, const f32x4 &v) {
        bf16x4 o = {(bf16_t)v[0], (bf16_t)v[1], (bf16_t)v[2], (bf16_t)v[3]};
        *(bf16x4 *)pos = o;
    };
    auto flush = [&](bf16_t *out) {
        __syncthreads();
        auto pass = [&](int p) {
            const int row = (tid >> 5) + 16 * p, gm = m0 + row, gn = n0 + (tid & 31) * 8;
            const u32x4 v = *(const u32x4 *)(st + row * CLD + (tid & 31) * 8);
            u32x4 *dst = (u32x4 *)(out + (int64_t)gm * d.ldc + gn);
            if (gm < mlim && gn < d.N) {
                // weight gradients are not read soon and would displace the operand panels from the L2
                if (AXC) __builtin_nontemporal_store(v, dst);
                else *dst = v;
            }
        };
#pragma unroll
        for (int p = 0; p < 16; ++p) pass(p);
        if (tall) { pass(16); pass(17); }
    };
    if (EPI == EPI_STORE) {
        for_each_quad([&](bf16_t *pos, const f32x4 &v) { put4(pos, v); });
        if (!scatter) {
            flush(C);
        } else {
            // result row (if C is given) and the scaled row at its target: the staged bf16 value times the
            // scale, rounded again -- exactly what a separate combine pass over C would produce
            bf16_t *S = (bf16_t *)d.C_scatter;
            const bool keep = d.C != nullptr;
            __syncthreads();
            auto spass = [&](int p) {
                const int row = (tid >> 5) + 16 * p, gm = m0 + row, gn = n0 + (tid & 31) * 8;
                const u32x4 v = *(const u32x4 *)(st + row * CLD + (tid & 31) * 8);
                const int trg = s_ctok[row];
                const float scl = s_cscl[row];
                if (gm < mlim && gn < d.N) {
                    if (keep) *(u32x4 *)(C + (int64_t)gm * d.ldc + gn) = v;
                    if (trg >= 0) {
                        const bf16x8 b = __builtin_bit_cast(bf16x8, v);
                        bf16x8 o;
#pragma unroll
                        for (int q = 0; q < 8; ++q) o[q] = (bf16_t)((float)b[q] * scl);
                        *(u32x4 *)(S + (int64_t)trg * d.ldc + gn) = __builtin_bit_cast(u32x4, o);
                    }
                }
            };
#pragma unroll
            for (int p = 0; p < 16; ++p) spass(p);
            if (tall) { spass(16); spass(17); }
        }
    } else if (EPI == EPI_GELU) {
        // The activation is a compile-time constant inside (one branch per tile, not per element).
        auto gelu_stage = [&](auto actc) __attribute__((always_inline)) {
            constexpr int ACT = decltype(actc)::value;
            if (d.C2) {
                // Second output act'(z), which is all the backward pass needs of z.  Both values are
                // computed in one go and staged side by side, so the tile goes out in three parts of
                // at most 128 rows (two staging areas of 128 rows fit the LDS): the tile's lower half,
                // its upper half, and the ninth block row of a tall tile.
                bf16_t *stG = st, *stH = st + 128 * CLD;
                bf16_t *outG = (bf16_t *)d.C2 + (int64_t)e * d.strideC;
                auto both4 = [&](const f32x4 &a, int srow, int col) __attribute__((always_inline)) {
                    f32x4 g, hv;
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        float h1, g1;
                        gelu_both_fast(a[q], ACT, h1, g1);
                        hv[q] = h1;
                        g[q] = g1;
                    }
                    const int off = srow * CLD + col + (lane >> 4) * 4;
                    put4(stG + off, g);
                    put4(stH + off, hv);
                };
                auto flush_part = [&](int part, int nrows) __attribute__((always_inline)) {
                    __syncthreads();
                    for (int p = 0; p < nrows / 16; ++p) {
                        const int sr = (tid >> 5) + 16 * p;
                        const int gm = m0 + part * 128 + sr, gn = n0 + (tid & 31) * 8;
                        const u32x4 vg = *(const u32x4 *)(stG + sr * CLD + (tid & 31) * 8);
                        const u32x4 vh = *(const u32x4 *)(stH + sr * CLD + (tid & 31) * 8);
                        if (gm < mlim && gn < d.N) {
                            *(u32x4 *)(outG + (int64_t)gm * d.ldc + gn) = vg;
                            *(u32x4 *)(C + (int64_t)gm * d.ldc + gn) = vh;
                        }
                    }
                    __syncthreads();
                };
#pragma unroll
                for (int part = 0; part < 2; ++part) {
#pragma unroll
                    for (int i = 0; i < 4; ++i)
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            both4(acc[4 * part + i][j], wr * 64 + i * 16 + (lane & 15), col_of(j));
                    flush_part(part, 128);
                }
                if (tall) {
#pragma unroll
                    for (int i = 0; i < 2; ++i)
#pragma unroll
                        for (int j = 0; j < 2; ++j) both4(accx[i][j], i * 16 + (lane & 15), wn + wr * 32 + j * 16);
                    flush_part(2, 32);
                }
            } else {
                for_each_quad([&](bf16_t *pos, const f32x4 &v) {
                    f32x4 g = {gelu_fast(v[0], ACT), gelu_fast(v[1], ACT), gelu_fast(v[2], ACT), gelu_fast(v[3], ACT)};
                    put4(pos, g);
                });
            }
        };
        if (act == MOE_GELU_TANH) gelu_stage(std::integral_constant<int, MOE_GELU_TANH>{});
        else gelu_stage(std::integral_constant<int, MOE_GELU_ERF>{});
        if (!d.C2) flush(C);
    } else {
        const bf16_t *Zin = (const bf16_t *)d.Zin + (int64_t)e * d.strideC;
        auto zpass = [&](int p) {
            const int row = (tid >> 5) + 16 * p, gm = m0 + row, gn = n0 + (tid & 31) * 8;
            u32x4 v = {0u, 0u, 0u, 0u};
            if (gm < mlim && gn < d.N) v = *(const u32x4 *)(Zin + (int64_t)gm * d.ldc + gn);
            *(u32x4 *)(st + row * CLD + (tid & 31) * 8) = v;
        };
#pragma unroll
        for (int p = 0; p < 16; ++p) zpass(p);
        if (tall) { zpass(16); zpass(17); }
        __syncthreads();
        for_each_quad([&](bf16_t *pos, const f32x4 &v) {     // Zin holds act'(z)
            const bf16x4 z = *(const bf16x4 *)pos;
            f32x4 g = {v[0] * (float)z[0], v[1] * (float)z[1], v[2] * (float)z[2], v[3] * (float)z[3]};
            put4(pos, g);
        });
        flush(C);
    }
    // the staging tile is reused by the next tile; s_next was last read before the main loop
    if (tid == 0) {
        publish(idx_n, ent_next);
        s_next[5] = (idx_n >= 0 && t_after < s_next[7]) ? s_next[6] + t_after : -1;
    }
    __syncthreads();
  }
}

static int num_compute_units() {
    static int cus = 0;                          // same value from every thread that races here
    if (cus == 0) {
        int dev = 0, n = 0;
        if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
            n <= 0)
            n = 256;
        cus = n;
    }
    return cus;
}

size_t gemm_bf16_plan_bytes(const GemmDesc &d) {
    const int64_t mt = (d.M + BM - 1) / BM, nt = (d.N + BN - 1) / BN;
    return (size_t)(PLAN_HDR_INTS * 4 + 16 * (int64_t)d.E * mt * nt + 255) / 256 * 256;
}

moe_status_t launch_gemm_bf16_plans(const GemmDesc *descs, int n, hipStream_t s) {
    if (n < 1 || n > MAX_PLANS) {
        set_error("gemm_bf16: %d plans in one launch", n);
        return MOE_ERR_INVALID_ARG;
    }
    PlanArgs args = {};
    int np = 0;
    for (int i = 0; i < n; ++i) {
        const GemmDesc &d = descs[i];
        if (gemm_rows_fits(d) || gemm_panel_fits(d) || gemm_wgrad_fits(d)) continue;
        if (d.plan == nullptr || d.E > 256) {
            set_error("gemm_bf16: no plan buffer, or more than 256 experts");
            return MOE_ERR_INVALID_ARG;
        }
        PlanDesc &p = args.p[np++];
        p.kept = d.kept; p.plan = (int32_t *)d.plan;
        p.E = d.E; p.M = d.M; p.K = d.K; p.nt = (d.N + BN - 1) / BN;
        p.rows_from_kept = d.rows_from_kept; p.maxb = d.a_xc ? 8 : MAXB;
        p.per_maxb = (uint32_t)((((uint64_t)1 << 32) + p.maxb - 1) / p.maxb);
        p.cus_per_xcd = num_compute_units() / 8 > 0 ? num_compute_units() / 8 : 1;
        if (p.rows_from_kept) {
            const int64_t room = (int64_t)p.E * ((p.M + BM - 1) / BM) * p.nt;          // tiles of the plan buffer
            p.low_tiles = (int)(room < 8 * p.cus_per_xcd ? room : 8 * p.cus_per_xcd);  // more never fit one round
        }
    }
    if (np == 0) return MOE_OK;
    hipLaunchKernelGGL(gemm_plan_kernel, dim3(np, PLAN_SLICES), dim3(PLAN_THREADS), 0, s, args);
    return check_launch("gemm_plan");
}

template <bool AXC, bool BXC, int EPI>
static void launch_one(const GemmDesc &d, hipStream_t s) {
    // persistent: one workgroup per compute unit (the LDS footprint allows no second one)
    hipLaunchKernelGGL((gemm_bf16_kernel<AXC, BXC, EPI>), dim3((unsigned)num_compute_units()), dim3(GEMM_THREADS), 0, s, d);
}

// The plan in d.plan must have been written (launch_gemm_bf16_plans) earlier on the same stream,
// for this descriptor's kept, E, M, N, K, rows_from_kept and A layout; a plan serves one launch.
moe_status_t launch_gemm_bf16(const GemmDesc &d, hipStream_t s) {
    if (gemm_rows_fits(d)) return launch_gemm_rows(d, s);
    if (gemm_panel_fits(d)) return launch_gemm_panel(d, s);
    if (gemm_wgrad_fits(d)) return launch_gemm_wgrad(d, s);
    if (d.plan == nullptr) {
        set_error("gemm_bf16: no plan");
        return MOE_ERR_INVALID_ARG;
    }
    if (!d.a_xc && d.b_xc && d.epi == EPI_GELU) launch_one<false, true, EPI_GELU>(d, s);          // forward: A [M,K], B [K,N]
    else if (!d.a_xc && d.b_xc && d.epi == EPI_STORE) launch_one<false, true, EPI_STORE>(d, s);
    else if (!d.a_xc && !d.b_xc && d.epi == EPI_DGELU) launch_one<false, false, EPI_DGELU>(d, s);  // data gradient: A [M,K], B [N,K]
    else if (!d.a_xc && !d.b_xc && d.epi == EPI_STORE) launch_one<false, false, EPI_STORE>(d, s);
    else if (d.a_xc && d.b_xc && d.epi == EPI_STORE) launch_one<true, true, EPI_STORE>(d, s);      // weight gradient: A [K,M], B [K,N]
    else {
        set_error("gemm_bf16: combination of operand layouts and epilogue not built");
        return MOE_ERR_UNSUPPORTED;
    }
    return check_launch("gemm_bf16");
}

}  // namespace moe
