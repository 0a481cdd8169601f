// Products for many prompt rows at once: C[R x 256 rows][N] = X W with BOTH operands tiled through LDS, so that a
// weight is read from HBM once per call instead of once per 256 rows (prompt processing, Section 1 stage (i) of the
// rollout; the step before decoding).  The streaming kernel of gemm.hip keeps one weight tile per wavefront in
// registers and is right for up to 256 rows; here a workgroup owns a 256 x 256 (or 256 x 192) tile of the output.
//
// Layouts are the decode step's (hx_internal.h): weights [n_tile][k_step][lane][8], activations of each 256-row block
// [k_step][8 m-groups][lane][8] in that block's workspace.  Both are already in matrix-core operand order, so
// staging is a plain copy of 1-KiB pieces and every LDS read is 16 contiguous bytes per lane (conflict-free).
//
// Workgroup = 8 wavefronts, two per SIMD: 2 x 4 sub-tiles of 128 x 64 (256 columns) or 4 x 2 of 64 x 96 (192 columns).
// A chunk is 2 k-steps: 16 pieces of X and 2 WNT of W, each copied global -> LDS directly by one wavefront, requested two
// chunks ahead into a ring of three stages; one barrier per chunk, passed BEFORE the chunk's last k-step is multiplied,
// so that the first operand reads of the next chunk hide behind those products, as the reads of its second k-step hide
// behind the first.  Reads, copies and products are laid out by hand in groups (sched_barrier).
// What bounds it is the matrix cores' power: with random operands a loop of 32x32x16 products out of registers reaches
// 1 550 TFLOP/s on this card (zeros: 2 410).  7B gate|up, 2048 rows, output stores left out: this kernel 1 253 TFLOP/s;
// with its copies removed 1 442, with its products removed 1 965.  The four-wavefront kernel before it (128 x 128 per
// wavefront, copies through registers) 1 195, and 951 against 1 086 with fp32 stores, which the second wavefront of a
// SIMD overlaps.  Four or five stages, or chunks of 4 k-steps in two stages, were not faster (1 095, 1 088, 995).
//
// Workgroup numbering: consecutive workgroup ids go to different XCDs, so id -> (xcd, slot); the workgroups of one
// XCD take all row blocks of a few column blocks and walk K in step: each XCD's L2 sees every weight once.
#include "hx_internal.h"
#include <algorithm>
#include <mutex>

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

namespace {

constexpr int WIDE_KC = 2;        // k-steps per chunk
constexpr int WIDE_STAGES = 3;
constexpr int WIDE_WAVES = 8;
constexpr int wide_lds_bytes(int wnt) { return WIDE_STAGES * WIDE_KC * (8 + wnt) * 1024; }

struct WideArgs {
    const uint4 *wp;              // packed weights of the matrix
    int k_steps, n_tiles, N;
    const char *xp0;              // block 0's packed activations; block b's are block_stride bytes further
    size_t block_stride;
    int R;                        // 256-row blocks
    float *y0;                    // fp32 output of block 0 ([splits][256][N]), same stride between blocks
    int steps_per_split;
    uint16_t *mp0;                // SiLU(gate)*up output of block 0 (packed activations, 8 m-groups)
};

// WNT: 32-column tiles per workgroup: 8 (a 256 x 256 output tile) or 6 (256 x 192, for products that would otherwise
// leave compute units idle).  Splits hold whole chunks.
template <int WNT, int EPI>
__global__ __launch_bounds__(64 * WIDE_WAVES) void gemm_wide_kernel(WideArgs a) {
    constexpr int KC = WIDE_KC, NST = WIDE_STAGES, WCOL = WNT == 8 ? 4 : 2, WROW = WIDE_WAVES / WCOL, TM = 8 / WROW, TW = WNT / WCOL;
    constexpr int PIECES = KC * (8 + WNT), STAGE_U4 = PIECES * 64;
    constexpr int LPW = (PIECES + WIDE_WAVES - 1) / WIDE_WAVES, FULL = PIECES - (LPW - 1) * WIDE_WAVES;   // waves < FULL copy LPW pieces, the others one less
    static_assert(KC == 2 && TM * TW == (WNT == 8 ? 8 : 6), "the operand registers alternate between two k-steps");
    extern __shared__ u32x4_t lds[];                    // [NST][PIECES][64 lanes]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int w = blockIdx.x, xcd = w & 7, slot = w >> 3;
    const int b = slot % a.R, nbl = (slot / a.R) * 8 + xcd;
    const int NB = (a.n_tiles + WNT - 1) / WNT;
    if (nbl >= NB) return;                              // whole workgroup, before any barrier
    const int nt0 = nbl * WNT;
    const int k_steps = a.k_steps;
    const int k0 = blockIdx.y * a.steps_per_split, k1 = min(k_steps, k0 + a.steps_per_split);
    const int n_chunks = (k1 - k0) / KC;
    const u32x4_t *xp = (const u32x4_t *)(a.xp0 + (size_t)b * a.block_stride);
    // this wavefront's share of the copies of a chunk: wave-uniform pointers that advance by a fixed step per chunk and
    // stop at the split's last one (requests past the end repeat it: never used)
    const bool full = wave < FULL;
    const u32x4_t *ptr[LPW];
    int step[LPW];
    uint32_t dst[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int p = min(i * WIDE_WAVES + wave, PIECES - 1);
        if (p < KC * 8) {
            const int kc = p >> 3, mg = p & 7;
            ptr[i] = xp + ((size_t)(k0 + kc) * 8 + mg) * 64; step[i] = KC * 8 * 64; dst[i] = (kc * 8 + mg) * 1024;
        } else {
            const int q = p - KC * 8, t = q / KC, kc = q % KC;
            const int nt = min(nt0 + t, a.n_tiles - 1);
            ptr[i] = (const u32x4_t *)a.wp + ((size_t)nt * k_steps + k0 + kc) * 64; step[i] = KC * 64; dst[i] = (KC * 8 + kc * WNT + t) * 1024;
        }
    }
    int next_c = 0;                                     // chunk the pointers stand at, and the stage it goes to
    uint32_t next_stage = 0;
    auto copy_one = [&](int i) {
        if (i + 1 < LPW || full) hx_copy_to_lds(ptr[i], lane * 16, next_stage * (STAGE_U4 * 16) + dst[i]);
    };
    auto advance = [&]() {
        ++next_c;
        const int go = -(int)(next_c < n_chunks);       // all ones while the next chunk exists
#pragma unroll
        for (int i = 0; i < LPW; ++i) ptr[i] += step[i] & go;
        next_stage = next_stage + 1 == NST ? 0 : next_stage + 1;
    };
    // this wavefront's copies of the chunk before the last requested one have landed, its LDS reads are done; then everyone's
    auto hand_over = [&]() {
        if (full) __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT((NST - 2) * LPW));
        else __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT((NST - 2) * (LPW - 1)));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    const int wm = wave / WCOL, wn = wave % WCOL;
    f32x16_t acc[TM][TW];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    u32x4_t x[2][TM], wt[2][TW];
    const u32x4_t *base = lds + lane;
    auto read_x = [&](uint32_t stage, int kc, int i) { x[kc & 1][i] = base[stage * STAGE_U4 + (kc * 8 + TM * wm + i) * 64]; };
    auto read_w = [&](uint32_t stage, int kc, int j) { wt[kc & 1][j] = base[stage * STAGE_U4 + (KC * 8 + kc * WNT + wn * TW + j) * 64]; };
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) copy_one(i);
        advance();
    }
    hand_over();                                        // chunk 0 is in its stage
#pragma unroll
    for (int j = 0; j < TW; ++j) read_w(0, 0, j);
#pragma unroll
    for (int i = 0; i < TM; ++i) read_x(0, 0, i);
    uint32_t rd = 0;                                    // stage of chunk c
    for (int c = 0; c < n_chunks; ++c) {
        const uint32_t nrd = rd + 1 == NST ? 0 : rd + 1;
#pragma unroll
        for (int kc = 0; kc < KC; ++kc) {
            // between the products of k-step kc: the operand reads of the next one (behind the barrier that hands over
            // chunk c + 1, if it is that chunk's first), and, in k-step 0, the copies of chunk c + NST - 1 into the stage
            // of chunk c - 1, which everybody has left
            const bool last = kc + 1 == KC;
            if (last) hand_over();
#pragma unroll
            for (int i = 0; i < TM; ++i) {
                if (i == 0) {
#pragma unroll
                    for (int j = 0; j < TW; ++j) read_w(last ? nrd : rd, last ? 0 : kc + 1, j);
                }
                read_x(last ? nrd : rd, last ? 0 : kc + 1, i);
                if (kc == 0) {
#pragma unroll
                    for (int q = 0; q < LPW; ++q) if (q * TM / LPW == i) copy_one(q);
                }
#pragma unroll
                for (int j = 0; j < TW; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, wt[kc & 1][j]),
                                                                        __builtin_bit_cast(bf16x8_t, x[kc & 1][i]), acc[i][j], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (kc == 0) advance();
        }
        rd = nrd;
    }
    __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT(0));        // no copy is in flight when the workgroup gives its LDS back

    // accumulator register r of lane l: batch row m = 32*(TM*wm + i) + l%32, column n = 32*nt + 8*(r/4) + 4*(l/32) + r%4
    const int hl = lane >> 5, ml = lane & 31;
    if (EPI == HX_EPI_PARTIAL) {
        float *y = a.y0 + ((size_t)b * a.block_stride) / 4 + (size_t)blockIdx.y * 256 * a.N;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = 32 * (TM * wm + i) + ml;
#pragma unroll
            for (int j = 0; j < TW; ++j) {
                const int nt = nt0 + wn * TW + j;
                if (nt < a.n_tiles) {
#pragma unroll
                    for (int j4 = 0; j4 < 4; ++j4) {
                        const int n = 32 * nt + 8 * j4 + 4 * hl;
                        if (n < a.N)
                            *(f32x4_t *)(y + (size_t)m * a.N + n) =
                                f32x4_t{acc[i][j][4 * j4], acc[i][j][4 * j4 + 1], acc[i][j][4 * j4 + 2], acc[i][j][4 * j4 + 3]};
                    }
                }
            }
        }
    } else {
        // SiLU(gate) * up: rows 0..15 of a tile are gate columns 16*nt + p, rows 16..31 the matching up columns
        uint16_t *mp = a.mp0 + ((size_t)b * a.block_stride) / 2;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = 32 * (TM * wm + i) + ml;
#pragma unroll
            for (int j = 0; j < TW; ++j) {
                const int nt = nt0 + wn * TW + j;
                if (nt < a.n_tiles) {
#pragma unroll
                    for (int j4 = 0; j4 < 2; ++j4) {
                        float v[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            const float gt = acc[i][j][4 * j4 + q], up = acc[i][j][8 + 4 * j4 + q];
                            v[q] = (gt / (1.0f + expf(-gt))) * up;
                        }
                        uint2 pk;
                        pk.x = hx_cvt_pk_bf16(v[0], v[1]);
                        pk.y = hx_cvt_pk_bf16(v[2], v[3]);
                        *(uint2 *)(mp + hx_xp_index(m, 16 * nt + 8 * j4 + 4 * hl, 8)) = pk;
                    }
                }
            }
        }
    }
}

template <int WNT, int EPI>
int launch_wide(dim3 grid, hipStream_t st, const WideArgs &a) {
    static std::once_flag once;
    static hipError_t configured = hipSuccess;
    std::call_once(once, [] {
        configured = hipFuncSetAttribute((const void *)gemm_wide_kernel<WNT, EPI>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                         wide_lds_bytes(WNT));
    });
    if (configured != hipSuccess) return hx_fail(HX_E_HIP, "hipFuncSetAttribute: %s", hipGetErrorString(configured));
    hipLaunchKernelGGL((gemm_wide_kernel<WNT, EPI>), grid, dim3(64 * WIDE_WAVES), wide_lds_bytes(WNT), st, a);
    return HX_OK;
}

template <int WNT>
int launch_wide_epi(int epilogue, dim3 grid, hipStream_t st, const WideArgs &a) {
    if (epilogue == HX_EPI_PARTIAL) return launch_wide<WNT, HX_EPI_PARTIAL>(grid, st, a);
    return launch_wide<WNT, HX_EPI_SWIGLU>(grid, st, a);
}

}  // namespace

// Tiles per workgroup and, for a product whose consumer sums partials, K-splits: the time of the busiest compute unit
// (rounds x tiles per workgroup x k-steps per split), with a charge per extra split for writing and re-reading its
// partial (measured: a 256 x N fp32 partial per row block is about 4 % of a 3584-deep product) and one per narrower
// tile (it draws more bytes per flop).  Splits hold whole chunks.
hx_wide_plan hx_plan_wide(const hx_matrix *m, int row_blocks, bool partial) {
    const int cus = hx_device_cus();
    hx_wide_plan best{8, 1};
    double best_cost = 1e300;
    for (int wnt : {8, 6}) {
        const int NB = (m->n_tiles + wnt - 1) / wnt;
        for (int s = 1; s <= (partial ? HX_MAX_SPLITS : 1); ++s) {
            if (s > 1 && m->k_steps / s < 32) break;
            const int wgs = NB * row_blocks * s;
            const int rounds = (wgs + cus - 1) / cus;
            const int sps = ((m->k_steps + s - 1) / s + 1) & ~1;
            const double cost = (double)rounds * wnt * sps * (1.0 + 0.04 * (s - 1)) * (1.0 + 0.03 * (8 - wnt));
            if (cost < best_cost - 1e-9) { best_cost = cost; best.wnt = wnt; best.splits = s; }
        }
    }
    return best;
}

// One wide product over `row_blocks` blocks of 256 rows.  xp_off / y_off / mp_off: byte offsets of the packed input,
// the fp32 output ([splits][256][N]) and the SiLU*mul output inside each block's workspace; ws0 = block 0's
// workspace, block_stride bytes between blocks.
int hx_launch_gemm_wide(const hx_engine *e, const hx_matrix *m, int row_blocks, char *ws0, size_t block_stride, size_t xp_off,
                        int epilogue, size_t y_off, size_t mp_off, hx_wide_plan plan, hipStream_t st) {
    int splits = plan.splits;
    const int wnt = plan.wnt;
    if (wnt != 8 && wnt != 6) return hx_fail(HX_E_RANGE, "%d tiles per workgroup: no such wide product", wnt);
    if (m->k_steps % WIDE_KC) return hx_fail(HX_E_SHAPE, "wide products need K to be a multiple of 32, not %d", m->k_steps * 16);
    if (epilogue != HX_EPI_PARTIAL && epilogue != HX_EPI_SWIGLU) return hx_fail(HX_E_RANGE, "epilogue %d has no wide product", epilogue);
    if (epilogue == HX_EPI_SWIGLU) splits = 1;
    if (block_stride % 16) return hx_fail(HX_E_RANGE, "block stride %zu is not a multiple of 16", block_stride);
    WideArgs a;
    a.wp = (const uint4 *)(e->weights + m->offset);
    a.k_steps = m->k_steps; a.n_tiles = m->n_tiles; a.N = m->N;
    a.xp0 = ws0 + xp_off; a.block_stride = block_stride; a.R = row_blocks;
    a.y0 = (float *)(ws0 + y_off);
    a.mp0 = (uint16_t *)(ws0 + mp_off);
    a.steps_per_split = ((m->k_steps + splits - 1) / splits + 1) & ~1;
    const int NB = (m->n_tiles + wnt - 1) / wnt;
    dim3 grid(((NB + 7) / 8) * 8 * row_blocks, splits);
    for (int sp = 0; sp < splits; ++sp)
        if (sp * a.steps_per_split >= m->k_steps) return hx_fail(HX_E_RANGE, "%d splits leave split %d of %d k-steps empty", splits, sp, m->k_steps);
    const int rc = wnt == 8 ? launch_wide_epi<8>(epilogue, grid, st, a) : launch_wide_epi<6>(epilogue, grid, st, a);
    if (rc) return rc;
    HX_CHECK_LAUNCH("gemm_wide");
    return HX_OK;
}
