// Products for many prompt rows at once: C[R x 256 rows][N] = X W with BOTH operands tiled through LDS, so that a
// weight is read from HBM once per call instead of once per 256 rows (prompt processing, Section 1 stage (i) of the
// rollout; the step before decoding), and for decode batches and prompt chunks of 129 to 256 rows.  The streaming kernel
// of gemm.hip keeps one weight tile per wavefront in registers and is right for up to 128 rows; here a workgroup owns a
// tile of the output of 256 rows by 128 to 256 columns.
//
// Layouts are the decode step's (hx_internal.h): weights [n_tile][k_step][lane][8], activations of each 256-row block
// [k_step][8 m-groups][lane][8] in that block's workspace.  Both are already in matrix-core operand order, so
// staging is a plain copy of 1-KiB pieces and every LDS read is 16 contiguous bytes per lane (conflict-free).
//
// Workgroup = 8 wavefronts, two per SIMD: 2 x 4 sub-tiles of 128 x 64 (256 columns), 4 x 2 of 64 x 96 or 64 x 64
// (192, 128 columns), or 8 of 32 rows by all 224 or 160 columns.
// A chunk is 2 k-steps: 16 pieces of X and 2 WNT of W, each copied global -> LDS directly by one wavefront, requested two
// chunks ahead into a ring of three stages (five ahead into six: wide_stages); one barrier per chunk, passed BEFORE the chunk's last k-step is multiplied,
// so that the first operand reads of the next chunk hide behind those products, as the reads of its second k-step (16x16x32: of the
// second half of the longer operand) hide behind the first.  Reads, copies and products are laid out by hand in groups (sched_barrier).
// What bounds it: the LDS path (operand reads and the copies that fill the stages) and the matrix cores, which cover each other only in
// part, and a last round that is paid whole (7B gate|up over 2048 rows 4.6 rounds, 14B over 4864 8.02).  us as it runs | without products | with
// copies for the first stages only | without output stores, each side with random operands: 7B, 2048 rows gate|up 449 | 307 | 428 | 409; 14B, 4864 rows gate|up
// 1053 | 816 | 953 | 990, down 499 | 417 | 434 | 456, QKV 306 | 275 | 264 | 280.  The same instructions out of registers would take 267, 662, 331 and 168
// (2 080 TFLOP/s; with 32x32x16 ones 1 810, on one card, which is why this kernel has the former): the reads alone take longer than that.
// A chunk of two k-steps is one 16x16x32 product's k, and its operands are read from the same stages (lane l: row l % 16 of a half group, k octet l / 16), so
// the layouts stay; the sums come out the same, bit for bit.  Six and more tiles per workgroup use them, us, 32x32x16 -> 16x16x32 in turn:
// 7B, 2048 rows gate|up 453 -> 422 (1.28 PFLOP/s), down 227 -> 215, O 52.3 -> 49.4; 14B, 4864 rows gate|up 1146 -> 1096, down 551 -> 501
// (1.38), QKV 322 -> 305.  Narrower tiles keep 32x32x16: most of them wait for memory (32x32x16 | 16x16x32: 1.5B gate|up 25.5 | 26.5 at 256 rows,
// 63.5 | 65.5 at 1024), but 7B QKV over 2048 rows, in five, does not (66.6 | 63.5).  The LM head, whose epilogue is written for that accumulator, has it, too.
// Four wavefronts of 128 x 128, one per SIMD, move a quarter less through LDS and are slower (575 against 437 in one session).

// Workgroup numbering: consecutive workgroup ids go to different XCDs, so XCD x takes the x-th eighth of the work, row
// blocks fastest, splits slowest: its workgroups take all row blocks of a few column blocks and walk K in step, so each XCD's L2 sees
// (nearly) every weight once, and all XCDs have the same number of workgroups.  (Whole column blocks dealt to the XCDs
// in turn left four of them with half as much again as the others at 20 column blocks: 724 us instead of 610 for the
// 14B down product over 4864 rows in two splits.)
#include "hx_internal.h"
#include "lm_epilogue.h"
#include <algorithm>
#include <mutex>

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

namespace {

constexpr int WIDE_KC = 2;        // k-steps per chunk
constexpr int WIDE_WAVES = 8;
// Stages of the ring: six of the narrow tiles, three of the others.  The narrow ones run where a product is small or has one
// block of rows, at a third of the matrix cores' rate, and wait for memory: six stages there, us at 201 rows: 7B gate|up
// 77 -> 75, down 50 -> 44, 14B gate|up 88 -> 82, O 25 -> 22, QKV 31.5 -> 30; 7B O, 1024 rows 34 -> 31.  Beyond 5 tiles the matrix
// cores bind: 2048 and 4864 rows 0.4 % slower with five stages.  Gate|up of more workgroups than compute units has three, too:
// five stages are requested anew at the start of every workgroup, which its few k-steps do not repay (us, three | six stages:
// 1.5B, 1024 rows 60.1 | 62.7; hidden size 896, 2048 rows 38.9 | 43.2; 2048, 768 rows 75.4 | 77.1; one workgroup for a compute
// unit: 1.5B, 256 rows 28 | 26).  The others of more than one round, whose k-steps are many, gain: 7B QKV, 4096 rows 141 | 135.
// A single block of at most 192 rows (narrow tiles: what such blocks get): the m-groups without rows are neither copied nor
// multiplied nor stored.  us at 129 / 192 rows, weights from memory: 14B gate|up 80.8 / 81.1 -> 68.5 / 73.4, down 45.0 / 46.6 -> 40.6 / 43.8, QKV 29.9 /
// 29.8 -> 25.6 / 26.1, O 25.1 / 24.4 -> 21.8 / 22.0; 7B gate|up 73.9 / 73.4 -> 65.9 / 68.9, down 45.9 / 44.8 -> 38.5 / 40.5; at 193 to 224 rows, where one
// group is left out, alike.  And its gate|up of 128 and more k-steps copies the weights non-temporally (a single block is all that reads
// them): 14B 68.5 / 73.4 / 82.6 at 129 / 192 / 256 rows -> 62.2 / 68.0 / 79.5, 7B 65.9 / 68.9 / 75.3 -> 63.7 / 63.2 / 70.0, 192 k-steps 43.4 / 48.6 / 50.7 -> 39.8 /
// 43.2 / 47.6, 128 30.7 / 35.6 / 41.0 -> 31.0 / 34.0 / 39.2, but 96 23.4 / 24.6 / 25.9 -> 24.6 / 25.6 / 27.1, and the split products 1 to 3 us slower.
constexpr int WIDE_PART_GROUPS = 6, WIDE_ONCE_STEPS = 128;
constexpr int wide_stages(int wnt, bool rounds) { return wnt <= 5 && !rounds ? 6 : 3; }
constexpr int wide_lds_bytes(int wnt, int stages) { return stages * WIDE_KC * (8 + wnt) * 1024; }

struct WideArgs {
    const uint4 *wp;              // packed weights of the matrix
    int k_steps, n_tiles, N;
    const char *xp0;              // block 0's packed activations; block b's are block_stride bytes further
    size_t block_stride;
    int R;                        // 256-row blocks
    float *y0;                    // fp32 output of block 0 ([splits][256][N]), same stride between blocks
    int steps_per_split, splits;
    uint16_t *mp0;                // SiLU(gate)*up output of block 0 (packed activations, 8 m-groups)
    int groups;                   // m-groups that hold rows: 8, of a single block 5 to 8
    hx_lm_args lm;                // LM head (one block)
};

// WNT: 32-column tiles per workgroup, 4 to 8 (a 256 x 128 to 256 x 256 output tile).  Splits hold whole chunks; ODD:
// but for the last, whose second k-step is missing.  (As a run-time condition in the loop this cost the narrow tiles 11 %.)
// PART: one block whose last m-groups hold no rows; wavefronts that have no others only copy.  ONCE: weights non-temporally.
template <int WNT, int EPI, bool ODD, int NST, bool PART = false, bool ONCE = false>
__global__ __launch_bounds__(64 * WIDE_WAVES) void gemm_wide_kernel(WideArgs a) {
    constexpr int KC = WIDE_KC, WCOL = WNT == 8 ? 4 : (WNT % 2 ? 1 : 2), WROW = WIDE_WAVES / WCOL, TM = 8 / WROW,
                  TW = WNT / WCOL;
    constexpr int PIECES = KC * (8 + WNT), STAGE_U4 = PIECES * 64;
    constexpr int LPW = (PIECES + WIDE_WAVES - 1) / WIDE_WAVES, FULL = PIECES - (LPW - 1) * WIDE_WAVES;   // waves < FULL copy LPW pieces, the others one less
    static_assert(KC == 2 && TM * TW == WNT, "the operand registers alternate between two k-steps");
    extern __shared__ u32x4_t lds[];                    // [NST][PIECES][64 lanes]
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NB = (a.n_tiles + WNT - 1) / WNT;
    const int item = (int)(blockIdx.x & 7) * (int)(gridDim.x >> 3) + (int)(blockIdx.x >> 3);
    const int split = item / (NB * a.R), tile = item - split * (NB * a.R);
    if (split >= a.splits) return;                      // whole workgroup, before any barrier
    const int b = tile % a.R, nbl = tile / a.R;
    const int nt0 = nbl * WNT;
    const int k_steps = a.k_steps;
    const int k0 = split * a.steps_per_split, k1 = min(k_steps, k0 + a.steps_per_split);
    const int n_chunks = (k1 - k0 + 1) / KC;            // an odd last k-step (a down product): its partner counts as zero
    const u32x4_t *xp = (const u32x4_t *)(a.xp0 + (size_t)b * a.block_stride);
    // This wavefront's share of the copies of a chunk: piece 8 i + wave, the 2 RG of X in the first two rounds and those of W behind;
    // wave-uniform pointers that advance by a fixed step per chunk and stop at the split's last one (requests past the end repeat
    // it: never used).  PART: X ends within the second round.
    const int RG = PART ? a.groups : 8;
    const bool full = FULL == WIDE_WAVES || wave < FULL, second = !PART || wave < KC * RG - WIDE_WAVES;
    const u32x4_t *ptr[LPW];
    int step[LPW];
    uint32_t dst[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int p = i * WIDE_WAVES + wave;
        if (i < 2) {
            const int x = min(p, KC * RG - 1), kc = PART ? x >= RG : x >> 3, mg = x - kc * RG;
            ptr[i] = xp + ((size_t)(k0 + kc) * 8 + mg) * 64; step[i] = KC * 8 * 64; dst[i] = (kc * 8 + mg) * 1024;
        } else {
            const int q = min(p, PIECES - 1) - KC * 8, t = q / KC, kc = q % KC;
            const int nt = min(nt0 + t, a.n_tiles - 1);
            ptr[i] = (const u32x4_t *)a.wp + ((size_t)nt * k_steps + k0 + kc) * 64; step[i] = KC * 64; dst[i] = (KC * 8 + kc * WNT + t) * 1024;
        }
    }
    int next_c = 0;                                     // chunk the pointers stand at, and the stage it goes to
    uint32_t next_stage = 0;
    auto copy_one = [&](int i) {
        if (i == 1 ? second : i + 1 < LPW || full) {
            if (ONCE && i >= 2) hx_copy_to_lds_once(ptr[i], lane * 16, next_stage * (STAGE_U4 * 16) + dst[i]);
            else hx_copy_to_lds(ptr[i], lane * 16, next_stage * (STAGE_U4 * 16) + dst[i]);
        }
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
        if (full && second) __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT((NST - 2) * LPW));
        else if (!PART || full || second) __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT((NST - 2) * (LPW - 1)));
        else __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT((NST - 2) * (LPW - 2)));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
    };
    const int wm = wave / WCOL, wn = wave % WCOL;
#pragma unroll
    for (int s = 0; s < NST - 1; ++s) {
#pragma unroll
        for (int i = 0; i < LPW; ++i) copy_one(i);
        advance();
    }
    hand_over();                                        // chunk 0 is in its stage
    if constexpr (WNT >= 6 && EPI <= HX_EPI_SWIGLU) {
        // 16x16x32 products: a chunk is their k; a 32-row group or a column tile is two fragments.  The longer operand is held once and
        // read half by half, the shorter one twice.
        constexpr int XF = 2 * TM, WF = 2 * TW;
        constexpr bool XL = XF >= WF;
        constexpr int NL = XL ? XF : WF, NS = XL ? WF : XF, H = NL / 2;
        static_assert(NS == 2 || NS == 4, "the hold behind the last products names every fragment of the shorter operand");
        f32x4_t acc[XF][WF];
#pragma unroll
        for (int i = 0; i < XF; ++i)
#pragma unroll
            for (int j = 0; j < WF; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        u32x4_t lo[NL], sh[2][NS];
        // lane l of a fragment: row l % 16 of its half, k octet l / 16 (k-step l / 32 of the chunk, half l / 16 % 2 of it)
        const int row = lane & 15, oct = lane >> 4;
        const u32x4_t *xbase = lds + ((oct >> 1) * 8 + TM * wm) * 64 + (oct & 1) * 32 + row;
        const u32x4_t *wbase = lds + (KC * 8 + (oct >> 1) * WNT + wn * TW) * 64 + (oct & 1) * 32 + row;
        auto frag = [&](bool x, uint32_t stage, int f) { return (x ? xbase : wbase)[stage * STAGE_U4 + (f >> 1) * 64 + (f & 1) * 16]; };
        auto read_l = [&](uint32_t stage, int f) { lo[f] = frag(XL, stage, f); };
        auto read_s = [&](uint32_t stage, int set, int f) { sh[set][f] = frag(!XL, stage, f); };
        auto multiply = [&](int l, int set) {
#pragma unroll
            for (int f = 0; f < NS; ++f) {
                f32x4_t &d = XL ? acc[l][f] : acc[f][l];
                d = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, XL ? sh[set][f] : lo[l]),
                                                            __builtin_bit_cast(bf16x8_t, XL ? lo[l] : sh[set][f]), d, 0, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        // the second k-step of an odd split's last chunk may hold anything: its lanes of both operands are zero
        auto clear = [&](u32x4_t &v) {
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = lane < 32 ? v[k] : 0u;
        };
#pragma unroll
        for (int f = 0; f < NS; ++f) read_s(0, 0, f);
#pragma unroll
        for (int l = 0; l < H; ++l) read_l(0, l);
        uint32_t rd = 0;                                // stage of chunk c
        auto chunk = [&](int c, int set) {
            const uint32_t nrd = rd + 1 == NST ? 0 : rd + 1;
            const bool odd = ODD && 2 * c + 1 >= k1 - k0;
            if (odd) {
#pragma unroll
                for (int f = 0; f < NS; ++f) clear(sh[set][f]);
#pragma unroll
                for (int l = 0; l < H; ++l) clear(lo[l]);
            }
            // first half: beside its products the reads of the second, and the copies of chunk c + NST - 1 into the stage of
            // chunk c - 1, which everybody has left
#pragma unroll
            for (int l = 0; l < H; ++l) {
                read_l(rd, H + l);
#pragma unroll
                for (int q = 0; q < LPW; ++q) if (q * H / LPW == l) copy_one(q);
                multiply(l, set);
            }
            advance();
            hand_over();
            if (odd) {
#pragma unroll
                for (int l = H; l < NL; ++l) clear(lo[l]);
            }
            // second half: beside its products the first reads of chunk c + 1
#pragma unroll
            for (int l = H; l < NL; ++l) {
#pragma unroll
                for (int f = 0; f < NS; ++f) if (f * H / NS == l - H) read_s(nrd, set ^ 1, f);
                read_l(nrd, l - H);
                multiply(l, set);
            }
            rd = nrd;
        };
        int c = 0;
        for (; c + 1 < n_chunks; c += 2) { chunk(c, 0); chunk(c + 1, 1); }
        if (c < n_chunks) chunk(c, 0);
        // nothing may be written into the last products' operands a few slots behind them (hx_hold_operands)
        f32x4_t &end = XL ? acc[NL - 1][NS - 1] : acc[NS - 1][NL - 1];
        asm volatile("s_nop 7" : "+v"(end) : "v"(lo[NL - 1]), "v"(lo[NL - 2]), "v"(lo[NL - 3]), "v"(sh[0][0]), "v"(sh[0][NS / 2 - 1]), "v"(sh[0][NS / 2]),
                     "v"(sh[0][NS - 1]), "v"(sh[1][0]), "v"(sh[1][NS / 2 - 1]), "v"(sh[1][NS / 2]), "v"(sh[1][NS - 1]));
        __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT(0));    // no copy is in flight when the workgroup gives its LDS back

        // register r of lane l of acc[i][j]: batch row 32 * TM * wm + 16 * i + l % 16, column 32 * (nt0 + wn * TW) + 16 * j + 4 * (l / 16) + r
        const int nt1 = nt0 + wn * TW, m0 = 32 * TM * wm + row;
        if (EPI == HX_EPI_PARTIAL) {
            float *y = a.y0 + ((size_t)b * a.block_stride) / 4 + (size_t)split * 256 * a.N;
#pragma unroll
            for (int i = 0; i < XF; ++i)
#pragma unroll
                for (int j = 0; j < WF; ++j) {
                    const int n = 32 * nt1 + 16 * j + 4 * oct;
                    if (n < a.N) *(f32x4_t *)(y + (size_t)(m0 + 16 * i) * a.N + n) = acc[i][j];
                }
        } else {
            // SiLU(gate) * up: the first 16 columns of a tile are gate columns 16 * nt + p, the others the matching up columns
            uint16_t *mp = a.mp0 + ((size_t)b * a.block_stride) / 2;
#pragma unroll
            for (int i = 0; i < XF; ++i)
#pragma unroll
                for (int j = 0; j < TW; ++j) {
                    if (nt1 + j >= a.n_tiles) continue;
                    float v[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float gt = acc[i][2 * j][q], up = acc[i][2 * j + 1][q];
                        v[q] = (gt / (1.0f + expf(-gt))) * up;
                    }
                    *(uint2 *)(mp + hx_xp_index(m0 + 16 * i, 16 * (nt1 + j) + 4 * oct, 8)) =
                        make_uint2(hx_cvt_pk_bf16(v[0], v[1]), hx_cvt_pk_bf16(v[2], v[3]));
                }
        }
        return;
    }
    f32x16_t acc[TM][TW];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TW; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    u32x4_t x[2][TM], wt[2][TW];
    const u32x4_t *base = lds + lane;
    if (PART && TM * wm >= RG) {                        // no rows: its copies, and everyone's barriers
        for (int c = 0; c < n_chunks; ++c) {
#pragma unroll
            for (int q = 0; q < LPW; ++q) copy_one(q);
            advance();
            hand_over();
        }
        __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT(0));
        return;
    }
    auto read_x = [&](uint32_t stage, int kc, int i) { x[kc & 1][i] = base[stage * STAGE_U4 + (kc * 8 + TM * wm + i) * 64]; };
    auto read_w = [&](uint32_t stage, int kc, int j) { wt[kc & 1][j] = base[stage * STAGE_U4 + (KC * 8 + kc * WNT + wn * TW + j) * 64]; };
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
            if (last) {
                hand_over();
                if (ODD && 2 * c + 1 >= k1 - k0) {          // both, as what lies behind either may hold anything; the copies stay
#pragma unroll
                    for (int i = 0; i < TM; ++i) x[kc & 1][i] = u32x4_t{0u, 0u, 0u, 0u};   // inside the buffers: a down
#pragma unroll
                    for (int j = 0; j < TW; ++j) wt[kc & 1][j] = u32x4_t{0u, 0u, 0u, 0u};  // matrix and its input are followed by others
                }
            }
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
        float *y = a.y0 + ((size_t)b * a.block_stride) / 4 + (size_t)split * 256 * a.N;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = 32 * (TM * wm + i) + ml;
            if (PART && TM * wm + i >= RG) continue;
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
    } else if (EPI == HX_EPI_SWIGLU) {
        // SiLU(gate) * up: rows 0..15 of a tile are gate columns 16*nt + p, rows 16..31 the matching up columns
        uint16_t *mp = a.mp0 + ((size_t)b * a.block_stride) / 2;
#pragma unroll
        for (int i = 0; i < TM; ++i) {
            const int m = 32 * (TM * wm + i) + ml;
            if (PART && TM * wm + i >= RG) continue;
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
    } else {
        // one copy of the tile's code, the accumulators moved up behind it
#pragma unroll 1
        for (int i = 0; i < TM; ++i) {
            const int m0 = 32 * (TM * wm + i);
#pragma unroll 1
            for (int j = 0; j < TW; ++j) {
                const int nt = nt0 + wn * TW + j;
                if (nt < a.n_tiles && m0 < a.lm.M) {
                    if (EPI == HX_EPI_LOGITS) hx_lm_greedy_tile(a.lm, acc[0][0], m0 + ml, nt, lane);
                    else                      hx_lm_sample_tile<false>(a.lm, acc[0][0], m0 + ml, nt, lane);
                }
#pragma unroll
                for (int k = 0; k + 1 < TM * TW; ++k) acc[k / TW][k % TW] = acc[(k + 1) / TW][(k + 1) % TW];
            }
        }
    }
}

template <int WNT, int EPI, bool ODD, bool ROUNDS = false, bool PART = false, bool ONCE = false>
int launch_wide(dim3 grid, hipStream_t st, const WideArgs &a) {
    constexpr int NST = wide_stages(WNT, ROUNDS), LDS = wide_lds_bytes(WNT, NST);
    static std::once_flag once;
    static hipError_t configured = hipSuccess;
    std::call_once(once, [] {
        configured = hipFuncSetAttribute((const void *)gemm_wide_kernel<WNT, EPI, ODD, NST, PART, ONCE>, hipFuncAttributeMaxDynamicSharedMemorySize, LDS);
    });
    if (configured != hipSuccess) return hx_fail(HX_E_HIP, "hipFuncSetAttribute: %s", hipGetErrorString(configured));
    hipLaunchKernelGGL((gemm_wide_kernel<WNT, EPI, ODD, NST, PART, ONCE>), grid, dim3(64 * WIDE_WAVES), LDS, st, a);
    return HX_OK;
}

template <int WNT>
int launch_wide_epi(int epilogue, dim3 grid, hipStream_t st, const WideArgs &a) {
    if (epilogue == HX_EPI_PARTIAL) {
        if (a.k_steps & 1) return launch_wide<WNT, HX_EPI_PARTIAL, true>(grid, st, a);
        if constexpr (WNT <= 5) if (a.groups <= WIDE_PART_GROUPS) return launch_wide<WNT, HX_EPI_PARTIAL, false, false, true>(grid, st, a);
        return launch_wide<WNT, HX_EPI_PARTIAL, false>(grid, st, a);
    }
    if (epilogue == HX_EPI_LOGITS) return launch_wide<WNT, HX_EPI_LOGITS, false>(grid, st, a);
    if (epilogue == HX_EPI_SAMPLE) return launch_wide<WNT, HX_EPI_SAMPLE, false>(grid, st, a);
    if ((int)grid.x > hx_device_cus()) return launch_wide<WNT, HX_EPI_SWIGLU, false, true>(grid, st, a);
    if constexpr (WNT <= 5) {
        const bool once = a.R == 1 && a.k_steps >= WIDE_ONCE_STEPS;
        if (a.groups <= WIDE_PART_GROUPS) {
            if (once) return launch_wide<WNT, HX_EPI_SWIGLU, false, false, true, true>(grid, st, a);
            return launch_wide<WNT, HX_EPI_SWIGLU, false, false, true>(grid, st, a);
        }
        if (once) return launch_wide<WNT, HX_EPI_SWIGLU, false, false, false, true>(grid, st, a);
    }
    return launch_wide<WNT, HX_EPI_SWIGLU, false>(grid, st, a);
}

}  // namespace

// Tiles per workgroup and, for a product whose consumer sums partials, K-splits: the plan with the least time by a
// model in microseconds, fitted to 7B and 14B products (224 to 1184 k-steps, 8 and 19 row blocks) when all of them were 32x32x16.  Of the
// present kernels, every plan of 4 to 8 tiles in 1 to 4 splits measured, it still takes the best or one within 3 % (14B O over 4864 rows 224 us, in two splits
// of 8 tiles 207 and the sum of a second split).  A 256 x 32 tile takes 46 ns
// per k-step on a compute unit when at most two thirds of them are busy and 52 when all are (the chip lowers its clock);
// a workgroup's start and end 8 per round, the launch 4; partial sums are written at 4.7 TB/s and the further ones
// read again at 10.  Narrow tiles read more operands per product.  The last round of many is only charged half.
// Measured, the plan taken (others), us: 7B, 2048 rows: QKV 67 with 5 tiles (6: 72, 7 in 3 splits: 73), down 213 with 7 in 2 (8 in 2: 207, 4: 237), O 50 with 7
// in 2 (8 in 2: 49, 4: 51), gate|up 423 to 504 with 8 as the clock has it (7: 483, 4: 482, 5: 518).  14B, 4864 rows: QKV 309 with 6 (8 in 2: 315, 7: 327), down
// 501 with 8 in 2 (7: 559), gate|up 1073 with 8 (6: 1154, 7: 1177, 5: 1244).  1.5B, 2048 rows: gate|up 108 with 6 (4: 109, 8: 119), down 53 with 6 in 4 (7 in 4: 56).
// One block of 256 rows, products that no other kernel takes (us; in brackets the streaming kernel of gemm.hip, which it replaces beyond 128 rows): 1.5B
// gate|up 27.6 (32.2); 7B QKV 20.4 (21.1), O 18.4 (19.5), gate|up 78.4 (88.6), down 46.7 (50.2); 14B 31.2 (32.9), 25.7 (27.3), 90.9 (89.7), 46.6 (51.5).
// The same two in turn on one card, with the packing of the input and the sum of the partials, at 129, 192 and 256 rows: 14B gate|up 95.9, 99.5, 102.2
// (98.8, 100.2, 105.5), the others 3 to 24 % faster.
int hx_wide_split_steps(const hx_matrix *m, int splits) { return ((m->k_steps + splits - 1) / splits + 1) & ~1; }

hx_wide_plan hx_plan_wide(const hx_matrix *m, int row_blocks, int epilogue, int max_splits) {
    const int cus = hx_device_cus();
    const bool partial = epilogue == HX_EPI_PARTIAL;
    const double out_mb = (double)row_blocks * 256 * m->N * (epilogue == HX_EPI_SWIGLU ? 1 : 4) * 1e-6;   // gate|up: bf16 of half the columns
    hx_wide_plan best{8, 1};
    double best_us = 1e300;
    for (int wnt : {8, 7, 6, 5, 4}) {
        const int NB = (m->n_tiles + wnt - 1) / wnt;
        const double narrow = wnt == 4 ? 1.2 : (wnt == 5 ? 1.12 : (wnt == 6 ? 1.03 : 1.0));
        for (int s = 1; s <= (partial ? max_splits : 1); ++s) {
            if (s > 1 && m->k_steps / s < 32) break;
            const int sps = hx_wide_split_steps(m, s);
            if ((s - 1) * sps >= m->k_steps) continue;          // whole chunks would leave the last split empty
            const double exact = (double)NB * row_blocks * s / cus;
            const int whole = (NB * row_blocks * s + cus - 1) / cus;
            const double rounds = whole <= 4 ? whole : 0.5 * (whole + exact);
            const double busy = exact / whole;
            const double tile_us = 0.046 + 0.018 * std::max(0.0, busy - 0.667);
            const double us = 4.0 + 8.0 * (whole - 1) + out_mb * (s / 4.7 + (s - 1) / 10.0) + rounds * wnt * sps * tile_us * narrow;
            if (us < best_us - 1e-9) { best_us = us; best.wnt = wnt; best.splits = s; }
        }
    }
    return best;
}

// One wide product over `row_blocks` blocks of 256 rows.  xp_off / y_off / mp_off: byte offsets of the packed input,
// the fp32 output ([splits][256][N]) and the SiLU*mul output inside each block's workspace; ws0 = block 0's
// workspace, block_stride bytes between blocks.
int hx_launch_gemm_wide(const hx_engine *e, const hx_matrix *m, int row_blocks, char *ws0, size_t block_stride, size_t xp_off,
                        int epilogue, size_t y_off, size_t mp_off, hx_wide_plan plan, hipStream_t st, const hx_lm_args *lm, int rows) {
    int splits = plan.splits;
    const int wnt = plan.wnt;
    if (wnt < 4 || wnt > 8) return hx_fail(HX_E_RANGE, "%d tiles per workgroup: no such wide product", wnt);
    if (m->k_steps % 2 && epilogue != HX_EPI_PARTIAL)   // hidden sizes are multiples of 32: only a down product's K can be odd
        return hx_fail(HX_E_SHAPE, "epilogue %d over %d k-steps has no wide product", epilogue, m->k_steps);
    const bool head = epilogue == HX_EPI_LOGITS || epilogue == HX_EPI_SAMPLE;
    if (head && (!lm || row_blocks != 1)) return hx_fail(HX_E_RANGE, "the LM head takes one block of rows");
    if (epilogue != HX_EPI_PARTIAL) splits = 1;
    if (block_stride % 16) return hx_fail(HX_E_RANGE, "block stride %zu is not a multiple of 16", block_stride);
    WideArgs a;
    a.wp = (const uint4 *)(e->weights + m->offset);
    a.k_steps = m->k_steps; a.n_tiles = m->n_tiles; a.N = m->N;
    a.xp0 = ws0 + xp_off; a.block_stride = block_stride; a.R = row_blocks;
    a.y0 = (float *)(ws0 + y_off);
    a.mp0 = (uint16_t *)(ws0 + mp_off);
    a.groups = row_blocks == 1 && rows > 128 ? (rows + 31) / 32 : 8;
    a.lm = head ? *lm : hx_lm_args{};
    a.steps_per_split = hx_wide_split_steps(m, splits);
    const int NB = (m->n_tiles + wnt - 1) / wnt;
    a.splits = splits;
    dim3 grid((NB * row_blocks * splits + 7) / 8 * 8);
    for (int sp = 0; sp < splits; ++sp)
        if (sp * a.steps_per_split >= m->k_steps) return hx_fail(HX_E_RANGE, "%d splits leave split %d of %d k-steps empty", splits, sp, m->k_steps);
    int rc;
    switch (wnt) {
        case 4: rc = launch_wide_epi<4>(epilogue, grid, st, a); break;
        case 5: rc = launch_wide_epi<5>(epilogue, grid, st, a); break;
        case 6: rc = launch_wide_epi<6>(epilogue, grid, st, a); break;
        case 7: rc = launch_wide_epi<7>(epilogue, grid, st, a); break;
        default: rc = launch_wide_epi<8>(epilogue, grid, st, a); break;
    }
    if (rc) return rc;
    HX_CHECK_LAUNCH("gemm_wide");
    return HX_OK;
}
