// Attention for prompt rows (prefill_rows, prefill_chunk): one schedule over all rows of
// the call, workgroups of four wavefronts that share a K/V stream through LDS.
//
// Consecutive rows of one sequence form a GROUP of up to 128 / G rows; its (row, query head of one KV head) pairs are
// up to 128 columns, 32 per wavefront.  A step is the K and V of 32 tokens (two cache blocks, 16 KiB in bf16), copied
// once per workgroup from the pool straight into LDS (three stages, requested two steps ahead):
//     S^T[token, column] = K . q           D/16 x v_mfma_f32_32x32x16_bf16   (A = K from LDS, B = q in registers)
//     O^T[d, column]    += V^T . P^T        D/32 x 2 blocks x (high, low part of P)
// The accumulator layout of the first product (lane = column, 16 registers = 16 of the 32 tokens) is taken as the
// B operand of the second by numbering the contraction index accordingly: the probabilities never cross lanes, and the
// V operand is read from LDS in the matching order.  P enters as a high + low bf16 pair, as in the decode step.
//
// What bounds it: a step is a chain (K reads, scores, maximum, exponentials, V reads, products) of which the matrix cores take
// 768 cycles at D = 128 and the arithmetic beside them about as many; the two wavefronts of a SIMD cover each other's only in
// part (2048 rows, 7B, one workgroup per compute unit 98 us, two 75).  Measured per layer, kernel + combine, against a
// kernel that served 8 rows per K/V stream with one wavefront each and 16-row products of half the rate: 7B, one prompt
// of 2048 tokens 75 + 13 us (214 + 69); 14B, 7 prompts of 5000 tokens together, 8-bit cache 97 + 6 us (273 + 136);
// 1.5B, 200 rows behind 3000 cached tokens 18 + 7 us (41 + 9).
//
// Schedule: a pair (group, KV head) of more than S steps is cut into equal parts of at most S steps; S follows from the
// work of the whole call (prompt_sched_kernel), so that a short call with a long cache fills the chip and a long one
// writes few partial results.  An uncut pair writes its output itself; the parts of a cut one are merged by
// prompt_combine_kernel.  Where there are more items than workgroups, groups are numbered by the length of their parts, items
// run from the last group to the first, and every second round of the workgroups, if it is not small, takes its items in reverse: who had a
// long part gets a short one.  (In the order of the rows, every round alike, one of 512 workgroups had up to 50 steps of a 2048-token
// prompt where the mean is 29.)  us per layer, the order of the rows | this: 7B, 2048 rows 83 | 75, 14B, 8-bit cache, 4864 rows of 7 prompts 118 | 97;
// the schedule, once for all layers, 11 -> 13 and 13.5 -> 18.
//
// Per-group arrays live where the 256-row workspaces keep their per-row ones: entry g in block g / 256 at g % 256.
#include "hx_internal.h"
#include <type_traits>

#define HX_NEG_BIG (-1.0e30f)
#define HX_PROMPT_COLS 128
#define HX_PROMPT_MIN_STEPS 8

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2_t __attribute__((ext_vector_type(2)));

struct PromptArgs {
    char *ws0;                          // workspace of the call's first 256 rows; the others follow at `stride` bytes
    size_t stride;
    size_t o_qp, o_pre, o_lens, o_ginfo, o_gslot, o_glist, o_sched, o_ap, o_ml, o_po;     // byte offsets in each
    int n_rows, n_blocks, slots_per_block;
    int n_kv, G, n_q, m_groups;
    float *attn_f32;                    // [n_rows, n_q * D] or NULL
};

template <typename T>
__device__ __forceinline__ T *group_entry(const PromptArgs &a, size_t off, int g) {
    return (T *)(a.ws0 + (size_t)(g >> 8) * a.stride + off) + (g & 255);
}

// ---- per row: RoPE angles, the block of its position, and whether it continues the row before it -----------------------
// grid = rows, 64 threads.  Row r continues row r - 1 if its length is one more and its table row repeats that of r - 1
// over the blocks r - 1 uses.  Angles as in step_setup_kernel.
__global__ __launch_bounds__(64) void prompt_rows_kernel(char *ws0, size_t stride, size_t o_cs, size_t o_blk, size_t o_cont,
                                                         const int32_t *__restrict__ positions,
                                                         const int32_t *__restrict__ seq_lens,
                                                         const int32_t *__restrict__ table, int max_blocks, int half,
                                                         double theta, int max_batch) {
    const int r = blockIdx.x, lane = threadIdx.x;
    char *ws = ws0 + (size_t)(r >> 8) * stride;
    const int b = r & 255;
    const int pos = positions[r];
    bool ok = false;
    if (r > 0) {
        const int Tp = seq_lens[r - 1], T = seq_lens[r];
        const int nb = (Tp + 15) >> 4;
        ok = (T == Tp + 1) && nb <= max_blocks;
        const int32_t *p = table + (size_t)(r - 1) * max_blocks, *q = table + (size_t)r * max_blocks;
        for (int i = lane; i < nb && ok; i += 64) ok = p[i] == q[i];
    }
    const bool all = __all(ok);
    if (lane == 0) {
        ((int32_t *)(ws + o_cont))[b] = (r > 0 && all) ? 1 : 0;
        ((int32_t *)(ws + o_blk))[b] = table[(size_t)r * max_blocks + (pos >> 4)];
    }
    float *cs = (float *)(ws + o_cs);
    for (int i = lane; i < half; i += 64) {
        const double ang = (double)pos * pow(theta, -(double)i / (double)half);
        cs[(size_t)b * half + i] = (float)cos(ang);
        cs[(size_t)max_batch * half + (size_t)b * half + i] = (float)sin(ang);
    }
}

// ---- groups and their schedule ------------------------------------------------------------------------------------------
// Inclusive scans over the 1024 threads of the one workgroup (wavefront shuffles, then the 16 wavefront totals).
template <bool MAX>
__device__ __forceinline__ int scan_1024(int v, int *red, int *total) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const int o = __shfl_up(v, off);
        if (lane >= off) v = MAX ? max(v, o) : v + o;
    }
    __syncthreads();                        // red may still be read from the scan before
    if (lane == 63) red[wave] = v;
    __syncthreads();
    int before = MAX ? -1 : 0, all = MAX ? -1 : 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) {
        if (w < wave) before = MAX ? max(before, red[w]) : before + red[w];
        all = MAX ? max(all, red[w]) : all + red[w];
    }
    *total = all;
    return MAX ? max(v, before) : v + before;
}

// Groups in the order of the rows, or of their parts' lengths, shortest first.
// pre[g] = items (group, KV head, part) of the groups before g, lens[g] = keys of the group's last row, ginfo[g] = first
// row | rows << 16, gslot[g] = first partial slot of a cut group, glist = the cut groups; sched (block 0) = {S, items,
// cut groups}.  n_rows <= 8192: up to 8 rows (later: groups) per thread.
__global__ __launch_bounds__(1024) void prompt_sched_kernel(PromptArgs a, const int32_t *__restrict__ seq_lens, size_t o_cont,
                                                            int group_rows, int n_wgs) {
    extern __shared__ int32_t sT[];                     // [n_rows] keys of each group's last row; then [n_rows] 16-bit groups in order
    uint16_t *order = (uint16_t *)(sT + a.n_rows);
    __shared__ int bin[1024];
    __shared__ int red[16];
    __shared__ long long redl[16];
    const int tid = threadIdx.x, E = (a.n_rows + 1023) >> 10, r0 = tid * E, r1 = min(a.n_rows, r0 + E);
    auto cont = [&](int r) { return *group_entry<int32_t>(a, o_cont, r); };
    int run = -1;                                       // start of the last run of consecutive rows that begins here
    for (int r = r0; r < r1; ++r) if (!cont(r)) run = r;
    int total;
    const int own = scan_1024<true>(run, red, &total);
    int before = __shfl_up(own, 1);                     // the run that is open on entry: the scan up to the thread before
    __syncthreads();
    if ((tid & 63) == 63) red[tid >> 6] = own;
    __syncthreads();
    if ((tid & 63) == 0) before = tid ? red[(tid >> 6) - 1] : 0;
    int n_start = 0, open = before;
    for (int r = r0; r < r1; ++r) {
        if (!cont(r)) open = r;
        n_start += (r - open) % group_rows == 0;
    }
    int n_groups;
    int gid = scan_1024<false>(n_start, red, &n_groups) - n_start - 1;
    open = before;
    for (int r = r0; r < r1; ++r) {
        if (!cont(r)) open = r;
        const int local = (r - open) % group_rows;
        gid += local == 0;
        const bool last = r + 1 == a.n_rows || !cont(r + 1) || local + 1 == group_rows;
        if (last) {
            sT[gid] = seq_lens[r];
            *group_entry<int32_t>(a, a.o_ginfo, gid) = (r - local) | ((local + 1) << 16);
        }
    }
    __syncthreads();                                    // sT is complete; nobody reads cont any more (glist replaces it)
    const int g0 = tid * E, g1 = min(n_groups, g0 + E);
    long long units = 0;
    for (int g = g0; g < g1; ++g) units += (sT[g] + 31) >> 5;
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) units += __shfl_xor(units, off);
    if ((tid & 63) == 0) redl[tid >> 6] = units;
    __syncthreads();
    units = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) units += redl[w];
    units *= a.n_kv;
    // The longest part: the share of one workgroup of the whole grid, at least HX_PROMPT_MIN_STEPS (a part costs its
    // workgroup the queries and a partial result of 64 KiB), and long enough for the partial slots: a cut pair has at
    // most 2 steps / S parts.
    const long long cap = (long long)a.slots_per_block * a.n_blocks;
    long long longest = (units + n_wgs - 1) / n_wgs;
    if (longest < HX_PROMPT_MIN_STEPS) longest = HX_PROMPT_MIN_STEPS;
    if (longest < (2 * units + cap - 1) / cap) longest = (2 * units + cap - 1) / cap;
    const int S = (int)longest;                         // 32 bits: the quotients by it are what this kernel's end takes
    auto parts = [&](int g) { return (((sT[g] + 31) >> 5) + S - 1) / S; };
    int want = 0;
    for (int g = g0; g < g1; ++g) want += parts(g);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) want += __shfl_xor(want, off);
    if ((tid & 63) == 0) red[tid >> 6] = want;
    bin[tid] = 0;
    __syncthreads();
    want = 0;
#pragma unroll
    for (int w = 0; w < 16; ++w) want += red[w];
    // Items in one round of the workgroups are not ordered; where there are more, the groups go by the length of their parts, in
    // 1024 steps of it; which of two equal ones comes first decides no result.  (Parts of half as much again would balance as well and be
    // fewer, 2374 us per 4-layer call instead of 2392, 7B, 2048 rows, and 1577 instead of 1620, 1024 rows behind 3000 tokens, but their longer sums
    // are 1 to 2.6 % further from exact.)
    const bool ordered = want * a.n_kv > n_wgs;
    auto group_at = [&](int g) { return ordered ? (int)order[g] : g; };
    if (ordered) {
        auto length = [&](int g) { const int st = (sT[g] + 31) >> 5, np = max(parts(g), 1); return (st + np - 1) / np * 1023 / S; };   // no keys: 0
        for (int g = g0; g < g1; ++g) atomicAdd(&bin[length(g)], 1);
        __syncthreads();
        int all;
        const int count = bin[tid], below = scan_1024<false>(count, red, &all) - count;
        bin[tid] = below;
        __syncthreads();
        for (int g = g0; g < g1; ++g) order[atomicAdd(&bin[length(g)], 1)] = (uint16_t)g;
        __syncthreads();
        int info[HX_PREFILL_MAX_ROWS / 1024];
#pragma unroll
        for (int k = 0; k < HX_PREFILL_MAX_ROWS / 1024; ++k) info[k] = g0 + k < g1 ? *group_entry<int32_t>(a, a.o_ginfo, order[g0 + k]) : 0;
        __syncthreads();                                // read by everybody, before the entries move
#pragma unroll
        for (int k = 0; k < HX_PREFILL_MAX_ROWS / 1024; ++k) if (g0 + k < g1) *group_entry<int32_t>(a, a.o_ginfo, g0 + k) = info[k];
    }
    for (int g = g0; g < g1; ++g) *group_entry<int32_t>(a, a.o_lens, g) = sT[group_at(g)];
    int items = 0, slots = 0, cut = 0;
    for (int g = g0; g < g1; ++g) {
        const int np = parts(group_at(g));
        items += np * a.n_kv;
        if (np > 1) { slots += np * a.n_kv; ++cut; }
    }
    int n_items, n_slots, n_cut;
    int at = scan_1024<false>(items, red, &n_items) - items;
    int slot = scan_1024<false>(slots, red, &n_slots) - slots;
    int ci = scan_1024<false>(cut, red, &n_cut) - cut;
    for (int g = g0; g < g1; ++g) {
        const int np = parts(group_at(g));
        *group_entry<int32_t>(a, a.o_pre, g) = at;
        at += np * a.n_kv;
        if (np > 1) {
            *group_entry<int32_t>(a, a.o_gslot, g) = slot;
            slot += np * a.n_kv;
            *group_entry<int32_t>(a, a.o_glist, ci++) = g;
        }
    }
    for (int g = n_groups + tid; g < a.n_blocks * 256; g += 1024) *group_entry<int32_t>(a, a.o_pre, g) = n_items;
    if (tid == 0) {
        int32_t *sched = (int32_t *)(a.ws0 + a.o_sched);
        sched[0] = S;
        sched[1] = n_items;
        sched[2] = n_cut;
    }
}

// ---- the attention kernel -----------------------------------------------------------------------------------------------
// The 32 columns of a wavefront, 16 of the 32 d of block i: the values d = 32 i + 8 (q + {0, 1}) + 4 (lane / 32) + 0..3 for one
// q of 0 and 2, bf16 into the packed operand of the output projection, unrounded if asked.
template <int D>
__device__ __forceinline__ void store_pair(const PromptArgs &a, f32x4_t v0, f32x4_t v1, float inv, int row, int head, int i, int q, int lane,
                                           bool used) {
    const int h = lane >> 5;
    v0 *= inv;
    v1 *= inv;
    const uint2 p0 = make_uint2(hx_cvt_pk_bf16(v0[0], v0[1]), hx_cvt_pk_bf16(v0[2], v0[3]));
    const uint2 p1 = make_uint2(hx_cvt_pk_bf16(v1[0], v1[1]), hx_cvt_pk_bf16(v1[2], v1[3]));
    // the two half-wavefronts hold 4 + 4 of every 8 consecutive d: exchange, so that each stores 8
    const uint2 give = h ? p0 : p1;
    uint2 got;
    got.x = __shfl_xor(give.x, 32);
    got.y = __shfl_xor(give.y, 32);
    const uint4 w = h ? make_uint4(got.x, got.y, p1.x, p1.y) : make_uint4(p0.x, p0.y, got.x, got.y);
    uint16_t *ap = (uint16_t *)(a.ws0 + (size_t)(row >> 8) * a.stride + a.o_ap);
    if (!used) return;
    *(uint4 *)(ap + hx_xp_index(row & 255, head * D + 32 * i + 8 * (q + h), a.m_groups)) = w;
    if (a.attn_f32) {
        float *dst = a.attn_f32 + ((size_t)row * a.n_q + head) * D + 32 * i + 4 * h + 8 * q;
        *(f32x4_t *)dst = v0;
        *(f32x4_t *)(dst + 8) = v1;
    }
}

// all of block i from an accumulator (register r: d = 32 i + 8 (r / 4) + 4 (lane / 32) + r % 4)
template <int D>
__device__ __forceinline__ void store_block(const PromptArgs &a, const f32x16_t &o, float inv, int row, int head, int i, int lane,
                                            bool used) {
#pragma unroll
    for (int q = 0; q < 4; q += 2)
        store_pair<D>(a, f32x4_t{o[4 * q], o[4 * q + 1], o[4 * q + 2], o[4 * q + 3]},
                      f32x4_t{o[4 * q + 4], o[4 * q + 5], o[4 * q + 6], o[4 * q + 7]}, inv, row, head, i, q, lane, used);
}

// group of item `it`: the last g with pre[g] <= it, by two ballots over the up to 32 x 256 entries
__device__ __forceinline__ int find_group(const PromptArgs &a, int it, int lane) {
    const int n = a.n_blocks * 256;
    const int i1 = lane * 128;
    const int v1 = i1 < n ? *group_entry<int32_t>(a, a.o_pre, i1) : 0x7fffffff;
    const int seg = __popcll(__ballot(v1 <= it)) - 1;
    const int i2 = seg * 128 + lane;
    const int va = *group_entry<int32_t>(a, a.o_pre, i2), vb = *group_entry<int32_t>(a, a.o_pre, i2 + 64);
    return __builtin_amdgcn_readfirstlane(seg * 128 + __popcll(__ballot(va <= it)) + __popcll(__ballot(vb <= it)) - 1);
}

// A group of at most 32 columns (one row of many sequences, the last row or two of a prompt) gives one wavefront something to
// multiply, and alone that takes it longer over a step of 4 or 8 KiB (1 us) than the memory takes to deliver one.  Where a step
// is that small (an 8-bit cache, or head size 64) the wavefronts of such a group each take every fourth step, in two LDS stages
// of their own and without a barrier, and are merged at the end; parts of one or two steps are not worth the merge.  us per
// 3-layer call, 8-bit cache, 64 rows of 64 sequences behind 8000 tokens (one K/V stream per wavefront with 16-row products, before
// this kernel | sharing every step | this): 14B 684 | 813 | 679, 7B 475 | 549 | 484, 1.5B 271 | 287 | 254; 256 rows of 256 sequences,
// 2000 tokens: 886 | 1080 | 935, 656 | 717 | 654, 375 | 371 | 338.  With steps of 16 KiB the sharing of one step is 1-2 % faster.
template <int D, bool FP8> constexpr int prompt_step_bytes() { return 4 * 16 * D * (FP8 ? 1 : 2); }
template <int D, bool FP8> constexpr bool prompt_split_steps() { return prompt_step_bytes<D, FP8>() <= 8192; }
template <int D, bool FP8> constexpr int prompt_lds_bytes() { return (prompt_split_steps<D, FP8>() ? 8 : 3) * prompt_step_bytes<D, FP8>(); }

template <int D, bool FP8>
__global__ __launch_bounds__(256, 2) void attn_prompt_kernel(PromptArgs a, const char *__restrict__ pool_layer, size_t block_bytes,
                                                             const int32_t *__restrict__ table, int max_blocks, float scale_log2e) {
    constexpr int TILE = 16 * D * (FP8 ? 1 : 2);        // bytes of a K (or V) tile
    constexpr int STAGE = prompt_step_bytes<D, FP8>();  // two blocks, K | V each
    constexpr int NP = STAGE / 4096;                    // 1-KiB copies per wavefront and step
    extern __shared__ char lds[];                       // [3][STAGE]; where the wavefronts take steps of their own [2][4][STAGE]
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, c32 = lane & 31;
    const int32_t *sched = (const int32_t *)(a.ws0 + a.o_sched);
    const int S = __builtin_amdgcn_readfirstlane(sched[0]), n_items = __builtin_amdgcn_readfirstlane(sched[1]);
    const int G = a.G, n_kv = a.n_kv;
    // (row of the group, query head) of this lane's column: among its wavefront's 32, or among the 32 all of them share
    const int rl_w = (wave * 32 + c32) / G, gq_w = wave * 32 + c32 - rl_w * G, rl_n = c32 / G, gq_n = c32 - rl_n * G;
    // this wavefront's part of a step: half a block (K or V) at most
    constexpr int PER_TILE = TILE / 1024;               // copies per tile: 4, 2 or 1
    for (int round = 0, w0 = 0; w0 < n_items; ++round, w0 += gridDim.x) {
        // A last round of less than a quarter of the workgroups goes to the first of them: the last ones may start behind the others,
        // and such a round then cost them a third part (us, in reverse | so: 256 rows behind 3000 tokens, 8-bit cache, 7B 51 | 37.7, 14B 66 | 43.8, bf16 7B 44 | 37.8;
        // 3 x 80 rows behind 6000 76 | 64.3; of 1.4 and 1.6 rounds, 7B, 2048 rows 74.5 and 200 single rows 206, not in reverse 75.5 and 243).
        const bool back = (round & 1) && 4 * (n_items - w0) >= (int)gridDim.x;
        const int w = w0 + (int)(back ? gridDim.x - 1 - blockIdx.x : blockIdx.x);
        if (w >= n_items) break;                        // only in the last round
        const int it = n_items - 1 - w;
        const int gi = find_group(a, it, lane);
        const int info = __builtin_amdgcn_readfirstlane(*group_entry<int32_t>(a, a.o_ginfo, gi));
        const int T = __builtin_amdgcn_readfirstlane(*group_entry<int32_t>(a, a.o_lens, gi));
        const int first = info & 0xffff, rows = info >> 16;
        const int steps = (T + 31) >> 5, np = (steps + S - 1) / S, nblk = (T + 15) >> 4;
        const int local = it - __builtin_amdgcn_readfirstlane(*group_entry<int32_t>(a, a.o_pre, gi));
        const int kvh = local / np, part = local - kvh * np;
        const int s0 = part * steps / np, s1 = (part + 1) * steps / np;          // steps <= 2^15: no overflow
        const size_t head_off = (size_t)kvh * 2 * TILE;
        const int32_t *trow = table + (size_t)(first + rows - 1) * max_blocks;   // the group reads through its last row
        const bool narrow = prompt_split_steps<D, FP8>() && rows * G <= 32 && steps > 2 * np;   // the same for the whole workgroup
        const int rl = narrow ? rl_n : rl_w, gq = narrow ? gq_n : gq_w;
        const bool used = rl < rows;
        const bool wave_used = narrow || wave * 32 < rows * G;  // wave-uniform
        // A group of at most 32 columns only streams: with a second step in flight it is 1-2 % slower (64 rows of 64 sequences,
        // 8000 tokens, 7B, us per 3-layer call: 649 | 660).
        const bool two_ahead = rows * G > 32;
        const int row = first + (used ? rl : 0);
        const int tcol = used ? T - (rows - 1 - rl) : 0;
        const int t_first = T - (rows - 1);

        u32x4_t q[D / 16];
        {
            const uint4 *qp = (const uint4 *)(a.ws0 + (size_t)(row >> 8) * a.stride + a.o_qp) +
                              ((size_t)(row & 255) * n_kv + kvh) * (D / 32) * 64;
#pragma unroll
            for (int s = 0; s < D / 16; ++s) {
                const uint4 v = qp[(s >> 1) * 64 + ((s & 1) * 2 + h) * 16 + (used ? gq : 0)];
                q[s] = used ? u32x4_t{v.x, v.y, v.z, v.w} : u32x4_t{0u, 0u, 0u, 0u};
            }
        }
        f32x16_t o[D / 32];
#pragma unroll
        for (int i = 0; i < D / 32; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) o[i][r] = 0.f;
        float m = HX_NEG_BIG, l = 0.f;

        int id0 = 2 * s0;                               // lane i holds the physical block of logical block id0 + i
        int32_t ids = trow[min(id0 + lane, nblk - 1)];
        // Waited for here and at the reload: at a use behind copies the wait for it would be one for all of them, every step (so it
        // was: 1.5B, 201 rows behind 3000 tokens 243 us per 3-layer call instead of 229).
        asm volatile("" : "+v"(ids));
        auto request = [&](int s, int stage, int p0) {  // copies NP pieces of step s, from p0 on, into a stage; blocks past the
            if (2 * s - id0 >= 64) {                    // last repeat it
                id0 += 64;
                ids = trow[min(id0 + lane, nblk - 1)];
                asm volatile("" : "+v"(ids));
            }
#pragma unroll
            for (int p = 0; p < NP; ++p) {
                const int piece = p0 + p, blk = piece / (2 * PER_TILE);
                const int32_t id = __builtin_amdgcn_readlane(ids, 2 * s + blk - id0);
                const uint64_t src = (uint64_t)(pool_layer + (size_t)id * block_bytes + head_off + (size_t)(piece % (2 * PER_TILE)) * 1024);
                const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)src), hi = __builtin_amdgcn_readfirstlane((uint32_t)(src >> 32));
                hx_copy_to_lds((const void *)(((uint64_t)hi << 32) | lo), lane * 16, stage * STAGE + piece * 1024);
            }
        };
        auto request_all = [&](int s, int stage) {      // a step of this wavefront's own
#pragma unroll 1
            for (int q = 0; q < 4; ++q) request(s, stage, q * NP);
        };
        // everybody has left the stages of the item before
        __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT(0));
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        auto attend = [&](int s, const char *st) {      // multiplies step s, which lies at st
            const int t0 = s * 32;
            // ---- scores of 32 tokens x 32 columns
            f32x16_t sc;
#pragma unroll
            for (int r = 0; r < 16; ++r) sc[r] = 0.f;
            const char *kb = st + (c32 >> 4) * 2 * TILE + (h * 16 + (c32 & 15)) * 16;
            constexpr int NK = FP8 ? D / 32 : D / 16;   // 16-byte reads of K, all requested before the first product
            u32x4_t kr[NK];
#pragma unroll
            for (int k = 0; k < NK; ++k) kr[k] = *(const u32x4_t *)(kb + (k >> 1) * 1024 + (k & 1) * 512);
            __builtin_amdgcn_sched_barrier(0);
            u32x4_t ko[D / 16];                         // the operand of every step of k
            if (!FP8) {
#pragma unroll
                for (int k = 0; k < D / 16; ++k) ko[k] = kr[k];
            } else {
                // 16 bytes hold the operand bytes of steps k and k + 2
#pragma unroll
                for (int kp = 0; kp < D / 32; ++kp) {
                    const int k = (kp >> 1) * 4 + (kp & 1);
                    const uint2 a0 = hx_e4m3x4_to_bf16x4(kr[kp].x), a1 = hx_e4m3x4_to_bf16x4(kr[kp].y);
                    const uint2 b0 = hx_e4m3x4_to_bf16x4(kr[kp].z), b1 = hx_e4m3x4_to_bf16x4(kr[kp].w);
                    ko[k] = u32x4_t{a0.x, a0.y, a1.x, a1.y};
                    ko[k + 2] = u32x4_t{b0.x, b0.y, b1.x, b1.y};
                }
            }
#pragma unroll
            for (int k = 0; k < D / 16; ++k)
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, ko[k]), __builtin_bit_cast(bf16x8_t, q[k]), sc, 0, 0, 0);
            hx_hold_operands(ko, sc);
            // ---- softmax; register r is token t0 + 8 (r / 4) + 4 h + r % 4
            float p[16];
#pragma unroll
            for (int r = 0; r < 16; ++r) p[r] = sc[r];
            if (t0 + 32 > t_first) {                // wave-uniform: some column ends inside these tokens
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (t0 + 8 * (r >> 2) + 4 * h + (r & 3) >= tcol) p[r] = -INFINITY;
            }
            float mx = p[0];
#pragma unroll
            for (int r = 1; r < 16; ++r) mx = fmaxf(mx, p[r]);
            mx = fmaxf(mx, __shfl_xor(mx, 32));
            // The scale of a column is its maximum, always: the largest probability is then 1 and exact.  (Left up to 2^8 behind it, as the
            // conditional rescaling known from FlashAttention-4, a layer of 2048 rows of 7B takes 70.5 us instead of 75, but that probability
            // is a high + low pair as the others are: 2.0e-6 from exact instead of 1.5e-6, 14B 2.2e-6 instead of 1.25e-6.)
            const float m_new = fmaxf(m, mx * scale_log2e);
#pragma unroll
            for (int r = 0; r < 16; ++r) p[r] = __builtin_amdgcn_exp2f(fmaf(p[r], scale_log2e, -m_new));
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; r += 4) sum += (p[r] + p[r + 1]) + (p[r + 2] + p[r + 3]);
            if (__builtin_amdgcn_ballot_w64(m_new != m) != 0ull) {     // rescale only when some maximum moved
                const float alpha = __builtin_amdgcn_exp2f(m - m_new);
                l *= alpha;
#pragma unroll
                for (int i = 0; i < D / 32; ++i) o[i] *= alpha;
                m = m_new;
            }
            l += sum;
            uint32_t ph[8], pl[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                ph[j] = hx_cvt_pk_bf16(p[2 * j], p[2 * j + 1]);
                pl[j] = hx_cvt_pk_bf16(p[2 * j] - __uint_as_float(ph[j] << 16), p[2 * j + 1] - __uint_as_float(ph[j] & 0xffff0000u));
            }
            // ---- O^T += V^T P^T, one block of 16 tokens after the other: contraction slots 0..3 of a lane are tokens
            // 4 h + 0..3 of the block, slots 4..7 tokens 8 + 4 h + 0..3
            const bool ragged = t0 + 32 > T;        // wave-uniform: V of positions that do not exist may hold anything
#pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                const char *vb = st + (2 * blk + 1) * TILE;
                u32x4_t v[D / 32];
                if (!FP8) {
                    const char *vl = vb + (h * 16 + (c32 & 15)) * 16 + (c32 >> 4) * 8;
#pragma unroll
                    for (int i = 0; i < D / 32; ++i) {
                        const u32x2_t x = *(const u32x2_t *)(vl + i * 1024), y = *(const u32x2_t *)(vl + i * 1024 + 512);
                        v[i] = u32x4_t{x.x, x.y, y.x, y.y};
                    }
                } else {
                    // 16 bytes: 4 tokens of d = c32 % 16 of four 16-wide d ranges
                    const char *vl = vb + (h * 16 + (c32 & 15)) * 16;
#pragma unroll
                    for (int ip = 0; ip < D / 64; ++ip) {
                        const u32x4_t x = *(const u32x4_t *)(vl + ip * 1024), y = *(const u32x4_t *)(vl + ip * 1024 + 512);
                        const bool up = (c32 >> 4) != 0;
                        const uint2 x0 = hx_e4m3x4_to_bf16x4(up ? x.y : x.x), y0 = hx_e4m3x4_to_bf16x4(up ? y.y : y.x);
                        const uint2 x1 = hx_e4m3x4_to_bf16x4(up ? x.w : x.z), y1 = hx_e4m3x4_to_bf16x4(up ? y.w : y.z);
                        v[2 * ip] = u32x4_t{x0.x, x0.y, y0.x, y0.y};
                        v[2 * ip + 1] = u32x4_t{x1.x, x1.y, y1.x, y1.y};
                    }
                }
                if (ragged) {
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const int valid = T - (t0 + 16 * blk + 8 * e + 4 * h);
                        const uint32_t m01 = valid >= 2 ? 0xffffffffu : (valid == 1 ? 0x0000ffffu : 0u);
                        const uint32_t m23 = valid >= 4 ? 0xffffffffu : (valid == 3 ? 0x0000ffffu : 0u);
#pragma unroll
                        for (int i = 0; i < D / 32; ++i) { v[i][2 * e] &= m01; v[i][2 * e + 1] &= m23; }
                    }
                }
                const u32x4_t pp[2] = {{ph[4 * blk], ph[4 * blk + 1], ph[4 * blk + 2], ph[4 * blk + 3]},
                                       {pl[4 * blk], pl[4 * blk + 1], pl[4 * blk + 2], pl[4 * blk + 3]}};
#pragma unroll
                for (int part = 0; part < 2; ++part)
#pragma unroll
                    for (int i = 0; i < D / 32; ++i)
                        o[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, v[i]), __builtin_bit_cast(bf16x8_t, pp[part]), o[i], 0, 0, 0);
                hx_hold_operands(v, pp, o);
            }
        };
        if (narrow) {                                   // every wavefront for itself, in stages of its own: no barrier
            if (s0 + wave < s1) {
                int stage = wave;
                request_all(s0 + wave, stage);
                for (int s = s0 + wave; s < s1; s += 4) {
                    const int next = stage ^ 4;
                    __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT(0));
                    asm volatile("" ::: "memory");
                    if (s + 4 < s1) request_all(s + 4, next);
                    attend(s, lds + stage * STAGE);
                    stage = next;
                }
            }
        } else {
            request(s0, 0, wave * NP);
            if (s0 + 1 < s1) request(s0 + 1, 1, wave * NP);
            int stage = 0;
            for (int s = s0; s < s1; ++s) {
                if (s + 1 < s1 && two_ahead) __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT(NP));
                else __builtin_amdgcn_s_waitcnt(HX_COPY_WAIT(0));
                __builtin_amdgcn_s_barrier();           // step s is in its stage; the stage of step s - 1 is free
                asm volatile("" ::: "memory");
                if (s + 2 < s1) request(s + 2, stage >= 1 ? stage - 1 : 2, wave * NP);
                if (wave_used) attend(s, lds + stage * STAGE);
                stage = stage == 2 ? 0 : stage + 1;
            }
        }
        if (!wave_used) continue;
        l += __shfl_xor(l, 32);
        if (narrow) {
            // merge the wavefronts' results in their order; wavefront i ends up with block i of d
            float *red = (float *)lds;
            __builtin_amdgcn_s_barrier();               // nobody reads a stage any more
            asm volatile("" ::: "memory");
            red[wave * 64 + lane] = h ? l : m;
            __syncthreads();
            float mw[4], lw[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { mw[j] = red[j * 64 + c32]; lw[j] = red[j * 64 + 32 + c32]; }
            __syncthreads();
            f32x4_t *ro = (f32x4_t *)lds + lane;
#pragma unroll
            for (int i = 0; i < D / 32; ++i)
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4)
                    ro[((wave * (D / 32) + i) * 4 + r4) * 64] = f32x4_t{o[i][4 * r4], o[i][4 * r4 + 1], o[i][4 * r4 + 2], o[i][4 * r4 + 3]};
            __syncthreads();
            m = mw[0];
#pragma unroll
            for (int j = 1; j < 4; ++j) m = fmaxf(m, mw[j]);
            l = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) o[0][r] = 0.f;
            if (wave >= D / 32) continue;               // the barrier before the next item's copies holds the others back
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const float wj = __builtin_amdgcn_exp2f(mw[j] - m);
                l += wj * lw[j];
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4) {
                    const f32x4_t x = ro[((j * (D / 32) + wave) * 4 + r4) * 64];
#pragma unroll
                    for (int r = 0; r < 4; ++r) o[0][4 * r4 + r] += wj * x[r];
                }
            }
        }
        if (np == 1) {
            const float inv = 1.0f / l;
            if (narrow) store_block<D>(a, o[0], inv, row, kvh * G + gq, wave, lane, used);
            else {
#pragma unroll
                for (int i = 0; i < D / 32; ++i) store_block<D>(a, o[i], inv, row, kvh * G + gq, i, lane, used);
            }
        } else {
            // partial result in register order: [slot][32 columns][d block, 4 registers][lane], and [max 32 | sum 32]
            const int slot = *group_entry<int32_t>(a, a.o_gslot, gi) + local;
            char *sb = a.ws0 + (size_t)(slot / a.slots_per_block) * a.stride;
            const size_t sub = (size_t)(slot % a.slots_per_block) * 4 + (narrow ? 0 : wave);
            if (!narrow || wave == 0) ((float *)(sb + a.o_ml))[sub * 64 + lane] = h ? l : m;
            f32x4_t *po = (f32x4_t *)(sb + a.o_po) + sub * (D / 8) * 64 + lane;
            if (narrow) po += wave * 4 * 64;
#pragma unroll
            for (int i = 0; i < D / 32; ++i) {
                if (narrow && i > 0) break;
#pragma unroll
                for (int r4 = 0; r4 < 4; ++r4)
                    po[(i * 4 + r4) * 64] = f32x4_t{o[i][4 * r4], o[i][4 * r4 + 1], o[i][4 * r4 + 2], o[i][4 * r4 + 3]};
            }
        }
    }
}

// ---- combine: the parts of the cut pairs ------------------------------------------------------------------------------
// Item = (cut group, KV head, 32 columns); two wavefronts per 32-wide block of d, 16 d each.  Same lane layout as the partials;
// parts are merged in order, four or eight requested at a time, in one pass: what bounds it is the latency of those requests.
// us per launch (two passes, four parts at a time, 32 d per wavefront, two divisions per part to find its slot): 2 pairs of 117
// parts (one row over 30 000 tokens, 1.5B) 46 -> 26, 12 pairs of 32 parts 15.1 -> 9.6, 1.5B, 201 rows behind 3000 tokens 9.4 -> 7.2.
template <int D>
__global__ __launch_bounds__(64 * (D / 16)) void prompt_combine_kernel(PromptArgs a) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, i = wave >> 1, q = 2 * (wave & 1), c32 = lane & 31;
    const int32_t *sched = (const int32_t *)(a.ws0 + a.o_sched);
    const int S = sched[0], n_items = sched[2] * a.n_kv * 4;
    const int G = a.G;
    for (int w = blockIdx.x; w < n_items; w += gridDim.x) {
        const int cb = w & 3, kvh = (w >> 2) % a.n_kv;
        const int gi = *group_entry<int32_t>(a, a.o_glist, (w >> 2) / a.n_kv);
        const int info = *group_entry<int32_t>(a, a.o_ginfo, gi), T = *group_entry<int32_t>(a, a.o_lens, gi);
        const int first = info & 0xffff, rows = info >> 16;
        if (cb * 32 >= rows * G) continue;
        const int np = __builtin_amdgcn_readfirstlane((((T + 31) >> 5) + S - 1) / S);
        const int slot0 = __builtin_amdgcn_readfirstlane(*group_entry<int32_t>(a, a.o_gslot, gi) + kvh * np);
        const int blk0 = slot0 / a.slots_per_block, rem0 = slot0 - blk0 * a.slots_per_block;
        const int col = cb * 32 + c32, rl = col / G, gq = col - rl * G;
        const bool used = rl < rows;
        float m = HX_NEG_BIG, den = 0.f;
        f32x4_t acc[2] = {f32x4_t{0.f, 0.f, 0.f, 0.f}, f32x4_t{0.f, 0.f, 0.f, 0.f}};
        auto merge = [&](int p, auto n) {                // parts p .. p + n - 1; past the last it again, with weight 0
            constexpr int U = decltype(n)::value;
            float pm[U], pl[U];
            f32x4_t v[U][2];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                int rem = rem0 + min(p + u, np - 1), blk = blk0;
                if (rem >= a.slots_per_block) { blk += rem / a.slots_per_block; rem %= a.slots_per_block; }      // wave-uniform, rare
                const char *sb = a.ws0 + (size_t)blk * a.stride;
                const size_t sub = (size_t)rem * 4 + cb;
                const float *ml = (const float *)(sb + a.o_ml) + sub * 64 + c32;
                pm[u] = ml[0];
                pl[u] = ml[32];
                const f32x4_t *po = (const f32x4_t *)(sb + a.o_po) + (sub * (D / 8) + i * 4 + q) * 64 + lane;
                v[u][0] = po[0];
                v[u][1] = po[64];
            }
            float m_new = m;
#pragma unroll
            for (int u = 0; u < U; ++u) m_new = fmaxf(m_new, pm[u]);
            const float alpha = __builtin_amdgcn_exp2f(m - m_new);
            m = m_new;
            den *= alpha;
            acc[0] *= alpha;
            acc[1] *= alpha;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const float wu = p + u < np ? __builtin_amdgcn_exp2f(pm[u] - m) : 0.f;
                den += wu * pl[u];
                acc[0] += wu * v[u][0];
                acc[1] += wu * v[u][1];
            }
        };
        if (np <= 4) merge(0, std::integral_constant<int, 4>{});
        else for (int p = 0; p < np; p += 8) merge(p, std::integral_constant<int, 8>{});
        store_pair<D>(a, acc[0], acc[1], 1.0f / den, first + (used ? rl : 0), kvh * G + gq, i, q, lane, used);
    }
}

// ---- launchers ------------------------------------------------------------------------------------------------------------
static PromptArgs prompt_args(const hx_engine *e, int n_rows, size_t stride, float *attn_f32) {
    const hx_ws_map &m = e->map;
    PromptArgs a;
    a.ws0 = e->ws;
    a.stride = stride;
    a.o_qp = m.qp; a.o_pre = m.pre; a.o_lens = m.lens; a.o_ginfo = m.prompt_ginfo; a.o_gslot = m.prompt_gslot; a.o_glist = m.prompt_cont;
    a.o_sched = m.sched; a.o_ap = m.ap; a.o_ml = m.prompt_part_ml; a.o_po = m.prompt_part_o;
    a.n_rows = n_rows;
    a.n_blocks = (n_rows + 255) / 256;
    a.slots_per_block = (e->attn_waves + e->cfg.max_batch * e->cfg.n_kv_heads) / 2;   // a slot here is two of that area's (64 columns)
    a.n_kv = e->cfg.n_kv_heads; a.G = e->G; a.n_q = e->cfg.n_q_heads;
    a.m_groups = hx_m_groups(n_rows < 256 ? n_rows : 256);
    a.attn_f32 = attn_f32;
    return a;
}

// e->ws: the workspace of the first 256 rows; `stride` bytes to the next (0 where n_rows <= 256)
int hx_launch_prompt_setup(const hx_engine *e, int n_rows, const int32_t *positions, const int32_t *seq_lens, const int32_t *table,
                           int max_blocks, hipStream_t st, size_t stride) {
    if (n_rows < 1 || n_rows > HX_PREFILL_MAX_ROWS) return hx_fail(HX_E_RANGE, "%d prompt rows in one call", n_rows);
    const PromptArgs a = prompt_args(e, n_rows, stride, nullptr);
    hipLaunchKernelGGL(prompt_rows_kernel, dim3(n_rows), dim3(64), 0, st, e->ws, stride, e->map.cs, e->map.blk_new, e->map.prompt_cont,
                       positions, seq_lens, table, max_blocks, e->D / 2, (double)e->cfg.rope_theta, e->cfg.max_batch);
    HX_CHECK_LAUNCH("prompt_rows");
    hipLaunchKernelGGL(prompt_sched_kernel, dim3(1), dim3(1024), (size_t)n_rows * 6, st, a, seq_lens, e->map.prompt_cont,
                       HX_PROMPT_COLS / e->G, e->attn_waves / 4);
    HX_CHECK_LAUNCH("prompt_sched");
    return HX_OK;
}

int hx_launch_prompt_attention(const hx_engine *e, const hx_kv *kv, int layer, int n_rows, const int32_t *table, int max_blocks,
                               float *attn_f32, hipStream_t st, size_t stride) {
    const PromptArgs a = prompt_args(e, n_rows, stride, attn_f32);
    const char *pool_layer = kv->pool + (size_t)layer * kv->layer_bytes;
    const float scale_log2e = (float)(1.4426950408889634 / sqrt((double)e->D));
    dim3 grid(e->attn_waves / 4), block(256);           // two workgroups of four wavefronts per compute unit
#define HX_PROMPT_LAUNCH(DD, F8) \
    hipLaunchKernelGGL((attn_prompt_kernel<DD, F8>), grid, block, (prompt_lds_bytes<DD, F8>()), st, a, pool_layer, kv->block_bytes, table, max_blocks, scale_log2e)
    if (e->D == 128) { if (kv->fp8) HX_PROMPT_LAUNCH(128, true); else HX_PROMPT_LAUNCH(128, false); }
    else             { if (kv->fp8) HX_PROMPT_LAUNCH(64, true);  else HX_PROMPT_LAUNCH(64, false); }
#undef HX_PROMPT_LAUNCH
    HX_CHECK_LAUNCH("attn_prompt");
    return HX_OK;
}

int hx_launch_prompt_combine(const hx_engine *e, int n_rows, float *attn_f32, hipStream_t st, size_t stride) {
    const PromptArgs a = prompt_args(e, n_rows, stride, attn_f32);
    const int items = n_rows * a.n_kv * 4;              // at most; the kernel strides over what there is
    dim3 grid(items < 2048 ? items : 2048);
    if (e->D == 128) hipLaunchKernelGGL((prompt_combine_kernel<128>), grid, dim3(512), 0, st, a);
    else             hipLaunchKernelGGL((prompt_combine_kernel<64>), grid, dim3(256), 0, st, a);
    HX_CHECK_LAUNCH("prompt_combine");
    return HX_OK;
}
