// Small-M weight-streaming matrix products  Y[M, N] = X[M, K] W[K, N]  (M = batch <= 128;
// more rows: gemm_wide.hip; matrices of few columns: gemm_slice.hip).
//
// The weights dominate the bytes, so the kernel is organised around streaming each packed weight
// tile exactly once, straight from HBM into the A operand of v_mfma_f32_32x32x16_bf16 (32 output
// columns n x 16 k per 1-KiB load).  The activations are the B operand (16 k x 32 batch rows per
// m-group); they are small, L2-resident, and shared by the consumer wavefronts of a workgroup through
// a multi-stage LDS copy made by dedicated producer wavefronts.  Each wavefront owns one 32-column n-tile and all batch rows, so the
// accumulator is MG tiles of 32 x 32 fp32.  Along K the product may be split over workgroups; the
// fp32 partial results are summed in split order by the consumer kernel (deterministic).
//
// Epilogues: plain fp32 partials; SiLU(gate) * up -> bf16 packed activations of the down
// projection; logits + per-tile argmax candidates; logits + per-tile sampling candidates and log-sum-exp pieces.
#include "hx_internal.h"
#include "lm_epilogue.h"
#include <algorithm>
#include <mutex>

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_any_t __attribute__((ext_vector_type(4), aligned(2)));     // at any element

// ---- weight packing ------------------------------------------------------------------------------------------
// A workgroup turns 32 k x 512 columns of the row-major source (two k-steps) into operand order.  Thread = 8 k x 8
// columns: eight 16-byte loads, a wavefront's each 1 KiB of one source row; transposed in registers to one 16-byte unit
// (8 k of a column) per column, through LDS into output order, and stored 1 KiB per wavefront and instruction.
// PHASE 0: tile column c = source column 32 * nt + c; PHASE 1 / 2 (gate / up): columns 0..15 / 16..31 of a tile, from
// source column 16 * nt + c % 16 (runs of 256 bytes).  What bounds it is memory: see hx_launch_pack.
#define HX_PACK_COLS 512
// The source may lie at any element: the 16-byte loads are from a 2-byte-aligned type (one load
// instruction, which the hardware takes at any alignment), and only a group of columns that ends past the row goes by elements.
// Loads and stores are non-temporal: everything passes once, and the globals take 764 us with them, 1020 without (see below).
// bx, by: 512 columns, two k-steps
template <int PHASE>
__device__ __forceinline__ void pack_matrix_block(const uint16_t *__restrict__ src, int64_t rows, int64_t cols, uint4 *__restrict__ dst,
                                                  int k_steps, int n_tiles, int bx, int by, uint4 *lds) {
    constexpr int TC = PHASE == 0 ? 32 : 16;            // source columns per tile
    const int tid = threadIdx.x, cg = tid & 63, rg = tid >> 6;            // rg = 2 * k-step + half
    const int64_t c0 = (int64_t)bx * HX_PACK_COLS, col = c0 + 8 * cg, k0 = (int64_t)by * 32 + 8 * rg;
    uint4 in[8];
#pragma unroll
    for (int r = 0; r < 8; ++r) {
        in[r] = make_uint4(0u, 0u, 0u, 0u);
        const uint16_t *p = src + (k0 + r) * cols + col;
        if (k0 + r < rows && col + 8 <= cols) in[r] = __builtin_bit_cast(uint4, __builtin_nontemporal_load((const u32x4_any_t *)p));
    }
    if (col < cols && col + 8 > cols) {
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            const uint16_t *p = src + (k0 + r) * cols + col;
            uint16_t e[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) e[j] = k0 + r < rows && col + j < cols ? p[j] : (uint16_t)0;
            in[r] = make_uint4(e[0] | ((uint32_t)e[1] << 16), e[2] | ((uint32_t)e[3] << 16), e[4] | ((uint32_t)e[5] << 16),
                               e[6] | ((uint32_t)e[7] << 16));
        }
    }
    // units in output order: [tile][k-step][half][column of the tile]; the 8 of a thread are neighbours, so they are spread
    // over the banks by the index of their group of 8
    auto place = [](int u) { return (u & ~7) | ((u ^ (u >> 3)) & 7); };
    const int first = (((8 * cg / TC) * 4 + rg) * TC) + (8 * cg) % TC;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        uint32_t w[4];
#pragma unroll
        for (int h = 0; h < 4; ++h) {
            const uint32_t a = ((const uint32_t *)&in[2 * h])[j >> 1], b = ((const uint32_t *)&in[2 * h + 1])[j >> 1];
            w[h] = (j & 1) ? (a >> 16) | (b & 0xffff0000u) : (a & 0xffffu) | (b << 16);
        }
        lds[place(first + j)] = make_uint4(w[0], w[1], w[2], w[3]);
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int u = i * 256 + tid;
        const int c = u % TC, kh = (u / TC) & 1, s = (u / (2 * TC)) & 1;
        const int64_t nt = c0 / TC + u / (4 * TC);
        const int ks = 2 * by + s;
        if (nt < n_tiles && ks < k_steps)
            __builtin_nontemporal_store(__builtin_bit_cast(u32x4_t, lds[place(u)]), (u32x4_t *)dst + ((size_t)nt * k_steps + ks) * 64 + kh * 32 + (PHASE == 2 ? 16 : 0) + c);
    }
}

// One tensor of a call.  first: its first workgroup; across: workgroups per two k-steps (vectors: all of them).
struct PackItem {
    const uint16_t *src;
    char *dst;
    int64_t rows, cols;
    int k_steps, n_tiles, phase, across;      // phase 0 plain, 1 gate, 2 up, 3 vector (copied)
    unsigned first;
};
struct PackList { PackItem item[HX_PACK_MANY]; int n; };
#define HX_PACK_COPY 4096                    // elements of a vector per workgroup

// All tensors of a call in one launch: the small ones fill the end of the large ones, and nothing waits between them.
__global__ __launch_bounds__(256) void pack_kernel(PackList list) {
    __shared__ uint4 lds[2048];               // unit of column c, k-step s, half kh: see place() above
    int i = 0;
    while (i + 1 < list.n && blockIdx.x >= list.item[i + 1].first) ++i;
    const PackItem &t = list.item[i];
    const unsigned blk = blockIdx.x - t.first;
    if (t.phase == 3) {
        const int64_t n = t.rows * t.cols, e0 = (int64_t)blk * HX_PACK_COPY + threadIdx.x * 8;
        uint16_t *dst = (uint16_t *)t.dst;
        constexpr int U = HX_PACK_COPY / 2048;
        u32x4_t v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) if (e0 + u * 2048 + 8 <= n) v[u] = __builtin_nontemporal_load((const u32x4_any_t *)(t.src + e0 + u * 2048));
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t e = e0 + u * 2048;
            if (e + 8 <= n) __builtin_nontemporal_store(v[u], (u32x4_t *)(dst + e));
            else for (int64_t k = e; k < n; ++k) dst[k] = t.src[k];
        }
        return;
    }
    const int by = (int)(blk / (unsigned)t.across), bx = (int)(blk % (unsigned)t.across);
    if (t.phase == 0) pack_matrix_block<0>(t.src, t.rows, t.cols, (uint4 *)t.dst, t.k_steps, t.n_tiles, bx, by, lds);
    else if (t.phase == 1) pack_matrix_block<1>(t.src, t.rows, t.cols, (uint4 *)t.dst, t.k_steps, t.n_tiles, bx, by, lds);
    else pack_matrix_block<2>(t.src, t.rows, t.cols, (uint4 *)t.dst, t.k_steps, t.n_tiles, bx, by, lds);
}

// 7B, source read and packed copy written: a layer 178 us = 5.2 TB/s (eight launches and copies 203, and as many boundaries),
// the globals 764 us = 5.7 TB/s (pack 412, the runtime's copy of the embedding 429, and a boundary; copying 16 384 elements per
// workgroup instead of 4 096: 827).  A device copy moves 4.8-5.3 here.
int hx_launch_pack(const hx_engine *e, const hx_pack_tensor *tensors, int n, hipStream_t st) {
    if (n < 1 || n > HX_PACK_MANY) return hx_fail(HX_E_RANGE, "%d tensors in one call, 1 to %d", n, HX_PACK_MANY);
    PackList list;
    list.n = n;
    int64_t at = 0;
    for (int i = 0; i < n; ++i) {
        const hx_pack_tensor &t = tensors[i];
        PackItem &o = list.item[i];
        o = PackItem{(const uint16_t *)t.src, e->weights + t.offset, t.rows, t.cols, 0, 0, t.phase, 1, (unsigned)at};
        if (t.phase == 3) {
            at += (t.rows * t.cols + HX_PACK_COPY - 1) / HX_PACK_COPY;
        } else {
            o.k_steps = t.m->k_steps; o.n_tiles = t.m->n_tiles;
            const int64_t all = (int64_t)t.m->n_tiles * (t.phase ? 16 : 32);      // columns of the tiles, zeros beyond `cols` included
            o.across = (int)((all + HX_PACK_COLS - 1) / HX_PACK_COLS);
            at += (int64_t)o.across * ((t.m->k_steps + 1) / 2);
        }
        if (at > 0x7fffffff) return hx_fail(HX_E_RANGE, "the tensors need %lld workgroups", (long long)at);
    }
    hipLaunchKernelGGL(pack_kernel, dim3((unsigned)at), dim3(256), 0, st, list);
    HX_CHECK_LAUNCH("pack");
    return HX_OK;
}

// ---- the streaming product ------------------------------------------------------------------------------------
// Workgroup = WN x WK consumer wavefronts + NP producer wavefronts.
// Consumers: WN adjacent n-tiles, each split into WK k-slices that are summed in slice order through LDS at
// the end.  Every consumer keeps RING weight loads (1 KiB each, non-temporal; 8 or 16: gemm_ring) in flight in a
// register ring and issues no other vector-memory load, so the in-order load counter never makes it wait for anything
// but the tile it is about to use.  Producers stage the activations of the coming chunks (KC k-steps of every
// k-slice, half a ring at most; four stages) in LDS through their own registers; one workgroup barrier per chunk
// hands a stage over.  A stage of one k-slice: 128 rows 32 KiB (16 with a ring of 8), 64 rows 16 (8), 32 rows 4.
#ifndef HX_GEMM_RING
#define HX_GEMM_RING 16
#endif

struct GemmArgs {
    const uint4 *wp;      // packed weights
    const uint4 *xp;      // packed activations
    int k_steps, n_tiles, steps_per_split, steps_per_wave;
    int M, N;
    float *y;             // PARTIAL: [splits][M][N]; LOGITS: [M][N] or NULL
    size_t split_stride;  // elements between splits of y
    uint16_t *mp;         // SWIGLU: packed bf16 output
    float *amax_val;      // LOGITS: [M][n_tiles]; SAMPLE: best perturbed score of the tile
    int32_t *amax_idx;
    // SAMPLE only
    const int32_t *positions, *row_ids;
    float inv_t;
    uint32_t key0, key1;
    float *samp_z, *samp_m, *samp_s;   // [M][n_tiles]
};

__device__ __forceinline__ u32x4_t hx_stream_load(const uint4 *p) {   // read-once data: non-temporal
    return __builtin_nontemporal_load((const u32x4_t *)p);
}

// Weight tiles in flight per consumer.  A compute unit keeps about 64 KiB outstanding: what goes beyond only queues up in front
// of the activations, and splits of few k-steps run in whole revolutions.  So 8, but for two shapes that lose by it: the four and
// five consumers of 128 rows, which wait for activations more than for weights, and four tiles of gate|up.  us, 16 -> 8: 7B at 3
// rows gate|up 44.0 -> 41.7, down 24.2 -> 22.5, QKV 7.8 -> 7.0, O 7.8 -> 7.1; at 37 rows 45.2 -> 44.2, 27.6 -> 26.6, 10.5 -> 9.7, 11.1 -> 10.2,
// LM head 188 -> 185, at 128 rows 227 -> 220; kept, at 16 (8): 7B at 128 rows gate|up 54.0 (57.2), down 37.1 (39.4); gate|up of four tiles
// at 33 / 48 / 64 rows 1.5B 16.6 / 16.1 / 16.3 (17.1 / 16.4 / 17.1), hidden 2048 22.6 / 21.6 / 22.7 (22.7 / 22.2 / 22.8), 14B 48.8 / 47.2 / 47.0
// (49.0 / 48.1 / 47.8).
// Ten tiles per workgroup (the LM head, in two rounds) of up to 64 rows: with at most 80 registers a compute unit holds two workgroups,
// and all run in one round.  So six wavefronts per SIMD are asked for, and a ring of 4.  Head, us, before -> now: 7B at 3 rows, drawn
// (136 registers before) 166 -> 162, 16 rows 179 -> 172, 37 rows (133) 195 -> 184, greedy (87) 187 -> 175; 64 rows greedy 1.5B 92 -> 88, 7B 190 -> 184,
// 14B 263 -> 255, drawn 270 -> 265.  Rings of 8 | 4 up to 32 rows 162.5 | 161.7 and 175.5 | 172.2, of 6 | 4 at 64 rows 14B 269 | 265.
template <int MG, int WN, int EPI> constexpr int gemm_resident() { return WN == 10 && MG <= 2 ? 6 : 1; }

template <int MG, int WN, int EPI> constexpr int gemm_ring() {
    if (WN == 10 && MG <= 2) return HX_GEMM_RING / 4;
    return WN == 10 || MG == 1 || (MG == 2 && !(WN == 4 && EPI == HX_EPI_SWIGLU)) ? HX_GEMM_RING / 2 : HX_GEMM_RING;
}

template <int MG, int WK, int RING> struct GemmGeom {
    static constexpr int NBUF = 4;                                  // stages of at most 32 KiB
    static constexpr int KC0 = 32 / (WK * MG);
    static constexpr int KC = KC0 > RING / 2 ? RING / 2 : (KC0 < 1 ? 1 : KC0);   // k-steps per LDS chunk
    static constexpr int SLICE_U4 = KC * MG * 64;                   // uint4 per k-slice per stage
    static constexpr int PVT = WK * KC * MG;                        // 1-KiB copies per stage
    static constexpr int NP = PVT > 16 ? 2 : 1;                     // producer wavefronts
    static constexpr int PVP = PVT / NP;                            // copies per producer per stage
    static constexpr int STAGE_BYTES = WK * SLICE_U4 * 16;
};
template <int MG, int WN, int WK, int RING> constexpr int gemm_lds_bytes() {
    constexpr int stages = GemmGeom<MG, WK, RING>::NBUF * GemmGeom<MG, WK, RING>::STAGE_BYTES;
    constexpr int red = (WK - 1) * WN * MG * 4096;
    return stages > red ? stages : red;
}

template <int MG, int WN, int WK, int EPI>
__global__ __launch_bounds__(64 * (WN * WK + GemmGeom<MG, WK, gemm_ring<MG, WN, EPI>()>::NP), (gemm_resident<MG, WN, EPI>())) void gemm_stream_kernel(
    const uint4 *__restrict__ a_wp, const uint4 *__restrict__ a_xp, int a_k_steps, int a_n_tiles,
    int a_steps_per_split, int a_steps_per_wave, int a_M, int a_N, float *__restrict__ a_y, size_t a_split_stride,
    uint16_t *__restrict__ a_mp, float *__restrict__ a_amax_val, int32_t *__restrict__ a_amax_idx,
    const int32_t *__restrict__ a_positions, const int32_t *__restrict__ a_row_ids, float a_inv_t, uint32_t a_key0,
    uint32_t a_key1, float *__restrict__ a_samp_z, float *__restrict__ a_samp_m, float *__restrict__ a_samp_s) {
    constexpr int RING = gemm_ring<MG, WN, EPI>();
    using GG = GemmGeom<MG, WK, RING>;
    constexpr int NBUF = GG::NBUF;
    constexpr int KC = GG::KC, CPR = RING / KC, SLICE_U4 = GG::SLICE_U4, NC = WN * WK;
    // with at most 8 wavefronts per workgroup each may use 256 registers: enough to read B operands ahead
    constexpr bool PREFETCH_B = NC + GG::NP <= 8;
    static_assert(RING % KC == 0, "ring must hold whole chunks");
    static_assert((RING / KC) % 2 == 0, "the producers' register sets alternate in pairs of chunks");
    extern __shared__ u32x4_t xs[];                      // [NBUF][WK][SLICE_U4]

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);       // wave-uniform, kept in a scalar register
    const bool producer = wave >= NC;                    // the last wavefronts only stage activations
    const int wn = producer ? 0 : wave % WN, wk = producer ? 0 : wave / WN;
    const int nt = blockIdx.x * WN + wn;
    const bool active = !producer && nt < a_n_tiles;
    const int split0 = blockIdx.y * a_steps_per_split;
    const int split1 = min(a_k_steps, split0 + a_steps_per_split);
    // every wavefront of the grid runs the same number of chunks: whole ring revolutions.  Steps past the end
    // of a k-slice re-read the slice's last (cached) weight tile and skip the multiply, so the load stream
    // carries no condition and the compiler keeps exactly RING - 1 loads outstanding.
    const int n_chunks = (a_steps_per_wave + RING - 1) / RING * CPR;

    if (producer) {
        // k-slice w of this workgroup covers k-steps [split0 + w*spw, min(split1, +spw)); chunk c of it is a
        // contiguous run of the packed activations.
        // The consumers spend their first ring revolution (CPR virtual chunks) only requesting weight tiles; real chunk
        // c is their virtual chunk c + CPR and lives in stage (c + CPR) % NBUF.
        const u32x4_t *xp4 = (const u32x4_t *)a_xp;
        const int last_u4 = a_k_steps * MG * 64 - 1;
        const int pid = wave - NC;
        // The copy goes through registers (global load, then LDS store): measured faster than the direct L2 -> LDS
        // path behind the compiler's builtin (timing lab: weights alone 27 us, direct copy alone 18 us, both 49 us for 60
        // workgroups), where every LDS read waits for all copies in flight; counted waits have not been tried here.
        u32x4_t ra[GG::PVP], rb[GG::PVP];
        auto load_chunk = [&](int c, u32x4_t (&r)[GG::PVP]) {
#pragma unroll
            for (int f = 0; f < GG::PVP; ++f) {
                const int ff = pid * GG::PVP + f;
                const int w = ff / (KC * MG), i = ff % (KC * MG);
                const int kb = min(split1, split0 + w * a_steps_per_wave);
                r[f] = xp4[min((kb + c * KC) * MG * 64 + i * 64 + lane, last_u4)];
            }
        };
        auto store_chunk = [&](int c, const u32x4_t (&r)[GG::PVP]) {
            const int buf = (c + CPR) % NBUF;
#pragma unroll
            for (int f = 0; f < GG::PVP; ++f) {
                const int ff = pid * GG::PVP + f;
                const int w = ff / (KC * MG), i = ff % (KC * MG);
                xs[(buf * WK + w) * SLICE_U4 + i * 64 + lane] = r[f];
            }
        };
        // Barrier v ends the consumers' virtual chunk v (one per KC k-steps, CPR of them before the first real chunk:
        // the revolution that fills their weight ring, which needs no activations).  The barriers of that revolution
        // but the last are passed at once, so the consumers have requested their whole ring before they first wait
        // for this wavefront; chunks 0 and 1 are handed over at the last of them, chunk c >= 2 at barrier c + CPR - 2,
        // one chunk ahead of its use.  Chunk c + 2 is requested as soon as chunk c has left its registers; the two
        // register sets alternate statically (n_chunks is even).
        load_chunk(0, ra);
        load_chunk(1, rb);
#pragma unroll
        for (int i = 0; i < CPR - 1; ++i) __syncthreads();
        store_chunk(0, ra);
        if (2 < n_chunks) load_chunk(2, ra);
        for (int c = 1; c < n_chunks - 1; c += 2) {
            store_chunk(c, rb);
            if (c + 2 < n_chunks) load_chunk(c + 2, rb);
            __syncthreads();
            store_chunk(c + 1, ra);
            if (c + 3 < n_chunks) load_chunk(c + 3, ra);
            __syncthreads();
        }
        store_chunk(n_chunks - 1, rb);
        __syncthreads();
        __syncthreads();
        __syncthreads();
        if (WK > 1) __syncthreads();
        return;
    }

    const int kb0 = split0 + wk * a_steps_per_wave;                  // this wavefront's k-slice [kb0, ke)
    const int ke = min(split1, kb0 + a_steps_per_wave);
    const int n_valid = active ? max(0, ke - kb0) : 0;               // steps that are multiplied
    const int kb = min(kb0, a_k_steps - 1);
    const int last = max(0, min(a_k_steps, kb + a_steps_per_wave) - kb - 1);   // last step whose tile may be read
    const uint4 *wrow = a_wp + ((size_t)(active ? nt : 0) * a_k_steps + kb) * 64 + lane;

    f32x16_t acc[MG];
#pragma unroll
    for (int g = 0; g < MG; ++g)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[g][r] = 0.f;

    // The loop starts one revolution early (c0 = -CPR): that revolution multiplies nothing, it only requests the
    // first RING tiles (at once: it does not wait for the activations); from then on step s multiplies the tile
    // requested RING steps earlier and then requests the tile of step s + RING into the same slot.
    // There is no separate prologue, so the only loads outstanding at any wait are the ring's own, in order.
    u32x4_t ring[RING];
#pragma unroll
    for (int r = 0; r < RING; ++r) ring[r] = u32x4_t{0u, 0u, 0u, 0u};

    int c_first = -CPR;
    asm volatile("" : "+s"(c_first));                   // opaque: the ring-filling revolution must not be peeled off the loop
    for (int c0 = c_first; c0 < n_chunks; c0 += CPR) {
#pragma unroll
        for (int cc = 0; cc < CPR; ++cc) {
            const int c = c0 + cc;
            const u32x4_t *xb = &xs[(((c + CPR) % NBUF) * WK + wk) * SLICE_U4 + lane];
            if (PREFETCH_B) {
                // B operands are read from LDS one k-step ahead of the multiplies that use them
                u32x4_t bcur[MG], bnxt[MG];
#pragma unroll
                for (int g = 0; g < MG; ++g) bcur[g] = xb[g * 64];
#pragma unroll
                for (int j = 0; j < KC; ++j) {
                    const int s = c * KC + j;
                    if (j + 1 < KC) {
#pragma unroll
                        for (int g = 0; g < MG; ++g) bnxt[g] = xb[((j + 1) * MG + g) * 64];
                    }
                    if (s >= 0 && s < n_valid) {
                        const bf16x8_t aop = __builtin_bit_cast(bf16x8_t, ring[cc * KC + j]);
#pragma unroll
                        for (int g = 0; g < MG; ++g)
                            acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aop, __builtin_bit_cast(bf16x8_t, bcur[g]), acc[g], 0, 0, 0);
                    }
                    // the slot is dead now: request the tile of step s + RING into the same registers
                    ring[cc * KC + j] = hx_stream_load(wrow + (size_t)min(s + RING, last) * 64);
                    if (j + 1 < KC) {
#pragma unroll
                        for (int g = 0; g < MG; ++g) bcur[g] = bnxt[g];
                    }
                }
            } else {
                // too many accumulators to hold two steps of B operands: read them DEPTH operands ahead of the
                // multiply that uses them, in the order (k-step, m-group) in which the stage stores them
                constexpr int DEPTH = 3, ITEMS = KC * MG;
                u32x4_t bq[DEPTH];
#pragma unroll
                for (int t = 0; t < DEPTH; ++t) bq[t] = xb[t * 64];
#pragma unroll
                for (int j = 0; j < KC; ++j) {
                    const int s = c * KC + j;
                    const bf16x8_t aop = __builtin_bit_cast(bf16x8_t, ring[cc * KC + j]);
#pragma unroll
                    for (int g = 0; g < MG; ++g) {
                        const int t = j * MG + g;
                        const u32x4_t bcur = bq[t % DEPTH];
                        if (t + DEPTH < ITEMS) bq[t % DEPTH] = xb[(t + DEPTH) * 64];
                        if (s >= 0 && s < n_valid)
                            acc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aop, __builtin_bit_cast(bf16x8_t, bcur), acc[g], 0, 0, 0);
                    }
                    ring[cc * KC + j] = hx_stream_load(wrow + (size_t)min(s + RING, last) * 64);
                }
            }
            __syncthreads();
        }
    }

    // sum the k-slices of each n-tile in slice order (the activation stages are free now)
    if (WK > 1) {
        float *red = (float *)xs;
        if (wk > 0 && active) {
            float *dst = red + ((size_t)((wk - 1) * WN + wn) * MG * 16) * 64 + lane;
#pragma unroll
            for (int g = 0; g < MG; ++g)
#pragma unroll
                for (int r = 0; r < 16; ++r) dst[(g * 16 + r) * 64] = acc[g][r];
        }
        __syncthreads();
        if (wk == 0 && active) {
#pragma unroll
            for (int w2 = 1; w2 < WK; ++w2) {
                const float *src = red + ((size_t)((w2 - 1) * WN + wn) * MG * 16) * 64 + lane;
#pragma unroll
                for (int g = 0; g < MG; ++g)
#pragma unroll
                    for (int r = 0; r < 16; ++r) acc[g][r] += src[(g * 16 + r) * 64];
            }
        }
    }
    if (!active || wk != 0) return;

    // accumulator register r of lane l: column m = 32*g + l%32, row n = 32*nt + 8*(r/4) + 4*(l/32) + r%4
    const int hl = lane >> 5, ml = lane & 31;
    if (EPI == HX_EPI_PARTIAL) {
        float *y = a_y + blockIdx.y * a_split_stride;
#pragma unroll
        for (int g = 0; g < MG; ++g) {
            const int m = 32 * g + ml;
            if (m < a_M) {
#pragma unroll
                for (int j4 = 0; j4 < 4; ++j4) {
                    const int n = 32 * nt + 8 * j4 + 4 * hl;
                    if (n < a_N)
                        *(f32x4_t *)(y + (size_t)m * a_N + n) =
                            f32x4_t{acc[g][4 * j4], acc[g][4 * j4 + 1], acc[g][4 * j4 + 2], acc[g][4 * j4 + 3]};
                }
            }
        }
    } else if (EPI == HX_EPI_SWIGLU) {
        // rows 0..15 of the tile are gate columns 16*nt + p, rows 16..31 the matching up columns
#pragma unroll
        for (int g = 0; g < MG; ++g) {
            const int m = 32 * g + ml;
            if (m < a_M) {
#pragma unroll
                for (int j4 = 0; j4 < 2; ++j4) {
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const float gt = acc[g][4 * j4 + i], up = acc[g][8 + 4 * j4 + i];
                        v[i] = (gt / (1.0f + expf(-gt))) * up;
                    }
                    uint2 pk;
                    pk.x = hx_cvt_pk_bf16(v[0], v[1]);
                    pk.y = hx_cvt_pk_bf16(v[2], v[3]);
                    *(uint2 *)(a_mp + hx_xp_index(m, 16 * nt + 8 * j4 + 4 * hl, MG)) = pk;
                }
            }
        }
    } else {
        const hx_lm_args lm{a_y, a_M, a_N, a_n_tiles, a_amax_val, a_amax_idx, a_positions, a_row_ids, a_inv_t, a_key0, a_key1,
                            a_samp_z, a_samp_m, a_samp_s};
        // one copy of the tile's code, the accumulators moved up behind it (unrolled it spills and leaves the instruction
        // cache; the last is cleared, or it would stay live; a drawn head's lane number is taken anew: kept, it was one register too many for two
        // workgroups, and went to scratch memory); m-groups that only pad the batch are left out
#pragma unroll 1
        for (int g = 0; g < MG && 32 * g < a_M; ++g) {
            const f32x16_t now = acc[0];
#pragma unroll
            for (int k = 0; k + 1 < MG; ++k) acc[k] = acc[k + 1];
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[MG - 1][r] = 0.f;
            if (EPI == HX_EPI_LOGITS) hx_lm_greedy_tile(lm, now, 32 * g + ml, nt, lane);
            else                      hx_lm_sample_tile<(MG <= 2)>(lm, now, 32 * g + (int)(__lane_id() & 31), nt, lane);
        }
    }
}

// ---- host side: one launch of a given shape -----------------------------------------------------------------------
#define HX_GEMM_ARGS a.wp, a.xp, a.k_steps, a.n_tiles, a.steps_per_split, a.steps_per_wave, a.M, a.N, a.y, a.split_stride, a.mp, \
                     a.amax_val, a.amax_idx, a.positions, a.row_ids, a.inv_t, a.key0, a.key1, a.samp_z, a.samp_m, a.samp_s

template <int MG, int WN, int WK, int EPI>
static int launch_one(dim3 grid, hipStream_t st, const GemmArgs &a) {
    constexpr int RING = gemm_ring<MG, WN, EPI>();
    constexpr int lds = gemm_lds_bytes<MG, WN, WK, RING>();
    // the opt-in for more than 64 KiB of LDS is per kernel: once per instantiation, whichever thread comes first
    static std::once_flag once;
    static hipError_t configured = hipSuccess;
    std::call_once(once, [] {
        configured = hipFuncSetAttribute((const void *)gemm_stream_kernel<MG, WN, WK, EPI>,
                                         hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    });
    if (configured != hipSuccess) return hx_fail(HX_E_HIP, "hipFuncSetAttribute: %s", hipGetErrorString(configured));
    dim3 block(64 * (WN * WK + GemmGeom<MG, WK, RING>::NP));
    hipLaunchKernelGGL((gemm_stream_kernel<MG, WN, WK, EPI>), grid, block, lds, st, HX_GEMM_ARGS);
    return HX_OK;
}

template <int MG, int WN, int WK>
static int launch_epi(int epilogue, dim3 grid, hipStream_t st, const GemmArgs &a) {
    if (epilogue == HX_EPI_PARTIAL) return launch_one<MG, WN, WK, HX_EPI_PARTIAL>(grid, st, a);
    if (epilogue == HX_EPI_SWIGLU) return launch_one<MG, WN, WK, HX_EPI_SWIGLU>(grid, st, a);
    if (epilogue == HX_EPI_SAMPLE) return launch_one<MG, WN, WK, HX_EPI_SAMPLE>(grid, st, a);
    return launch_one<MG, WN, WK, HX_EPI_LOGITS>(grid, st, a);
}

template <int MG>
static int launch_shape(int wn, int wk, int epilogue, dim3 grid, hipStream_t st, const GemmArgs &a) {
    if (wk == 1) {
        if (wn == 4) return launch_epi<MG, 4, 1>(epilogue, grid, st, a);
        if (wn == 5) return launch_epi<MG, 5, 1>(epilogue, grid, st, a);
        if (wn == 6) return launch_epi<MG, 6, 1>(epilogue, grid, st, a);
    }
    if (wn == 4 && wk == 2) return launch_epi<MG, 4, 2>(epilogue, grid, st, a);
    // ten n-tiles per workgroup (twelve wavefronts): only for products that run in several rounds (the LM head)
    if (wn == 10 && wk == 1 && epilogue != HX_EPI_PARTIAL) {
        if (epilogue == HX_EPI_SWIGLU) return launch_one<MG, 10, 1, HX_EPI_SWIGLU>(grid, st, a);
        if (epilogue == HX_EPI_SAMPLE) return launch_one<MG, 10, 1, HX_EPI_SAMPLE>(grid, st, a);
        return launch_one<MG, 10, 1, HX_EPI_LOGITS>(grid, st, a);
    }
    return hx_fail(HX_E_RANGE, "unsupported product shape wn=%d wk=%d for %d m-groups", wn, wk, MG);
}

// ---- host side: how to cut one product into launches ---------------------------------------------------------------
// Measured on MI355X, wn x 1 shapes (wn n-tiles sharing one activation stream) are the fastest.  The planner picks wn in
// {4, 5, 6, 10} -- and, for products whose consumer kernel sums split partials, the number of K-splits (at most
// HX_MAX_SPLITS, at least 16 k-steps each) -- that minimises the time of the busiest compute unit in a model fitted at 128 rows,
// where a workgroup occupies a compute unit (128 KiB of LDS), a launch runs in rounds of as many workgroups as the device has
// compute units (hx_device_cus) and a partly filled last round costs a full one: rounds x (wn tiles + 3 tile-times for the
// round's own copy of the activations, which every workgroup draws from the L2 whatever its width) x revolutions of
// PLAN_STEPS k-steps; split products, which run in one round and read only a K-slice of the activations, keep a small charge
// per extra tile instead (five consumers on four SIMDs); ties go to the smaller wn and fewer splits.  Fewer rows take
// the same plan, though their rings are of 8 and their workgroups take a quarter of the LDS or less: the splits decide
// in which order a row's products are added, and so a row comes out alike in every batch of up to 128.
// Examples: the 1184 tiles of the 7B gate|up matrix make 296 workgroups of 4 (two rounds on 256 compute
// units) but 237 workgroups of 5 (one round); the 4752 tiles of the LM head make five rounds of 4, four of 5 or
// two of 10, measured 253 / 244 / 230 us.  Ten tiles per workgroup are twelve wavefronts (three per SIMD): only
// for products without split partials.  Matrices of few columns go to gemm_slice.hip (hx_plan_slice).  HX_GEMM_SHAPE="wn,wk,splits" overrides
// (tuning).  Batches of more than 128 rows: hx_plan_wide, under the same two knobs.
constexpr int PLAN_STEPS = 16;

struct gemm_launch { int wn, wk, splits, slice_tiles; };     // slice_tiles > 0: gemm_slice.hip, with these K-splits

// HX_GEMM_MAX_SPLITS, and HX_GEMM_SHAPE="wn,wk,splits"
static int splits_allowed(int most) {
    const char *cap = getenv("HX_GEMM_MAX_SPLITS");
    return cap ? std::max(1, std::min(most, atoi(cap))) : most;
}
static bool forced_shape(int *wn, int *wk, int *splits) {
    const char *ov = getenv("HX_GEMM_SHAPE");
    return ov && sscanf(ov, "%d,%d,%d", wn, wk, splits) == 3 && *splits >= 1;
}

// Up to 128 rows.
static gemm_launch plan_product(int n_tiles, int k_steps, int rows, int epilogue) {
    const int cus = hx_device_cus();
    const bool partial = epilogue == HX_EPI_PARTIAL;
    gemm_launch best{4, 1, 1, 0};
    double best_cost = 1e300;
    const int max_s = partial ? splits_allowed(HX_MAX_SPLITS) : 1;
    int a, b, c;
    if (forced_shape(&a, &b, &c) && c <= max_s && ((b == 1 && a >= 4 && a <= 6) || (a == 4 && b == 2)) && k_steps / (b * c) >= 1)
        return gemm_launch{a, b, c, 0};
    const hx_slice_plan slice = hx_plan_slice(n_tiles, k_steps, rows, epilogue, max_s);
    if (slice.tiles) return gemm_launch{4, 1, slice.splits, slice.tiles};
    static const int widths[] = {4, 5, 6, 10};
    for (int wn : widths) {
        if (wn == 10 && partial) continue;
        for (int s = 1; s <= max_s; ++s) {
            if (s > 1 && k_steps / s < 16) break;
            const int wgs = ((n_tiles + wn - 1) / wn) * s;
            const int rounds = (wgs + cus - 1) / cus;
            const int sps = (k_steps + s - 1) / s;
            // busiest compute unit: rounds x (wn tiles + the activations) x whole revolutions (one more to fill
            // the ring), plus a small charge per split for writing and re-reading its partial tile
            const int revolutions = (sps + PLAN_STEPS - 1) / PLAN_STEPS + 1;
            const double width = partial ? wn + 0.35 * (wn - 4) : wn + 3.0;   // as measured on each kind
            const double cost = (double)rounds * width * revolutions * (1.0 + 0.02 * (s - 1));
            if (cost < best_cost - 1e-9) { best_cost = cost; best.wn = wn; best.splits = s; }
        }
    }
    return best;
}

// Beyond 128 rows: the workgroup-tiled product of gemm_wide.hip, one block of 256 rows, those past the batch computed and never
// read; its partials are 256 rows apart, so fewer splits fit the buffer of an engine for fewer rows.  Matrices of few columns
// (slice.tiles > 0): gemm_slice.hip, unless a shape is forced.  knobs: whether the environment has a say (a block of prompt rows plans its own).
static bool wide_rows(int batch) { return batch > 128; }
struct batch_plan { hx_wide_plan wide; hx_slice_plan slice; };
static batch_plan plan_wide_batch(const hx_matrix *m, int epilogue, int max_batch, bool knobs) {
    const bool partial = epilogue == HX_EPI_PARTIAL;
    auto allowed = [&](int most) { return !partial ? 1 : knobs ? splits_allowed(most) : most; };
    const int max_s = allowed(HX_MAX_SPLITS * max_batch / 256);
    batch_plan plan{hx_plan_wide(m, 1, epilogue, max_s), hx_slice_plan{0, 1}};
    int wn, wk, sp;                                      // forced: 4 to 8 tiles, no k-slices, no split without k-steps
    if (knobs && forced_shape(&wn, &wk, &sp) && wk == 1 && wn >= 4 && wn <= 8 && sp <= max_s && (sp - 1) * hx_wide_split_steps(m, sp) < m->k_steps)
        plan.wide = hx_wide_plan{wn, sp};
    else
        plan.slice = hx_plan_slice(m->n_tiles, m->k_steps, 256, epilogue, allowed(HX_MAX_SPLITS));
    return plan;
}

// The plan of one product, for inspection: tiles per workgroup, k-slices per workgroup, K-splits.  Beyond 128 rows as an
// engine for 256 rows runs it; of few columns only the splits are the plan's.
extern "C" int hx_plan_product(int32_t n_tiles, int32_t k_steps, int32_t batch, int32_t partial, int32_t *wn_out,
                               int32_t *wk_out, int32_t *splits_out) {
    if (!wn_out || !wk_out || !splits_out) return hx_fail(HX_E_NULL, "an output pointer is NULL");
    if (n_tiles < 1 || k_steps < 1 || batch < 1 || batch > 256) return hx_fail(HX_E_RANGE, "product %d x %d for batch %d", n_tiles, k_steps, batch);
    if (wide_rows(batch)) {
        const hx_matrix m{0, 16 * k_steps, 32 * n_tiles, k_steps, n_tiles};
        const batch_plan plan = plan_wide_batch(&m, partial ? HX_EPI_PARTIAL : HX_EPI_SWIGLU, 256, true);
        *wn_out = plan.slice.tiles ? 4 : plan.wide.wnt; *wk_out = 1; *splits_out = plan.slice.tiles ? plan.slice.splits : plan.wide.splits;
        return HX_OK;
    }
    const gemm_launch plan = plan_product(n_tiles, k_steps, batch, partial ? HX_EPI_PARTIAL : HX_EPI_SWIGLU);
    *wn_out = plan.wn; *wk_out = plan.wk; *splits_out = plan.splits;
    return HX_OK;
}

int hx_launch_gemm(const hx_engine *e, const hx_matrix *m, int batch, const void *xp, int epilogue, float *y,
                   void *mp_out, hipStream_t st, const hx_sample_params *sample, hx_partials *parts, bool prompt_block) {
    if (epilogue == HX_EPI_SAMPLE && !sample) return hx_fail(HX_E_NULL, "sampling parameters missing");
    const int mg = hx_m_groups(batch);
    const bool partial = epilogue == HX_EPI_PARTIAL;
    const hx_lm_args lm{y, batch, m->N, m->n_tiles, (float *)(e->ws + e->map.amax_val), (int32_t *)(e->ws + e->map.amax_idx),
                        sample ? sample->positions : nullptr, sample ? sample->row_ids : nullptr,
                        sample ? sample->inv_temperature : 1.0f, sample ? sample->key0 : 0u, sample ? sample->key1 : 0u,
                        (float *)(e->ws + e->map.samp_z), (float *)(e->ws + e->map.samp_m), (float *)(e->ws + e->map.samp_s)};
    if (wide_rows(batch)) {
        const batch_plan plan = plan_wide_batch(m, epilogue, e->cfg.max_batch, !prompt_block);
        if (parts) *parts = plan.slice.tiles ? hx_partials{plan.slice.splits, (size_t)batch * m->N} : hx_partials{plan.wide.splits, (size_t)256 * m->N};
        if (plan.slice.tiles) return hx_launch_gemm_slice(e, m, batch, plan.slice, xp, epilogue, y, mp_out, lm, st);
        // The streaming kernel has one wavefront per SIMD with all rows' accumulators, and nothing beside its multiplications
        // or its epilogue; the workgroup-tiled product has two.  LM head, 1.5B, 256 rows, sampled: 327 -> 204 us; the other
        // products: see hx_plan_wide.
        return hx_launch_gemm_wide(e, m, 1, e->ws, 0, (const char *)xp - e->ws, epilogue, partial ? (char *)y - e->ws : 0,
                                   mp_out ? (char *)mp_out - e->ws : 0, plan.wide, st, &lm, batch);
    }
    const gemm_launch pl = plan_product(m->n_tiles, m->k_steps, batch, epilogue);
    if (parts) *parts = hx_partials{pl.splits, (size_t)batch * m->N};
    if (pl.slice_tiles)
        return hx_launch_gemm_slice(e, m, batch, hx_slice_plan{pl.slice_tiles, pl.splits}, xp, epilogue, y, mp_out, lm, st);
    GemmArgs a;
    a.wp = (const uint4 *)(e->weights + m->offset);
    a.xp = (const uint4 *)xp;
    a.k_steps = m->k_steps;
    a.n_tiles = m->n_tiles;
    a.steps_per_split = (m->k_steps + pl.splits - 1) / pl.splits;
    a.steps_per_wave = (a.steps_per_split + pl.wk - 1) / pl.wk;
    a.M = batch;
    a.N = m->N;
    a.y = y;
    a.split_stride = (size_t)batch * m->N;
    a.mp = (uint16_t *)mp_out;
    a.amax_val = lm.amax_val;
    a.amax_idx = lm.amax_idx;
    a.positions = lm.positions;
    a.row_ids = lm.row_ids;
    a.inv_t = lm.inv_t;
    a.key0 = lm.key0;
    a.key1 = lm.key1;
    a.samp_z = lm.samp_z;
    a.samp_m = lm.samp_m;
    a.samp_s = lm.samp_s;
    dim3 grid((m->n_tiles + pl.wn - 1) / pl.wn, pl.splits);
    int rc;
    switch (mg) {
        case 1: rc = launch_shape<1>(pl.wn, pl.wk, epilogue, grid, st, a); break;
        case 2: rc = launch_shape<2>(pl.wn, pl.wk, epilogue, grid, st, a); break;
        case 4: rc = launch_shape<4>(pl.wn, pl.wk, epilogue, grid, st, a); break;
        default: return hx_fail(HX_E_RANGE, "%d rows for the streaming product", batch);
    }
    if (rc) return rc;
    HX_CHECK_LAUNCH("gemm_stream");
    return HX_OK;
}

// ---- the token of each row from its per-tile candidates -------------------------------------------------------
// One workgroup per row, of 1024 threads (256 where a row has at most 1024 tiles).  A row's 4752 tiles (7B) are 5 per thread,
// all requested before the first is used: what bounds these kernels is the latency of their loads and of the merges behind them,
// not their bytes.  Of the sums every lane weighs its own once, and the wavefronts' results are merged by one of them: 37 rows of
// 4752 tiles 5.5 us sampled, 3 rows 4.9, 128 rows 6.1, 256 rows 8.0 (four tiles per trip, every merge weighed, the wavefronts' one
// after the other by one thread: 9.1, 8.6, 10.1, 12.0).
#define HX_FINAL_THREADS 1024
#define HX_FINAL_UNROLL 5

// Largest value wins, ties go to the smaller index; fixed order, so the result does not depend on the timing.
__device__ __forceinline__ void keep_best(float &v, int32_t &i, float &z, float ov, int32_t oi, float oz) {
    if (ov > v || (ov == v && oi < i)) { v = ov; i = oi; z = oz; }
}

__global__ __launch_bounds__(HX_FINAL_THREADS) void argmax_final_kernel(const float *__restrict__ val, const int32_t *__restrict__ idx,
                                                                        int n_tiles, int32_t *__restrict__ out) {
    __shared__ float sv[HX_FINAL_THREADS / 64];
    __shared__ int32_t si[HX_FINAL_THREADS / 64];
    const int m = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const size_t base = (size_t)m * n_tiles;
    float best = -INFINITY, none = 0.f;
    int32_t bi = 0x7fffffff;
    for (int t0 = tid; t0 < n_tiles; t0 += nt * HX_FINAL_UNROLL) {
        float v[HX_FINAL_UNROLL];
        int32_t ix[HX_FINAL_UNROLL];
#pragma unroll
        for (int u = 0; u < HX_FINAL_UNROLL; ++u) {
            const int t = min(t0 + u * nt, n_tiles - 1);      // past the end: the last again, which changes nothing
            v[u] = val[base + t]; ix[u] = idx[base + t];
        }
#pragma unroll
        for (int u = 0; u < HX_FINAL_UNROLL; ++u) keep_best(best, bi, none, v[u], ix[u], 0.f);
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) keep_best(best, bi, none, __shfl_xor(best, off), __shfl_xor(bi, off), 0.f);
    if ((tid & 63) == 0) { sv[tid >> 6] = best; si[tid >> 6] = bi; }
    __syncthreads();
    if (tid >= 64) return;
    const int w = min(tid, nt / 64 - 1);
    best = sv[w];
    bi = si[w];
#pragma unroll
    for (int off = HX_FINAL_THREADS / 128; off > 0; off >>= 1) keep_best(best, bi, none, __shfl_xor(best, off), __shfl_xor(bi, off), 0.f);
    if (tid == 0) out[m] = bi;
}

int hx_launch_argmax_final(const hx_engine *e, int batch, int32_t *tokens_out, hipStream_t st) {
    hipLaunchKernelGGL(argmax_final_kernel, dim3(batch), dim3(e->wlm.n_tiles <= 1024 ? 256 : HX_FINAL_THREADS), 0, st, (const float *)(e->ws + e->map.amax_val),
                       (const int32_t *)(e->ws + e->map.amax_idx), e->wlm.n_tiles, tokens_out);
    HX_CHECK_LAUNCH("argmax_final");
    return HX_OK;
}

// The sampled token and its log-probability: largest perturbed score (ties: smaller column); log-sum-exp of the scaled
// logits = M + log(S) from the tiles' (max, sum of exp(z - max)): the maximum over the lanes first, so that each weighs its own sum
// once, and the sums in a fixed order.
__device__ __forceinline__ void lse_over_lanes(float &M, float &S, int lanes) {
    const float own = M;
    for (int off = lanes / 2; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
    if (M > -INFINITY) S *= expf(own - M);                         // all -inf: nothing to weigh
    for (int off = lanes / 2; off > 0; off >>= 1) S += __shfl_xor(S, off);
}

__global__ __launch_bounds__(HX_FINAL_THREADS) void sample_final_kernel(const float *__restrict__ val, const int32_t *__restrict__ idx,
                                                                        const float *__restrict__ zc, const float *__restrict__ tm,
                                                                        const float *__restrict__ tsum, int n_tiles,
                                                                        int32_t *__restrict__ tok_out, float *__restrict__ lp_out) {
    constexpr int NW = HX_FINAL_THREADS / 64, U = HX_FINAL_UNROLL;
    __shared__ float sv[NW], sz[NW], sm[NW], ss[NW];
    __shared__ int32_t si[NW];
    const int m = blockIdx.x, tid = threadIdx.x, nt = blockDim.x;
    const size_t base = (size_t)m * n_tiles;
    float best = -INFINITY, bz = 0.f, M = -INFINITY, S = 0.f;
    int32_t bi = 0x7fffffff;
    for (int t0 = tid; t0 < n_tiles; t0 += nt * U) {
        float v[U], z[U], mt[U], st[U];
        int32_t ix[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int t = min(t0 + u * nt, n_tiles - 1);
            v[u] = val[base + t]; ix[u] = idx[base + t]; z[u] = zc[base + t];
            mt[u] = tm[base + t]; st[u] = tsum[base + t];
        }
        float mc = M;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            keep_best(best, bi, bz, v[u], ix[u], z[u]);
            mc = fmaxf(mc, mt[u]);
        }
        if (mc > -INFINITY) {
            S *= expf(M - mc);
#pragma unroll
            for (int u = 0; u < U; ++u)
                if (t0 + u * nt < n_tiles) S += st[u] * expf(mt[u] - mc);
        }
        M = mc;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) keep_best(best, bi, bz, __shfl_xor(best, off), __shfl_xor(bi, off), __shfl_xor(bz, off));
    lse_over_lanes(M, S, 64);
    if ((tid & 63) == 0) { const int w = tid >> 6; sv[w] = best; si[w] = bi; sz[w] = bz; sm[w] = M; ss[w] = S; }
    __syncthreads();
    if (tid >= 64) return;
    const int w = min(tid, nt / 64 - 1);
    best = sv[w];
    bi = si[w];
    bz = sz[w];
    M = sm[w];
    S = tid < nt / 64 ? ss[w] : 0.f;
#pragma unroll
    for (int off = NW / 2; off > 0; off >>= 1) keep_best(best, bi, bz, __shfl_xor(best, off), __shfl_xor(bi, off), __shfl_xor(bz, off));
    lse_over_lanes(M, S, NW);
    if (tid == 0) {
        tok_out[m] = bi;
        lp_out[m] = bz - (M + logf(S));
    }
}

int hx_launch_sample_final(const hx_engine *e, int batch, int32_t *tokens_out, float *logprobs_out, hipStream_t st) {
    hipLaunchKernelGGL(sample_final_kernel, dim3(batch), dim3(e->wlm.n_tiles <= 1024 ? 256 : HX_FINAL_THREADS), 0, st, (const float *)(e->ws + e->map.amax_val),
                       (const int32_t *)(e->ws + e->map.amax_idx), (const float *)(e->ws + e->map.samp_z),
                       (const float *)(e->ws + e->map.samp_m), (const float *)(e->ws + e->map.samp_s), e->wlm.n_tiles,
                       tokens_out, logprobs_out);
    HX_CHECK_LAUNCH("sample_final");
    return HX_OK;
}
