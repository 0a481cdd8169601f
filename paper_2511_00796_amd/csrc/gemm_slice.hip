// Small products: those whose matrix has too few column tiles to give the streaming kernel of gemm.hip (four
// and more tiles per workgroup, at most 9 K-splits, none of gate|up) a workgroup for every compute unit.
//
// Workgroup = four wavefronts on one or two 32-column tiles: k-step i of the split goes to wavefront i % 4, so the
// workgroup reads its tile's weights as one contiguous run.  A wavefront loads its weights and activations straight into
// registers, R steps ahead; no LDS stages, no barrier until the end, where the four sums are added in order through LDS, laid out
// so that the outputs leave in whole 128-byte lines.
// What bounds it is the round trips of a launch: a ring's fill, and the end.  That the activations of every tile come through
// the ring, which returns in order behind the weights, makes it slower than the streaming kernel wherever the weights are
// many: 14B gate|up at 64 rows 73 us (two tiles per workgroup 56), 48 there.  us, streaming -> this, 1 / 64 / 128 rows:
// 1.5B QKV 3.9 / 7.5 / 10.5 -> 2.7 / 4.3 / 7.0, O 4.5 / 7.1 / 9.5 -> 3.4 / 4.1 / 6.0, down 10.0 / 14.3 / 16.8 -> 8.6 / 11.2 / 13.0
// (two tiles; one: 7.6 / 10.4 / 13.6), with weights that are partly in the memory-side cache.
// Beyond 128 rows a workgroup takes 64 of them (two tiles: 128), and the row blocks of a tile, numbered so that one XCD takes them all, read its
// weights again, from that XCD's L2 (so they are ordinary loads there).  Numbered block by block, tiles times splits that were no multiple of 8 put
// them on different XCDs, and each fetched the weights from memory: down products at 129 rows with the packing of the
// input and the sum of the splits, weights from memory: 62 tiles of 1024 k-steps 47.6 -> 39.8 us, 68 of 512 32.7 -> 28.0, 68 of 688 41.3 -> 35.4.  The workgroup-tiled kernel of gemm_wide.hip would give these matrices 40 to 112 of 256
// compute units a workgroup.  us, there -> this, 160 / 256
// rows, weights from memory: 1.5B QKV 14.1 / 14.6 -> 7.4 / 7.7, O 14.1 / 15.0 -> 7.2 / 7.3, down 22.2 / 22.1 -> 15.6 / 16.6 (five splits; nine 21.2 / 22.2,
// one tile per workgroup 23.9 / 23.8); the tiny model's 9 to 13 -> 3 to 4.
#include "hx_internal.h"
#include "lm_epilogue.h"
#include <algorithm>

typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

namespace {

constexpr int SLICES = 4;         // wavefronts of a workgroup

// TN tiles per workgroup, MG of XG m-groups, R k-steps in flight per wavefront
template <int MG, int XG, int TN, int R, int EPI>
__global__ __launch_bounds__(64 * SLICES) void gemm_slice_kernel(const uint4 *__restrict__ a_wp, const uint4 *__restrict__ a_xp,
                                                               int a_k_steps, int a_n_tiles, int a_steps_per_split, int a_M, int a_N,
                                                               int a_split_stride, float *__restrict__ a_y, uint16_t *__restrict__ a_mp,
                                                               hx_lm_args a_lm) {
    constexpr int S = SLICES;
    constexpr int Q = TN * MG * 4;                       // 16-byte quads of accumulators per lane
    __shared__ u32x4_t red[S * Q * 64];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    int tg = blockIdx.x, split = blockIdx.y, g0 = 0;     // tile group, split, first m-group
    if (XG > MG) {
        // consecutive workgroup ids go to different XCDs: blockIdx.x is the XCD that takes all row blocks of a (group, split)
        const unsigned pair = 8 * blockIdx.z + blockIdx.x, groups = (unsigned)(a_n_tiles + TN - 1) / TN;
        split = pair / groups;
        tg = pair - split * groups;
        g0 = MG * blockIdx.y;
        if (split * a_steps_per_split >= a_k_steps) return;             // behind the last pair: no split is empty
    }
    const int t0 = tg * TN;
    const int split0 = split * a_steps_per_split, split1 = min(a_k_steps, split0 + a_steps_per_split);
    // step i of this wavefront is k-step split0 + wave + S * i
    const int n = (split1 - split0 - wave + S - 1) / S;
    const u32x4_t *wrow[TN];
#pragma unroll
    for (int t = 0; t < TN; ++t) wrow[t] = (const u32x4_t *)a_wp + ((size_t)min(t0 + t, a_n_tiles - 1) * a_k_steps + split0 + wave) * 64 + lane;
    const u32x4_t *xrow = (const u32x4_t *)a_xp + ((size_t)(split0 + wave) * XG + g0) * 64 + lane;
    f32x16_t acc[TN][MG];
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int g = 0; g < MG; ++g)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][g][r] = 0.f;
    if (n > 0) {
        u32x4_t w[R][TN], x[R][MG];
        auto request = [&](int r, int i) {
            const int j = S * min(i, n - 1);
#pragma unroll
            for (int t = 0; t < TN; ++t) w[r][t] = XG > MG ? wrow[t][(size_t)j * 64] : __builtin_nontemporal_load(wrow[t] + (size_t)j * 64);
#pragma unroll
            for (int g = 0; g < MG; ++g) x[r][g] = xrow[((size_t)j * XG + g) * 64];
            __builtin_amdgcn_sched_barrier(0);
        };
        auto multiply = [&](int r) {
#pragma unroll
            for (int t = 0; t < TN; ++t)
#pragma unroll
                for (int g = 0; g < MG; ++g)
                    acc[t][g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, w[r][t]), __builtin_bit_cast(bf16x8_t, x[r][g]),
                                                                        acc[t][g], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
#pragma unroll
        for (int r = 0; r < R; ++r) request(r, r);
        int i = 0;
        for (; i + R < n; i += R) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                multiply(r);
                request(r, i + r + R);
            }
        }
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (i + r < n) multiply(r);
    }
    // the slices' sums, added in order
#pragma unroll
    for (int t = 0; t < TN; ++t)
#pragma unroll
        for (int g = 0; g < MG; ++g)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4_t v = {acc[t][g][4 * j], acc[t][g][4 * j + 1], acc[t][g][4 * j + 2], acc[t][g][4 * j + 3]};
                // the row's place is turned by the quad's column group, so that eight lanes reading one row's eight groups of
                // columns meet eight different banks
                const int place = EPI == HX_EPI_PARTIAL ? (lane & 32) | ((lane & 31) ^ (2 * j + (lane >> 5))) : lane;
                red[(wave * Q + (t * MG + g) * 4 + j) * 64 + place] = __builtin_bit_cast(u32x4_t, v);
            }
    __syncthreads();
    auto sum = [&](int quad, int place) {
        f32x4_t v = __builtin_bit_cast(f32x4_t, red[quad * 64 + place]);
#pragma unroll
        for (int s = 1; s < S; ++s) v += __builtin_bit_cast(f32x4_t, red[(s * Q + quad) * 64 + place]);
        return v;
    };
    if (EPI == HX_EPI_PARTIAL) {
        // lane = (row of 8, group of 4 columns): 128 contiguous bytes per row
        float *y = a_y + (size_t)split * a_split_stride;
        const int nq = lane & 7;
        for (int u = wave; u < Q; u += S) {              // 8 rows of one tile
            const int t = u / (MG * 4), g = u / 4 % MG, ml = (u & 3) * 8 + (lane >> 3);
            const int m = 32 * (g0 + g) + ml, nn = 32 * (t0 + t) + 4 * nq;
            if (m < a_M && nn < a_N) {
                const f32x4_t v = sum((t * MG + g) * 4 + (nq >> 1), (nq & 1) * 32 + (ml ^ nq));
                *(f32x4_t *)(y + (size_t)m * a_N + nn) = v;
            }
        }
    } else if (EPI == HX_EPI_SWIGLU) {
        for (int u = wave; u < TN * MG; u += S) {
            const int t = u / MG, g = u % MG, h = lane >> 5, ml = lane & 31, m = 32 * (g0 + g) + ml;
            if (m < a_M && t0 + t < a_n_tiles) {
                uint32_t pk[4];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const f32x4_t gt = sum(u * 4 + h, q * 32 + ml), up = sum(u * 4 + h + 2, q * 32 + ml);
                    float v[4];
#pragma unroll
                    for (int i = 0; i < 4; ++i) v[i] = (gt[i] / (1.0f + expf(-gt[i]))) * up[i];
                    pk[2 * q] = hx_cvt_pk_bf16(v[0], v[1]);
                    pk[2 * q + 1] = hx_cvt_pk_bf16(v[2], v[3]);
                }
                *(uint4 *)(a_mp + hx_xp_index(m, 16 * (t0 + t) + 8 * h, XG)) = make_uint4(pk[0], pk[1], pk[2], pk[3]);
            }
        }
    } else {
        for (int u = (wave + tg) % S; u < TN * MG; u += S) {
            const int t = u / MG, g = u % MG;
            if (32 * (g0 + g) >= a_M || t0 + t >= a_n_tiles) continue;
            f32x16_t v;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x4_t q = sum(u * 4 + j, lane);
#pragma unroll
                for (int i = 0; i < 4; ++i) v[4 * j + i] = q[i];
            }
            if (EPI == HX_EPI_LOGITS) hx_lm_greedy_tile(a_lm, v, 32 * (g0 + g) + (lane & 31), t0 + t, lane);
            else                      hx_lm_sample_tile<true>(a_lm, v, 32 * (g0 + g) + (lane & 31), t0 + t, lane);
        }
    }
}

struct SliceArgs {
    const uint4 *wp, *xp;         // packed weights, packed activations
    int k_steps, n_tiles, steps_per_split, M, N, split_stride;      // split_stride: elements between the splits of y
    float *y;                     // PARTIAL: [splits][M][N]
    uint16_t *mp;                 // SWIGLU: packed bf16 output
    hx_lm_args lm;                // LM head
};

template <int MG, int XG, int TN, int R>
int launch_slice(int epilogue, const SliceArgs &a, int splits, hipStream_t st) {
    const int groups = (a.n_tiles + TN - 1) / TN, blocks = (a.M + 32 * MG - 1) / (32 * MG);
    const dim3 grid = XG > MG ? dim3(8, blocks, (groups * splits + 7) / 8) : dim3(groups, splits), block(64 * SLICES);
#define HX_SLICE(EPI)                                                                                                      \
    hipLaunchKernelGGL((gemm_slice_kernel<MG, XG, TN, R, EPI>), grid, block, 0, st, a.wp, a.xp, a.k_steps, a.n_tiles, a.steps_per_split, \
                       a.M, a.N, a.split_stride, a.y, a.mp, a.lm)
    if (epilogue == HX_EPI_PARTIAL) {
        HX_SLICE(HX_EPI_PARTIAL);
    } else if (epilogue == HX_EPI_SWIGLU) {
        HX_SLICE(HX_EPI_SWIGLU);
    } else if constexpr (TN == 1) {
        if (epilogue == HX_EPI_SAMPLE) HX_SLICE(HX_EPI_SAMPLE);
        else HX_SLICE(HX_EPI_LOGITS);
    } else {                                             // small heads are planned with one
        return hx_fail(HX_E_RANGE, "epilogue %d with %d tiles per workgroup: no such small product", epilogue, TN);
    }
#undef HX_SLICE
    HX_CHECK_LAUNCH("gemm_slice");
    return HX_OK;
}

}  // namespace

// Whether a product runs here: the streaming kernel's most workgroups, a quarter of the tiles times the
// most splits, would leave two fifths of the compute units without one (up to 68 tiles on 256: 17 workgroups of four in 9 splits are
// 153).  us at 1 / 64 / 128 rows, 68 tiles, there with its best splits -> here: 128 k-steps 4.4 / 7.4 / 11.9 -> 4.0 / 5.4 / 7.3, 544 k-steps
// 10.2 / 15.7 / 18.7 -> 8.4 / 13.3 / 16.6, LM head 11.5 / 20.1 / 23.1 -> 5.2 / 8.7 / 11.0; 112 tiles, 7B O, at 3 / 37 rows 7.7 / 11.4 there,
// 7.9 / 13.7 here.  K-splits: at least 24 k-steps each (1.5B QKV at 64 rows in 6 / 4 / 2 splits: 5.6 / 4.4 /
// 5.2 us) and no more workgroups than compute units; two tiles per workgroup where that still leaves long ones.  Up to 128 rows are one
// block; more are four of 64 or two of 128, whatever their number, so that a row's sums are added in one order in all such batches.
// Of more than 64 tiles only three such splits fit beyond 128 rows, and long ones lose (us at 129 / 256 rows, workgroup-tiled -> this, with packing and
// sum: 68 tiles of 512 k-steps 29.3 / 33.6 -> 28.0 / 31.3, 688 35.1 / 40.4 -> 35.4 / 39.2, 768 36.5 / 41.4 -> 37.8 / 41.6, 1280 50.1 / 56.8 -> 55.2 / 60.6; in four,
// 64 tiles of 1792 k-steps 62.5 / 69.1 -> 61.0 / 67.6): more than 240 k-steps each go to the workgroup-tiled kernel.
// Gate|up, which is not split, runs here in one round of one or two tiles per workgroup.  us, streaming -> this, 1 / 33 / 128 rows: 256 tiles of
// 128 k-steps 16.8 / 18.6 / 23.6 -> 8.8 / 10.5 / 14.4, 512 of 128 18.7 / 20.6 / 25.2 -> 13.5 / 14.6 / 19.6, 384 of 192 24.0 / 26.6 / 33.7 -> 17.0 /
// 18.2 / 25.2; 816 tiles, in two rounds of two, 21.7 / 25.4 / 29.8 -> 21.6 / 24.9 / 34.2.  Three tiles (up to 768) gain up to 64 rows and lose beyond: 560 of
// 96 (1.5B) 15.2 / 17.0 / 21.8 -> 13.2 / 14.8 / 26, 768 of 192 26.9 / 30.2 / 38.0 -> 25.3 / 26.4 / 46; as row blocks of 64 rows, two workgroups to a
// compute unit, still 2 to 4 % and 11 to 13 % at 65 to 128 rows.  One plan serves all batches of up to 128 rows (a row's products are added in
// one order in all of them), so three are left to the streaming kernel.
hx_slice_plan hx_plan_slice(int n_tiles, int k_steps, int rows, int epilogue, int max_splits) {
    const int cus = hx_device_cus();
    const bool partial = epilogue == HX_EPI_PARTIAL;
    hx_slice_plan p{0, 1};
    if (epilogue == HX_EPI_SWIGLU && rows <= 128) {
        const int t = (n_tiles + cus - 1) / cus;
        if (t <= 2) p.tiles = t;
        return p;
    }
    if ((n_tiles + 3) / 4 * HX_MAX_SPLITS * 5 > cus * 3) return p;
    p.tiles = partial && k_steps > 24 * HX_MAX_SPLITS ? 2 : 1;
    const int groups = (n_tiles + p.tiles - 1) / p.tiles * (rows <= 128 ? 1 : 4 / p.tiles);
    if (partial && rows > 128 && cus / groups < 4 && k_steps > 240 * (cus / groups)) return hx_slice_plan{0, 1};
    if (partial) p.splits = std::max(1, std::min({max_splits, k_steps / 24, cus / groups}));
    return p;
}

int hx_launch_gemm_slice(const hx_engine *e, const hx_matrix *m, int batch, hx_slice_plan plan, const void *xp, int epilogue, float *y,
                         void *mp_out, const hx_lm_args &lm, hipStream_t st) {
    SliceArgs a;
    a.wp = (const uint4 *)(e->weights + m->offset);
    a.xp = (const uint4 *)xp;
    a.k_steps = m->k_steps; a.n_tiles = m->n_tiles;
    a.steps_per_split = (m->k_steps + plan.splits - 1) / plan.splits;
    if ((plan.splits - 1) * a.steps_per_split >= m->k_steps) return hx_fail(HX_E_RANGE, "%d splits of %d k-steps: one is empty", plan.splits, m->k_steps);
    a.M = batch; a.N = m->N;
    a.y = y; a.split_stride = batch * m->N;
    a.mp = (uint16_t *)mp_out;
    a.lm = lm;
    // k-steps in flight: with eight of the fewest rows the first products wait for loads past the split's end (1.5B, 16 rows, QKV
    // 4.7 -> 4.1 us, O 4.5 -> 3.7 with four); at more rows 2 to 6 are alike, but for two tiles of 128 rows (2: 13.3, 3: 12.4)
    switch (hx_m_groups(batch) * 10 + plan.tiles) {
        case 11: return launch_slice<1, 1, 1, 4>(epilogue, a, plan.splits, st);
        case 21: return launch_slice<2, 2, 1, 6>(epilogue, a, plan.splits, st);
        case 41: return launch_slice<4, 4, 1, 4>(epilogue, a, plan.splits, st);
        case 81: return launch_slice<2, 8, 1, 6>(epilogue, a, plan.splits, st);
        case 12: return launch_slice<1, 1, 2, 6>(epilogue, a, plan.splits, st);
        case 22: return launch_slice<2, 2, 2, 6>(epilogue, a, plan.splits, st);
        case 42: return launch_slice<4, 4, 2, 3>(epilogue, a, plan.splits, st);
        case 82: return launch_slice<4, 8, 2, 3>(epilogue, a, plan.splits, st);
        default: return hx_fail(HX_E_RANGE, "%d rows, %d tiles per workgroup: no such small product", batch, plan.tiles);
    }
}
