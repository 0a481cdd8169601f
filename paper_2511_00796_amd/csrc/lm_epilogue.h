// What the LM head does with a 32 x 32 tile of logits out of its accumulators, shared by the streaming product (gemm.hip)
// and the workgroup-tiled one (gemm_wide.hip): store the logits, and leave per (row, tile) the candidates from which the
// row kernels choose the token.
#pragma once
#include "hx_internal.h"

struct hx_lm_args {
    float *y;                     // logits [M][N] or NULL
    int M, N, n_tiles;
    float *amax_val;              // [M][n_tiles]: largest logit, or best perturbed score, of the tile
    int32_t *amax_idx;            // its column
    // sampling only
    const int32_t *positions, *row_ids;
    float inv_t;
    uint32_t key0, key1;
    float *samp_z, *samp_m, *samp_s;   // [M][n_tiles]: scaled logit of the candidate, tile max, tile sum of exp(z - max)
};

// exp(t) for t <= 0, to about one unit in the last place: 2^(t log2 e) with the rounding error of the product and the low
// part of log2 e put back to first order.  Below e^-100 (it only enters sums of at least 1) and at -inf: 0.
__device__ __forceinline__ float hx_exp_nonpositive(float t) {
    const float r = t * 1.44269502f;
    const float lost = fmaf(t, 1.44269502f, -r) + t * 1.92596299e-8f;
    const float e = __builtin_amdgcn_exp2f(r);
    return t < -100.0f ? 0.0f : fmaf(e * 0.693147182f, lost, e);
}

// accumulator register r of lane l: row m = m0 + l % 32, column 32 * nt + 8 * (r / 4) + 4 * (l / 32) + r % 4
__device__ __forceinline__ void hx_lm_greedy_tile(const hx_lm_args &a, const f32x16_t &acc, int m, int nt, int lane) {
    const int hl = lane >> 5;
    float best = -INFINITY;
    int best_n = 0x7fffffff;
#pragma unroll
    for (int j4 = 0; j4 < 4; ++j4) {
        const int n = 32 * nt + 8 * j4 + 4 * hl;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = acc[4 * j4 + i];
            if (n + i < a.N && v > best) { best = v; best_n = n + i; }
        }
        if (a.y != nullptr && m < a.M && n < a.N)
            *(f32x4_t *)(a.y + (size_t)m * a.N + n) = f32x4_t{acc[4 * j4], acc[4 * j4 + 1], acc[4 * j4 + 2], acc[4 * j4 + 3]};
    }
    const float ov = __shfl_xor(best, 32);
    const int on = __shfl_xor(best_n, 32);
    if (ov > best || (ov == best && on < best_n)) { best = ov; best_n = on; }
    if (hl == 0 && m < a.M) {
        a.amax_val[(size_t)m * a.n_tiles + nt] = best;
        a.amax_idx[(size_t)m * a.n_tiles + nt] = best_n;
    }
}

// Temperature sample by Gumbel-max, and the pieces of the log-sum-exp: per (row, tile) the best perturbed score y = z + g
// with its column and its z, the tile's max of z and its sum of exp(z - max).  z = logit * (1/T); g = -log(-log(u)); u from
// one generator block per 4 consecutive columns.
// This arithmetic bounds the LM head of a sampled step (about 100 vector operations per logit at first: a third of the
// head's time at 256 rows).  The tile's winner is therefore found with the two logarithms straight from v_log_f32, which
// are within 2e-5 of the exact score, and only the winner's score is computed exactly; where a lane's second best comes
// within a margin above twice that error, the whole tile is done exactly.  So the candidate is always the exact one.
// 7B head: 128 rows 249 -> 240 us, 37 rows 207 -> 200.
// LEAN, for kernels whose registers decide how many workgroups a compute unit holds (gemm_resident): the generator's blocks are kept
// one behind the other, and none of their products moves out of the caller's loop over rows; z takes the logits' registers, the exact
// pass is a loop, and a ragged tile has no copy of the code (136 registers -> 70).  With two or three wavefronts per SIMD the blocks
// hide each other's latencies: 7B at 128 rows 231 us, LEAN 234; 1.5B at 256 rows 187, LEAN 194.
template <bool LEAN>
__device__ __forceinline__ void hx_lm_sample_columns(const hx_lm_args &a, f32x16_t &z, uint32_t row, uint32_t pos, int n0,
                                                     float &best, int &best_n, float &best_z, float &zmax) {
    const auto uniform = [](uint32_t w) { return ((float)(w >> 9) + 0.5f) * (1.0f / 8388608.0f); };
    float top = -INFINITY, second = -INFINITY, top_u = 0.5f;
#pragma unroll
    for (int j4 = 0; j4 < 4; ++j4) {
        const int n = n0 + 8 * j4;
        uint32_t w[4];
        hx_philox4x32_10((uint32_t)(n >> 2), row, pos, 0x53414D50u, a.key0, a.key1, w);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = 4 * j4 + i;
            z[r] *= a.inv_t;
            const float u = uniform(w[i]);
            const float g2 = __builtin_amdgcn_logf(-__builtin_amdgcn_logf(u));          // log2(-log2(u))
            const float ya = fmaf(-0.693147182f, g2, z[r]);                             // y, less the constant log(log 2)
            second = fmaxf(second, fminf(top, ya));
            if (ya > top) { top = ya; top_u = u; best_z = z[r]; best_n = n + i; }
            zmax = fmaxf(zmax, z[r]);
        }
        if (LEAN) __builtin_amdgcn_sched_barrier(0);
    }
    best = best_z - logf(-logf(top_u));
    if (__any(second >= top - (1e-4f + 1e-6f * fabsf(top)))) {         // also both -inf, or a lane with an infinite score
        best = -INFINITY; best_z = 0.f; best_n = 0x7fffffff;          // rare: the numbers are generated again, not kept
#pragma unroll 1
        for (int j4 = 0; j4 < 4; ++j4) {
            const int n = n0 + 8 * j4;
            uint32_t w[4];
            hx_philox4x32_10((uint32_t)(n >> 2), row, pos, 0x53414D50u, a.key0, a.key1, w);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float zi = j4 == 0 ? z[i] : j4 == 1 ? z[4 + i] : j4 == 2 ? z[8 + i] : z[12 + i];
                const float y = zi - logf(-logf(uniform(w[i])));
                if (y > best) { best = y; best_z = zi; best_n = n + i; }
            }
        }
    }
}

template <bool LEAN>
__device__ __forceinline__ void hx_lm_sample_tile(const hx_lm_args &a, f32x16_t z, int m, int nt, int lane) {
    const int hl = lane >> 5;
    int n0 = 32 * nt + 4 * hl;
    if (LEAN) asm volatile("" : "+v"(n0));               // opaque
    const bool row_ok = m < a.M;
    const uint32_t row = row_ok ? (a.row_ids ? (uint32_t)a.row_ids[m] : (uint32_t)m) : 0u;
    const uint32_t pos = row_ok ? (uint32_t)a.positions[m] : 0u;
    float best = -INFINITY, best_z = 0.f, zmax = -INFINITY;
    int best_n = 0x7fffffff;
    if (a.y != nullptr && row_ok) {
#pragma unroll
        for (int j4 = 0; j4 < 4; ++j4) {
            const int n = n0 + 8 * j4;
            if (n < a.N) *(f32x4_t *)(a.y + (size_t)m * a.N + n) = f32x4_t{z[4 * j4], z[4 * j4 + 1], z[4 * j4 + 2], z[4 * j4 + 3]};
        }
    }
    if (32 * nt + 32 > a.N) {                            // columns that do not exist: neither drawn nor weighed
#pragma unroll
        for (int r = 0; r < 16; ++r) if (n0 + 8 * (r >> 2) + (r & 3) >= a.N) z[r] = -INFINITY;
    }
    if (LEAN) __builtin_amdgcn_sched_barrier(0);
    hx_lm_sample_columns<LEAN>(a, z, row, pos, n0, best, best_n, best_z, zmax);
    // the two half-wavefronts hold the two halves of the tile's 32 columns
    const float tmax = fmaxf(zmax, __shfl_xor(zmax, 32));
    float sum = 0.f;
    if (tmax > -INFINITY) {
#pragma unroll
        for (int i = 0; i < 16; ++i) sum += hx_exp_nonpositive(z[i] - tmax);     // 0 for columns past N
    }
    sum += __shfl_xor(sum, 32);
    const float oy = __shfl_xor(best, 32), oz = __shfl_xor(best_z, 32);
    const int on = __shfl_xor(best_n, 32);
    if (oy > best || (oy == best && on < best_n)) { best = oy; best_n = on; best_z = oz; }
    if (hl == 0 && row_ok) {
        const size_t o = (size_t)m * a.n_tiles + nt;
        a.amax_val[o] = best;
        a.amax_idx[o] = best_n;
        a.samp_z[o] = best_z;
        a.samp_m[o] = tmax;
        a.samp_s[o] = sum;
    }
}
