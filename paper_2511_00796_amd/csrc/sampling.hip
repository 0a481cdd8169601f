// Nucleus (top-p) sampling of one step's logits (Holtzman et al., ICLR 2020), after temperature scaling:
// keep the most probable entries whose mass reaches top_p -- all entries with z_i >= tau, tau the largest
// threshold for which mass{z_i >= tau} >= top_p * total, so entries equal to the last kept one are kept --
// and draw from the kept set by Gumbel-max with the noise of the temperature sampler.
//
// One workgroup per row.  tau is found by a radix select on the 32-bit order-preserving key of z, most
// significant digit first (11, 11, 10 bits): each pass builds a histogram of probability MASS per digit among the
// entries that match the digits chosen so far, and walks it from the largest z down to the digit where the
// running mass reaches the target.  Mass is 40-bit fixed point, w_i = floor(exp(z_i - max z) * 2^40), added with
// integer LDS atomics: the sums are exact, so the kept set does not depend on the order of the additions and the
// kernel is deterministic.  The draw takes the tile winners that the LM head's sampling epilogue has left, on the whole
// chip (here, one workgroup per row, drawing again for every kept entry was 90 of 144 us at 64 rows of 152 064 logits).
// Three reads of the row (from the memory-side cache: the LM head has just written it).
#include "hx_internal.h"
#include <type_traits>

#define HX_NUC_THREADS 1024
#define HX_NUC_BINS 2048
#define HX_NUC_UNROLL 8
#define HX_NUC_TILES 4
#define HX_NUC_SCALE 1099511627776.0f   // 2^40

// ascending key order = descending z; -0 and +0 share a key
__device__ __forceinline__ uint32_t nucleus_key(float z) {
    const uint32_t b = __float_as_uint(z + 0.0f);
    return ~(b ^ ((b >> 31) ? 0xFFFFFFFFu : 0x80000000u));
}

// group q: entries 4 q .. 4 q + 3 of the row
__device__ __forceinline__ void load_group(const float *__restrict__ x, int V, int q, bool vec, float (&v)[4]) {
    const size_t at = 4 * (size_t)q;
    if (vec) {
        const f32x4_t t = *(const f32x4_t *)(x + at);
        v[0] = t[0]; v[1] = t[1]; v[2] = t[2]; v[3] = t[3];
    } else {
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = x[at + i < (size_t)V ? at + i : (size_t)V - 1];
    }
}
// groups q0, q0 + HX_NUC_THREADS, ..., all requested before the first is used (one group at a time, the
// passes waited for one load after the other: 38 round trips each over a 152 064-entry row); groups past the end repeat
// the last one and are skipped by the caller
__device__ __forceinline__ void load_groups(const float *__restrict__ x, int V, int q0, int n_groups, bool vec,
                                            float (&v)[HX_NUC_UNROLL][4]) {
#pragma unroll
    for (int u = 0; u < HX_NUC_UNROLL; ++u) load_group(x, V, min(q0 + u * HX_NUC_THREADS, n_groups - 1), vec, v[u]);
}

__global__ __launch_bounds__(HX_NUC_THREADS) void nucleus_kernel(
    const float *__restrict__ logits, int V, const float *__restrict__ cand_y, const int32_t *__restrict__ cand_i,
    const float *__restrict__ cand_z, const float *__restrict__ tile_zmax, int n_tiles,
    const int32_t *__restrict__ positions, const int32_t *__restrict__ row_ids, float inv_t, float top_p, uint32_t key0,
    uint32_t key1, int32_t *__restrict__ tok_out, float *__restrict__ lp_out, int32_t *__restrict__ size_out) {
    __shared__ unsigned long long hist[HX_NUC_BINS];
    __shared__ unsigned long long scan[HX_NUC_THREADS];
    __shared__ float redf[HX_NUC_THREADS / 64];
    __shared__ int32_t redi[HX_NUC_THREADS / 64], redc[HX_NUC_THREADS / 64];
    __shared__ float redz[HX_NUC_THREADS / 64];
    __shared__ unsigned long long sh_before, sh_mass;
    __shared__ uint32_t sh_digit;

    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *x = logits + (size_t)m * V;
    const bool vec = (V & 3) == 0;                // rows then start on 16-byte boundaries
    const int n_groups = (V + 3) >> 2;

    // max z from the LM head's per-tile maxima
    float mx = -INFINITY;
    for (int t = tid; t < n_tiles; t += HX_NUC_THREADS) mx = fmaxf(mx, tile_zmax[(size_t)m * n_tiles + t]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
    if (lane == 0) redf[wave] = mx;
    __syncthreads();
    mx = redf[0];
#pragma unroll
    for (int w = 1; w < HX_NUC_THREADS / 64; ++w) mx = fmaxf(mx, redf[w]);
    const float zmax = mx;
    __syncthreads();

    uint32_t prefix = 0;                          // digits chosen so far (the high bits of tau's key)
    unsigned long long before = 0, target = 0;    // mass of the entries above the chosen digits; mass to reach
    int shift = 32;
#pragma unroll 1
    for (int pass = 0; pass < 3; ++pass) {
        const int bits = pass < 2 ? 11 : 10;
        const int hi_shift = shift;               // entries must match prefix in the bits above hi_shift
        shift -= bits;
        for (int i = tid; i < HX_NUC_BINS; i += HX_NUC_THREADS) hist[i] = 0ull;
        __syncthreads();
        for (int q0 = tid; q0 < n_groups; q0 += HX_NUC_THREADS * HX_NUC_UNROLL) {
            float v[HX_NUC_UNROLL][4];
            load_groups(x, V, q0, n_groups, vec, v);
#pragma unroll
            for (int u = 0; u < HX_NUC_UNROLL; ++u) {
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if (4 * (q0 + u * HX_NUC_THREADS) + i >= V) continue;
                    const float z = v[u][i] * inv_t;
                    const uint32_t key = nucleus_key(z);
                    if (pass == 0 || (key >> hi_shift) == prefix) {
                        const unsigned long long w = (unsigned long long)(expf(z - zmax) * HX_NUC_SCALE);
                        if (w) atomicAdd(&hist[(key >> shift) & ((1u << bits) - 1u)], w);
                    }
                }
            }
        }
        __syncthreads();
        // inclusive scan of the bins in key order, two bins per thread
        const unsigned long long h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
        unsigned long long incl = h0 + h1;
        scan[tid] = incl;
        __syncthreads();
#pragma unroll 1
        for (int off = 1; off < HX_NUC_THREADS; off <<= 1) {
            const unsigned long long add = tid >= off ? scan[tid - off] : 0ull;
            __syncthreads();
            incl += add;
            scan[tid] = incl;
            __syncthreads();
        }
        if (pass == 0) {
            // every entry was counted: the total fixes the target, at least one unit and at most everything
            const unsigned long long total = scan[HX_NUC_THREADS - 1];
            const double want = ceil((double)top_p * (double)total);
            target = want < 1.0 ? 1ull : (unsigned long long)want;
            if (target > total) target = total;
        }
        const unsigned long long excl = incl - (h0 + h1);
        if (before + excl < target && target <= before + incl) {       // exactly one thread
            const bool first = before + excl + h0 >= target;
            sh_digit = 2 * tid + (first ? 0 : 1);
            sh_before = before + excl + (first ? 0ull : h0);
            sh_mass = before + excl + h0 + (first ? 0ull : h1);         // through the chosen bin
        }
        __syncthreads();
        prefix = (prefix << bits) | sh_digit;
        before = sh_before;
    }
    const uint32_t key_tau = prefix;
    const unsigned long long mass = sh_mass;      // of all entries with key <= key_tau, i.e. z >= tau

    // The draw: largest z_i - log(-log(u_i)) among the kept entries, smaller index on ties.  The LM head has left the best
    // perturbed score of every 32-column tile: where that entry is kept it is the tile's best kept one, too.  Of the other
    // tiles those whose largest z is not kept hold nothing kept; only the rest are gone through again, by eight lanes each,
    // 32 tiles requested at a time (a wavefront with at most 8 of them: those).  Head + draw, us, 151 936 logits (drawing again for
    // every kept entry | all other tiles gone through, eight at a time | this): one kept entry 163 | 203 | 166 at 1 row, 210 | 230 | 196
    // at 64; top_p 0.3 of flat logits 226 | 241 | 224 and 269 | 269 | 255; 0.95: 226 | 199 | 192 and 269 | 224 | 222.  What is left
    // of the first column's lead, few rows and few kept entries, is the sampling epilogue of the head (10 us at 14B).
    const uint32_t row = row_ids ? (uint32_t)row_ids[m] : (uint32_t)m;
    const uint32_t pos = (uint32_t)positions[m];
    float best = -INFINITY, best_z = 0.f;
    int32_t best_i = 0x7fffffff, count = 0;
    auto consider = [&](float y, int32_t i, float z) { if (y > best || (y == best && i < best_i)) { best = y; best_i = i; best_z = z; } };
    for (int t0 = tid - lane; t0 < n_tiles; t0 += HX_NUC_THREADS) {      // whole wavefronts
        const int t = t0 + lane;
        bool again = false;
        if (t < n_tiles) {
            const size_t o = (size_t)m * n_tiles + t;
            const float z = cand_z[o], y = cand_y[o], zm = tile_zmax[o];
            const int32_t i = cand_i[o];
            if (nucleus_key(z) <= key_tau) consider(y, i, z);
            else again = nucleus_key(zm) <= key_tau;
        }
        const unsigned long long todo = __ballot(again);
        const int n = __popcll(todo);
        if (n == 0) continue;
        // lanes 0..n-1 get the tiles to go through, in order; the other lanes what is left
        const int rank = __popcll(todo & ((1ull << lane) - 1ull));
        const int packed = __builtin_amdgcn_ds_permute(4 * (again ? rank : n + lane - rank), t);
        auto look_again = [&](int k0, auto rounds) {                         // tiles k0 .. k0 + 8 * rounds - 1 of them
            constexpr int U = decltype(rounds)::value;
            float v[U][4];
            int q[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int k = k0 + 8 * u + (lane >> 3);
                const int g = __shfl(packed, min(k, n - 1)) * 8 + (lane & 7);        // a group of four entries
                q[u] = k < n && g < n_groups ? g : -1;
                load_group(x, V, min(g, n_groups - 1), vec, v[u]);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (q[u] < 0) continue;
                bool keep[4], any = false;
#pragma unroll
                for (int i = 0; i < 4; ++i) { keep[i] = 4 * q[u] + i < V && nucleus_key(v[u][i] * inv_t) <= key_tau; any |= keep[i]; }
                if (any) {
                    uint32_t w[4];
                    hx_philox4x32_10((uint32_t)q[u], row, pos, 0x53414D50u, key0, key1, w);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        if (!keep[i]) continue;
                        const float z = v[u][i] * inv_t;
                        const float un = ((float)(w[i] >> 9) + 0.5f) * (1.0f / 8388608.0f);
                        consider(z - logf(-logf(un)), 4 * q[u] + i, z);
                    }
                }
            }
        };
        if (n <= 8) look_again(0, std::integral_constant<int, 1>{});
        else for (int k0 = 0; k0 < n; k0 += 8 * HX_NUC_TILES) look_again(k0, std::integral_constant<int, HX_NUC_TILES>{});
    }
    if (size_out) {                               // the number of kept entries, where it is asked for
        for (int q0 = tid; q0 < n_groups; q0 += HX_NUC_THREADS * HX_NUC_UNROLL) {
            float v[HX_NUC_UNROLL][4];
            load_groups(x, V, q0, n_groups, vec, v);
#pragma unroll
            for (int u = 0; u < HX_NUC_UNROLL; ++u)
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    count += 4 * (q0 + u * HX_NUC_THREADS) + i < V && nucleus_key(v[u][i] * inv_t) <= key_tau;
        }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float oy = __shfl_xor(best, off), oz = __shfl_xor(best_z, off);
        const int32_t oi = __shfl_xor(best_i, off);
        if (oy > best || (oy == best && oi < best_i)) { best = oy; best_i = oi; best_z = oz; }
        count += __shfl_xor(count, off);
    }
    if (lane == 0) { redf[wave] = best; redi[wave] = best_i; redz[wave] = best_z; redc[wave] = count; }
    __syncthreads();
    if (tid == 0) {
#pragma unroll 1
        for (int w = 1; w < HX_NUC_THREADS / 64; ++w) {
            if (redf[w] > best || (redf[w] == best && redi[w] < best_i)) { best = redf[w]; best_i = redi[w]; best_z = redz[w]; }
            count += redc[w];
        }
        tok_out[m] = best_i;
        lp_out[m] = (float)((double)best_z - ((double)zmax + log((double)mass * (1.0 / 1099511627776.0))));
        if (size_out) size_out[m] = count;
    }
}

int hx_launch_nucleus(const hx_engine *e, int batch, const float *logits, const hx_sample_params *sample,
                      int32_t *tokens_out, float *logprobs_out, hipStream_t st) {
    hipLaunchKernelGGL(nucleus_kernel, dim3(batch), dim3(HX_NUC_THREADS), 0, st, logits, e->cfg.vocab,
                       (const float *)(e->ws + e->map.amax_val), (const int32_t *)(e->ws + e->map.amax_idx),
                       (const float *)(e->ws + e->map.samp_z), (const float *)(e->ws + e->map.samp_m), e->wlm.n_tiles, sample->positions, sample->row_ids,
                       sample->inv_temperature, sample->top_p, sample->key0, sample->key1, tokens_out, logprobs_out,
                       sample->nucleus_sizes);
    HX_CHECK_LAUNCH("nucleus");
    return HX_OK;
}
