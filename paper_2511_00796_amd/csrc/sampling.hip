// Nucleus (top-p) sampling of one step's logits (Holtzman et al., ICLR 2020), after temperature scaling:
// keep the most probable entries whose mass reaches top_p -- all entries with z_i >= tau, tau the largest
// threshold for which mass{z_i >= tau} >= top_p * total, so entries equal to the last kept one are kept --
// and draw from the kept set by Gumbel-max with the noise of the temperature sampler.
//
// Mass is 40-bit fixed point, w_i = floor(exp(z_i - max z) * 2^40), added with integer LDS atomics: the sums are exact, so the
// kept set does not depend on the order of the additions and the result is deterministic.  tau is found in two steps.  The
// entries' mass is summed in 2048 bins of max z - z, as wide as the row's spread asks for (nucleus_scale), and the bins are walked
// from the largest z down to the one where the running mass reaches the target.  The entries of that bin, a thousand of 152 064 or
// fewer, are then collected in LDS and selected among by their order-preserving 32-bit keys, up to 11 bits of their range at a
// time; a bin of more than HX_NUC_LIST entries (many equal logits, or a cut far below the bulk) is read from the row again for each
// digit instead.
// A short row, or one of many, is one workgroup's (nucleus_parts).  Of others the bins are filled and the bin's keys
// listed by as many workgroups per row as give the chip two on every compute unit: exponentials and atomics of the whole row,
// three times over, by one workgroup were four fifths of the time.  64 rows of 152 064 logits: 94 -> 17 + 17 + 24 us, bound by
// the LDS atomics, the chains of small steps, and the launches.
// The draw takes the tile winners that the LM head's sampling epilogue has left, on the whole
// chip (here, one workgroup per row, drawing again for every kept entry was 90 of 144 us at 64 rows of 152 064 logits).
#include "hx_internal.h"
#include <algorithm>

#define HX_NUC_THREADS 1024
#define HX_NUC_BINS 2048
#define HX_NUC_UNROLL 8
#define HX_NUC_LIST 8192
#define HX_NUC_PART 16384
#define HX_NUC_MAX_PARTS 16
#define HX_NUC_PART_LIST 1024
#define HX_NUC_PRELOAD 5         // rounds of 1024 tiles: all of 152 064 entries
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

// An entry's mass, and its bin: rounding is monotone, so a larger z is never in a later bin.  expf, within 0.86 units in the last
// place (0.30 root mean square) of the exact value; the LM head's hx_exp_nonpositive, 1.26 (0.41), would move entries at the cut.
__device__ __forceinline__ unsigned long long nucleus_mass(float z, float zmax) { return (unsigned long long)(expf(z - zmax) * HX_NUC_SCALE); }
struct NucleusScale { float zmax, per_z; };       // largest z of the row; bins per unit of z below it
__device__ __forceinline__ uint32_t nucleus_bin(float z, const NucleusScale &s) {
    return (uint32_t)fminf((s.zmax - z) * s.per_z, (float)(HX_NUC_BINS - 1));
}

// The row's scale, from the LM head's per-tile maxima.  The bins reach 32 below the largest z, where the mass has long been 0, or
// six times as far as the smallest of the tiles' maxima: of normally distributed logits that is 22 standard deviations, so that a
// bin holds the same few entries whatever their spread (with bins of 1/64 always, the cut bin of a flat row overflowed the lists:
// 128 and 256 rows of 151 936, standard deviation 0.2, took 330 and 401 us with the head, 175 and 238 now).  Entries further
// down are the last bin's.
__device__ __forceinline__ NucleusScale nucleus_scale(const float *__restrict__ tile_zmax, int n_tiles, float (*redf)[HX_NUC_THREADS / 64]) {
    const int tid = threadIdx.x;
    float mx = -INFINITY, mn = INFINITY;
    for (int t = tid; t < n_tiles; t += HX_NUC_THREADS) { mx = fmaxf(mx, tile_zmax[t]); mn = fminf(mn, tile_zmax[t]); }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) { mx = fmaxf(mx, __shfl_xor(mx, off)); mn = fminf(mn, __shfl_xor(mn, off)); }
    if ((tid & 63) == 0) { redf[0][tid >> 6] = mx; redf[1][tid >> 6] = mn; }
    __syncthreads();
    mx = redf[0][0]; mn = redf[1][0];
#pragma unroll
    for (int w = 1; w < HX_NUC_THREADS / 64; ++w) { mx = fmaxf(mx, redf[0][w]); mn = fminf(mn, redf[1][w]); }
    __syncthreads();
    return NucleusScale{mx, HX_NUC_BINS / fmaxf(fminf(6.0f * (mx - mn), 32.0f), 1e-30f)};
}

// f(z) for the entries of groups [q0, q1) of the row.  One copy of f per entry of a group, the groups moved up behind it: with
// all of them unrolled the kernels spent most of their time fetching their own code.
template <typename F>
__device__ __forceinline__ void each_entry(const float *__restrict__ x, int V, int q0, int q1, bool vec, float inv_t, F f) {
    for (int q = q0 + threadIdx.x; q < q1; q += HX_NUC_THREADS * HX_NUC_UNROLL) {
        float v[HX_NUC_UNROLL][4];
        load_groups(x, V, q, q1, vec, v);
#pragma unroll 1
        for (int g = q, u = 0; u < HX_NUC_UNROLL && g < q1; ++u, g += HX_NUC_THREADS) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                if (4 * g + i < V) f(v[0][i] * inv_t);
#pragma unroll
            for (int k = 0; k + 1 < HX_NUC_UNROLL; ++k)
#pragma unroll
                for (int i = 0; i < 4; ++i) v[k][i] = v[k + 1][i];
        }
    }
}

// the bins of one part of a row (hist is cleared here; the caller synchronises)
__device__ __forceinline__ void fill_bins(unsigned long long *hist, const float *__restrict__ x, int V, int q0, int q1, bool vec, float inv_t,
                                          const NucleusScale &scale) {
    for (int i = threadIdx.x; i < HX_NUC_BINS; i += HX_NUC_THREADS) hist[i] = 0ull;
    __syncthreads();
    each_entry(x, V, q0, q1, vec, inv_t, [&](float z) {
        const unsigned long long w = nucleus_mass(z, scale.zmax);
        if (w) atomicAdd(&hist[nucleus_bin(z, scale)], w);
    });
}

// What the walk over the bins leaves: the chosen bin, the mass above it and through it, and the mass to reach.
struct NucleusState { unsigned long long before, through, target; uint32_t digit; };

// What the two kernels before nucleus_kernel leave of a row, beside the lists
struct NucleusRow { NucleusState st; NucleusScale scale; uint32_t count[HX_NUC_MAX_PARTS]; };

// grid (rows, parts), so that the parts of a row mostly share an XCD's L2: bins of each part, to be added by nucleus_collect_kernel; the scale of each row
__global__ __launch_bounds__(HX_NUC_THREADS) void nucleus_bins_kernel(const float *__restrict__ logits, const float *__restrict__ tile_zmax,
                                                                      int V, int n_tiles, float inv_t, int part_groups,
                                                                      unsigned long long *__restrict__ bins, NucleusRow *__restrict__ heads) {
    __shared__ unsigned long long hist[HX_NUC_BINS];
    __shared__ float redf[2][HX_NUC_THREADS / 64];
    const int m = blockIdx.x, part = blockIdx.y;
    const NucleusScale scale = nucleus_scale(tile_zmax + (size_t)m * n_tiles, n_tiles, redf);
    const int q0 = part * part_groups, q1 = min((V + 3) >> 2, q0 + part_groups);
    fill_bins(hist, logits + (size_t)m * V, V, q0, q1, (V & 3) == 0, inv_t, scale);
    __syncthreads();
    unsigned long long *out = bins + ((size_t)m * gridDim.y + part) * HX_NUC_BINS;
    for (int i = threadIdx.x; i < HX_NUC_BINS; i += HX_NUC_THREADS) out[i] = hist[i];
    if (part == 0 && threadIdx.x == 0) heads[m].scale = scale;
}

// The bin, two per thread, in which the running mass from st.before on reaches st.target; `first`: the total of all bins fixes the
// target.  `sh` is the workgroup's copy (zeroed before the first walk), through which every thread learns the outcome.
__device__ __forceinline__ NucleusState walk_bins(const unsigned long long *hist, unsigned long long *wave_sum, NucleusState *sh,
                                                  NucleusState st, bool first, float top_p) {
    constexpr int NW = HX_NUC_THREADS / 64;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned long long h0 = hist[2 * tid], h1 = hist[2 * tid + 1];
    unsigned long long incl = h0 + h1;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long o = __shfl_up(incl, off);
        if (lane >= off) incl += o;
    }
    if (lane == 63) wave_sum[wave] = incl;
    __syncthreads();
    unsigned long long base = 0, total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (w < wave) base += wave_sum[w];
        total += wave_sum[w];
    }
    incl += base;
    if (first) {                                  // at least one unit and at most everything
        const double want = ceil((double)top_p * (double)total);
        st.target = want < 1.0 ? 1ull : (unsigned long long)want;
        if (st.target > total) st.target = total;
    }
    const unsigned long long excl = incl - (h0 + h1);
    if (st.before + excl < st.target && st.target <= st.before + incl) {       // exactly one thread
        const bool low = st.before + excl + h0 >= st.target;
        *sh = NucleusState{st.before + excl + (low ? 0ull : h0), st.before + excl + h0 + (low ? 0ull : h1), st.target,
                           (uint32_t)(2 * tid + (low ? 0 : 1))};
    }
    __syncthreads();
    return *sh;
}

// grid (rows, parts): every part adds the bins of all parts and walks them, then lists the keys of its own entries in the chosen
// bin (their number, and as many as fit)
__global__ __launch_bounds__(HX_NUC_THREADS) void nucleus_collect_kernel(const float *__restrict__ logits,
                                                                         const unsigned long long *__restrict__ bins,
                                                                         NucleusRow *__restrict__ heads, uint32_t *__restrict__ lists, int V,
                                                                         float inv_t, float top_p, int part_groups) {
    __shared__ unsigned long long hist[HX_NUC_BINS];
    __shared__ unsigned long long wave_sum[HX_NUC_THREADS / 64];
    __shared__ NucleusState sh;
    __shared__ uint32_t n;
    const int m = blockIdx.x, part = blockIdx.y, parts = gridDim.y, tid = threadIdx.x;
    const unsigned long long *in = bins + (size_t)m * parts * HX_NUC_BINS;
#pragma unroll
    for (int k = 0; k < HX_NUC_BINS / HX_NUC_THREADS; ++k) {
        unsigned long long h = 0;
#pragma unroll
        for (int p = 0; p < HX_NUC_MAX_PARTS; ++p)
            if (p < parts) h += in[(size_t)p * HX_NUC_BINS + k * HX_NUC_THREADS + tid];
        hist[k * HX_NUC_THREADS + tid] = h;
    }
    if (tid == 0) { sh = NucleusState{0ull, 0ull, 0ull, 0u}; n = 0; }
    const NucleusScale scale = heads[m].scale;
    __syncthreads();
    const NucleusState st = walk_bins(hist, wave_sum, &sh, NucleusState{0ull, 0ull, 0ull, 0u}, true, top_p);
    uint32_t *list = lists + ((size_t)m * parts + part) * HX_NUC_PART_LIST;
    const int q0 = part * part_groups, q1 = min((V + 3) >> 2, q0 + part_groups);
    each_entry(logits + (size_t)m * V, V, q0, q1, (V & 3) == 0, inv_t, [&](float z) {
        if (nucleus_bin(z, scale) == st.digit && nucleus_mass(z, scale.zmax)) {
            const uint32_t at = atomicAdd(&n, 1u);
            if (at < HX_NUC_PART_LIST) list[at] = nucleus_key(z);
        }
    });
    __syncthreads();
    if (tid == 0) {
        heads[m].count[part] = n;
        if (part == 0) heads[m].st = st;
    }
}

// One workgroup per row: selection among the entries of the chosen bin, and the draw.  PARTS: bins and lists come from the kernels
// above; else from here.
template <bool PARTS>
__global__ __launch_bounds__(HX_NUC_THREADS) void nucleus_kernel(
    const float *__restrict__ logits, const float *__restrict__ tile_zmax, int V, int n_tiles, float inv_t, float top_p,
    const NucleusRow *__restrict__ heads, const uint32_t *__restrict__ lists, int parts, const float *__restrict__ cand_y,
    const int32_t *__restrict__ cand_i, const float *__restrict__ cand_z, const int32_t *__restrict__ positions,
    const int32_t *__restrict__ row_ids, uint32_t key0, uint32_t key1, int32_t *__restrict__ tok_out, float *__restrict__ lp_out,
    int32_t *__restrict__ size_out) {
    constexpr int NW = HX_NUC_THREADS / 64, PRE = HX_NUC_PRELOAD;
    __shared__ unsigned long long hist[HX_NUC_BINS];
    __shared__ unsigned long long wave_sum[NW];
    __shared__ uint32_t list[HX_NUC_LIST];
    __shared__ float redf[2][NW];
    __shared__ int32_t redi[NW], redc[NW];
    __shared__ float redz[NW];
    __shared__ NucleusState sh;
    __shared__ uint32_t sh_lo, sh_hi, sh_n;

    const int m = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const float *x = logits + (size_t)m * V;
    const bool vec = (V & 3) == 0;                // rows then start on 16-byte boundaries
    const int n_groups = (V + 3) >> 2;
    // the first tiles' candidates for the draw, requested now
    float pz[PRE], py[PRE], pm[PRE];
    int32_t pi[PRE];
#pragma unroll
    for (int u = 0; u < PRE; ++u) {
        const size_t o = (size_t)m * n_tiles + min(tid + u * HX_NUC_THREADS, n_tiles - 1);
        pz[u] = cand_z[o]; py[u] = cand_y[o]; pm[u] = tile_zmax[o]; pi[u] = cand_i[o];
    }
    if (tid == 0) { sh = NucleusState{0ull, 0ull, 0ull, 0u}; sh_lo = 0xffffffffu; sh_hi = 0; sh_n = 0; }
    NucleusScale scale;
    NucleusState st{0ull, 0ull, 0ull, 0u};
    uint32_t bin, n_in_bin;
    bool listed = true;                           // `list` holds all keys of the bin
    if (PARTS) {
        scale = heads[m].scale;
        st = heads[m].st;
        bin = st.digit;
        n_in_bin = 0;
        uint32_t n[HX_NUC_MAX_PARTS], key[HX_NUC_MAX_PARTS];       // all counts, then all lists, one entry per thread, at once
        static_assert(HX_NUC_PART_LIST <= HX_NUC_THREADS, "a thread takes one entry of each list");
#pragma unroll
        for (int p = 0; p < HX_NUC_MAX_PARTS; ++p) n[p] = p < parts ? heads[m].count[p] : 0u;
#pragma unroll
        for (int p = 0; p < HX_NUC_MAX_PARTS; ++p)
            if ((uint32_t)tid < min(n[p], (uint32_t)HX_NUC_PART_LIST)) key[p] = lists[((size_t)m * parts + p) * HX_NUC_PART_LIST + tid];
#pragma unroll
        for (int p = 0; p < HX_NUC_MAX_PARTS; ++p) {
            listed = listed && n[p] <= HX_NUC_PART_LIST && n_in_bin + n[p] <= HX_NUC_LIST;
            if (listed && (uint32_t)tid < n[p]) list[n_in_bin + tid] = key[p];
            n_in_bin += n[p];
        }
        __syncthreads();                          // `sh` was cleared by one thread above
        if (tid == 0) sh = st;
    } else {
        scale = nucleus_scale(tile_zmax + (size_t)m * n_tiles, n_tiles, redf);
        fill_bins(hist, x, V, 0, n_groups, vec, inv_t, scale);
        __syncthreads();
        st = walk_bins(hist, wave_sum, &sh, st, true, top_p);
        bin = st.digit;
        each_entry(x, V, 0, n_groups, vec, inv_t, [&](float z) {
            if (nucleus_bin(z, scale) == bin && nucleus_mass(z, scale.zmax)) {
                const uint32_t at = atomicAdd(&sh_n, 1u);
                if (at < HX_NUC_LIST) list[at] = nucleus_key(z);
            }
        });
        __syncthreads();
        n_in_bin = sh_n;
        listed = n_in_bin <= HX_NUC_LIST;
    }
    __syncthreads();
    const auto key_value = [](uint32_t key) { const uint32_t b = ~key; return __uint_as_float(b ^ ((b >> 31) ? 0x80000000u : 0xffffffffu)); };
    auto each_key = [&](auto f) {                 // f(key, z) of the entries of the bin
        if (listed) {
            for (uint32_t i = tid; i < n_in_bin; i += HX_NUC_THREADS) f(list[i], key_value(list[i]));
        } else {
            each_entry(x, V, 0, n_groups, vec, inv_t, [&](float z) {
                if (nucleus_bin(z, scale) == bin && nucleus_mass(z, scale.zmax)) f(nucleus_key(z), z);
            });
        }
    };
    {                                             // the range of the keys
        uint32_t lo = 0xffffffffu, hi = 0;
        each_key([&](uint32_t key, float) { lo = min(lo, key); hi = max(hi, key); });
        if (lo <= hi) { atomicMin(&sh_lo, lo); atomicMax(&sh_hi, hi); }
    }
    __syncthreads();
    const uint32_t key_lo = sh_lo;
    uint32_t prefix = 0;                          // digits chosen so far, of key - key_lo
    int shift = sh_hi > key_lo ? 32 - __clz(sh_hi - key_lo) : 0;       // its bits still open (none: all keys are one)
    while (shift > 0) {
        const int bits = min(shift, 11), hi_shift = shift;
        shift -= bits;
        for (int i = tid; i < HX_NUC_BINS; i += HX_NUC_THREADS) hist[i] = 0ull;
        __syncthreads();
        each_key([&](uint32_t key, float z) {
            const uint32_t d = key - key_lo;
            if (hi_shift == 32 || (d >> hi_shift) == prefix) atomicAdd(&hist[(d >> shift) & ((1u << bits) - 1u)], nucleus_mass(z, scale.zmax));
        });
        __syncthreads();
        st = walk_bins(hist, wave_sum, &sh, st, false, top_p);
        prefix = (prefix << bits) | st.digit;
    }
    const uint32_t key_tau = key_lo + prefix;
    const unsigned long long mass = st.through;   // of all entries with key <= key_tau, i.e. z >= tau

    // The draw: largest z_i - log(-log(u_i)) among the kept entries, smaller index on ties.  The LM head has left the best
    // perturbed score of every 32-column tile: where that entry is kept it is the tile's best kept one, too.  Of the other
    // tiles those whose largest z is not kept hold nothing kept; only the rest are gone through again, listed first, so that all
    // threads share them.  Against drawing again for every kept entry this loses with few rows and few kept entries (one kept
    // entry, 1 row, 151 936 logits: 163 against 166 us with the head) and wins elsewhere (64 rows, top_p 0.95: 269 against 222).
    const uint32_t row = row_ids ? (uint32_t)row_ids[m] : (uint32_t)m;
    const uint32_t pos = (uint32_t)positions[m];
    float best = -INFINITY, best_z = 0.f;
    int32_t best_i = 0x7fffffff, count = 0, ahead = PRE;     // ahead: rounds whose candidates are in registers, the next one's first
    auto consider = [&](float y, int32_t i, float z) { if (y > best || (y == best && i < best_i)) { best = y; best_i = i; best_z = z; } };
    auto look_again = [&](const float (&v)[4], int q) {
        bool any = false;
#pragma unroll
        for (int i = 0; i < 4; ++i) any |= 4 * q + i < V && nucleus_key(v[i] * inv_t) <= key_tau;
        if (!any) return;
        uint32_t w[4];
        hx_philox4x32_10((uint32_t)q, row, pos, 0x53414D50u, key0, key1, w);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float z = v[i] * inv_t;
            if (4 * q + i >= V || nucleus_key(z) > key_tau) continue;
            const float un = ((float)(w[i] >> 9) + 0.5f) * (1.0f / 8388608.0f);
            consider(z - logf(-logf(un)), 4 * q + i, z);
        }
    };
    for (int c0 = 0; c0 < n_tiles; c0 += HX_NUC_LIST) {                  // once, but for rows of more than 262 144 entries
        __syncthreads();                          // `list` and its counter are free
        if (tid == 0) sh_n = 0;
        __syncthreads();
        const int c1 = min(n_tiles, c0 + HX_NUC_LIST);
#pragma unroll 1
        for (int t = c0 + tid; t < c1; t += HX_NUC_THREADS) {
            if (ahead-- <= 0) {
                const size_t o = (size_t)m * n_tiles + t;
                pz[0] = cand_z[o]; py[0] = cand_y[o]; pm[0] = tile_zmax[o]; pi[0] = cand_i[o];
            }
            if (nucleus_key(pz[0]) <= key_tau) consider(py[0], pi[0], pz[0]);
            else if (nucleus_key(pm[0]) <= key_tau) list[atomicAdd(&sh_n, 1u)] = t;
#pragma unroll
            for (int u = 0; u + 1 < PRE; ++u) { pz[u] = pz[u + 1]; py[u] = py[u + 1]; pm[u] = pm[u + 1]; pi[u] = pi[u + 1]; }
        }
        __syncthreads();
        const int items = 8 * sh_n;               // groups of four entries, two per thread and round
#pragma unroll 1
        for (int i = tid; i < items; i += 2 * HX_NUC_THREADS) {
            const int j = min(i + HX_NUC_THREADS, items - 1);
            int q[2] = {(int)list[i >> 3] * 8 + (i & 7), (int)list[j >> 3] * 8 + (j & 7)};
            float v[2][4];
#pragma unroll
            for (int u = 0; u < 2; ++u) load_group(x, V, min(q[u], n_groups - 1), vec, v[u]);
#pragma unroll 1
            for (int u = 0; u < 2; ++u) {
                if (q[0] < n_groups && (u == 0 || i + HX_NUC_THREADS < items)) look_again(v[0], q[0]);
                q[0] = q[1];
#pragma unroll
                for (int k = 0; k < 4; ++k) v[0][k] = v[1][k];
            }
        }
    }
    if (size_out) {                               // the number of kept entries, where it is asked for
        each_entry(x, V, 0, n_groups, vec, inv_t, [&](float z) { count += nucleus_key(z) <= key_tau; });
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) {
        const float oy = __shfl_xor(best, off), oz = __shfl_xor(best_z, off);
        const int32_t oi = __shfl_xor(best_i, off);
        if (oy > best || (oy == best && oi < best_i)) { best = oy; best_i = oi; best_z = oz; }
        count += __shfl_xor(count, off);
    }
    if (lane == 0) { redf[0][wave] = best; redi[wave] = best_i; redz[wave] = best_z; redc[wave] = count; }
    __syncthreads();
    if (tid == 0) {
#pragma unroll 1
        for (int w = 1; w < HX_NUC_THREADS / 64; ++w) {
            if (redf[0][w] > best || (redf[0][w] == best && redi[w] < best_i)) { best = redf[0][w]; best_i = redi[w]; best_z = redz[w]; }
            count += redc[w];
        }
        tok_out[m] = best_i;
        lp_out[m] = (float)((double)best_z - ((double)scale.zmax + log((double)mass * (1.0 / 1099511627776.0))));
        if (size_out) size_out[m] = count;
    }
}

// Workgroups per row that fill the bins and list the keys: two on every compute unit, parts of HX_NUC_PART entries or more.  One
// workgroup does it all in one launch where the row is short or the rows alone fill the chip: beyond a row per two compute units, or
// 768 entries for each row.  us with the head, one workgroup -> several: 151 936 entries 1 row 114 -> 81, 64 rows 138 -> 114, 128 rows
// 158 -> 150, 170 rows 194 -> 191, 256 rows 208 -> 216; 65 536 entries 64 rows 75.3 -> 70.1, 96 rows 81.2 -> 80.9, 128 rows 85.2 -> 88.5;
// 49 152 entries 1 row 54.5 -> 50.6, 64 rows 62.8 -> 61.5, 96 rows 69.1 -> 71.9; 32 768 entries 1 row 42.6 -> 45.8, 128 rows 59.1 -> 64.3.
static int nucleus_parts(int vocab, int batch) {
    const int cus = hx_device_cus();
    if (vocab < 3 * HX_NUC_PART || batch > cus / 2 || vocab / batch < 768) return 1;
    return std::max(1, std::min({HX_NUC_MAX_PARTS, 2 * cus / batch, vocab / HX_NUC_PART}));
}

// heads of `max_batch` rows, then lists and bins of at most `most` parts
static size_t nucleus_most_parts(int vocab, int max_batch) {
    size_t most = 0;
    for (int b = 1; b <= max_batch; ++b) {
        const int parts = nucleus_parts(vocab, b);
        if (parts > 1) most = std::max(most, (size_t)parts * b);
    }
    return most;
}
size_t hx_nucleus_bytes(int vocab, int max_batch) {
    const size_t most = nucleus_most_parts(vocab, max_batch);
    return most ? (size_t)max_batch * sizeof(NucleusRow) + most * (HX_NUC_BINS * sizeof(unsigned long long) + HX_NUC_PART_LIST * sizeof(uint32_t)) : 0;
}

int hx_launch_nucleus(const hx_engine *e, int batch, const float *logits, const hx_sample_params *sample,
                      int32_t *tokens_out, float *logprobs_out, hipStream_t st) {
    const int V = e->cfg.vocab, parts = nucleus_parts(V, batch), n_tiles = e->wlm.n_tiles;
    const float *tile_zmax = (const float *)(e->ws + e->map.samp_m);
    char *ws = e->ws + e->map.nucleus;
    NucleusRow *heads = (NucleusRow *)ws;
    unsigned long long *bins = (unsigned long long *)(ws + (size_t)e->cfg.max_batch * sizeof(NucleusRow));
    uint32_t *lists = (uint32_t *)(bins + (size_t)batch * parts * HX_NUC_BINS);
    if (parts > 1) {
        const int part_groups = ((V + 3) / 4 + parts - 1) / parts;
        hipLaunchKernelGGL(nucleus_bins_kernel, dim3(batch, parts), dim3(HX_NUC_THREADS), 0, st, logits, tile_zmax, V, n_tiles,
                           sample->inv_temperature, part_groups, bins, heads);
        HX_CHECK_LAUNCH("nucleus_bins");
        hipLaunchKernelGGL(nucleus_collect_kernel, dim3(batch, parts), dim3(HX_NUC_THREADS), 0, st, logits, (const unsigned long long *)bins,
                           heads, lists, V, sample->inv_temperature, sample->top_p, part_groups);
        HX_CHECK_LAUNCH("nucleus_collect");
    }
    hipLaunchKernelGGL(parts > 1 ? nucleus_kernel<true> : nucleus_kernel<false>, dim3(batch), dim3(HX_NUC_THREADS), 0, st, logits, tile_zmax, V,
                       n_tiles, sample->inv_temperature, sample->top_p, (const NucleusRow *)heads, (const uint32_t *)lists, parts,
                       (const float *)(e->ws + e->map.amax_val), (const int32_t *)(e->ws + e->map.amax_idx),
                       (const float *)(e->ws + e->map.samp_z), sample->positions, sample->row_ids, sample->key0, sample->key1, tokens_out,
                       logprobs_out, sample->nucleus_sizes);
    HX_CHECK_LAUNCH("nucleus");
    return HX_OK;
}
