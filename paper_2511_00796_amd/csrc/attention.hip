// Split-K flash-decoding attention over the paged cache: the per-step schedule that cuts the ragged
// batch into equal shares of K/V tiles, the attention kernel, and the combine kernel that merges the
// partial results.
//
// Work decomposition ("stream-K").  A tile is the K and V of 16 tokens of one KV head.  All tiles of the
// batch are lined up in (sequence, KV head, block) order and cut into W equal runs of S = ceil(Nt / W)
// tiles, one run per wavefront, W = 8 per compute unit.
// Every wavefront therefore streams the same
// number of bytes whatever the length mix, all of them are resident at once and finish together, and a
// run is long (about 1 MiB at the 7B shape), so start-up latency is paid once.  A run that crosses from
// one (sequence, KV head) pair into the next emits one partial result per pair it touches; run w and pair
// p write slot w + p, which is unique and makes the slots of a pair contiguous (w0 + p .. w1 + p).
//
// One wavefront serves all G query heads of its KV head at once, so every K and V byte is read exactly once:
//     S^T[token, g] = K_tile[token, :] . q[g, :]        v_mfma_f32_16x16x32_bf16 (A = K tile, B = packed q)
//     O^T[d, g]    += V_tile^T[d, token] . P^T[token, g] v_mfma_f32_16x16x16_bf16 (A = V tile, B = P)
// The accumulator layout of the first product (lane = query head g, 4 registers = 4 tokens) is
// exactly the B-operand layout of the second, so the probabilities never cross lanes; only the
// running maximum is exchanged between the four 16-lane groups, with two register swaps per
// tile, and the running sum is reduced once at the end.  K/V tiles are stored in operand order
// in the pool, so they go from HBM to registers with contiguous 1-KiB loads and need no LDS.
#include "hx_internal.h"
#include "step_setup.h"

#define HX_NEG_BIG (-1.0e30f)

// ---- per-step setup: schedule + RoPE angles (step_setup.h) ------------------------------------------------------
// block 0: the schedule; blocks 1..batch: the rows
__global__ __launch_bounds__(256) void step_setup_kernel(hx_setup_args a) {
    if (blockIdx.x == 0) {
        if (a.seq_lens != nullptr) hx_setup_schedule(a);
    } else if (a.positions != nullptr) {
        hx_setup_row(a, blockIdx.x - 1);
    }
}

hx_attn_bufs hx_attn_bufs_of(const hx_engine *e) {
    char *ws = e->ws;
    return hx_attn_bufs{(uint16_t *)(ws + e->map.qp), (int32_t *)(ws + e->map.pre), (int32_t *)(ws + e->map.lens),
                        (int32_t *)(ws + e->map.sched), (float *)(ws + e->map.part_ml), (float *)(ws + e->map.part_o),
                        (uint16_t *)(ws + e->map.ap)};
}

hx_setup_args hx_setup_args_of(const hx_engine *e, int batch, const int32_t *positions, const int32_t *seq_lens, const int32_t *table,
                               int max_blocks, const hx_attn_bufs &bufs) {
    return hx_setup_args{batch, e->cfg.n_kv_heads, e->attn_waves, positions, seq_lens, table, max_blocks, bufs.pre, bufs.lens, bufs.sched,
                         (int32_t *)(e->ws + e->map.blk_new), (float *)(e->ws + e->map.cs), e->D / 2, (double)e->cfg.rope_theta,
                         e->cfg.max_batch};
}

int hx_launch_step_setup(const hx_engine *e, int batch, const int32_t *positions, const int32_t *seq_lens,
                         const int32_t *table, int max_blocks, hipStream_t st, const hx_attn_bufs *bufs) {
    if (bufs && positions) return hx_fail(HX_E_RANGE, "the schedule-only set-up takes no positions");
    // without positions only block 0 runs: the per-row blocks would write the engine's RoPE tables
    hipLaunchKernelGGL(step_setup_kernel, dim3(positions ? batch + 1 : 1), dim3(256), 0, st,
                       hx_setup_args_of(e, batch, positions, seq_lens, table, max_blocks, bufs ? *bufs : hx_attn_bufs_of(e)));
    HX_CHECK_LAUNCH("step_setup");
    return HX_OK;
}

// ---- split-K attention -----------------------------------------------------------------------------------
typedef unsigned int u32x4_t __attribute__((ext_vector_type(4)));

// One K/V tile in registers: D/32 K operands then D/32 V operands, 16 bytes per lane each.
// K/V are read exactly once per step: non-temporal loads keep them from displacing reusable lines.
template <int D>
__device__ __forceinline__ void load_tile(u32x4_t (&r)[D / 16], const char *tile, int lane) {
    const u32x4_t *p = (const u32x4_t *)tile + lane;
#pragma unroll
    for (int i = 0; i < D / 16; ++i) r[i] = __builtin_nontemporal_load(p + i * 64);
}

// State of one (sequence, KV head) pair while its tiles stream through.
template <int D>
struct AttnState {
    f32x4_t o[D / 16];
    float m;   // running maximum of the scaled scores (base-2 domain), same in the 4 lane groups
    float l;   // this lane's share of the running sum
};

// Streams `nblk` (1..128) consecutive blocks of one pair: tokens [t0, t1), t0 a multiple of 16.  blk_lo / blk_hi
// hold the physical ids: lane i of blk_lo = block i, lane i of blk_hi = block 64 + i.
// PF = tiles in flight (register ring): 8 KiB per wavefront, 64 KiB per compute unit, which is what a compute unit keeps
// outstanding; more only queues up, and a run of few tiles asks for more past its end.  us per launch with 3 / 2 / 1 tiles of
// 8 KiB: 7B, 128 sequences 351 / 347 / 339, 1.5B, 256 of them 157.5 / 151.5 / 147.5, 64 53.4 / 51.1 / 49.3; 7B, 8 short ones 15.6 / - / 9.2.
// The loop has no prologue and no conditional load: it starts PF tiles early (iterations that only request) and every
// iteration requests the tile PF ahead into the slot it has just finished with; past the end of the run the request goes to the
// packed query (small, cache-resident, finite), so the load stream is unconditional and the compiler keeps exactly
// PF - 1 tiles outstanding behind every wait.
template <int D, int PF>
__device__ __forceinline__ void stream_tiles(AttnState<D> &st, const bf16x8_t (&qop)[D / 32], const char *pool_layer,
                                             size_t block_bytes, size_t head_off, const char *qtile, int32_t blk_lo,
                                             int32_t blk_hi, int nblk, int t0, int t1, float scale_log2e, int lane) {
    const int qd = lane >> 4;
    u32x4_t ring[PF][D / 16];
#pragma unroll
    for (int s = 0; s < PF; ++s)
#pragma unroll
        for (int i = 0; i < D / 16; ++i) ring[s][i] = u32x4_t{0u, 0u, 0u, 0u};

    const int n_rounds = (nblk + PF - 1) / PF + 1;
    for (int rd = 0; rd < n_rounds; ++rd) {
#pragma unroll
        for (int s = 0; s < PF; ++s) {
            const int i = (rd - 1) * PF + s;                   // tile of this iteration; < 0 while the ring fills
            const int tok0 = t0 + i * 16 + qd * 4;             // this lane's 4 tokens
            if (rd > 0) {
                // scores of 16 tokens x 16 query heads
                f32x4_t sc = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < D / 32; ++kk)
                    sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, ring[s][kk]), qop[kk], sc, 0, 0, 0);
                {
                    // The K operands of the slot die with these products, so the compiler may hand their registers to the
                    // next vector instruction (at head size 64 it did: the mask arithmetic of a ragged tile, a few
                    // instructions behind the product that was still to read them).  Keep them live past the products
                    // (hx_hold_operands) at both head sizes.
                    u32x4_t kheld[D / 32];
#pragma unroll
                    for (int kk = 0; kk < D / 32; ++kk) kheld[kk] = ring[s][kk];
                    hx_hold_operands(kheld, sc);
                }
                float s4[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) s4[r] = sc[r] * scale_log2e;
                // V of positions that do not exist must not reach the product as NaN/Inf
                u32x4_t vv[D / 32];
#pragma unroll
                for (int q = 0; q < D / 32; ++q) vv[q] = ring[s][D / 32 + q];
                if (t0 + (i + 1) * 16 > t1) {                      // wave-uniform: a tile with missing tokens
                    const int valid = t1 - tok0;
#pragma unroll
                    for (int r = 0; r < 4; ++r) s4[r] = r < valid ? s4[r] : -INFINITY;
                    const uint32_t m01 = valid >= 2 ? 0xffffffffu : (valid == 1 ? 0x0000ffffu : 0u);
                    const uint32_t m23 = valid >= 4 ? 0xffffffffu : (valid == 3 ? 0x0000ffffu : 0u);
#pragma unroll
                    for (int q = 0; q < D / 32; ++q) { vv[q].x &= m01; vv[q].y &= m23; vv[q].z &= m01; vv[q].w &= m23; }
                }
                float mx = fmaxf(fmaxf(s4[0], s4[1]), fmaxf(s4[2], s4[3]));
                mx = hx_max_of_16_lane_groups(mx);
                const float m_new = fmaxf(st.m, mx);
                const float alpha = __builtin_amdgcn_exp2f(st.m - m_new);
                float p[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) p[r] = __builtin_amdgcn_exp2f(s4[r] - m_new);
                st.l = st.l * alpha + ((p[0] + p[1]) + (p[2] + p[3]));
                st.m = m_new;
#pragma unroll
                for (int nn = 0; nn < D / 16; ++nn) st.o[nn] *= alpha;
                // P enters the matrix core as bf16; split it into a high and a low bf16 part so that the
                // product keeps ~16 significant bits of every probability
                uint2 ph, pl;
                ph.x = hx_cvt_pk_bf16(p[0], p[1]);
                ph.y = hx_cvt_pk_bf16(p[2], p[3]);
                pl.x = hx_cvt_pk_bf16(p[0] - __uint_as_float(ph.x << 16), p[1] - __uint_as_float(ph.x & 0xffff0000u));
                pl.y = hx_cvt_pk_bf16(p[2] - __uint_as_float(ph.y << 16), p[3] - __uint_as_float(ph.y & 0xffff0000u));
                const s16x4_t pop_hi = __builtin_bit_cast(s16x4_t, ph);
                const s16x4_t pop_lo = __builtin_bit_cast(s16x4_t, pl);
#pragma unroll
                for (int q = 0; q < D / 32; ++q) {
                    uint2 lo = make_uint2(vv[q].x, vv[q].y), hi = make_uint2(vv[q].z, vv[q].w);
                    st.o[2 * q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, lo), pop_hi, st.o[2 * q], 0, 0, 0);
                    st.o[2 * q + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, hi), pop_hi, st.o[2 * q + 1], 0, 0, 0);
                }
#pragma unroll
                for (int q = 0; q < D / 32; ++q) {
                    uint2 lo = make_uint2(vv[q].x, vv[q].y), hi = make_uint2(vv[q].z, vv[q].w);
                    st.o[2 * q] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, lo), pop_lo, st.o[2 * q], 0, 0, 0);
                    st.o[2 * q + 1] = __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s16x4_t, hi), pop_lo, st.o[2 * q + 1], 0, 0, 0);
                }
            }
            // the slot is free: request tile i + PF into it (or the query once the run is exhausted)
            const int nx = i + PF;
            const int32_t blk = (nx < 64) ? __builtin_amdgcn_readlane(blk_lo, nx & 63) : __builtin_amdgcn_readlane(blk_hi, nx & 63);
            const char *src = (nx < nblk) ? pool_layer + (size_t)blk * block_bytes + head_off : qtile;
            load_tile<D>(ring[s], src, lane);
        }
    }
}

template <int D, int PF>
__global__ __launch_bounds__(64) void attn_splitk_kernel(const int32_t *__restrict__ sched, const int32_t *__restrict__ pre,
                                         const int32_t *__restrict__ lens, const char *__restrict__ pool_layer, size_t block_bytes,
                                         const uint16_t *__restrict__ qp, const int32_t *__restrict__ table, int max_blocks,
                                         int n_kv, int G, float scale_log2e, float *__restrict__ part_ml,
                                         float *__restrict__ part_o) {
    const int w = blockIdx.x;
    const int lane = threadIdx.x;
    const int S = sched[0], Nt = sched[1];
    int f = w * S;
    const int f1 = min(Nt, f + S);
    if (f >= f1) return;
    const int g = lane & 15, qd = lane >> 4;

    // the whole schedule sits in registers: lane l holds pre[l + 64 i] and lens[l + 64 i]
    int32_t pr[HX_PREFIX_LEN / 64], ln[4];
#pragma unroll
    for (int i = 0; i < HX_PREFIX_LEN / 64; ++i) pr[i] = pre[lane + 64 * i];
#pragma unroll
    for (int i = 0; i < 4; ++i) ln[i] = lens[lane + 64 * i];
    auto pick = [&](const int32_t *regs, int n, int idx) -> int32_t {   // regs[idx / 64] of lane idx % 64
        int32_t v = 0;
#pragma unroll
        for (int i = 0; i < HX_PREFIX_LEN / 64; ++i)
            if (i < n && (idx >> 6) == i) v = __builtin_amdgcn_readlane(regs[i], idx & 63);
        return v;
    };

    while (f < f1) {                                     // one iteration per (sequence, KV head) pair touched
        // sequence of tile f: the last b with pre[b] * n_kv <= f
        int cnt = 0;
#pragma unroll
        for (int i = 0; i < HX_PREFIX_LEN / 64; ++i) cnt += __popcll(__ballot((long long)pr[i] * n_kv <= (long long)f));
        const int b = __builtin_amdgcn_readfirstlane(cnt) - 1;
        const int pb = pick(pr, HX_PREFIX_LEN / 64, b);
        const int T = pick(ln, 4, b);
        const int nblk_b = (T + 15) >> 4;
        const int local = f - pb * n_kv;
        const int kvh = local / nblk_b;
        const int blk0 = local - kvh * nblk_b;
        const int n = min(f1 - f, nblk_b - blk0);        // tiles of this pair in this run
        const size_t head_off = (size_t)kvh * 2 * (16 * D * 2);

        // packed query: B operand of the score product
        const char *qtile = (const char *)(qp + ((size_t)b * n_kv + kvh) * (D / 32) * 512);
        bf16x8_t qop[D / 32];
        {
            const uint4 *q4 = (const uint4 *)qtile + lane;
#pragma unroll
            for (int kk = 0; kk < D / 32; ++kk) qop[kk] = __builtin_bit_cast(bf16x8_t, q4[kk * 64]);
        }
        AttnState<D> st;
#pragma unroll
        for (int nn = 0; nn < D / 16; ++nn) st.o[nn] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        st.m = HX_NEG_BIG;
        st.l = 0.f;

        for (int done = 0; done < n; done += 128) {      // at most 128 block ids fit the two id registers
            const int nsub = min(128, n - done);
            const int32_t *row = table + (size_t)b * max_blocks + blk0 + done;
            int32_t blk_lo = (lane < nsub) ? row[lane] : 0;
            int32_t blk_hi = (64 + lane < nsub) ? row[64 + lane] : 0;
            const int t0 = (blk0 + done) * 16;
            // Everything requested so far must have landed before the tile loop is entered: its waits count
            // outstanding loads, and a load still in flight on entry would make every wait in the loop drain
            // the tile ring to match.
#pragma unroll
            for (int kk = 0; kk < D / 32; ++kk) asm volatile("" : "+v"(qop[kk]));
            asm volatile("" : "+v"(blk_lo), "+v"(blk_hi));
            stream_tiles<D, PF>(st, qop, pool_layer, block_bytes, head_off, qtile, blk_lo, blk_hi, nsub, t0,
                                min(T, t0 + nsub * 16), scale_log2e, lane);
        }

        // total of the running sum over the four lane groups
        float l = st.l;
        l += __shfl_xor(l, 16);
        l += __shfl_xor(l, 32);
        const size_t slot = (size_t)w + (size_t)b * n_kv + kvh;
        if (qd == 0) {
            part_ml[slot * 32 + g] = st.m;
            part_ml[slot * 32 + 16 + g] = l;
        }
        if (g < G) {
            float *po = part_o + (slot * G + g) * D;
#pragma unroll
            for (int nn = 0; nn < D / 16; ++nn) *(f32x4_t *)(po + nn * 16 + qd * 4) = st.o[nn];
        }
        f += n;
    }
}

// ---- combine ---------------------------------------------------------------------------------------------
// o = sum_c 2^(m_c - M) o_c / sum_c 2^(m_c - M) l_c over the partial results of the pair (sequence, KV head):
// the runs w0..w1 that cover its tiles, found from the schedule, in slots w + pair.
// WPP wavefronts per (sequence, query head).  Maximum and denominator: lane i takes partials i, i+64, ..., reduced by
// a fixed shuffle tree (every wavefront for itself).  Numerator: lane = (phase 0..3, d8 0..15); phase p of wavefront w
// takes partials 16 w + p + 4 u (u < 4), then those 16 WPP further, in order, then the phases are summed by a fixed shuffle tree and the
// wavefronts in order (deterministic).  Lanes of phase 0
// write the bf16-rounded result into the packed activation buffer of the output projection and, if asked,
// the unrounded fp32 values.  D = 64 uses lanes d8 < 8 only.
// WPP = 1, four pairs per workgroup: batches whose pairs have a few partials.  WPP = 8: batches whose pairs may have a hundred and
// more (its one wavefront went through them in a dozen dependent steps); a pair that has at most HX_COMBINE_FEW all the same is
// done by its first wavefront as with WPP = 1, bit for bit.
#define HX_COMBINE_FEW 32
template <int D, int WPP>
__global__ __launch_bounds__(WPP == 1 ? 256 : 64 * WPP) void attn_combine_kernel(const int32_t *__restrict__ sched,
                                                           const int32_t *__restrict__ pre,
                                                           const int32_t *__restrict__ lens, int n_q, int n_kv, int G,
                                                           const float *__restrict__ part_ml,
                                                           const float *__restrict__ part_o,
                                                           uint16_t *__restrict__ ap, int m_groups,
                                                           float *__restrict__ attn_f32) {
    __shared__ float part[WPP == 1 ? 1 : WPP][WPP == 1 ? 1 : D];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), pw = WPP == 1 ? 0 : wave;   // of the workgroup / of the pair
    const int b = blockIdx.y, h = WPP == 1 ? blockIdx.x * 4 + wave : blockIdx.x;
    if (h >= n_q) return;                                // whole wavefronts; for WPP > 1 the grid is exact
    const int lane = threadIdx.x & 63, d8 = lane & 15, ph = lane >> 4;
    const bool has_d = d8 < D / 8;
    const int T = lens[b], P = pre[b];
    const unsigned S = max(sched[0], 1);
    __builtin_amdgcn_sched_barrier(0);                   // three loads in one round trip, beside the division by G
    const int kvh = (unsigned)h / (unsigned)G, g = h - kvh * G;
    const int nblk_b = (T + 15) >> 4;
    const int start = P * n_kv + kvh * nblk_b;           // tiles of this pair: [start, start + nblk_b)
    const int pair = b * n_kv + kvh;
    // its slots, inclusive; a sequence without keys has no partials: it reads one slot, whatever that holds, and no other row does
    const int s0 = (unsigned)start / S + pair, s1 = (unsigned)(start + max(nblk_b, 1) - 1) / S + pair;
    const int n = s1 - s0 + 1;
    const int waves = WPP > 1 && n > HX_COMBINE_FEW ? WPP : 1;      // that share the pair: the same for the whole workgroup
    if (pw >= waves) return;
    float M = HX_NEG_BIG, den = 0.f;
    float acc[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] = 0.f;
    // U partials of this 16-lane group, four slots apart; past the end the last again, with weight 0
    constexpr int U = 4;
    float m[U], l[U];
    f32x4_t a[U], c[U];
    auto request = [&](int it, int u) {
        const int iu = min(it + 4 * u, s1);
        const float *ml = part_ml + (size_t)iu * 32 + g;
        m[u] = ml[0]; l[u] = ml[16];
        if (has_d) {
            const float *po = part_o + ((size_t)iu * G + g) * D + d8 * 8;
            a[u] = *(const f32x4_t *)po; c[u] = *(const f32x4_t *)(po + 4);
        }
    };
    auto add = [&](float w, int u) {
        if (has_d) {
            acc[0] += w * a[u][0]; acc[1] += w * a[u][1]; acc[2] += w * a[u][2]; acc[3] += w * a[u][3];
            acc[4] += w * c[u][0]; acc[5] += w * c[u][1]; acc[6] += w * c[u][2]; acc[7] += w * c[u][3];
        }
    };
    if (n <= 8) {       // the usual case (a few partials per pair): each 16-lane group takes every fourth
#pragma unroll
        for (int u = 0; u < 2; ++u) request(s0 + ph, u);
        M = fmaxf(m[0], m[1]);
        M = fmaxf(M, __shfl_xor(M, 16));
        M = fmaxf(M, __shfl_xor(M, 32));
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const float w = s0 + ph + 4 * u <= s1 ? __builtin_amdgcn_exp2f(m[u] - M) : 0.f;
            den += w * l[u];
            add(w, u);
        }
        den += __shfl_xor(den, 16);
        den += __shfl_xor(den, 32);
    } else {
        // More than 8 partials (a short batch of long sequences has a hundred): maximum and denominator take one
        // partial per lane, 64 at a time; the weighted sum four per 16-lane group and round, the first round's requested with them.
        const int first = s0 + 16 * pw + ph;
        const float *ml = part_ml + (size_t)(s0 + min(lane, n - 1)) * 32 + g;
        const float m0 = ml[0], l0 = lane < n ? ml[16] : 0.f;
#pragma unroll
        for (int u = 0; u < U; ++u) request(first, u);
        M = m0;
        for (int i = lane + 64; i < n; i += 64) M = fmaxf(M, part_ml[(size_t)(s0 + i) * 32 + g]);
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1) M = fmaxf(M, __shfl_xor(M, sh));
        den = __builtin_amdgcn_exp2f(m0 - M) * l0;
        for (int i = lane + 64; i < n; i += 64) {
            const float *mi = part_ml + (size_t)(s0 + i) * 32 + g;
            den += __builtin_amdgcn_exp2f(mi[0] - M) * mi[16];
        }
#pragma unroll
        for (int sh = 1; sh < 64; sh <<= 1) den += __shfl_xor(den, sh);
        for (int it = first; it <= s1; it += 16 * waves) {
            if (it != first) {
#pragma unroll
                for (int u = 0; u < U; ++u) request(it, u);
            }
#pragma unroll
            for (int u = 0; u < U; ++u) add(it + 4 * u <= s1 ? __builtin_amdgcn_exp2f(m[u] - M) : 0.f, u);
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        acc[j] += __shfl_xor(acc[j], 16);
        acc[j] += __shfl_xor(acc[j], 32);
    }
    if (WPP > 1 && waves > 1) {
        if (ph == 0 && has_d)
#pragma unroll
            for (int j = 0; j < 8; ++j) part[pw][d8 * 8 + j] = acc[j];
        __syncthreads();
        if (pw != 0) return;
#pragma unroll
        for (int w = 1; w < WPP; ++w)
            if (has_d)
#pragma unroll
                for (int j = 0; j < 8; ++j) acc[j] += part[w][d8 * 8 + j];
    }
    if (ph != 0 || !has_d) return;
    const float inv = 1.0f / den;
#pragma unroll
    for (int j = 0; j < 8; ++j) acc[j] *= inv;
    if (attn_f32) {
        float *dst = attn_f32 + ((size_t)b * n_q + h) * D + d8 * 8;
        *(f32x4_t *)dst = f32x4_t{acc[0], acc[1], acc[2], acc[3]};
        *(f32x4_t *)(dst + 4) = f32x4_t{acc[4], acc[5], acc[6], acc[7]};
    }
    if (ap == nullptr) return;
    uint4 pk;
    pk.x = hx_cvt_pk_bf16(acc[0], acc[1]); pk.y = hx_cvt_pk_bf16(acc[2], acc[3]);
    pk.z = hx_cvt_pk_bf16(acc[4], acc[5]); pk.w = hx_cvt_pk_bf16(acc[6], acc[7]);
    *(uint4 *)(ap + hx_xp_index(b, h * D + d8 * 8, m_groups)) = pk;
}

int hx_launch_attention(const hx_engine *e, const hx_kv *kv, int layer, int batch, const int32_t *seq_lens,
                        const int32_t *table, int max_blocks, hipStream_t st, const hx_attn_bufs *bufs) {
    const char *pool_layer = kv->pool + (size_t)layer * kv->layer_bytes;
    const hx_attn_bufs own = hx_attn_bufs_of(e);
    const hx_attn_bufs &a = bufs ? *bufs : own;
    const float scale_log2e = (float)(1.4426950408889634 / sqrt((double)e->D));
    (void)seq_lens; (void)batch;
    dim3 grid(e->attn_waves), block(64);
#define HX_ATTN_ARGS                                                                                             \
    (const int32_t *)a.sched, (const int32_t *)a.pre, (const int32_t *)a.lens, pool_layer, kv->block_bytes,      \
        (const uint16_t *)a.qp, table, max_blocks, e->cfg.n_kv_heads, e->G, scale_log2e, a.part_ml, a.part_o
    if (e->D == 128) hipLaunchKernelGGL((attn_splitk_kernel<128, 1>), grid, block, 0, st, HX_ATTN_ARGS);
    else             hipLaunchKernelGGL((attn_splitk_kernel<64, 2>), grid, block, 0, st, HX_ATTN_ARGS);
#undef HX_ATTN_ARGS
    HX_CHECK_LAUNCH("attn_splitk");
    return HX_OK;
}

int hx_launch_combine(const hx_engine *e, int batch, float *attn_f32_out, hipStream_t st, const hx_attn_bufs *bufs) {
    const hx_attn_bufs own = hx_attn_bufs_of(e);
    const hx_attn_bufs &a = bufs ? *bufs : own;
    const int n_kv = e->cfg.n_kv_heads, n_q = e->cfg.n_q_heads;
    const int m_groups = hx_m_groups(batch);
    // A pair has about attn_waves / (batch * n_kv) partials, if its sequence has as many blocks (which only the device knows): with
    // more than 32 its eight wavefronts pay (170 partials, 3 rows of 7B: 13.0 -> 8.0 us; 1 row of 1.5B, 200 blocks: 11.5 -> 7.6), and
    // for shorter sequences the seven that leave at once cost nothing (1 to 8 rows, 20 to 400 tokens: 17.3-18.3 us with the
    // attention kernel either way).
    const bool many = e->attn_waves > HX_COMBINE_FEW * batch * n_kv;
    dim3 cgrid(many ? n_q : (n_q + 3) / 4, batch), cblock(many ? 512 : 256);
#define HX_COMB_ARGS                                                                                             \
    (const int32_t *)a.sched, (const int32_t *)a.pre, (const int32_t *)a.lens, n_q, n_kv, e->G,                  \
        (const float *)a.part_ml, (const float *)a.part_o, a.ap, m_groups, attn_f32_out
#define HX_COMB_LAUNCH(DD)                                                                                         \
    do {                                                                                                         \
        if (many) hipLaunchKernelGGL((attn_combine_kernel<DD, 8>), cgrid, cblock, 0, st, HX_COMB_ARGS);          \
        else      hipLaunchKernelGGL((attn_combine_kernel<DD, 1>), cgrid, cblock, 0, st, HX_COMB_ARGS);          \
    } while (0)
    if (e->D == 128) HX_COMB_LAUNCH(128);
    else             HX_COMB_LAUNCH(64);
#undef HX_COMB_LAUNCH
#undef HX_COMB_ARGS
    HX_CHECK_LAUNCH("attn_combine");
    return HX_OK;
}
