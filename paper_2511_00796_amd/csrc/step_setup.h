// The per-step set-up of a decode step, shared by the launch that does it beside the embedding (elementwise.hip) and the one
// that does it alone (attention.hip, stage hooks).
#pragma once
#include "hx_internal.h"

struct hx_setup_args {
    int batch, n_kv, n_waves;
    const int32_t *positions, *seq_lens, *table;     // positions NULL: schedule only; seq_lens NULL: rows only; table may be NULL
    int max_blocks;
    int32_t *pre, *lens, *sched, *blk_new;
    float *cs;
    int half;
    double theta;
    int max_batch;
};

// The schedule, by one workgroup of at least 256 threads: sched[0] = S (tiles per wavefront), sched[1] = Nt (tiles in all),
// pre[b] = blocks of the sequences before b (pre[b] = total for b >= batch, HX_PREFIX_LEN entries), lens[b] = seq_lens[b]
// (0 for b >= batch).
__device__ __forceinline__ void hx_setup_schedule(const hx_setup_args &a) {
    __shared__ int32_t scan[256];
    const int b = threadIdx.x;
    const bool on = b < 256;
    const int T = b < a.batch ? a.seq_lens[b] : 0;
    const int cnt = (T + 15) >> 4;
    if (on) scan[b] = cnt;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {       // inclusive Hillis-Steele scan
        const int v = (on && b >= off) ? scan[b - off] : 0;
        __syncthreads();
        if (on) scan[b] += v;
        __syncthreads();
    }
    if (!on) return;
    const int total = scan[255];
    a.pre[b] = scan[b] - cnt;                        // b >= batch: cnt = 0, so pre[b] = total
    a.lens[b] = T;
    for (int i = 256 + b; i < HX_PREFIX_LEN; i += 256) a.pre[i] = total;
    if (b == 0) {
        const long long nt = (long long)total * a.n_kv;
        a.sched[0] = (int)((nt + a.n_waves - 1) / a.n_waves);
        a.sched[1] = (int)nt;
    }
}

// Row b: cos/sin of pos * theta^(-2i/D), evaluated in double, stored fp32; and the physical block that holds the new
// position (one look-up per step instead of one per layer in the append kernel).
__device__ __forceinline__ void hx_setup_row(const hx_setup_args &a, int b) {
    if (threadIdx.x == 0 && a.table != nullptr) a.blk_new[b] = a.table[(size_t)b * a.max_blocks + (a.positions[b] >> 4)];
    const double pos = (double)a.positions[b];
    for (int i = threadIdx.x; i < a.half; i += blockDim.x) {
        const double ang = pos * pow(a.theta, -(double)i / (double)a.half);
        a.cs[(size_t)b * a.half + i] = (float)cos(ang);
        a.cs[(size_t)a.max_batch * a.half + (size_t)b * a.half + i] = (float)sin(ang);
    }
}

hx_setup_args hx_setup_args_of(const hx_engine *e, int batch, const int32_t *positions, const int32_t *seq_lens, const int32_t *table,
                               int max_blocks, const hx_attn_bufs &bufs);
