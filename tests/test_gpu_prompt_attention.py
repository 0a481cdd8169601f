"""The attention of prompt calls where its schedule can go wrong: one or two rows over a long cache, groups that end at a
workspace of 256 rows, and pairs cut into few or many parts (HX_ATTN_WAVES sets the number of workgroups the work is cut for).  Reference: the same call with HX_CHUNK_ATTENTION=0, which sends every
row through the decode step's attention (held to the oracle by its own tests); same products, other order of sums."""
import numpy as np
import pytest
import torch

from paper_2511_00796_amd import synth
from test_gpu_prefill import build, dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    from paper_2511_00796_amd import binding
    binding.load()
    return binding


def layer0_attention(hx, s, plan, kv_dtype, waves, monkeypatch, seed=31):
    ctx = np.array([c for c, _ in plan], dtype=np.int32)
    n_new = np.array([n for _, n in plan], dtype=np.int32)
    final = ctx + n_new
    n = int(n_new.sum())
    table, nb = synth.block_table(final, s.block_size, seed)
    toks = np.random.default_rng(seed).integers(0, s.vocab, size=n).astype(np.int32)
    bs = np.concatenate([np.full(m, b) for b, m in enumerate(n_new)])
    ps = np.concatenate([np.arange(c, c + m) for c, m in plan]).astype(np.int32)
    start = np.concatenate([[0], np.cumsum(ctx)]).astype(np.int32)
    out = []
    for flag in ("0", "1"):
        monkeypatch.setenv("HX_CHUNK_ATTENTION", flag)
        if waves and flag == "1":
            monkeypatch.setenv("HX_ATTN_WAVES", str(waves))
        eng = build(hx, s, seed, 256, int(final.max()) + 1, kv_dtype)
        monkeypatch.delenv("HX_ATTN_WAVES", raising=False)
        kv = hx.KVCache(eng, nb)
        kv.pool.fill_(0xFF)                            # NaN in both cache types: nothing outside a sequence may be used
        if int(ctx.sum()):
            k, v = synth.kv_fill(s, 0, int(ctx.sum()), seed, device="cuda")
            kv.prefill_fill(0, k, v, dev(start), dev(table))
        cap = torch.zeros(s.n_layers, n, s.q_dim, dtype=torch.float32, device="cuda")
        eng.set_attn_capture(cap)
        args = (dev(toks), dev(ps), dev(ps + 1), dev(table[bs]))
        if n > 256:
            ws = torch.empty(hx.prefill_workspace_bytes(eng.cfg, n), dtype=torch.uint8, device="cuda")
            ws.fill_(0xFF)
            eng.prefill_rows(kv, *args, ws)
        else:
            eng.prefill_chunk(kv, *args)
        eng.set_attn_capture(None)
        torch.cuda.synchronize()
        out.append(cap[0].cpu().numpy())
    return out


# (heads, KV heads, head size, plan of (keys cached, rows)).  128 / G rows are one group, 32 columns a wavefront; 32 tokens are a step, 8 steps the
# shortest part.  In groups of at most 32 columns the wavefronts may take steps of their own.
CASES = {
    "16-columns-1000-blocks": (16, 2, 128, [(15990, 2)]),
    "16-columns-999-blocks": (16, 2, 128, [(15982, 2)]),
    "24-columns-1001-blocks": (16, 2, 128, [(16005, 3)]),
    "one-row-64-1000-blocks": (4, 1, 64, [(15999, 1)]),
    "group-of-18": (7, 1, 128, [(255, 18)]),
    "group-of-19": (7, 1, 128, [(255, 19), (256, 1), (257, 18)]),
    "one-step": (8, 2, 64, [(0, 32)]),
    "one-token-beyond": (8, 2, 64, [(0, 33)]),
    "cut-at-the-last-token": (4, 2, 128, [(3040, 33), (15, 31)]),
    "narrow-3-to-9-steps": (8, 1, 128, [(70, 1), (97, 1), (128, 2), (160, 1), (290, 4), (290, 5), (0, 2)]),
    "narrow-32-and-33-columns": (11, 1, 64, [(300, 3), (301, 2), (95, 2), (64, 3)]),
    "narrow-long-and-cut": (16, 2, 128, [(9000, 1), (777, 2), (8191, 2), (40, 1)]),
    "all-single": (4, 4, 64, [(40 * i + i % 17, 1) for i in range(40)]),
    "across-workspaces": (6, 2, 128, [(0, 250), (1500, 13), (3, 500), (33, 5)]),
    "across-workspaces-64": (16, 1, 64, [(900, 255), (0, 2), (64, 511)]),
}


@pytest.mark.parametrize("waves", [0, 64])
@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("name", sorted(CASES))
def test_prompt_attention_equals_row_at_a_time(hx, name, cache, waves, monkeypatch):
    n_q, n_kv, d, plan = CASES[name]
    s = synth.ModelShape("prompt-attn", 2, 256, n_q, n_kv, d, 704, 1024)
    kv_dtype = hx.HX_KV_FP8_E4M3 if cache == "fp8" else hx.HX_KV_BF16
    rowwise, grouped = layer0_attention(hx, s, plan, kv_dtype, waves, monkeypatch)
    assert np.isfinite(grouped).all()
    scale = max(float(np.abs(rowwise).max()), 1.0)
    diff = float(np.abs(grouped - rowwise).max())
    print("%s %s waves %d: max |grouped - row-wise| %.2e (max |o| %.2f)" % (name, cache, waves, diff, scale))
    # P enters both kernels as a high + low bf16 pair: 2^-17 of each probability, plus fp32 sums in another order
    assert diff <= 2e-5 * scale


def scale_moves(s, plan, cache, steepness, parts, seed=31):
    """Host copy of layer 0's scores over the cached keys, 32 at a time, in that many parts per pair: -> (moves of a column's scale, its maximum,
    after the first step of a part; those by 2^8 and more; per column; largest sum of magnitudes behind a score, in powers of two)."""
    w, glob = synth.layer_weights(s, 0, seed), synth.global_weights(s, seed)
    n = sum(m for _, m in plan)
    toks = np.random.default_rng(seed).integers(0, s.vocab, size=n)
    x = glob["embed"].float()[torch.from_numpy(toks)]
    x = x * torch.rsqrt((x * x).mean(-1, keepdim=True) + s.rms_eps) * w["g1"].float()
    D, half = s.head_dim, s.head_dim // 2
    q = (x @ w["wqkv"].float() + w["bqkv"].float())[:, :s.q_dim].view(n, s.n_q_heads, D)
    pos = torch.cat([torch.arange(c, c + m) for c, m in plan]).float()
    ang = pos[:, None, None] * s.rope_theta ** (-torch.arange(half) / half)
    q = torch.cat([q[..., :half] * ang.cos() - q[..., half:] * ang.sin(), q[..., half:] * ang.cos() + q[..., :half] * ang.sin()], -1)
    total = sum(c for c, _ in plan)
    k = rising_keys(synth.kv_fill(s, 0, total, seed, device="cuda")[0], steepness).cpu().float()
    k = k.clamp(-448, 448).to(torch.float8_e4m3fn).float() if cache == "fp8" else k
    moves, leaps, largest, r0, t0 = [], [], 0.0, 0, 0
    for c, m in plan:
        kb = k[t0:t0 + c].repeat_interleave(s.group, 1)                              # the KV head of every query head
        qb = q[r0:r0 + m] * (1.4426950408889634 / D ** 0.5)
        sc = torch.einsum("rhd,thd->rht", qb, kb)
        largest = max(largest, float(torch.einsum("rhd,thd->rht", qb.abs(), kb.abs()).max()))
        mx = sc[..., :c // 32 * 32].view(m, s.n_q_heads, -1, 32).amax(-1)
        mv, lp = torch.zeros(m, s.n_q_heads), torch.zeros(m, s.n_q_heads)
        for i in range(mx.shape[-1]):
            if i % -(-mx.shape[-1] // parts) == 0:
                top = mx[..., i]
            mv += mx[..., i] > top
            lp += mx[..., i] > top + 8
            top = torch.maximum(top, mx[..., i])
        moves.append(mv.flatten())
        leaps.append(lp.flatten())
        r0, t0 = r0 + m, t0 + c
    return torch.cat(moves), torch.cat(leaps), largest


def rising_keys(k, steepness):
    ramp = torch.linspace(0.02, 1.0, k.shape[0], device=k.device) * steepness
    return (k.float() * ramp.view(-1, *[1] * (k.dim() - 1))).to(k.dtype)


@pytest.mark.parametrize("d,plan", [(128, [(4000, 40), (3000, 1)]), (64, [(4000, 70), (2500, 2)])], ids=["128", "64"])
@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("waves,parts", [(64, 2), (2048, 16)])       # pairs in at most two parts; in parts of the shortest length, 8 steps
@pytest.mark.parametrize("steepness", [16.0, 50.0, 200.0])
def test_scores_that_rise_along_the_keys(hx, d, plan, cache, waves, parts, steepness, monkeypatch):
    """Keys that grow along the sequence move a column's scale in step after step of a part, by little and by 2^8 and more (counted on the
    host), and with it what the column has summed so far."""
    s = synth.ModelShape("prompt-attn", 2, 256, 8, 2, d, 704, 1024)
    moves, leaps, largest = scale_moves(s, plan, cache, steepness, parts)
    print("moves per column %d..%d (median %d), by 2^8 and more: median %d" % (moves.min(), moves.max(), moves.median(), leaps.median()))
    assert moves.median() >= 10 and moves.max() >= 20 and (leaps.median() >= 2 or steepness < 200)
    fill = synth.kv_fill

    def rising(*args, **kwargs):
        k, v = fill(*args, **kwargs)
        return rising_keys(k, steepness), v

    monkeypatch.setattr(synth, "kv_fill", rising)
    rowwise, grouped = layer0_attention(hx, s, plan, hx.HX_KV_FP8_E4M3 if cache == "fp8" else hx.HX_KV_BF16, waves, monkeypatch)
    assert np.isfinite(grouped).all()
    scale = max(float(np.abs(rowwise).max()), 1.0)
    diff = float(np.abs(grouped - rowwise).max())
    print("%s %d x %g: max |grouped - row-wise| %.2e (max |o| %.2f, scores' magnitudes up to %.0f)" % (cache, d, steepness, diff, scale, largest))
    # as above, and scores (in powers of two) that are fp32 sums in two orders: 2^-23 of the largest sum of magnitudes
    assert diff <= (2e-5 + largest * 2.0 ** -23) * scale


@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("rows", [2, 40])                # one wavefront's columns, or steps of their own; several wavefronts
def test_the_largest_probability_is_exact(hx, rows, d, cache):
    """Probabilities are relative to the largest of their column so far, which is 1 and needs no second bf16: a column that two keys share,
    the larger one four steps behind the smaller (the same wavefront's, where each takes every fourth step) and 2^0.5 to 2^7.5 times its weight, errs by fp32 roundings alone, where a high + low pair of the
    larger one's probability would err by up to 2^-18.  The smaller key's values are 0, so nothing else hides that."""
    s = synth.ModelShape("prompt-attn", 2, 256, 8, 1, d, 704, 1024)
    kv_dtype = hx.HX_KV_FP8_E4M3 if cache == "fp8" else hx.HX_KV_BF16
    eng = build(hx, s, 3, 256, 256, kv_dtype)
    slow = d // 2 - 1                                    # the rotation's slowest pair: queries of all rows are nearly the same
    q = torch.zeros(8, d)
    q[:, slow] = torch.linspace(0.5, 7.5, 8) * d ** 0.5 / (1.4426950408889634 * 2)      # (score of 2) - (score of 0) = 0.5 .. 7.5
    k_new = torch.zeros(d)
    k_new[slow] = -200.0
    for l in range(2):
        w = synth.layer_weights(s, l, 3)
        w["wqkv"] = torch.zeros_like(w["wqkv"])
        w["bqkv"] = torch.cat([q.flatten(), k_new, torch.zeros(d)]).to(w["bqkv"].dtype)
        eng.pack_layer(l, w)
    ctx, T = 200, 200 + rows
    table = torch.arange((T + 15) // 16, dtype=torch.int32, device="cuda").view(1, -1)
    kv = hx.KVCache(eng, table.numel())
    kv.pool.fill_(0xFF)
    k, v = torch.zeros(ctx, 1, d), torch.randn(ctx, 1, d, generator=torch.Generator().manual_seed(3))
    k[:, 0, slow] = -200.0
    k[5, 0, slow], k[140, 0, slow], v[5] = 0.0, 2.0, 0.0
    start = lambda n: torch.tensor([0, n], dtype=torch.int32, device="cuda")
    for l in range(2):
        kv.prefill_fill(l, k.bfloat16().cuda(), v.bfloat16().cuda(), start(ctx), table)
    pos = torch.arange(ctx, T, dtype=torch.int32, device="cuda")
    rows_table = table.expand(rows, -1).contiguous()
    cap = torch.zeros(2, rows, s.q_dim, dtype=torch.float32, device="cuda")
    eng.set_attn_capture(cap)
    eng.prefill_chunk(kv, torch.zeros_like(pos), pos, pos + 1, rows_table)
    eng.set_attn_capture(None)
    qr = eng.stage_rope_append(kv, 0, torch.zeros(rows, s.qkv_dim, device="cuda"), pos, rows_table).view(rows, 8, d).double()
    K, V = (t[:, 0].double() for t in kv.gather(0, T, start(T), table))
    sc = (qr @ K.t().contiguous() / d ** 0.5).masked_fill(torch.arange(T, device="cuda")[None, None] > pos[:, None, None], -np.inf)
    ref = torch.softmax(sc, -1) @ V
    err = ((cap[0].double().view_as(ref) - ref).abs() / ref.abs().clamp_min(1e-3)).max().item()
    print("%s %d x %d: largest relative error 2^%.1f" % (cache, d, rows, np.log2(max(err, 1e-12))))
    # the smaller weight: exp2 and a score of up to 8 (in powers of two), the sum, the reciprocal and the product: 2^-20 in all
    assert err <= 2.0 ** -20
