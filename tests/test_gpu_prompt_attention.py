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


@pytest.mark.parametrize("d,plan", [(128, [(700, 40), (1300, 1)]), (64, [(900, 70), (333, 2)])], ids=["128", "64"])
@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("steepness", [1.0, 4.0, 16.0])
def test_scores_that_rise_along_the_keys(hx, d, plan, cache, steepness, monkeypatch):
    """A column's scale is moved only when its maximum is 2^8 past it: keys that grow along the sequence make maxima rise by less
    than that, by about that and by more, over and over."""
    fill = synth.kv_fill

    def rising(*args, **kwargs):
        k, v = fill(*args, **kwargs)
        ramp = torch.linspace(0.05, 1.0, k.shape[0], device=k.device) * steepness
        return (k.float() * ramp.view(-1, *[1] * (k.dim() - 1))).to(k.dtype), v

    monkeypatch.setattr(synth, "kv_fill", rising)
    s = synth.ModelShape("prompt-attn", 2, 256, 8, 2, d, 704, 1024)
    rowwise, grouped = layer0_attention(hx, s, plan, hx.HX_KV_FP8_E4M3 if cache == "fp8" else hx.HX_KV_BF16, 0, monkeypatch)
    assert np.isfinite(grouped).all()
    scale = max(float(np.abs(rowwise).max()), 1.0)
    diff = float(np.abs(grouped - rowwise).max())
    print("%s %d x %g: max |grouped - row-wise| %.2e (max |o| %.2f)" % (cache, d, steepness, diff, scale))
    # as above, and scores of up to about 8 steepness (in powers of two) that are sums in another order: 2^-20 of that at most
    assert diff <= (2e-5 + 8 * steepness * 2.0 ** -20) * scale
