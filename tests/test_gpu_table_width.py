"""The width of the block table is the caller's allocation (the longest sequence it allows), not a property of the sequences: the
same call through a table as wide as its longest sequence and through one of 2 048 entries gives the same bits."""
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


def tables(final, seed):
    table, nb = synth.block_table(np.asarray(final, dtype=np.int32), 16, seed)
    wide = np.full((table.shape[0], 2048), -1, dtype=np.int32)       # entries past a sequence's blocks are never read
    wide[:, :table.shape[1]] = table
    return (table, wide), nb


@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("plan", [[(300, 1)], [(4000, 2)], [(700, 1), (30, 7)]])
def test_prompt_chunk(hx, plan, cache):
    s = synth.ModelShape("width", 2, 256, 16, 2, 128, 688, 1024)
    eng = build(hx, s, 3, 8, 8192, hx.HX_KV_FP8_E4M3 if cache == "fp8" else hx.HX_KV_BF16)
    ctx, new = np.array([c for c, _ in plan], dtype=np.int32), np.array([n for _, n in plan], dtype=np.int32)
    both, nb = tables(ctx + new, 5)
    start = np.concatenate([[0], np.cumsum(ctx)]).astype(np.int32)
    seq = np.repeat(np.arange(len(plan)), new)
    pos = np.concatenate([np.arange(c, c + n) for c, n in plan]).astype(np.int32)
    toks = np.random.default_rng(1).integers(0, s.vocab, len(pos)).astype(np.int32)
    out = []
    for table in both:
        kv = hx.KVCache(eng, nb)
        k, v = synth.kv_fill(s, 0, int(ctx.sum()), 3, device="cuda")
        kv.prefill_fill(0, k, v, dev(start), dev(table))
        cap = torch.zeros(2, len(pos), s.q_dim, device="cuda")
        eng.set_attn_capture(cap)
        eng.prefill_chunk(kv, dev(toks), dev(pos), dev(pos + 1), dev(table[seq]))
        eng.set_attn_capture(None)
        out.append(cap[0].clone())
    torch.cuda.synchronize()
    assert float(out[0].abs().max()) > 0 and torch.equal(out[0], out[1])


@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("d,lens", [(128, [500]), (128, [512, 17, 300]), (64, [100, 512]), (128, [8000, 30, 3000])])
def test_decode_attention(hx, d, lens, cache):
    s = synth.ModelShape("width", 1, 256, 6, 2, d, 688, 1000)
    eng = build(hx, s, 3, len(lens), 8192, hx.HX_KV_FP8_E4M3 if cache == "fp8" else hx.HX_KV_BF16)
    both, nb = tables(lens, 5)
    start = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    q = torch.randn(len(lens), s.q_dim, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda")
    out = []
    for table in both:
        kv = hx.KVCache(eng, nb)
        k, v = synth.kv_fill(s, 0, int(np.sum(lens)), 3, device="cuda")
        kv.prefill_fill(0, k, v, dev(start), dev(table))
        out.append(eng.stage_attention(kv, 0, q, dev(np.array(lens, dtype=np.int32)), dev(table)))
    torch.cuda.synchronize()
    assert torch.equal(out[0], out[1])
