"""Rows without keys (length 0).  They are outside the contract of a step (a row attends at least its own token) and what comes out
for them means nothing, but every access they cause stays inside the buffers and the other rows are what they are without them."""
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


@pytest.mark.parametrize("waves", [64, 500, 2048])       # runs of 13 to 37 tiles; of 2 to 5; every tile, or two, a run of its own
@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("heads", [(8, 2, 128), (4, 1, 64)], ids=["8-2-128", "4-1-64"])
@pytest.mark.parametrize("lens", [[0, 0, 3700, 0, 2500, 16], [33, 0, 9000, 9700, 0, 0]], ids=["first", "last"])
def test_the_other_rows_of_a_decode_batch(hx, lens, heads, cache, waves, monkeypatch):
    """The first pairs of a batch empty, some between, and the last ones: the runs of tiles are the same as without them, and so is
    every bit of the others' attention."""
    n_q, n_kv, d = heads
    s = synth.ModelShape("empty", 1, 256, n_q, n_kv, d, 704, 1024)
    monkeypatch.setenv("HX_ATTN_WAVES", str(waves))
    eng = build(hx, s, 3, len(lens), 16384, hx.HX_KV_FP8_E4M3 if cache == "fp8" else hx.HX_KV_BF16)
    lens = np.array(lens, dtype=np.int32)
    table, nb = synth.block_table(np.maximum(lens, 1), s.block_size, 3)
    kv = hx.KVCache(eng, nb)
    k, v = synth.kv_fill(s, 0, int(lens.sum()), 3, device="cuda")
    kv.prefill_fill(0, k, v, dev(np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)), dev(table))
    q = torch.randn(len(lens), s.q_dim, device="cuda", generator=torch.Generator(device="cuda").manual_seed(3))
    on = np.nonzero(lens)[0]
    alone = eng.stage_attention(kv, 0, q[dev(on)].contiguous(), dev(lens[on]), dev(table[on]))
    out = eng.stage_attention(kv, 0, q, dev(lens), dev(table))
    assert torch.isfinite(alone).all() and torch.equal(out[dev(on)], alone)


def test_a_batch_of_nothing_but_empty_rows_ends(hx):
    s = synth.ModelShape("empty", 1, 256, 8, 2, 128, 704, 1024)
    eng = build(hx, s, 3, 4, 64)
    kv = hx.KVCache(eng, 4)
    lens = torch.zeros(4, dtype=torch.int32, device="cuda")
    eng.stage_attention(kv, 0, torch.randn(4, s.q_dim, device="cuda"), lens, torch.arange(4, dtype=torch.int32, device="cuda").view(4, 1).contiguous())
    torch.cuda.synchronize()


@pytest.mark.parametrize("waves", [64, 2048])            # 16 workgroups, fewer than items, so that the groups are ordered; 512
@pytest.mark.parametrize("heads", [(8, 2, 128), (8, 4, 64)], ids=["8-2-128", "8-4-64"])
def test_the_other_rows_of_a_prompt_call(hx, heads, waves, monkeypatch):
    """Rows without keys as groups of their own (first, last, several in a row) and in front of the first row of a sequence, which
    then counts as its continuation."""
    n_q, n_kv, d = heads
    s = synth.ModelShape("empty", 2, 256, n_q, n_kv, d, 704, 1024)
    monkeypatch.setenv("HX_ATTN_WAVES", str(waves))
    plan = [(0, 0), (700, 40), (0, 0), (0, 0), (90, 3), (0, 0), (0, 33), (5, 1), (1200, 20), (0, 0)]     # (cached, rows); no rows: an empty one
    ctx = np.array([c for c, _ in plan], dtype=np.int32)
    rows = [(b, c + i, c + i + 1) for b, (c, n) in enumerate(plan) for i in range(n)] + [(b, 0, 0) for b, (_, n) in enumerate(plan) if n == 0]
    rows.sort(key=lambda r: (r[0], r[1]))
    table, nb = synth.block_table(np.array([c + max(n, 1) for c, n in plan]), s.block_size, 5)
    toks = np.random.default_rng(5).integers(0, s.vocab, size=len(rows)).astype(np.int32)
    k, v = synth.kv_fill(s, 0, int(ctx.sum()), 5, device="cuda")
    eng = build(hx, s, 5, 256, 2048)
    start = np.concatenate([[0], np.cumsum(ctx)]).astype(np.int32)

    def attention(keep):
        kv = hx.KVCache(eng, nb)
        kv.pool.fill_(0xFF)
        for l in range(s.n_layers):
            kv.prefill_fill(l, k, v, dev(start), dev(table))
        cap = torch.zeros(s.n_layers, len(keep), s.q_dim, dtype=torch.float32, device="cuda")
        eng.set_attn_capture(cap)
        seq, pos, lens = (np.array([rows[i][j] for i in keep], dtype=np.int32) for j in range(3))
        eng.prefill_chunk(kv, dev(toks[keep]), dev(pos), dev(lens), dev(table[seq]))
        eng.set_attn_capture(None)
        torch.cuda.synchronize()
        return cap[0].cpu().numpy()

    on = [i for i, r in enumerate(rows) if r[2] > 0]
    alone, among = attention(on), attention(list(range(len(rows))))[on]
    assert np.isfinite(alone).all() and np.isfinite(among).all()
    # other parts at most: P enters as a high + low bf16 pair, 2^-17 of each probability, plus fp32 sums in another order
    assert float(np.abs(among - alone).max()) <= 2e-5 * max(float(np.abs(alone).max()), 1.0)
