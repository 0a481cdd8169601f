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


@pytest.mark.parametrize("waves", [1, 7, 2048])          # one run over everything; runs of a few tiles; every tile a run of its own
@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("heads", [(8, 2, 128), (4, 1, 64)], ids=["8-2-128", "4-1-64"])
@pytest.mark.parametrize("lens", [[0, 0, 37, 0, 250, 16], [33, 0, 900, 0, 0]], ids=["first", "last"])
def test_the_other_rows_of_a_decode_batch(hx, lens, heads, cache, waves, monkeypatch):
    """The first pairs of a batch empty, some between, and the last ones: the runs of tiles are the same as without them, and so is
    every bit of the others' attention."""
    n_q, n_kv, d = heads
    s = synth.ModelShape("empty", 1, 256, n_q, n_kv, d, 704, 1024)
    monkeypatch.setenv("HX_ATTN_WAVES", str(waves))
    eng = build(hx, s, 3, len(lens), 1024, hx.HX_KV_FP8_E4M3 if cache == "fp8" else hx.HX_KV_BF16)
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
