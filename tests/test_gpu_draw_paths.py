"""The draw where its kernels change: batches beyond 128 rows (the workgroup-tiled LM head leaves the candidates), a
vocabulary that ends inside a tile, and kept sets from one entry to nearly all of them (which tiles the nucleus draw
goes through again).  Reference: the oracle's samplers on the step's own logits."""
import numpy as np
import pytest
import torch

import oracle
import test_gpu_sampling
import test_gpu_top_p
from paper_2511_00796_amd import synth, workload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    from paper_2511_00796_amd import binding
    binding.load()
    return binding


# 1000 = 31 tiles and 8 columns, 33324 = 1041 and 12: more tiles than the 1024 threads that first look at them
@pytest.mark.parametrize("batch,max_batch", [(129, 129), (130, 200), (200, 200), (256, 256)])
@pytest.mark.parametrize("vocab", [1000, 33324])
def test_draws_beyond_128_rows(hx, vocab, batch, max_batch):
    s = synth.ModelShape("draw", 1, 256, 4, 2, 64, 688, vocab)
    dw = workload.build(synth.Workload("draw", s, max_batch, "uniform", 1, 40, 77))
    args = (dw.tokens[:batch].contiguous(), dw.positions[:batch].contiguous(), dw.seq_lens_d[:batch].contiguous(),
            dw.table_d[:batch].contiguous())
    pos = args[1].cpu().numpy()
    logits = torch.empty(batch, vocab, device="cuda")
    tok = torch.empty(batch, dtype=torch.int32, device="cuda")
    lp = torch.empty(batch, device="cuda")
    n = torch.empty(batch, dtype=torch.int32, device="cuda")
    dw.engine.decode_step(dw.kv, *args, logits, tok)
    greedy = logits.clone()
    assert torch.equal(tok.long(), greedy.argmax(1))
    ids = torch.from_numpy(np.random.default_rng(2).permutation(5000)[:batch].astype(np.int32)).cuda()
    for row_ids, rows in ((None, np.arange(batch)), (ids, ids.cpu().numpy())):
        logits.fill_(float("nan"))
        dw.engine.decode_step_sample(dw.kv, *args, 0.7, 9, logits, tok, lp, row_ids)
        assert torch.equal(logits, greedy)
        test_gpu_sampling.check_against_oracle(tok.cpu().numpy(), lp.cpu().numpy(), greedy.cpu().numpy(), 0.7, 9, rows, pos, "sample")
        logits.fill_(float("nan"))
        dw.engine.decode_step_top_p(dw.kv, *args, 0.3, 0.8, 9, logits, tok, lp, row_ids, n)
        assert torch.equal(logits, greedy)
        test_gpu_top_p.check_against_oracle(tok.cpu().numpy(), lp.cpu().numpy(), n.cpu().numpy(), greedy.cpu().numpy(), 0.3, 0.8, 9,
                                            rows, pos, "top-p")


# (temperature, top_p): one kept entry, a few, some in every tile, all but the least likely
@pytest.mark.parametrize("temperature,top_p", [(0.002, 0.9), (0.02, 0.5), (0.1, 0.3), (1.0, 0.05), (1.0, 0.5), (1.0, 0.9999)])
@pytest.mark.parametrize("vocab,batch", [(1000, 5), (33324, 64), (70000, 3)])
def test_kept_sets_of_every_size(hx, vocab, batch, temperature, top_p):
    s = synth.ModelShape("kept", 1, 256, 4, 2, 64, 688, vocab)
    eng = hx.Engine(s, batch, 64)
    g = torch.Generator(device="cuda").manual_seed(13)
    eng.weights_pack(hx.HX_T_WLM, 0, torch.empty(256, vocab, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g))
    x = torch.randn(batch, 256, generator=g, device="cuda")
    pos = torch.arange(100, 100 + batch, dtype=torch.int32, device="cuda")
    y, tok, lp, n = (t.cpu().numpy() for t in eng.stage_lm_head_top_p(x, pos, temperature, top_p, 31))
    print("kept %d..%d of %d" % (n.min(), n.max(), vocab))
    test_gpu_top_p.check_against_oracle(tok, lp, n, y, temperature, top_p, 31, np.arange(batch), pos.cpu().numpy(), "kept")


@pytest.mark.parametrize("vocab,batch", [(70000, 5), (70000, 37), (70000, 100), (33324, 200)])
def test_near_ties_are_decided_exactly(hx, vocab, batch):
    """All logits of a row equal and large, so the noise alone decides and one wavefront in twenty meets a second best within the
    margin of the fast scores: its tiles are scored again, exactly.  Ten tiles per workgroup (up to 32, 64, 128 rows) and the
    workgroup-tiled head."""
    s = synth.ModelShape("near", 1, 256, 4, 2, 64, 688, vocab)
    eng = hx.Engine(s, batch if batch <= 128 else 256, 64)
    g = torch.Generator(device="cuda").manual_seed(9)
    column = torch.empty(256, 1, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.02, generator=g)
    eng.weights_pack(hx.HX_T_WLM, 0, column.expand(256, vocab).contiguous())
    x = torch.randn(batch, 256, generator=g, device="cuda")
    pos = torch.arange(100, 100 + batch, dtype=torch.int32, device="cuda")
    for seed in (31, 32):
        y, tok, lp, n = (t.cpu().numpy() for t in eng.stage_lm_head_top_p(x, pos, 1e-3, 0.5, seed))
        assert (n == vocab).all()
        test_gpu_top_p.check_against_oracle(tok, lp, n, y, 1e-3, 0.5, seed, np.arange(batch), pos.cpu().numpy(), "near")


# 2, 63, 257 tiles of 256 threads; 1024 (the last of them), 1025; 5 per thread of 1024: 5120 (the last in one trip) and 5121
@pytest.mark.parametrize("tiles", [2, 63, 257, 1024, 1025, 5120, 5121])
def test_tokens_from_any_number_of_tiles(hx, tiles):
    vocab = 32 * tiles - 8
    s = synth.ModelShape("tiles", 1, 256, 4, 2, 64, 688, vocab)
    dw = workload.build(synth.Workload("tiles", s, 4, "uniform", 1, 40, 78))
    for seed in (3, 4):
        tok, lp, logits = test_gpu_sampling.sample_once(dw, 1.3, seed)
        test_gpu_sampling.check_against_oracle(tok, lp, logits, 1.3, seed, np.arange(4), dw.positions.cpu().numpy(), "tiles")
    greedy = torch.empty(4, dtype=torch.int32, device="cuda")
    dw.engine.decode_step(dw.kv, dw.tokens, dw.positions, dw.seq_lens_d, dw.table_d, dw.logits, greedy)
    assert torch.equal(greedy.long(), dw.logits.argmax(1))
