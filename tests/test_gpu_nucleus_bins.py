"""Nucleus selection by bins: rows at the edges of one and several workgroups per row, with so many equal logits that no list
takes the cut bin's entries, that one list of several overflows, that each takes its own but all are too many together, or that the
cut falls on a bin of one entry.  Logits are planted
through the LM head (one input column is 1, so column j's logit is the weight of row 0); the oracle is the sort of the definition."""
import numpy as np
import pytest
import torch

import oracle
from paper_2511_00796_amd import synth
from test_gpu_prefill import build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    from paper_2511_00796_amd import binding
    binding.load()
    return binding


def planted(law, V):
    r = np.random.default_rng(V)
    if law == "normal":
        return r.normal(0, 2, V)
    if law == "equal":                       # one bin holds the whole row
        return np.zeros(V)
    if law == "two_levels":                  # 5 000 equal entries in front, more than a part's list
        z = np.full(V, -3.0)
        z[: min(5000, V // 2)] = 1.0
        return z
    if law == "spread":                      # as many all over the row, which every part's list takes
        z = np.full(V, -3.0)
        z[:: max(2, V // 5000)] = 1.0
        return z
    if law == "two_in_a_bin":                # two in every other tile of 32 columns, neighbouring bf16 values that share a bin: in the
        z = np.full(V, -20.0)                # longest row 9 376, which every part's list takes its own of, but all together are too many
        z[::64] = 1.0
        z[7::64] = 1.0078125
        return z
    z = r.normal(0, 1, V)                     # peaked: one entry carries nearly everything
    z[V // 3] = 30.0
    return z


@pytest.mark.parametrize("law", ["normal", "equal", "two_levels", "spread", "two_in_a_bin", "peaked"])
@pytest.mark.parametrize("vocab", [8, 1000, 32764, 32768, 65540, 300000])
def test_kept_sets_of_planted_rows(hx, vocab, law):
    s = synth.ModelShape("nb", 1, 32, 1, 1, 64, 16, vocab)
    rows = 3
    eng = hx.Engine(s, rows, 64)
    z = torch.from_numpy(planted(law, vocab)).to(torch.bfloat16)
    wlm = torch.zeros(s.hidden, vocab, dtype=torch.bfloat16)
    wlm[0] = z
    eng.pack_globals({"embed": torch.zeros(vocab, s.hidden, dtype=torch.bfloat16).cuda(),
                      "gf": torch.ones(s.hidden, dtype=torch.bfloat16).cuda(), "wlm": wlm.cuda()})
    x = torch.zeros(rows, s.hidden, device="cuda")
    x[:, 0] = torch.tensor([1.0, 0.5, 2.0])
    pos = torch.tensor([3, 4, 5], dtype=torch.int32, device="cuda")
    compared = 0
    for share in (0.05, 0.5, 0.97):
        top_p = (int(share * vocab) + 0.5) / vocab          # between two multiples of 1 / vocab: never on a cut of equal entries
        y, tok, lp, n = [t.cpu().numpy() for t in eng.stage_lm_head_top_p(x, pos, 1.0, top_p, 99)]
        assert np.array_equal(y, x[:, :1].cpu().numpy() * z.float().numpy()[None])
        otok, olp, on, margin, gap = oracle.sample_top_p(y, 1.0, top_p, 99, np.arange(rows), pos.cpu().numpy())
        firm = margin > 1e-6                  # further from the cut than a sum of 3e5 fp32 exponentials is exact
        assert np.array_equal(n[firm], on[firm]), (top_p, n, on, margin)
        same = firm & (gap > 1e-4)            # fp32 perturbed scores on both sides
        assert np.array_equal(tok[same], otok[same])
        assert np.abs(lp[same] - olp[same]).max(initial=0.0) <= 2e-4
        compared += int(same.sum())
    assert compared >= 3


def test_masses_are_the_exponentials_of_the_definition(hx):
    """Rows of two entries that count, z = 0 and z = t: the second is kept unless the first alone reaches top_p of the sum, so the
    kept set turns over at one value of t.  128 neighbouring values around it, for many top_p: the sizes are those of the masses
    floor(exp(t) 2^40) of the device's fp32 exponential, not of one that is a unit in the last place away."""
    s = synth.ModelShape("nm", 1, 32, 1, 1, 64, 16, 4)
    rows = 128
    eng = hx.Engine(s, rows, 64)
    wlm = torch.zeros(s.hidden, s.vocab, dtype=torch.bfloat16)
    wlm[0:3, 1] = 1.0                         # logit 1 = x0 + x1 + x2: any fp32 number, as three bf16 pieces
    wlm[3, 2:] = 1.0
    eng.pack_globals({"embed": torch.zeros(s.vocab, s.hidden, dtype=torch.bfloat16).cuda(),
                      "gf": torch.ones(s.hidden, dtype=torch.bfloat16).cuda(), "wlm": wlm.cuda()})
    pos = torch.zeros(rows, dtype=torch.int32, device="cuda")
    turned = 0
    for top_p in np.linspace(0.51, 0.999, 64).astype(np.float32):
        mid = np.float32(np.log(1.0 / float(top_p) - 1.0))
        t = (np.full(rows, mid).view(np.int32) + np.arange(rows, dtype=np.int32) - rows // 2).view(np.float32)
        x = torch.zeros(rows, s.hidden, device="cuda")
        left = torch.from_numpy(t).cuda()
        for i in range(3):
            x[:, i] = left.bfloat16().float()
            left = left - x[:, i]
        assert not left.any()
        x[:, 3] = -100.0                      # no mass
        y, _, _, n = eng.stage_lm_head_top_p(x, pos, 1.0, float(top_p), 7)
        assert np.array_equal(y[:, 1].cpu().numpy(), t) and not y[:, 0].any()
        w = (torch.exp(y[:, :2]) * 2.0 ** 40).to(torch.int64).cpu().numpy()
        target = np.ceil(float(top_p) * w.sum(1).astype(np.float64))
        want = np.where(w[:, 0] >= target, 1, 2)
        assert np.array_equal(n.cpu().numpy(), want), (float(top_p), np.nonzero(n.cpu().numpy() != want)[0])
        turned += len(set(want.tolist())) == 2
    assert turned >= 48


def top_p_engine(hx, rows, vocab, std, seed=3):
    """An engine whose LM head gives normally distributed logits of standard deviation `std`, and its input."""
    s = synth.ModelShape("nt", 1, 64, 1, 1, 64, 16, vocab)
    eng = hx.Engine(s, rows, 64)
    g = torch.Generator(device="cuda").manual_seed(seed)
    w = [torch.randn(sh, generator=g, device="cuda").mul_(sd).bfloat16() for sh, sd in (((vocab, 64), 1.0), ((64,), 1.0), ((64, vocab), std / 8))]
    eng.pack_globals({"embed": w[0], "gf": w[1], "wlm": w[2]})
    return eng, torch.randn(rows, 64, generator=g, device="cuda"), torch.arange(rows, dtype=torch.int32, device="cuda")


def test_flat_rows_cost_what_others_do(hx):
    """The entries of the cut bin are listed, whatever the spread of the logits: rows whose bins overflow the lists are gone
    through again by one workgroup, which took twice as long."""
    eng, x, pos = top_p_engine(hx, 128, 151936, 1.0)

    def us(temperature):
        best = 1e9
        for _ in range(5):
            a, b = torch.cuda.Event(True), torch.cuda.Event(True)
            a.record()
            for _ in range(10):
                eng.stage_lm_head_top_p(x, pos, temperature, 0.5, 9)
            b.record()
            torch.cuda.synchronize()
            best = min(best, a.elapsed_time(b) * 100)
        return best
    us(1.0)
    usual = us(1.0)
    for temperature in (5.0, 30.0, 1000.0):
        assert us(temperature) <= 1.4 * usual, (temperature, usual)


@pytest.mark.parametrize("vocab,rows", [(49148, 8), (49152, 8), (49152, 64), (49152, 65), (98304, 128), (98304, 129), (151936, 200)])
def test_kept_sets_beside_the_edges_of_the_split(hx, vocab, rows):
    """One workgroup per row and several: both sides of the row's length and of the number of rows where it turns."""
    eng, x, pos = top_p_engine(hx, rows, vocab, 2.0)
    for top_p in (0.2, 0.9):
        y, tok, lp, n = [t.cpu().numpy() for t in eng.stage_lm_head_top_p(x, pos, 0.7, top_p, 5)]
        otok, olp, on, margin, gap = oracle.sample_top_p(y, 0.7, top_p, 5, np.arange(rows), pos.cpu().numpy())
        firm = margin > 1e-7                  # as in test_gpu_top_p.py: a sum of 1e5 fp32 exponentials
        same = firm & (gap > 1e-4)
        assert firm.sum() > rows // 2 and np.array_equal(n[firm], on[firm])
        assert np.array_equal(tok[same], otok[same]) and np.abs(lp[same] - olp[same]).max(initial=0.0) <= 2e-4


def test_draws_between_prompt_chunks(hx):
    """A draw's lists lie where prompt attention keeps its partial results: chunks and draws of one engine in turn, each as alone."""
    s = synth.ModelShape("nd", 2, 64, 2, 1, 64, 96, 65536)
    eng = build(hx, s, 11, 256, 4096)
    n = 3000
    kv = hx.KVCache(eng, 200)
    table = torch.arange(200, dtype=torch.int32, device="cuda").flip(0)[None].contiguous()
    start = torch.tensor([0, n], dtype=torch.int32, device="cuda")
    g = torch.Generator(device="cuda").manual_seed(5)
    for l in range(s.n_layers):
        k, v = torch.randn(2, n, s.n_kv_heads, s.head_dim, generator=g, device="cuda").bfloat16()
        kv.prefill_fill(l, k, v, start, table)
    pos = torch.arange(n - 256, n, dtype=torch.int32, device="cuda")
    toks = torch.arange(256, dtype=torch.int32, device="cuda")
    rows_table = table.expand(256, -1).contiguous()
    x = torch.randn(16, s.hidden, generator=g, device="cuda")
    step = torch.arange(16, dtype=torch.int32, device="cuda")

    def chunk():
        eng.prefill_chunk(kv, toks, pos, pos + 1, rows_table)
        return torch.stack(kv.gather(s.n_layers - 1, n, start, table)).clone()

    def draw():
        return [t.clone() for t in eng.stage_lm_head_top_p(x, step, 1.0, 0.9, 3)]
    alone = chunk()
    drawn = draw()
    for _ in range(3):
        assert torch.equal(chunk(), alone)
        assert all(torch.equal(a, b) for a, b in zip(draw(), drawn))
