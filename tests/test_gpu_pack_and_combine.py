"""Weight packing where its loads change (sources off a 16-byte boundary, rows that end inside a group of 8 columns, an odd
number of k-steps, column counts inside a workgroup's 512), and the attention combine at the number of partials where it changes kernels."""
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


@pytest.mark.parametrize("shift", [0, 1, 4])
@pytest.mark.parametrize("intermediate,vocab", [(688, 1000), (16, 1004), (528, 2052)])
def test_products_of_packed_weights(hx, intermediate, vocab, shift):
    """shift: elements by which the source lies beyond a 16-byte boundary; 1004 and 2052 columns are no multiple of 8."""
    s = synth.ModelShape("pack", 1, 256, 4, 2, 64, intermediate, vocab)
    eng = build(hx, s, 3, 8, 64)
    g = torch.Generator(device="cuda").manual_seed(11)

    def fresh(rows, cols):
        flat = torch.empty(rows * cols + 8, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.05, generator=g)
        return flat[shift:shift + rows * cols].view(rows, cols)

    wd, wg, wu, wlm = fresh(intermediate, 256), fresh(256, intermediate), fresh(256, intermediate), fresh(256, vocab)
    for kind, w in ((hx.HX_T_WD, wd), (hx.HX_T_WG, wg), (hx.HX_T_WU, wu), (hx.HX_T_WLM, wlm)):
        eng.weights_pack(kind, 0, w)
    for kind, w in ((hx.HX_T_WD, wd), (hx.HX_T_WLM, wlm), (hx.HX_T_WG, None)):
        x = torch.randn(5, 256 if w is None else w.shape[0], generator=g, device="cuda").bfloat16().float()
        y = eng.stage_linear(kind, 0, x)
        y = (y[0] if isinstance(y, tuple) else y).double()
        xd = x.double()
        if w is None:
            gate = xd @ wg.double()
            ref = gate * torch.sigmoid(gate) * (xd @ wu.double())
            assert ((y - ref).abs() <= ref.abs() * 2.0 ** -7 + 1e-5).all()       # one bf16 rounding of the result
        else:
            assert ((y - xd @ w.double()).abs() <= 1e-5 * (xd.abs() @ w.double().abs())).all()   # fp32 sums of exact products


@pytest.mark.parametrize("shift", [0, 1, 4])
@pytest.mark.parametrize("intermediate,vocab", [(688, 1000), (16, 132), (2064, 40004)])
def test_tensors_packed_together_and_one_by_one(hx, intermediate, vocab, shift):
    """One launch for all tensors of a layer, or of the model, leaves the bytes that one call per tensor leaves; tensors on the
    host go along; a refused tensor keeps the others from being packed."""
    s = synth.ModelShape("many", 2, 96, 3, 1, 64, intermediate, vocab)
    nbytes = hx.Engine(s, 4, 64).weights.numel()
    one, many, mixed = [hx.Engine(s, 4, 64, weights=torch.zeros(nbytes, dtype=torch.uint8, device="cuda")) for _ in range(3)]
    g = torch.Generator(device="cuda").manual_seed(5)

    def fresh(*shape):
        n = int(np.prod(shape))
        return torch.empty(n + 8, dtype=torch.bfloat16, device="cuda").normal_(0.0, 0.05, generator=g)[shift:shift + n].view(*shape)

    kinds = {"g1": (hx.HX_T_G1, (96,)), "wqkv": (hx.HX_T_WQKV, (96, 320)), "bqkv": (hx.HX_T_BQKV, (320,)), "wo": (hx.HX_T_WO, (192, 96)),
             "g2": (hx.HX_T_G2, (96,)), "wg": (hx.HX_T_WG, (96, intermediate)), "wu": (hx.HX_T_WU, (96, intermediate)),
             "wd": (hx.HX_T_WD, (intermediate, 96))}
    top = {"embed": (hx.HX_T_EMBED, (vocab, 96)), "gf": (hx.HX_T_GF, (96,)), "wlm": (hx.HX_T_WLM, (96, vocab))}
    for layer, group in ((0, kinds), (1, kinds), (None, top)):
        w = {n: fresh(*sh) for n, (_, sh) in group.items()}
        for n, (k, _) in group.items():
            one.weights_pack(k, layer or 0, w[n])
        half = {n: t.cpu() if i % 2 else t for i, (n, t) in enumerate(w.items())}
        if layer is None:
            many.pack_globals(w)
            mixed.pack_globals(half)
        else:
            many.pack_layer(layer, w)
            mixed.pack_layer(layer, half)
    torch.cuda.synchronize()
    assert torch.equal(one.weights, many.weights) and torch.equal(one.weights, mixed.weights)
    bad = {n: fresh(*sh) for n, (_, sh) in kinds.items()}
    bad["wd"] = fresh(intermediate, 95)
    with pytest.raises(hx.HexError):
        many.pack_layer(1, bad)
    torch.cuda.synchronize()
    assert torch.equal(one.weights, many.weights)


@pytest.mark.parametrize("cache", ["bf16", "fp8"])
@pytest.mark.parametrize("d,lens", [(128, [500]), (128, [520]), (128, [8000, 17, 3000]), (64, [4096]), (64, [1, 900])])
def test_combine_of_many_partials(hx, d, lens, cache, monkeypatch):
    """32 and 33 blocks are the edge of the eight-wavefront combine.  Reference: 64 wavefronts, few partials per pair."""
    s = synth.ModelShape("comb", 1, 256, 6, 2, d, 688, 1000)
    kv_dtype = hx.HX_KV_FP8_E4M3 if cache == "fp8" else hx.HX_KV_BF16
    n = np.array(lens, dtype=np.int32)
    table, nb = synth.block_table(n, 16, 3)
    start = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    q = torch.randn(len(lens), s.q_dim, generator=torch.Generator(device="cuda").manual_seed(2), device="cuda").bfloat16().float()
    out = []
    for waves in (None, "64"):
        if waves:
            monkeypatch.setenv("HX_ATTN_WAVES", waves)
        eng = build(hx, s, 3, len(lens), int(n.max()) + 1, kv_dtype)
        kv = hx.KVCache(eng, nb)
        kv.pool.fill_(0xFF)
        k, v = synth.kv_fill(s, 0, int(n.sum()), 3, device="cuda")
        kv.prefill_fill(0, k, v, dev(start), dev(table))
        out.append(eng.stage_attention(kv, 0, q, dev(n), dev(table)))
    torch.cuda.synchronize()
    assert torch.isfinite(out[0]).all()
    assert float((out[0] - out[1]).abs().max()) <= 2e-5 * max(float(out[1].abs().max()), 1.0)
