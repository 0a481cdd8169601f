"""Products of matrices with few columns (gemm_slice.hip): every number of k-steps that leaves wavefronts without work or the ring
part-filled, odd numbers of tiles, ragged last tiles, both sides of the row groups' edges, one and two tiles per workgroup, and
the step to the streaming kernel (68 | 69 tiles on 256 compute units).  Reference: the product in float64."""
import pytest
import torch

from paper_2511_00796_amd import synth
from test_gpu_prefill import build

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hx():
    from paper_2511_00796_amd import binding
    binding.load()
    return binding


# hidden x (heads) x intermediate x vocab.  k-steps of the down product: 1, 5, 23, 48 (two splits), 217 (one more than nine
# splits of 24: two tiles per workgroup); columns: 64 to 2080, 1000 (the last tile holds 8)
SHAPES = {"k1": synth.ModelShape("sp-k1", 1, 64, 1, 1, 64, 16, 64), "k5": synth.ModelShape("sp-k5", 1, 96, 3, 1, 64, 80, 1000),
          "k23": synth.ModelShape("sp-k23", 1, 352, 4, 2, 128, 368, 36), "k48": synth.ModelShape("sp-k48", 1, 768, 6, 1, 128, 768, 2048),
          "k217": synth.ModelShape("sp-k217", 1, 480, 2, 2, 128, 3472, 2080)}
# 68 and 69 tiles: a head of 2176 and of 2180 columns (its last tile holds 4), O and down products (split) of hidden sizes 2176 and 2208
for hidden, vocab in ((2176, 2180), (2208, 2176)):
    SHAPES["t%d" % (hidden // 32)] = synth.ModelShape("sp-t%d" % (hidden // 32), 1, hidden, 6, 1, 128, 800, vocab)


@pytest.mark.parametrize("batch", [1, 31, 33, 64, 65, 100, 128])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_products_of_few_columns(hx, name, batch):
    s = SHAPES[name]
    eng = build(hx, s, 5, batch, 64)
    w = {k: v.double().cuda() for k, v in synth.layer_weights(s, 0, 5).items()}
    head = synth.global_weights(s, 5)["wlm"].double().cuda()
    g = torch.Generator(device="cuda").manual_seed(7)
    for kind, mat in ((hx.HX_T_WQKV, w["wqkv"]), (hx.HX_T_WO, w["wo"]), (hx.HX_T_WD, w["wd"]), (hx.HX_T_WG, None), (hx.HX_T_WLM, head)):
        K = s.hidden if mat is None else mat.shape[0]
        x = torch.randn(batch, K, generator=g, device="cuda").bfloat16().float()
        y = eng.stage_linear(kind, 0, x, want_argmax=True) if kind == hx.HX_T_WLM else eng.stage_linear(kind, 0, x)
        torch.cuda.synchronize()
        if kind == hx.HX_T_WLM:
            y, am = y
            assert (am.long() == y.argmax(-1)).all()
        xd = x.double()
        if mat is None:
            gate = xd @ w["wg"]
            ref = gate * torch.sigmoid(gate) * (xd @ w["wu"])
            # one bf16 rounding of the result (2^-8 at most with ties and the fp32 sums' own error)
            assert y.shape == ref.shape and ((y.double() - ref).abs() <= ref.abs() * 2.0 ** -7 + 1e-5).all(), (name, kind)
        else:
            # fp32 sums of exact products: a few units of 2^-24 of the sum of magnitudes
            ref = xd @ mat
            assert y.shape == ref.shape and ((y.double() - ref).abs() <= 1e-5 * (xd.abs() @ mat.abs())).all(), (name, kind)


@pytest.mark.parametrize("batch,max_batch", [(129, 129), (192, 256), (193, 193), (256, 256)])
@pytest.mark.parametrize("name", ["k1", "k5", "k23", "k48", "k217", "t68"])
def test_products_of_few_columns_beyond_128_rows(hx, name, batch, max_batch):
    """Blocks of 64 rows (two tiles per workgroup: 128), the last of which may hold one row; what lies behind the rows is not a number."""
    s = SHAPES[name]
    eng = build(hx, s, 5, max_batch, 64)
    w = {k: v.double().cuda() for k, v in synth.layer_weights(s, 0, 5).items()}
    head = synth.global_weights(s, 5)["wlm"].double().cuda()
    g = torch.Generator(device="cuda").manual_seed(7)
    eng.workspace.fill_(0xFF)
    for kind, mat in ((hx.HX_T_WQKV, w["wqkv"]), (hx.HX_T_WO, w["wo"]), (hx.HX_T_WD, w["wd"]), (hx.HX_T_WG, None), (hx.HX_T_WLM, head)):
        x = torch.randn(batch, s.hidden if mat is None else mat.shape[0], generator=g, device="cuda").bfloat16().float()
        y, am = eng.stage_linear(kind, 0, x, want_argmax=True) if kind == hx.HX_T_WLM else (eng.stage_linear(kind, 0, x), None)
        torch.cuda.synchronize()
        assert am is None or (am.long() == y.argmax(-1)).all()
        xd = x.double()
        if mat is None:
            gate = xd @ w["wg"]
            ref = gate * torch.sigmoid(gate) * (xd @ w["wu"])
            # one bf16 rounding of the result and the fp32 sums' own error
            assert y.shape == ref.shape and ((y.double() - ref).abs() <= ref.abs() * 2.0 ** -7 + 1e-5).all(), (name, kind)
        else:
            # fp32 sums of exact products
            ref = xd @ mat
            assert y.shape == ref.shape and ((y.double() - ref).abs() <= 1e-5 * (xd.abs() @ mat.abs())).all(), (name, kind)


@pytest.mark.parametrize("batch", [1, 32, 33, 64, 65, 128])
@pytest.mark.parametrize("tiles,hidden", [(69, 32), (256, 96), (257, 192), (512, 160), (513, 96), (770, 64)])
def test_gate_up_of_one_and_two_tiles_per_workgroup(hx, tiles, hidden, batch):
    """Both sides of the steps between one and two tiles per workgroup (256 on 256 compute units) and to the streaming kernel (512),
    last workgroups with tiles that do not exist, fewer k-steps than wavefronts."""
    s = synth.ModelShape("sp-gu", 1, hidden, 1, 1, 64, 16 * tiles, 64)
    eng = build(hx, s, 5, batch, 64)
    w = {k: v.double().cuda() for k, v in synth.layer_weights(s, 0, 5).items()}
    eng.workspace.fill_(0xFF)
    x = torch.randn(batch, hidden, generator=torch.Generator(device="cuda").manual_seed(7), device="cuda").bfloat16().float()
    y = eng.stage_linear(hx.HX_T_WG, 0, x)
    torch.cuda.synchronize()
    gate = x.double() @ w["wg"]
    ref = gate * torch.sigmoid(gate) * (x.double() @ w["wu"])
    # one bf16 rounding of the result and the fp32 sums' own error
    assert y.shape == ref.shape and ((y.double() - ref).abs() <= ref.abs() * 2.0 ** -7 + 1e-5).all()


@pytest.mark.parametrize("tiles,hidden", [(256, 512), (257, 512), (512, 512), (513, 512), (560, 1536), (768, 512), (769, 512)])
def test_a_row_comes_out_alike_in_every_batch_of_up_to_128(hx, tiles, hidden):
    """The order in which a row's products are added hangs on the matrix alone, at every number of gate|up tiles where a plan ends:
    the rows of 1, 32, 33, 64 and 65 are those of 128, bit for bit, and so are those of the other products."""
    s = synth.ModelShape("sp-alike", 1, hidden, 4, 2, 64, 16 * tiles, 70000 if tiles == 513 else 2180)     # a head in ten tiles per workgroup, too
    eng = build(hx, s, 5, 128, 64)
    g = torch.Generator(device="cuda").manual_seed(7)
    for kind, K in ((hx.HX_T_WG, hidden), (hx.HX_T_WQKV, hidden), (hx.HX_T_WO, s.q_dim), (hx.HX_T_WD, s.intermediate), (hx.HX_T_WLM, hidden)):
        x = torch.randn(128, K, generator=g, device="cuda")
        whole = eng.stage_linear(kind, 0, x)
        for batch in (1, 32, 33, 64, 65):
            assert torch.equal(eng.stage_linear(kind, 0, x[:batch].contiguous()), whole[:batch]), (kind, batch)


# (tile, split) pairs that are no multiple of 8 (one workgroup in 8 of the last ones has nothing to do), one and two tiles per workgroup, an odd
# last tile group; 1 pair, 7 (one tile of 168 k-steps), 68, 25 x 5, 31 x 4, 34 x 3
# (the last two: 720 and 721 k-steps of 65 tiles, the step to the workgroup-tiled kernel)
@pytest.mark.parametrize("hidden,intermediate", [(32, 16), (32, 2688), (2176, 368), (1568, 3472), (1984, 3488), (2176, 3472), (2080, 11520), (2080, 11536)])
def test_row_blocks_of_pairs_that_do_not_fill_the_xcds(hx, hidden, intermediate):
    """Every number of row blocks: against float64 at 256 rows, and fewer rows are, bit for bit, the first of those."""
    s = synth.ModelShape("sp-xcd", 1, hidden, 1, 1, 64, intermediate, 64)
    eng = build(hx, s, 5, 256, 64)
    w = synth.layer_weights(s, 0, 5)["wd"].double().cuda()
    x = torch.randn(256, intermediate, generator=torch.Generator(device="cuda").manual_seed(7), device="cuda").bfloat16().float()
    eng.workspace.fill_(0xFF)
    whole = eng.stage_linear(hx.HX_T_WD, 0, x)
    # fp32 sums of exact products
    assert ((whole.double() - x.double() @ w).abs() <= 1e-5 * (x.double().abs() @ w.abs())).all()
    for batch in (129, 160, 192, 193, 255):
        eng.workspace.fill_(0xFF)
        assert torch.equal(eng.stage_linear(hx.HX_T_WD, 0, x[:batch].contiguous()), whole[:batch]), batch
