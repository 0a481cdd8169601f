"""Products of more than 128 rows outside prefill_rows: batches at the edges of the workgroup-tiled kernel, an odd number of
k-steps, engines for fewer than 256 rows (whose partial buffer caps the K-splits), column blocks that end inside a
workgroup's tile; the sampled heads: test_gpu_draw_paths.py.  Reference: the product in float64."""
import numpy as np
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


# intermediate 688 = 43 k-steps, 16 = one; 2080 = 130; vocab 1000: the last head tile holds 8 columns
SHAPES = {"odd": synth.ModelShape("wb-odd", 1, 256, 4, 2, 64, 688, 1000), "one": synth.ModelShape("wb-one", 1, 64, 1, 1, 64, 16, 64),
          "splits": synth.ModelShape("wb-splits", 1, 1536, 12, 2, 128, 2080, 2048)}


@pytest.mark.parametrize("batch,max_batch", [(129, 129), (130, 200), (255, 256), (256, 256)])
@pytest.mark.parametrize("name", sorted(SHAPES))
def test_products_beyond_128_rows(hx, name, batch, max_batch):
    s = SHAPES[name]
    eng = build(hx, s, 5, max_batch, 64)
    w = {k: v.double().cuda() for k, v in synth.layer_weights(s, 0, 5).items()}
    g = torch.Generator(device="cuda").manual_seed(7)
    head = synth.global_weights(s, 5)["wlm"].double().cuda()
    for kind, mat in ((hx.HX_T_WQKV, w["wqkv"]), (hx.HX_T_WO, w["wo"]), (hx.HX_T_WD, w["wd"]), (hx.HX_T_WG, None), (hx.HX_T_WLM, head)):
        K = s.hidden if mat is None else mat.shape[0]
        N = s.intermediate if mat is None else mat.shape[1]
        x = torch.randn(batch, K, generator=g, device="cuda").bfloat16().float()
        y = eng.stage_linear(kind, 0, x)
        y = y[0] if isinstance(y, tuple) else y
        torch.cuda.synchronize()
        assert y.shape == (batch, N)
        xd = x.double()
        if mat is None:
            gate = xd @ w["wg"]
            ref = gate * torch.sigmoid(gate) * (xd @ w["wu"])
            # one bf16 rounding of the result (2^-8 at most with ties and the fp32 sums' own error)
            assert ((y.double() - ref).abs() <= ref.abs() * 2.0 ** -7 + 1e-5).all(), (name, kind)
        else:
            # fp32 sums of exact products: a few units of 2^-24 of the sum of magnitudes
            bound = xd.abs() @ mat.abs()
            assert ((y.double() - (xd @ mat)).abs() <= 1e-5 * bound).all(), (name, kind)


@pytest.mark.parametrize("knob,value", [("HX_GEMM_MAX_SPLITS", "1"), ("HX_GEMM_SHAPE", "5,1,2"), ("HX_GEMM_SHAPE", "8,1,3"), ("HX_GEMM_SHAPE", "4,2,1")])
@pytest.mark.parametrize("batch,max_batch", [(130, 130), (256, 256)])
def test_forced_plans_beyond_128_rows(hx, batch, max_batch, knob, value, monkeypatch):
    """The knobs that force plans hold beyond 128 rows, too; a shape that does not exist there, or needs more partial results
    than the engine's buffer holds, is ignored."""
    s = SHAPES["splits"]
    eng = build(hx, s, 5, max_batch, 64)
    wd = synth.layer_weights(s, 0, 5)["wd"].double().cuda()
    x = torch.randn(batch, s.intermediate, generator=torch.Generator(device="cuda").manual_seed(7), device="cuda").bfloat16().float()
    monkeypatch.setenv(knob, value)
    y = eng.stage_linear(hx.HX_T_WD, 0, x)
    torch.cuda.synchronize()
    assert ((y.double() - x.double() @ wd).abs() <= 1e-5 * (x.double().abs() @ wd.abs())).all()


@pytest.mark.parametrize("tiles", [4, 5, 6])
@pytest.mark.parametrize("k_steps", [1, 2, 9, 10, 11, 12, 13, 14])
def test_fewer_and_more_chunks_than_stages(hx, k_steps, tiles, monkeypatch):
    """Products of 1 to 7 chunks: the ring of LDS stages (six of the narrow tiles, three of the others) holds all of them, or not."""
    s = synth.ModelShape("wb-ring", 1, 192, 2, 1, 64, 16 * k_steps, 64)
    eng = build(hx, s, 5, 130, 64)
    wd = synth.layer_weights(s, 0, 5)["wd"].double().cuda()
    x = torch.randn(130, s.intermediate, generator=torch.Generator(device="cuda").manual_seed(7), device="cuda").bfloat16().float()
    monkeypatch.setenv("HX_GEMM_SHAPE", "%d,1,1" % tiles)
    y = eng.stage_linear(hx.HX_T_WD, 0, x)
    torch.cuda.synchronize()
    # fp32 sums of exact products, as above
    assert ((y.double() - x.double() @ wd).abs() <= 1e-5 * (x.double().abs() @ wd.abs())).all()


@pytest.mark.parametrize("rows", [127, 128, 129, 135, 136, 137, 200, 255, 256])
def test_every_row_is_normalised_once(hx, rows):
    """Beyond 128 rows the row kernels deal their rows to the XCDs in eighths, the last of which may be short or empty."""
    s = SHAPES["odd"]
    eng = build(hx, s, 5, 256, 64)
    x = torch.randn(rows, s.hidden, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    y = eng.stage_rmsnorm(hx.HX_T_G1, 0, x)
    torch.cuda.synchronize()
    xd = x.double()
    ref = xd * torch.rsqrt((xd * xd).mean(-1, keepdim=True) + s.rms_eps) * synth.layer_weights(s, 0, 5)["g1"].double().cuda()
    # one bf16 rounding (2^-9 relative) and the fp32 norm's own error
    assert y.shape == x.shape and ((y.double() - ref).abs() <= ref.abs() * 2.0 ** -8 + 1e-6).all()


@pytest.mark.parametrize("tiles,blocks,hidden", [(512, 2, 32), (338, 6, 32), (640, 2, 32), (640, 2, 192), (1026, 2, 32), (1026, 2, 96), (1026, 2, 192)])
def test_gate_up_of_one_and_two_rounds(hx, tiles, blocks, hidden):
    """Narrow tiles of gate|up on as many workgroups as compute units (256 of 4 and of 5 tiles), and on more (510 of 4, 412 of 5),
    which have another number of LDS stages: products of 1, 3 and 6 chunks."""
    s = synth.ModelShape("wb-gu", 1, hidden, 1, 1, 64, 16 * tiles, 64)
    eng = build(hx, s, 5, 256, 64)
    w = {k: v.double().cuda() for k, v in synth.layer_weights(s, 0, 5).items()}
    ws = torch.empty(hx.prefill_workspace_bytes(eng.cfg, 256 * blocks), dtype=torch.uint8, device="cuda")
    x = torch.randn(256 * blocks, hidden, generator=torch.Generator(device="cuda").manual_seed(7), device="cuda").bfloat16().float()
    y = eng.stage_linear_rows(hx.HX_T_WG, 0, x, ws)
    torch.cuda.synchronize()
    gate = x.double() @ w["wg"]
    ref = gate * torch.sigmoid(gate) * (x.double() @ w["wu"])
    # one bf16 rounding of the result and the fp32 sums' own error
    assert y.shape == ref.shape and ((y.double() - ref).abs() <= ref.abs() * 2.0 ** -7 + 1e-5).all()


@pytest.mark.parametrize("tiles", [6, 7, 8])
@pytest.mark.parametrize("k_steps,batch", [(1, 129), (2, 130), (3, 255), (5, 256), (8, 129), (13, 256)])
def test_wide_tiles(hx, k_steps, batch, tiles, monkeypatch):
    """Six and more column tiles per workgroup (16x16x32 products): 1 to 7 chunks, the last of them half empty (what lies behind it
    is not a number here), column blocks that end inside a workgroup, and gate|up."""
    s = synth.ModelShape("wb-wide", 1, 288, 2, 1, 64, 16 * k_steps, 64)
    eng = build(hx, s, 5, 256, 64)
    w = {k: v.double().cuda() for k, v in synth.layer_weights(s, 0, 5).items()}
    monkeypatch.setenv("HX_GEMM_SHAPE", "%d,1,1" % tiles)
    g = torch.Generator(device="cuda").manual_seed(7)
    eng.workspace.fill_(0xFF)
    x = torch.randn(batch, s.intermediate, generator=g, device="cuda").bfloat16().float()
    y = eng.stage_linear(hx.HX_T_WD, 0, x)
    u = torch.randn(batch, s.hidden, generator=g, device="cuda").bfloat16().float()
    m = eng.stage_linear(hx.HX_T_WG, 0, u)
    torch.cuda.synchronize()
    # fp32 sums of exact products; one bf16 rounding of gate|up's result and the fp32 sums' own error
    assert ((y.double() - x.double() @ w["wd"]).abs() <= 1e-5 * (x.double().abs() @ w["wd"].abs())).all()
    gate = u.double() @ w["wg"]
    ref = gate * torch.sigmoid(gate) * (u.double() @ w["wu"])
    assert m.shape == ref.shape and ((m.double() - ref).abs() <= ref.abs() * 2.0 ** -7 + 1e-5).all()


@pytest.mark.parametrize("tiles", [4, 5])
@pytest.mark.parametrize("batch", [129, 160, 161, 192, 193])
@pytest.mark.parametrize("hidden,k_steps", [(96, 2), (160, 14), (2080, 26)])
def test_blocks_with_groups_that_hold_no_rows(hx, hidden, k_steps, batch, tiles, monkeypatch):
    """Five and six m-groups of a single block (seven and eight: the kernel of full blocks), few and many chunks, splits, column blocks
    that end inside a workgroup; gate|up of 128 and more k-steps copies its weights non-temporally.  What lies behind the rows is not
    a number."""
    s = synth.ModelShape("wb-part", 1, hidden, 2, 1, 64, 16 * k_steps, 64)
    eng = build(hx, s, 5, 256, 64)
    w = {k: v.double().cuda() for k, v in synth.layer_weights(s, 0, 5).items()}
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(batch, s.intermediate, generator=g, device="cuda").bfloat16().float()
    u = torch.randn(batch, s.hidden, generator=g, device="cuda").bfloat16().float()
    for splits in (1, 2):
        monkeypatch.setenv("HX_GEMM_SHAPE", "%d,1,%d" % (tiles, splits))
        eng.workspace.fill_(0xFF)
        y = eng.stage_linear(hx.HX_T_WD, 0, x)
        # fp32 sums of exact products
        assert ((y.double() - x.double() @ w["wd"]).abs() <= 1e-5 * (x.double().abs() @ w["wd"].abs())).all()
    monkeypatch.setenv("HX_GEMM_SHAPE", "%d,1,1" % tiles)
    eng.workspace.fill_(0xFF)
    m = eng.stage_linear(hx.HX_T_WG, 0, u)
    torch.cuda.synchronize()
    gate = u.double() @ w["wg"]
    ref = gate * torch.sigmoid(gate) * (u.double() @ w["wu"])
    # one bf16 rounding of the result and the fp32 sums' own error
    assert m.shape == ref.shape and ((m.double() - ref).abs() <= ref.abs() * 2.0 ** -7 + 1e-5).all()


@pytest.mark.parametrize("k_steps,splits", [(1, 1), (2, 1), (65, 1), (66, 1), (131, 1), (216, 1), (65, 2), (66, 2), (131, 2), (216, 2)])
def test_both_matrix_instructions_give_the_same_bits(hx, k_steps, splits, monkeypatch):
    """Six and more tiles per workgroup add a row's products with 16x16x32 instructions, fewer with 32x32x16: the same sums, bit for
    bit, with one and two splits (the second behind an odd last k-step too), of values of very different sizes, and gate|up of them."""
    s = synth.ModelShape("wb-bits", 1, 416, 2, 1, 64, 16 * k_steps, 64)
    eng = build(hx, s, 5, 256, 64)
    g = torch.Generator(device="cuda").manual_seed(7)
    x = torch.randn(256, s.intermediate, generator=g, device="cuda") * torch.exp(3 * torch.randn(256, s.intermediate, generator=g, device="cuda"))
    u = torch.randn(256, s.hidden, generator=g, device="cuda") * torch.exp(torch.randn(256, s.hidden, generator=g, device="cuda"))
    out = []
    for tiles in (4, 5, 6, 7, 8):
        monkeypatch.setenv("HX_GEMM_SHAPE", "%d,1,%d" % (tiles, splits))
        eng.workspace.fill_(0xFF)
        y = eng.stage_linear(hx.HX_T_WD, 0, x)
        monkeypatch.setenv("HX_GEMM_SHAPE", "%d,1,1" % tiles)
        out.append((y, eng.stage_linear(hx.HX_T_WG, 0, u)))
    for y, m in out[1:]:
        assert torch.equal(y, out[0][0]) and torch.equal(m, out[0][1])
