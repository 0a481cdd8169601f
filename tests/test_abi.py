"""Host-side checks of the C-ABI library that need no GPU: it loads, exports every symbol the header
declares, its pure-host entry points (size queries, argument validation) behave as documented."""
import ctypes as C
import dataclasses
import os
import re

import pytest

from paper_2511_00796_amd import binding, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def declared_functions():
    text = open(os.path.join(ROOT, "include", "hexdecode.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    names = re.findall(r"\b(?:int|const char \*)\s*\*?\s*([a-z_0-9]+)\s*\(", text)
    return sorted(set(names))


def test_library_exports_every_declared_symbol():
    lib = binding.load()
    names = declared_functions()
    assert set(names) == set(binding.EXPORTS), sorted(set(names) ^ set(binding.EXPORTS))
    for n in names:
        assert hasattr(lib, n), n


def test_size_queries_are_consistent_with_the_shapes():
    for wl in synth.WORKLOADS.values():
        s = wl.shape
        cfg = binding.make_config(s, wl.batch, 16400)
        wb = binding.weights_bytes(cfg)
        # packed weights = streamed weights + embedding table, plus padding only
        logical = 2 * (s.weight_elements() + s.vocab * s.hidden)
        assert logical <= wb <= logical * 1.01 + (1 << 20)
        assert binding.kv_bytes(cfg, 1000) == s.n_layers * 1000 * s.n_kv_heads * 2 * 16 * s.head_dim * 2
        assert binding.workspace_bytes(cfg) > 0


def test_bad_configurations_are_rejected_with_codes_not_crashes():
    s = synth.TINY
    good = binding.make_config(s, 4, 256)
    assert binding.weights_bytes(good) > 0

    def expect(code, **kw):
        cfg = binding.make_config(s, 4, 256)
        for k, v in kw.items():
            setattr(cfg, k, v)
        out = C.c_size_t()
        rc = binding.load().hx_weights_bytes(C.byref(cfg), C.byref(out))
        assert rc == code, (kw, rc, binding.last_error())
        assert binding.last_error()

    expect(binding.HX_E_CONFIG, struct_size=8)
    expect(binding.HX_E_CONFIG, head_dim=96)
    expect(binding.HX_E_CONFIG, n_q_heads=5)
    expect(binding.HX_E_CONFIG, n_q_heads=34)          # 17 query heads per KV head
    expect(binding.HX_E_CONFIG, hidden=250)
    expect(binding.HX_E_CONFIG, intermediate=100)
    expect(binding.HX_E_CONFIG, block_size=32)
    expect(binding.HX_E_CONFIG, max_batch=0)
    expect(binding.HX_E_CONFIG, max_batch=257)
    expect(binding.HX_E_CONFIG, vocab=1023)
    lib = binding.load()
    assert lib.hx_weights_bytes(None, C.byref(C.c_size_t())) == binding.HX_E_NULL
    assert lib.hx_weights_bytes(C.byref(good), None) == binding.HX_E_NULL
    out = C.c_size_t()
    assert lib.hx_kv_bytes(C.byref(good), 0, C.byref(out)) == binding.HX_E_RANGE


def test_engine_create_validates_buffers_on_the_host():
    lib = binding.load()
    cfg = binding.make_config(synth.TINY, 4, 256)
    wb, sb = binding.weights_bytes(cfg), binding.workspace_bytes(cfg)
    h = C.c_void_p()
    fake = 0x10000000   # never dereferenced: creation only records addresses
    assert lib.hx_engine_create(C.byref(cfg), None, wb, fake, sb, C.byref(h)) == binding.HX_E_NULL
    assert lib.hx_engine_create(C.byref(cfg), fake + 8, wb, fake, sb, C.byref(h)) == binding.HX_E_ALIGN
    assert lib.hx_engine_create(C.byref(cfg), fake, wb - 1, fake, sb, C.byref(h)) == binding.HX_E_TOO_SMALL
    assert lib.hx_engine_create(C.byref(cfg), fake, wb, fake, sb - 1, C.byref(h)) == binding.HX_E_TOO_SMALL
    assert lib.hx_engine_create(C.byref(cfg), fake, wb, fake, sb, C.byref(h)) == binding.HX_OK
    eng = h
    kvh = C.c_void_p()
    kb = binding.kv_bytes(cfg, 10)
    assert lib.kv_alloc(eng, fake, kb - 1, 10, C.byref(kvh)) == binding.HX_E_TOO_SMALL
    assert lib.kv_alloc(eng, fake, kb, 10, C.byref(kvh)) == binding.HX_OK
    # scalar validation of the step happens before anything is enqueued
    p = C.c_void_p(fake)
    assert lib.decode_step(eng, kvh, 0, p, p, p, p, 4, None, p, None) == binding.HX_E_RANGE
    assert lib.decode_step(eng, kvh, 5, p, p, p, p, 4, None, p, None) == binding.HX_E_RANGE
    assert lib.decode_step(eng, kvh, 4, p, p, p, p, 0, None, p, None) == binding.HX_E_RANGE
    assert lib.decode_step(eng, kvh, 4, None, p, p, p, 4, None, p, None) == binding.HX_E_NULL
    assert lib.decode_step(None, kvh, 4, p, p, p, p, 4, None, p, None) == binding.HX_E_NULL
    f32 = C.c_float
    assert lib.decode_step_sample(eng, kvh, 4, p, p, p, p, 4, f32(0.0), 1, None, None, p, p, None) == binding.HX_E_RANGE
    assert lib.decode_step_sample(eng, kvh, 4, p, p, p, p, 4, f32(-2.0), 1, None, None, p, p, None) == binding.HX_E_RANGE
    assert lib.decode_step_sample(eng, kvh, 4, p, p, p, p, 4, f32(float("nan")), 1, None, None, p, p, None) == binding.HX_E_RANGE
    assert lib.decode_step_sample(eng, kvh, 4, p, p, p, p, 4, f32(1.0), 1, None, None, p, None, None) == binding.HX_E_NULL
    assert lib.decode_step_sample(eng, kvh, 9, p, p, p, p, 4, f32(1.0), 1, None, None, p, p, None) == binding.HX_E_RANGE
    assert lib.hx_weights_pack(eng, binding.HX_T_WO, 0, p, 3, 3, None) == binding.HX_E_SHAPE
    assert lib.hx_weights_pack(eng, binding.HX_T_WO, 9, p, 256, 256, None) == binding.HX_E_SHAPE
    assert lib.hx_weights_pack(eng, 99, 0, p, 256, 256, None) == binding.HX_E_SHAPE
    assert lib.kv_free(kvh) == binding.HX_OK
    assert lib.hx_engine_destroy(eng) == binding.HX_OK
    assert lib.hx_engine_destroy(None) == binding.HX_E_NULL


def test_product_plans_fill_the_chip_and_respect_their_limits(monkeypatch):
    """Host-side launch planner: every plan keeps at least 16 k-steps per split, never splits a product whose epilogue
    needs the whole sum, stays within 9 splits and 4..6 tiles per workgroup (10 only for unsplit products; 4..8 beyond 128 rows),
    and for the 7B shapes picks the plans the design rests on (gate|up: 237 workgroups of 5 = one round on 256 compute
    units; O and QKV: 7 splits of exactly two revolutions of 16 k-steps, the planner's unit; down: 9 splits; LM head: two rounds of 10 tiles)."""
    lib = binding.load()

    def plan(n_tiles, k_steps, batch, partial):
        wn, wk, sp = C.c_int32(), C.c_int32(), C.c_int32()
        assert lib.hx_plan_product(n_tiles, k_steps, batch, int(partial), C.byref(wn), C.byref(wk), C.byref(sp)) == binding.HX_OK
        return wn.value, wk.value, sp.value

    for s in (synth.TINY, synth.QWEN_1P5B, synth.QWEN_7B, synth.QWEN_14B):
        for K, N, partial in ((s.hidden, s.qkv_dim, True), (s.q_dim, s.hidden, True), (s.hidden, 2 * s.intermediate, False),
                              (s.intermediate, s.hidden, True), (s.hidden, s.vocab, False)):
            for batch in (1, 4, 64, 128, 256):
                wn, wk, sp = plan((N + 31) // 32, K // 16, batch, partial)
                if batch <= 128:
                    assert (4 <= wn <= 6 or (wn == 10 and not partial)) and wk == 1 and 1 <= sp <= 9
                else:                                   # the workgroup-tiled product
                    assert 4 <= wn <= 8 and wk == 1 and 1 <= sp <= 9
                assert sp == 1 or (K // 16) // sp >= 16
                assert partial or sp == 1
    # the splits tell the products for few columns from the others: up to 68 tiles, at any number of rows, and beyond 128 rows no three
    # splits of more than 240 k-steps; up to 128 rows the number of rows decides nothing
    for batch in (1, 64, 65, 128):
        assert [plan(n, 160, batch, True)[2] for n in (64, 68, 69)] == [4, 3, 5] and plan(64, 217, batch, True)[2] == 8
    for batch in (129, 256):
        assert plan(64, 1792, batch, True)[2] == 4
        assert plan(65, 720, batch, True)[2] == 3 and plan(65, 721, batch, True)[2] == 9
    s = synth.QWEN_7B
    assert plan(2 * s.intermediate // 32, s.hidden // 16, 128, False) == (5, 1, 1)
    assert plan(s.hidden // 32, s.q_dim // 16, 128, True) == (4, 1, 7)
    assert plan(s.qkv_dim // 32, s.hidden // 16, 128, True) == (4, 1, 7)
    assert plan(s.hidden // 32, s.intermediate // 16, 128, True) == (4, 1, 9)
    assert plan(s.vocab // 32, s.hidden // 16, 128, False) == (10, 1, 1)
    # beyond 128 rows the answer is the plan of the product that runs there, under the same knobs
    assert plan(s.vocab // 32, s.hidden // 16, 256, False) == (7, 1, 1)
    down = (s.hidden // 32, s.intermediate // 16)
    assert plan(*down, 256, True)[2] > 2
    monkeypatch.setenv("HX_GEMM_MAX_SPLITS", "2")
    assert plan(*down, 256, True)[2] <= 2 and plan(*down, 128, True)[2] <= 2
    monkeypatch.delenv("HX_GEMM_MAX_SPLITS")
    monkeypatch.setenv("HX_GEMM_SHAPE", "7,1,3")
    assert plan(*down, 256, True) == (7, 1, 3) and plan(*down, 128, True) == (4, 1, 9)       # 7 tiles: only beyond 128 rows
    monkeypatch.setenv("HX_GEMM_SHAPE", "4,2,2")
    assert plan(*down, 128, True) == (4, 2, 2) and plan(*down, 256, True)[1] == 1            # k-slices: only up to 128
    monkeypatch.delenv("HX_GEMM_SHAPE")
    none = C.c_int32()
    assert lib.hx_plan_product(0, 10, 4, 1, C.byref(none), C.byref(none), C.byref(none)) == binding.HX_E_RANGE
    assert lib.hx_plan_product(10, 10, 300, 1, C.byref(none), C.byref(none), C.byref(none)) == binding.HX_E_RANGE
    assert lib.hx_plan_product(10, 10, 4, 1, None, C.byref(none), C.byref(none)) == binding.HX_E_NULL


def test_a_nucleus_draw_takes_no_workspace_of_its_own():
    """The vocabulary enters the workspace by the LM head's five arrays of one number per row and tile, nothing else: neither an
    engine's nor that of a prompt call, which holds one per 256 rows and never draws."""
    def arrays(vocab, batch):
        return 5 * ((batch * ((vocab + 31) // 32) * 4 + 255) // 256 * 256)
    for shape in (synth.QWEN_1P5B, synth.QWEN_14B):
        for batch in (1, 3, 64, 128, 256):
            small, large = [binding.make_config(dataclasses.replace(shape, vocab=v), batch, 1024) for v in (1024, 152064)]
            more = arrays(152064, batch) - arrays(1024, batch)
            assert binding.workspace_bytes(large) - binding.workspace_bytes(small) == more
            if batch == 256:
                blocks = [binding.prefill_workspace_bytes(c, 256) for c in (small, large)]
                assert abs(blocks[1] - blocks[0] - more) < 4096            # blocks are a multiple of 4096 bytes


def test_the_step_from_few_columns_to_the_streaming_product():
    """68 tiles are the last whose product gets one workgroup per tile and splits of 24 k-steps; 69 take the streaming plan, in
    splits of whole revolutions of 16 (256 compute units: no device is asked here)."""
    lib = binding.load()
    out = [C.c_int32() for _ in range(3)]

    def splits(n_tiles, k_steps, batch=64):
        assert lib.hx_plan_product(n_tiles, k_steps, batch, 1, *[C.byref(o) for o in out]) == binding.HX_OK
        return out[2].value
    for batch in (1, 64, 128):
        assert [splits(t, 48, batch) for t in (64, 65, 68, 69)] == [2, 2, 2, 3]
        assert [splits(t, 128, batch) for t in (68, 69)] == [3, 8]


def test_row_kernels_take_several_blocks_only_beyond_128_rows():
    """The row kernels of at most 128 rows do not look at the block's index: several blocks of so few rows are refused instead of
    the first being written again and again.  Internal launches, over an engine of zeros: nothing is read behind the check."""
    lib = binding.load()
    zeros = C.create_string_buffer(1 << 14)
    e, none, size = C.cast(zeros, C.c_void_p), C.c_void_p(), C.c_size_t

    def launch(name, *args):
        f = getattr(lib, name)
        f.restype = C.c_int
        return f(*args)
    for blocks, rows in ((2, 128), (3, 1)):
        for rc in (launch("_Z20hx_launch_embed_normPK9hx_engineiPKimP12ihipStream_tim", e, rows, none, size(0), none, blocks, size(4096)),
                   launch("_Z21hx_launch_reduce_normPK9hx_engineiPKfimmP12ihipStream_tim", e, rows, none, 1, size(0), size(0), none, blocks,
                          size(4096)),
                   launch("_Z21hx_launch_rope_appendPK9hx_enginePK5hx_kviiPKfimPKiP12ihipStream_tim", e, e, 0, rows, none, 1, size(0), none,
                          none, blocks, size(4096))):
            assert rc == binding.HX_E_RANGE and "blocks of" in lib.hx_last_error().decode()


def test_packing_many_refuses_a_tensor_given_twice():
    """All tensors of a call are written by one launch, in no order.  Refused on the host: the buffers are never touched."""
    lib = binding.load()
    s = synth.TINY
    cfg = binding.make_config(s, 4, 64)
    engine = C.c_void_p()
    at = C.c_void_p(1 << 20)
    assert lib.hx_engine_create(C.byref(cfg), at, binding.weights_bytes(cfg), at, binding.workspace_bytes(cfg), C.byref(engine)) == binding.HX_OK
    try:
        def pack(*kinds):
            n = len(kinds)
            rows = [s.intermediate if k == binding.HX_T_WD else s.hidden for k in kinds]
            cols = [s.hidden if k == binding.HX_T_WD else s.intermediate for k in kinds]
            return lib.hx_weights_pack_many(engine, n, (C.c_int32 * n)(*kinds), 0, (C.c_void_p * n)(*[1 << 20] * n), (C.c_int64 * n)(*rows),
                                            (C.c_int64 * n)(*cols), None)
        assert pack(binding.HX_T_WG, binding.HX_T_WU, binding.HX_T_WG) == binding.HX_E_SHAPE
        assert pack(binding.HX_T_WD, binding.HX_T_WD) == binding.HX_E_SHAPE
        assert lib.hx_weights_pack_many(engine, 0, None, 0, None, None, None, None) == binding.HX_E_NULL
    finally:
        lib.hx_engine_destroy(engine)


@pytest.mark.parametrize("missing", ["_raw_stream", "_raw_device", "not set up"])
def test_the_stream_falls_back_to_the_public_way(monkeypatch, missing):
    """A torch without one of its unpromised functions, or whose GPU is not set up yet, is asked for the current stream."""
    class Stream:
        cuda_stream = 1234

    monkeypatch.setattr(binding, "_raw_device", lambda: 3)
    monkeypatch.setattr(binding, "_raw_stream", lambda device: 100 + device)
    monkeypatch.setattr(binding.torch.cuda, "is_initialized", lambda: missing != "not set up")
    monkeypatch.setattr(binding.torch.cuda, "current_stream", Stream)
    if missing != "not set up":
        assert binding._stream().value == 103
        monkeypatch.setattr(binding, missing, None)
    assert binding._stream().value == 1234
