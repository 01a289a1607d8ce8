"""GPU parity: the HIP path through the C ABI against the CPU oracle, element by element, on the same
seeded inputs.  Tolerances (per output tensor): max|g-o|/max|o| <= 2e-2 for bf16 storage, 1e-4 for fp32,
plus an elementwise rtol/atol gate (helpers.assert_close); cache entries within one storage ulp plus the slack that
the bf16 rounding of the normed row causes (helpers.CACHE_SLACK_BF16, measured in tests/test_cache_gate_model.py);
slots, and everything the call must not touch, bit-exact."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2603_13281_amd import binding, synth
from helpers import assert_cache_close, assert_close, assert_fp8_cache_close, e4m3_spacing, fill_pool, filled_batch, mark_unwritten, oracle_config, read_pool
from gpu_util import bf16_ulp, dev, fp8_pool_to_float, host, make_layer, pool_from_device_layout, pool_to_device_layout

pytestmark = pytest.mark.gpu

TOL = {True: 2e-2, False: 1e-4}
MODES = [0, 1]  # 0: automatic kernel choice, 1: generic vector kernels


def _say(*a):
    print(*a, flush=True)


def _cache_close(shape, got_pool, want_pool, what):
    # pools in the oracle's layout [blocks, 2, Hkv, Bk, D]; K and V are different tensors (with QK-norm K has unit
    # rms per head, V the scale of the weights), so each plane is gated against the rms of its own written entries
    for plane, nm in ((0, "K"), (1, "V")):
        assert_cache_close(got_pool[:, plane], want_pool[:, plane], shape.bf16, f"{what} {nm}")


def _decode_case(shape, ctx, n_active, seed, mode, norm_ones=False):
    base = synth.make_base(shape, seed=seed, norm_ones=norm_ones)
    lora = synth.make_lora(shape, seed=seed)
    batch = synth.make_batch(shape, ctx, n_active, seed=seed)
    pool = filled_batch(shape, batch, seed=seed)
    pool[pool == 0] = -3.0                                   # sentinel in unfilled slots
    x = synth.make_hidden(shape, batch.R, seed=seed)
    orc = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, lora)
    want_pool = pool.copy()
    want, want_slots = orc.decode_step(want_pool, batch.block_tables, batch.ctx_lens, batch.row_seq, batch.row_model, x)

    layer = make_layer(shape, base, lora, batch.num_blocks)
    layer.set_kernel_mode(mode)
    dpool = dev(pool_to_device_layout(pool), shape.bf16)
    bt = torch.from_numpy(batch.block_tables).cuda()
    slots = torch.full((batch.S,), -1, dtype=torch.int64, device="cuda")
    got = layer.decode_step(dpool, bt, batch.ctx_lens, batch.row_seq, batch.row_model, dev(x, shape.bf16), slot_out=slots)
    torch.cuda.synchronize()
    got_pool = pool_from_device_layout(host(dpool), shape.block_size, shape.head_dim)
    return batch, want, want_slots, want_pool, pool, host(got), slots.cpu().numpy(), got_pool


def _check_decode(shape, ctx, n_active, seed, mode, **kw):
    batch, want, want_slots, want_pool, pool0, got, slots, got_pool = _decode_case(shape, ctx, n_active, seed, mode, **kw)
    assert np.array_equal(slots, want_slots)
    # only the appended slots changed, and they match the oracle's entries
    changed = np.argwhere((got_pool != pool0).any(axis=(1, 2, 4)))
    assert sorted(int(b) * shape.block_size + int(o) for b, o in changed) == sorted(int(s) for s in want_slots)
    _cache_close(shape, got_pool, want_pool, "kv cache")
    assert_close(got, want, TOL[shape.bf16], "x_out")


@pytest.mark.parametrize("mode", MODES)
def test_config1_tiny_fp32_prefill_then_decode(mode):
    # Config 1: d 256, 4 heads of 64, FFN 688, M = 2 rank-8 adapters on q/v/o, one sequence, 128-token shared
    # prefix built by the frozen encoder's prefill, then one decode step with both models active.
    _say("case: config 1 tiny fp32, mode", mode)
    shape = synth.TINY
    base = synth.make_base(shape, seed=0)
    lora = synth.make_lora(shape, seed=0)
    batch = synth.make_batch(shape, [128], [2], seed=0)
    orc = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, lora)
    xp = synth.make_hidden(shape, 128, seed=0, tag=1)
    want_pool = orc.new_pool()
    want_y, want_s = orc.prefill(want_pool, batch.block_tables, [0], [128], xp)

    layer = make_layer(shape, base, lora, batch.num_blocks)
    layer.set_kernel_mode(mode)
    dpool = torch.zeros(layer.cfg.pool_shape(), dtype=torch.float32, device="cuda")
    bt = torch.from_numpy(batch.block_tables).cuda()
    slots = torch.zeros(128, dtype=torch.int64, device="cuda")
    got_y = layer.prefill_kv(dpool, bt, [0], [128], dev(xp, False), slot_out=slots)
    torch.cuda.synchronize()
    assert np.array_equal(slots.cpu().numpy(), want_s)
    assert_close(host(got_y), want_y, 1e-4, "prefill x_out")
    _cache_close(shape, pool_from_device_layout(host(dpool), 16, 64), want_pool, "prefill cache")

    x = synth.make_hidden(shape, batch.R, seed=0)
    want, ws = orc.decode_step(want_pool, batch.block_tables, batch.ctx_lens, batch.row_seq, batch.row_model, x)
    s1 = torch.zeros(1, dtype=torch.int64, device="cuda")
    got = layer.decode_step(dpool, bt, batch.ctx_lens, batch.row_seq, batch.row_model, dev(x, False), slot_out=s1)
    torch.cuda.synchronize()
    assert int(s1[0]) == int(ws[0])
    assert_close(host(got), want, 1e-4, "decode x_out")
    _cache_close(shape, pool_from_device_layout(host(dpool), 16, 64), want_pool, "decode cache")


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
def test_decode_ragged_batch(shape, mode):
    # several tiles and ragged tails: lengths around block boundaries, empty context, 0..M active models
    _say("case: ragged decode", shape.name, "mode", mode)
    ctx = [0, 1, 15, 16, 17, 300, 1030, 47]
    M = shape.n_models
    n_active = [1, 0, M, 2, 1, M, min(3, M), 0]
    _check_decode(shape, ctx, n_active, seed=11, mode=mode)


@pytest.mark.parametrize("rows", [100, 129, 230, 300, 385])
def test_decode_row_counts_of_every_gemm_tile(rows):
    # The GEMM launcher picks its tile from the stacked row count: up to 64, up to 128, 193-256 (fused gate/up),
    # up to 384, more.  The other cases of this file stay below 64 rows; these reach the other tiles, each with a
    # ragged last row tile, and the first row count past a boundary (129, 385).  More than 256 rows also take the
    # row and RoPE kernels with one workgroup per row instead of several.
    _say("case: decode with", rows, "stacked rows")
    shape = synth.LLAMA_SMALL
    S = rows // 5
    ctx = [(7 * i) % 45 for i in range(S)]
    n_active = [4] * S
    extra = rows - 5 * S                       # one shorter sequence makes up the exact count
    if extra:
        ctx.append(33)
        n_active.append(extra - 1)
    _check_decode(shape, ctx, n_active, seed=21, mode=MODES[0])


@pytest.mark.parametrize("rows,d_ffn", [(330, 10304), (150, 20608), (131, 20608), (160, 20608), (161, 20608)])
def test_decode_wide_ffn_takes_the_wide_projection_gemm(rows, d_ffn):
    # A fused gate/up projection wide enough for 160 tiles of 192 x 256 goes to the 256 wide tiles
    # (two row tiles of 192 at 330 rows; at most 160 rows: the 160 x 256 tile, partly filled at 131 and 150 rows, full at 160; 161 rows: one 192-row tile again; the last column tile is
    # ragged: d_ffn is not a multiple of 128).  Element by element against the oracle; the down projection then
    # contracts over the same odd width.
    _say("case: wide ffn", rows, "rows, d_ffn", d_ffn)
    # d_model 512: eight 64-wide slabs of base weights, so the kernel's steady-state loop runs as well as its tail
    shape = synth.QWEN_SMALL.replace(d_model=512, n_q_heads=2, n_kv_heads=2, d_ffn=d_ffn)
    S = rows // 4
    ctx = [(5 * i) % 40 for i in range(S)]
    n_active = [3] * S
    extra = rows - 4 * S
    if extra:
        ctx.append(17)
        n_active.append(extra - 1)
    _check_decode(shape, ctx, n_active, seed=23, mode=MODES[0])


@pytest.mark.parametrize("mode", MODES)
def test_decode_long_context_many_models(mode):
    _say("case: long context decode mode", mode)
    shape = synth.LLAMA_SMALL.replace(n_models=8)
    _check_decode(shape, [5000, 2049], [8, 5], seed=5, mode=mode)


def test_config2_llama8b_layer_decode():
    # Config 2 whole: Llama-3-8B-shaped layer, M = 8 rank-16 adapters on all seven projections, one sequence
    # with a 4096-token shared prefix (directly filled), one decode step, all eight models active.
    _say("case: config 2 llama-8b layer")
    _check_decode(synth.LLAMA8B, [4096], [8], seed=0, mode=0, norm_ones=True)


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [synth.TINY, synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
def test_attn_shared_kv(shape, mode):
    _say("case: attention only", shape.name, "mode", mode)
    lens = [1, 16, 33, 700, 2500]
    rows_per_seq = [1, 3, 1 + shape.n_models, 2, 1 + shape.n_models]
    batch = synth.make_batch(shape, lens, [0] * len(lens), seed=3, headroom=0)
    pool = filled_batch(shape, batch, seed=3)
    row_seq = np.repeat(np.arange(len(lens)), rows_per_seq).astype(np.int32)
    R = len(row_seq)
    rng = np.random.default_rng(7)
    q = synth.to_storage(rng.standard_normal((R, shape.n_q_heads, shape.head_dim)).astype(np.float32), shape.bf16)
    orc = oracle.Oracle(oracle_config(shape, batch.num_blocks), synth.make_base(shape), None)
    want = orc.attn_shared_kv(q, pool, batch.block_tables, lens, row_seq)
    layer = make_layer(shape, synth.make_base(shape), None, batch.num_blocks)
    layer.set_kernel_mode(mode)
    dpool = dev(pool_to_device_layout(pool), shape.bf16)
    got = layer.attn_shared_kv(dev(q, shape.bf16), dpool, torch.from_numpy(batch.block_tables).cuda(), lens, row_seq)
    torch.cuda.synchronize()
    assert_close(host(got), want, TOL[shape.bf16], "attention out")
    assert np.array_equal(host(dpool), pool_to_device_layout(pool))     # read-only


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
def test_prefill_chunk_over_paged_prefix_then_decode(shape, mode):
    # Config 4's structure at reduced size: cached prefixes, a chunk appended by the frozen encoder (starting
    # mid-block, spanning blocks), then a decode step by a model that never ran on the sequence: no recompute.
    _say("case: prefill chunk", shape.name, "mode", mode)
    pre = [37, 0, 160]
    chunk = [45, 20, 0]
    base = synth.make_base(shape, seed=2, norm_ones=False)
    lora = synth.make_lora(shape, seed=2)
    batch = synth.make_batch(shape, pre, [1, 2, 1], seed=2, headroom=64)
    pool = filled_batch(shape, batch, seed=2)
    pool[pool == 0] = 5.0
    x = synth.make_hidden(shape, sum(chunk), seed=2, tag=3)
    orc = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, lora)
    want_pool = pool.copy()
    want, want_slots = orc.prefill(want_pool, batch.block_tables, pre, chunk, x)

    layer = make_layer(shape, base, lora, batch.num_blocks)
    layer.set_kernel_mode(mode)
    dpool = dev(pool_to_device_layout(pool), shape.bf16)
    bt = torch.from_numpy(batch.block_tables).cuda()
    slots = torch.zeros(sum(chunk), dtype=torch.int64, device="cuda")
    got = layer.prefill_kv(dpool, bt, pre, chunk, dev(x, shape.bf16), slot_out=slots)
    torch.cuda.synchronize()
    assert np.array_equal(slots.cpu().numpy(), want_slots)
    got_pool = pool_from_device_layout(host(dpool), shape.block_size, shape.head_dim)
    changed = np.argwhere((got_pool != pool).any(axis=(1, 2, 4)))
    assert sorted(int(b) * shape.block_size + int(o) for b, o in changed) == sorted(int(s) for s in want_slots)
    _cache_close(shape, got_pool, want_pool, "prefill cache")
    assert_close(host(got), want, TOL[shape.bf16], "prefill x_out")

    # cache-only prefill writes the same bytes
    dpool2 = dev(pool_to_device_layout(pool), shape.bf16)
    layer.prefill_kv(dpool2, bt, pre, chunk, dev(x, shape.bf16), want_out=False)
    torch.cuda.synchronize()
    assert torch.equal(dpool2, dpool)

    # decode on top of the GPU-written cache, against the oracle on the oracle-written cache
    ctx2 = [p + c for p, c in zip(pre, chunk)]
    b2 = synth.make_batch(shape, ctx2, [1, 2, 1], seed=2, headroom=1)
    xd = synth.make_hidden(shape, b2.R, seed=2, tag=4)
    wd, _ = orc.decode_step(want_pool, batch.block_tables, ctx2, b2.row_seq, b2.row_model, xd)
    gd = layer.decode_step(dpool, bt, ctx2, b2.row_seq, b2.row_model, dev(xd, shape.bf16))
    torch.cuda.synchronize()
    assert_close(host(gd), wd, TOL[shape.bf16], "decode after prefill")


@pytest.mark.parametrize("mode", MODES)
def test_cache_bits_do_not_depend_on_adapters(mode):
    # Sec. 3.2 / 3.3: the cache is written by the frozen encoder alone -> bit-identical on the GPU whatever
    # adapter weights are loaded and whichever models are active; K/V adapters are never read.
    _say("case: adapter independence mode", mode)
    shape = synth.LLAMA_SMALL
    base = synth.make_base(shape, seed=4)
    ctx = [33, 250]
    pools, outs = [], []
    for lora_seed, n_act, scale_kv in ((4, [2, 4], 1.0), (9, [2, 4], 1.0), (4, [0, 1], 1.0), (4, [2, 4], 50.0)):
        lora = synth.make_lora(shape, seed=lora_seed)
        lora["k"] = (lora["k"][0] * scale_kv, lora["k"][1])
        lora["v"] = (lora["v"][0], lora["v"][1] * scale_kv)
        batch = synth.make_batch(shape, ctx, n_act, seed=4)
        pool = filled_batch(shape, batch, seed=4)
        x_seq = synth.make_hidden(shape, 2, seed=4)
        layer = make_layer(shape, base, lora, batch.num_blocks)
        layer.set_kernel_mode(mode)
        dpool = dev(pool_to_device_layout(pool), True)
        y = layer.decode_step(dpool, torch.from_numpy(batch.block_tables).cuda(), ctx, batch.row_seq, batch.row_model,
                              dev(x_seq[batch.row_seq], True))
        torch.cuda.synchronize()
        pools.append(dpool.cpu())
        outs.append(y.cpu())
    assert all(torch.equal(pools[0], p) for p in pools[1:])
    assert torch.equal(outs[0], outs[3])            # K/V adapter perturbation is a no-op on outputs too
    assert not torch.equal(outs[0], outs[1])


@pytest.mark.parametrize("mode", MODES)
def test_zero_B_rows_equal_encoder_row_and_runs_are_deterministic(mode):
    _say("case: zero B, determinism, mode", mode)
    shape = synth.LLAMA_SMALL
    base = synth.make_base(shape, seed=6)
    lora = synth.make_lora(shape, seed=6, zero_b=True)
    batch = synth.make_batch(shape, [129, 64], [4, 2], seed=6)
    pool = filled_batch(shape, batch, seed=6)
    x = synth.make_hidden(shape, 2, seed=6)[batch.row_seq]
    layer = make_layer(shape, base, lora, batch.num_blocks)
    layer.set_kernel_mode(mode)
    bt = torch.from_numpy(batch.block_tables).cuda()
    ys = []
    for _ in range(2):
        dpool = dev(pool_to_device_layout(pool), True)
        ys.append(layer.decode_step(dpool, bt, batch.ctx_lens, batch.row_seq, batch.row_model, dev(x, True)).cpu())
    assert torch.equal(ys[0], ys[1])
    y = ys[0].float().numpy()
    orc = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, lora)
    want, _ = orc.decode_step(pool.copy(), batch.block_tables, batch.ctx_lens, batch.row_seq, batch.row_model, x)
    assert_close(y, want, 2e-2, "zero-B x_out")
    # Sec. 3.2: with B = 0 a decoder is the base model.  On the device too, bit for bit: a row's arithmetic does not
    # depend on its place in a tile, the adapter's K-steps add exact zeros, and equal queries of one sequence see
    # equal scores, so every step of a decoder row repeats the encoder row's.
    for r in range(batch.R):
        enc = int(np.flatnonzero((batch.row_seq == batch.row_seq[r]) & (batch.row_model == -1))[0])
        assert torch.equal(ys[0][r], ys[0][enc]), f"row {r} differs from its sequence's encoder row {enc}"


def test_errors_surface_through_the_binding():
    from paper_2603_13281_amd.binding import IcarusError
    shape = synth.LLAMA_SMALL
    batch = synth.make_batch(shape, [20], [1], seed=0)
    layer = make_layer(shape, synth.make_base(shape), synth.make_lora(shape), batch.num_blocks)
    dpool = torch.zeros(layer.cfg.pool_shape(), dtype=torch.bfloat16, device="cuda")
    bt = torch.from_numpy(batch.block_tables).cuda()
    x = torch.zeros(2, shape.d_model, dtype=torch.bfloat16, device="cuda")
    with pytest.raises(IcarusError) as e:
        layer.decode_step(dpool, bt, [20], [0, 0], [-1, 99], x)
    assert e.value.status_name == "MODEL_ID"
    with pytest.raises(IcarusError) as e:
        layer.decode_step(dpool, bt, [20], [0, 0], [-1, 0], x, workspace=torch.zeros(64, dtype=torch.uint8, device="cuda"))
    assert e.value.status_name == "CAPACITY"
    with pytest.raises(IcarusError) as e:
        layer.decode_step(dpool, bt, [10_000], [0, 0], [-1, 0], x)
    assert e.value.status_name == "CAPACITY"


@pytest.mark.parametrize("chunk", [0, 128, 256])
@pytest.mark.parametrize("g,rows", [(4, 1), (4, 4), (4, 9), (8, 2), (8, 7), (8, 9), (1, 3)])
def test_attn_mfma_tiles_splits_and_tails(g, rows, chunk):
    # matrix-core attention: every query-tile count (1..5 tiles of 16 stacked queries), single-chunk and
    # split sequences, lengths around the 16-token block, 32-token group and 128-token chunk boundaries
    _say("case: mfma attention g", g, "rows", rows, "chunk", chunk)
    shape = synth.LLAMA_SMALL.replace(n_q_heads=2 * g, n_kv_heads=2, d_model=256, n_models=8)
    lens = [1, 15, 16, 17, 31, 32, 33, 127, 128, 129, 255, 257, 1000, 3001]
    rows_per_seq = [rows if i % 3 else max(1, rows - 1) for i in range(len(lens))]
    batch = synth.make_batch(shape, lens, [0] * len(lens), seed=8, headroom=0)
    pool = filled_batch(shape, batch, seed=8)
    mark_unwritten(shape, batch, pool, np.nan)   # unwritten slots hold NaN: masked positions must not leak
    row_seq = np.repeat(np.arange(len(lens)), rows_per_seq).astype(np.int32)
    R = len(row_seq)
    rng = np.random.default_rng(9)
    q = synth.to_storage(rng.standard_normal((R, shape.n_q_heads, shape.head_dim)).astype(np.float32) * 2, True)
    orc = oracle.Oracle(oracle_config(shape, batch.num_blocks), synth.make_base(shape), None)
    want = orc.attn_shared_kv(q, pool, batch.block_tables, lens, row_seq)
    layer = make_layer(shape, synth.make_base(shape), None, batch.num_blocks)
    layer.set_attn_piece_limit(chunk)          # 0: automatic; else sequences longer than this are cut into pieces
    dpool = dev(pool_to_device_layout(pool), True)
    got = layer.attn_shared_kv(dev(q, True), dpool, torch.from_numpy(batch.block_tables).cuda(), lens, row_seq)
    torch.cuda.synchronize()
    assert_close(host(got), want, 2e-2, "attention out")


@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
def test_prefill_causal_groups_and_boundaries(shape):
    # prefill attention on the matrix cores: chunks cut into groups of consecutive tokens with a causal
    # stagger; prefixes and chunk lengths around the 16-token block, 32-token group and group-size boundaries
    _say("case: prefill causal boundaries", shape.name)
    pre = [0, 1, 20, 31, 32, 33, 63, 64, 500, 27]
    chunk = [1, 5, 12, 13, 25, 7, 66, 3, 130, 40]
    base = synth.make_base(shape, seed=13, norm_ones=False)
    batch = synth.make_batch(shape, pre, [0] * len(pre), seed=13, headroom=140)
    pool = filled_batch(shape, batch, seed=13)
    mark_unwritten(shape, batch, pool, np.nan)    # never-written slots hold NaN: masked positions must not leak
    x = synth.make_hidden(shape, sum(chunk), seed=13, tag=5)
    orc = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, None)
    want_pool = pool.copy()
    want, want_slots = orc.prefill(want_pool, batch.block_tables, pre, chunk, x)
    layer = make_layer(shape, base, None, batch.num_blocks)
    dpool = dev(pool_to_device_layout(pool), True)
    bt = torch.from_numpy(batch.block_tables).cuda()
    slots = torch.zeros(sum(chunk), dtype=torch.int64, device="cuda")
    got = layer.prefill_kv(dpool, bt, pre, chunk, dev(x, True), slot_out=slots)
    torch.cuda.synchronize()
    assert np.array_equal(slots.cpu().numpy(), want_slots)
    assert_close(host(got), want, 2e-2, "prefill x_out")
    # generic kernels give the same answer (GPU vs GPU, to tolerance)
    layer.set_kernel_mode(1)
    dpool2 = dev(pool_to_device_layout(pool), True)
    got2 = layer.prefill_kv(dpool2, bt, pre, chunk, dev(x, True))
    torch.cuda.synchronize()
    assert_close(host(got2), want, 2e-2, "prefill x_out (generic kernels)")


@pytest.mark.parametrize("pre,chunk", [([16379, 16384, 40001], [9, 33, 70]),          # around the longest decode piece, and beyond
                                       ([131072 - 20], [20]), ([131072 - 19], [20])],  # the longest context a workgroup's LDS covers, one more
                         ids=["beyond-16384", "longest", "past-longest"])
def test_prefill_over_long_contexts(pre, chunk):
    _say("case: prefill long contexts", pre, chunk)
    shape = synth.LLAMA_SMALL
    base = synth.make_base(shape, seed=17, norm_ones=False)
    batch = synth.make_batch(shape, pre, [0] * len(pre), seed=17, headroom=max(chunk) + 16, pool_factor=1.0)
    pool = filled_batch(shape, batch, seed=17)
    mark_unwritten(shape, batch, pool, np.nan)
    x = synth.make_hidden(shape, sum(chunk), seed=17, tag=5)
    dpool = dev(pool_to_device_layout(pool), True)
    orc = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, None)
    want, want_slots = orc.prefill(pool, batch.block_tables, pre, chunk, x)
    layer = make_layer(shape, base, None, batch.num_blocks, max_position=1 << 18)
    slots = torch.zeros(sum(chunk), dtype=torch.int64, device="cuda")
    got = layer.prefill_kv(dpool, torch.from_numpy(batch.block_tables).cuda(), pre, chunk, dev(x, True), slot_out=slots)
    torch.cuda.synchronize()
    assert np.array_equal(slots.cpu().numpy(), want_slots)
    assert_close(host(got), want, 2e-2, "prefill x_out")


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("limit", [0, 128, 384])
def test_prefill_walks_cut_into_pieces(limit, fp8):
    # the walks of a few token groups are cut into pieces (128-token rounds) and their partial results merged: a part shorter
    # than a round joins the piece before it, so last pieces have 128 to 255 tokens, and with at most 32 rows to a group every
    # query reaches every piece; whole and cut walks in one call; groups that fill one wave or all
    _say("case: prefill pieces, limit", limit, "fp8", fp8)
    shape = synth.QWEN_SMALL                        # g = 8: 32 chunk tokens per group
    pre = [0, 127, 128, 255, 380, 1000, 2303, 5]
    chunk = [129, 2, 128, 1, 133, 40, 33, 31]
    ks, vs = 0.02, 0.013
    base = synth.make_base(shape, seed=19, norm_ones=False)
    batch = synth.make_batch(shape, pre, [0] * len(pre), seed=19, headroom=140)
    x = synth.make_hidden(shape, sum(chunk), seed=19, tag=5)
    cfg = oracle_config(shape, batch.num_blocks)
    if fp8:
        layer = make_layer(shape, base, None, batch.num_blocks, kv_fp8=True, k_scale=ks, v_scale=vs)
        gen = torch.Generator(device="cuda:0")
        gen.manual_seed(19)
        dpool = torch.randint(0, 256, layer.cfg.pool_shape(), generator=gen, device="cuda:0", dtype=torch.uint8)
        dpool[(dpool & 0x7f) == 0x7f] = 0x38        # no NaN codes inside the contexts
        dpool[(dpool & 0x78) == 0x78] &= 0xbf
        pool = pool_from_device_layout(fp8_pool_to_float(dpool, ks, vs), shape.block_size, shape.head_dim)
        cfg = dataclasses.replace(cfg, kv_fp8=True, k_scale=ks, v_scale=vs)
    else:
        layer = make_layer(shape, base, None, batch.num_blocks)
        pool = filled_batch(shape, batch, seed=19)
        mark_unwritten(shape, batch, pool, np.nan)
        dpool = dev(pool_to_device_layout(pool), True)
    want, _ = oracle.Oracle(cfg, base, None).prefill(pool, batch.block_tables, pre, chunk, x)
    layer.set_attn_piece_limit(limit)
    got = layer.prefill_kv(dpool, torch.from_numpy(batch.block_tables).cuda(), pre, chunk, dev(x, True))
    torch.cuda.synchronize()
    assert_close(host(got), want, 2e-2, "prefill x_out")


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
def test_prefill_pieces_that_queries_do_not_reach(fp8):
    # a query head per kv-head: groups of up to 256 rows, and a last piece of 128-255 tokens lies past what the first rows of
    # the group attend to; they leave a maximum of -inf and a sum of 0 there, which the merge must weigh with zero
    _say("case: unreached prefill pieces, fp8", fp8)
    shape = synth.LLAMA_SMALL.replace(n_q_heads=4, n_kv_heads=4)
    pre, chunk = [100, 0, 37, 260], [300, 513, 257, 256]
    ks, vs = 0.02, 0.013
    base = synth.make_base(shape, seed=47, norm_ones=False)
    batch = synth.make_batch(shape, pre, [0] * len(pre), seed=47, headroom=max(chunk))
    x = synth.make_hidden(shape, sum(chunk), seed=47, tag=5)
    cfg = oracle_config(shape, batch.num_blocks)
    kw = dict(kv_fp8=True, k_scale=ks, v_scale=vs) if fp8 else {}
    layer = make_layer(shape, base, None, batch.num_blocks, **kw)
    if fp8:
        gen = torch.Generator(device="cuda:0")
        gen.manual_seed(47)
        dpool = torch.randint(0, 0x70, layer.cfg.pool_shape(), generator=gen, device="cuda:0", dtype=torch.uint8)
        pool = pool_from_device_layout(fp8_pool_to_float(dpool, ks, vs), shape.block_size, shape.head_dim)
        cfg = dataclasses.replace(cfg, **kw)
    else:
        pool = filled_batch(shape, batch, seed=47)
        mark_unwritten(shape, batch, pool, np.nan)
        dpool = dev(pool_to_device_layout(pool), True)
    layer.set_attn_piece_limit(128)
    pieces = layer.prefill_plan(pre, chunk)
    first = {}                                      # tokens the first row of each group attends to
    row = 0
    for c, n in zip(pre, chunk):
        first.update({row + t: c + t + 1 for t in range(0, n, 256)})
        row += n
    assert any(p[2] >= first[int(p[0])] for p in pieces), "no piece that a query does not reach"
    want, _ = oracle.Oracle(cfg, base, None).prefill(pool, batch.block_tables, pre, chunk, x)
    got = layer.prefill_kv(dpool, torch.from_numpy(batch.block_tables).cuda(), pre, chunk, dev(x, True))
    torch.cuda.synchronize()
    assert_close(host(got), want, 2e-2, "prefill x_out")


def test_append_by_tiles_sums_the_slices_of_the_projection():
    # the tiles add up the K slices that the QKV projection leaves; chunks that start inside a block
    _say("case: append tiles over slices")
    shape = synth.QWEN_SMALL.replace(d_model=3072, n_q_heads=48, n_kv_heads=8, d_ffn=512)
    pre, chunk = [5, 30], [230, 100]
    n = [shape.n_q_heads * 128, shape.n_kv_heads * 128, shape.n_kv_heads * 128]
    assert binding.gemm_choice(sum(chunk), shape.d_model, n, max_slices=12, taken=True)[3] == 2
    base = synth.make_base(shape, seed=53, norm_ones=False)
    batch = synth.make_batch(shape, pre, [0, 0], seed=53, headroom=max(chunk))
    layer = make_layer(shape, base, None, batch.num_blocks)
    assert layer.append_in_tiles(sum(chunk), 24)
    pool = filled_batch(shape, batch, seed=53)
    x = synth.make_hidden(shape, sum(chunk), seed=53, tag=5)
    dpool = dev(pool_to_device_layout(pool), True)
    want, want_slots = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, None).prefill(pool, batch.block_tables, pre, chunk, x)
    slots = torch.zeros(sum(chunk), dtype=torch.int64, device="cuda")
    got = layer.prefill_kv(dpool, torch.from_numpy(batch.block_tables).cuda(), pre, chunk, dev(x, True), slot_out=slots)
    torch.cuda.synchronize()
    assert np.array_equal(slots.cpu().numpy(), want_slots)
    _cache_close(shape, pool_from_device_layout(host(dpool), shape.block_size, shape.head_dim), pool, "cache")
    assert_close(host(got), want, 2e-2, "prefill x_out")


@pytest.mark.parametrize("rows", [65, 129, 161, 250, 321, 449, 577, 770, 1100])
@pytest.mark.parametrize("d_ffn", [4096, 8256])
def test_prefill_row_counts_over_the_gemm_tiles(rows, d_ffn):
    # whole prefill layers at row counts one past a tile edge or well inside, a ragged last column tile (8256 outputs), panels
    # that do not divide.  At 1024 columns nearly all projections run in 128 x 128 tiles, sliced and whole, gate/up also in the
    # larger ones; every tile and slice count by itself is in test_gpu_gemm.py
    _say("case: prefill rows", rows, "d_ffn", d_ffn)
    shape = synth.LLAMA_SMALL.replace(d_model=1024, d_ffn=d_ffn)
    base = synth.make_base(shape, seed=23, norm_ones=False)
    pre, chunk = [40, 0], [rows - 20, 20]
    batch = synth.make_batch(shape, pre, [0, 0], seed=23, headroom=max(chunk))
    pool = filled_batch(shape, batch, seed=23)
    x = synth.make_hidden(shape, rows, seed=23, tag=5)
    dpool = dev(pool_to_device_layout(pool), True)
    want, _ = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, None).prefill(pool, batch.block_tables, pre, chunk, x)
    layer = make_layer(shape, base, None, batch.num_blocks)
    got = layer.prefill_kv(dpool, torch.from_numpy(batch.block_tables).cuda(), pre, chunk, dev(x, True))
    torch.cuda.synchronize()
    assert_close(host(got), want, 2e-2, "prefill x_out")
    got_pool = pool_from_device_layout(host(dpool), shape.block_size, shape.head_dim)
    _cache_close(shape, got_pool, pool, "prefill cache")


SKINNY_SHAPES = {
    # whole 16-byte pieces; rows and heads that are not (one element at a time, blocks of 6 tokens); bf16 outside the matrix cores
    "fp32": synth.TINY.replace(n_models=8, lora_target_mask=synth.ALL_TARGETS),
    "fp32-odd": synth.TINY.replace(d_model=90, n_q_heads=6, n_kv_heads=2, head_dim=18, d_ffn=70, lora_rank=3, n_models=8, block_size=6,
                                   lora_target_mask=synth.ALL_TARGETS),
    "fp32-gate-only": synth.TINY.replace(n_models=8, lora_target_mask=0b0010000, n_q_heads=8, n_kv_heads=2, head_dim=32),
    "bf16-d64": synth.LLAMA_SMALL.replace(d_model=256, head_dim=64, d_ffn=200, n_models=8),
    "bf16-up-only": synth.LLAMA_SMALL.replace(d_model=256, head_dim=96, d_ffn=344, n_models=8, lora_target_mask=0b0100001),
}


@pytest.mark.parametrize("shape", list(SKINNY_SHAPES.values()), ids=list(SKINNY_SHAPES))
@pytest.mark.parametrize("ctx,n_active", [([128], [2]), ([0, 37], [0, 3]), ([5, 1023, 1030, 2050], [1, 3, 0, 8]), ([3, 40], [6, 8]), ([70, 11], [8, 7])],
                         ids=["r3", "r5", "r16", "r16b", "r17"])
def test_decode_of_a_few_rows_on_vector_kernels(shape, ctx, n_active):
    _say("case: few rows", shape.name, "d", shape.d_model, "ctx", ctx, "active", n_active)
    _check_decode(shape, ctx, n_active, seed=29, mode=0)


@pytest.mark.parametrize("shape", list(SKINNY_SHAPES.values()), ids=list(SKINNY_SHAPES))
def test_prefill_of_a_few_rows_on_vector_kernels(shape):
    _say("case: few rows prefill", shape.name)
    base = synth.make_base(shape, seed=31, norm_ones=False)
    pre, chunk = [33, 0], [6, 9]
    batch = synth.make_batch(shape, pre, [0, 0], seed=31, headroom=16)
    pool = filled_batch(shape, batch, seed=31)
    mark_unwritten(shape, batch, pool, np.nan)
    x = synth.make_hidden(shape, sum(chunk), seed=31, tag=5)
    dpool, dpool2 = (dev(pool_to_device_layout(pool), shape.bf16) for _ in range(2))
    want, _ = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, None).prefill(pool, batch.block_tables, pre, chunk, x)
    layer = make_layer(shape, base, None, batch.num_blocks)
    bt = torch.from_numpy(batch.block_tables).cuda()
    got = layer.prefill_kv(dpool, bt, pre, chunk, dev(x, shape.bf16))
    layer.prefill_kv(dpool2, bt, pre, chunk, dev(x, shape.bf16), want_out=False)   # cache only: the same bytes
    torch.cuda.synchronize()
    assert_close(host(got), want, TOL[shape.bf16], "prefill x_out")
    assert np.array_equal(host(dpool).view(np.uint32), host(dpool2).view(np.uint32))


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
def test_cache_entries_do_not_depend_on_the_append_path(shape, fp8):
    # the same chunks in one call (appended by tiles) and in calls of too few rows for tiles leave the same bytes;
    # K = 256 keeps the projections in one slice, so each row's products are summed in the same order in all calls
    _say("case: append paths agree", shape.name, "fp8", fp8)
    shape = shape.replace(d_model=256)
    heads = shape.n_q_heads + 2 * shape.n_kv_heads
    pre, chunk = [0, 3, 21], [-(-20480 // heads) - 250, 201, 60]
    base = synth.make_base(shape, seed=43, norm_ones=False)
    batch = synth.make_batch(shape, pre, [0] * len(pre), seed=43, headroom=max(chunk))
    layer = make_layer(shape, base, None, batch.num_blocks, **(dict(kv_fp8=True, k_scale=0.02, v_scale=0.013) if fp8 else {}))
    x = dev(synth.make_hidden(shape, sum(chunk), seed=43, tag=5), True)
    pools = [torch.zeros(layer.cfg.pool_shape(), dtype=layer.cfg.pool_dtype, device="cuda:0") for _ in range(2)]
    bt = torch.from_numpy(batch.block_tables).cuda()
    whole = layer.prefill_kv(pools[0], bt, pre, chunk, x)
    row = 0
    for s, n in enumerate(chunk):
        for t in range(0, n, 320):
            m = min(320, n - t)
            layer.prefill_kv(pools[1], bt[s:s + 1].clone(), [pre[s] + t], [m], x[row + t:row + t + m].clone())
        row += n
    torch.cuda.synchronize()
    assert torch.isfinite(whole).all()
    assert torch.equal(pools[0].view(torch.uint8), pools[1].view(torch.uint8))


@pytest.mark.parametrize("tiles", [False, True], ids=["rows", "tiles"])
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
def test_prefill_appends_by_block_tiles(shape, fp8, tiles):
    # chunk rows appended one by one or, from 20480 (row, head) pairs on, in tiles that lie within one block: a single
    # token anywhere in it, whole blocks, the end of one and the start of the next; every slot right, every other byte of
    # the pool as it was, also in a cache-only call
    _say("case: append tiles", shape.name, "fp8", fp8, "tiles", tiles)
    pre = [0, 1, 15, 16, 17, 31, 5, 64]
    chunk = [1, 15, 17, 16, 33, 1, 40, 3]
    if tiles:
        more = -(-20480 // (shape.n_q_heads + 2 * shape.n_kv_heads)) - sum(chunk)  # the least that takes the tiles
        pre, chunk = pre + [3, 0, 30, 8], chunk + [more // 4] * 3 + [more - more // 4 * 3]
    ks, vs = 0.02, 0.013
    base = synth.make_base(shape, seed=37, norm_ones=False)
    batch = synth.make_batch(shape, pre, [0] * len(pre), seed=37, headroom=max(chunk))
    kw = dict(kv_fp8=True, k_scale=ks, v_scale=vs) if fp8 else {}
    layer = make_layer(shape, base, None, batch.num_blocks, **kw)
    x = synth.make_hidden(shape, sum(chunk), seed=37, tag=5)
    pool = filled_batch(shape, batch, seed=37)
    cfg = oracle_config(shape, batch.num_blocks)
    if fp8:
        cfg = dataclasses.replace(cfg, **kw)
        gen = torch.Generator(device="cuda:0")
        gen.manual_seed(37)
        dpool = torch.randint(0, 0x70, layer.cfg.pool_shape(), generator=gen, device="cuda:0", dtype=torch.uint8)
        pool = pool_from_device_layout(fp8_pool_to_float(dpool, ks, vs), shape.block_size, shape.head_dim)
    else:
        dpool = dev(pool_to_device_layout(pool), True)
    before, cache_only = dpool.clone(), dpool.clone()
    orc = oracle.Oracle(cfg, base, None)
    want_pool = pool.copy()
    _, want_slots = orc.prefill(want_pool, batch.block_tables, pre, chunk, x)
    bt = torch.from_numpy(batch.block_tables).cuda()
    slots = torch.zeros(sum(chunk), dtype=torch.int64, device="cuda")
    layer.prefill_kv(dpool, bt, pre, chunk, dev(x, True), slot_out=slots)
    layer.prefill_kv(cache_only, bt, pre, chunk, dev(x, True), want_out=False)
    torch.cuda.synchronize()
    assert np.array_equal(slots.cpu().numpy(), want_slots)
    assert torch.equal(dpool, cache_only)
    if fp8:
        got = pool_from_device_layout(fp8_pool_to_float(dpool, ks, vs), shape.block_size, shape.head_dim)
        was = pool_from_device_layout(fp8_pool_to_float(before, ks, vs), shape.block_size, shape.head_dim)
        if tiles:
            # the same call into a bf16 cache rounds the same fp32 K and V: half a grid step here, 2^-8 of the value there
            # (which the bf16 case compares with the oracle)
            plain = make_layer(shape, base, None, batch.num_blocks)
            bpool = dev(pool_to_device_layout(pool), True)
            plain.prefill_kv(bpool, bt, pre, chunk, dev(x, True), want_out=False)
            same = pool_from_device_layout(host(bpool), shape.block_size, shape.head_dim).astype(np.float64)
            written = np.unique(want_slots)
            at = lambda a, plane: a[written // shape.block_size, plane, :, written % shape.block_size].astype(np.float64)
            for plane, scale in ((0, ks), (1, vs)):
                g, b = at(got, plane), np.clip(at(same, plane), -448 * scale, 448 * scale)
                step = e4m3_spacing(np.maximum(np.abs(g), np.abs(b)), scale)
                assert (np.abs(g - b) <= 0.501 * step + 2.0 ** -8 * np.abs(b)).all(), "fp8 cache against the bf16 cache"
        else:
            for plane, scale in ((0, ks), (1, vs)):
                assert_fp8_cache_close(got[:, plane], want_pool[:, plane], scale, True, "cache")
    else:
        got, was = (pool_from_device_layout(host(t), shape.block_size, shape.head_dim) for t in (dpool, before))
        _cache_close(shape, got, want_pool, "cache")
    changed = np.argwhere((got != was).any(axis=(1, 2, 4)))
    assert sorted(int(b) * shape.block_size + int(o) for b, o in changed) == sorted(int(s) for s in want_slots)
