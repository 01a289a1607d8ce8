"""Prefill calls whose QKV projection rotates, normalises and appends in its epilogue, against the same rows in calls of up to 128, which
leave the projections in memory for the append kernels."""
import numpy as np
import pytest
import torch

from gpu_util import dev, fp8_pool_to_float, host, make_layer
from paper_2603_13281_amd import binding, synth

pytestmark = pytest.mark.gpu

SHAPES = {"plain": synth.LLAMA8B.replace(d_ffn=512), "norms": synth.QWEN32B.replace(d_ffn=512),
          "ungrouped": synth.LLAMA8B.replace(d_model=512, n_q_heads=16, n_kv_heads=16, d_ffn=512)}
# rows -> the projection's tile; chunks whose rows begin and end anywhere in a block of 16 tokens, in a tile and in a group of 32 rows.  192 x 128: full
# tiles of up to 256 workgroups (eight waves) and of more (four), and tiles of 160 rows (four)
CASES = [("plain", 500, (128, 128)), ("norms", 300, (128, 128)), ("plain", 700, (192, 128)), ("plain", 780, (192, 128)), ("plain", 1003, (160, 256)), ("plain", 1701, (192, 256)), ("plain", 2011, (256, 256)),
         ("norms", 400, (192, 128)), ("norms", 601, (160, 256)), ("norms", 1001, (192, 256)), ("norms", 1203, (256, 256)), ("ungrouped", 2700, (192, 128))]


def _bits(pool, layer):
    return fp8_pool_to_float(pool, layer.cfg.k_scale, layer.cfg.v_scale) if layer.cfg.kv_fp8 else pool.float().cpu().numpy()


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("kind,rows,tile", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_projection_that_appends(kind, rows, tile, fp8):
    print("case: fused append", kind, rows, tile, "fp8", fp8, flush=True)
    shape = SHAPES[kind]
    d, kvd = shape.d_model, shape.n_kv_heads * 128
    assert binding.gemm_choice(rows, d, [shape.n_q_heads * 128, kvd, kvd], taken=True) == (*tile, tile[1] == 256 and tile[0] < 256, 1)
    chunk = [1, 15, 16, 9, 0, 33]
    chunk = np.int32(chunk + [rows - sum(chunk)])
    ctx = np.int32([0, 7, 16, 31, 5, 3, 13])
    base = synth.make_base(shape, seed=4, norm_ones=False)
    batch = synth.make_batch(shape, list(ctx), [0] * len(ctx), seed=4, headroom=int(chunk.max()))
    layer = make_layer(shape, base, None, batch.num_blocks, **(dict(kv_fp8=True, k_scale=0.02, v_scale=0.02) if fp8 else {}))
    gen = torch.Generator(device="cuda").manual_seed(4)
    pool = torch.randn(layer.cfg.pool_shape(), generator=gen, device="cuda").clamp(-4, 4)
    pool = (pool / 0.02).to(torch.float8_e4m3fn).view(torch.uint8) if fp8 else pool.to(torch.bfloat16)
    bt = torch.from_numpy(batch.block_tables).cuda()
    x = dev(synth.make_hidden(shape, rows, seed=4, tag=5), True)
    fused, slots = pool.clone(), torch.full((rows,), -1, dtype=torch.int64, device="cuda")
    got = host(layer.prefill_kv(fused, bt, ctx, chunk, x, slot_out=slots))
    parts, want, want_slots, row = pool.clone(), [], [], 0
    for s, n in enumerate(chunk):
        for t in range(0, int(n), 128):
            m = min(128, int(n) - t)
            at = torch.empty(m, dtype=torch.int64, device="cuda")
            want.append(layer.prefill_kv(parts, bt[s:s + 1].clone(), ctx[s:s + 1] + np.int32(t), np.int32([m]), x[row + t:row + t + m], slot_out=at))
            want_slots.append(at)
        row += int(n)
    torch.cuda.synchronize()
    assert torch.equal(slots, torch.cat(want_slots))
    # the products are summed in another order: some entries round to the neighbouring value, 2^-8 (FP8: 2^-3) of their own size apart
    a, b = _bits(fused, layer), _bits(parts, layer)
    off = a != b
    assert off.mean() < (2e-3 if fp8 else 0.05)
    assert (np.abs(a - b)[off] <= (0.13 if fp8 else 0.008) * np.abs(b)[off] + 0.02 * 2.0 ** -8).all()
    untouched = np.ones(a.shape[0], bool)
    untouched[np.unique(slots.cpu().numpy() // shape.block_size)] = False
    assert not off[untouched].any()
    want = host(torch.cat(want))
    assert np.linalg.norm(got - want) <= 1e-2 * np.linalg.norm(want)


@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
def test_entries_of_one_call_that_append_to_one_block(fp8):
    """Token 8 and tokens 12-15 of one block from two entries of the call with another conversation's three rows between them: eight rows,
    of which the first and the last alone are where eight tokens in line would be."""
    print("case: fused append, shared block", "fp8", fp8, flush=True)
    shape = SHAPES["plain"]
    chunk, ctx = np.int32([1, 3, 4, 492]), np.int32([8, 5, 12, 0])
    rows = int(chunk.sum())
    kvd = shape.n_kv_heads * 128
    assert binding.gemm_choice(rows, shape.d_model, [shape.n_q_heads * 128, kvd, kvd], taken=True) == (128, 128, False, 1)
    base = synth.make_base(shape, seed=4, norm_ones=False)
    batch = synth.make_batch(shape, list(ctx), [0] * len(ctx), seed=4, headroom=int(chunk.max()))
    layer = make_layer(shape, base, None, batch.num_blocks, **(dict(kv_fp8=True, k_scale=0.02, v_scale=0.02) if fp8 else {}))
    tables = batch.block_tables.copy()
    tables[2] = tables[0]
    bt = torch.from_numpy(tables).cuda()
    pool = torch.zeros(layer.cfg.pool_shape(), dtype=layer.cfg.pool_dtype, device="cuda")
    x = dev(synth.make_hidden(shape, rows, seed=4, tag=5), True)
    fused, parts, row = pool.clone(), pool.clone(), 0
    layer.prefill_kv(fused, bt, ctx, chunk, x)
    for s, n in enumerate(chunk):
        for t in range(0, int(n), 128):
            m = min(128, int(n) - t)
            layer.prefill_kv(parts, bt[s:s + 1].clone(), ctx[s:s + 1] + np.int32(t), np.int32([m]), x[row + t:row + t + m])
        row += int(n)
    torch.cuda.synchronize()
    a, b = _bits(fused, layer), _bits(parts, layer)
    # the products are summed in another order: some entries round to the neighbouring value, 2^-8 (FP8: 2^-3) of their own size apart
    assert (np.abs(a - b) <= (0.13 if fp8 else 0.008) * np.abs(b) + 0.02 * 2.0 ** -8).all()
