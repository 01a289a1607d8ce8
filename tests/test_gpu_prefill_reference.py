"""The softmax reference of the prefill walk: scores that leave it by hundreds of powers of two, upwards (the reference moves)
and downwards (they vanish), at every place of a 32-token group, a round of four and a piece; and the same bits from both prefill kernels."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, fp8_pool_to_float, host, make_layer, pool_from_device_layout, pool_to_device_layout
from helpers import filled_batch, mark_unwritten, oracle_config
from paper_2603_13281_amd import synth

pytestmark = pytest.mark.gpu

PRE = [32, 64, 95, 127, 128, 129, 300, 513, 11000]
CHUNK = [1, 16, 33, 64, 65, 70, 5, 40, 9]


def _pool(shape, batch, kind, reach, pre=PRE):
    """Cached tokens whose keys are one direction u times a factor that runs from -reach to reach: a query's scores rise or fall
    by up to a few hundred, as its product with u is positive or negative.  Values differ between the two halves only, so that
    the output does not hang on the last bits of such scores."""
    rng = np.random.default_rng(5)
    D, Bk = shape.head_dim, shape.block_size
    u = rng.choice([-1.0, 1.0], size=(shape.n_kv_heads, D)) / np.sqrt(D)
    values = rng.normal(size=(2, shape.n_kv_heads, D))
    pool = np.zeros((batch.num_blocks, 2, shape.n_kv_heads, Bk, D), dtype=np.float32)
    for s, n in enumerate(pre):
        for p in range(n):
            second = p >= (n + 1) // 2
            c = (2.0 * p / (n - 1) - 1.0) if kind == "slope" else (1.0 if second else -1.0)
            blk, off = batch.block_tables[s, p // Bk], p % Bk
            pool[blk, 0, :, off] = reach * c * u
            pool[blk, 1, :, off] = values[int(second)]
    return torch.from_numpy(pool).to(torch.bfloat16).float().numpy()


@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("kind", ["slope", "step"])
@pytest.mark.parametrize("limit", [0, 128, 5504, 16384])  # 5504: pieces, 16384: whole walks, by the kernel for long pieces (more than 5120 tokens)
def test_scores_far_from_the_reference(shape, fp8, kind, limit):
    print("case: far scores", shape.name, "fp8", fp8, kind, "pieces", limit, flush=True)
    base = synth.make_base(shape, seed=3, norm_ones=False)
    batch = synth.make_batch(shape, PRE, [0] * len(PRE), seed=3, headroom=max(CHUNK))
    pool = _pool(shape, batch, kind, 1000.0)
    kw = dict(kv_fp8=True, k_scale=1.0, v_scale=0.02) if fp8 else {}
    layer = make_layer(shape, base, None, batch.num_blocks, **kw)
    if fp8:
        dpool = torch.from_numpy(pool_to_device_layout(pool))
        dpool[:, :, 1] /= kw["v_scale"]
        dpool = dpool.to(torch.float8_e4m3fn).view(torch.uint8).cuda()
        pool = pool_from_device_layout(fp8_pool_to_float(dpool, kw["k_scale"], kw["v_scale"]), shape.block_size, shape.head_dim)
    else:
        dpool = dev(pool_to_device_layout(pool), True)
    x = synth.make_hidden(shape, sum(CHUNK), seed=3, tag=5)
    cfg = dataclasses.replace(oracle_config(shape, batch.num_blocks), **kw)
    want, _ = oracle.Oracle(cfg, base, None).prefill(pool, batch.block_tables, PRE, CHUNK, x)
    layer.set_attn_piece_limit(limit)
    got = layer.prefill_kv(dpool, torch.from_numpy(batch.block_tables).cuda(), PRE, CHUNK, dev(x, True))
    torch.cuda.synchronize()
    got = host(got)
    assert np.isfinite(got).all()
    # in the 2-norm: q is rounded to bf16, 2^-9 of a score, and of scores in the hundreds the few queries nearly at right angles to
    # u weigh both halves, by a ratio that this rounding moves by tenths (the vector kernel, on the same rounded q: 0.004-0.008)
    assert np.sqrt(((got - want) ** 2).sum() / (want ** 2).sum()) <= 2e-2


# ---- attention by itself: O is the identity, the MLP adds nothing, the residual is small ------------------------------------------------
def _bare(shape):
    shape = shape.replace(d_model=shape.n_q_heads * shape.head_dim)
    base = synth.make_base(shape, seed=3, norm_ones=False)
    base["o"], base["down"] = np.eye(shape.d_model, dtype=np.float32), np.zeros_like(base["down"])
    return shape, base


@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
@pytest.mark.parametrize("kind", ["normal", "slope", "step"])
@pytest.mark.parametrize("longest", [470, 1200])
def test_both_prefill_kernels_give_the_same_bits(shape, kind, longest):
    # Walks of up to 5120 tokens go to the kernel for short pieces, unless a longer one is in the call: the same chunks
    # with another chunk beside them, over 100 tokens and over 6004.
    print("case: same bits", shape.name, kind, longest, flush=True)
    pre, chunk = [min(n, longest) for n in PRE[:-1]] + [longest], CHUNK + [3]
    shape, base = _bare(shape)
    x = synth.make_hidden(shape, sum(chunk), seed=3, tag=5) / 16
    out = []
    for last in (100, 6004):
        batch = synth.make_batch(shape, pre + [last], [0] * len(chunk), seed=3, headroom=max(chunk))
        pool = filled_batch(shape, batch, seed=3) if kind == "normal" else _pool(shape, batch, kind, 1000.0, pre)
        mark_unwritten(shape, batch, pool, np.nan)                     # positions past the context must not leak
        layer = make_layer(shape, base, None, batch.num_blocks)
        layer.set_attn_piece_limit(8192)
        out.append(layer.prefill_kv(dev(pool_to_device_layout(pool), True), torch.from_numpy(batch.block_tables).cuda(), pre + [last], chunk, dev(x, True)))
    torch.cuda.synchronize()
    n = sum(CHUNK)
    assert torch.isfinite(out[0]).all() and torch.equal(out[0][:n], out[1][:n])


@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
@pytest.mark.parametrize("kind", ["slope", "step"])
@pytest.mark.parametrize("limit", [128, 5504, 16384])
def test_every_query_far_from_the_reference(shape, fp8, kind, limit):
    print("case: far scores by query", shape.name, "fp8", fp8, kind, "pieces", limit, flush=True)
    shape, base = _bare(shape)
    batch = synth.make_batch(shape, PRE, [0] * len(PRE), seed=3, headroom=max(CHUNK))
    pool = _pool(shape, batch, kind, 1000.0)
    kw = dict(kv_fp8=True, k_scale=4.0, v_scale=0.02) if fp8 else {}
    layer = make_layer(shape, base, None, batch.num_blocks, **kw)
    if fp8:
        dpool = torch.from_numpy(pool_to_device_layout(pool))
        dpool[:, :, 0] /= kw["k_scale"]
        dpool[:, :, 1] /= kw["v_scale"]
        dpool = dpool.to(torch.float8_e4m3fn).view(torch.uint8).cuda()
        pool = pool_from_device_layout(fp8_pool_to_float(dpool, kw["k_scale"], kw["v_scale"]), shape.block_size, shape.head_dim)
    else:
        dpool = dev(pool_to_device_layout(pool), True)
    x = synth.make_hidden(shape, sum(CHUNK), seed=3, tag=5) / 16
    cfg = dataclasses.replace(oracle_config(shape, batch.num_blocks), **kw)
    want, _ = oracle.Oracle(cfg, base, None).prefill(pool.copy(), batch.block_tables, PRE, CHUNK, x)
    layer.set_attn_piece_limit(limit)
    got = layer.prefill_kv(dpool, torch.from_numpy(batch.block_tables).cuda(), PRE, CHUNK, dev(x, True))
    torch.cuda.synchronize()
    heads = (len(x), shape.n_q_heads, shape.head_dim)
    got, want, attn = host(got).reshape(heads), want.reshape(heads), (want - x).reshape(heads)
    # A query whose weights lie on one half but for 2^-8: its attention is that half's values, whatever the last bits of its scores are.
    g = shape.n_q_heads // shape.n_kv_heads
    decided = np.zeros(heads[:2], dtype=bool)
    row = 0
    for s, n in enumerate(CHUNK):
        for p in (0, PRE[s] - 1):
            v = pool[batch.block_tables[s, p // shape.block_size], 1, :, p % shape.block_size]          # [Hkv, D]
            decided[row:row + n] |= np.abs(attn[row:row + n] - np.repeat(v, g, 0)[None]).max(-1) <= 2.0 ** -8 * np.abs(v).max()
        row += n
    assert decided.mean() >= 0.75 and decided.any(1).all()
    # that rest, whose share the rounding of q may double, and probabilities, attention and (both sides) residual sum rounded to bf16
    bound = 2.0 ** -7 * np.abs(attn).max(-1, keepdims=True) + 2.0 ** -8 * np.abs(want)
    assert (np.abs(got - want) <= bound)[decided].all(), np.argwhere(~(np.abs(got - want) <= bound).all(-1) & decided)[:8]


@pytest.mark.parametrize("ctx,chunk", [([2531, 3671], [841, 802]), ([316, 3859, 3623, 1796], [463, 642, 800, 805])], ids=["two", "four"])
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
def test_walks_cut_with_remainders(ctx, chunk, fp8):
    """A plan of equal parts and remainders against whole walks of the same calls."""
    print("case: remainders", ctx, chunk, "fp8", fp8, flush=True)
    shape = synth.LLAMA_SMALL
    base = synth.make_base(shape, seed=3, norm_ones=False)
    batch = synth.make_batch(shape, ctx, [0] * len(ctx), seed=3, headroom=max(chunk))
    layer = make_layer(shape, base, None, batch.num_blocks, **(dict(kv_fp8=True, k_scale=0.02, v_scale=0.02) if fp8 else {}))
    pool = torch.randn(layer.cfg.pool_shape(), generator=torch.Generator().manual_seed(1)).clamp(-4, 4)
    pool = (pool / 0.02).to(torch.float8_e4m3fn).view(torch.uint8).cuda() if fp8 else pool.to(torch.bfloat16).cuda()
    pieces = layer.prefill_plan(ctx, chunk)
    assert (np.diff(pieces[:, 3][pieces[:, 4] >= 0]) < 0).sum() > 3  # remainders of several lengths
    x = dev(synth.make_hidden(shape, sum(chunk), seed=3, tag=5), True)
    bt = torch.from_numpy(batch.block_tables).cuda()
    out = []
    for limit in (0, 16384):
        layer.set_attn_piece_limit(limit)
        p = pool.clone()
        out.append((host(layer.prefill_kv(p, bt, ctx, chunk, x)), p))
    torch.cuda.synchronize()
    (a, pa), (b, pb) = out
    assert torch.equal(pa, pb)
    # attention outputs that differ in the last bit of float32 sums round to neighbouring bf16 values, half of 2^-8 apart at most
    assert np.linalg.norm(a - b) <= 2 ** -8 * np.linalg.norm(b)
