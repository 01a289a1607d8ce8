"""The vector attention kernel at its edges: positions around a quad, a block and a chunk of 1024, head sizes and block sizes that are
whole quads and not, workgroups of 256 and of 1024 threads."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, fp8_pool_to_float, host, make_layer, pool_from_device_layout, pool_to_device_layout
from helpers import filled_batch, mark_unwritten, oracle_config
from paper_2603_13281_amd import synth

pytestmark = pytest.mark.gpu

LENS = [1, 3, 4, 5, 15, 16, 17, 255, 256, 258, 1023, 1024, 1025, 1028, 2051]


@pytest.mark.parametrize("rows", [1, 6], ids=["wide", "narrow"])       # 60 and 360 workgroups
@pytest.mark.parametrize("D,Bk", [(64, 16), (64, 8), (40, 4), (256, 16), (4, 16), (64, 6), (30, 16)])
def test_edges(D, Bk, rows):
    print("case: vector attention, head size", D, "block size", Bk, "rows", rows, flush=True)
    shape = synth.TINY.replace(head_dim=D, block_size=Bk, d_model=4 * D, n_kv_heads=2)
    batch = synth.make_batch(shape, LENS, [0] * len(LENS), seed=8, headroom=0)
    pool = filled_batch(shape, batch, seed=8)
    mark_unwritten(shape, batch, pool, np.nan)                         # positions past the context must not leak
    row_seq = np.repeat(np.arange(len(LENS)), rows).astype(np.int32)
    q = np.random.default_rng(9).standard_normal((len(row_seq), shape.n_q_heads, D)).astype(np.float32)
    base = synth.make_base(shape)
    want = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, None).attn_shared_kv(q, pool, batch.block_tables, LENS, row_seq)
    layer = make_layer(shape, base, None, batch.num_blocks)
    got = layer.attn_shared_kv(dev(q, False), dev(pool_to_device_layout(pool), False), torch.from_numpy(batch.block_tables).cuda(), LENS, row_seq)
    torch.cuda.synchronize()
    # a score is D products of about one over sqrt(D): off by at most D 2^-24 sqrt(D) <= 2.5e-4 for D = 256 and in practice by the
    # root of that count; a probability by as much and its own rounding, an output by that times the largest value
    assert np.abs(host(got) - want).max() <= 5e-5 * np.abs(pool[np.isfinite(pool)]).max()


@pytest.mark.parametrize("rows", [1, 6], ids=["wide", "narrow"])
@pytest.mark.parametrize("bf16,fp8", [(True, False), (True, True), (False, True)], ids=["bf16", "bf16-fp8", "fp32-fp8"])
@pytest.mark.parametrize("D,Bk", [(64, 16), (80, 8), (40, 4), (32, 16), (28, 8), (8, 16), (30, 6)])
def test_edges_of_the_narrow_types(D, Bk, bf16, fp8, rows):
    print("case: vector attention, head size", D, "block size", Bk, "rows", rows, "bf16", bf16, "fp8", fp8, flush=True)
    shape = synth.TINY.replace(head_dim=D, block_size=Bk, d_model=4 * D, n_kv_heads=2, bf16=bf16)
    batch = synth.make_batch(shape, LENS, [0] * len(LENS), seed=8, headroom=0)
    pool = filled_batch(shape, batch, seed=8)
    kw = dict(kv_fp8=True, k_scale=0.02, v_scale=0.01) if fp8 else {}
    if fp8:
        mark_unwritten(shape, batch, pool, 0.0)
        dpool = torch.from_numpy(pool_to_device_layout(pool))
        dpool[:, :, 0] /= kw["k_scale"]
        dpool[:, :, 1] /= kw["v_scale"]
        dpool = dpool.clamp(-448.0, 448.0).to(torch.float8_e4m3fn).view(torch.uint8).cuda()
        pool = pool_from_device_layout(fp8_pool_to_float(dpool, kw["k_scale"], kw["v_scale"]), Bk, D)
    else:
        mark_unwritten(shape, batch, pool, np.nan)
        dpool = dev(pool_to_device_layout(pool), True)
    row_seq = np.repeat(np.arange(len(LENS)), rows).astype(np.int32)
    q = synth.to_storage(np.random.default_rng(9).standard_normal((len(row_seq), shape.n_q_heads, D)), bf16)
    base = synth.make_base(shape)
    cfg = dataclasses.replace(oracle_config(shape, batch.num_blocks), **kw)
    want = oracle.Oracle(cfg, base, None).attn_shared_kv(q, pool, batch.block_tables, LENS, row_seq)
    layer = make_layer(shape, base, None, batch.num_blocks, **kw)
    got = layer.attn_shared_kv(dev(q, bf16), dpool, torch.from_numpy(batch.block_tables).cuda(), LENS, row_seq)
    torch.cuda.synchronize()
    # as above, and with bf16 storage each side's output rounded to it, 2^-9
    bound = 5e-5 * np.abs(pool[np.isfinite(pool)]).max() + (2.0 ** -8 * np.abs(want) if bf16 else 0.0)
    assert (np.abs(host(got) - want) <= bound).all()
