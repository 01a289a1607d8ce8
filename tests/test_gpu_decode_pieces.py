"""The decode attention's walk from piece to piece: shares of several pieces of several sequences, pieces that leave some of a
workgroup's waves without a group, partial last groups, one to three query tiles mixed within a share."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from paper_2603_13281_amd import synth
from helpers import assert_close, filled_batch, mark_unwritten, oracle_config
from gpu_util import dev, fp8_pool_to_float, host, make_layer, pool_from_device_layout, pool_to_device_layout

pytestmark = pytest.mark.gpu

LENS = np.int32([1, 31, 32, 33, 127, 128, 129, 159, 160, 161, 255, 257, 290, 16, 48, 640])


@pytest.mark.parametrize("limit", [32, 64, 96, 128, 160, 288, 0])
@pytest.mark.parametrize("most", [4, 8, 12])        # rows of the fullest sequence: 1, 2 and 3 tiles of 4 heads a row
@pytest.mark.parametrize("fp8", [False, True], ids=["bf16", "fp8"])
def test_walk_from_piece_to_piece(fp8, most, limit):
    rng = np.random.default_rng([17, most, limit])
    shape = synth.LLAMA_SMALL.replace(n_q_heads=8, n_kv_heads=2, d_model=256, n_models=8)
    lens = rng.permutation(LENS)
    rows = [int(rng.integers(1, most + 1)) for _ in lens]
    rows[int(rng.integers(len(rows)))] = most
    print("case: pieces", fp8, most, limit, lens.tolist(), rows, flush=True)
    base = synth.make_base(shape)
    batch = synth.make_batch(shape, lens.tolist(), [0] * len(lens), seed=7, headroom=0)
    row_seq = np.repeat(np.arange(len(lens)), rows).astype(np.int32)
    q = synth.to_storage(rng.standard_normal((len(row_seq), shape.n_q_heads, shape.head_dim)).astype(np.float32), True)
    cfg, scales = oracle_config(shape, batch.num_blocks), {}
    if fp8:
        scales = dict(kv_fp8=True, k_scale=0.02, v_scale=0.013)
        cfg = dataclasses.replace(cfg, **scales)
    layer = make_layer(shape, base, None, batch.num_blocks, **scales)
    if fp8:
        gen = torch.Generator(device="cuda:0").manual_seed(3)
        dpool = torch.randint(0, 256, layer.cfg.pool_shape(), generator=gen, device="cuda:0", dtype=torch.uint8)
        dpool[(dpool & 0x7f) == 0x7f] = 0x38         # no NaN codes
        dpool[(dpool & 0x78) == 0x78] &= 0xbf        # |code value| < 32: scores stay in a sane range
        pool = pool_from_device_layout(fp8_pool_to_float(dpool, 0.02, 0.013), shape.block_size, shape.head_dim)
    else:
        pool = filled_batch(shape, batch, seed=7)
        mark_unwritten(shape, batch, pool, np.nan)   # masked positions must not leak
        dpool = dev(pool_to_device_layout(pool), True)
    want = oracle.Oracle(cfg, base, None).attn_shared_kv(q, pool, batch.block_tables, lens, row_seq)
    layer.set_attn_piece_limit(limit)                # 0: pieces as the plan makes them
    got = layer.attn_shared_kv(dev(q, True), dpool, torch.from_numpy(batch.block_tables).cuda(), lens, row_seq)
    torch.cuda.synchronize()
    assert_close(host(got).reshape(want.shape), want, 2e-2, "attention out")
    layer.close()
