"""The vector attention kernel at its edges: positions around a quad, a block and a chunk of 1024, head sizes and block sizes that are
whole quads and not, workgroups of 256 and of 1024 threads."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host, make_layer, pool_to_device_layout
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
