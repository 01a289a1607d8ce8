"""A call's metadata reaches the device as kernel arguments up to 960 ints and by a copy from pinned memory beyond; the calls without a
workspace pass all of it as arguments.  The same bits either way, also for calls that follow one another without a wait."""
import numpy as np
import pytest
import torch

from gpu_util import dev, make_layer, pool_to_device_layout
from helpers import filled_batch
from paper_2603_13281_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [synth.TINY, synth.LLAMA_SMALL], ids=lambda s: s.name)
def test_metadata_sizes_around_one_launch(shape):
    lens = [20 + i for i in range(330)]
    batch = synth.make_batch(shape, lens, [0] * len(lens), seed=8, headroom=0)
    layer = make_layer(shape, synth.make_base(shape), None, batch.num_blocks)
    pool = dev(pool_to_device_layout(filled_batch(shape, batch, seed=8)), shape.bf16)
    tables = torch.from_numpy(batch.block_tables).cuda()
    q = dev(np.random.default_rng(9).standard_normal((len(lens), shape.n_q_heads, shape.head_dim)), shape.bf16)
    got, want = [], []
    sizes = [1, 40, 80, 96, 100, 106, 107, 119, 120, 121, 136, 137, 160, 192, 200, 239, 240, 241, 300, 330]   # 4 to 9 ints a row
    for n in sizes * 2:                       # more calls than staging buffers
        print("case: metadata of", n, "rows", shape.name, flush=True)
        args = (q[-n:].clone(), pool, tables[-n:].clone(), lens[-n:], np.arange(n))
        out = torch.empty_like(args[0])
        got.append(layer.attn_shared_kv(*args))
        want.append(layer.attn_shared_kv_static(*args, out))
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) and torch.isfinite(a).all() for a, b in zip(got, want))
