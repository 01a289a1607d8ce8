"""The softmax reference of the prefill walk: scores that leave it by hundreds of powers of two, upwards (the reference moves and the
scores are formed again) and downwards (they vanish), at every place of a 32-token group, a round of four and a piece."""
import dataclasses

import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, fp8_pool_to_float, host, make_layer, pool_from_device_layout, pool_to_device_layout
from helpers import oracle_config
from paper_2603_13281_amd import synth

pytestmark = pytest.mark.gpu

PRE = [32, 64, 95, 127, 128, 129, 300, 513]
CHUNK = [1, 16, 33, 64, 65, 70, 5, 40]


def _pool(shape, batch, kind, reach):
    """Cached tokens whose keys are one direction u times a factor that runs from -reach to reach: a query's scores rise or fall
    by up to a few hundred, as its product with u is positive or negative.  Values differ between the two halves only, so that
    the output does not hang on the last bits of such scores."""
    rng = np.random.default_rng(5)
    D, Bk = shape.head_dim, shape.block_size
    u = rng.choice([-1.0, 1.0], size=(shape.n_kv_heads, D)) / np.sqrt(D)
    values = rng.normal(size=(2, shape.n_kv_heads, D))
    pool = np.zeros((batch.num_blocks, 2, shape.n_kv_heads, Bk, D), dtype=np.float32)
    for s, n in enumerate(PRE):
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
@pytest.mark.parametrize("limit", [0, 128, 1024])  # 1024: whole walks, of more than 512 tokens: the kernel for long pieces
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
