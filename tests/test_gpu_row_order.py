"""Row kernels whose workgroups take the rows in runs of one model (97 rows and more): every row once, whatever the models are."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import dev, host, make_layer, pool_to_device_layout
from helpers import assert_close, filled_batch, oracle_config
from paper_2603_13281_amd import synth

pytestmark = pytest.mark.gpu


def _active(kind, n_seq, n_models):
    """Active models of each sequence; with its encoder row the call has n_seq + their number rows."""
    if kind == "none":
        return [[] for _ in range(n_seq)]
    if kind == "one model":
        return [[1] for _ in range(n_seq)]
    if kind == "one row":
        return [[n_models - 1] if s == 5 else [] for s in range(n_seq)]
    return [list(range(s % (n_models + 1))) for s in range(n_seq)]  # 0, 1, .. models in turn


@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
@pytest.mark.parametrize("kind,n_seq", [("mixed", 32), ("mixed", 33), ("one model", 48), ("one model", 49), ("none", 97), ("one row", 103)], ids=str)
def test_every_row_once(shape, kind, n_seq):
    print("case: row order", shape.name, kind, n_seq, flush=True)
    base, lora = synth.make_base(shape, seed=9, norm_ones=False), synth.make_lora(shape, seed=9)
    lens = [3 + 7 * s % 50 for s in range(n_seq)]
    batch = synth.make_batch(shape, lens, [0] * n_seq, seed=9)
    pool = filled_batch(shape, batch, seed=9)
    seq, model = [], []
    for s, act in enumerate(_active(kind, n_seq, shape.n_models)):
        seq += [s] * (1 + len(act))
        model += [-1] + act
    x = synth.make_hidden(shape, len(seq), seed=9)
    want_pool = pool.copy()
    want, _ = oracle.Oracle(oracle_config(shape, batch.num_blocks), base, lora).decode_step(want_pool, batch.block_tables, lens, seq, model, x)
    layer = make_layer(shape, base, lora, batch.num_blocks)
    got = layer.decode_step(dev(pool_to_device_layout(pool), True), torch.from_numpy(batch.block_tables).cuda(), lens, np.asarray(seq, np.int32),
                            np.asarray(model, np.int32), dev(x, True))
    torch.cuda.synchronize()
    assert_close(host(got), want, 2e-2, "x_out")


@pytest.mark.parametrize("shape", [synth.LLAMA_SMALL, synth.QWEN_SMALL], ids=lambda s: s.name)
@pytest.mark.parametrize("n_seq", [1, 4, 5, 8, 9, 16, 17, 32, 33])
def test_few_rows_split_over_workgroups(shape, n_seq):
    """2 n_seq rows: an adapter's products are split over 16, 8, 4 or 2 workgroups a row, fewer for more rows; both sides of each line."""
    test_every_row_once(shape, "one model", n_seq)
