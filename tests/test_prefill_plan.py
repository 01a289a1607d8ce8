"""The plan of the prefill attention, on the host: what pieces a call's walks are cut into and where their partial results go."""
import numpy as np
import pytest

from paper_2603_13281_amd import binding
from test_abi_host import _cfg, _weights

WALK = 131072  # tokens one workgroup can walk


def _layer(g, n_kv, n_blocks=1 << 16):
    base, lora = _weights()
    return binding.IcarusLayer(_cfg(d_model=1024, n_q_heads=g * n_kv, n_kv_heads=n_kv, head_dim=128, num_blocks=n_blocks, max_position=1 << 20), base, lora)


def _check(layer, g, ctx, chunk):
    """Every group of every chunk walked once from its first token to its last; partial slots of cut walks distinct, in
    token order; inner boundaries on whole rounds."""
    pieces = layer.prefill_plan(ctx, chunk)
    assert len(pieces), ("vector kernel", ctx, chunk)
    tq, row, groups = max(1, 256 // g), 0, {}
    for c, n in zip(ctx, chunk):
        for t in range(0, n, tq):
            groups[row + t] = (min(tq, n - t), c + min(n, t + tq))
        row += n
    slots = []
    assert sorted(set(int(r) for r in pieces[:, 0])) == sorted(groups)
    for r, (rows, kv) in groups.items():
        mine = pieces[pieces[:, 0] == r]
        mine = mine[np.argsort(mine[:, 2])]
        assert (mine[:, 1] == rows).all()
        at = 0
        for _, _, begin, n, slot in mine:
            assert begin == at and 0 < n <= WALK and begin % 128 == 0
            at += n
            slots.append(int(slot))
        assert at == kv
        if len(mine) == 1:
            assert mine[0, 4] == -1
        else:
            assert (np.diff(mine[:, 4]) == 1).all() and mine[0, 4] >= 0
    slots = [s for s in slots if s >= 0]
    assert sorted(slots) == list(range(len(slots)))


@pytest.mark.parametrize("g,n_kv", [(1, 8), (4, 8), (8, 8), (8, 2), (16, 1)])
@pytest.mark.parametrize("ctx,chunk", [
    ([135000], [4096]), ([135000], [8192]), ([135000] * 4, [2048] * 4), ([131000], [200]), ([131072], [1]), ([400000, 5], [3000, 700]),
    ([200000], [60000]), ([262144 - 100, 131072, 0, 90], [300, 1, 5000, 64]),
], ids=lambda v: "+".join(map(str, v)))
def test_contexts_beyond_a_workgroup_stay_on_the_matrix_cores(g, n_kv, ctx, chunk):
    layer = _layer(g, n_kv)
    _check(layer, g, ctx, chunk)
    layer.close()


def test_plans_of_drawn_calls():
    rng = np.random.default_rng(11)
    for _ in range(300):
        g, n_kv = [(1, 8), (2, 8), (4, 8), (8, 8), (4, 4), (8, 1)][rng.integers(0, 6)]
        layer = _layer(g, n_kv)
        S = int(rng.integers(1, 9))
        ctx = [int(x) for x in 2 ** rng.uniform(0, 18, S)]
        chunk = [int(x) for x in 2 ** rng.uniform(0, 12, S)]
        layer.set_attn_piece_limit(int(rng.choice([0, 0, 128, 1000, 5000])))
        _check(layer, g, ctx, chunk)
        layer.close()


def test_a_shorter_call_needs_no_more_workspace():
    # room for forced pieces only where a context asks for them
    layer = _layer(8, 8)
    small, at, past = (layer.workspace_bytes(4096, 1, n) for n in (WALK - 20000, WALK, WALK + 4000))
    assert small <= at < past
    assert layer.workspace_bytes(9, 1, WALK + 4000) - layer.workspace_bytes(9, 1, WALK) < 1 << 24
    layer.close()


@pytest.mark.parametrize("ctx,chunk", [([2522, 6657, 8161, 4188], [113, 345, 72, 223]), ([3366, 3809], [568, 469]), ([1933, 1832, 2744], [24, 89, 426])],
                         ids=lambda v: "+".join(map(str, v)))
def test_remainders_of_walks_follow_their_equal_parts(ctx, chunk):
    layer = _layer(4, 8)
    _check(layer, 4, ctx, chunk)
    pieces = layer.prefill_plan(ctx, chunk)
    cut = [p for p in pieces if (pieces[:, 0] == p[0]).sum() > 1]
    last = {p[0]: max(q[2] for q in cut if q[0] == p[0]) for p in cut}
    tail = [i for i, p in enumerate(pieces) if p[0] in last and p[2] == last[p[0]]]
    assert tail == list(range(len(pieces) - len(tail), len(pieces)))  # after all others,
    assert all(pieces[a][3] >= pieces[b][3] for a, b in zip(tail, tail[1:]))  # longest first
    assert len({p[3] for i, p in enumerate(pieces) if p[0] in last and i not in tail}) == 1
    layer.close()


@pytest.mark.parametrize("n_kv,ctx,chunk", [(8, [9000], [632]), (8, [14000], [300]), (8, [24000], [300]), (4, [9000] * 5, [317] * 5), (4, [24000], [326])],
                         ids=lambda v: "+".join(map(str, v)) if isinstance(v, list) else str(v))
def test_no_short_remainders_behind_a_full_round_of_equal_parts(n_kv, ctx, chunk):
    """Pieces are dealt to the engines of 8 CUs in turn, whoever is free: what is dealt to an engine after eight of its CUs have a long piece waits for
    one of them.  The call's longest engine is no longer than with equal parts of the shortest length that still makes whole rounds of CUs."""
    layer = _layer(4, n_kv)
    _check(layer, 4, ctx, chunk)
    pieces, engines = layer.prefill_plan(ctx, chunk), 32 // n_kv
    cus = 8 * engines
    assert any((pieces[:, 4] >= 0))

    def longest(lens):
        free, end = np.zeros((engines, 8), np.int64), 0
        for i, n in enumerate(lens):
            h = free[i % engines]
            k = int(h.argmin())
            h[k] += n + 160
            end = max(end, int(h[k]))
        return end

    groups = sum(-(-n // 64) for n in chunk)
    best = None
    for rounds in (1, 2, 3, 4):
        parts = rounds * cus // groups
        if parts:
            top = max(c + n for c, n in zip(ctx, chunk))
            n = -(-top // parts // 128) * 128 + 128
            best = min(best or 1 << 60, rounds * (n + 160))
    assert longest(pieces[:, 3]) <= best
    layer.close()
