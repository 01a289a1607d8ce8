"""The GEMM kernels in every tile and number of K slices that the launch choice can name, against float64 products of the same bf16
inputs.  The choice itself is checked in test_gemm_plan.py; here a launch is asked for by name (icarus_gemm), so that a choice that
only a 5120-wide layer makes is covered at sizes of a few hundred."""
import numpy as np
import pytest
import torch

from paper_2603_13281_amd import binding

pytestmark = pytest.mark.gpu

TILES = [(64, 128, False), (128, 128, False), (192, 128, False), (256, 256, False), (192, 256, True), (160, 256, True)]
SLABS = {1: (4, 7, 40), 2: (12, 13), 3: (13, 36), 5: (24, 37), 12: (49, 96)}  # slices -> K / 64: even, odd, slices of unequal length and empty ones


def _draw(shape, seed, std=1.0):
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(seed)
    return (torch.randn(*shape, generator=gen, device="cuda:0") * std).to(torch.bfloat16)


def _adapters(rows, n, models, rank, sides, seed):
    """t with one model's columns per row (none for every fourth row, as the layers leave it) and B per side."""
    t = _draw((rows, sides, models, rank), seed)
    keep = torch.arange(rows, device="cuda:0") % (models + 1)
    t *= (keep[:, None] == torch.arange(1, models + 1, device="cuda:0")[None]).to(t.dtype)[:, None, :, None]
    return t.reshape(rows, -1).contiguous(), [_draw((models, n, rank), seed + 1 + s, 0.2) for s in range(sides)]


def _product(x, w, t=None, b=None):
    """float64 product and the sum of the absolute values of its terms."""
    y, s = x.double() @ w.double().T, x.double().abs() @ w.double().abs().T
    if t is not None:
        cat = b.permute(1, 0, 2).reshape(b.shape[1], -1).double()
        y, s = y + t.double() @ cat.T, s + t.double().abs() @ cat.abs().T
    return y, s


def _check(got, want, bound, what):
    """bound: |error| of fp32 sums of these terms in any order (terms * 2^-23 * sum of their absolute values), plus the rounding of the store."""
    assert torch.isfinite(got).all(), what
    worst = ((got.double() - want).abs() / bound).max().item()
    assert worst <= 1.0, (what, worst)


@pytest.mark.parametrize("tile", TILES, ids=lambda t: f"{t[0]}x{t[1]}" + ("r" if t[2] else ""))
@pytest.mark.parametrize("slices", list(SLABS))
@pytest.mark.parametrize("models,rank", [(0, 0), (1, 8), (3, 16), (8, 32)], ids=["plain", "8", "48", "256"])
def test_projection(tile, slices, models, rank):
    # three stacked matrices with ragged last column tiles (q, k and v: adapters on the first only), and one with a residual;
    # one row tile, one row more, and a row tile count that panels do not divide
    bm, bn, _ = tile
    for slabs in SLABS[slices]:
        for rows in (1, bm + 1, 3 * bm - 5):
            k, n = 64 * slabs, [bn + 8, 16, 2 * bn - 40]
            x, w = _draw((rows, k), slabs), [_draw((m, k), 10 + i, 0.05) for i, m in enumerate(n)]
            t, b = _adapters(rows, n[0], models, rank, 1, 20) if models else (None, None)
            what = (tile, "slices", slices, "slabs", slabs, "rows", rows, "adapters", models * rank)
            print("case:", *what, flush=True)
            eps = (k + models * rank + 16) * 2.0 ** -23
            parts = [_product(x, v, t if i == 0 else None, b[0] if t is not None else None) for i, v in enumerate(w)]
            want, size = (torch.cat([p[j] for p in parts], 1) for j in (0, 1))
            _check(binding.gemm(x, w, tile, slices, t=t, b=b), want, eps * size + 1e-30, what)
            resid = _draw((rows, n[0]), 30)
            want = parts[0][0] + resid.double()
            _check(binding.gemm(x, w[:1], tile, slices, t=t, b=b, resid=resid), want,
                   eps * (parts[0][1] + resid.double().abs()) + 2.0 ** -8 * want.abs() + 1e-30, what + ("residual",))


@pytest.mark.parametrize("tile", TILES, ids=lambda t: f"{t[0]}x{t[1]}" + ("r" if t[2] else ""))
@pytest.mark.parametrize("models,rank", [(0, 0), (1, 8), (3, 16), (8, 32)], ids=["plain", "8", "48", "256"])
def test_gate_up(tile, models, rank):
    # silu(gate) * up, adapters on both; |d silu| <= 1.1 |d gate|
    bm, bn, _ = tile
    for slabs in SLABS[1]:
        for rows in (1, bm + 1, 3 * bm - 5):
            for n in (bn // 2 + 8, 3 * bn // 2 - 24):
                k = 64 * slabs
                x, w = _draw((rows, k), slabs), [_draw((n, k), 10 + i, 0.05) for i in range(2)]
                t, b = _adapters(rows, n, models, rank, 2, 20) if models else (None, None)
                what = (tile, "fused", "slabs", slabs, "rows", rows, "n", n, "adapters", models * rank)
                print("case:", *what, flush=True)
                half = (lambda s: t[:, s * models * rank:(s + 1) * models * rank]) if models else (lambda s: None)
                (g, gs), (u, us) = (_product(x, w[s], half(s), b[s] if models else None) for s in range(2))
                silu = g * torch.sigmoid(g)
                eps = (k + models * rank + 16) * 2.0 ** -23
                bound = 1.1 * eps * gs * u.abs() + eps * us * silu.abs() + (2.0 ** -8 + (2 + g.abs()) * 2.0 ** -21) * (silu * u).abs() + 2.0 ** -100
                _check(binding.gemm(x, w, tile, fused=True, t=t, b=b), silu * u, bound, what)


@pytest.mark.parametrize("tile", TILES, ids=lambda t: f"{t[0]}x{t[1]}" + ("r" if t[2] else ""))
@pytest.mark.parametrize("slabs,slices", [(7, 1), (8, 1), (13, 2), (37, 5)])
@pytest.mark.parametrize("models", [0, 3])
def test_infinite_activations_reach_only_their_products(tile, slabs, slices, models):
    # a launch pads K (odd slab counts, slices, adapter columns up to a whole slab) with zeros on both sides: an infinity gives
    # infinities of the weights' signs, no NaN, wherever in K it is
    print("case: infinities", tile, slabs, slices, models, flush=True)
    rows, n, k = slabs, tile[1] + 8, 64 * slabs
    x, w = _draw((rows, k), 1), _draw((n, k), 2, 0.05)
    w = torch.where(w == 0, torch.ones_like(w), w)
    at = torch.arange(rows, device="cuda:0") * 64 + 9            # an infinity in every slab, one row each
    x[torch.arange(rows, device="cuda:0"), at] = float("inf")
    t, b = _adapters(rows, n, models, 16, 1, 20) if models else (None, None)
    got = binding.gemm(x, [w], tile, slices, t=t, b=b)
    want = torch.sign(w[:, at].T.float()) * float("inf")
    assert torch.equal(got, want)
    if models:                                                   # the last adapter column, next to the padding
        x, t = _draw((rows, k), 1), t.clone()
        t[0, -1] = float("inf")
        b[0][-1, :, -1] = 1.0
        got = binding.gemm(x, [w], tile, slices, t=t, b=b)
        assert torch.isposinf(got[0]).all() and torch.isfinite(got[1:]).all()


@pytest.mark.parametrize("rows", [128, 129, 160, 161, 192, 193, 256, 257, 320, 321, 384, 480, 481])
def test_lower_tiles_where_as_many_hold_the_rows(rows):
    # a launch in 192 x 128 tiles is one of 128 or 160 rows each, if it needs no more of them
    print("case: 192 x 128", rows, flush=True)
    k, n, models, rank = 64 * 9, 136, 3, 16
    x, w = _draw((rows, k), 1), [_draw((n, k), 10 + i, 0.05) for i in range(2)]
    t, b = _adapters(rows, n, models, rank, 1, 20)
    eps = (k + models * rank + 16) * 2.0 ** -23
    want, size = _product(x, w[0], t, b[0])
    _check(binding.gemm(x, w[:1], (192, 128, False), 2, t=t, b=b), want, eps * size + 1e-30, rows)
    (g, gs), (u, us) = (_product(x, v) for v in w)
    silu = g * torch.sigmoid(g)
    bound = 1.1 * eps * gs * u.abs() + eps * us * silu.abs() + (2.0 ** -8 + (2 + g.abs()) * 2.0 ** -21) * (silu * u).abs() + 2.0 ** -100
    _check(binding.gemm(x, w, (192, 128, False), fused=True), silu * u, bound, (rows, "fused"))


@pytest.mark.parametrize("fused", [False, True], ids=["plain", "fused"])
@pytest.mark.parametrize("rows,cols", [(250, 128), (250, 129), (576, 85), (576, 86)])
def test_narrow_tiles_by_eight_waves_and_by_four(rows, cols, fused):
    # 192 x 128 tiles, two of 128 rows or three of 192: up to 256 workgroups have a CU to themselves and eight waves, more share one with four each
    print("case: waves of a narrow tile", rows, cols, fused, flush=True)
    k, n, models, rank = 64 * 9, (64 if fused else 128) * cols - 24, 3, 16
    x, w = _draw((rows, k), 1), [_draw((n, k), 10 + i, 0.05) for i in range(1 + fused)]
    t, b = _adapters(rows, n, models, rank, 1 + fused, 20)
    eps = (k + models * rank + 16) * 2.0 ** -23
    got = binding.gemm(x, w, (192, 128, False), fused=fused, t=t, b=b)
    parts = [_product(x, w[s], t[:, s * models * rank:(s + 1) * models * rank], b[s]) for s in range(1 + fused)]
    if not fused:
        return _check(got, parts[0][0], eps * parts[0][1] + 1e-30, (rows, cols))
    (g, gs), (u, us) = parts
    silu = g * torch.sigmoid(g)
    bound = 1.1 * eps * gs * u.abs() + eps * us * silu.abs() + (2.0 ** -8 + (2 + g.abs()) * 2.0 ** -21) * (silu * u).abs() + 2.0 ** -100
    _check(got, silu * u, bound, (rows, cols, "fused"))


@pytest.mark.parametrize("tile", TILES, ids=lambda t: f"{t[0]}x{t[1]}" + ("r" if t[2] else ""))
@pytest.mark.parametrize("rows", [100, 200, 384, 385])
@pytest.mark.parametrize("models", [0, 8])
def test_column_tiles_that_start_at_different_places_along_k(tile, rows, models):
    # K a multiple of 2048, up to 384 rows: column tile n starts at slab n modulo their number -- 34 column tiles (fused: 67) on 32 slabs, on three
    # slices of 11 and 10, and on twelve of three slabs, of which with adapters one ends in and one is nothing but adapter columns and without one is empty
    print("case: turn", tile, rows, models, flush=True)
    k, n, rank = 2048, 33 * tile[1] + 8, 32
    x, w = _draw((rows, k), 1), [_draw((n, k), 10 + i, 0.05) for i in range(2)]
    t, b = _adapters(rows, n, models, rank, 2, 20) if models else (None, None)
    half = (lambda s: t[:, s * models * rank:(s + 1) * models * rank].contiguous()) if models else (lambda s: None)
    (g, gs), (u, us) = (_product(x, w[s], half(s), b[s] if models else None) for s in range(2))
    eps = (k + models * rank + 16) * 2.0 ** -23
    for slices in (1, 3, 12):
        got = binding.gemm(x, w[:1], tile, slices, t=half(0), b=b[:1] if models else None)
        _check(got, g, eps * gs + 1e-30, (tile, rows, models, slices))
    silu = g * torch.sigmoid(g)
    bound = 1.1 * eps * gs * u.abs() + eps * us * silu.abs() + (2.0 ** -8 + (2 + g.abs()) * 2.0 ** -21) * (silu * u).abs() + 2.0 ** -100
    _check(binding.gemm(x, w, tile, fused=True, t=t, b=b), silu * u, bound, (tile, rows, models, "fused"))


@pytest.mark.parametrize("rows", [160, 161, 192, 193, 320, 321, 384, 480, 481])
@pytest.mark.parametrize("k", [64 * 9, 64 * 257])
def test_full_192_row_tiles_with_many_adapter_columns(rows, k):
    # 8 adapters of rank 32: up to K = 16384 k_gemm_mfma takes the tiles that are needed in full, k_gemm_quad the lower ones and longer K
    print("case: 192 x 128, 256 adapter columns", rows, k, flush=True)
    n, models, rank = [136, 24], 8, 32
    x, w = _draw((rows, k), 1), [_draw((m, k), 10 + i, 0.05) for i, m in enumerate(n)]
    t, b = _adapters(rows, n[0], models, rank, 1, 20)
    eps = (k + models * rank + 16) * 2.0 ** -23
    (q, qs), (v, vs) = _product(x, w[0], t, b[0]), _product(x, w[1])
    for slices in (1, 3):
        _check(binding.gemm(x, w, (192, 128, False), slices, t=t, b=b), torch.cat([q, v], 1), eps * torch.cat([qs, vs], 1) + 1e-30, (rows, k, slices))


@pytest.mark.parametrize("k", [2 ** 23, 2 ** 23 + 64])
@pytest.mark.parametrize("tile,rows", [((192, 128, False), 192), ((160, 256, True), 160)], ids=["192x128", "160x256"])
def test_rows_gigabytes_apart(tile, rows, k):
    # K = 2^23: the last row of a tile is more than 2^31 bytes behind its first, within the 32 bits that k_gemm_quad keeps; one slab
    # more and the launch goes to the kernel with 64-bit row addresses.  A few columns of small whole numbers: exact in any order.
    print("case: rows gigabytes apart", tile, rows, k, flush=True)
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    cols = torch.tensor([0, 63, 64, k // 12, k // 2 - 1, k // 2, k - 65, k - 64, k - 1], device="cuda:0")
    x, w = (torch.zeros((n, k), dtype=torch.bfloat16, device="cuda:0") for n in (rows, 8))
    xs, ws = (torch.randint(-8, 9, (n, len(cols)), generator=gen, device="cuda:0").to(torch.bfloat16) for n in (rows, 8))
    x[:, cols], w[:, cols] = xs, ws
    got = binding.gemm(x, [w], tile, 12)
    assert torch.equal(got.double(), xs.double() @ ws.double().T)


def test_gemm_refuses_what_the_kernels_do_not_take():
    x, w = _draw((4, 128), 1), _draw((16, 128), 2)
    for kw in (dict(tile=(96, 128, False)), dict(tile=(256, 256, True)), dict(tile=TILES[0], slices=13), dict(tile=TILES[0], slices=0)):
        with pytest.raises(binding.IcarusError):
            binding.gemm(x, [w], **kw)
    with pytest.raises(binding.IcarusError):
        binding.gemm(_draw((4, 96), 1), [_draw((16, 96), 2)], TILES[0])      # K not a multiple of 64
    with pytest.raises(binding.IcarusError):
        binding.gemm(x, [_draw((12, 128), 2)], TILES[0])                      # outputs not a multiple of 8
    with pytest.raises(binding.IcarusError):
        binding.gemm(x, [w, w], TILES[0], slices=2, fused=True)
