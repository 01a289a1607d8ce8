"""How the GEMMs' tiles are laid over the chip, on the host."""
import numpy as np
import pytest

from paper_2603_13281_amd import binding

XCDS, CUS = 8, 256


@pytest.mark.parametrize("tile", [(64, 128, 2), (128, 128, 1), (192, 128, 1), (256, 256, 1), (160, 256, 1)], ids=str)
@pytest.mark.parametrize("rows,cols,slices", [(1, 1, 1), (1, 7, 12), (1, 33, 4), (1, 224, 1), (1, 448, 1), (1, 1002, 1), (1, 80, 3), (2, 20, 12),
                                              (3, 448, 1), (9, 56, 2), (17, 112, 1), (64, 5, 3), (257, 31, 1)])
def test_every_tile_of_every_slice_once(rows, cols, slices, tile):
    order = binding.gemm_tile_order(rows, cols, slices, *tile)
    assert len(order) == rows * cols * slices
    assert len(np.unique(order[:, 1:], axis=0)) == len(order)
    assert (order.min(axis=0) >= 0).all() and (order.max(axis=0) < [XCDS, rows, cols, slices]).all()


@pytest.mark.parametrize("tile", [(64, 128, 2), (128, 128, 1), (160, 256, 1)], ids=str)
@pytest.mark.parametrize("cols", [112, 128, 200, 224, 250, 448, 512, 1002])
def test_one_row_tile_keeps_neighbouring_columns_on_an_xcd(cols, tile):
    # dealt over the XCDs, a quarter of the time is lost where the columns' strides line up (K = 8192, and K = 4096 with 65536 outputs)
    order = binding.gemm_tile_order(1, cols, 1, *tile)
    xcd = np.empty(cols, dtype=np.int64)
    xcd[order[:, 2]] = order[:, 0]
    changes = int((np.diff(xcd) != 0).sum())
    assert changes <= cols // 4, (changes, cols)


@pytest.mark.parametrize("vocab", [32000, 49152, 65536, 128256, 131072, 151936, 202048])
@pytest.mark.parametrize("rows", [1, 8, 64])
def test_lm_head_of_a_few_rows(rows, vocab):
    # 64 x 256 tiles lost up to a tenth of the step where the last round of workgroups is short
    assert binding.gemm_choice(rows, 4096, vocab, max_slices=1) == (64, 128, False, 1)


# (rows, K, outputs, adapter columns, most slices, slices taken by a later kernel) -> the launch that was fastest inside a layer
CHOICES = [
    ((162, 28672, [8192], 128, 12, False), (192, 128, False, 4)),     # modelled 1 % slower than 192 x 256 in 8 slices, measured 22 % faster
    ((189, 28672, [8192], 128, 12, False), (192, 128, False, 4)),
    ((374, 4096, [4096], 128, 12, True), (192, 128, False, 4)),
    ((360, 25600, [5120], 256, 12, False), (192, 256, True, 6)),      # 112 us, 119 us in 192 x 128 and 3 slices: no near tie
    ((270, 8192, [8192], 128, 12, True), (192, 128, False, 2)),
    ((720, 8192, [5120], 256, 12, True), (128, 128, False, 1)),
    ((385, 8192, [8192], 0, 12, True), (128, 128, False, 1)),
    ((10000, 4096, [4096], 0, 1, True), (256, 256, False, 1)),        # 349 us in 160 x 256, 327 us
    ((8000, 8192, [5120], 0, 1, True), (256, 256, False, 1)),
    ((4337, 14336, [4096], 0, 2, True), (192, 256, True, 2)),         # 457 us + 26 in the row kernel that sums them; 160 x 256 whole 502
]


@pytest.mark.parametrize("call,want", CHOICES, ids=[str(c[0][:3]) for c in CHOICES])
def test_near_ties_keep_the_plain_launch(call, want):
    rows, k, n, cols, most, taken = call
    assert binding.gemm_choice(rows, k, n, False, cols, most, taken) == want


@pytest.mark.parametrize("groups,want", [
    ([1] * 9, (64, 128)), ([64] + [8] * 8, (64, 128)), ([64, 64, 0, 1], (64, 128)),
    ([66] + [8] * 8, (64, 128)), ([300] + [38] * 8, (64, 128)),       # one group past the tile does not pad all the others
    ([66] * 9, (128, 128)), ([100] * 9, (128, 128)), ([130] * 9, (192, 128)), ([300] + [150] * 8, (192, 128)),
    ([200] * 9, (256, 256)), ([256] * 9, (256, 256)), ([1024] * 9, (256, 256)), ([0, 0], (64, 128)),
], ids=str)
def test_tile_of_grouped_projections(groups, want):
    assert binding.gemm_group_tile(groups) == want


# what the layers of the benchmark shapes run: (rows, K, outputs, fused, most slices, taken) -> launch
LAYERS = [
    ((374, 4096, [4096, 1024, 1024], False, 12, True), (192, 128, False, 2)),
    ((374, 4096, [14336], True, 1, False), (192, 256, True, 1)),
    ((374, 14336, [4096], False, 12, False), (192, 128, False, 4)),
    ((512, 25600, [5120], False, 12, False), (256, 256, False, 6)),
    ((512, 5120, [25600], True, 1, False), (256, 256, False, 1)),
    ((753, 14336, [4096], False, 12, False), (192, 256, True, 4)),
    ((753, 4096, [14336], True, 1, False), (192, 256, True, 1)),
    ((753, 5120, [8192, 1024, 1024], False, 8, True), (160, 256, True, 1)),
    ((4337, 4096, [4096], False, 2, True), (160, 256, True, 1)),
    ((4337, 14336, [4096], False, 2, False), (160, 256, True, 1)),
    ((16384, 4096, [14336], True, 1, False), (256, 256, False, 1)),
]


@pytest.mark.parametrize("call,want", LAYERS, ids=[str(c[0][:3]) for c in LAYERS])
def test_launches_of_the_benchmark_layers(call, want):
    rows, k, n, fused, most, taken = call
    assert binding.gemm_choice(rows, k, n, fused, 0, most, taken) == want


def test_choices_are_launches_the_workspace_holds():
    # never more slices than asked for, none empty, K slices of four slabs or more
    rng = np.random.default_rng(5)
    for _ in range(3000):
        rows, slabs = int(2 ** rng.uniform(0, 16)), int(2 ** rng.uniform(0, 9))
        n = [int(2 ** rng.uniform(6, 15)) // 8 * 8 for _ in range(rng.integers(1, 4))]
        cols, most, fused = int(rng.choice([0, 8, 128, 256])), int(rng.integers(1, 13)), bool(rng.integers(0, 2))
        bm, bn, reg, slices = binding.gemm_choice(rows, 64 * slabs, n[:1] if fused else n, fused, cols, most, bool(rng.integers(0, 2)))
        assert (bm, bn, reg) in ((64, 128, False), (128, 128, False), (192, 128, False), (256, 256, False), (192, 256, True), (160, 256, True))
        assert 1 <= slices <= (1 if fused else most)
        if slices > 1 and rows > 384:
            total = slabs + -(-cols // 64)
            per = -(-total // slices)
            assert per >= 6 and (slices - 1) * per < total


def test_append_of_short_chunks_goes_row_by_row():
    # a tile takes as long for one row as for sixteen: 4000 chunks of one token 71 us row by row, 143 us in tiles
    from test_abi_host import _cfg, _weights
    base, lora = _weights()
    layer = binding.IcarusLayer(_cfg(d_model=512, n_q_heads=32, n_kv_heads=8, head_dim=128), base, lora)
    assert not layer.append_in_tiles(400, 25)                 # too few rows
    assert layer.append_in_tiles(512, 33) and layer.append_in_tiles(4000, 1000) and layer.append_in_tiles(16384, 1024)
    assert not layer.append_in_tiles(4000, 4000) and not layer.append_in_tiles(4000, 2000) and not layer.append_in_tiles(3000, 1000)
    layer.close()
    other = binding.IcarusLayer(_cfg(n_q_heads=32, n_kv_heads=8, head_dim=64), base, lora)
    assert not other.append_in_tiles(16384, 1024)
    other.close()
