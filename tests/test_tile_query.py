"""Which tile of the whole-input batched kernel, and of the bf16 product, the library's own choice takes (host arithmetic, no GPU)."""
import random

from paper_2305_02299_amd import binding as B_


def test_tiles_of_named_layers():
    assert B_.srigl_fwd_tile_query(256, 768, 3072, 77, 3072) == (32, 6)           # one workgroup per compute unit
    assert B_.srigl_fwd_tile_query(1024, 768, 3072, 154, 3072) == (32, 24)
    assert B_.srigl_fwd_tile_query(256, 2160, 768, 216, 768)[0] in (8, 16)        # 32 rows of 2160 columns do not fit the LDS
    assert B_.srigl_fwd_tile_query(256, 3072, 768, 307, 768) == (8, 6)             # nor do 16 rows of 3072
    assert B_.srigl_fwd_tile_query(300, 1000, 700, 50, 777, has_active=True)[0] in (16, 32)
    for sizes in ((1, 768, 3072, 77, 3072), (16, 768, 3072, 77, 3072), (256, 4112, 768, 307, 768), (0, 768, 3072, 77, 3072), (64, 8, 3072, 4, 3072)):
        assert B_.srigl_fwd_tile_query(*sizes) == (0, 0), sizes                    # one row, a few rows, too wide, nothing, too narrow


def test_every_tile_taken_fits():
    rng = random.Random(11)
    taken = 0
    for _ in range(400):
        d_in, d_out = rng.randint(1, 4096), rng.randint(1, 16384)
        n = max(1, d_out - rng.choice([0, rng.randint(0, d_out // 2)]))
        K, B = max(1, d_in * rng.randint(1, 30) // 100), rng.choice([1, 2, 8, 16, 33, 100, 256, 777, 2048, 5000])
        tile, rows = B_.srigl_fwd_tile_query(B, d_in, n, K, d_out, rng.choice([B_.F32, B_.BF16]), rng.choice([16, 32]), n != d_out, rng.random() < 0.9)
        assert (tile == 0) == (rows == 0)
        if tile:
            taken += 1
            unit = 32 if tile == 8 else 16
            cols = -(-d_in // unit) * unit
            assert tile in (8, 16, 32, 64) and 16 <= d_in and B > 1
            assert ((cols + 1) * tile + tile * (16 * rows | 1)) * 4 <= 160 * 1024
    assert taken > 50


def test_shapes_of_bf16_products_that_only_the_choice_takes():
    """(B, d_in, stored, d_out): products measured behind in 128 x 96 and 64 x 128 go into 128 x 128 and 64 x 64, the ones around them measured ahead stay."""
    tile = lambda *sizes: B_.srigl_structured_tile_query(*sizes, B_.BF16)   # noqa: E731
    for sizes in ((314, 544, 7906, 13632), (331, 1120, 7918, 12416), (1127, 456, 2423, 3904), (428, 448, 5660, 8256)):
        assert tile(*sizes) == B_.TILE_128x128, sizes
    for sizes in ((616, 2416, 1728, 1728), (1116, 2680, 899, 899), (524, 2976, 1894, 3392)):
        assert tile(*sizes) == B_.TILE_64x64, sizes
    for sizes in ((1057, 208, 2196, 4032), (391, 3368, 5960, 11328), (1104, 672, 2017, 2164)):
        assert tile(*sizes) == B_.TILE_128x96, sizes
    for sizes in ((1192, 3952, 1026, 1472), (118, 3840, 10524, 10919), (188, 3160, 5494, 5494)):
        assert tile(*sizes) == B_.TILE_64x128, sizes
    assert tile(1500, 2048, 11440, 11440) == B_.TILE_192x192
