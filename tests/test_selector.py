"""Host-side choice between the condensed and the structured-only representation (Sec. 4.4 / Fig. 4): properties that
hold whatever the calibration, plus the two ends of the paper's comparison.  No GPU work: the function is arithmetic on sizes."""
import pytest

import synth_inputs as si


@pytest.fixture(scope="module")
def B_():
    from paper_2305_02299_amd import binding
    return binding


def test_small_batches_stay_condensed(B_):
    """Online inference (one row) in either storage type, and batches up to 16 in fp32 (where the matrix pipe is slow)."""
    for (d_in, d_out, sp, K, B) in si.sweep_points():
        for dt in (B_.F32, B_.BF16):
            if B == 1 or (B <= 16 and dt == B_.F32):
                r, c, s = B_.srigl_choose_representation(B, d_in, d_out, K, d_out, dt)
                assert r == B_.REPR_CONDENSED, (d_in, d_out, K, B, dt, c, s)


def test_large_bf16_batch_at_modest_sparsity_goes_structured(B_):
    L = si.config("c5")
    r, c, s = B_.srigl_choose_representation(L.B, L.d_in, L.d_out, L.K, L.d_out, B_.BF16)
    assert r == B_.REPR_STRUCTURED and s < c


def test_online_inference_config_stays_condensed(B_):
    L = si.config("c1")
    r, c, s = B_.srigl_choose_representation(1, L.d_in, L.d_out, L.K, L.d_out, B_.F32)
    assert r == B_.REPR_CONDENSED and c < s


@pytest.mark.parametrize("dt", [0, 1])
def test_denser_rows_never_move_the_choice_towards_condensed(B_, dt):
    """The structured estimate does not depend on K, the condensed one grows with it."""
    for B in (64, 256, 1024, 4096):
        seen_structured = False
        prev_c = None
        for K in (1, 8, 39, 77, 154, 307, 768):
            r, c, s = B_.srigl_choose_representation(B, 768, 3072, K, 3072, dt)
            if prev_c is not None:
                assert c >= prev_c
            prev_c = c
            if seen_structured:
                assert r == B_.REPR_STRUCTURED
            seen_structured = seen_structured or r == B_.REPR_STRUCTURED


def test_rows_that_are_not_whole_16_byte_pieces_stay_condensed(B_):
    r, c, s = B_.srigl_choose_representation(4096, 770, 3072, 385, 3072, B_.F32)
    assert r == B_.REPR_CONDENSED
    r, c, s = B_.srigl_choose_representation(4096, 772, 3072, 385, 3072, B_.BF16)
    assert r == B_.REPR_CONDENSED


def test_parts_of_d_in_for_the_structured_only_product(B_):
    """Host-only plan: a wide fp32 layer with few stored neurons at a modest batch is cut into parts (its tiles alone reach a
    fraction of the compute units); a product with thousands of tiles is not; the workspace is parts x B x n_active floats."""
    L = si.config("c3", B=256)
    n = 538
    parts, need = B_.srigl_structured_split_plan(256, L.d_in, n, L.d_out, B_.F32)
    assert 2 <= parts <= 16 and need == parts * 256 * n * 4
    L5 = si.config("c5")
    assert B_.srigl_structured_split_plan(L5.B, L5.d_in, 13108, L5.d_out, B_.BF16) == (1, 0)
    # every part keeps at least four stages of 128 bytes: 64 fp32 columns are two stages, so one part
    assert B_.srigl_structured_split_plan(16, 64, 64, 64, B_.F32) == (1, 0)
    for (B, d_in, n_active) in [(1, 768, 3072), (64, 3072, 538), (300, 1024, 96), (2048, 4096, 100)]:
        for dt in (B_.F32, B_.BF16):
            parts, need = B_.srigl_structured_split_plan(B, d_in, n_active, n_active, dt)
            stages = (d_in * (4 if dt == B_.F32 else 2) + 127) // 128
            assert 1 <= parts <= max(1, min(16, stages // 4))
            assert need == (parts * B * n_active * 4 if parts > 1 else 0)
    assert B_.srigl_structured_split_plan(0, 768, 0, 3072, B_.F32) == (1, 0)


def test_the_condensed_estimate_is_that_of_the_form_the_call_takes(B_):
    """bf16 at sizes where the layer's call goes to the matrix cores: the choice compares that form, not the gathering kernels (measured, with its
    copy made in the call: 4096 -> 16384 with 13108 stored 211 us at batch 2048, 112 at 1024; the gathering kernels need 620 and 312)."""
    for (B, d_in, n, K, d_out, condensed, structured) in ((2048, 4096, 13108, 205, 16384, 211.1, 193.4), (1024, 4096, 13108, 205, 16384, 111.5, 98.5),
                                                         (2048, 4096, 16384, 205, 16384, 204.4, 189.4), (512, 4096, 4096, 410, 4096, 44.9, 29.2),
                                                         (1024, 768, 3072, 77, 3072, 21.3, 12.6), (512, 1024, 4096, 102, 4096, 18.9, 10.9)):
        assert B_.srigl_blocked_tile_with_copy(B, d_in, n, K, d_out) != 0
        r, c, s = B_.srigl_choose_representation(B, d_in, n, K, d_out, B_.BF16)
        assert abs(c / condensed - 1) < 0.15 and abs(s / structured - 1) < 0.15
    # rows the structured form cannot hold: the estimate is still the matrix-core form's
    r, c, s = B_.srigl_choose_representation(1024, 546, 16192, 98, 16192, B_.BF16)
    assert r == B_.REPR_CONDENSED and abs(c / 40.1 - 1) < 0.15


def test_bf16_products_that_the_condensed_form_does_not_reach(B_):
    """us measured beside each other, condensed / structured.  While the product's estimate was 13 % too high the condensed form was taken here."""
    for (B, d_in, n, K, d_out) in ((64, 4096, 4096, 410, 4096),      # 17.7 / 13.9
                                   (128, 768, 3072, 154, 3072),      # 9.2 / 7.8
                                   (512, 2048, 2048, 102, 2048)):    # 16.4 / 13.1
        r, c, s = B_.srigl_choose_representation(B, d_in, n, K, d_out, B_.BF16)
        assert r == B_.REPR_STRUCTURED, (B, d_in, K, c, s)
    for (B, d_in, n, K, d_out) in ((128, 4096, 1024, 205, 1024),     # 8.8 / 12.3
                                   (32, 4096, 13108, 205, 16384),    # 16.1 / 24.6
                                   (64, 768, 3072, 77, 3072)):       # 6.4 / 7.7
        r, c, s = B_.srigl_choose_representation(B, d_in, n, K, d_out, B_.BF16)
        assert r == B_.REPR_CONDENSED, (B, d_in, K, c, s)
