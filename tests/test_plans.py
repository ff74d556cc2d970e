"""The launch forms that the plans choose (host only), for a device of 256 compute
units: what each rule is there for."""
import pytest

# without a GPU the library plans for 256 compute units, as on an MI355X


@pytest.mark.parametrize("m,n,r,b,launches", [
    (1024, 4096, 800, 1, 1), (4096, 4096, 2016, 1, 1),
    (4096, 4096, 2016, 2, 2),      # one batch row only
    (32, 32, 32, 1, 2),            # fewer than sixteen workgroups
    (4096, 5120, 2240, 1, 2),      # more than two workgroups a unit
    # rows so long that a workgroup's LDS leaves no room for a second one
    (4096, 16384, 4096, 1, 2), (3072, 16384, 4096, 1, 2), (4096, 15680, 4096, 1, 2),
    (4096, 15648, 4096, 1, 1),
])
def test_one_launch_decode(test_lib, m, n, r, b, launches):
    assert test_lib.af1_test_gemv_launches(m, n, r, b) == launches


@pytest.mark.parametrize("m,n,r,count,two", [
    (4096, 16384, 3264, 2, True), (2560, 16384, 2176, 3, True),
    (4096, 15680, 3232, 2, True), (4096, 4096, 2016, 3, True),
    (4096, 16384, 2048, 2, False),   # no more workgroups than units
])
def test_fused_projections_leave_room_for_two(test_lib, m, n, r, count, two):
    """Where the launch has more workgroups than units, two fit a unit's LDS."""
    lds = test_lib.af1_test_multi_lds(m, n, r, count, 1)
    assert (2 * (lds + 256) <= 160 * 1024) == two


@pytest.mark.parametrize("m,n,r,T,product,form", [
    # small tiles measured slower than the large ones (us, small / large)
    (6912, 4672, 4672, 1525, 1, (128, 256, 1, 1)),   # 114 / 97
    (12128, 608, 608, 936, 1, (128, 256, 1, 0)),     # 28.9 / 24.9
    (10656, 704, 704, 400, 1, (64, 256, 1, 0)),      # 19.6 / 16.5
    (2432, 8096, 2432, 961, 0, (64, 256, 3, 0)),     # 55.3 / 48.8
    (27424, 544, 544, 272, 1, (128, 256, 1, 0)),     # 25.1 / 23.2
    (8160, 6176, 6176, 1329, 1, (128, 256, 1, 1)),   # 147 / 137
    # and faster
    (4096, 4096, 2016, 45, 0, (32, 64, 1, 0)),       # 6 / 11
    (8192, 8192, 4064, 500, 1, (64, 128, 1, 0)),
    (4096, 4096, 2016, 200, 3, (32, 128, 1, 0)),
])
def test_small_tiles_where_they_are_faster(gemm_form, m, n, r, T, product, form):
    assert gemm_form(m, n, r, T, product) == form


def test_no_partials_where_the_tiles_fill_the_device(gemm_form):
    """K ranges (whose partials take workspace) only where units would be idle."""
    for m, n, r, T in [(26784, 13312, 4480, 994), (28384, 12000, 2816, 1660), (24032, 576, 5568, 789)]:
        for product, (N, kind) in enumerate([(r, "f"), (m, "f"), (r, "b"), (n, "b")]):
            bm, bn, splits, _ = gemm_form(m, n, r, T, product)
            tiles = -(-T // bm) * -(-N // bn)
            assert splits == 1 or tiles < 256, (m, n, r, T, product)
