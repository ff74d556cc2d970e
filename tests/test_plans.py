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
