"""The decode forward as one launch when the second product's wait ends before
the first product's values are there: the waiting workgroups compute them, so
the call ends with the same outputs whatever keeps the first product's
workgroups from starting.

The test build of the library forces that: its second product does not wait, and
its first product starts some 60 us late."""
import importlib.util

import numpy as np
import pytest
import torch

from paper_2609_06161_amd import af1, build_lib, synth
from paper_2609_06161_amd.layer import DeviceLayer, to_device

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def late():
    """The binding on the test build."""
    spec = importlib.util.spec_from_file_location("paper_2609_06161_amd.af1_late", af1.__file__)
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    mod.LIB_PATH = build_lib.TEST_LIB
    mod.lib()
    return mod


def call(late, L, x, y, ws):
    d = late.make_layer(L.m, L.n, L.r, L.Bu, L.Bv, L.s_out, L.s_mid, L.s_in)
    late.af1_linear_gemv(d, x, 1, y, ws, ws.numel())


def nan_out(m):
    return torch.full((1, m), 0x7FC0, dtype=torch.int16, device="cuda")


# few and many second-product workgroups, ranks that end inside a row tile, one
# and two column halves of the first product, up to the largest grid
SHAPES = [(224, 32, 32), (480, 1056, 96), (1024, 1024, 480), (32, 2048, 3360), (1024, 4096, 800),
          (3072, 3072, 1504), (4096, 4096, 2016)]


@pytest.mark.parametrize("m,n,r", SHAPES)
def test_values_computed_instead(late, m, n, r):
    print(f"late first product m={m} n={n} r={r}", flush=True)
    lin = synth.make_linear(m + n + r, m, n, r, 1)
    lin.s_mid[:5] = 0  # zeros are values too
    L, x = DeviceLayer.from_host(lin), to_device(lin.x)
    two = nan_out(m)
    af1.af1_linear_gemv_noalloc(L.desc, x, 1, two)
    ws = torch.zeros(af1.af1_gemv_workspace_bytes(m, n, r, 1), dtype=torch.uint8, device="cuda")
    for _ in range(4):  # both link buffers, each cleared by the other's call
        y = nan_out(m)
        call(late, L, x, y, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, two)


def test_late_and_ordinary_calls_share_a_workspace(late):
    """The header that a late call leaves serves the next call of any shape."""
    cases = []
    for i, (m, n, r) in enumerate(SHAPES[2:]):
        lin = synth.make_linear(40 + i, m, n, r, 1)
        L, x, two = DeviceLayer.from_host(lin), to_device(lin.x), nan_out(m)
        af1.af1_linear_gemv_noalloc(L.desc, x, 1, two)
        cases.append((L, x, two))
    ws = torch.zeros(max(af1.af1_gemv_workspace_bytes(L.m, L.n, L.r, 1) for L, _, _ in cases),
                     dtype=torch.uint8, device="cuda")
    rng = np.random.default_rng(8)
    for k, slow in zip(rng.integers(0, len(cases), 40), rng.integers(0, 2, 40)):
        L, x, two = cases[k]
        y = nan_out(L.m)
        if slow:
            call(late, L, x, y, ws)
        else:
            L.gemv(x, y, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, two), (L.m, L.n, L.r, slow)
