"""Every small-tile launch form (32 x 64 with one, two and four K ranges, 32 x 128,
64 x 128) in each of the four contractions (the forward's two, with and without
the saved intermediates, and the backward's two), on ragged tiles, against the
fp64 oracle.  Each case first asserts that the plan takes the form, so that a
change of the plan cannot move the tests off a path.

Bars: those of the prefill and training tests (y and dx rounded to bfloat16,
operands rounded once to fp16: 5e-3 relative L2 per token; fp32 scale
gradients 1e-3)."""
import numpy as np
import pytest
import torch

from paper_2609_06161_amd import synth
from paper_2609_06161_amd.layer import DeviceLayer, bf16_bits_to_f64, to_device

pytestmark = pytest.mark.gpu


def rows_rel(y, ref):
    return max(np.linalg.norm(a - e) / max(np.linalg.norm(e), 1e-300) for a, e in zip(y, ref))


# layers with two narrow dimensions, so that the one contraction is wide or long
# enough for its form and the oracle stays small; no token count or output width
# is a multiple of its tile's
TRAIN = [((32, 7168, 4256, 6), {0: (32, 64, 2)}), ((4128, 32, 7456, 5), {1: (32, 64, 2)}),
         ((7040, 32, 4320, 5), {2: (32, 64, 2)}), ((256, 4640, 7168, 5), {3: (32, 64, 2)}),
         ((64, 4736, 32, 5), {0: (32, 64, 4)}), ((32, 32, 5024, 5), {1: (32, 64, 4), 3: (32, 64, 4)}),
         ((4640, 64, 32, 5), {2: (32, 64, 4)}),
         ((32, 32, 5664, 67), {0: (32, 128, 1), 2: (32, 128, 1)}),
         ((5600, 96, 32, 65), {1: (32, 128, 1)}), ((32, 6048, 32, 66), {3: (32, 128, 1)}),
         ((32, 32, 4640, 203), {0: (64, 128, 1)}), ((6720, 96, 32, 132), {1: (64, 128, 1)}),
         ((1312, 64, 736, 1376), {2: (64, 128, 1)}), ((96, 6624, 32, 134), {3: (64, 128, 1)})]


@pytest.mark.parametrize("shape,forms", TRAIN)
def test_form_in_every_product(oracle, gemm_form, shape, forms):
    m, n, r, T = shape
    print(f"tile form m={m} n={n} r={r} T={T} {forms}", flush=True)
    for product, form in forms.items():
        assert gemm_form(m, n, r, T, product)[:3] == form
    lin = synth.make_linear(m + n + r + T, m, n, r, T)
    dy = synth.make_output_grad(T, T, m)
    L = DeviceLayer.from_host(lin)
    x = to_device(lin.x)
    y = torch.full((T, m), 0x7FC0, dtype=torch.int16, device="cuda")
    L.gemm(x, y=y)
    yt, saved = L.forward_train(x)
    dx, grads = L.backward(x, to_device(dy), saved)
    torch.cuda.synchronize()
    args = (m, n, r, lin.Bu, lin.Bv, lin.s_out, lin.s_mid, lin.s_in, lin.x)
    assert torch.equal(y, yt)
    assert rows_rel(bf16_bits_to_f64(y), oracle.forward(*args)) <= 5e-3
    rdx, *rds = oracle.backward(*args, dy)
    assert rows_rel(bf16_bits_to_f64(dx), rdx) <= 5e-3
    for g, ref in zip(grads, rds):
        g = g.cpu().numpy().astype(np.float64)
        assert np.linalg.norm(g - ref) <= 1e-3 * np.linalg.norm(ref)


# the second product's sum over more row-sum entries than its threads hold in
# registers (32 a token for 64-token tiles, 64 for 32-token ones), just past the
# line and far past it; and two K ranges of 32 x 128 tiles
FORWARD = [((5760, 32, 2176, 162), {0: (32, 64, 1), 1: (64, 128, 1)}),
           ((5664, 128, 4384, 65), {0: (32, 64, 1), 1: (32, 128, 1)}),
           ((32, 32, 4192, 3), {0: (32, 64, 1), 1: (32, 64, 1)}),
           ((32, 32, 5024, 5), {0: (32, 64, 1), 1: (32, 64, 4)}),
           ((1024, 32, 4192, 35), {0: (32, 64, 1), 1: (32, 64, 1)}),
           ((9696, 17088, 6144, 62), {0: (32, 64, 1), 1: (32, 128, 1)}),
           ((28672, 8192, 6336, 126), {0: (32, 128, 1), 1: (64, 128, 1)}),
           ((32, 26304, 1120, 280), {0: (32, 128, 2)})]


@pytest.mark.parametrize("shape,forms", FORWARD)
def test_many_row_sums(oracle, gemm_form, shape, forms):
    m, n, r, T = shape
    print(f"row sums m={m} n={n} r={r} T={T} {forms}", flush=True)
    for product, form in forms.items():
        assert gemm_form(m, n, r, T, product)[:3] == form
    lin = synth.make_linear(m + T, m, n, r, T)
    L = DeviceLayer.from_host(lin)
    y = torch.full((T, m), 0x7FC0, dtype=torch.int16, device="cuda")
    L.gemm(to_device(lin.x), y=y)
    again = L.gemm(to_device(lin.x))
    torch.cuda.synchronize()
    assert torch.equal(y, again)
    idx = np.unique(np.array([0, 31, 32, T // 2, T - 1]) % T)
    ref = oracle.forward(m, n, r, lin.Bu, lin.Bv, lin.s_out, lin.s_mid, lin.s_in, lin.x[idx])
    assert rows_rel(bf16_bits_to_f64(y)[idx], ref) <= 5e-3
