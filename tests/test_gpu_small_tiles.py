"""The small-tile contractions at the edges of their tiles and K steps, through
the prefill forward and the scale-only training step, against the fp64 oracle
(layers this small take 32-token tiles; 64 x 128 ones are in
test_gpu_tile_forms.py).

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


# token counts around the 32- and 64-token tiles; widths one group below, at
# and above the 64- and 128-row tiles and the 128- and 256-column K steps
@pytest.mark.parametrize("T", [1, 31, 32, 33, 63, 65, 129])
@pytest.mark.parametrize("m,n,r", [(32, 32, 32), (96, 224, 64), (160, 288, 128), (544, 992, 416),
                                   (1056, 1024, 480)])
def test_small_tile_edges(oracle, T, m, n, r):
    print(f"small tiles m={m} n={n} r={r} T={T}", flush=True)
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


# ordinary layers whose two products take different forms (the plan's choices on
# one device; test_gpu_tile_forms.py asserts the form of each of its cases)
@pytest.mark.parametrize("m,n,r,T", [(4096, 4096, 2016, 500), (4096, 4096, 2016, 130),
                                     (4096, 14336, 3136, 20), (2048, 28672, 1536, 40),
                                     (14336, 4096, 3136, 700)])
def test_small_tile_forms(oracle, m, n, r, T):
    print(f"small tile form m={m} n={n} r={r} T={T}", flush=True)
    lin = synth.make_linear(m + T, m, n, r, T)
    L = DeviceLayer.from_host(lin)
    y = torch.full((T, m), 0x7FC0, dtype=torch.int16, device="cuda")
    L.gemm(to_device(lin.x), y=y)
    torch.cuda.synchronize()
    idx = np.unique(np.concatenate([[0, 31, T - 1], np.random.default_rng(T).integers(0, T, 9)]) % T)
    ref = oracle.forward(m, n, r, lin.Bu, lin.Bv, lin.s_out, lin.s_mid, lin.s_in, lin.x[idx])
    assert rows_rel(bf16_bits_to_f64(y)[idx], ref) <= 5e-3


def test_neighbour_token_does_not_leak():
    """A token whose row holds infinities leaves the other tokens of its tile
    as they are (a partial last K step reads nothing past the row's end)."""
    m, n, r, T = 160, 288, 96, 40
    lin = synth.make_linear(5, m, n, r, T)
    L = DeviceLayer.from_host(lin)
    clean = L.gemm(to_device(lin.x))
    x = lin.x.copy()
    x[7, :] = 0x7F80
    dirty = L.gemm(to_device(x))
    torch.cuda.synchronize()
    keep = [t for t in range(T) if t != 7]
    assert torch.equal(clean[keep], dirty[keep])
