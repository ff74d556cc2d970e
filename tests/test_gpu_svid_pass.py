"""The fused SVID pass and the surrogate's column statistics at the edges of
their tiles, against the fp64 oracle.

Bars: the signs bit-exact; left, right and the RMS vectors within 2e-6
relative: fp32 sums of up to 2^14 positive terms taken in trees no deeper than
64 sequential additions, whose error is below 64 * 2^-24 = 3.8e-6 in the worst
case and about its square root's share of that (5e-7) in practice."""
import numpy as np
import pytest
import torch

from oracle import nabf as onabf
from paper_2609_06161_amd import nabf, synth
from paper_2609_06161_amd.layer import bf16_bits_to_f64, to_device

pytestmark = pytest.mark.gpu


def rel(t, e):
    a = t.cpu().numpy().astype(np.float64)
    return float(np.linalg.norm(a - e) / max(np.linalg.norm(e), 1e-300))


# every width class of the register tile (1024, 2048, 4096, 8192, 16384
# columns), one float4 group below and above each edge, the wide path past
# the last; rows below, at and past a workgroup's block
@pytest.mark.parametrize("rows,cols", [(32, 32), (32, 1024), (96, 1056), (160, 2048), (64, 2080),
                                       (2080, 4096), (96, 4128), (64, 8192), (96, 8224),
                                       (32, 16384), (32, 16416), (4128, 96)])
@pytest.mark.parametrize("iters", [0, 1, 7])
@pytest.mark.parametrize("roomy", [False, True])
def test_svid_pass(rows, cols, iters, roomy):
    print(f"svid {rows}x{cols} iters={iters} roomy={roomy}", flush=True)
    rng = np.random.default_rng(rows * 7 + cols + iters)
    Z = (rng.standard_normal((rows, cols)) * rng.uniform(0.2, 3.0, (rows, 1))).astype(np.float32)
    Z[0, 0], Z[-1, -1] = -0.0, -1.5
    bits = torch.empty((rows, cols // 32), dtype=torch.int32, device="cuda")
    left = torch.empty(rows, dtype=torch.float32, device="cuda")
    right = torch.empty(cols, dtype=torch.float32, device="cuda")
    # the scratch of the entry point alone (64-row partial sums), or a
    # layer's workspace
    al = lambda v: (v + 255) // 256 * 256
    need = (al((rows + 63) // 64 * cols * 4) + al(cols * 4) + al((cols + 255) // 256 * 4))
    ws = torch.empty(need if not roomy else nabf.af1_nabf_workspace_bytes(rows, cols, 64),
                     dtype=torch.uint8, device="cuda")
    nabf.af1_svid(to_device(Z), rows, cols, iters, bits, left, right, ws, ws.numel())
    torch.cuda.synchronize()
    rb, ra, rv = onabf.svid(Z, iters)
    assert np.array_equal(bits.cpu().numpy().view(np.uint32), rb)
    assert rel(left, ra) < 2e-6 and rel(right, rv) < 2e-6


def test_svid_zero_matrix_keeps_the_right_vector():
    rows, cols = 96, 1056
    Z = torch.zeros((rows, cols), dtype=torch.float32, device="cuda")
    bits = torch.empty((rows, cols // 32), dtype=torch.int32, device="cuda")
    left = torch.empty(rows, dtype=torch.float32, device="cuda")
    right = torch.empty(cols, dtype=torch.float32, device="cuda")
    ws = torch.empty(nabf.af1_nabf_workspace_bytes(rows, cols, 64), dtype=torch.uint8,
                     device="cuda")
    nabf.af1_svid(Z, rows, cols, 3, bits, left, right, ws, ws.numel())
    torch.cuda.synchronize()
    assert not bits.any() and not left.any()
    assert torch.equal(right, torch.full_like(right, np.float32(1.0 / np.sqrt(np.float32(cols)))))


@pytest.mark.parametrize("m,n,T", [(32, 32, 1), (288, 544, 63), (256, 1056, 65), (4128, 224, 200),
                                   (64, 96, 1100)])
def test_surrogate_edges(m, n, T):
    print(f"surrogate {m}x{n} T={T}", flush=True)
    rng = np.random.default_rng(m + n + T)
    W = rng.standard_normal((m, n)).astype(np.float32)
    X, G = synth.make_activations(2, T, n), synth.make_output_grad(3, T, m)
    Wp = torch.empty((m, n), dtype=torch.float32, device="cuda")
    i = torch.empty(n, dtype=torch.float32, device="cuda")
    o = torch.empty(m, dtype=torch.float32, device="cuda")
    ws = torch.empty(nabf.af1_nabf_workspace_bytes(m, n, 32, T), dtype=torch.uint8, device="cuda")
    nabf.af1_nabf_surrogate(to_device(W), m, n, to_device(X), to_device(G), T, Wp, i, o, ws,
                            ws.numel())
    torch.cuda.synchronize()
    f64 = lambda a: bf16_bits_to_f64(torch.from_numpy(a.view(np.int16)))
    rWp, ri, ro = onabf.surrogate(W, f64(X), f64(G))
    assert rel(i, ri) < 2e-6 and rel(o, ro) < 2e-6 and rel(Wp, rWp) < 2e-6
