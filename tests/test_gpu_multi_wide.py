"""Fused projections on rows so long that their LDS decides how many workgroups
share a unit (both forms of the cross-wave sums), against the fp64 oracle."""
import numpy as np
import pytest
import torch

from paper_2609_06161_amd import synth
from paper_2609_06161_amd.layer import DeviceLayer, bf16_bits_to_f64, gemv_multi, to_device

pytestmark = pytest.mark.gpu


# (rank rows summed over the layers: above 256 tiles of 16, 256, and few)
@pytest.mark.parametrize("n", [15648, 15680, 16384])
@pytest.mark.parametrize("shapes", [((544, 3264), (96, 1056)), ((544, 3264), (96, 832)),
                                    ((544, 1056), (96, 96))])
def test_wide_projections(oracle, n, shapes):
    print(f"wide projections n={n} shapes={shapes}", flush=True)
    lins = [synth.make_linear(n + m + r, m, n, r, 1) for m, r in shapes]
    Ls = [DeviceLayer.from_host(l) for l in lins]
    ys = gemv_multi(Ls, to_device(lins[0].x))
    torch.cuda.synchronize()
    for l, y in zip(lins, ys):
        ref = oracle.forward(l.m, l.n, l.r, l.Bu, l.Bv, l.s_out, l.s_mid, l.s_in, lins[0].x)
        err = np.linalg.norm(bf16_bits_to_f64(y) - ref) / np.linalg.norm(ref)
        # bf16 rounds each output by up to 2^-9; the fp32 sums add far less
        assert err <= 2.0 ** -8, (l.m, l.r, err)
