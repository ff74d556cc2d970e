"""Decode forward over every count of word groups a wave can own (one to eight,
whole and ragged), in both products, against the fp64 oracle.

A wave takes groups of eight sign words in turn; its loads and matrix products
end at its own count, so each count is another exit of the unrolled code."""
import numpy as np
import pytest

from paper_2609_06161_amd import synth
from paper_2609_06161_amd.layer import DeviceLayer, bf16_bits_to_f64, to_device

pytestmark = pytest.mark.gpu

WAVE_COLS = 8 * 8 * 32  # columns that give each of a workgroup's 8 waves one group


@pytest.mark.parametrize("groups", range(1, 9))
@pytest.mark.parametrize("b", [1, 3, 12])
def test_every_group_count(oracle, groups, b):
    # the same width for n (first product) and r (second), the last group cut
    # to one word, and one word more than a whole count of groups
    for k, width in enumerate((WAVE_COLS * groups, WAVE_COLS * groups - 7 * 32,
                               WAVE_COLS * (groups - 1) + 32)):
        print(f"gemv groups={groups} width={width} b={b}", flush=True)
        for m, n, r in ((96, width, 64), (96, 64, width)):
            lin = synth.make_linear(7000 + 10 * groups + k, m, n, r, b)
            y = bf16_bits_to_f64(DeviceLayer.from_host(lin).gemv(to_device(lin.x)))
            ref = oracle.forward(m, n, r, lin.Bu, lin.Bv, lin.s_out, lin.s_mid, lin.s_in, lin.x)
            # bf16 rounds each output by up to 2^-9; the fp32 sums add far less
            err = np.linalg.norm(y - ref, axis=1) / np.linalg.norm(ref, axis=1)
            assert np.all(err <= 2.0 ** -8), (m, n, r, b, err.max())
