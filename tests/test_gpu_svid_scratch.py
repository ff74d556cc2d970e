"""af1_svid's results do not depend on how large its workspace is: the least
scratch that it accepts (one row of partial sums per 64 rows, where the pass and
the column sums are separate launches), a layer's workspace, and a much larger
one give the same bits."""
import numpy as np
import pytest
import torch

from oracle import nabf as onabf
from paper_2609_06161_amd import nabf
from paper_2609_06161_amd.layer import to_device

pytestmark = pytest.mark.gpu


def least_scratch(rows, cols):
    def al(v):
        return (v + 255) // 256 * 256
    return al((rows + 63) // 64 * cols * 4) + al(cols * 4) + al((cols + 255) // 256 * 4)


# every width class of the row pass; rows for runs of 4, 8, 16 and 32 rows (2048,
# 4096 and 8192 rows are the edges), whole chunks of 64 and ragged ones.  The
# scratches of `rooms` hold one to all of a chunk's runs (96 workgroups and
# more take several runs each there, fewer leave w to the launch of its own).
@pytest.mark.parametrize("rows,cols", [(32, 32), (96, 96), (192, 4576), (352, 2496), (2048, 1024),
                                       (2080, 2048), (2016, 4096), (2112, 5120), (4096, 544), (4128, 32), (8224, 64), (8192, 2080),
                                       (64, 8224),
                                       (96, 16384), (96, 16416), (20000, 32)])
def test_same_bits_for_every_workspace(rows, cols):
    print(f"svid scratch {rows}x{cols}", flush=True)
    rng = np.random.default_rng(rows + cols)
    Z = (rng.standard_normal((rows, cols)) * rng.uniform(0.2, 3.0, (rows, 1))).astype(np.float32)
    Zd = to_device(Z)
    layer = nabf.af1_nabf_workspace_bytes(rows, cols, 32)
    outs = []
    least = least_scratch(rows, cols)
    rooms = [least + n * ((rows + 63) // 64) * cols * 4 for n in (2, 4, 8, 16)]
    for size in (least, least + 4096, *rooms, layer, 2 * layer):
        bits = torch.empty((rows, cols // 32), dtype=torch.int32, device="cuda")
        left = torch.empty(rows, dtype=torch.float32, device="cuda")
        right = torch.empty(cols, dtype=torch.float32, device="cuda")
        ws = torch.full((size,), 0xFF, dtype=torch.uint8, device="cuda")  # NaN patterns
        nabf.af1_svid(Zd, rows, cols, 5, bits, left, right, ws, size)
        outs.append((bits, left, right))
    torch.cuda.synchronize()
    for o in outs[1:]:
        assert all(torch.equal(a, b) for a, b in zip(o, outs[0]))
    rb, ra, rv = onabf.svid(Z, 5)
    for got, ref in ((outs[0][1], ra), (outs[0][2], rv)):
        # fp32 sums of positive terms in trees of at most 64 sequential additions
        g = got.cpu().numpy().astype(np.float64)
        assert np.linalg.norm(g - ref) <= 2e-6 * np.linalg.norm(ref)
    assert np.array_equal(outs[0][0].cpu().numpy().view(np.uint32), rb)
