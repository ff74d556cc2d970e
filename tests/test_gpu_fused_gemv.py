"""The decode forward as one launch (small layers at batch 1): against
the fp64 oracle and bit for bit against the two-launch form, which the
no-allocation entry point runs; workspaces shared by calls of other shapes and
batches in any order, graph replays, and two streams at once."""
import numpy as np
import pytest
import torch

from paper_2609_06161_amd import af1, synth
from paper_2609_06161_amd.layer import DeviceLayer, bf16_bits_to_f64, to_device

pytestmark = pytest.mark.gpu


def nan_out(b, m):
    return torch.full((b, m), 0x7FC0, dtype=torch.int16, device="cuda")


def workspace(L, b):
    return torch.zeros(af1.af1_gemv_workspace_bytes(L.m, L.n, L.r, b), dtype=torch.uint8,
                       device="cuda")


# from one row group and one word (below the sixteen workgroups that the
# one-launch form needs) up to its largest grid (4096^2: 508 workgroups of 512)
# and past it (4096x5120)
@pytest.mark.parametrize("m,n,r", [(32, 32, 32), (128, 64, 96), (224, 32, 32), (480, 1056, 96),
                                   (1024, 1024, 480), (1024, 4096, 800), (2048, 4096, 1344),
                                   (4096, 4096, 2016), (4096, 5120, 2240)])
@pytest.mark.parametrize("b", [1, 2])
def test_one_launch_matches(oracle, m, n, r, b):
    print(f"fused gemv m={m} n={n} r={r} b={b}", flush=True)
    lin = synth.make_linear(m + n + r + b, m, n, r, b)
    L, x = DeviceLayer.from_host(lin), to_device(lin.x)
    ws = workspace(L, b)
    two = nan_out(b, m)
    af1.af1_linear_gemv_noalloc(L.desc, x, b, two)
    for _ in range(5):  # both link buffers, each cleared by the other's call
        y = nan_out(b, m)
        L.gemv(x, y, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, two)
    got = bf16_bits_to_f64(y)
    ref = oracle.forward(m, n, r, lin.Bu, lin.Bv, lin.s_out, lin.s_mid, lin.s_in, lin.x)
    for a, e in zip(got, ref):
        assert np.linalg.norm(a - e) <= 5e-3 * np.linalg.norm(e)


def test_zero_input_and_zero_scales():
    """Zeros in the intermediate are values too: the call must not wait for
    them."""
    lin = synth.make_linear(3, 1024, 1024, 480, 1)
    lin.s_mid[:200] = 0
    L = DeviceLayer.from_host(lin)
    ws = workspace(L, 1)
    for x in (to_device(lin.x), torch.zeros((1, 1024), dtype=torch.int16, device="cuda")):
        two, y = nan_out(1, 1024), nan_out(1, 1024)
        af1.af1_linear_gemv_noalloc(L.desc, x, 1, two)
        L.gemv(x, y, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, two)


def test_shared_workspace_shapes_in_any_order():
    """One workspace for calls of every kind: one launch, two launches, and
    the last-slab reduction, whose counters lie in the same header."""
    shapes = [(2048, 4096, 1344, 1), (1024, 1024, 480, 1), (4096, 4096, 2016, 1), (4096, 4096, 2016, 8),
              (544, 4128, 96, 16), (1024, 4096, 800, 1), (4096, 14336, 3136, 4)]
    cases, need = [], 0
    for i, (m, n, r, b) in enumerate(shapes):
        lin = synth.make_linear(70 + i, m, n, r, b)
        L, x = DeviceLayer.from_host(lin), to_device(lin.x)
        ref = nan_out(b, m)
        L.gemv(x, ref, workspace(L, b))
        cases.append((L, x, b, ref))
        need = max(need, af1.af1_gemv_workspace_bytes(m, n, r, b))
    ws = torch.zeros(need, dtype=torch.uint8, device="cuda")
    order = np.random.default_rng(4).integers(0, len(cases), 60)
    for k in order:
        L, x, b, ref = cases[k]
        y = nan_out(b, L.m)
        L.gemv(x, y, ws)
        torch.cuda.synchronize()
        assert torch.equal(y, ref), shapes[k]


def test_graph_replays():
    lins = [synth.make_linear(90 + i, 1024, 1024, 480, 1) for i in range(3)]
    Ls = [DeviceLayer.from_host(l) for l in lins]
    ws = workspace(Ls[0], 1)
    x = to_device(lins[0].x)
    ys = [nan_out(1, 1024) for _ in Ls]

    def chain():
        h = x
        for L, y in zip(Ls, ys):
            L.gemv(h, y, ws)
            h = y

    chain()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        chain()
    for rep in range(6):
        x.copy_(to_device(synth.make_activations(200 + rep, 1, 1024)))
        for y in ys:
            y.fill_(0x7FC0)
        g.replay()
        torch.cuda.synchronize()
        got = [y.clone() for y in ys]
        chain()
        torch.cuda.synchronize()
        assert all(torch.equal(a, y) for a, y in zip(got, ys))


def test_two_streams_at_once():
    """Calls that overlap in time on workspaces of their own."""
    lins = [synth.make_linear(300 + i, 2048, 4096, 1344, 1) for i in range(2)]
    Ls = [DeviceLayer.from_host(l) for l in lins]
    xs = [to_device(l.x) for l in lins]
    wss = [workspace(L, 1) for L in Ls]
    refs = []
    for L, x in zip(Ls, xs):
        y = nan_out(1, 2048)
        af1.af1_linear_gemv_noalloc(L.desc, x, 1, y)
        refs.append(y)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    outs = [[nan_out(1, 2048) for _ in range(40)] for _ in range(2)]
    torch.cuda.synchronize()
    for k in range(40):
        for i in range(2):
            Ls[i].gemv(xs[i], outs[i][k], wss[i], stream=streams[i])
    torch.cuda.synchronize()
    for i in range(2):
        assert all(torch.equal(y, refs[i]) for y in outs[i])
