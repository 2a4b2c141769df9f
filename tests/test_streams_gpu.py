"""GPU tests of calls that overlap in time: those that share no workspace by the library's own query may run side by side."""
import pytest

import workloads
from tests.util import to_device, upload

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def rl():
    import paper_2405_05751_amd as pkg
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return pkg


def _linear(rl, M, K, N, dtype, seed):
    w = workloads.make(M, K, N, dtype, 1e-5, seed)
    X, g, W = upload(w)
    assert rl.rl_workspace_bytes(M, K, N, X.dtype) == 0
    return lambda Y: rl.rmsnorm_linear(X, g, W, w.eps, Y)


def _attention(rl, B, H, S, D, dtype, seed):
    c = workloads.make_attention(B, H, S, D, dtype, seed)
    t = [to_device(c[k], dtype) for k in ("Q", "K", "V", "gq", "bq", "gk", "bk")]
    return lambda O: rl.rl_qknorm_attention(*t, 1e-5, O)


CALLS = {
    "odd sizes, split": (_linear, (8, 4095, 3001, "bf16"), (8, 3001)),
    "odd sizes, f16": (_linear, (40, 1001, 2050, "f16"), (40, 2050)),
    "X-hat in a kernel of its own": (_linear, (300, 1024, 10000, "bf16"), (300, 10000)),
    "X-hat formed by the tiles": (_linear, (654, 2392, 4352, "f16"), (654, 4352)),
    "row blocks": (_linear, (509, 512, 1024, "bf16"), (509, 1024)),
    "attention, many heads": (_attention, (8, 40, 700, 128, "bf16"), (8, 40, 128)),
    "attention, short sequence": (_attention, (1, 32, 300, 128, "f16"), (1, 32, 128)),
}


@pytest.mark.parametrize("what", CALLS)
def test_two_streams_and_a_graph(rl, what):
    """The same shape with other inputs on two streams, a replayed graph of a third call beside them: every result is, bit for
    bit, what the call gives by itself (the captured one what it gives in a graph by itself)."""
    import torch
    make, args, shape = CALLS[what]
    dt = {"bf16": torch.bfloat16, "f16": torch.float16}[args[-1]]
    calls = [make(rl, *args, 7100 + i) for i in range(3)]
    out = [[torch.empty(shape, dtype=dt, device="cuda") for _ in range(12)] for _ in calls]
    streams = [torch.cuda.Stream() for _ in calls]
    want = []
    for i in range(2):
        with torch.cuda.stream(streams[i]):
            calls[i](out[i][0])
        torch.cuda.synchronize()
        want.append(out[i][0].clone())
    calls[2](out[2][0])
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        for Y in out[2]:
            calls[2](Y)
    graph.replay()
    torch.cuda.synchronize()
    want.append(out[2][0].clone())
    for i in range(3):
        for Y in out[i]:
            Y.zero_()
    torch.cuda.synchronize()
    with torch.cuda.stream(streams[2]):
        graph.replay()
    for n in range(12):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                calls[i](out[i][n])
    torch.cuda.synchronize()
    for i in range(3):
        for n, Y in enumerate(out[i]):
            assert torch.equal(Y, want[i]), (what, i, n)
