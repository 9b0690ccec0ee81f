"""Runs of one handle on streams: the answers are those of the last run whatever else is still queued, and
a stream that is being captured is refused."""
from __future__ import annotations

import numpy as np
import pytest

import oracle
from paper_1909_05631_amd import sdnn
from tests.gpu_util import GpuNet, log, oracle_run, torch_cuda

pytestmark = pytest.mark.gpu


def small_net(n=256, nl=3, seed=4):
    rng = np.random.default_rng(seed)
    layers = []
    for _ in range(nl):
        src = np.stack([np.sort(rng.choice(n, size=32, replace=False)) for _ in range(n)]).astype(np.int32)
        layers.append((np.arange(n + 1, dtype=np.int64) * 32, src.reshape(-1),
                       rng.uniform(0.02, 0.11, size=src.size).astype(np.float32), np.full(n, -0.3, np.float32)))
    gpu = GpuNet(n, nl)
    for l, layer in enumerate(layers):
        gpu.load(l, *layer)
    return gpu, layers


def inputs(rng, m, n, dead):
    y = rng.random((m, n)).astype(np.float32)
    y[dead] = 0.0
    return y


def test_earlier_run_queued_on_another_stream():
    """A run whose work is still queued on one stream (behind matrix products) ends after a second run of the
    handle on another stream: categories, counts and rows are the second run's."""
    torch = torch_cuda()
    gpu, layers = small_net()
    rng = np.random.default_rng(5)
    m, n = 12, gpu.n
    first, second = inputs(rng, m, n, [0, 1, 2, 3, 4, 5, 6]), inputs(rng, m, n, [3, 9])
    ya, yb = torch.from_numpy(first).cuda(), torch.from_numpy(second).cuda()
    nb = gpu.net.workspace_bytes(m)
    wa, wb = (torch.empty(nb, dtype=torch.uint8, device="cuda") for _ in range(2))
    a = torch.rand(4096, 4096, device="cuda")
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    torch.cuda.synchronize()
    log("two streams, one handle")
    with torch.cuda.stream(sa):
        for _ in range(20):
            a = torch.mm(a, a) * 1e-3
    gpu.net.infer(ya, m, wa, nb, sa)
    gpu.net.infer(yb, m, wb, nb, sb)
    torch.cuda.synchronize()
    o = oracle_run(second, layers)
    cats = gpu.net.categories()
    np.testing.assert_array_equal(cats, o.categories())
    np.testing.assert_array_equal(gpu.net.live_counts(), oracle.padded_live_counts(o, gpu.n_layers))
    np.testing.assert_array_equal(gpu.net.final_rows(cats), o.rows(cats))


def test_captured_stream_is_refused():
    """Categories are read after a wait for the handle's stream, which a replay need not run on: a capturing
    stream is refused before anything is enqueued, and the handle goes on working."""
    torch = torch_cuda()
    gpu, layers = small_net()
    y = inputs(np.random.default_rng(6), 12, gpu.n, [3])
    yd = torch.from_numpy(y).cuda()
    torch.cuda.synchronize()
    log("captured stream")
    with torch.cuda.graph(torch.cuda.CUDAGraph()):
        with pytest.raises(sdnn.SdnnError) as e:
            gpu.net.infer_static(yd, 12, torch.cuda.current_stream())
    assert e.value.name == "SDNN_ESTATE"
    gpu.net.infer_static(yd, 12, torch.cuda.current_stream())
    np.testing.assert_array_equal(gpu.net.categories(), oracle_run(y, layers).categories())
