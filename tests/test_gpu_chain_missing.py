"""The chained kernel of one image where workgroups do not run, or run late: those that wait for them compute the tasks themselves."""
import numpy as np
import pytest

from paper_1901_05350_amd import inputs
from util import dev, dev16, host

pytestmark = pytest.mark.gpu


def model_of(half, q, size, classes, seed=97):
    import paper_1901_05350_amd as tfx
    make, net, up = (inputs.mobilenet_v1_f16, tfx.MobileNetV1F16, dev16) if half else (inputs.mobilenet_v1, tfx.MobileNetV1, dev)
    d = make(seed=seed, batch=1, image_size=size, width_quarters=q, classes=classes)
    return (lambda: net(d["weights"], batch=1, image_size=size, width_quarters=q)), up(d["image"])


@pytest.mark.parametrize("workgroups", [64, 100, 255])
@pytest.mark.parametrize("half,q,size,classes", [(True, 1, 64, 10), (True, 2, 97, 129), (True, 3, 192, 1000), (True, 4, 224, 1024),
                                                 (False, 1, 65, 1000), (False, 2, 192, 10), (False, 3, 96, 7), (False, 4, 224, 1000)])
def test_workgroups_that_never_run(monkeypatch, half, q, size, classes, workgroups):
    """The same bits: whoever computes a task does it in the same order."""
    make, image = model_of(half, q, size, classes)
    model = make()
    want = [host(t).copy() for t in model.forward(image)]
    assert not np.isnan(want[0]).any()
    monkeypatch.setenv("TFX_CHAIN_WORKGROUPS", str(workgroups))
    got = [host(t).copy() for t in model.forward(image)]
    monkeypatch.delenv("TFX_CHAIN_WORKGROUPS")
    after = [host(t) for t in model.forward(image)]
    for i in range(2):
        assert np.array_equal(got[i], want[i]) and np.array_equal(after[i], want[i])


@pytest.mark.parametrize("half,q,size", [(True, 4, 160), (True, 1, 128), (False, 2, 128)])
def test_replays_and_calls_on_streams(half, q, size):
    """Captured passes replayed on three streams at once, among calls on them: nothing orders them against each other."""
    import torch
    make, image = model_of(half, q, size, 100)
    models = [make() for _ in range(4)]
    want = host(models[0].forward(image)[1]).copy()
    streams = [torch.cuda.Stream() for _ in range(3)]
    graphs, logits = [], []
    for m in models[:3]:
        m.forward(image)
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            logits.append(m.forward(image)[1])
        graphs.append(graph)
    for turn in range(10):
        for l in logits:
            l.zero_()
        torch.cuda.synchronize()
        for _ in range(2):
            for graph, stream in zip(graphs, streams):
                with torch.cuda.stream(stream):
                    graph.replay()
        direct = models[3].forward(image)[1]
        for l in logits + [direct]:
            assert np.array_equal(host(l), want), turn
