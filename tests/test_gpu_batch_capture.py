"""Batch.output recorded into a graph: the batch's stream joins the capture, and
every replay reads the step that was made before it."""
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1408_3526_amd import binding, scenes  # noqa: E402


def test_outputs_recorded_and_replayed():
    g = scenes.grid(-2, 2, 0.5)
    sizes = [(21, 30), (33, 17)]
    fr = [torch.from_numpy(scenes.flow_scene(7 + i, H=H, W=W, T=8, n_targets=1).frames).cuda() for i, (H, W) in enumerate(sizes)]
    b = binding.Batch([dict(H=H, W=W, M=(8, 8, 4), gx=g, gy=g) for H, W in sizes])
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        b.push([f[0] for f in fr])
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            rec = [b.output(i) for i in range(2)]
        for t in range(1, 8):
            b.push([f[t] for f in fr])
            s.wait_stream(b.torch_stream)
            graph.replay()
            got = [[x.clone() for x in r] for r in rec]
            torch.cuda.synchronize()
            for r, i in zip(got, range(2)):
                assert all(torch.equal(x, y) for x, y in zip(r, b.output(i))), (t, i)
            if t > 1:                            # the recorded arrays hold this step's values, not the last one's
                assert not torch.equal(got[0][0], last)
            last = got[0][0]
    torch.cuda.synchronize()
    del rec, graph
    b.close()
