"""A frame's results copied out by one launch: odd sizes, destinations aligned to
4 bytes only, nothing written beside them, destinations in host memory (which
take the copies of their own), outputs of a batch on the caller's stream."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1408_3526_amd import binding, scenes  # noqa: E402


@pytest.mark.parametrize("H,W", [(1, 1), (3, 5), (5, 13), (16, 64), (33, 47)])
@pytest.mark.parametrize("off", [0, 1, 2, 3, 4])
def test_velocity_into_views(H, W, off):
    g = scenes.grid(-2, 2, 0.5)
    f = binding.Filter(H, W, 8, 8, 4, g, g)
    rng = np.random.default_rng(H * W)
    fr = torch.from_numpy((rng.normal(size=(5, H, W)) * 10).astype(np.float32)).cuda()
    for t in range(5):
        f.push_frame(fr[t])
    n = H * W
    vx, ix = torch.empty(2 * n, device="cuda"), torch.empty(n, dtype=torch.int32, device="cuda")
    L = binding.lib()
    assert L.rmdf_velocity(f.ctx, vx.data_ptr(), None) == 0 and L.rmdf_velocity(f.ctx, None, ix.data_ptr()) == 0
    bv = torch.full((2 * n + 12,), -7.0, device="cuda")
    bi = torch.full((n + 12,), -7, dtype=torch.int32, device="cuda")
    f.velocity(bv[off:off + 2 * n], bi[off:off + n])
    assert torch.equal(bv[off:off + 2 * n], vx) and torch.equal(bi[off:off + n], ix)
    assert bool((bv[:off] == -7).all()) and bool((bv[off + 2 * n:] == -7).all())
    assert bool((bi[:off] == -7).all()) and bool((bi[off + n:] == -7).all())
    hv, hi = torch.empty(2 * n).pin_memory(), torch.empty(n, dtype=torch.int32).pin_memory()
    assert L.rmdf_velocity(f.ctx, ctypes.c_void_p(hv.data_ptr()), ctypes.c_void_p(hi.data_ptr())) == 0
    torch.cuda.synchronize()
    assert torch.equal(hv, vx.cpu()) and torch.equal(hi, ix.cpu())
    f.close()


def test_batch_outputs_are_ordered_with_the_callers_stream():
    """Outputs read on a stream of the caller's, their memory given back and taken
    again between steps: every step's values are those of the stream alone."""
    H, W, T = 40, 56, 8
    g = scenes.grid(-2, 2, 0.5)
    fr = [torch.from_numpy(scenes.flow_scene(s, H=H, W=W, T=T, n_targets=1).frames).cuda() for s in range(3)]
    b = binding.Batch([dict(H=H, W=W, M=(8, 8, 4), gx=g, gy=g)] * 3)
    fs = [binding.Filter(H, W, 8, 8, 4, g, g) for _ in range(3)]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    got = []
    with torch.cuda.stream(side):
        for t in range(T):
            b.push([f[t] for f in fr])
            got.append([torch.cat([o.reshape(-1).double() for o in b.output(s)]) for s in range(3)])
    torch.cuda.current_stream().wait_stream(side)
    for t in range(T):
        for s in range(3):
            fs[s].push_frame(fr[s][t])
            v, i = fs[s].velocity()
            assert torch.equal(got[t][s], torch.cat([o.reshape(-1).double() for o in (fs[s].output(), v, i)])), (t, s)
    for f in fs:
        f.close()
    b.close()


def test_velocity_under_capture():
    """A captured read-out, replayed between frames pushed outside the graph,
    gives each frame's velocity and index."""
    H, W, T = 21, 30, 6
    g = scenes.grid(-2, 2, 0.5)
    fr = torch.from_numpy(scenes.flow_scene(4, H=H, W=W, T=T, n_targets=1).frames).cuda()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    f = binding.Filter(H, W, 8, 8, 4, g, g, stream=s.cuda_stream)
    v, i = torch.empty(H, W, 2, device="cuda"), torch.empty(H, W, dtype=torch.int32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        f.push_frame(fr[0])
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s):
            f.velocity(v, i)
        for t in range(1, T):
            f.push_frame(fr[t])
            graph.replay()
            a, b = (x.clone() for x in (v, i))
            c, d = f.velocity()
            assert torch.equal(a, c) and torch.equal(b, d), t
    torch.cuda.synchronize()
    f.close()
