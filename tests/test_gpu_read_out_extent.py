"""Results read into arrays that are too small for them: refused, as a copy is,
whether one array is asked for or several (which share a launch)."""
import ctypes

import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

from paper_1408_3526_amd import binding, scenes  # noqa: E402

H, W = 64, 64
N = H * W


class DeviceArray:
    """An allocation of its own (not from torch's pools), filled with 0x55."""

    def __init__(self, nbytes):
        self.hip = ctypes.CDLL("libamdhip64.so")
        self.hip.hipMalloc.argtypes = [ctypes.c_void_p, ctypes.c_size_t]
        self.hip.hipFree.argtypes = [ctypes.c_void_p]
        self.hip.hipMemset.argtypes = [ctypes.c_void_p, ctypes.c_int, ctypes.c_size_t]
        self.hip.hipMemcpy.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_int]
        p = ctypes.c_void_p()
        assert self.hip.hipMalloc(ctypes.byref(p), nbytes) == 0
        self.p, self.nbytes = p.value, nbytes
        assert self.hip.hipMemset(self.p, 0x55, nbytes) == 0

    def host(self):
        a = np.empty(self.nbytes, np.uint8)
        torch.cuda.synchronize()
        assert self.hip.hipMemcpy(a.ctypes.data, self.p, self.nbytes, 2) == 0
        return a

    def free(self):
        torch.cuda.synchronize()
        assert self.hip.hipFree(self.p) == 0


# (each short array's last page is mapped to its end, whatever its size)
@pytest.mark.parametrize("short", ["vxy", "idx"])
@pytest.mark.parametrize("inside", [0, 4096])
def test_a_short_velocity_array_is_refused(short, inside):
    g = scenes.grid(-2, 2, 0.5)
    f = binding.Filter(H, W, 8, 8, 4, g, g)
    f.push_frame(torch.randn(H, W, device="cuda"))
    L = binding.lib()
    v = DeviceArray(inside + 8 * N - (64 if short == "vxy" else 0))
    i = DeviceArray(inside + 4 * N - (64 if short == "idx" else 0))
    bad = v if short == "vxy" else i
    one = [v.p + inside, None] if short == "vxy" else [None, i.p + inside]
    assert L.rmdf_velocity(f.ctx, *one) == binding.RMDF_E_DEVICE
    assert L.rmdf_velocity(f.ctx, v.p + inside, i.p + inside) == binding.RMDF_E_DEVICE
    assert (bad.host() == 0x55).all()
    f.velocity()                                 # the context goes on
    f.push_frame(torch.zeros(H, W, device="cuda"))
    v.free()
    i.free()
    f.close()


@pytest.mark.parametrize("short", [0, 1, 2])
def test_a_short_batch_output_is_refused(short):
    g = scenes.grid(-2, 2, 0.5)
    b = binding.Batch([dict(H=H, W=W, M=(8, 8, 4), gx=g, gy=g)])
    b.push([torch.randn(H, W, device="cuda")])
    a = [DeviceArray(k * N - (64 if q == short else 0)) for q, k in enumerate((4, 8, 4))]
    assert binding.lib().rmdf_batch_output(b.b, 0, *(x.p for x in a)) == binding.RMDF_E_DEVICE
    assert (a[short].host() == 0x55).all()
    b.output(0)
    for x in a:
        x.free()
    b.close()


@pytest.mark.parametrize("shift", [0, 1, N - 1, 2 * N - 1, -1, 1 - N])
def test_overlapping_arrays_hold_the_index(shift):
    """An index array that shares memory with the velocity array: the index is
    written after the velocities."""
    g = scenes.grid(-2, 2, 0.5)
    f = binding.Filter(H, W, 8, 8, 4, g, g)
    for _ in range(5):
        f.push_frame(torch.randn(H, W, device="cuda") * 10)
    v, i = (x.reshape(-1) for x in f.velocity())
    buf = torch.zeros(4 * N, device="cuda")
    want = buf.clone()
    want[N:3 * N] = v
    want[N + shift:2 * N + shift] = i.view(torch.float32)
    f.velocity(buf[N:3 * N], buf.view(torch.int32)[N + shift:2 * N + shift])
    assert torch.equal(buf.view(torch.int32), want.view(torch.int32))
    f.close()


def test_an_error_left_by_another_call_is_not_reported():
    """HIP keeps the status of a program's last failed call until it is asked for."""
    g = scenes.grid(-2, 2, 0.5)
    f = binding.Filter(H, W, 8, 8, 4, g, g)
    f.push_frame(torch.randn(H, W, device="cuda"))
    want = f.velocity()
    v, i = torch.empty(H, W, 2, device="cuda"), torch.empty(H, W, dtype=torch.int32, device="cuda")
    torch.cuda.synchronize()
    hip = ctypes.CDLL("libamdhip64.so")
    assert hip.hipMemcpy(None, None, ctypes.c_size_t(16), 3) != 0      # refused for its NULL arguments
    st = binding.lib().rmdf_velocity(f.ctx, v.data_ptr(), i.data_ptr())
    hip.hipGetLastError()
    assert st == binding.RMDF_OK
    assert torch.equal(v, want[0]) and torch.equal(i, want[1])
    f.close()


@pytest.mark.parametrize("mode", ["global", "thread_local", "relaxed"])
def test_velocity_under_each_capture_mode(mode):
    """The arrays are looked up while their stream captures: the graph gives each
    frame's results."""
    g = scenes.grid(-2, 2, 0.5)
    fr = torch.from_numpy(scenes.flow_scene(4, H=21, W=30, T=6, n_targets=1).frames).cuda()
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    f = binding.Filter(21, 30, 8, 8, 4, g, g, stream=s.cuda_stream)
    v, i = torch.empty(21, 30, 2, device="cuda"), torch.empty(21, 30, dtype=torch.int32, device="cuda")
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        f.push_frame(fr[0])
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=s, capture_error_mode=mode):
            f.velocity(v, i)
        for t in range(1, 6):
            f.push_frame(fr[t])
            graph.replay()
            a, b = v.clone(), i.clone()
            c, d = f.velocity()
            assert torch.equal(a, c) and torch.equal(b, d), t
    torch.cuda.synchronize()
    f.close()
