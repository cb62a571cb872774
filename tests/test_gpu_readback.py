"""Readback of both eyes as one copy, where they lie side by side in one allocation on the device and on the host, and as
two where they do not: the host's bytes are the device's, also in a captured graph's replays."""
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_01530_amd import rt
    rt.lib()
    return torch


def _pair(torch, shape, layout, **kw):
    """The two eyes' buffers: side by side, the right eye first, with a gap of one pixel, or two allocations."""
    if layout == "apart":
        return [torch.zeros(shape, dtype=torch.float32, **kw) for _ in range(2)]
    n = shape[0] * shape[1] * 3
    flat = torch.zeros(2 * n + 3, dtype=torch.float32, **kw)
    first, second = flat[:n].view(shape), (flat[n + 3:] if layout == "gap" else flat[n:2 * n]).view(shape)
    return [second, first] if layout == "swapped" else [first, second]


@pytest.mark.parametrize("size", [(1, 1), (33, 21), (160, 90)])
@pytest.mark.parametrize("device,host", [("together", "together"), ("apart", "together"), ("together", "apart"),
                                         ("swapped", "swapped"), ("gap", "together"), ("gap", "gap"),
                                         ("together", "swapped")])
@pytest.mark.parametrize("captured", [False, True])
def test_readback_of_eyes_side_by_side_or_not(torch_cuda, size, device, host, captured):
    torch = torch_cuda
    from paper_1702_01530_amd import rt
    from paper_1702_01530_amd.stereo import GpuScene, alloc_outputs, output_struct, render_stereo
    scene, cam = sg.make_small_terrain(seed=5, grid=12, n_spheres=3, level=1, lights=2, depth=2)
    cam = cam.resized(*size)
    gs = GpuScene(scene)
    print(f"[readback] {size} {device} {host} captured={captured}", flush=True)
    ref = render_stereo(gs, cam)
    torch.cuda.synchronize()
    out = alloc_outputs(cam, gs.num_lights, gs.device, counts=False)
    shape = (size[1], size[0], 3)
    out["radiance"] = _pair(torch, shape, device, device="cuda")
    out["host_radiance"] = _pair(torch, shape, host, pin_memory=True)
    st, camst, s = output_struct(out), rt.make_camera_struct(cam), torch.cuda.Stream()
    rt.rt_render_stereo_noalloc(gs.handle, camst, st, 0, s.cuda_stream, None)
    s.synchronize()
    graph = None
    if captured:
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=s):
            rt.rt_render_stereo_noalloc(gs.handle, camst, st, 0, s.cuda_stream, None)
    for _ in range(3 if captured else 1):
        if captured:
            for h in out["host_radiance"]:
                h.fill_(-7.0)
            render_stereo(gs, cam)  # eager work between replays
            torch.cuda.synchronize()
            graph.replay()
            torch.cuda.synchronize()
        for eye in range(2):
            assert torch.equal(out["radiance"][eye], ref["radiance"][eye])
            assert torch.equal(out["host_radiance"][eye], ref["radiance"][eye].cpu())
    del graph
    gs.close()
