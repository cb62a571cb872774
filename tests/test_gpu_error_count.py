"""RT_COUNT_ERRORS counts the launches that stopped a ray on a consistency check, however many rays and workgroups did:
the root's child references are overwritten with ones past the last node, which the traversal finds before it reads."""
import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def broken():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_01530_amd.stereo import GpuScene
    scene, cam = sg.make_small_terrain(seed=5, grid=20, n_spheres=3, level=1, lights=2, depth=2)
    gs = GpuScene(scene)
    n = gs.info()["num_nodes"]
    torch.cuda.synchronize()
    root = gs._storage[gs.storage_offset:gs.storage_offset + 64].cpu().view(torch.int32)
    assert n > 4 and ((root[4:8] >= 0) & (root[4:8] < n)).any()
    root[4:8] = n + 7  # a reference below 2^31 - 1 and past the last node: checked before it is used
    gs._storage[gs.storage_offset:gs.storage_offset + 64] = root.view(torch.uint8).cuda()
    torch.cuda.synchronize()
    yield torch, gs, cam
    gs.close()


# frames of one launch with a batch for every wave and with several, and of queues
@pytest.mark.parametrize("size", [(33, 21), (256, 256), (480, 360), (1400, 900)])
@pytest.mark.parametrize("ids", [False, True])
def test_one_error_a_frame(broken, size, ids):
    torch, gs, cam = broken
    from paper_1702_01530_amd.stereo import Workspace, alloc_outputs, render_stereo
    cam = cam.resized(*size)
    print(f"[errors] {size} ids={ids}", flush=True)
    ws, out = Workspace.for_camera(cam, gs.num_lights), alloc_outputs(cam, gs.num_lights, gs.device, path_ids=ids)
    for k in range(1, 4):
        render_stereo(gs, cam, workspace=ws, outputs=out, path_ids=ids)
        torch.cuda.synchronize()
        assert int(out["ray_counts"][-1]) == k


@pytest.mark.parametrize("size", [(33, 21), (480, 360)])
def test_one_error_a_replay(broken, size):
    torch, gs, cam = broken
    from paper_1702_01530_amd import rt
    from paper_1702_01530_amd.stereo import alloc_outputs, output_struct, render_stereo
    cam = cam.resized(*size)
    print(f"[errors] captured {size}", flush=True)
    out = alloc_outputs(cam, gs.num_lights, gs.device)
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    camst, st = rt.make_camera_struct(cam), output_struct(out)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=stream):
        rt.rt_render_stereo_noalloc(gs.handle, camst, st, 0, stream.cuda_stream, None)
    for k in range(1, 4):
        graph.replay()
        torch.cuda.synchronize()
        assert int(out["ray_counts"][-1]) == k
        render_stereo(gs, cam)
