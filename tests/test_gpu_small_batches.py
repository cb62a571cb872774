"""Batches of small images, whose waves hold rays and entries of several of them: each image is that of the item alone,
byte for byte, also where the items share scenes, differ in lights and depth, or have no tree."""
import pytest

import scenegen as sg

from tests.helpers import make_scene, material

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_01530_amd import rt
    rt.lib()
    return torch


def _scenes(n):
    """Small terrains of one to three lights; every fourth is two spheres over a plane, without a tree."""
    from paper_1702_01530_amd.stereo import GpuScene
    out = []
    for i in range(n):
        if i % 4 == 3:
            out.append(GpuScene(make_scene(spheres=[[-1, 1, 6, 1], [1.2, 0.8, 5, 0.8]], planes=[[0, 1, 0, -0.2]],
                                           lights=[[3, 6, 1, 1, 1, 1]], ambient=(0.05,) * 3,
                                           materials=[material(kr=(0.6,) * 3)])))
        else:
            out.append(GpuScene(sg.make_small_terrain(seed=90 + i, grid=10 + i, n_spheres=3, level=1, lights=1 + i % 3)[0]))
    return out


@pytest.mark.parametrize("size,count", [((8, 8), 5), ((8, 8), 70), ((5, 3), 33), ((16, 16), 40), ((40, 24), 12)])
@pytest.mark.parametrize("scenes", [1, 2, 9])
@pytest.mark.parametrize("graph", [False, True])
def test_small_images(torch_cuda, size, count, scenes, graph):
    from paper_1702_01530_amd.stereo import BatchGraph, GpuScene, Workspace, batch_items, batch_outputs, render_batch, \
        render_stereo
    from paper_1702_01530_amd import rt
    torch = torch_cuda
    cam = sg.make_small_terrain(seed=90)[1]
    gs = _scenes(scenes)
    pairs = [(gs[i % scenes], cam.resized(*size).with_(max_depth=(4, 2, 0, 8)[i % 4],
                                                        center=[0.1 * i, 2.5, -4])) for i in range(count)]
    print(f"[small batch] {size} x {count}, {scenes} scenes, graph={graph}", flush=True)
    outs = batch_outputs(pairs)
    ws = Workspace(rt.rt_render_batch_workspace_size(batch_items(pairs, outs)))
    if graph:
        g = BatchGraph(pairs, outs, ws)
        for _ in range(3):
            for o in outs:
                o["radiance"].zero_()
            g.launch(pairs, outs)
        torch.cuda.synchronize()
        g.close()
    else:
        render_batch(pairs, outputs=outs, workspace=ws)
        torch.cuda.synchronize()
    for i, (scene, c) in enumerate(pairs):
        one = render_stereo(scene, c, path_ids=True)
        torch.cuda.synchronize()
        for k in ("radiance", "hit_t", "hit_prim"):
            assert torch.equal(one[k], outs[i][k]), (i, k)
    if not graph:
        assert int(outs[0]["ray_counts"][-1]) == 0
        ids = render_batch(pairs, path_ids=True)
        counted = render_batch(pairs, count_work=True)
        torch.cuda.synchronize()
        assert torch.equal(ids[0]["ray_counts"][:3], counted[0]["ray_counts"][:3])
        for i in range(count):
            assert torch.equal(ids[i]["radiance"], outs[i]["radiance"]), i
            assert torch.equal(counted[i]["radiance"], outs[i]["radiance"]), i
    for s in gs:
        s.close()
