"""What a caller without ray-tree signatures gets: frames that one launch takes through the whole recursion, and frames by
queues whose traversal adds the lights' terms.  Against the FP64 oracle with the plain frame's own radiance and hits, and
byte for byte against the launches with signatures on scenes of exact ties, boxes without height, spheres and planes
beside a tree, both builders, and every triangle of a tree without it."""
import dataclasses

import numpy as np
import pytest

import scenegen as sg

from tests.helpers import coincident_scene, corners_scene, flat_scene, nested_scene, oracle_sampled
from tests.parity import assert_parity, compare, gpu_flat

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_01530_amd import rt
    rt.lib()
    return torch


def _mixed():
    """A small terrain between mirror planes, with spheres on it, one of them twice."""
    scene, cam = sg.make_small_terrain(seed=13, grid=20, n_spheres=5, level=1, lights=3, depth=4)
    m = scene.materials.shape[0]
    mirror = np.float32([[0.05, 0.05, 0.05, 0, 0, 0, 0.8, 0.8, 0.8, 16]])
    return dataclasses.replace(
        scene, spheres=np.float32([[-2, 1.5, 6, 0.8], [2, 1.2, 9, 1.1], [-2, 1.5, 6, 0.8]]),
        sphere_material=np.uint32([0, m, m]), planes=np.float32([[1, 0, 0, -9], [-1, 0, 0, -9], [0, 0, -1, -30]]),
        plane_material=np.uint32([m, m, m]), materials=np.vstack([scene.materials, mirror])), cam


SCENES = {"coincident": coincident_scene, "flat": flat_scene, "corners": corners_scene, "nested": nested_scene,
          "mixed": _mixed}


@pytest.mark.parametrize("what", sorted(SCENES))
@pytest.mark.parametrize("accel,brute", [("ploc", False), ("karras", False), ("none", False), ("ploc", True),
                                         ("karras", True)])
@pytest.mark.parametrize("size", [(1, 1), (64, 40), (200, 131), (500, 301)])
def test_plain_frames_equal_the_queues(torch_cuda, what, accel, brute, size):
    torch = torch_cuda
    from paper_1702_01530_amd.stereo import GpuScene, render_stereo
    scene, cam = SCENES[what]()
    cam = cam.resized(*size)
    print(f"[plain] {what} {accel} brute={brute} {size}", flush=True)
    gs = GpuScene(scene, accel=accel)
    plain = render_stereo(gs, cam, brute_force=brute)
    ids = render_stereo(gs, cam, path_ids=True, brute_force=brute)
    torch.cuda.synchronize()
    for k in ("radiance", "hit_t", "hit_prim", "ray_counts"):
        assert torch.equal(plain[k], ids[k]), k
    gs.close()


# 1700x1021 with two lights takes the queues, the others one launch
@pytest.mark.parametrize("what,size,samples", [("terrain", (96, 64), None), ("coincident", (48, 32), None),
                                               ("mixed", (64, 48), None), ("spheres", (128, 96), None),
                                               ("terrain", (1700, 1021), 4096)])
def test_plain_frames_against_the_oracle(torch_cuda, what, size, samples):
    torch = torch_cuda
    import oracle
    from paper_1702_01530_amd.stereo import GpuScene, render_stereo
    if what == "terrain":
        scene, cam = sg.make_small_terrain(seed=21, grid=20, n_spheres=4, level=1, lights=2, depth=3)
    elif what == "spheres":
        scene, cam = sg.make_spheres_scene(seed=3)
    else:
        scene, cam = SCENES[what]()
    cam = cam.resized(*size)
    print(f"[plain] oracle {what} {size}", flush=True)
    gs = GpuScene(scene)
    plain, ids = render_stereo(gs, cam), render_stereo(gs, cam, path_ids=True)
    torch.cuda.synchronize()
    gs.close()
    assert int(plain["ray_counts"][-1]) == 0
    g = gpu_flat({**plain, "path_prims": ids["path_prims"], "shadow_state": ids["shadow_state"]})
    orc = oracle.render(scene, cam) if samples is None else oracle_sampled(
        scene, cam, sg.sample_paths(cam, samples, seed=5), say=lambda *a: print(*a, flush=True))
    assert_parity(compare(g, orc, scene=scene, cam=cam))
