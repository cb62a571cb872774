"""The traversal's wave-wide ray sharing (a wave with few rays left spreads their stacks over its idle lanes) against
brute force and against one-at-a-time renders, byte for byte: the closest hit and a shadow ray's answer do not depend
on which lane visits a node, or in which order."""
import pytest

import scenegen as sg

from tests.helpers import coincident_scene, corners_scene, flat_scene

pytestmark = pytest.mark.gpu

KEYS = ("radiance", "hit_t", "hit_prim", "path_prims", "shadow_state")


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_01530_amd import rt
    rt.lib()
    return torch


def _same(torch, a, b, what):
    for k in KEYS:
        assert torch.equal(a[k], b[k]), (what, k)
    assert torch.equal(a["ray_counts"][:3], b["ray_counts"][:3]) and int(b["ray_counts"][-1]) == 0, what


# Paths per frame around the sizes where a launch's batches go from 8 to 16, 32 and 64 rays (8 x, 16 x and 32 x the
# 8,192 waves of a full grid), and down to a single path of each eye.
@pytest.mark.parametrize("size", [(1, 1), (3, 2), (8, 8), (17, 9), (179, 183), (181, 181), (255, 257), (363, 361), (420, 400)])
def test_every_batch_width_equals_brute_force(torch_cuda, size):
    torch = torch_cuda
    from paper_1702_01530_amd.stereo import GpuScene, render_stereo
    scene, cam = sg.make_small_terrain(seed=31, grid=18, n_spheres=5, level=1, lights=4, depth=4)
    cam = cam.resized(*size)
    print(f"[shared rays] {size}", flush=True)
    gs = GpuScene(scene)
    tree, brute = render_stereo(gs, cam, path_ids=True), render_stereo(gs, cam, path_ids=True, brute_force=True)
    torch.cuda.synchronize()
    _same(torch, brute, tree, size)
    # the kernels that count work trace one lane per ray
    counted = render_stereo(gs, cam, path_ids=True, count_work=True)
    torch.cuda.synchronize()
    _same(torch, brute, counted, size)
    gs.close()


# Exact ties in t (the smaller id wins, whichever lane reaches it), zero-area triangles, boxes without height, grazing
# and axis-parallel rays.
@pytest.mark.parametrize("make", [coincident_scene, flat_scene, corners_scene])
@pytest.mark.parametrize("size", [(48, 32), (190, 181)])
def test_ties_and_flat_boxes_equal_brute_force(torch_cuda, make, size):
    torch = torch_cuda
    from paper_1702_01530_amd.stereo import GpuScene, render_stereo
    scene, cam = make()
    cam = cam.resized(*size)
    print(f"[shared rays] {make.__name__} {size}", flush=True)
    gs = GpuScene(scene)
    tree, brute = render_stereo(gs, cam, path_ids=True), render_stereo(gs, cam, path_ids=True, brute_force=True)
    torch.cuda.synchronize()
    _same(torch, brute, tree, make.__name__)
    gs.close()


def test_waves_that_hold_several_items(torch_cuda):
    """A batch of tiny images: from the first mirror bounce on, one wave's rays belong to several items (and scenes),
    which it traverses one after the other."""
    torch = torch_cuda
    from paper_1702_01530_amd.stereo import GpuScene, render_batch, render_stereo
    scenes = [sg.make_small_terrain(seed=40 + k, grid=10 + 3 * k, n_spheres=2 + k, level=1, lights=1 + k % 4, depth=3)
              for k in range(4)] + [sg.make_spheres_scene(seed=9)]
    built = [GpuScene(s) for s, _ in scenes]
    pairs = [(built[i % 5], scenes[i % 5][1].with_(width=5 + i % 9, height=11 - i % 7, max_depth=1 + i % 4)) for i in range(40)]
    print("[shared rays] batch of 40", flush=True)
    outs = render_batch(pairs, path_ids=True)
    torch.cuda.synchronize()
    for i, (gs, cam) in enumerate(pairs):
        one = render_stereo(gs, cam, path_ids=True)
        torch.cuda.synchronize()
        for k in KEYS:
            assert torch.equal(one[k], outs[i][k]), (i, k)
    for gs in built:
        gs.close()


def _flat(n):
    """n triangles and no tree."""
    scene, cam = sg.make_small_terrain(seed=50, grid=18, n_spheres=2, level=1, lights=2, depth=3)
    from dataclasses import replace
    return replace(scene, triangles=scene.triangles[-n:], tri_material=scene.tri_material[-n:]), cam


# Frames that one launch takes through the whole recursion against the queue kernels (which frames with ray-tree
# signatures take): sizes around every batch width, no light to eight, no mirror to eight, no tree and no triangle.
@pytest.mark.parametrize("size", [(1, 1), (3, 2), (17, 9), (181, 181), (255, 257), (420, 400)])
@pytest.mark.parametrize("lights,depth", [(0, 2), (1, 0), (4, 4), (8, 8)])
@pytest.mark.parametrize("what", ["tree", "spheres", "flat256", "flat257"])
def test_whole_paths_equal_the_queues(torch_cuda, what, lights, depth, size):
    torch = torch_cuda
    from paper_1702_01530_amd.stereo import GpuScene, render_stereo
    if what == "tree":
        scene, cam = sg.make_small_terrain(seed=33, grid=18, n_spheres=5, level=1)
    elif what == "spheres":
        scene, cam = sg.make_spheres_scene(seed=3)
    else:
        scene, cam = _flat(int(what[4:]))
    all_lights = [[-6, 8, 2], [6, 6, 12], [-3, 9, 9], [5, 7, 3], [0, 8, 5], [-7, 5, 11], [3, 4, 14], [0.5, 3, -2]]
    scene = scene.with_lights([p + [0.4, 0.4, 0.4] for p in all_lights[:lights]])
    cam = cam.resized(*size).with_(max_depth=depth)
    print(f"[whole paths] {what} L={lights} D={depth} {size}", flush=True)
    gs = GpuScene(scene, accel="none" if what.startswith("flat") else "ploc")
    one, queues = render_stereo(gs, cam), render_stereo(gs, cam, path_ids=True)
    torch.cuda.synchronize()
    for k in ("radiance", "hit_t", "hit_prim", "ray_counts"):
        assert torch.equal(one[k], queues[k]), k
    gs.close()


# A batch of scenes with no light to eight, cut into passes in the middle of items: the queues' layout (entries, light
# arrays, eye positions) against each image in one launch.
@pytest.mark.parametrize("max_pass_paths", [4096, 4992, 1 << 25])
def test_batch_passes_equal_whole_paths(torch_cuda, max_pass_paths):
    torch = torch_cuda
    from paper_1702_01530_amd import rt
    from paper_1702_01530_amd.stereo import GpuScene, render_batch, render_stereo
    all_lights = [[-6, 8, 2], [6, 6, 12], [-3, 9, 9], [5, 7, 3], [0, 8, 5], [-7, 5, 11], [3, 4, 14], [0.5, 3, -2]]
    pairs = []
    for i, n in enumerate((0, 8, 1, 5)):
        scene, cam = sg.make_small_terrain(seed=60 + i, grid=12, n_spheres=4, level=1)
        scene = scene.with_lights([p + [0.4, 0.4, 0.4] for p in all_lights[:n]])
        pairs.append((GpuScene(scene), cam.resized(61 + 6 * i, 43 - 5 * i).with_(max_depth=i + 1)))
    print(f"[batch passes] {max_pass_paths}", flush=True)
    saved = rt.rt_get_tuning()
    rt.rt_set_tuning(**{**saved, "max_pass_paths": max_pass_paths})
    try:
        outs = render_batch(pairs)
        torch.cuda.synchronize()
    finally:
        rt.rt_set_tuning(**saved)
    for i, (gs, cam) in enumerate(pairs):
        one = render_stereo(gs, cam)
        torch.cuda.synchronize()
        for k in ("radiance", "hit_t", "hit_prim"):
            assert torch.equal(one[k], outs[i][k]), (i, k)
    for gs, _ in pairs:
        gs.close()


@pytest.mark.parametrize("size", [(480, 360), (720, 560)])
@pytest.mark.parametrize("what", ["tree", "flat256"])
def test_whole_paths_in_several_batches_equal_the_queues(torch_cuda, what, size):
    """Frames of more batches than waves run at once, which take them one by one: of 32 paths and of 64."""
    torch = torch_cuda
    from paper_1702_01530_amd.stereo import GpuScene, render_stereo
    scene, cam = sg.make_small_terrain(seed=33, grid=18, n_spheres=5, level=1, lights=2) if what == "tree" else _flat(256)
    cam = cam.resized(*size).with_(max_depth=3)
    print(f"[whole paths] {what} {size}", flush=True)
    gs = GpuScene(scene, accel="ploc" if what == "tree" else "none")
    queues = render_stereo(gs, cam, path_ids=True)
    for _ in range(2):  # the counters of the first launch are no concern of the second
        one = render_stereo(gs, cam)
        torch.cuda.synchronize()
        for k in ("radiance", "hit_t", "hit_prim", "ray_counts"):
            assert torch.equal(one[k], queues[k]), k
    gs.close()


@pytest.mark.parametrize("lights,depth", [(1, 0), (4, 1), (8, 2), (2, 5)])
def test_terms_added_by_the_traversal_equal_the_launches(torch_cuda, lights, depth):
    """Frames by queues: the traversal of depth d adds the lights' terms of depth d - 2, but not with ray-tree signatures
    or the timer, whose frames take launches of their own for them."""
    torch = torch_cuda
    from paper_1702_01530_amd.stereo import GpuScene, render_stereo
    scene, cam = sg.make_small_terrain(seed=33, grid=18, n_spheres=5, level=1)
    all_lights = [[-6, 8, 2], [6, 6, 12], [-3, 9, 9], [5, 7, 3], [0, 8, 5], [-7, 5, 11], [3, 4, 14], [0.5, 3, -2]]
    scene = scene.with_lights([p + [0.4, 0.4, 0.4] for p in all_lights[:lights]])
    cam = cam.resized(1700, 1021).with_(max_depth=depth)
    print(f"[queues] L={lights} D={depth}", flush=True)
    gs = GpuScene(scene)
    one, ids, counted = (render_stereo(gs, cam, **kw) for kw in ({}, {"path_ids": True}, {"count_work": True}))
    torch.cuda.synchronize()
    for k in ("radiance", "hit_t", "hit_prim"):
        assert torch.equal(one[k], ids[k]) and torch.equal(one[k], counted[k]), k
    assert torch.equal(one["ray_counts"][:3], ids["ray_counts"][:3])
    gs.close()
