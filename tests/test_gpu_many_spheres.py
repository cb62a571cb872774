"""Scenes of many spheres and planes: the kernels that share a walk over them between waves, load several at a time and
stop early, against the walk of one lane per ray (the kernels that count work), byte for byte."""
import numpy as np
import pytest

from tests.helpers import make_scene, material, mono_camera

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_01530_amd import rt
    rt.lib()
    return torch


def _scene(S, P, T, lights=2):
    """Spheres (the last a copy of the first: an exact tie), planes around them (the last a copy of the first) and
    triangles, all mirrors."""
    r = np.random.default_rng([S, P, T])
    balls = np.concatenate([r.uniform((-4, 0, 3), (4, 4, 11), (S, 3)), r.uniform(0.1, 0.7, (S, 1))], 1)
    n = r.normal(size=(P, 3))
    n /= np.linalg.norm(n, axis=1, keepdims=True)
    planes = np.concatenate([n, (n @ [0, 2, 7])[:, None] - r.uniform(6, 20, (P, 1))], 1)
    if S > 1:
        balls[-1] = balls[0]
    if P > 1:
        planes[-1] = planes[0]
    tris = r.uniform((-4, 0, 3), (4, 4, 11), (T, 1, 3)) + r.uniform(-0.4, 0.4, (T, 3, 3))
    where = [[-3, 6, 1], [4, 5, 4], [0, 7, 8], [-5, 3, 9]]
    return make_scene(tris=tris, spheres=balls, sphere_mat=np.arange(S) % 2, planes=planes, plane_mat=np.arange(P) % 2,
                      materials=[material(ks=(0.3,) * 3, kr=(0.5,) * 3), material(kd=(0.7, 0.3, 0.2), kr=(0.4,) * 3)],
                      lights=[p + [0.5] * 3 for p in where[:lights]], ambient=(0.05,) * 3)


def _same(torch, gs, cam, what):
    from paper_1702_01530_amd.stereo import render_stereo
    counted = render_stereo(gs, cam, path_ids=True, count_work=True)
    queues, plain = render_stereo(gs, cam, path_ids=True), render_stereo(gs, cam)
    torch.cuda.synchronize()
    for k in ("radiance", "hit_t", "hit_prim", "path_prims", "shadow_state"):
        assert torch.equal(counted[k], queues[k]), (what, k)
    for k in ("radiance", "hit_t", "hit_prim"):
        assert torch.equal(counted[k], plain[k]), (what, k)
    assert torch.equal(counted["ray_counts"][:3], plain["ray_counts"][:3]) and int(plain["ray_counts"][-1]) == 0, what


# around the loads of four, the steps of 64, the limit of the frames in one launch (256 with two lights) and the sizes
# from which eight waves share a walk (512 in all)
@pytest.mark.parametrize("S,P,T", [(1, 0, 0), (3, 1, 0), (4, 4, 7), (5, 5, 1), (63, 0, 0), (65, 66, 0), (255, 1, 0),
                                   (256, 1, 0), (510, 1, 0), (511, 1, 0), (0, 513, 0), (300, 7, 206), (5, 3, 520),
                                   (700, 130, 600)])
@pytest.mark.parametrize("size", [(1, 1), (33, 21), (130, 97)])
def test_walks_without_a_tree(torch_cuda, S, P, T, size):
    from paper_1702_01530_amd.stereo import GpuScene
    print(f"[spheres] {S} {P} {T} {size}", flush=True)
    gs = GpuScene(_scene(S, P, T), accel="none")
    _same(torch_cuda, gs, mono_camera(center=(0, 2, 0), width=size[0], height=size[1], depth=3, baseline=0.065,
                                      convergence=5.0), (S, P, T, size))
    gs.close()


# beside a tree: around the limit of the frames in one launch (128 in all) and the steps of 64; 180x130 has batches of 8
# rays a wave, 420x400 of 32
@pytest.mark.parametrize("S,P,T", [(1, 0, 2), (5, 4, 40), (64, 0, 40), (65, 63, 300), (66, 63, 300), (300, 70, 2000)])
@pytest.mark.parametrize("size", [(1, 1), (180, 130), (420, 400)])
@pytest.mark.parametrize("accel", ["ploc", "karras"])
def test_walks_beside_a_tree(torch_cuda, S, P, T, size, accel):
    from paper_1702_01530_amd.stereo import GpuScene
    print(f"[spheres] {S} {P} {T} {size} {accel}", flush=True)
    gs = GpuScene(_scene(S, P, T), accel=accel)
    _same(torch_cuda, gs, mono_camera(center=(0, 2, 0), width=size[0], height=size[1], depth=3, baseline=0.065,
                                      convergence=5.0), (S, P, T, size))
    gs.close()


# batches of scenes without a tree, and of both kinds: a batch walks in the traversal's own kernel
@pytest.mark.parametrize("sizes", [[(40, 30)] * 4, [(8, 8)] * 9, [(1, 1), (70, 51), (5, 3), (16, 16)]])
@pytest.mark.parametrize("brute", [False, True])
def test_batches_of_scenes_without_a_tree(torch_cuda, sizes, brute):
    from paper_1702_01530_amd.stereo import GpuScene, render_batch, render_stereo
    torch = torch_cuda
    kinds = [(3, 1, 130, "none"), (70, 2, 0, "none"), (0, 0, 67, "none"), (4, 5, 300, "ploc")]
    scenes = [GpuScene(_scene(*k[:3]), accel=k[3]) for k in kinds]
    pairs = [(scenes[i % 4], mono_camera(center=(0, 2, 0.1 * i), width=w, height=h, depth=i % 4, baseline=0.065,
                                         convergence=5.0)) for i, (w, h) in enumerate(sizes)]
    print(f"[spheres] batch {sizes[:4]} brute={brute}", flush=True)
    outs = render_batch(pairs, brute_force=brute)
    torch.cuda.synchronize()
    for i, (gs, cam) in enumerate(pairs):
        one = render_stereo(gs, cam, path_ids=True, count_work=True)
        torch.cuda.synchronize()
        for k in ("radiance", "hit_t", "hit_prim"):
            assert torch.equal(one[k], outs[i][k]), (i, k)
    for gs in scenes:
        gs.close()
