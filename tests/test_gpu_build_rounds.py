"""The tree build at the sizes where its steps change hands: the clustering's rounds go from many workgroups to one at
1,024 clusters, a level of the collapse at 1,024 nodes, and a search or sort tile ends at a few hundred or thousand
triangles.  Each tree is walked: every node and triangle is reached once, levels are contiguous, every child's box (as
the traversal reads it) contains the triangles under it; and a frame equals brute force, byte for byte."""
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


def _soup(n, kind):
    r = np.random.default_rng(n)
    c = {"uniform": lambda: r.uniform(-4, 4, (n, 1, 3)), "grid": lambda: np.round(r.uniform(-4, 4, (n, 1, 3))),
         "same": lambda: np.zeros((n, 1, 3)),
         "line": lambda: np.stack([np.linspace(-4, 4, n)[:, None], np.zeros((n, 1)), np.zeros((n, 1))], -1),
         "grow": lambda: np.stack([1.0005 ** np.arange(n)[:, None], np.zeros((n, 1)), np.zeros((n, 1))], -1)}[kind]()
    d = r.uniform(-0.4, 0.4, (1 if kind == "same" else n, 3, 3))
    return make_scene(tris=c + [0, 0, 6] + d, lights=[[1, 5, -2, 1, 1, 1]], ambient=(0.05,) * 3,
                      materials=[material(kr=(0.5, 0.5, 0.5))])


def _walk(gs, T, tris):
    info = gs.info()
    n = info["num_nodes"]
    raw = gs._storage[gs.storage_offset:].cpu().numpy()
    u = raw[:64 * n].view(np.uint32).reshape(n, 16)
    f = u.view(np.float32)
    rec = raw[-(-64 * (T - 1) // 256) * 256:][:48 * T].view(np.int32).reshape(T, 12)[:, 3]
    assert np.array_equal(np.sort(rec), np.arange(T))
    lo, hi = tris[rec].astype(np.float64).min(1), tris[rec].astype(np.float64).max(1)
    step = np.stack([f[:, 3], f[:, 14], f[:, 15]], 1).astype(np.float64) / 2.0 ** 24
    p = f[:, 0:3].astype(np.float64)
    byte = lambda w, k: ((u[:, w] >> np.uint32(8 * k)) & np.uint32(255)).astype(np.float64)  # noqa: E731
    level, levels, first, seen, box = np.zeros(1, np.int64), 0, 0, np.zeros(T, np.int64), None
    inf = np.full((1, 3), np.inf)
    box = (-inf, inf)
    while len(level):
        levels += 1
        assert np.array_equal(np.sort(level), np.arange(first, first + len(level)))  # a level's nodes are contiguous
        first += len(level)
        nxt, nlo, nhi = [], [], []
        for k in range(4):
            ql = np.stack([byte(8, k), byte(10, k), byte(12, k)], 1)[level]
            qh = np.stack([byte(9, k), byte(11, k), byte(13, k)], 1)[level]
            ok = (ql <= qh).all(1)
            clo = np.maximum(box[0], p[level] + ql * step[level])[ok]
            chi = np.minimum(box[1], p[level] + qh * step[level])[ok]
            ref = u[level, 4 + k].view(np.int32)[ok]
            leaf = ref < 0
            at = (~ref[leaf]) >> 2
            assert np.all((~ref[leaf]) & 3 == 0)
            np.add.at(seen, at, 1)
            assert np.all(lo[at] >= clo[leaf]) and np.all(hi[at] <= chi[leaf])
            nxt.append(ref[~leaf].astype(np.int64)), nlo.append(clo[~leaf]), nhi.append(chi[~leaf])
        level, box = np.concatenate(nxt), (np.concatenate(nlo), np.concatenate(nhi))
    assert first == n and levels == info["bvh_depth"] and np.all(seen == 1)


@pytest.mark.parametrize("accel", ["ploc", "karras"])
@pytest.mark.parametrize("n,kind", [(2, "uniform"), (3, "line"), (65, "grid"), (1023, "uniform"), (1024, "grid"),
                                    (1025, "uniform"), (1025, "same"), (2049, "line"), (4000, "grow"), (4097, "uniform"),
                                    (40001, "uniform"), (40000, "same"), (70000, "grid")])
def test_tree_at_the_edges_of_its_steps(torch_cuda, n, kind, accel):
    torch = torch_cuda
    from paper_1702_01530_amd.stereo import GpuScene, render_stereo
    scene = _soup(n, kind)
    print(f"[build] {n} {kind} {accel}", flush=True)
    gs = GpuScene(scene, accel=accel)
    torch.cuda.synchronize()
    _walk(gs, n, scene.triangles)
    cam = mono_camera(center=(0, 0.5, 0), width=33, height=21, depth=2, baseline=0.065, convergence=5.0)
    tree, brute = render_stereo(gs, cam, path_ids=True), render_stereo(gs, cam, path_ids=True, brute_force=True)
    torch.cuda.synchronize()
    for k in ("radiance", "hit_t", "hit_prim", "path_prims", "shadow_state"):
        assert torch.equal(tree[k], brute[k]), k
    gs.close()


@pytest.mark.parametrize("n", [5, 3000, 100000])
@pytest.mark.parametrize("bad", [float("nan"), float("inf"), 3e12])
def test_refused_triangles_stay_refused(torch_cuda, n, bad):
    """A bad vertex anywhere (or everywhere) gives the same error at every size, and the build ends."""
    from paper_1702_01530_amd import rt
    from paper_1702_01530_amd.stereo import GpuScene
    for at in (slice(n // 2, n // 2 + 1), slice(0, n)):
        scene = _soup(n, "uniform")
        scene.triangles[at, 1, 2] = bad
        print(f"[build] refused {n} {bad} {at}", flush=True)
        for accel in ("ploc", "karras"):
            with pytest.raises(rt.RtError) as e:
                GpuScene(scene, accel=accel)
            assert e.value.status == rt.RT_ERR_INVALID_ARGUMENT


@pytest.mark.parametrize("n", [255, 1024, 1025, 32768, 32769, 262143, 262144, 300001])
def test_sort_at_the_edges_of_its_tiles(torch_cuda, n):
    """The record order is a stable sort of the Morton codes where the sort's tile size and its prefix change (262,144
    triangles; 32 blocks), with a tenth of the triangles duplicated (equal codes keep their order)."""
    from paper_1702_01530_amd.stereo import GpuScene
    from tests.test_gpu_render import _morton_keys, _record_ids
    scene = _soup(n, "uniform")
    r = np.random.default_rng(n + 1)
    scene.triangles[r.integers(0, n, n // 10)] = scene.triangles[r.integers(0, n, n // 10)]
    print(f"[build] sort {n}", flush=True)
    gs = GpuScene(scene)
    assert np.array_equal(_record_ids(gs, n), np.argsort(_morton_keys(scene.triangles), kind="stable"))
    gs.close()


@pytest.mark.parametrize("n", [1, 3, 5, 511, 512, 519, 1030])
@pytest.mark.parametrize("size", [(1, 1), (33, 21), (150, 140)])
def test_scenes_without_a_tree(torch_cuda, n, size):
    """RT_ACCEL_NONE around the sizes where eight waves share a batch's triangles (512) and where a wave's records, taken
    four at a time, leave a rest: equal to the tree's render and to brute force on the tree's records, byte for byte."""
    torch = torch_cuda
    from dataclasses import replace
    from paper_1702_01530_amd.stereo import GpuScene, render_stereo
    scene = replace(_soup(n, "grid"), spheres=np.asarray([[0.5, 0.3, 4, 0.4], [-1, 0, 9, 1.5]], np.float32),
                    sphere_material=np.zeros(2, np.uint32), planes=np.asarray([[0, 1, 0, -3]], np.float32),
                    plane_material=np.zeros(1, np.uint32))
    cam = mono_camera(center=(0, 0.5, 0), width=size[0], height=size[1], depth=2, baseline=0.065, convergence=5.0)
    print(f"[flat] {n} {size}", flush=True)
    a, b = GpuScene(scene, accel="none"), GpuScene(scene)
    outs = [render_stereo(a, cam, path_ids=True), render_stereo(b, cam, path_ids=True),
            render_stereo(b, cam, path_ids=True, brute_force=True), render_stereo(a, cam, path_ids=True, count_work=True)]
    torch.cuda.synchronize()
    for o in outs[1:]:
        for k in ("radiance", "hit_t", "hit_prim", "path_prims", "shadow_state"):
            assert torch.equal(outs[0][k], o[k]), k
    a.close()
    b.close()


@pytest.mark.parametrize("n", [2, 63, 64, 65, 127, 1087, 1088, 16384, 16385])
@pytest.mark.parametrize("kind", ["uniform", "grid", "same"])
def test_sort_of_few_keys(torch_cuda, n, kind):
    """Small builds place each key by counting the keys before it, in tiles of 64 and shares of 64 a wave: the record order
    is a stable sort of the Morton codes, with few distinct codes and with one."""
    from paper_1702_01530_amd.stereo import GpuScene
    from tests.test_gpu_render import _morton_keys, _record_ids
    scene = _soup(n, kind)
    print(f"[build] sort {n} {kind}", flush=True)
    gs = GpuScene(scene)
    assert np.array_equal(_record_ids(gs, n), np.argsort(_morton_keys(scene.triangles), kind="stable"))
    gs.close()


@pytest.mark.parametrize("accel", ["ploc", "karras"])
@pytest.mark.parametrize("n,kind", [(12288, "uniform"), (12288, "line"), (12288, "same"), (12289, "uniform"),
                                    (12289, "grow")])
def test_small_trees_level_by_level(torch_cuda, n, kind, accel):
    """Trees of at most 12,288 triangles are collapsed by one workgroup, several nodes a thread; larger ones by a launch
    a level where a level is wide."""
    from paper_1702_01530_amd.stereo import GpuScene
    scene = _soup(n, kind)
    print(f"[build] levels {n} {kind} {accel}", flush=True)
    gs = GpuScene(scene, accel=accel)
    _walk(gs, n, scene.triangles)
    gs.close()
