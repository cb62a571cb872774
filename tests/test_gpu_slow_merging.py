"""Scenes whose clustering rounds merge few pairs, so that a build takes more rounds than are launched at first: the tree
reaches every triangle once and two builds store the same bytes."""
import numpy as np
import pytest

from tests.helpers import make_scene
from tests.test_gpu_build_rounds import _walk

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_01530_amd import rt
    rt.lib()
    return torch


def _scene(n, kind):
    """Triangles around one point, of random sizes, or needles of random lengths along an axis."""
    r = np.random.default_rng(n)
    if kind == "shells":
        tris = r.uniform(0.01, 4, (n, 1, 1)) * np.asarray([[-1, -1, -1], [1, 1, 1], [1, -1, 1]], float)
    else:
        x, size = r.uniform(0, 1e3, n), 500 * r.uniform(0, 1, n) ** 8
        tris = np.zeros((n, 3, 3))
        tris[:, :, 0] = x[:, None] + size[:, None] * np.asarray([0, 1, 0.5])
        tris[:, 1, 1] = tris[:, 2, 2] = 0.01
    return make_scene(tris=tris, lights=[[1, 5, -2, 1, 1, 1]])


@pytest.mark.parametrize("n", [1025, 5000, 40000, 300000])
@pytest.mark.parametrize("kind", ["shells", "needles"])
def test_rounds_that_merge_slowly(torch_cuda, n, kind):
    from paper_1702_01530_amd.stereo import GpuScene
    scene = _scene(n, kind)
    print(f"[build] {n} {kind}", flush=True)
    first, second = GpuScene(scene), GpuScene(scene)
    _walk(first, n, scene.triangles)
    nbytes = -(-64 * (n - 1) // 256) * 256 + 48 * n  # nodes and triangle records
    a, b = (g._storage[g.storage_offset:g.storage_offset + nbytes] for g in (first, second))
    assert torch_cuda.equal(a, b)
    first.close()
    second.close()
