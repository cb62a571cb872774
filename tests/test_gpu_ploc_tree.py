"""The tree that the clustering kernels build is the one that the partner rule gives: the rounds, the cost table and the
collapse are run on the host with the rule's own function (ploc_tree.cpp), and every child reference of every node is
compared."""
import os
import subprocess

import numpy as np
import pytest

from tests.helpers import coincident_scene, corners_scene, flat_scene
from tests.test_gpu_build_rounds import _soup

pytestmark = pytest.mark.gpu
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_01530_amd import rt
    rt.lib()
    return torch


@pytest.fixture(scope="module")
def host(tmp_path_factory):
    exe = tmp_path_factory.mktemp("ploc") / "ploc_tree"
    subprocess.run(["g++", "-O2", "-ffp-contract=off", "-std=c++17", os.path.join(ROOT, "tests", "ploc_tree.cpp"), "-o",
                    str(exe)], check=True)
    return exe


def _compare(torch, host, tmp_path, scene, what):
    from paper_1702_01530_amd import rt
    from paper_1702_01530_amd.stereo import GpuScene
    print(f"[ploc] {what}", flush=True)
    T = scene.num_triangles
    gs = GpuScene(scene)
    info = gs.info()
    assert info["builder"] == rt.RT_ACCEL_PLOC
    torch.cuda.synchronize()
    raw = gs._storage[gs.storage_offset:].cpu().numpy()
    gs.close()
    device = raw[:64 * info["num_nodes"]].view(np.int32).reshape(-1, 16)[:, 4:8]
    order = raw[-(-64 * (T - 1) // 256) * 256:][:48 * T].view(np.int32).reshape(T, 12)[:, 3]
    tris = scene.triangles[order]
    boxes, refs = tmp_path / "boxes", tmp_path / "refs"
    np.concatenate([tris.min(1), tris.max(1)], 1).astype(np.float32).tofile(boxes)
    subprocess.run([str(host), str(boxes), str(refs)], check=True, timeout=100)
    assert np.array_equal(device, np.fromfile(refs, np.int32).reshape(-1, 4)), what


# the one-workgroup rounds (to 1,024 clusters), the search of few clusters (below 65,536) and the one-sided search of
# many, and the collapse with one workgroup (to 12,288 triangles) and with launches a level
@pytest.mark.parametrize("n,kind", [(2, "uniform"), (3, "line"), (33, "grid"), (64, "same"), (1023, "uniform"),
                                    (1024, "grid"), (1025, "uniform"), (1090, "same"), (4000, "grow"), (5000, "grid"),
                                    (12289, "uniform"), (40001, "line"), (65536, "uniform"), (70000, "grid"),
                                    (70001, "same"), (300001, "uniform")])
def test_tree_of_the_rule(torch_cuda, host, tmp_path, n, kind):
    _compare(torch_cuda, host, tmp_path, _soup(n, kind), (n, kind))


@pytest.mark.parametrize("make", [coincident_scene, corners_scene, flat_scene])
def test_tree_of_the_rule_with_ties(torch_cuda, host, tmp_path, make):
    _compare(torch_cuda, host, tmp_path, make()[0], make.__name__)
