"""Display composition where its two kernels meet: widths and heights that make whole groups of four pixels and ones that
do not.  Buffers that are only 4-byte aligned take the one-pixel kernel; the bytes are the same, and nothing outside the
image is written."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _compose(torch, eyes, mode, shifts):
    from paper_1702_01530_amd import rt
    from paper_1702_01530_amd.stereo import stream_handle
    h, w = eyes.shape[1:3]
    dev = []
    for e in range(2):  # so many floats past a 16-byte aligned start
        t = torch.empty(h * w * 3 + 4, dtype=torch.float32, device="cuda")[shifts[e]:shifts[e] + h * w * 3]
        t.copy_(torch.from_numpy(eyes[e].reshape(-1)))
        dev.append(t)
    n = h * w * (2 if mode == rt.RT_COMPOSE_SIDE_BY_SIDE else 1)
    out = torch.zeros(n + 8, dtype=torch.int32, device="cuda")
    img = out[shifts[2]:shifts[2] + n]
    rt.rt_compose_stereo(dev[0].data_ptr(), dev[1].data_ptr(), w, h, mode, 1.25, img.data_ptr(), stream_handle())
    torch.cuda.synchronize()
    assert not out[:shifts[2]].any() and not out[shifts[2] + n:].any()
    return img.cpu()


@pytest.mark.parametrize("size", [(1, 1), (3, 1), (4, 1), (2, 2), (5, 4), (8, 3), (64, 33), (65, 32), (1023, 9), (1024, 1030)])
@pytest.mark.parametrize("mode", [0, 1])
def test_compose_groups_and_alignment(size, mode):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    w, h = size
    eyes = np.random.default_rng(w * 1000 + h).uniform(-0.1, 1.6, (2, h, w, 3)).astype(np.float32)
    print(f"[compose] {size} {mode}", flush=True)
    aligned = _compose(torch, eyes, mode, (0, 0, 0))
    for shifts in ((1, 0, 0), (0, 2, 0), (0, 0, 3), (1, 1, 1)):
        assert torch.equal(aligned, _compose(torch, eyes, mode, shifts)), shifts
