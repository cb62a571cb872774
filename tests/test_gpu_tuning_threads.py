"""A thread that sets the launch tuning while others render: each call takes one tuning throughout (the no-allocation entry
point lays its traversal-stack spill area out for the grid that it launches), so the images are those of a quiet render."""
import threading

import pytest

import scenegen as sg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ids", [True, False])
def test_noalloc_while_the_tuning_changes(ids):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1702_01530_amd import rt
    from paper_1702_01530_amd.stereo import GpuScene, alloc_outputs, output_struct, render_stereo, stream_handle
    scene, cam = sg.make_terrain_1080p()
    cam = cam.resized(640, 360)
    gs = GpuScene(scene)
    ref = render_stereo(gs, cam, path_ids=ids)
    out = alloc_outputs(cam, gs.num_lights, gs.device, ids, False)
    st, camst, flags = output_struct(out), rt.make_camera_struct(cam), rt.RT_FLAG_PATH_IDS if ids else 0
    saved, stop = rt.rt_get_tuning(), threading.Event()

    def change():
        k = 0
        while not stop.is_set():
            k += 1
            rt.rt_set_tuning(**{**saved, "trace_blocks_per_cu": 0 if k % 2 else 1})

    thread = threading.Thread(target=change)
    thread.start()
    try:
        for k in range(100):
            out["radiance"].fill_(-7.0)
            rt.rt_render_stereo_noalloc(gs.handle, camst, st, flags, stream_handle(None), None)
            torch.cuda.synchronize()
            for key in ("radiance", "hit_t", "hit_prim"):
                assert torch.equal(out[key], ref[key]), (k, key)
    finally:
        stop.set()
        thread.join()
        rt.rt_set_tuning(**saved)
    gs.close()
