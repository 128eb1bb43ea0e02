"""GPU: the stage clocks add up to the carve they belong to, whoever carves it and in however many calls."""
import ctypes

import numpy as np
import pytest
import torch

from gpu_helpers import dev, log

pytestmark = pytest.mark.gpu

from paper_2410_21207_amd import _lib, api  # noqa: E402


def _image(H, W):
    return dev(np.random.default_rng(H + W).integers(0, 256, size=(H, W, 3), dtype=np.uint8))


def _adds_up(ws, n=1, gaps=False):
    for (t0, t1), st in zip(api.read_times(ws, n), api.read_stages(ws, n)):
        log("stages", ["%.1f us" % (1e6 * s) for s in st], "of %.1f us" % (1e6 * (t1 - t0)))
        assert all(0 <= s <= t1 - t0 for s in st) and st[0] > 0 and st[1] > 0
        assert sum(st) <= (t1 - t0) * 1.001 and (gaps or sum(st) >= 0.6 * (t1 - t0))


@pytest.mark.parametrize("team", [1, 4])
def test_stages_of_a_carve(team):
    img = _image(300, 700)
    ws = api.workspace(1 << 23, "cuda")
    api.carve(img, 660, team=team, variant=7, ws=ws)
    _adds_up(ws)


def test_stages_of_forward_and_batches():
    ws = api.workspace(1 << 24, "cuda")
    api.carve_forward(_image(300, 700), 660, ws=ws)
    torch.cuda.synchronize()
    _adds_up(ws)
    srcs = [_image(100 + 20 * i, 300 + 10 * i) for i in range(6)]
    for b in (api.BatchCarver([torch.empty_like(x) for x in srcs], [250] * 6, srcs=srcs),
              api.ForwardBatch([torch.empty_like(x) for x in srcs], [250] * 6, srcs=srcs)):
        for _ in range(2):
            b.launch()
            _adds_up(b.ws, 6)


def test_stages_of_steps_and_of_one_seam():
    lib = _lib.load()
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    st = ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)
    img, ws, table = _image(200, 400), api.workspace(1 << 23, "cuda"), api.workspace(lib.sc_slot_table_bytes(1), "cuda")
    job = _lib.sc_job(img.data_ptr(), 200, 400, 3, 1200, 370, None, None, None)
    _lib.call("sc_slot_start", ctypes.byref(job), p(ws), ws.numel(), p(table), 1, 0, st)
    team = (ctypes.c_int32 * 1)(3)
    done = torch.zeros(1, dtype=torch.int32, device="cuda")
    for i in range(30):  # by a team and by one workgroup in turn, with and without a budget
        if i % 2:
            _lib.call("sc_slots_step", p(table), 1, 1, p(done), st)
        else:
            _lib.call("sc_slots_step_teams", p(table), 1, 1, team, 1, 1000 * (i % 4), p(done), st)
    assert int(done.cpu()[0]) == 30
    _adds_up(ws, gaps=True)
    e = torch.randint(0, 200, (300, 500), dtype=torch.int32, device="cuda")
    api.dp_seam(e, ws=ws)
    assert api.read_stages(ws)[0] == (0, 0, 0)  # clocks belong to carves
