"""GPU: calls of every kind at once on several streams, whose teams want more workgroups of one XCD
than it holds, each equal to the oracle.  A team takes whoever is there in time, so nobody waits for
a workgroup that another team keeps out."""
import threading

import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev, host, log

pytestmark = pytest.mark.gpu

from paper_2410_21207_amd import api  # noqa: E402


def _image(seed, H, W, C=3):
    return np.random.default_rng(seed).integers(0, 256, size=(H, W, C), dtype=np.uint8)


def test_calls_on_several_streams():
    """Three carves by teams of 32, two by the default team, forward energy, one seam, insertion and
    (from its own thread, being synchronous) object removal, twice over, all in flight together."""
    carves = [(_image(i, 300 + 40 * i, 900 - 50 * i), 24, 32 if i < 3 else None) for i in range(5)]
    fwd = [_image(20 + i, 260 + 60 * i, 700) for i in range(2)]
    e = np.random.default_rng(3).integers(0, 200, size=(500, 1200)).astype(np.int32)
    ins = _image(30, 240, 640)
    obj, mask = _image(31, 300, 500), np.zeros((300, 500), np.uint8)
    mask[100:180, 200:215] = 1
    want_c = [oracle.carve(img, img.shape[1] - k) for img, k, _ in carves]
    want_f = [oracle.carve_forward(img, img.shape[1] - 20) for img in fwd]
    want_s, want_cost = oracle.dp_seam(e)[:2]
    want_i = oracle.insert_seams(ins, 20)
    want_o = oracle.remove_object(obj, mask, 0)
    dc, df, de, di, do, dm = [dev(c[0]) for c in carves], [dev(x) for x in fwd], dev(e), dev(ins), dev(obj), dev(mask)
    streams = [torch.cuda.Stream() for _ in range(10)]
    torch.cuda.synchronize()
    for turn in range(2):
        log("streams, turn", turn)
        box = {}

        def remove():
            with torch.cuda.stream(streams[9]):
                box["object"] = api.remove_object(do, dm, 0)

        t = threading.Thread(target=remove)
        t.start()
        got_c, got_f, keep = [], [], []
        for i, (img, k, team) in enumerate(carves):
            with torch.cuda.stream(streams[i]):
                ws = api.workspace(1 << 23, "cuda")
                keep.append(ws)
                got_c.append(api.carve(torch.empty_like(dc[i]), img.shape[1] - k, src=dc[i], team=team, ws=ws,
                                       variant=7 if team else None, check=False))
        for i, img in enumerate(fwd):
            with torch.cuda.stream(streams[5 + i]):
                got_f.append(api.carve_forward(torch.empty_like(df[i]), img.shape[1] - 20, src=df[i]))
        with torch.cuda.stream(streams[7]):
            got_s = [api.dp_seam(de, check=False) for _ in range(6)]
        with torch.cuda.stream(streams[8]):
            got_i = api.insert_seams(di, 20, check=False)
        t.join()
        torch.cuda.synchronize()
        for ws in keep:
            assert api.read_status(ws, 1) == [0]
        for got, want in list(zip(got_c, want_c)) + list(zip(got_f, want_f)):
            assert np.array_equal(host(got[1]), want[1]) and np.array_equal(host(got[2]), want[2])
            assert np.array_equal(host(got[0]), want[0])
        for seam, cost in got_s:
            assert np.array_equal(host(seam), want_s) and int(host(cost)[0]) == want_cost
        assert np.array_equal(host(got_i[0]), want_i[0]) and np.array_equal(host(got_i[1]), want_i[1])
        out, info, seams, costs = box["object"]
        assert info["k"] == want_o[1]["k"] and np.array_equal(host(seams), want_o[2])
        assert np.array_equal(host(out), want_o[0])


@pytest.mark.parametrize("team", [2, 16, 32])
def test_batch_of_whole_teams(team):
    """Sixteen images that may have a team of up to 32 each, as many workgroups as the device holds."""
    imgs = [_image(50 + i, 220 + 9 * i, 400 + 13 * i) for i in range(16)]
    srcs = [dev(x) for x in imgs]
    log("batch of teams of", team)
    bc = api.BatchCarver([torch.empty_like(x) for x in srcs], [x.shape[1] - 10 for x in imgs], srcs=srcs, team=team)
    for _ in range(2):
        bc.launch()
        for img, (out, seams, costs) in list(zip(imgs, bc.results()))[::5]:
            o_out, o_seams, o_costs = oracle.carve(img, img.shape[1] - 10)
            assert np.array_equal(host(seams), o_seams) and np.array_equal(host(costs), o_costs)
            assert np.array_equal(host(out), o_out)
