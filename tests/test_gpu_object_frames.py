"""GPU: object removal on the frames that choose its kernels, bit-exact against the oracle.

Half a frame's rows times the bias of its masked costs decide: up to 31 bits (1672 rows of three
channels) a team of the carve engine takes the frame, above that one workgroup of 1024 threads with
64-bit keys.  The frames below it that are wide enough for several waves, for ancestors that do not fit in
LDS, for eight columns per thread and for several passes of a row's shift are all above the bound; flat
wide frames make the teams take strips of eight columns per lane."""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev, host, log

pytestmark = pytest.mark.gpu

from paper_2410_21207_amd import api  # noqa: E402

LIMIT = 1 << 31


def _by_teams(H, C):
    half = min(((H + 1) // 2 + 3) & ~3, H) if H > 32 else H
    return (half + 1) * (H * 510 * C + 1) < LIMIT


# H, W, C, columns of the mask, values
FRAMES = [
    (1676, 700, 3, 3, 256),    # several waves, cross-wave keys, rows of several passes
    (1700, 130, 3, 4, 3),      # few waves, ties
    (1700, 2300, 3, 2, 4),     # 29 phases x 2300 columns of ancestors do not fit in LDS
    (1690, 4300, 3, 2, 256),   # eight columns per thread
    (2100, 1030, 2, 2, 5),
    (1500, 900, 4, 3, 256),
    (2920, 520, 1, 3, 4),
    (1672, 300, 3, 3, 4),      # the tallest of three channels that a team takes
    (64, 8000, 3, 3, 4),       # strips of eight columns per lane
    (33, 8000, 1, 4, 256),
]


@pytest.mark.parametrize("H,W,C,cols,alpha", FRAMES)
def test_object_frames(H, W, C, cols, alpha):
    log("object frame", H, W, C, "by teams" if _by_teams(H, C) else "by one workgroup")
    rng = np.random.default_rng(H + W)
    img = rng.integers(0, alpha, size=(H, W, C), dtype=np.uint8)
    mask = np.zeros((H, W), np.uint8)
    x = W * 2 // 3
    mask[H // 5:H // 5 + H // 2, x:x + cols] = 7
    mask[H - 2, 1] = 1  # a stray pixel far from the rest
    o_out, o_info, o_seams, o_costs = oracle.remove_object(img, mask, 0)
    out, info, seams, costs = api.remove_object(dev(img), dev(mask), 0)
    assert info["k"] == o_info["k"] >= cols and info["left"] == o_info["left"] == 0
    assert np.array_equal(host(seams), o_seams) and np.array_equal(host(costs), o_costs)
    assert np.array_equal(host(out), o_out)


def test_tall_frame_from_a_wide_mask():
    """Horizontal seams of an image wider than the bound's rows: its transpose is carved by one workgroup, and
    the size comes back by insertion."""
    H, W = 500, 1800
    img = np.random.default_rng(4).integers(0, 256, size=(H, W, 3), dtype=np.uint8)
    mask = np.zeros((H, W), np.uint8)
    mask[200:203, 300:1500] = 1
    assert not _by_teams(W, 3)
    o_out, o_info, o_seams, o_costs = oracle.remove_object(img, mask, -1, True)
    out, info, seams, costs = api.remove_object(dev(img), dev(mask), -1, True)
    assert info["direction"] == o_info["direction"] == 1 and info["k"] == o_info["k"]
    assert np.array_equal(host(seams), o_seams) and np.array_equal(host(costs), o_costs)
    assert np.array_equal(host(out), o_out)
