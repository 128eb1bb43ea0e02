"""GPU: the carve at the sizes where its tiling changes shape, bit-exact against the oracle.

Strips of the cost sweep (a window of 256 columns, or 504 of a 512-column one when there are too few
waves for narrow strips), halves and blocks of 24 or 32 rows, rows that share an access of the row
shifter (up to 208 bytes to move) or take several passes (63 slots of 16 bytes each).
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev, host, log

pytestmark = pytest.mark.gpu

from paper_2410_21207_amd import api  # noqa: E402


def _check(H, W, C, k, alpha=256, **kw):
    log("carve shape", H, W, C, k, alpha, kw)
    img = np.random.default_rng(H * 7919 + W + C).integers(0, alpha, size=(H, W, C), dtype=np.uint8)
    out, seams, costs = api.carve(dev(img), W - k, **kw)
    o_out, o_seams, o_costs = oracle.carve(img, W - k)
    assert np.array_equal(host(seams), o_seams) and np.array_equal(host(costs), o_costs)
    assert np.array_equal(host(out), o_out)


@pytest.mark.parametrize("team", [1, 2, 3])
@pytest.mark.parametrize("W", [257, 385, 505, 513, 954, 1403, 1852])
def test_strip_edges(W, team):
    """Widths that cross a strip boundary while they shrink, one workgroup to three."""
    _check(150, W, 3, 6, alpha=5 if team == 2 else 256, team=team)


@pytest.mark.parametrize("H", [1, 2, 3, 4, 5, 8, 9, 31, 32, 33, 63, 64, 65, 66, 128, 129, 130, 260])
@pytest.mark.parametrize("variant", [7, 9])
def test_split_rows(H, variant):
    """Heights around the split of the image in halves and in blocks."""
    _check(H, 90, 1, 8, alpha=3, variant=variant, team=2 if H % 2 else 1)


@pytest.mark.parametrize("C,W", [(1, 207), (1, 420), (2, 209), (3, 138), (3, 141), (4, 103), (4, 106), (3, 1400), (4, 1100)])
@pytest.mark.parametrize("minside", [True, False])
def test_row_shifts(C, W, minside):
    """Every pixel size at the widths where rows stop sharing accesses, and where a row takes
    several passes; moving either side or only the right one."""
    _check(37, W, C, 20, minside=minside, team=1)


@pytest.mark.parametrize("team", [1, 4])
def test_path_leaves_its_window(team):
    """A seam that runs diagonally across the image: the backtrack needs several rounds."""
    H, W = 700, 1000
    img = np.full((H, W, 1), 128, np.uint8)
    img[::2, ::2] = 255
    for y in range(H):  # a quiet diagonal of constant pixels, five wide
        x = 100 + y
        img[y, x:x + 5] = 128
    log("diagonal seam", team)
    out, seams, costs = api.carve(dev(img), W - 3, team=team)
    o_out, o_seams, o_costs = oracle.carve(img, W - 3)
    assert np.array_equal(host(seams), o_seams) and np.array_equal(host(costs), o_costs)
    assert np.array_equal(host(out), o_out)


@pytest.mark.parametrize("H,W", [(1, 5), (2, 900), (63, 64), (65, 513), (300, 1403), (700, 257), (1100, 700)])
@pytest.mark.parametrize("dirs", [False, True])
def test_one_seam_by_a_team(H, W, dirs):
    """The seam of a given energy map, by the team its size gets, with and without the direction map."""
    e = np.random.default_rng(H * 7 + W).integers(0, 12, size=(H, W)).astype(np.int32)
    want, cost, _, D = oracle.dp_seam(e, full=True)
    got = api.dp_seam(dev(e), dirs=dirs)
    assert np.array_equal(host(got[0]), want)
    assert int(host(got[1])[0]) == cost
    if dirs:
        assert np.array_equal(host(got[2])[1:], D[1:])


def _check_forward(img, k, got):
    out, seams, costs = oracle.carve_forward(img, img.shape[1] - k)
    assert np.array_equal(host(got[1]), seams)
    assert np.array_equal(host(got[2]), costs)
    assert np.array_equal(host(got[0]), out)


@pytest.mark.parametrize("H,W,C", [(1, 9, 3), (2, 300, 1), (4, 257, 3), (5, 1403, 2), (33, 256, 4), (64, 513, 3),
                                   (66, 255, 1), (130, 385, 3), (300, 954, 1), (640, 70, 3)])
def test_forward_shapes(H, W, C):
    """Forward energy at the edges of strips, halves and blocks; few values, so that ties abound."""
    img = np.random.default_rng(H * 11 + W).integers(0, 3, size=(H, W, C)).astype(np.uint8)
    k = min(W - 1, 6)
    _check_forward(img, k, api.carve_forward(dev(img), W - k))


def test_forward_batch_of_lone_workgroups():
    """More images than workgroups' teams: wide strips, several to a wave, carved by one workgroup each."""
    rng = np.random.default_rng(5)
    imgs = [rng.integers(0, 4, size=(33 + i % 40, 505 + 3 * i, 3)).astype(np.uint8) for i in range(150)]
    srcs = [dev(i) for i in imgs]
    fb = api.ForwardBatch([torch.empty_like(x) for x in srcs], [i.shape[1] - 3 for i in imgs], srcs=srcs)
    fb.launch()
    res = fb.results()
    for i in range(0, len(imgs), 14):
        _check_forward(imgs[i], 3, res[i])


# the last two: costs of half the image above 31 bits, which one workgroup carves with wider keys
@pytest.mark.parametrize("H,W,C", [(1, 40, 1), (3, 300, 3), (64, 513, 3), (131, 257, 2), (300, 70, 4), (500, 1100, 3), (1640, 40, 3),
                                   (2040, 24, 4), (2400, 30, 3)])
def test_object_shapes(H, W, C):
    """Masked costs at the edges of strips, halves and blocks, and on both sides of the 31-bit limit."""
    rng = np.random.default_rng(H * 13 + W)
    img = rng.integers(0, 3, size=(H, W, C)).astype(np.uint8)
    mask = np.zeros((H, W), np.uint8)
    for _ in range(3):
        y, x = int(rng.integers(0, H)), int(rng.integers(0, W - 3))
        mask[y:y + max(1, H // 5), x:x + 3] = 255
    log("object shape", H, W, C)
    o_out, o_info, o_seams, o_costs = oracle.remove_object(img, mask, 0)
    out, info, seams, costs = api.remove_object(dev(img), dev(mask), 0)
    assert info["k"] == o_info["k"] and info["left"] == o_info["left"]
    assert np.array_equal(host(seams), o_seams) and np.array_equal(host(costs), o_costs)
    assert np.array_equal(host(out), o_out)


@pytest.mark.parametrize("k", [1, 63, 64, 65, 128, 130, 299])
def test_insert_blocks_of_seams(k):
    """Original columns are found in blocks of 64 seams."""
    img = np.random.default_rng(k).integers(0, 4, size=(7, 300, 1)).astype(np.uint8)
    o_out, o_seams = oracle.insert_seams(img, k)
    out, seams = api.insert_seams(dev(img), k)
    assert np.array_equal(host(seams), o_seams) and np.array_equal(host(out), o_out)


@pytest.mark.parametrize("C", [1, 2, 3, 4])
@pytest.mark.parametrize("H,W", [(1, 1), (2, 3), (4, 4), (5, 5), (9, 1023), (3, 1025), (8, 1028)])
def test_energy_map_groups(H, W, C):
    """The energy map in groups of 4 columns by 4 rows, of rows that start at any byte."""
    img = np.random.default_rng(H * W + C).integers(0, 256, size=(H, W, C), dtype=np.uint8)
    flat = torch.zeros(H * (W * C + 5) + 1, dtype=torch.uint8, device="cuda")
    rows = torch.as_strided(flat, (H, W, C), (W * C + 5, C, 1), 1)
    rows.copy_(dev(img))
    assert np.array_equal(host(api.energy(rows)), oracle.energy(img))
