"""Sphere insertion at the sizes where its work splits change, against the
oracle: balls wider than a wave along z (rows in pieces), balls cut by the
image on every side, boxes of caps without and with points, caps larger than
those dealt together, centres of one step beside each other. Everything is an
integer: equality."""
import numpy as np
import pytest

import oracle
import paper_2101_03240_amd as ibip
from paper_2101_03240_amd import synth

pytestmark = pytest.mark.gpu


def _open(shape, solid):
    img = np.ones(shape, np.uint8)
    for s in solid:
        img[s] = 0
    return img


def _image(name):
    rng = np.random.default_rng(11)
    if name == "line":  # one row: caps of one point
        return _open((1, 1, 3000), [(0, 0, 0), (0, 0, 2049)])
    if name == "column":  # along x: L of every ball is 1
        return _open((700, 1, 1), [(13, 0, 0)])
    if name == "plane":  # balls of more than 64 voxels across
        return _open((1, 190, 210), [(0, 3, 5), (0, 180, 200)])
    if name == "box":  # plateaus: many centres of one step, caps across the whole image (over 1024 points)
        return _open((20, 22, 180), [(slice(None), slice(None), 0), (slice(None), slice(None), 179)])
    if name == "noise":
        return synth.blurred_noise((61, 64, 67), 5.0, 0.6, 3)
    return (rng.random((40, 33, 65)) < 0.9).astype(np.uint8)  # balls of a few voxels


@pytest.mark.parametrize("integer_ball", [False, True])
@pytest.mark.parametrize("name", ["line", "column", "plane", "box", "noise", "salt"])
def test_insertion_equals_oracle(name, integer_ball):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    img = _image(name)
    inl = synth.face_mask(img.shape, 2 if img.shape[2] > 1 else 0, 0)
    want = oracle.invade(img, inl, integer_ball=integer_ball)
    got = ibip.invade(torch.from_numpy(img).cuda(), torch.from_numpy(inl).cuda(), integer_ball=integer_ball)
    assert got["K"] == want["K"]
    assert np.array_equal(got["seq"].cpu().numpy(), want["seq"])
