"""The opening's levels, several to a launch and one by one, against the oracle:
more levels than a launch takes, planes and volumes, rows of every alignment,
radii and lines on both sides of those that the shared launches take. Everything
is an integer, and the saturations are quotients of integers: equality."""
import numpy as np
import pytest

import oracle
import paper_2101_03240_amd as ibip
from paper_2101_03240_amd import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape,T", [
    ((1, 50, 61), range(70, 0, -1)),
    ((1, 64, 72), range(33, 0, -1)),
    ((9, 17, 24), range(40, 0, -1)),
    ((12, 13, 18), range(32, 0, -1)),
    ((20, 7, 11), [65535, 50, 20, 3, 1]),
    ((20, 7, 11), [65536, 50, 20, 3, 1]),
    ((1, 30, 600), [90, 40, 2, 1]),
    ((1, 1030, 9), [90, 40, 2, 1]),
    ((1, 40, 40), range(4096, 0, -1)),
    ((1, 40, 40), range(4097, 0, -1)),
])
def test_levels_equal_oracle(shape, T):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    img = synth.blurred_noise(shape, 3.0, 0.7, 4)
    img.flat[0] = 0
    inl = synth.face_mask(shape, 1, 0)
    T = np.array(list(T), np.uint32)
    want = oracle.mio(img, inl, T)
    got = ibip.opening_drainage(torch.from_numpy(img).cuda(), torch.from_numpy(inl).cuda(), T.tolist())
    assert np.array_equal(got["mio_r2"].cpu().numpy().view(np.uint32), want["mio_r2"])
    assert np.array_equal(np.asarray(got["mio_sat"]), np.asarray(want["mio_sat"]))
