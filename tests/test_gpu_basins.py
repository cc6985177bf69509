"""Reconstruction by basins where its paths change, against the oracle: planes
and volumes at the edges of the tiles, climbs longer than one labelling pass,
chains of hooks longer than one compression, one basin, no seed, all seeds, and
more basins than the lists hold (the sweeps take over). Everything is an integer:
equality."""
import numpy as np
import pytest

import oracle
import paper_2101_03240_amd as ibip

pytestmark = pytest.mark.gpu


def _case(name):
    rng = np.random.default_rng(5)
    if name == "climb":  # one climb through 2048 tiles
        seq = np.arange(1, 65536, dtype=np.int32).reshape(1, 1, -1)
    elif name == "chain":  # teeth of rising height, each hooking to the next
        seq = np.zeros((1, 1, 60000), np.int32)
        seq[0, 0, 0::2] = np.arange(1, 30001) + 40000
        seq[0, 0, 1::2] = np.arange(1, 30001)
    elif name == "noise":  # a top for every seventh voxel
        seq = rng.integers(1, 1000, (104, 104, 104)).astype(np.int32)
    elif name == "plateau":
        seq = np.zeros((9, 65, 33), np.int32)
        seq[4, 1:, :] = 7
    else:
        shape = {"tile": (8, 8, 32), "tile+1": (9, 9, 33), "tile-1": (7, 15, 31), "plane": (1, 64, 32),
                 "plane+1": (1, 129, 97), "thin": (70, 2, 3), "few": (3, 1, 2)}[name]
        seq = rng.integers(-1, 9, shape).astype(np.int32)
    return seq


@pytest.mark.parametrize("conn", [6, 26])
@pytest.mark.parametrize("name", ["climb", "chain", "noise", "plateau", "tile", "tile+1", "tile-1", "plane", "plane+1",
                                  "thin", "few"])
def test_trap_equals_oracle(name, conn):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    seq = _case(name)
    faces = np.zeros(seq.shape, np.uint8)
    faces[..., -1] = 1
    for outlets in (faces, np.zeros_like(faces), np.ones_like(faces)):
        want = oracle.trap(seq, outlets, conn)
        got = ibip.trap(torch.from_numpy(seq).cuda(), torch.from_numpy(outlets).cuda(), connectivity=conn)
        assert got["K_after"] == want["K_after"]
        assert np.array_equal(got["trapped"].cpu().numpy(), want["trapped"])
        assert np.array_equal(got["seq_trapped"].cpu().numpy(), want["seq_trapped"])
