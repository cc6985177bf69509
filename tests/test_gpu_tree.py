"""The invasion by levels of the component tree, at the sizes where its paths
change, against the oracle: levels of few voxels (one workgroup) and of many,
searches that fit in LDS or not, more peaks than there is room for (the step
loop takes over), and step limits on both sides of the one below which the
step loop runs. Everything is an integer: equality."""
import numpy as np
import pytest

from paper_2101_03240_amd import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dev():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    return torch.device("cuda:0")


def _serpentine(n):
    """One channel of width 1 that runs through n x n pixels: as many rounds of
    one level as it has pixels."""
    img = np.zeros((1, n, n), np.uint8)
    img[0, 1::2] = 1
    for i, y in enumerate(range(2, n, 2)):
        img[0, y, n - 1 if i % 2 == 0 else 0] = 1
    return img


def _comb(n, depth):
    """A corridor of width 1 with a dead-end chamber of width 3 at each step:
    components entered one by one in the rounds of one level."""
    img = np.zeros((1, depth + 8, n), np.uint8)
    img[0, 1] = 1
    for x in range(2, n - 4, 6):
        img[0, 2:4, x + 1] = 1
        img[0, 4:4 + depth, x:x + 3] = 1
    return img


def _image(name):
    rng = np.random.default_rng(7)
    if name == "serpentine":
        return _serpentine(161)
    if name == "comb":
        return _comb(2000, 9)
    if name == "salt":  # few ranks, levels of many voxels, long searches
        return (rng.random((48, 50, 52)) < 0.62).astype(np.uint8)
    if name == "isolated":  # more peaks than an eighth of the pore voxels
        img = np.zeros((40, 60, 80), np.uint8)
        img[::2, ::2, ::2] = 1
        img[0] = 1
        return img
    if name == "open":  # one solid voxel: one component, levels of growing shells
        img = np.ones((40, 41, 43), np.uint8)
        img[20, 20, 20] = 0
        return img
    if name == "wide levels":
        return synth.blurred_noise((90, 120, 130), 3.0, 0.6, 3)
    return synth.overlapping_spheres((100, 90, 80), r2=40, porosity=0.5, seed=2)


@pytest.mark.parametrize("name", ["serpentine", "comb", "salt", "isolated", "open", "wide levels", "grains"])
def test_tree_equals_oracle(dev, name):
    import torch

    import oracle
    import paper_2101_03240_amd as ibip

    img = _image(name)
    axis = 2 if name == "comb" else 1 if img.shape[0] == 1 else 0
    inl = synth.face_mask(img.shape, axis, 0)
    ref = oracle.invade(img, inl)
    r = ibip.invade(torch.from_numpy(img).to(dev), torch.from_numpy(inl).to(dev))
    assert r["K"] == ref["K"]
    for k in ("centre_step", "seq", "rad2", "M"):
        assert np.array_equal(r[k].cpu().numpy().view(np.uint32), np.asarray(ref[k]).astype(np.uint32)), k


@pytest.mark.parametrize("steps", [1, 1023, 1024, 1500, 10 ** 6])
def test_tree_step_limit(dev, steps):
    import torch

    import oracle
    import paper_2101_03240_amd as ibip

    img = synth.blurred_noise((1, 260, 300), 5.0, 0.6, 5)
    inl = synth.face_mask(img.shape, 1, 0)
    ref = oracle.invade(img, inl, max_steps=steps)
    r = ibip.invade(torch.from_numpy(img).to(dev), torch.from_numpy(inl).to(dev), max_steps=steps)
    assert r["K"] == ref["K"]
    for k in ("centre_step", "seq", "rad2", "M"):
        assert np.array_equal(r[k].cpu().numpy().view(np.uint32), np.asarray(ref[k]).astype(np.uint32)), k


@pytest.mark.parametrize("limits", [[5, 40, 900, 7], [5, 0, 900, 7], [0, 2000, 0, 0]])
def test_batch_step_limits(dev, limits):
    """Batches of uneven images whose jobs all stop after few steps (the step
    loops) and others (one tree for all): each job as the oracle alone."""
    import torch

    import oracle
    import paper_2101_03240_amd as ibip

    imgs = [synth.blurred_noise((20, 61, 33), 2.5, 0.6, 1), synth.overlapping_spheres((45, 30, 70), 16, 0.6, 2),
            synth.blurred_noise((1, 120, 90), 4.0, 0.55, 3), synth.overlapping_spheres((9, 64, 8), 9, 0.7, 4)]
    inls = [synth.face_mask(i.shape, 1, 0) for i in imgs]
    out = ibip.invade_batch([torch.from_numpy(i).to(dev) for i in imgs],
                            [torch.from_numpy(i).to(dev) for i in inls], max_steps=limits, sat=True)
    for img, inl, lim, b in zip(imgs, inls, limits, out):
        ref = oracle.invade(img, inl, max_steps=lim)
        assert b["status"] == 0 and b["K"] == ref["K"]
        for k in ("centre_step", "seq", "rad2", "M"):
            assert np.array_equal(b[k].cpu().numpy().view(np.uint32), np.asarray(ref[k]).astype(np.uint32)), k
        n = np.bincount(ref["seq"][ref["seq"] > 0], minlength=ref["K"] + 1)[1:]
        assert np.array_equal(b["sat"].cpu().numpy(), np.cumsum(n) / float((img != 0).sum()))


@pytest.mark.parametrize("budget", [3 << 20, 64 << 20])
def test_served_with_and_without_room_for_the_tree(dev, budget):
    """A server whose pool holds one job's scratch but not its tree's (the step
    loop runs), and one with room for both; a step limit below the tree's."""
    import torch

    import oracle
    import paper_2101_03240_amd as ibip

    img = synth.blurred_noise((44, 46, 40), 3.0, 0.6, 8)
    inl = synth.face_mask(img.shape, 0, 0)
    with ibip.Server(dev, hbm_budget_bytes=budget, max_inflight=2) as srv:
        ts = [srv.submit(torch.from_numpy(img).to(dev), torch.from_numpy(inl).to(dev), max_steps=k)
              for k in (0, 50, 0)]
        res = [srv.wait(t) for t in ts]
        assert srv.stats()["bytes_in_use"] == 0
    for k, b in zip((0, 50, 0), res):
        ref = oracle.invade(img, inl, max_steps=k)
        assert b["status"] == 0 and b["K"] == ref["K"]
        for f in ("centre_step", "seq", "rad2", "M"):
            assert np.array_equal(b[f].cpu().numpy().view(np.uint32), np.asarray(ref[f]).astype(np.uint32)), f
