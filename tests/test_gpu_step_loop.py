"""The step loop where calls of size run it: wide steps over the whole GPU and
the insertion beside them, resumed calls, batches (continued jobs, replayed
setups) and served jobs, told by the counters of the timing, which the component
tree leaves at 0. Everything is an integer: equality with the oracle, or with the
steps that an image of parallel plates has by construction."""
import time

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


def _put(dev, a):
    import torch
    return torch.from_numpy(a).to(dev)


def _timed(fn):
    import paper_2101_03240_amd as ibip

    ibip.reset_timing()
    ibip.enable_timing(True)
    try:
        return fn(), ibip.get_timing()
    finally:
        ibip.enable_timing(False)


def _same(r, ref, keys=("centre_step", "seq", "rad2", "M")):
    assert r["K"] == ref["K"]
    for k in keys:
        assert np.array_equal(r[k].cpu().numpy().view(np.uint32), np.asarray(ref[k]).astype(np.uint32)), k


def _plates(dev, shape):
    """Plates one voxel apart: from the face x = 0 each step takes the next x of all
    of them (the first one x = 0 and 1), and its spheres hold their centres alone."""
    import torch

    img = torch.zeros(shape, dtype=torch.uint8, device=dev)
    img[:, :, ::2] = 1
    x = torch.arange(shape[0], dtype=torch.int32, device=dev).clamp(min=1)[:, None, None]
    return img, torch.where(img != 0, x.expand(shape), torch.full_like(x, -1).expand(shape))


def test_wide_steps_and_the_insertion_beside_them(dev):
    """16,384 centres a step (the whole GPU takes steps of more than 8,192), 4.9 M in
    all (the insertion starts at 2^21); then the same resumed from its 100th step."""
    import torch

    import paper_2101_03240_amd as ibip

    shape = (300, 256, 128)
    img, want = _plates(dev, shape)
    inl = _put(dev, synth.face_mask(shape, 0, 0))
    r, t = _timed(lambda: ibip.invade(img, inl))
    assert t["loop_launches"] > 0 and t["wide_launches"] > 200
    assert r["K"] == 299 and torch.equal(r["seq"], want)
    assert torch.equal(r["centre_step"], want.clamp(min=0))
    part = ibip.invade(img, inl, max_steps=100)
    assert torch.equal(part["centre_step"], torch.where(want > 100, 0, want).clamp(min=0))
    r, t = _timed(lambda: ibip.invade_resume(img, inl, part["centre_step"], 100))
    assert t["wide_launches"] > 150
    assert r["K"] == 299 and torch.equal(r["seq"], want)


@pytest.mark.parametrize("name", ["noise", "grains", "salt", "plane"])
def test_resumed_from_the_start(dev, name):
    """A call resumed from step 0 runs the step loop from its first step to its last,
    on images that the tree would take."""
    import torch

    import oracle
    import paper_2101_03240_amd as ibip

    img = {"noise": lambda: synth.blurred_noise((110, 120, 100), 3.0, 0.6, 3),
           "grains": lambda: synth.overlapping_spheres((120, 100, 110), r2=40, porosity=0.5, seed=2),
           "salt": lambda: (np.random.default_rng(1).random((90, 100, 110)) < 0.75).astype(np.uint8),
           "plane": lambda: synth.blurred_noise((1, 600, 500), 4.0, 0.6, 5)}[name]()
    inl = synth.face_mask(img.shape, 2, 0)
    none = torch.zeros(img.shape, dtype=torch.int32, device=dev)
    r, t = _timed(lambda: ibip.invade_resume(_put(dev, img), _put(dev, inl), none, 0))
    assert t["loop_launches"] > 0
    _same(r, oracle.invade(img, inl))


def _uneven(n, lo, hi, seed):
    rng = np.random.default_rng(seed)
    imgs = []
    for i in range(n):
        L = int(rng.integers(lo, hi))
        imgs.append(synth.blurred_noise((L, L + 3, L - 5), 3.0, 0.6, 50 + i) if i % 2 else
                    synth.overlapping_spheres((L, L - 2, L + 4), r2=16, porosity=0.65, seed=50 + i))
    return imgs, [synth.face_mask(i.shape, 0, 0) for i in imgs]


# several jobs with limits, and a few small ones without: both by their step loops,
# whose steps above the threshold leave the launch
@pytest.mark.parametrize("wide", [128, 300, 1000, -1])
@pytest.mark.parametrize("n, lo, hi, limit", [(9, 40, 90, 900), (3, 38, 46, 0)])
def test_batch_continued_jobs(dev, wide, n, lo, hi, limit):
    import oracle
    import paper_2101_03240_amd as ibip

    imgs, inls = _uneven(n, lo, hi, 7)
    lims = [limit if i != 1 else 57 for i in range(n)]
    imgs.append(np.ones((20, 20, 24), np.uint8))  # no solid: fails alone
    inls.append(synth.face_mask(imgs[-1].shape, 0, 0))
    out, t = _timed(lambda: ibip.invade_batch([_put(dev, a) for a in imgs], [_put(dev, a) for a in inls],
                                              max_steps=lims + [limit], raise_on_error=False,
                                              tuning={"batch_wide": wide}))
    assert t["loop_launches"] == 1
    # (the inlet face is a step of 2,000 to 9,000 centres)
    assert (t["wide_launches"] > 0) == (wide > 0)
    assert out[-1]["status"] == -3
    for img, inl, lim, b in zip(imgs[:-1], inls[:-1], lims, out):
        assert b["status"] == 0
        _same(b, oracle.invade(img, inl, max_steps=lim))


def test_replayed_setups(dev):
    """The same batch of more jobs than there are streams comes back: its setups are
    captured, then replayed, with the program's own work and other batches between,
    and read what the inputs hold by then."""
    import torch

    import paper_2101_03240_amd as ibip

    imgs, inls = _uneven(12, 40, 70, 3)
    da, ia = [_put(dev, a) for a in imgs], [_put(dev, a) for a in inls]
    out = [torch.empty(0)]

    def run():
        r, t = _timed(lambda: ibip.invade_batch(da, ia, max_steps=300))
        assert t["loop_launches"] == 1
        return r

    def want():
        return [ibip.invade(x, y, max_steps=300) for x, y in zip(da, ia)]

    def check(got, ref):
        for b, s in zip(got, ref):
            assert b["status"] == 0 and b["K"] == s["K"]
            assert all(torch.equal(b[k], s[k]) for k in ("seq", "rad2", "centre_step", "M"))

    ref = want()
    for _ in range(3):
        out = run()
        check(out, ref)
        out = run()
        check(out, ref)
        torch.cuda.synchronize()
        ibip.invade_batch(da[:2], ia[:2], max_steps=50)
        ibip.invade_batch([torch.ones_like(da[0]) * da[0] for _ in range(2)] + da, ia[:1] * 2 + ia)  # (trees)
    for x, a in zip(da, imgs):
        x.copy_(_put(dev, np.flip(a, axis=-1).copy()))
    ref = want()
    check(run(), ref)
    check(run(), ref)


@pytest.mark.parametrize("wide", [128, 1000])
def test_served_jobs_with_wide_steps(dev, wide):
    import oracle
    import paper_2101_03240_amd as ibip

    imgs, inls = _uneven(10, 30, 50, wide)
    with ibip.Server(dev, hbm_budget_bytes=1 << 30, max_inflight=4) as srv:
        srv.set_tuning({"batch_wide": wide, "edt_tile_y": 64})
        ts = [srv.submit(_put(dev, a), _put(dev, b), max_steps=41 if i == 3 else 0)
              for i, (a, b) in enumerate(zip(imgs, inls))]
        res = [srv.wait(t) for t in ts]
    for i, (img, inl, r) in enumerate(zip(imgs, inls, res)):
        assert r["status"] == 0
        _same(r, oracle.invade(img, inl, max_steps=41 if i == 3 else 0))


@pytest.mark.parametrize("wide", [-1, 500])
def test_cancelled_in_its_loop(dev, wide):
    """A job whose loop takes long (4,000 steps of 4,096 centres: in one workgroup, or
    each over the whole GPU) stops at a check or between its segments."""
    import paper_2101_03240_amd as ibip

    shape = (4000, 128, 64)
    img, _ = _plates(dev, shape)
    inl = _put(dev, synth.face_mask(shape, 0, 0))
    small = synth.blurred_noise((40, 44, 48), 3.0, 0.6, 80)
    sinl = synth.face_mask(small.shape, 0, 0)
    with ibip.Server(dev, hbm_budget_bytes=4 << 30, max_inflight=4) as srv:
        srv.set_tuning({"batch_wide": wide})
        t = srv.submit(img, inl)
        t0 = time.time()
        while srv.stats()["running"] < 1 and time.time() - t0 < 30:
            time.sleep(0.0005)
        time.sleep(0.02)  # (past its setup)
        assert not srv.done(t)
        assert srv.cancel(t)
        ts = srv.submit(_put(dev, small), _put(dev, sinl))
        r, rs = srv.wait(t), srv.wait(ts)
        st = srv.stats()
    assert r["status"] == -6 and rs["status"] == 0
    assert st["cancelled"] == 1 and st["bytes_in_use"] == 0 and st["running"] == 0
    s = ibip.invade(_put(dev, small), _put(dev, sinl))
    assert rs["K"] == s["K"] and np.array_equal(rs["seq"].cpu().numpy(), s["seq"].cpu().numpy())
