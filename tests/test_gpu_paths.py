"""Which path an invasion takes, told by the timing counters (the component
tree launches no step loop), and the same results on each, against the oracle.
Everything is an integer: equality."""
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


def _loops(fn):
    """fn's result and the step loops that it launched on this thread's context."""
    import paper_2101_03240_amd as ibip

    ibip.reset_timing()
    ibip.enable_timing(True)
    try:
        r = fn()
        return r, ibip.get_timing()["loop_launches"]
    finally:
        ibip.enable_timing(False)


def _put(dev, a):
    import torch
    return torch.from_numpy(a).to(dev)


def _same(r, ref):
    assert r["K"] == ref["K"]
    for k in ("centre_step", "seq", "rad2", "M"):
        assert np.array_equal(r[k].cpu().numpy().view(np.uint32), np.asarray(ref[k]).astype(np.uint32)), k


def test_the_tree_launches_no_step_loop(dev):
    import oracle
    import paper_2101_03240_amd as ibip

    img = synth.blurred_noise((90, 80, 100), 3.0, 0.6, 4)
    inl = synth.face_mask(img.shape, 0, 0)
    ref = oracle.invade(img, inl)
    r, loops = _loops(lambda: ibip.invade(_put(dev, img), _put(dev, inl)))
    assert loops == 0
    _same(r, ref)
    r, loops = _loops(lambda: ibip.invade(_put(dev, img), _put(dev, inl), max_steps=100))
    assert loops > 0
    _same(r, oracle.invade(img, inl, max_steps=100))


# (numbers of steps above a sixteenth of the pore voxels + 4,096)
@pytest.mark.parametrize("side, sigma", [(500, 3.0), (620, 2.0), (1000, 6.0)])
def test_planes_of_many_steps_take_the_tree(dev, side, sigma):
    import oracle
    import paper_2101_03240_amd as ibip

    img = synth.blurred_noise((1, side, side), sigma, 0.6, 1)
    inl = synth.face_mask(img.shape, 1, 0)
    ref = oracle.invade(img, inl)
    assert ref["K"] > int(img.sum()) // 16 + 4096
    r, loops = _loops(lambda: ibip.invade(_put(dev, img), _put(dev, inl)))
    assert loops == 0
    _same(r, ref)


def _plates(shape, width):
    """Parallel plates `width` voxels apart: each distance is one plateau, and the
    one in the middle is searched from the inlet face voxel by voxel."""
    img = np.zeros(shape, np.uint8)
    for i in range(width):
        img[:, :, i::width + 1] = 1
    img[-1, -1, -1] = 0
    return img


# levels that leave more than 2^15 voxels after their first rounds, for 40 to 240
# rounds more (they come back for more rounds once, or twice)
@pytest.mark.parametrize("name, shape", [("plates 1", (120, 90, 40)), ("plates 2", (60, 100, 63)),
                                         ("plates 7", (250, 100, 64)), ("salt", (90, 100, 110))])
def test_plateaus(dev, name, shape):
    import oracle
    import paper_2101_03240_amd as ibip

    rng = np.random.default_rng(3)
    img = ((rng.random(shape) < 0.6).astype(np.uint8) if name == "salt"
           else _plates(shape, int(name.split()[1])))
    inl = synth.face_mask(img.shape, 0, 0)
    ref = oracle.invade(img, inl)
    r = ibip.invade(_put(dev, img), _put(dev, inl))
    _same(r, ref)
    b = ibip.invade_batch([_put(dev, img)] * 2, [_put(dev, inl)] * 2)
    for x in b:
        _same(x, ref)
    with ibip.Server(dev, hbm_budget_bytes=1 << 30, max_inflight=2) as srv:
        _same(srv.wait(srv.submit(_put(dev, img), _put(dev, inl))), ref)


def _in_thread(fn):
    """fn on a thread of its own: a context that holds no scratch yet."""
    import concurrent.futures as cf
    with cf.ThreadPoolExecutor(1) as pool:
        return pool.submit(fn).result()


def _fill(dev, left):
    """Tensors that leave `left` bytes of the device (what is free is known a little late)."""
    import torch

    fill = []
    for _ in range(3):
        room = torch.cuda.mem_get_info(dev)[0] - left
        if room > 0:
            fill.append(torch.empty(room, dtype=torch.uint8, device=dev))
    return fill


def test_no_room_for_the_tree(dev):
    """On a device that is nearly full the invasion runs its step loop in the
    scratch that it has; the tree's scratch, once there, makes room for other calls'."""
    import torch

    import paper_2101_03240_amd as ibip

    img = synth.blurred_noise_device((256, 256, 256), 4.0, 0.6, 2, dev)
    img[-1, -1, -1] = 0
    inl = _put(dev, synth.face_mask(img.shape, 0, 0))
    long_img = torch.cat([img, img])
    d = _in_thread(lambda: ibip.edt(long_img))

    def work():
        ibip.invade(img, inl, max_steps=3)  # the step loop's scratch
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        keep = [torch.empty(img.numel() * 4, dtype=torch.uint8, device=dev) for _ in range(8)]
        fill = _fill(dev, 96 << 20)  # (the tree takes 550 MB)
        del keep  # (the results' memory)
        r, loops = _loops(lambda: ibip.invade(img, inl))
        del fill
        torch.cuda.empty_cache()
        r2, loops2 = _loops(lambda: ibip.invade(img, inl))
        torch.cuda.empty_cache()
        keep = torch.empty(long_img.numel() * 4, dtype=torch.uint8, device=dev)
        fill = _fill(dev, 32 << 20)  # (the distances' scratch grows by 100 MB)
        del keep
        return r, loops, r2, loops2, ibip.edt(long_img)

    try:
        r, loops, r2, loops2, d2 = _in_thread(work)
    finally:
        torch.cuda.empty_cache()  # (the memory that filled the device)
    assert loops > 0 and loops2 == 0
    assert r["K"] == r2["K"]
    for k in ("centre_step", "seq", "rad2", "M"):
        assert torch.equal(r[k], r2[k]), k
    assert torch.equal(d, d2)


# thin images, whose tiles hold few voxels: lists for whatever the image holds, and
# for an eighth and half of the voxels
@pytest.mark.parametrize("shape", [(900, 700, 1), (1500, 1000, 1), (1100, 1, 1200), (900, 800, 2), (4, 3, 30000)])
def test_thin_images(dev, shape):
    import oracle
    import paper_2101_03240_amd as ibip

    img = np.ascontiguousarray(synth.blurred_noise((1, 1500, 1200), 3.0, 0.6, 6)[0].reshape(-1)[:np.prod(shape)]
                               .reshape(shape))
    img[-1, -1, -1] = 0
    axis = 2 if shape[2] > 2 else 0
    inl, out = synth.face_mask(shape, axis, 0), synth.face_mask(shape, axis, shape[axis] - 1)
    ref = oracle.invade(img, inl)
    r = ibip.invade(_put(dev, img), _put(dev, inl))
    _same(r, ref)
    t, rt = ibip.trap(r["seq"], _put(dev, out)), oracle.trap(ref["seq"], out)
    assert np.array_equal(t["seq_trapped"].cpu().numpy(), rt["seq_trapped"])
    T = [25, 9, 4, 1]
    m, rm = ibip.opening_drainage(_put(dev, img), _put(dev, inl), T), oracle.mio(img, inl, np.array(T, np.uint32))
    assert np.array_equal(m["mio_r2"].cpu().numpy().view(np.uint32), rm["mio_r2"])


def _beside(a, b):
    """Two images side by side along x or y, a wall of solid between them, and
    inlets: the first face of `a` along that axis, of `b` along the last axis."""
    axis = 1 if a.shape[0] == 1 else 0
    wall = np.zeros([1 if i == axis else n for i, n in enumerate(a.shape)], np.uint8)
    return (np.concatenate([a, wall, b], axis=axis),
            np.concatenate([synth.face_mask(a.shape, axis, 0), wall, synth.face_mask(b.shape, 2, 0)], axis=axis))


def _serpentine(n):
    """One channel of width 1 that runs through n x n pixels, from y = 1, z = 0."""
    img = np.zeros((1, n, n), np.uint8)
    img[0, 1::2] = 1
    for i, y in enumerate(range(2, n, 2)):
        img[0, y, n - 1 if i % 2 == 0 else 0] = 1
    return img


def _comb(n, depth):
    """A corridor of width 1 with a dead-end chamber of width 3 every six pixels."""
    img = np.zeros((1, depth + 8, n), np.uint8)
    img[0, 1] = 1
    for x in range(2, n - 4, 6):
        img[0, 2:4, x + 1] = 1
        img[0, 4:4 + depth, x:x + 3] = 1
    return img


def _form(name):
    rng = np.random.default_rng(11)
    if name == "serpentine":  # as many rounds of one level as it has pixels
        return _beside(_serpentine(161), synth.blurred_noise((1, 700, 161), 2.0, 0.6, 3))
    if name == "long serpentine":  # more steps than a quarter of the pore voxels
        return _beside(_serpentine(401), synth.blurred_noise((1, 160, 401), 2.0, 0.6, 3))
    if name == "comb":  # components entered one by one in the rounds of one level
        return _beside(_comb(2000, 9), synth.blurred_noise((1, 90, 2000), 2.0, 0.6, 4))
    if name == "salt":  # levels of many voxels, long searches
        return _beside((rng.random((48, 60, 62)) < 0.62).astype(np.uint8),
                       synth.blurred_noise((90, 60, 62), 2.0, 0.6, 5))
    if name == "isolated":  # more peaks than an eighth of the pore voxels
        img = np.zeros((80, 80, 100), np.uint8)
        img[::2, ::2, ::2] = 1
        img[0] = 1
        return _beside(img, synth.blurred_noise((60, 80, 100), 2.0, 0.6, 6))
    if name == "wide levels":
        img = synth.blurred_noise((120, 130, 140), 3.0, 0.6, 3)
    else:
        img = synth.overlapping_spheres((130, 110, 100), r2=40, porosity=0.5, seed=2)
    return img, synth.face_mask(img.shape, 2, 0)


# (gives up: the tree starts, runs out of room for peaks or for steps, and the step
# loop takes over)
@pytest.mark.parametrize("name, gives_up", [("serpentine", False), ("long serpentine", True), ("comb", False),
                                            ("salt", False), ("isolated", True), ("wide levels", False),
                                            ("grains", False)])
def test_forms_of_the_tree(dev, name, gives_up):
    import oracle
    import paper_2101_03240_amd as ibip

    img, inl = _form(name)
    ref = oracle.invade(img, inl)
    r, loops = _loops(lambda: ibip.invade(_put(dev, img), _put(dev, inl)))
    assert (loops > 0) == gives_up
    _same(r, ref)
    K = ref["K"]
    for lim in (K - 1, K, 10 ** 9):
        r, loops = _loops(lambda: ibip.invade(_put(dev, img), _put(dev, inl), max_steps=lim))
        if lim > K or K > 3000:  # (below, the loop ends sooner)
            assert (loops > 0) == gives_up
        _same(r, oracle.invade(img, inl, max_steps=lim))


# small images, step limits that come before the tree would be done, and images of
# one rank, or of one rank for almost all of them
@pytest.mark.parametrize("name, limit", [("small", 0), ("small plane", 0), ("limit", 1023), ("limit", 1024),
                                         ("limit", 6000), ("plates", 0), ("salt", 0)])
def test_calls_that_the_step_loop_does_sooner(dev, name, limit):
    import oracle
    import paper_2101_03240_amd as ibip

    img = {"small": lambda: synth.blurred_noise((24, 30, 28), 2.0, 0.6, 1),
           "small plane": lambda: synth.blurred_noise((1, 90, 88), 4.0, 0.6, 2),
           "limit": lambda: synth.blurred_noise((180, 180, 180), 4.0, 0.6, 3),
           "plates": lambda: _plates((120, 90, 40), 2),
           "salt": lambda: (np.random.default_rng(3).random((60, 70, 80)) < 0.6).astype(np.uint8)}[name]()
    inl = synth.face_mask(img.shape, 2, 0)
    r, loops = _loops(lambda: ibip.invade(_put(dev, img), _put(dev, inl), max_steps=limit))
    assert loops > 0
    _same(r, oracle.invade(img, inl, max_steps=limit))


def _corner(shape):
    """One solid voxel, in the corner: as many ranks as its box has distances."""
    img = np.ones(shape, np.uint8)
    img[0, 0, 0] = 0
    return img


def _batch_form(name):
    noise = [synth.blurred_noise((90 + 3 * i, 80, 90 - 2 * i), 2.5, 0.6, i) for i in range(5)]
    if name == "isolated":  # more peaks than the group has room for
        img = np.zeros((160, 120, 120), np.uint8)
        img[::2, ::2, ::2] = 1
        img[0] = 1
        return noise[:2] + [img]
    if name == "ranks":  # each has fewer than 8,192, all together more
        return noise + [_corner((1, 120, 120)), _corner((24, 24, 90))]
    if name == "plates":
        return [_plates((160, 90, 80), 1), _plates((140, 80, 90), 2), _plates((1, 70, 60), 1)]
    return noise


# (which the tree gives up or does not take: one launch runs all step loops)
@pytest.mark.parametrize("name, gives_up", [("noise", False), ("isolated", True), ("ranks", True), ("plates", True)])
def test_batches_that_give_up_stay_batches(dev, name, gives_up):
    import oracle
    import paper_2101_03240_amd as ibip

    imgs = _batch_form(name)
    inls = [synth.face_mask(i.shape, 2, 0) for i in imgs]
    out, loops = _loops(lambda: ibip.invade_batch([_put(dev, i) for i in imgs], [_put(dev, i) for i in inls], sat=True))
    assert loops == (1 if gives_up else 0)
    for img, inl, b in zip(imgs, inls, out):
        ref = oracle.invade(img, inl)
        assert b["status"] == 0
        _same(b, ref)
        n = np.bincount(ref["seq"][ref["seq"] > 0], minlength=ref["K"] + 1)[1:]
        assert np.array_equal(b["sat"].cpu().numpy(), np.cumsum(n) / float((img != 0).sum()))


def test_a_batch_without_room_for_its_tree(dev):
    import torch

    import paper_2101_03240_amd as ibip

    imgs = [synth.blurred_noise_device((128, 128, 128), 3.0, 0.6, i, dev) for i in range(4)]
    for i in imgs:
        i[-1, -1, -1] = 0
    inls = [_put(dev, synth.face_mask((128, 128, 128), 0, 0))] * 4

    def work():
        ibip.invade_batch(imgs, inls, max_steps=9)  # the step loops' scratch
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        keep = [torch.empty(4 * imgs[0].numel(), dtype=torch.uint8, device=dev) for _ in range(20)]
        fill = _fill(dev, 64 << 20)  # (the tree takes 250 MB)
        del keep
        a = _loops(lambda: ibip.invade_batch(imgs, inls))
        del fill
        torch.cuda.empty_cache()
        return a, _loops(lambda: ibip.invade_batch(imgs, inls))

    try:
        (a, la), (b, lb) = _in_thread(work)
    finally:
        torch.cuda.empty_cache()
    assert (la, lb) == (1, 0)
    for x, y in zip(a, b):
        assert x["K"] == y["K"]
        for k in ("centre_step", "seq", "rad2", "M"):
            assert torch.equal(x[k], y[k]), k


def _scratch():
    """Bytes of scratch that this thread's context holds."""
    import torch

    import paper_2101_03240_amd as ibip
    return ibip.load_library().ibip_ctx_scratch_bytes(ibip._context(torch.device("cuda", torch.cuda.current_device())))


# images of other rows, planes and orientations than their neighbours': groups of
# their own instead of up to 256 times their voxels of padding, each in its layout
@pytest.mark.parametrize("shapes", [[(8, 400, 400), (400, 400, 8), (400, 8, 400)],
                                    [(1, 900, 910), (900, 1, 910), (910, 900, 1), (1, 7, 9), (61, 1, 1), (1, 1, 53)],
                                    [(200, 200, 200)] + [(20, 21, 22)] * 20,
                                    [(40, 100, 105), (105, 40, 100), (100, 105, 40), (120, 27, 600), (600, 120, 27)],
                                    [(13, 33, 35), (35, 13, 33), (33, 35, 13)]])
def test_batches_of_uneven_shapes(dev, shapes):
    import oracle
    import paper_2101_03240_amd as ibip

    rng = np.random.default_rng(5)
    imgs = [synth.blurred_noise(s, 1.5, 0.65, i) if min(s) > 5 else (rng.random(s) < 0.85).astype(np.uint8)
            for i, s in enumerate(shapes)]
    inls = [(rng.random(s) < 0.01).astype(np.uint8) for s in shapes]
    for i in imgs:
        i[-1, -1, -1] = 0

    def work():
        return ibip.invade_batch([_put(dev, i) for i in imgs], [_put(dev, i) for i in inls], sat=True), _scratch()

    out, scratch = _in_thread(work)
    assert scratch < 200 * sum(i.size for i in imgs) + (2200 << 20)
    for img, inl, b in zip(imgs, inls, out):
        ref = oracle.invade(img, inl)
        assert b["status"] == 0
        _same(b, ref)
        n = np.bincount(ref["seq"][ref["seq"] > 0], minlength=ref["K"] + 1)[1:]
        assert np.array_equal(b["sat"].cpu().numpy(), np.cumsum(n) / float((img != 0).sum()))


# served jobs: by the step loop at once (small), by the tree, by a tree that gives up
# (the loop takes over), by the loop after their ranks are known, and without room for
# the tree; told by the pool's peak
@pytest.mark.parametrize("name, room, tree", [("small", 1 << 30, False), ("wide levels", 1 << 30, True),
                                              ("isolated", 1 << 30, True), ("long serpentine", 1 << 30, True),
                                              ("plates", 1 << 30, False), ("wide levels", 80 << 20, False)])
def test_served_paths(dev, name, room, tree):
    import oracle
    import paper_2101_03240_amd as ibip

    if name == "small":
        img = synth.blurred_noise((20, 24, 26), 2.0, 0.6, 1)
        inl = synth.face_mask(img.shape, 0, 0)
    elif name == "plates":
        img = _plates((160, 90, 80), 1)
        inl = synth.face_mask(img.shape, 0, 0)
    else:
        img, inl = _form(name)
    d_img, d_inl = _put(dev, img), _put(dev, inl)
    with ibip.Server(dev, hbm_budget_bytes=room, max_inflight=2) as srv:
        srv.wait(srv.submit(d_img, d_inl, max_steps=2))
        loop_peak = srv.stats()["peak_bytes"]
        b = srv.wait(srv.submit(d_img, d_inl))
        assert (srv.stats()["peak_bytes"] > loop_peak) == tree
        assert srv.stats()["bytes_in_use"] == 0
    assert b["status"] == 0
    _same(b, oracle.invade(img, inl))


# 26-connected: with room for all edges, and (volumes of more) by the tiles' sweeps
@pytest.mark.parametrize("shape", [(60, 70, 80), (110, 100, 104), (2, 800, 900), (1, 1100, 1000)])
def test_trapping_26_connected(dev, shape):
    import oracle
    import paper_2101_03240_amd as ibip

    img = synth.blurred_noise(shape, 2.0, 0.6, 9)
    inl, out = synth.face_mask(shape, 2, 0), synth.face_mask(shape, 2, shape[2] - 1)
    seq = oracle.invade(img, inl)["seq"]
    t, r = ibip.trap(_put(dev, seq), _put(dev, out), connectivity=26), oracle.trap(seq, out, conn=26)
    assert np.array_equal(t["trapped"].cpu().numpy(), r["trapped"])
    assert np.array_equal(t["seq_trapped"].cpu().numpy(), r["seq_trapped"])


def test_served_trees_short_of_room(dev):
    """A pool with room for three jobs' scratch and one tree: some jobs have a tree,
    some run their loops, and every ticket comes back."""
    import oracle
    import paper_2101_03240_amd as ibip

    img = synth.blurred_noise((120, 130, 128), 3.0, 0.6, 3)
    inl = synth.face_mask(img.shape, 0, 0)
    ref = oracle.invade(img, inl)
    n = img.size
    d_img, d_inl = _put(dev, img), _put(dev, inl)
    with ibip.Server(dev, hbm_budget_bytes=3 * 27 * n + 36 * n, max_inflight=4) as srv:
        ts = [srv.submit(d_img, d_inl) for _ in range(7)]
        res = [srv.wait(t) for t in ts]
        st = srv.stats()
    assert st["bytes_in_use"] == 0 and st["running"] == 0 and st["completed"] == 7
    for b in res:
        assert b["status"] == 0
        _same(b, ref)
