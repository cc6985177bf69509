"""The work that users of this library have it do, as measurable cases.

Every case goes through the public entry points of ``paper_2101_03240_amd``
on inputs made from a seed: the distance transform alone, the drainage
(invasion, then trapping) of one image, trapping alone, the opening drainage,
the 2D comparison of the two methods, a batch of uneven images and a stream of
served requests. Sizes are those of the benchmark and the tests, and odd ones
between them.
"""
from __future__ import annotations

import heapq
import math

import numpy as np
import torch

import paper_2101_03240_amd as ibip
from paper_2101_03240_amd import synth


def _case(name, op, x, y, z, kind, porosity, sigma=6.0, r2=16, conn=6, radii=0, count=1):
    """kind: "noise" (blurred noise of width sigma) or "balls" (overlapping
    solid balls of squared radius r2). conn: trapping connectivity. radii:
    opening radii. count: images of a batch or a stream, their sides drawn
    between z and y."""
    return {"name": name, "op": op, "x": x, "y": y, "z": z, "kind": kind, "porosity": porosity, "sigma": sigma,
            "r2": r2, "conn": conn, "radii": radii, "count": count}


def listed():
    return [
        # one 2D image of the size the paper shows: the smallest call, launches and latency
        _case("edt 2d 500", "edt", 1, 500, 500, "noise", 0.60),
        # a scan cropped to odd sides
        _case("edt odd 301", "edt", 301, 287, 313, "noise", 0.55),
        # the distance transform of the benchmark's image
        _case("edt 512", "edt", 512, 512, 512, "noise", 0.55),
        # the 2D comparison of invasion, opening and trapping (every call once), a study's inner loop
        _case("figure 2d 500", "figure", 1, 500, 500, "noise", 0.60),
        # a small subvolume: drainage with trapping, bound by latency
        _case("drain 64", "drain", 64, 64, 64, "balls", 0.65),
        # an ordinary bead pack, inlet to outlet
        _case("drain grains 200", "drain", 200, 200, 200, "balls", 0.40, r2=144),
        # the benchmark's image, the largest single call
        _case("drain 512", "drain", 512, 512, 512, "noise", 0.55),
        # trapping of an invasion already at hand (other outlets), ragged sides
        _case("trap ragged", "trap", 230, 171, 199, "noise", 0.55),
        # pressure-based drainage of the bead pack at the comparison's radii
        _case("opening grains 200", "opening", 200, 200, 200, "balls", 0.40, r2=144, radii=25),
        # one opening of the benchmark's image
        _case("opening 512", "opening", 512, 512, 512, "noise", 0.55, radii=1),
        # many subvolumes of uneven size in one call
        _case("batch 20", "batch", 0, 192, 32, "noise", 0.55, count=20),
        # requests that arrive together at a server kept open
        _case("serve 12", "serve", 0, 256, 64, "noise", 0.55, count=12),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["edt", "edt", "drain", "drain", "drain", "trap", "opening", "opening", "figure", "batch",
                     "serve"])
    porosity = round(rng.uniform(0.40, 0.65), 3)
    if op in ("batch", "serve"):
        lo, hi = (32, 192) if op == "batch" else (64, 256)
        return _case("", op, 0, _log_int(rng, 2 * lo, hi), lo, "noise", porosity, sigma=round(rng.uniform(3, 6), 2),
                     count=rng.randint(6, 20 if op == "batch" else 12))
    if op == "figure":
        return _case("", op, 1, _log_int(rng, 120, 500), _log_int(rng, 120, 500), rng.choice(["noise", "balls"]),
                     porosity=round(rng.uniform(0.5, 0.65), 3), r2=rng.randint(16, 144))
    top = {"edt": 512, "drain": 360, "trap": 360, "opening": 360}[op]
    x, y, z = (_log_int(rng, 40, top) for _ in range(3))
    if rng.random() < 0.2:
        x = 1  # a 2D image
    if rng.random() < 0.3:
        z = min(top, (z + 7) // 8 * 8)
    kind = "balls" if rng.random() < 0.4 else "noise"
    # grains of a size that a few thousand of them fill the image
    r = max(3.0, (x * y * z / 12000.0) ** (1 / 3) * rng.uniform(1.0, 1.8))
    return _case("", op, x, y, z, kind, porosity, sigma=round(rng.uniform(3, 8), 2), r2=int(min(r * r, 400)),
                 conn=rng.choice([6, 6, 26]) if op == "trap" else 6,
                 radii=rng.choice([1, 5, 25]) if op == "opening" else 0)


def _device():
    return torch.device("cuda", torch.cuda.current_device())


def _balls(shape, porosity, r2, seed):
    """Boolean model: solid balls (disks in 2D) of three radii about
    sqrt(r2), integer centres uniform in the box extended by a radius, as many
    as leave `porosity` on average."""
    rng = np.random.Generator(np.random.PCG64(seed))
    dims = [n for n in shape if n > 1] or [1]
    flat = torch.ones(math.prod(dims), dtype=torch.uint8, device=_device())
    for f in (0.75, 1.0, 1.25):
        r = max(1, int(round(math.sqrt(r2) * f)))
        o = np.stack(np.meshgrid(*[np.arange(-r, r + 1)] * len(dims), indexing="ij"), -1).reshape(-1, len(dims))
        o = o[(o * o).sum(1) <= r * r]
        count = int(math.ceil(-math.log(porosity) / 3 * math.prod(n + 2 * r + 1 for n in dims) / len(o)))
        c = np.stack([rng.integers(-r, n + r + 1, size=count) for n in dims], 1)
        o_d, c_d = torch.from_numpy(o).to(flat.device), torch.from_numpy(c).to(flat.device)
        per = max(1, (1 << 25) // len(o))
        for i in range(0, count, per):
            ok, at = True, 0
            for a, n in enumerate(dims):
                p = c_d[i:i + per, None, a] + o_d[None, :, a]
                ok = ok & (p >= 0) & (p < n)
                at = at * n + p
            flat[at[ok]] = 0
    return flat.reshape(tuple(shape))


def _image(shape, kind, porosity, sigma, r2, seed):
    if kind == "balls":
        img = _balls(shape, porosity, r2, seed)
    else:
        # a crop of a field with sides of a power of two, whose transforms are ready sooner
        side = max(64, 1 << (max(shape) - 1).bit_length())
        field = synth.blurred_noise_device(tuple(side if n > 1 else 1 for n in shape), sigma, porosity, seed, _device())
        img = field[tuple(slice(0, n) for n in shape)].contiguous()
    img[-1, -1, -1] = 0  # an image without solid has no distance transform
    return img


def _face(shape, axis, index):
    m = torch.zeros(tuple(shape), dtype=torch.uint8, device=_device())
    m.select(axis, index).fill_(1)
    return m


def _case_image(case, seed):
    return _image((case["x"], case["y"], case["z"]), case["kind"], case["porosity"], case["sigma"], case["r2"], seed)


def _thresholds(dt2_max, n):
    """T_i = max(1, ceil((r_max i / n)^2)) for i = n..1, duplicates removed."""
    r = math.sqrt(dt2_max)
    return sorted({max(1, math.ceil((r * i / n) ** 2)) for i in range(1, n + 1)}, reverse=True)


_kept = {}


def _server():
    # a server lives as long as its program
    if "server" not in _kept:
        _kept["server"] = ibip.Server(hbm_budget_bytes=4 << 30)
    return _kept["server"]


class _Table:
    """Per-step (or per-level) arrays of one image, kept in rows of a fixed
    length as a study keeps them: their true length depends on the image."""

    def __init__(self, rows):
        self.rows, self.cols = rows, {}

    def put(self, name, a):
        t = self.cols.get(name)
        if t is None:
            t = self.cols[name] = torch.zeros(self.rows, dtype=a.dtype, device=a.device)
        t[:a.numel()].copy_(a)
        return t


_STEPS = ("M", "n_new", "sat", "pc")


def _filed(table, prefix, d):
    """The dict `d` of a call, its per-step arrays filed in the table."""
    return {k: table.put(prefix + k, v) if k in _STEPS else v for k, v in d.items()}


def _step_rows(n):
    return max(n // 32, 65536)


def _sides(case):
    """The sides of a batch's or a stream's images: log-uniform between z and
    y, the same for every seed."""
    rng = np.random.Generator(np.random.PCG64(1000 * case["y"] + case["count"]))
    u = rng.uniform(math.log(case["z"]), math.log(case["y"]), size=case["count"])
    return [case["y"]] + [int(round(math.exp(v))) for v in u[1:]]


def prepare(case, seed):
    op = case["op"]
    if op in ("batch", "serve"):
        imgs = [_image((s, s, s), "noise", case["porosity"], min(case["sigma"], 2 + s / 40), 0, seed * 1000 + i)
                for i, s in enumerate(_sides(case))]
        st = {"case": case, "imgs": imgs, "inlets": [_face(i.shape, 0, 0) for i in imgs],
              "tables": [_Table(_step_rows(i.numel())) for i in imgs]}
        if op == "serve":
            st["server"] = _server()
        return st
    img = _case_image(case, seed)
    axis = 0 if img.shape[0] > 1 else 1
    st = {"case": case, "img": img, "inlets": _face(img.shape, axis, 0), "outlets": _face(img.shape, axis, -1),
          "steps": _Table(_step_rows(img.numel())), "levels": _Table(4096)}
    if op == "trap":
        st["seq"] = ibip.invade(img, st["inlets"], rad2=False, centre_step=False, steps=False)["seq"]
    if op == "opening":
        d = ibip.edt(img)
        if case["radii"] == 1:
            st["T"] = [int(torch.median(d[d > 0].to(torch.int64)).item())]
        else:
            st["T"] = _thresholds(int(d.max().item()), case["radii"])
    return st


def run(st):
    case = st["case"]
    op = case["op"]
    if op == "edt":
        return {"dt2": ibip.edt(st["img"])}
    if op == "drain":
        r = ibip.invade(st["img"], st["inlets"])
        t = ibip.trap(r["seq"], st["outlets"])
        return {"invasion": _filed(st["steps"], "", r), "trapping": t}
    if op == "trap":
        return ibip.trap(st["seq"], st["outlets"], connectivity=case["conn"])
    if op == "opening":
        o = ibip.opening_drainage(st["img"], st["inlets"], st["T"])
        return {"mio_r2": o["mio_r2"], "mio_sat": np.array(o["mio_sat"] + [0.0] * (case["radii"] - len(st["T"])))}
    if op == "figure":
        r = ibip.invade(st["img"], st["inlets"])
        s = ibip.saturation(r["seq"], r["M"])
        t = ibip.trap(r["seq"], st["outlets"])
        Ma = ibip.remap_steps(r["seq"], t["seq_trapped"], r["M"], t["K_after"])
        sa = ibip.saturation(t["seq_trapped"], Ma)
        T = torch.unique(r["M"]).flip(0).tolist()
        o = ibip.opening_drainage(st["img"], st["inlets"], T)
        c = ibip.compare_opening(s["satmap"], o["mio_r2"], T, o["mio_sat"], t["trapped"])
        steps, levels = st["steps"], st["levels"]
        return {"invasion": _filed(steps, "", r), "curves": _filed(steps, "curves ", s), "trapping": t,
                "M_after": steps.put("M after", Ma), "curves_after": _filed(steps, "after ", sa),
                "mio_r2": o["mio_r2"],
                "mio_sat": levels.put("mio_sat", torch.tensor(o["mio_sat"], dtype=torch.float64)),
                "comparison": {k: levels.put(k, v) for k, v in c.items()}}
    if op == "batch":
        out = ibip.invade_batch(st["imgs"], st["inlets"], rad2=False, centre_step=False)
        return [{"seq": o["seq"], "M": t.put("M", o["M"]), "K": o["K"]} for o, t in zip(out, st["tables"])]
    srv = st["server"]
    tickets = [srv.submit(i, l, rad2=False, centre_step=False) for i, l in zip(st["imgs"], st["inlets"])]
    out = [srv.wait(t) for t in tickets]
    return [{"seq": o["seq"], "M": t.put("M", o["M"]), "K": o["K"]} for o, t in zip(out, st["tables"])]


def work(case):
    """Inputs read once, outputs written once. The operations are those of the
    definitions at one comparison or addition per voxel and neighbour."""
    op, c = case["op"], case
    n = c["x"] * c["y"] * c["z"]
    pore = c["porosity"]
    if op in ("batch", "serve"):
        n = sum(a ** 3 for a in _sides(c))
        return {"bytes": 6.0 * n, "flops": 20.0 * pore * n}  # image, inlets; seq
    if op == "edt":
        return {"bytes": 5.0 * n, "flops": 6.0 * n}  # image; dt2
    if op == "trap":
        return {"bytes": 10.0 * n, "flops": 6.0 * pore * n}  # seq, outlets; trapped, seq_trapped
    if op == "opening":
        return {"bytes": 6.0 * n, "flops": 6.0 * n * (1 + c["radii"])}  # image, inlets; mio_r2
    if op == "drain":
        # image, inlets, outlets; seq, rad2, centre_step, trapped, seq_trapped
        return {"bytes": 20.0 * n, "flops": 30.0 * pore * n}
    # figure: as drain, and satmap, satmap after trapping, mio_r2
    return {"bytes": 40.0 * n, "flops": 60.0 * pore * n}


# ---------------------------------------------------------------------------
# The values of the definitions, for images small enough to take in plain
# numpy and torch.
# ---------------------------------------------------------------------------
def _edt_exact(img):
    """Squared distances to the nearest solid voxel, axis by axis, in int64."""
    big = 1 << 40
    d = torch.where(img != 0, big, 0).to(torch.int64)
    for ax in range(3):
        L = d.shape[ax]
        m = d.movedim(ax, -1).contiguous()
        flat = m.reshape(-1, L)
        i = torch.arange(L, device=d.device)
        sq = (i[:, None] - i[None, :]) ** 2
        out = torch.empty_like(flat)
        step = max(1, (1 << 26) // (L * L))
        for r in range(0, flat.shape[0], step):
            out[r:r + step] = (flat[r:r + step, None, :] + sq[None]).amin(2)
        d = out.reshape(m.shape).movedim(-1, ax).contiguous()
    return d


def _invade_exact(img, inlets, dt2):
    """The invasion loop of the definition: seq, rad2, centre_step and M."""
    X, Y, Z = img.shape
    dims = (X, Y, Z)

    def around(v):
        z, y, x = v % Z, v // Z % Y, v // (Y * Z)
        if x > 0:
            yield v - Y * Z
        if x < X - 1:
            yield v + Y * Z
        if y > 0:
            yield v - Z
        if y < Y - 1:
            yield v + Z
        if z > 0:
            yield v - 1
        if z < Z - 1:
            yield v + 1

    d = dt2.reshape(-1).tolist()
    seen = [False] * len(d)
    heap = []

    def push(v):
        if d[v] and not seen[v]:
            seen[v] = True
            heapq.heappush(heap, (-d[v], v))

    for v in np.flatnonzero(inlets.reshape(-1)).tolist():
        push(v)
        for u in around(v):
            push(u)
    seq = np.where(img != 0, 0, -1).astype(np.int64)
    rad2 = np.zeros(dims, np.int64)
    cs = np.zeros(img.size, np.int64)
    M = []
    balls = {}
    while heap:
        m = -heap[0][0]
        M.append(m)
        k = len(M)
        popped = []
        while heap and -heap[0][0] == m:
            popped.append(heapq.heappop(heap)[1])
        for v in popped:
            cs[v] = k
            for u in around(v):
                push(u)
        r = math.isqrt(m - 1)
        if m not in balls:
            o = np.arange(-r, r + 1) ** 2
            balls[m] = (o[:, None, None] + o[None, :, None] + o[None, None, :]) < m
        for v in popped:
            at = (v // (Y * Z), v // Z % Y, v % Z)
            lo = [max(0, a - r) for a in at]
            hi = [min(n, a + r + 1) for a, n in zip(at, dims)]
            part = tuple(slice(a, b) for a, b in zip(lo, hi))
            b = balls[m][tuple(slice(l - a + r, h - a + r) for l, h, a in zip(lo, hi, at))]
            new = b & (seq[part] == 0)
            seq[part][new] = k
            rad2[part][new] = m
    return seq, rad2, cs.reshape(dims), np.array(M, np.int64)


def _trap_exact(seq, outlets):
    """Trapped voxels, the re-ranked sequence and the steps left: the widest
    path from the outlets, by decreasing smallest step along it."""
    X, Y, Z = seq.shape
    s = seq.reshape(-1).tolist()
    top = max(max(s), 0) + 1
    w = [-1] * len(s)
    heap = []
    for v in np.flatnonzero(outlets.reshape(-1)).tolist():
        if s[v] >= 0:
            w[v] = s[v] or top
            heapq.heappush(heap, (-w[v], v))
    while heap:
        c, v = heapq.heappop(heap)
        c = -c
        if c < w[v]:
            continue
        z, y, x = v % Z, v // Z % Y, v // (Y * Z)
        for ok, u in ((x > 0, v - Y * Z), (x < X - 1, v + Y * Z), (y > 0, v - Z), (y < Y - 1, v + Z),
                      (z > 0, v - 1), (z < Z - 1, v + 1)):
            if ok and s[u] >= 0:
                t = min(c, s[u] or top)
                if t > w[u]:
                    w[u] = t
                    heapq.heappush(heap, (-t, u))
    a, wa = seq.reshape(-1), np.array(w, np.int64)
    trapped = (a > 0) & (wa < a)
    left = np.unique(a[(a > 0) & ~trapped])
    after = np.where(a < 0, -1, 0)
    keep = (a > 0) & ~trapped
    after[keep] = np.searchsorted(left, a[keep]) + 1
    return trapped.reshape(seq.shape), after.reshape(seq.shape), left


def _curves_exact(seq, M, satmap=True):
    n_new = np.bincount(seq[seq > 0], minlength=len(M) + 1)[1:]
    sat = np.cumsum(n_new) / float((seq >= 0).sum())
    out = {"n_new": n_new, "sat": sat, "pc": 2.0 / np.sqrt(M.astype(np.float64))}
    if satmap:
        m = np.where(seq < 0, -1.0, 0.0)
        m[seq > 0] = sat[seq[seq > 0] - 1]
        out["satmap"] = m
    return out


def _opening_exact(img, inlets, dt2, T):
    """Opening at each squared radius: centres of dt2 >= T joined to the inlet
    candidates, dilated by the ball. The join is a widest path over dt2."""
    X, Y, Z = img.shape
    d = dt2.reshape(-1).tolist()
    K = [0] * len(d)
    heap = []

    def around(v):
        z, y, x = v % Z, v // Z % Y, v // (Y * Z)
        return [u for ok, u in ((x > 0, v - Y * Z), (x < X - 1, v + Y * Z), (y > 0, v - Z), (y < Y - 1, v + Z),
                                (z > 0, v - 1), (z < Z - 1, v + 1)) if ok]

    def offer(u, c):
        t = min(c, d[u])
        if t > K[u]:
            K[u] = t
            heapq.heappush(heap, (-t, u))

    for v in np.flatnonzero(inlets.reshape(-1)).tolist():
        for u in [v] + around(v):
            offer(u, 1 << 40)
    while heap:
        c, v = heapq.heappop(heap)
        if -c == K[v]:
            for u in around(v):
                offer(u, -c)
    kept = torch.from_numpy(np.array(K, np.int64).reshape(img.shape)).to(_device())
    r2 = torch.zeros(img.shape, dtype=torch.int64, device=kept.device)
    for t in T:
        near = _edt_exact((kept < t).to(torch.uint8)) < t
        r2[near & (r2 == 0)] = t
    n_pore = float((img != 0).sum())
    return r2.cpu().numpy(), np.array([float((r2 >= t).sum()) / n_pore for t in T])


def _padded(a, rows):
    return np.concatenate([a, np.zeros(rows - len(a), a.dtype)])


def exact(case, seed):
    op = case["op"]
    n = case["x"] * case["y"] * case["z"]
    if op == "edt":
        if n > 1 << 25:
            return None
        return {"dt2": _edt_exact(_case_image(case, seed))}
    if op not in ("drain", "figure") or n > 300000:
        return None
    img_d = _case_image(case, seed)
    axis = 0 if img_d.shape[0] > 1 else 1
    img, dt2 = img_d.cpu().numpy(), _edt_exact(img_d).cpu().numpy()
    inlets = _face(img_d.shape, axis, 0).cpu().numpy()
    outlets = _face(img_d.shape, axis, -1).cpu().numpy()
    seq, rad2, cs, M = _invade_exact(img, inlets, dt2)
    trapped, after, left = _trap_exact(seq, outlets)
    rows = _step_rows(n)

    def curves(q, m, satmap):
        return {k: _padded(v, rows) if k in _STEPS else v for k, v in _curves_exact(q, m, satmap).items()}

    r = dict(curves(seq, M, False), seq=seq, rad2=rad2, centre_step=cs, K=len(M), M=_padded(M, rows))
    t = {"trapped": trapped, "seq_trapped": after, "K_after": len(left)}
    if op == "drain":
        return {"invasion": r, "trapping": t}
    s = curves(seq, M, True)
    Ma = M[left - 1]
    T = np.unique(M)[::-1].tolist()
    if n * len(T) * max(img.shape) > 4e10:
        mio_r2 = mio_sat = dis = held = None
    else:
        mio_r2, mio_sat = _opening_exact(img, inlets, dt2, T)
        dis = np.array([int((((s["satmap"] > 0) & (s["satmap"] <= b)) != (mio_r2 >= a)).sum())
                        for a, b in zip(T, mio_sat)])
        held = np.array([int(((mio_r2 >= a) & trapped).sum()) for a in T])
        mio_sat, dis, held = (_padded(a, 4096) for a in (mio_sat, dis, held))
    return {"invasion": r, "curves": s, "trapping": t, "M_after": _padded(Ma, rows),
            "curves_after": curves(after, Ma, True), "mio_r2": mio_r2, "mio_sat": mio_sat,
            "comparison": {"disagree": dis, "mio_trapped": held}}
