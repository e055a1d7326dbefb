"""Timed workloads of the framework: what a program that uses it has it compute.

A simulation keeps a tree and asks for J (``forward``), or rebuilds the tree of
moved elements in every step and asks for J of the active ones (``step``); a fit
of opacities, densities or luminosities takes J and its gradients (``gradient``);
a study of many small media runs them as one forest (``forest``, ``forest_gradient``).
Media, sizes and options are those of the repository's scene generators, its
benchmark and its tests.

``exact`` evaluates the same method in 64-bit torch operations, written here from
its definition (HEALPix rays, radix tree over Morton keys, transmission averages,
opening criterion, particle-particle sphere); derivatives come from autograd with
the discrete decisions frozen.
"""
import math

import numpy as np
import torch

from paper_2310_15235_amd import api, scenes

BANDS = (1.0, 10.0, 100.0, 1000.0)


# ------------------------------------------------------------------ the cases
def _case(name, kind, medium, n, **kw):
    c = dict(name=name, kind=kind, medium=medium, n=n, bands=1, nside=2, leaf=8, theta=0.75,
             active=1.0, keep_depths=False, directed=False, absorption_avg=False,
             scenes=1, mix=0)
    c.update(kw)
    return c


def listed():
    return [
        # The smallest call: J of a test-sized medium on a kept tree (latency, launches).
        _case("forward_1k", "forward", "uniform", 1000, nside=1),
        # A time step of the small named workload: build, then J of every element.
        _case("step_4k", "step", "uniform", 4096, nside=1),
        # A fit on the small differentiation workload: J and its gradients, tree included.
        _case("gradient_4k", "gradient", "lognormal", 4096, bands=2),
        # A fine angular grid (192 rays) on a small clumpy medium of odd size: the
        # particle-particle sets grow with the narrower beams.
        _case("forward_fine_rays", "forward", "lognormal", 9973, bands=3, nside=4),
        # Ten frequency bands, the paper's spectral experiment, on an odd size.
        _case("forward_ten_bands", "forward", "lognormal", 65537, bands=10),
        # A time step of the clumpy workload: build, then J of every element.
        _case("step_clumpy", "step", "lognormal", 2 ** 18, bands=3),
        # The differentiation workload at full size, with the kept far-field depths.
        _case("gradient_clumpy", "gradient", "lognormal", 2 ** 18, bands=2, keep_depths=True),
        # An individual time step: a large diffuse medium rebuilt for 1% active elements.
        _case("step_diffuse_1pct", "step", "isothermal", 2 ** 21, bands=2, nside=4, active=0.01),
        # Gradients of a large diffuse medium, every element a source, 10% receivers.
        _case("gradient_diffuse", "gradient", "isothermal", 1500001, bands=2, nside=4,
              active=0.1),
        # The fixed-opacity cloud test with the paper's bucket size, its receivers a shell
        # and one ray aimed at the source.
        _case("forward_clouds", "forward", "clouds", 297000, leaf=12, directed=True),
        # Many small media at once (forward), as in a scan over parameters.
        _case("forest_small", "forest", "mixed", 4096, scenes=48, mix=1),
        # The benchmark's batch (a third of its scenes): J and gradients, job log kept.
        _case("forest_gradient", "forest_gradient", "mixed", 2 ** 17, scenes=20, mix=2),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("forward", "step", "gradient", "forest", "forest_gradient"))
    c = _case("", kind, "mixed", 0)
    del c["name"]
    if kind.startswith("forest"):
        c["scenes"] = _log_uniform(rng, 2, 48 if kind == "forest" else 20)
        c["n"] = _log_uniform(rng, 2000, 2 ** 15)
        c["mix"] = rng.randrange(3, 1 << 20)
        return c
    c["medium"] = rng.choice(("uniform", "lognormal", "lognormal", "isothermal", "clouds"))
    c["bands"] = rng.choice((1, 2, 2, 3, 4, 10))
    c["nside"] = rng.choice((1, 2, 2, 4))
    top = 2 ** 18 if c["bands"] <= 4 else 2 ** 16
    if c["medium"] == "lognormal" and c["nside"] == 4:
        top = 2 ** 13
    if c["medium"] == "isothermal":
        c["bands"] = 2
        top = 2 ** 20
        c["active"] = rng.choice((0.01, 0.1, 0.3))
    if c["medium"] == "clouds":
        c["bands"] = 1
        c["directed"] = rng.random() < 0.5
        c["absorption_avg"] = rng.random() < 0.5
    if kind == "gradient":
        top //= 2
        c["keep_depths"] = rng.random() < 0.5
    elif c["medium"] in ("uniform", "lognormal"):
        c["active"] = rng.choice((1.0, 1.0, 0.1, 0.01))
    c["n"] = _log_uniform(rng, 1000, top)
    c["leaf"] = rng.choice((8, 8, 12))
    c["theta"] = rng.choice((0.75, 0.75, 0.6, 0.9))
    return c


# ----------------------------------------------------------------- the inputs
def _one_scene(medium, n, bands, nside, leaf, theta, seed, **kw):
    kappa = tuple(BANDS[:bands]) if bands <= 4 else tuple(np.geomspace(1.0, 1000.0, bands))
    if medium == "uniform":
        return scenes.uniform_scene(n=n, seed=seed, n_src=max(1, n // 64), bands=kappa,
                                    nside=nside, leaf_size=leaf, theta=theta, **kw)
    if medium == "lognormal":
        grid = 16 if n < 2 ** 13 else 32 if n < 2 ** 15 else 64
        return scenes.lognormal_scene(n=n, seed=seed, grid=grid, bands=kappa, nside=nside,
                                      leaf_size=leaf, theta=theta, **kw)
    if medium == "isothermal":
        return scenes.isothermal_scene(n=n, seed=seed, bands=kappa, nside=nside,
                                       leaf_size=leaf, theta=theta, **kw)
    more = 1.0
    while True:   # the lattice's count varies with its jitter: thin a fuller one to n
        more *= 1.02
        coarser = (290000.0 / (n * more)) ** (1.0 / 3.0)
        sc = scenes.source_features_scene("clouds", seed=seed, nside=nside, theta=theta,
                                          leaf_size=leaf, outer=0.0625 * coarser,
                                          inner=0.0209 * coarser)
        if sc.n >= n:
            break
    keep = np.sort(np.random.default_rng(seed).choice(sc.n - 1, n - 1, replace=False))
    keep = np.append(keep, sc.n - 1)    # the source is the last element
    sc = sc.with_(active=scenes.shell_active(sc, 0.0625 * coarser))
    cut = {k: np.ascontiguousarray(getattr(sc, k)[..., keep])
           for k in ("x", "y", "z", "m", "rho", "kappa", "lum", "active")}
    return sc.with_(**cut)


def _scenes(case, seed):
    """The scenes of a case with their active flags, from the seed alone."""
    if case["kind"].startswith("forest"):
        mix = np.random.default_rng(case["mix"])
        out = []
        for s in range(case["scenes"]):
            n = int(round(math.exp(mix.uniform(math.log(case["n"] / 32), math.log(case["n"])))))
            out.append(_one_scene("uniform" if mix.random() < 0.5 else "lognormal", max(n, 64),
                                  int(mix.integers(1, 5)), int(mix.choice([1, 2, 4])),
                                  case["leaf"], case["theta"], seed * 64 + s))
        return [_uneven(s, seed + i) for i, s in enumerate(out)]
    sc = _one_scene(case["medium"], case["n"], case["bands"], case["nside"], case["leaf"],
                    case["theta"], seed)
    if case["medium"] == "clouds":
        if case["directed"]:
            sc = sc.with_(directed=tuple(float(v) for v in sc.meta["centre"]))
    elif case["active"] < 1.0:
        sc = sc.with_(active=scenes.active_subset(sc, case["active"], seed + 1))
    return [_uneven(sc.with_(absorption_avg=case["absorption_avg"]), seed)]


def _uneven(sc, seed):
    """Masses jittered by up to 1%: no two elements of one size, as in a simulation
    (the derivative of a maximum over equal sizes has a kink)."""
    u = np.random.default_rng(seed + 13).uniform(-0.01, 0.01, sc.n)
    return sc.with_(m=(sc.m * (1.0 + u)).astype(np.float32))


def _adjoint(scene_list, seed):
    """dE/dJ of a fit, per scene [B, n]."""
    rng = np.random.default_rng(seed + 7)
    return [rng.normal(size=(s.n_bands, s.n)) for s in scene_list]


def prepare(case, seed):
    scs = _scenes(case, seed)
    st = {"kind": case["kind"]}
    if case["kind"].startswith("forest"):
        F = api.Forest(scs)
        st["F"] = F
        if case["kind"] == "forest_gradient":
            F.compute_J()
            F.set_job_log(2 * F.counters()["pp_log_entries"] + (1 << 28))
            st["gJ"] = torch.as_tensor(np.concatenate([g.ravel() for g in _adjoint(scs, seed)]),
                                       device="cuda")
        return st
    sc = scs[0]
    t = lambda a: torch.as_tensor(np.ascontiguousarray(a, np.float32), device="cuda")  # noqa: E731
    st["x"] = [t(a) for a in (sc.x, sc.y, sc.z, sc.m, sc.rho, sc.kappa, sc.lum)]
    st["active"] = torch.as_tensor(sc.active, device="cuda")
    st["bg"] = t(sc.bg) if sc.background else None
    flags = api.scene_flags(sc) | (api.KEEP_DEPTHS if case["keep_depths"] else 0)
    st["opts"] = dict(nside=sc.nside, leaf_size=sc.leaf_size, theta=sc.theta, flags=flags,
                      rpp_min=sc.rpp_min, box=sc.box, target=sc.directed)
    if case["kind"] == "gradient":
        for a in st["x"][4:]:
            a.requires_grad_(True)
        st["gJ"] = torch.as_tensor(_adjoint(scs, seed)[0], device="cuda")
    elif case["kind"] == "forward":
        st["tree"] = api.Tree(*st["x"], **st["opts"])
    else:
        st["scratch"] = None   # handed from one step's tree to the next
    return st


def run(st):
    kind = st["kind"]
    if kind == "forward":
        return st["tree"].compute_J(st["active"], st["bg"])
    if kind == "step":
        T = api.Tree(*st["x"], scratch=st["scratch"], **st["opts"])
        J = T.compute_J(st["active"], st["bg"])
        st["scratch"] = T.scratch
        T.close()
        return J
    if kind == "gradient":
        J = api.TrevrJ.apply(*st["x"], st["active"], st["bg"], st["opts"])
        rho, kappa, lum = st["x"][4:]
        return (J.detach(),) + torch.autograd.grad(J, (lum, kappa, rho), st["gJ"])
    J = st["F"].compute_J()
    if kind == "forest":
        return J
    return (J,) + tuple(st["F"].compute_J_backward(st["gJ"]))


# ------------------------------------------------------------------- the work
def _per_receiver(medium, n, nside):
    """Far sources per receiver, cell chords per bucket, particle-particle elements and
    hits of the particle-particle source paths per receiver: fits to the counters of the
    generators' media."""
    k = 12 * nside * nside
    chords = 0.8 * k * math.log2(1 + n / 150)
    fine = max(1.0, nside / 2) ** 2
    if medium == "uniform":
        return 37 * math.log2(1 + n / 3000), chords, 45.0 * fine, 4.0 * fine
    if medium == "lognormal":
        src = 45 * math.log2(1 + n / 1200)
        if nside >= 4:
            near = n / (1 + n / 20000)
            return src / 2, chords / 8, near, 3.5 * near
        return src, chords, (52.0, 185.0)[nside - 1], (38.0, 240.0)[nside - 1]
    if medium == "isothermal":
        return 36 * math.log2(1 + n / 7), chords, 50.0 * fine, 300.0 * fine ** 1.4
    return 1.0, chords, 55.0 * fine, 0.0


def work(case):
    """Bytes: every input read and every output written once.  Operations: the
    method's arithmetic for the far sources, cell chords, particle-particle columns
    (an element lies on some 15% of the rays) and paths of the receivers (adds, multiplies, divides, roots, exponentials)."""
    back = "gradient" in case["kind"]
    if case["kind"].startswith("forest"):
        mix = np.random.default_rng(case["mix"])
        parts = []
        for _ in range(case["scenes"]):
            n = int(round(math.exp(mix.uniform(math.log(case["n"] / 32), math.log(case["n"])))))
            med = "uniform" if mix.random() < 0.5 else "lognormal"
            parts.append((med, max(n, 64), int(mix.integers(1, 5)), int(mix.choice([1, 2, 4])),
                          1.0))
    else:
        act = 0.07 if case["medium"] == "clouds" else case["active"]
        parts = [(case["medium"], case["n"], case["bands"], case["nside"], act)]
    total = {"bytes": 0.0, "flops": 0.0}
    for medium, n, B, nside, act in parts:
        src, chords, near, hits = _per_receiver(medium, n, nside)
        rec, k = act * n, 12 * nside * nside
        buckets = min(n / (0.7 * case["leaf"]), rec)
        total["bytes"] += n * (20 + 8 * B + 1 + 8 * B * act)
        flops = rec * (src * (37 + 6 * B) + 0.15 * k * near * 24.0 + hits * (29 + 2 * B))
        flops += buckets * chords * (20 + 2 * B)
        if back:
            per = 8 if case["kind"] == "forest_gradient" else 4
            total["bytes"] += n * (20 + 8 * B + 8 * B + per * (2 * B + 1))
            flops += rec * (src * (61 + 19 * B) + 0.15 * k * near * 32.0 + hits * (35 + 5 * B))
            flops += buckets * chords * (40 + 8 * B)
        total["flops"] += flops
    return total


# ------------------------------------------- the method in 64-bit torch operations
MOST_PATHS = 6e10   # particle-particle source paths that fit some seconds


def _ragged(count):
    """Row and position within the row of every entry of rows of `count` entries."""
    row = torch.repeat_interleave(torch.arange(count.numel(), device=count.device), count)
    start = torch.cumsum(count, 0) - count
    return row, torch.arange(row.numel(), device=count.device) - start[row]


def _healpix(nside):
    """Pixel centres in ring order."""
    out = []
    for i in range(1, 4 * nside):
        j = min(i, 4 * nside - i)
        if j < nside:
            z, cnt, half = 1.0 - j * j / (3.0 * nside * nside), 4 * j, True
            z = z if i < nside else -z
        else:
            z, cnt, half = 4 / 3 - 2.0 * i / (3.0 * nside), 4 * nside, (i - nside) % 2 == 0
        for q in range(cnt):
            phi = (q + (0.5 if half else 0.0)) * 2.0 * math.pi / cnt
            st = math.sqrt((1.0 - z) * (1.0 + z))
            out.append((st * math.cos(phi), st * math.sin(phi), z))
    return out


def _pixel(N, v):
    """Ring-order pixel that holds each direction."""
    z = v[:, 2] / v.square().sum(1).sqrt()
    za = z.abs()
    phi = torch.atan2(v[:, 1], v[:, 0])
    tt = torch.where(phi < 0, phi + 2 * math.pi, phi) / (0.5 * math.pi)
    up, dn = N * (0.5 + tt) - N * z * 0.75, N * (0.5 + tt) + N * z * 0.75
    jp, jm = up.floor().long(), dn.floor().long()
    ring = N + 1 + jp - jm
    ip = torch.div(jp + jm - N + 1 - (ring & 1) + 1, 2, rounding_mode="floor") % (4 * N)
    belt = 2 * N * (N - 1) + (ring - 1) * 4 * N + ip
    tp, root = tt - tt.floor(), N * (3.0 * (1.0 - za)).clamp(min=0).sqrt()
    cap = (tp * root).floor().long() + ((1.0 - tp) * root).floor().long() + 1
    ic = (tt * cap).floor().long() % (4 * cap)
    polar = torch.where(z > 0, 2 * cap * (cap - 1) + ic, 12 * N * N - 2 * cap * (cap + 1) + ic)
    return torch.where(za <= 2.0 / 3.0, belt, polar)


def _intensity(r, h):
    """Intensity of a unit source at distance r averaged over a sphere of the
    element's size (1/(4 pi r^2) far away, 1/h^2 at r = 0)."""
    x = r / (math.sqrt(3.0 / (4.0 * math.pi)) * h)
    one = torch.ones_like(x)
    a = torch.where((x > 0) & (x < 1), x, 0.5 * one)
    b = torch.where((x > 1) & (x < 10), x, 2.0 * one)
    y = 1.0 / torch.where(x >= 10, x, 10.0 * one).square()
    far = sum(2.0 * y ** k / (4.0 * k * k - 1.0) for k in range(1, 13))
    f = torch.where(x < 1, 1.0 + (1.0 - a * a) * torch.atanh(a) / a,
                    torch.where(x < 10, 1.0 - (b * b - 1.0) * torch.atanh(1.0 / b) / b, far))
    f = torch.where(x == 0, 2.0 * one, torch.where(x == 1, one, f))
    return f / (2.0 * h * h)


def _dist2_box(lo, hi, c):
    return (torch.clamp(lo - c, min=0) + torch.clamp(c - hi, min=0)).square().sum(1)


class _Exact:
    def __init__(self, sc, grad):
        dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        t = lambda a: torch.as_tensor(np.asarray(a), device=dev).double()  # noqa: E731
        self.sc, self.dev, self.n, self.B = sc, dev, sc.n, sc.n_bands
        pos = torch.stack([t(sc.x), t(sc.y), t(sc.z)], 1)
        lo, side = torch.tensor(sc.box[:3], dtype=torch.float64, device=dev), float(sc.box[3])
        q = ((pos - lo) * (2.0 ** 21 / side)).floor().clamp(0, 2097151).long()
        key = torch.zeros(sc.n, dtype=torch.long, device=dev)
        for b in range(20, -1, -1):
            for a in range(3):
                key = (key << 1) | ((q[:, a] >> b) & 1)
        self.key, self.perm = torch.sort(key, stable=True)
        self.pos, self.q, self.lo, self.side = pos[self.perm], q[self.perm], lo, side
        self.m = t(sc.m)[self.perm]
        self.rho, self.kappa, self.lum = t(sc.rho), t(sc.kappa), t(sc.lum)
        for a in (self.rho, self.kappa, self.lum) if grad else ():
            a.requires_grad_(True)
        self.act = torch.as_tensor(sc.active, device=dev)[self.perm] > 0
        self.dirs = torch.tensor(_healpix(sc.nside), dtype=torch.float64, device=dev)
        self.K = self.dirs.shape[0]
        # exact powers of two: empty cells meet the opening criterion with equality
        self.sides = side * torch.tensor([2.0 ** -k for k in range(24)], dtype=torch.float64,
                                         device=dev)
        _, self.cls = torch.unique((self.dirs.abs() * 1e9).round(), dim=0, return_inverse=True)
        self.rep = torch.stack([(self.cls == c).nonzero()[0, 0] for c in range(int(self.cls.max()) + 1)])
        self._topology()
        self._moments()

    def _topology(self):
        dev, leaf = self.dev, self.sc.leaf_size
        first = torch.zeros(1, dtype=torch.long, device=dev)
        count = torch.full((1,), self.n, dtype=torch.long, device=dev)
        own = torch.zeros(1, dtype=torch.long, device=dev)
        levels, base = [], 0
        while first.numel():
            k0, k1 = self.key[first], self.key[first + count - 1]
            inner = (count > leaf) & (k0 != k1)
            x, top = k0 ^ k1, torch.zeros_like(k0)       # highest differing bit
            for w in (32, 16, 8, 4, 2, 1):
                big = (x >> w) > 0
                top, x = top + big * w, torch.where(big, x >> w, x)
            split = torch.where(inner, 62 - top, -1)
            pre = (k1 >> top) << top
            mid = torch.searchsorted(self.key, pre)
            base += first.numel()
            i = inner.nonzero()[:, 0]
            child = torch.full_like(first, -1)
            child[i] = base + 2 * torch.arange(i.numel(), device=dev)
            levels.append((first, count, own, split, child))
            f, c, s, m = first[i], count[i], split[i], mid[i]
            first = torch.stack([f, m], 1).reshape(-1)
            count = torch.stack([m - f, f + c - m], 1).reshape(-1)
            own = torch.stack([s + 1, s + 1], 1).reshape(-1)
        self.levels = [l[0].numel() for l in levels]
        self.first, self.count, self.own, self.split, self.child = (
            torch.cat([l[j] for l in levels]) for j in range(5))
        self.leaf = self.split < 0
        nb = torch.div(self.own[:, None] + 2 - torch.arange(3, device=dev), 3, rounding_mode="floor")
        w = self.sides[nb]
        k = self.q[self.first] >> (21 - nb)
        self.blo, self.bhi = self.lo + k * w, self.lo + (k + 1) * w

    def _combine(self, length, a1, a2):
        """Transmission average of two halves of the prefix boxes of the given
        lengths, per direction class; a1, a2 [nodes, classes, B]."""
        ax = length % 3
        order = torch.stack([ax, (ax + 1) % 3, (ax + 2) % 3], 1)
        nb = torch.div(length[:, None] + 2 - order, 3, rounding_mode="floor")
        s = self.sides[nb]
        n = self.dirs[self.rep].abs()[None].expand(length.numel(), -1, -1)
        n = torch.gather(n, 2, order[:, None, :].expand(-1, n.shape[1], -1))
        sa, sb, sc = s[:, None, 0], s[:, None, 1], s[:, None, 2]
        tb, tc = n[..., 1] / n[..., 0], n[..., 2] / n[..., 0]
        u = torch.minimum(0.5 * sa, torch.minimum(sb / tb, sc / tc))
        v12 = 2.0 * (sb * sc * u - (sb * tc + sc * tb) * u * u / 2 + tb * tc * u ** 3 / 3)
        vol = sa * sb * sc
        v12 = torch.where(n[..., 0] > 0, v12, torch.zeros_like(v12))
        w1, w12 = ((vol - v12) / 2).clamp(min=0) / vol, (v12 / vol).clamp(max=1)
        d = (s[:, None, :] / n).amin(2)[..., None]
        w1, w12 = w1.log()[..., None], w12.log()[..., None]
        terms = torch.stack([w1 - d * a1, w1 - d * a2, w12 - d * (a1 + a2) / 2])
        return -torch.logsumexp(terms, 0) / d

    def _moments(self):
        p, B = self.perm, self.B
        self.rho_s, self.kap, self.L = self.rho[p], self.kappa[:, p].T, self.lum[:, p].T
        self.h = (self.m / self.rho_s) ** (1.0 / 3.0)
        self.Lbol = self.L.sum(1)
        leaf_of = torch.zeros(self.n, dtype=torch.long, device=self.dev)
        li = self.leaf.nonzero()[:, 0]
        row, at = _ragged(self.count[li])
        leaf_of[self.first[li][row] + at] = li[row]
        self.leaf_of, nn = leaf_of, self.first.numel()
        add = lambda v: torch.zeros((nn,) + v.shape[1:], dtype=v.dtype, device=self.dev).index_add(0, leaf_of, v)  # noqa: E731
        Lb, SL = add(self.L), add(self.Lbol[:, None] * self.pos)
        vol = add(self.m / self.rho_s)
        bucket = add(self.kap * self.m[:, None]) / torch.where(vol > 0, vol, 1.0)[:, None]
        C = self.rep.numel()
        end, below = nn, None
        got = []
        for size in reversed(self.levels):
            sl = slice(end - size, end)
            lb, s1, al = Lb[sl], SL[sl], bucket[sl][:, None, :].expand(-1, C, -1)
            inner = (~self.leaf[sl]).nonzero()[:, 0]
            if inner.numel():
                c0 = self.child[sl][inner] - end
                lb = lb.index_put((inner,), below[0][c0] + below[0][c0 + 1])
                s1 = s1.index_put((inner,), below[1][c0] + below[1][c0 + 1])
                a1, a2 = below[2][c0], below[2][c0 + 1]
                split, own = self.split[sl][inner], self.own[sl][inner]
                empty = split - own               # vacuum boxes above the split one
                if self.sc.absorption_avg:
                    A = (a1 + a2) / 2 * (self.sides[empty] / self.side)[:, None, None]
                else:
                    A = self._combine(split, a1, a2)
                    for e in range(1, int(empty.max()) + 1):
                        i = (empty >= e).nonzero()[:, 0]
                        A = A.index_put((i,), self._combine(split[i] - e, A[i], torch.zeros_like(A[i])))
                al = al.index_put((inner,), A)
            below, end = (lb, s1, al), end - size
            got.append(below)
        self.Lb, SL, self.alpha = (torch.cat([g[j] for g in reversed(got)]) for j in range(3))
        self.Lnode = self.Lb.sum(1)
        dark = self.Lnode <= 0
        self.cen = torch.where(dark[:, None], 0.5 * (self.blo + self.bhi),
                               SL / torch.where(dark, 1.0, self.Lnode)[:, None])
        zero = torch.zeros(self.n + 1, dtype=torch.float64, device=self.dev)
        zero[1:] = torch.cumsum((self.kap.detach() * self.m[:, None]).sum(1), 0)
        self.absorbs = zero[self.first + self.count] - zero[self.first] > 0

    def _near(self, c, r2):
        """(bucket, slot) pairs with |x - c| < r, by bucket and slot."""
        b = torch.arange(c.shape[0], device=self.dev)
        nd = torch.zeros_like(b)
        got_b, got_l = [], []
        while b.numel():
            keep = _dist2_box(self.blo[nd], self.bhi[nd], c[b]) <= r2[b] * (1 + 1e-9)
            b, nd = b[keep], nd[keep]
            lf = self.leaf[nd]
            got_b.append(b[lf])
            got_l.append(nd[lf])
            b, nd = b[~lf].repeat_interleave(2), self.child[nd[~lf]].repeat_interleave(2)
            nd[1::2] += 1
        b, nd = torch.cat(got_b), torch.cat(got_l)
        row, at = _ragged(self.count[nd])
        b, s = b[row], self.first[nd][row] + at
        keep = (self.pos[s] - c[b]).square().sum(1) < r2[b]
        code = torch.sort(b[keep] * self.n + s[keep])[0]
        return torch.div(code, self.n, rounding_mode="floor"), code % self.n

    def _sphere(self, leaf, c):
        """Particle-particle radius of the buckets (and which element sets it), and
        the pairs inside."""
        nb, h = leaf.numel(), self.h.detach()
        r = torch.full((nb,), float(self.sc.rpp_min), dtype=torch.float64, device=self.dev)
        who = torch.full((nb,), -1, dtype=torch.long, device=self.dev)
        off, div = torch.zeros_like(r), torch.ones_like(r)
        if not self.sc.near_field:
            none = torch.zeros(0, dtype=torch.long, device=self.dev)
            return torch.zeros_like(r), who, off, div, none, none

        def grow(b, s, value, o, d):
            best = torch.full_like(r, -1.0).scatter_reduce(0, b, value, "amax")
            up = best > r
            top = (value == best[b]) & up[b]
            at = torch.full_like(who, self.n).scatter_reduce(0, b[top], s[top], "amin")
            pick = top & (s == at[b])
            r[b[pick]], who[b[pick]] = value[pick], s[pick]
            off[b[pick]], div[b[pick]] = o[pick], d
            return up

        row, k = _ragged(self.count[leaf])
        s = self.first[leaf][row] + k
        dist = (self.pos[s] - c[row]).square().sum(1).sqrt()
        grow(row, s, dist + h[s], dist, 1.0)
        w = 2.0 * math.tan(math.acos(1.0 - 2.0 / self.K))
        while True:
            b, s = self._near(c, r * r)
            if not bool(grow(b, s, h[s] / w, torch.zeros_like(h[s]), w).any()):
                return r, who, off, div, b, s

    def _walk(self, c, r2):
        b = torch.arange(c.shape[0], device=self.dev)
        nd = torch.zeros_like(b)
        cen, got = self.cen.detach(), []
        while b.numel():
            lo, hi, cb = self.blo[nd], self.bhi[nd], c[b]
            keep = torch.maximum((lo - cb).square(), (hi - cb).square()).sum(1) >= r2[b]
            b, nd, lo, hi, cb = b[keep], nd[keep], lo[keep], hi[keep], cb[keep]
            d2 = _dist2_box(lo, hi, cb)
            far = torch.maximum((cen[nd] - lo).square(), (hi - cen[nd]).square()).sum(1)
            op = (d2 < r2[b]) | (far > self.sc.theta ** 2 * d2)
            down = op & ~self.leaf[nd]
            got.append((b[~down], nd[~down], op[~down]))
            b, nd = b[down].repeat_interleave(2), self.child[nd[down]].repeat_interleave(2)
            nd[1::2] += 1
        return (torch.cat([g[j] for g in got]) for j in range(3))

    def _chunk(self, leaf, tab, bg):
        """J of the active elements of some buckets: (slots, J [receivers, B])."""
        rho, kap, L, h, Lb, cen, alpha = tab
        K, B, dev, N = self.K, self.B, self.dev, self.sc.nside
        c = 0.5 * (self.blo[leaf] + self.bhi[leaf])
        nb = leaf.numel()
        rv, who, off, div, nb_b, nb_s = self._sphere(leaf, c)
        r2 = rv * rv
        r = torch.where(who >= 0, off + h[who.clamp(min=0)] / div, rv)
        dirs = self.dirs[None].expand(nb, -1, -1)
        if self.sc.directed is not None:
            v = torch.tensor(self.sc.directed, dtype=torch.float64, device=dev) - c
            dirs = dirs.clone()
            dirs[torch.arange(nb, device=dev), _pixel(N, v)] = v / v.square().sum(1).sqrt()[:, None]
        b, nd, op = self._walk(c, r2)
        # chords of the absorbing cells beyond the sphere
        hit_b, hit_k, hit_n, hit_t0, hit_t1 = [], [], [], [], []
        ab, an = b[self.absorbs[nd]], nd[self.absorbs[nd]]
        for at in range(0, ab.numel(), 1 + 20000000 // K):
            eb, en = ab[at:at + 1 + 20000000 // K], an[at:at + 1 + 20000000 // K]
            tin = torch.full((eb.numel(), K), -math.inf, dtype=torch.float64, device=dev)
            tout, ok = -tin, torch.ones_like(tin, dtype=torch.bool)
            for a in range(3):
                nv = dirs[eb, :, a]
                u, v = (self.blo[en, a] - c[eb, a])[:, None], (self.bhi[en, a] - c[eb, a])[:, None]
                t1, t2, flat = u * (1.0 / nv), v * (1.0 / nv), nv == 0
                tin = torch.where(flat, tin, torch.maximum(tin, torch.minimum(t1, t2)))
                tout = torch.where(flat, tout, torch.minimum(tout, torch.maximum(t1, t2)))
                ok &= ~flat | ((u <= 0) & (v >= 0))
            e, k = (ok & (tin < tout) & (tout > rv[eb][:, None])).nonzero(as_tuple=True)
            hit_b.append(eb[e]), hit_k.append(k), hit_n.append(en[e])
            hit_t0.append(tin[e, k]), hit_t1.append(tout[e, k])
        empty = torch.zeros(0, dtype=torch.long, device=dev)
        hb, hk, hn = (torch.cat(v) if v else empty for v in (hit_b, hit_k, hit_n))
        t0, t1 = (torch.cat(v) if v else empty.double() for v in (hit_t0, hit_t1))
        code, order = torch.sort(hb * K + hk, stable=True)
        hb, hk, hn, t0, t1 = hb[order], hk[order], hn[order], t0[order], t1[order]
        t0 = torch.where(t0 < rv[hb], r[hb], t0)
        # far sources: whole cells, and the elements of opened buckets
        cell = ~op & (self.Lnode[nd] > 0)
        row, at = _ragged(self.count[nd[op]])
        eb, es = b[op][row], self.first[nd[op]][row] + at
        keep = (self.Lbol[es] > 0) & ((self.pos[es] - c[eb]).square().sum(1) >= r2[eb])
        eb, es = eb[keep], es[keep]
        sb = torch.cat([b[cell], eb])
        sp = torch.cat([cen[nd[cell]], self.pos[es]])
        sL = torch.cat([Lb[nd[cell]], L[es]])
        v = sp - c[sb]
        at_c = (v.detach() == 0).all(1)
        sk = torch.where(at_c, 0, _pixel(N, torch.where(at_c[:, None], torch.ones_like(v), v.detach())))
        ss = torch.where(at_c, torch.zeros_like(v[:, 0]), (v * dirs[sb, sk]).sum(1))
        order = torch.argsort(sb, stable=True)
        sb, sk, ss, sp, sL = sb[order], sk[order], ss[order], sp[order], sL[order]
        nsrc = sb.numel()
        if bg is not None:   # the way out of the root cube, as one more end per ray
            wall = torch.where(dirs > 0, self.lo + self.side - c[:, None], self.lo - c[:, None]) / dirs
            out = torch.where(dirs == 0, math.inf, wall).amin(2)
            sb = torch.cat([sb, torch.arange(nb, device=dev).repeat_interleave(K)])
            sk = torch.cat([sk, torch.arange(K, device=dev).repeat(nb)])
            ss = torch.cat([ss, out.reshape(-1)])
        ray = sb * K + sk
        begin = torch.searchsorted(code, ray)
        cnt = torch.searchsorted(code, ray, right=True) - begin
        tau = torch.zeros((ss.numel(), B), dtype=torch.float64, device=dev)
        edge = torch.cumsum(cnt, 0)
        at = 0
        while at < cnt.numel():
            done = int(edge[at - 1]) if at else 0
            to = max(at + 1, int(torch.searchsorted(edge, done + 60000000)))
            row, pos = _ragged(cnt[at:to])
            row = row + at
            g = begin[row] + pos
            end = torch.where(ss[row] < t1[g], ss[row], t1[g])
            use = (end > t0[g]).nonzero()[:, 0]
            row, g = row[use], g[use]
            tau = tau.index_add(0, row, alpha[hn[g], self.cls[hk[g]]] * (end[use] - t0[g])[:, None])
            at = to
        # receivers
        row, at = _ragged(self.count[leaf])
        rs = self.first[leaf][row] + at
        row, rs = row[self.act[rs]], rs[self.act[rs]]
        nr = rs.numel()
        J = torch.zeros((nr, B), dtype=torch.float64, device=dev)
        near0 = torch.searchsorted(nb_b, row)
        nearc = torch.searchsorted(nb_b, row, right=True) - near0
        # columns along the rays
        col = torch.zeros((nr * K, B), dtype=torch.float64, device=dev)
        rr, at = _ragged(nearc)
        el = nb_s[near0[rr] + at]
        for part in torch.split(torch.arange(rr.numel(), device=dev), 1 + 30000000 // K):
            i, l = rr[part], el[part]
            d = (self.pos[l] - self.pos[rs[i]])[:, None]
            n = dirs[row[i]]
            b2 = torch.linalg.cross(d.expand_as(n), n, dim=2).square().sum(2)
            ok = ((d * n).sum(2) > 0) & (b2.sqrt() < h.detach()[l][:, None]) & (l != rs[i])[:, None]
            e, k = ok.nonzero(as_tuple=True)
            le, hl = l[e], h[l[e]]
            sig = 3.0 * self.m[le] / (math.pi * hl * hl) * (1.0 - b2[e, k].sqrt() / hl)
            col = col.index_add(0, i[e] * K + k, kap[le] * sig[:, None])
        # far sources at each receiver
        s0 = torch.searchsorted(sb[:nsrc], row)
        sc = torch.searchsorted(sb[:nsrc], row, right=True) - s0
        edge, at = torch.cumsum(sc, 0), 0
        while at < nr:
            done = int(edge[at - 1]) if at else 0
            to = max(at + 1, int(torch.searchsorted(edge, done + 60000000)))
            i, pos = _ragged(sc[at:to])
            i = i + at
            e = s0[i] + pos
            dist = (sp[e] - self.pos[rs[i]]).square().sum(1).sqrt()
            dark = tau[e] <= 0
            ex = torch.where(dark, torch.zeros_like(tau[e]),
                             tau[e] * (dist / torch.where(ss[e] != 0, ss[e], torch.ones_like(dist)))[:, None])
            J = J.index_add(0, i, sL[e] * (_intensity(dist, h[rs[i]])[:, None]
                                           * torch.exp(-col[i * K + sk[e]] - ex)))
            at = to
        # near sources
        lum = (self.Lbol[nb_s] > 0).nonzero()[:, 0]
        l0 = torch.searchsorted(nb_b[lum], row)
        lc = torch.searchsorted(nb_b[lum], row, right=True) - l0
        i, pos = _ragged(lc)
        j = nb_s[lum[l0[i] + pos]]
        path = torch.zeros((i.numel(), B), dtype=torch.float64, device=dev)
        e_ = self.pos[j] - self.pos[rs[i]]
        r2ij = e_.square().sum(1)
        edge, at = torch.cumsum(nearc[i], 0), 0
        while at < i.numel():
            done = int(edge[at - 1]) if at else 0
            to = max(at + 1, int(torch.searchsorted(edge, done + 60000000)))
            p, pos = _ragged(nearc[i[at:to]])
            p = p + at
            l = nb_s[near0[i[p]] + pos]
            ok = (l != rs[i[p]]) & (l != j[p]) & ((self.pos[l] - self.pos[j[p]]).square().sum(1) < r2ij[p])
            p, l = p[ok], l[ok]
            w = self.pos[l] - self.pos[rs[i[p]]]
            u = ((w * e_[p]).sum(1) / r2ij[p]).clamp(0, 1)
            bb = (w - u[:, None] * e_[p]).square().sum(1).sqrt()
            ok = bb < h.detach()[l]
            p, l, bb = p[ok], l[ok], bb[ok]
            sig = 3.0 * self.m[l] / (math.pi * h[l] * h[l]) * (1.0 - bb / h[l])
            path = path.index_add(0, p, kap[l] * sig[:, None])
            at = to
        J = J.index_add(0, i, L[j] * (_intensity(r2ij.sqrt(), h[rs[i]])[:, None] * torch.exp(-path)))
        if bg is not None:
            J = J + (4.0 * math.pi / K) * bg * torch.exp(
                -col.reshape(nr, K, B) - tau[nsrc:].reshape(nb, K, B)[row]).sum(1)
        if self.sc.thick_corr:
            th = kap[rs] * (rho[rs] * h[rs])[:, None]
            some = th.detach() != 0
            safe = torch.where(some, th, torch.ones_like(th))
            J = J * torch.where(some, -torch.expm1(-safe) / safe, torch.ones_like(th))
        return rs, J

    def _paths(self, leaves):
        """Particle-particle source paths, from a sample of the buckets."""
        some = leaves[:: max(1, leaves.numel() // 256)]
        b, s = self._sphere(some, 0.5 * (self.blo[some] + self.bhi[some]))[4:]
        near = torch.bincount(b, minlength=some.numel()).double()
        lum = torch.bincount(b[self.Lbol[s] > 0], minlength=some.numel()).double()
        return float((near * lum).mean()) * float(self.act.sum())

    def evaluate(self, gJ=None):
        """J [B, n], and with gJ the gradients (lum, kappa, rho); None if it would
        take long."""
        any_act = torch.zeros(self.first.numel(), device=self.dev).index_add(
            0, self.leaf_of, self.act.float()) > 0
        leaves = (self.leaf & any_act).nonzero()[:, 0]
        paths = self._paths(leaves)
        if paths * (4 if gJ is not None else 1) > MOST_PATHS:
            return None
        bg = torch.as_tensor(self.sc.bg, device=self.dev).double() if self.sc.background else None
        whole = (self.rho_s, self.kap, self.L, self.h, self.Lb, self.cen, self.alpha)
        tab = whole if gJ is None else tuple(a.detach().requires_grad_(True) for a in whole)
        J = torch.zeros((self.B, self.n), dtype=torch.float64, device=self.dev)
        step = 2048 if gJ is None else 1024
        for part in torch.split(leaves, step):
            with torch.set_grad_enabled(gJ is not None):
                s, Jr = self._chunk(part, tab, bg)
                i = self.perm[s]
                if gJ is not None:
                    (Jr * gJ[:, i].T).sum().backward()
            J[:, i] = Jr.detach().T
        if gJ is None:
            return J
        torch.autograd.backward([w for w, t in zip(whole, tab) if w.requires_grad and t.grad is not None],
                                [t.grad for w, t in zip(whole, tab) if w.requires_grad and t.grad is not None])
        return J, self.lum.grad, self.kappa.grad, self.rho.grad


def exact(case, seed):
    scs = _scenes(case, seed)
    back = "gradient" in case["kind"]
    gJ = _adjoint(scs, seed) if back else None
    out = []
    for s, sc in enumerate(scs):
        E = _Exact(sc, back)
        g = None if gJ is None else torch.as_tensor(gJ[s], device=E.dev)
        v = E.evaluate(g)
        if v is None:
            return None
        out.append(v)
    if not case["kind"].startswith("forest"):
        return out[0]
    if not back:
        return torch.cat([v.reshape(-1) for v in out])
    return tuple(torch.cat([v[j].reshape(-1) for v in out]) for j in range(4))
