"""Workloads of the library, from its smallest calls to its largest, for timing
and for checking results: dense entries, per-frequency H-matrices, the 3D-ACA
operator, its products, the FMM-based product, the batched solve and gCQ
stepping, each through the calls a program makes.

Meshes are ellipsoids (geodesic spheres of 20 f^2 triangles, stretched) and
finned cylinders shaped like a machine housing; their semi-axes and
orientation, the time step behind the frequencies and the vectors come from the
seed.
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_2505_00715_amd as g

PREC = {"c128": g.C128, "c64": g.C64, "split": g.C64_SPLIT_BF16}
DEV = "cuda:0"


def listed():
    return [
        # one small dense block, as a first check of an installation asks for
        # it: nothing but latency
        dict(name="entries_small_c128", op="entries", mesh="sphere", size=4, freqs=32, use=3, rows=64, cols=320,
             prec="c128", dlp=False, leaf=16, eta=1.0),
        # sampled rows and columns of a mid-sized housing at many frequencies:
        # the reference values an operator is checked against
        dict(name="entries_housing_c64", op="entries", mesh="housing", size=20480, freqs=256, use=17, rows=2048,
             cols=2048, prec="c64", dlp=False, leaf=64, eta=1.0),
        # per-frequency H-matrices of a sphere built and applied once: the
        # plain method in single precision
        dict(name="hmatrix_sphere5120_c64", op="hmatrix", mesh="sphere", size=16, freqs=64, prec="c64", dlp=False,
             leaf=64, eta=1.0, tol=1e-5),
        # the same in double precision for the double layer, small, with an odd
        # number of frequencies and the ragged leaves of an odd subdivision
        dict(name="hmatrix_dlp_sphere1620_c128", op="hmatrix", mesh="sphere", size=9, freqs=31, prec="c128", dlp=True,
             leaf=32, eta=0.8, tol=1e-6),
        # the 3D-ACA operator of a housing over a whole frequency set, built
        # and applied once: what a program pays for each new geometry
        dict(name="operator_housing3k_c64", op="operator", mesh="housing", size=3000, freqs=256, prec="c64",
             dlp=False, leaf=64, eta=1.0, tol=3e-6),
        # the smallest product: launches and latency
        dict(name="product_sphere320_c64", op="product", mesh="sphere", size=4, freqs=32, prec="c64", dlp=False,
             leaf=64, eta=1.0, tol=1e-5),
        # the benchmark's product: 41 k triangles, 256 frequencies
        dict(name="product_housing40k_split", op="product", mesh="housing", size=40960, freqs=256, prec="split",
             dlp=False, leaf=64, eta=1.0, tol=3e-6),
        # the double-precision product of the plain method's sphere
        dict(name="product_sphere5120_c128", op="product", mesh="sphere", size=16, freqs=64, prec="c128", dlp=False,
             leaf=64, eta=1.0, tol=1e-5),
        # the frequency-weighted sum of eq. product on the 20480-triangle sphere
        dict(name="wsum_sphere20480_c64", op="wsum", mesh="sphere", size=32, freqs=64, prec="c64", dlp=False, leaf=64,
             eta=1.0, tol=1e-5),
        # the FMM-based operator's product
        dict(name="fmm_housing10k_c64", op="fmm", mesh="housing", size=10000, freqs=128, prec="c64", leaf=64, eta=1.0,
             tol=1e-5, order=4),
        # all frequencies of a housing solved to 1e-6
        dict(name="solve_housing3k_split", op="solve", mesh="housing", size=3000, freqs=256, prec="split", leaf=64,
             eta=1.0, tol=3e-6, rtol=1e-6),
        # sixteen implicit Euler steps of the forward convolution, 64 frequencies
        dict(name="stepping_sphere5120_c64", op="stepping", mesh="sphere", size=16, freqs=64, prec="c64", leaf=64,
             eta=1.0, tol=1e-5, stages=1, steps=16),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["entries", "entries", "hmatrix", "hmatrix", "operator", "product", "product", "product", "wsum",
                     "fmm", "solve", "stepping"])
    c = dict(op=op, mesh=rng.choice(["sphere", "housing"]), leaf=rng.choice([20, 32, 48, 64]),
             eta=rng.choice([0.8, 1.0]))
    most = {"entries": 20480, "hmatrix": 4000, "operator": 4000, "product": 10000, "wsum": 20000, "fmm": 10000,
            "solve": 3000, "stepping": 5000}[op]
    n = _log_int(rng, 1000 if c["mesh"] == "housing" else 320, most)
    c["size"] = n if c["mesh"] == "housing" else max(4, round(math.sqrt(n / 20.0)))
    c["freqs"] = _log_int(rng, 5, 64 if op in ("hmatrix", "wsum", "stepping", "solve") else 256)
    if op in ("entries", "hmatrix", "operator", "product", "wsum"):
        c["dlp"] = rng.random() < 0.25
    if op == "entries":
        c["prec"] = rng.choice(["c128", "c64"])
        c["use"] = min(c["freqs"], _log_int(rng, 1, 33))
        c["rows"] = min(n - n // 8, _log_int(rng, 1, 4096))
        room = (6e7 if c["prec"] == "c64" else 2e7) / (c["use"] * c["rows"])
        c["cols"] = max(1, min(n - n // 8, int(room), _log_int(rng, 16, 4096)))
        return c
    c["tol"] = rng.choice([1e-5, 3e-6])
    c["prec"] = rng.choice({"hmatrix": ["c64", "c64", "c128"], "operator": ["c64"],
                            "product": ["c64", "split", "c128"], "wsum": ["c64"], "fmm": ["c64"],
                            "solve": ["split", "c64"], "stepping": ["c64"]}[op])
    if op == "fmm":
        c["order"] = rng.choice([3, 4, 5])
        c["freqs"] = min(c["freqs"], 128)
        c["leaf"] = max(c["leaf"], 48)
    if op == "solve":
        c["rtol"] = rng.choice([1e-4, 1e-6])
    if op == "stepping":
        c["stages"] = rng.choice([1, 1, 2])
        c["freqs"] = max(c["freqs"], 16)
        c["steps"] = rng.randint(4, 16)
    return c


# ---- meshes and frequencies -----------------------------------------------------------

def _merge(soup):
    """(vertices, triangles) of a triangle soup (t, 3, 3): equal corners become one vertex."""
    p = soup.reshape(-1, 3)
    span = np.abs(p).max()
    q = np.rint(p / span * (1 << 19)).astype(np.int64) + (1 << 20)
    _, first, inv = np.unique((q[:, 0] << 42) + (q[:, 1] << 21) + q[:, 2], return_index=True, return_inverse=True)
    return np.ascontiguousarray(p[first]), np.ascontiguousarray(inv.reshape(-1, 3).astype(np.int32))


def _sphere(f):
    """Geodesic unit sphere: every face of an icosahedron cut into f^2 triangles."""
    h = (1.0 + math.sqrt(5.0)) / 2.0
    v = np.array([[-1, h, 0], [1, h, 0], [-1, -h, 0], [1, -h, 0], [0, -1, h], [0, 1, h], [0, -1, -h], [0, 1, -h],
                  [h, 0, -1], [h, 0, 1], [-h, 0, -1], [-h, 0, 1]])
    # the faces: triples of vertices at the edge length 2 from each other
    near = np.abs(np.linalg.norm(v[:, None] - v[None], axis=-1) - 2.0) < 1e-9
    faces = [(a, b, c) for a in range(12) for b in range(a + 1, 12) for c in range(b + 1, 12)
             if near[a, b] and near[b, c] and near[a, c]]
    ij = [(i, j) for i in range(f) for j in range(f - i)]
    bary = []
    for i, j in ij:
        bary.append([(i, j), (i + 1, j), (i, j + 1)])
        if i + j < f - 1:
            bary.append([(i + 1, j), (i + 1, j + 1), (i, j + 1)])
    bary = np.asarray(bary, float) / f                               # (f^2, 3, 2)
    soup = []
    for a, b, c in faces:
        x = v[a] + bary[..., 0:1] * (v[b] - v[a]) + bary[..., 1:2] * (v[c] - v[a])
        soup.append(x / np.linalg.norm(x, axis=-1, keepdims=True))
    return _outward(np.concatenate(soup))


def _outward(soup):
    nrm = np.cross(soup[:, 1] - soup[:, 0], soup[:, 2] - soup[:, 0])
    flip = (nrm * soup.mean(1)).sum(-1) < 0
    soup[flip] = soup[flip][:, [0, 2, 1]]
    return soup


def _quads(a, b, c, d):
    """Two triangles each of the quadrilaterals a b c d (arrays of points)."""
    return np.concatenate([np.stack([a, b, c], 1), np.stack([a, c, d], 1)])


def _zip_rings(outer, inner):
    """Triangles between two closed rings of points of the plane, both sorted by angle."""
    ao, ai = (np.arctan2(r[:, 1], r[:, 0]) % (2 * math.pi) for r in (outer, inner))
    outer, ao, inner, ai = outer[np.argsort(ao)], np.sort(ao), inner[np.argsort(ai)], np.sort(ai)
    no, ni, o, i, tri = len(outer), len(inner), 0, 0, []
    while o < no or i < ni:
        to = ao[(o + 1) % no] + (2 * math.pi if o + 1 >= no else 0.0)
        ti = ai[(i + 1) % ni] + (2 * math.pi if i + 1 >= ni else 0.0)
        if i >= ni or (o < no and to <= ti):
            tri.append((outer[o % no], outer[(o + 1) % no], inner[i % ni]))
            o += 1
        else:
            tri.append((outer[o % no], inner[(i + 1) % ni], inner[i % ni]))
            i += 1
    return np.asarray(tri)


def _housing(target, radius, length, thick, height, fins=24):
    """Closed finned cylinder of about `target` triangles: an outline with `fins`
    rectangular fins extruded along z, its ends closed by a disk of concentric
    rings and a grid on every fin."""
    base = math.sqrt(radius ** 2 - thick ** 2 / 4)
    top = radius + height
    area = (2 * math.pi * radius + fins * 2 * height) * length + 2 * (math.pi * radius ** 2 + fins * thick * height)
    h = math.sqrt(2.0 * area / target)
    ns, nt, nz = (max(1, round(x / h)) for x in (height, thick, length))
    half = math.asin(thick / 2 / radius)
    gap = 2 * math.pi / fins - 2 * half
    na = max(1, round(gap * radius / h))
    rr, tt = np.linspace(base, top, ns + 1), np.linspace(-thick / 2, thick / 2, nt + 1)
    outline, circle, caps = [], [], []
    for k in range(fins):
        th = 2 * math.pi * k / fins
        er, et = np.array([math.cos(th), math.sin(th)]), np.array([-math.sin(th), math.cos(th)])
        grid = rr[:, None, None] * er + tt[None, :, None] * et       # (ns + 1, nt + 1, 2)
        ang = th + half + gap * np.arange(na + 1) / na
        arc = radius * np.stack([np.cos(ang), np.sin(ang)], 1)
        outline += [grid[:-1, 0], grid[-1, :-1], grid[:0:-1, -1], arc[:-1]]
        circle += [grid[0, :-1], arc[:-1]]
        caps.append(_quads(*(x.reshape(-1, 2) for x in (grid[:-1, :-1], grid[1:, :-1], grid[1:, 1:], grid[:-1, 1:]))))
    outline, prev = np.concatenate(outline), np.concatenate(circle)
    rings, count = max(1, round(radius / h)), len(prev)
    for k in range(rings - 1, 0, -1):
        m = max(6, round(count * k / rings))
        ang = 2 * math.pi * (np.arange(m) + 0.5 * (k % 2)) / m
        ring = radius * k / rings * np.stack([np.cos(ang), np.sin(ang)], 1)
        caps.append(_zip_rings(prev, ring))
        prev = ring
    prev = prev[np.argsort(np.arctan2(prev[:, 1], prev[:, 0]) % (2 * math.pi))]
    caps.append(np.stack([prev, np.roll(prev, -1, 0), np.zeros_like(prev)], 1))
    cap = np.concatenate(caps)                                       # counter-clockwise in the plane
    e1, e2 = cap[:, 1] - cap[:, 0], cap[:, 2] - cap[:, 0]
    flip = e1[:, 0] * e2[:, 1] - e1[:, 1] * e2[:, 0] < 0
    cap[flip] = cap[flip][:, [0, 2, 1]]
    nxt = np.roll(outline, -1, 0)
    z = np.linspace(0.0, length, nz + 1)

    def lift(p, zz):
        return np.concatenate([p, np.full(p.shape[:-1] + (1,), zz)], -1)

    soup = [_quads(lift(outline, a), lift(nxt, a), lift(nxt, b), lift(outline, b)) for a, b in zip(z[:-1], z[1:])]
    return np.concatenate(soup + [lift(cap, length), lift(cap[:, [0, 2, 1]], 0.0)])


def _geometry(case, seed):
    """(xyz, tri, wave speed) of the case's mesh."""
    rng = np.random.default_rng([seed, 1])
    if case["mesh"] == "sphere":
        soup, c = _sphere(case["size"]) * rng.uniform(0.9, 1.1, 3), 1.0
    else:
        soup = _housing(case["size"], 0.1, 0.3, 0.01, 0.02) - np.array([0.0, 0.0, 0.15])
        soup, c = soup * rng.uniform(0.95, 1.05, 3), 343.0
    q, _ = np.linalg.qr(rng.standard_normal((3, 3)))
    xyz, tri = _merge(soup @ (q if np.linalg.det(q) > 0 else -q))
    return xyz, tri, c


def _frequencies(case, seed):
    """The frequency set, the step sizes (stepping) and the contour weights (stepping)."""
    rng = np.random.default_rng([seed, 2])
    L = case["freqs"]
    dt = (1e-4 if case["mesh"] == "housing" else 0.02) * rng.uniform(0.9, 1.1)
    if case["op"] != "stepping":
        # the BDF2 generating function on a circle, closed under conjugation
        z = 10.0 ** (-16.0 / max(L, 64)) * np.exp(2j * np.pi * np.arange(L) / L)
        s = ((1.0 - z) + 0.5 * (1.0 - z) ** 2) / dt
        k = np.arange(1, (L + 1) // 2)
        s[L - k] = np.conj(s[k])
        s[0] = s[0].real
        if L % 2 == 0:
            s[L // 2] = s[L // 2].real
        return s, dt, None
    if case["mesh"] == "sphere":
        dt *= 2.5 * case["stages"]
    # step points first, then the contour of a slightly larger step range (with
    # one step point and an odd contour the set pairs up as k <-> L - k)
    A = _butcher(case)
    lam = np.linalg.eigvals(np.linalg.inv(A))
    m = len(lam)
    nq = L - m - (1 if m == 1 and (L - m) % 2 == 0 else 0)
    s, w = g.contour(nq, *g.contour_steps(A, dt, 1.5 * dt))
    return np.concatenate([lam / dt, s]), dt, w


def _butcher(case):
    return np.array([[1.0]]) if case["stages"] == 1 else np.array([[5 / 12, -1 / 12], [3 / 4, 1 / 4]])


def _vector(shape, seed, k=0, dtype=torch.complex128):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(8 * seed + k)
    return torch.randn(shape, dtype=dtype, device=DEV, generator=gen)


def _dtype(case):
    return torch.complex128 if case["prec"] == "c128" else torch.complex64


def _sample(case, seed, n):
    rng = np.random.default_rng([seed, 3])
    rows, cols = (np.sort(rng.choice(n, min(k, n), replace=False)).astype(np.int32)
                  for k in (case["rows"], case["cols"]))
    fidx = np.sort(rng.choice(case["freqs"], case["use"], replace=False)).astype(np.int32)
    return rows, cols, fidx


# ---- the cases ------------------------------------------------------------------------

def prepare(case, seed):
    xyz, tri, c = _geometry(case, seed)
    s, dt, w = _frequencies(case, seed)
    ctx = g.Context(0)
    ctx.upload_mesh(xyz, tri, c)
    # (the step points of a method of several stages break the pairing k <-> L - k)
    ctx.set_frequencies(s, case.get("stages", 1) == 1)
    ctx.build_cluster_tree(case["leaf"], case["eta"])
    st = dict(case=case, ctx=ctx, prec=PREC[case["prec"]])
    op, n, L = case["op"], len(tri), len(s)
    if op == "entries":
        st["rows"], st["cols"], st["fidx"] = _sample(case, seed, n)
        st["out"] = torch.empty((len(st["fidx"]), len(st["cols"]), len(st["rows"])), dtype=_dtype(case), device=DEV)
        return st
    build = g.C128 if case["prec"] == "c128" else g.C64
    flags = g.FLAG_DOUBLE_LAYER if case.get("dlp") else 0
    st.update(build=build, flags=flags)
    if op in ("product", "wsum", "solve", "stepping"):
        # the launch parameters the autotuner picks on the housings
        ctx.set_tuning(aca3d_waves=(2, 4, 4, 4), aca3d_stack_slices=4)
        ctx.aca3d(case["tol"], case["tol"], 64, build, flags)
    elif op == "fmm":
        ctx.fmm3d(case["order"], case["tol"], 64, build)
    if op == "stepping":
        st.update(dt=dt, w=w, A=_butcher(case), Q=_vector((case["steps"], case["stages"], n), seed,
                                                          dtype=torch.float64))
        st["F"] = torch.empty_like(st["Q"])
    else:
        st["X"] = _vector((L, n), seed, dtype=torch.complex128 if op == "solve" else _dtype(case))
        st["Y"] = torch.empty((n,) if op == "wsum" else (L, n), dtype=st["X"].dtype, device=DEV)
    if op not in ("hmatrix", "operator"):
        ctx.trim()   # the build's working memory, not needed by what follows
    return st


def run(st):
    case, ctx, prec = st["case"], st["ctx"], st["prec"]
    op = case["op"]
    if op == "entries":
        call = ctx.assemble_dlp_slices if case["dlp"] else ctx.assemble_slices
        return call(st["rows"], st["cols"], st["fidx"], prec, st["out"])
    if op == "hmatrix":
        ctx.aca_blocks(case["tol"], 64, st["build"], g.FLAG_RECOMPRESS | st["flags"])
        return ctx.compressed_matvec(g.PLAIN_H, prec, st["X"], st["Y"])
    if op == "operator":
        ctx.aca3d(case["tol"], case["tol"], 64, st["build"], st["flags"])
        return ctx.compressed_matvec(g.PER_FREQUENCY, prec, st["X"], st["Y"])
    if op == "product":
        return ctx.compressed_matvec(g.PER_FREQUENCY, prec, st["X"], st["Y"])
    if op == "wsum":
        return ctx.compressed_matvec(g.WEIGHTED_SUM, prec, st["X"], st["Y"])
    if op == "fmm":
        return ctx.fmm3d_matvec(st["X"], st["Y"])
    if op == "solve":
        ctx.solve(st["X"], st["Y"], rtol=case["rtol"], precision=prec)
        # the densities in the operator's precision, as its products take them
        return st["Y"].to(torch.complex64)
    ctx.gcq_convolve(st["dt"], st["w"], st["Q"], st["F"], precision=prec, A=st["A"], n_step_points=case["stages"])
    return st["F"].to(torch.float32)   # as above


def _storage(case, n):
    """About the stored numbers of the compressed operator: dense near blocks of
    seven or so terms along the frequencies (one term per frequency in an
    H-matrix), and factors that grow with the tree's depth."""
    near = n * 10.0 * 0.65 * case["leaf"]
    far = n * max(1.0, math.log2(n / case["leaf"]))
    if case["op"] == "hmatrix":
        K = case["freqs"] // 2 + 1
        return K * (near + 60.0 * far)
    return 7.0 * near + 3500.0 * far


def work(case):
    n = 20 * case["size"] ** 2 if case["mesh"] == "sphere" else case["size"]
    L, op = case["freqs"], case["op"]
    z = 16 if case["prec"] == "c128" else 8
    if op == "entries":
        e = case["rows"] * case["cols"] * case["use"]
        return {"bytes": e * z, "flops": e * 7 * 20}
    stored = _storage(case, n)
    vec = 2 * n * L * z
    if op == "hmatrix":
        # every stored factor element is one kernel entry of its row or column
        return {"bytes": stored * z * 2 + vec, "flops": stored * (140 + 8 * L / (L // 2 + 1))}
    if op == "operator":
        return {"bytes": stored * z * 2 + vec, "flops": stored * (140 + 8 * L)}
    if op == "wsum":
        return {"bytes": stored * z + vec / 2, "flops": stored * 16}
    if op == "fmm":
        p3 = case["order"] ** 3
        stored = 7 * (n * 10.0 * 0.65 * case["leaf"] + 1.4 * n * p3 * p3)
        return {"bytes": stored * z + vec, "flops": 8.0 * L * stored}
    passes = {"product": 1, "solve": 30, "stepping": case.get("steps", 1) * case.get("stages", 1)}[op]
    return {"bytes": passes * (stored * z + vec), "flops": passes * 8.0 * L * stored}


# ---- plain values in 64 bits ------------------------------------------------------------

class _Panels:
    """The collocation matrix of the single or double layer with flat triangles,
    written out: centroids, a 7-point rule of degree 5 on far panels, the same
    on 16 sub-triangles of near ones (centroids closer than twice the longest
    edge), polar coordinates with 16 Gauss-Legendre angles per edge on the
    panel itself (0 for the double layer)."""

    def __init__(self, xyz, tri, c, dlp):
        self.c, self.dlp = c, dlp
        v = torch.from_numpy(xyz[tri]).to(DEV)                        # (n, 3, 3)
        self.v, self.x = v, (v[:, 0] + v[:, 1] + v[:, 2]) / 3.0
        cr = torch.linalg.cross(v[:, 1] - v[:, 0], v[:, 2] - v[:, 0])
        self.area = 0.5 * cr.norm(dim=1)
        self.nrm = cr / cr.norm(dim=1, keepdim=True)
        self.h2 = torch.stack([((v[:, i] - v[:, j]) ** 2).sum(1) for i, j in ((0, 1), (1, 2), (2, 0))]).amax(0)
        q = math.sqrt(15.0)
        a, b = (6 - q) / 21, (6 + q) / 21
        pts = [(1 / 3, 1 / 3, 1 / 3), (a, a, 1 - 2 * a), (a, 1 - 2 * a, a), (1 - 2 * a, a, a), (b, b, 1 - 2 * b),
               (b, 1 - 2 * b, b), (1 - 2 * b, b, b)]
        wts = [9 / 40] + [(155 - q) / 1200] * 3 + [(155 + q) / 1200] * 3
        subs = [np.eye(3)]
        for _ in range(2):
            cut = []
            for p in subs:
                m = [(p[0] + p[1]) / 2, (p[1] + p[2]) / 2, (p[2] + p[0]) / 2]
                cut += [np.stack(x) for x in ((p[0], m[0], m[2]), (m[0], p[1], m[1]), (m[2], m[1], p[2]), tuple(m))]
            subs = cut
        self.far = tuple(torch.tensor(np.asarray(x), device=DEV) for x in (pts, wts))
        self.near = (torch.tensor(np.concatenate([np.asarray(pts) @ p for p in subs]), device=DEV),
                     torch.tensor(np.asarray(wts * 16) / 16.0, device=DEV))

    def _sum(self, d, w, nrm, freqs):
        """Per frequency s the sum over the last axis of w U(|d|, s), or of its
        normal derivative."""
        r = d.norm(dim=-1)
        f = w / (4 * math.pi * r)
        if self.dlp:
            f = f * (d * nrm).sum(-1) / (r * r)
        for s in freqs:
            k = complex(s) / self.c
            e = f * torch.exp(-k.real * r)
            re, im = e * torch.cos(k.imag * r), -e * torch.sin(k.imag * r)
            if self.dlp:
                pr, pi = 1.0 + k.real * r, k.imag * r
                re, im = re * pr - im * pi, re * pi + im * pr
            yield torch.complex(re.sum(-1), im.sum(-1))

    def _self(self, i, s):
        if self.dlp:
            return torch.zeros(len(i), dtype=torch.complex128, device=DEV)
        gx, gw = (torch.tensor(x, device=DEV) for x in np.polynomial.legendre.leggauss(16))
        k = complex(s) / self.c
        total = 0
        for e in range(3):
            p, q = self.v[i, e] - self.x[i], self.v[i, (e + 1) % 3] - self.x[i]
            t = (q - p) / (q - p).norm(dim=1, keepdim=True)
            tp, tq = (p * t).sum(1), (q * t).sum(1)
            d = (p - tp[:, None] * t).norm(dim=1)
            ta, tb = torch.atan2(tp, d), torch.atan2(tq, d)
            R = d[:, None] / torch.cos(ta[:, None] + (tb - ta)[:, None] * (gx + 1) / 2)
            a = k * R
            # (1 - exp(-a)) / a, by its series where the difference would cancel
            series = 1 - a / 2 * (1 - a / 3 * (1 - a / 4 * (1 - a / 5)))
            phi = torch.where(a.abs() < 1e-3, series, (1 - torch.exp(-a)) / a)
            total = total + (tb - ta) / (4 * math.pi) * ((R * phi) * (gw / 2)).sum(1)
        return total

    def blocks(self, rows, cols, freqs):
        """Yields (first row, (F, rows, cols) entries) over slabs of rows."""
        bary, wt = self.far
        y = torch.einsum("qc,jcd->jqd", bary, self.v[cols])
        w = wt * self.area[cols][:, None]
        step = max(1, int(2e7 / len(cols) / 7))
        for a in range(0, len(rows), step):
            ra = rows[a:a + step]
            d = self.x[ra][:, None, None, :] - y[None]
            out = torch.stack(list(self._sum(d, w[None], self.nrm[cols][None, :, None, :], freqs)))
            d2 = ((self.x[ra][:, None, :] - self.x[cols][None]) ** 2).sum(-1)
            same = ra[:, None] == cols[None, :]
            i, j = torch.nonzero((d2 < 4.0 * self.h2[cols][None]) & ~same, as_tuple=True)
            nb, nw = self.near
            for p in range(0, len(i), 200000):
                ip, jp = i[p:p + 200000], j[p:p + 200000]
                cj = cols[jp]
                dn = self.x[ra[ip]][:, None, :] - torch.einsum("qc,jcd->jqd", nb, self.v[cj])
                for f, v in enumerate(self._sum(dn, nw * self.area[cj][:, None], self.nrm[cj][:, None, :], freqs)):
                    out[f, ip, jp] = v
            i, j = torch.nonzero(same, as_tuple=True)
            for f, s in enumerate(freqs):
                out[f, i, j] = self._self(ra[i], s)
            yield a, out


def exact(case, seed):
    op = case["op"]
    xyz, tri, c = _geometry(case, seed)
    s, dt, w = _frequencies(case, seed)
    n, L = len(tri), len(s)
    P = _Panels(xyz, tri, c, bool(case.get("dlp")))
    if op == "entries":
        rows, cols, fidx = _sample(case, seed, n)
        tr, tc = torch.from_numpy(rows).long().to(DEV), torch.from_numpy(cols).long().to(DEV)
        A = torch.cat([b for _, b in P.blocks(tr, tc, s[fidx])], 1)
        return A.transpose(1, 2).contiguous()
    K = L if case.get("stages", 1) > 1 else L // 2 + 1
    if 7.0 * n * n * K > 1.2e11 or (op == "solve" and 16.0 * n * n * K > 4e10):
        return None
    every = torch.arange(n, device=DEV)
    if op == "stepping":
        return _steps(case, seed, P, every, s, dt, w)
    X = _vector((L, n), seed, dtype=torch.complex128 if op == "solve" else _dtype(case)).to(torch.complex128)
    # V(conj s) x = conj(V(s) conj(x)): the upper half of the set comes with the lower
    Y = torch.zeros((L, n), dtype=torch.complex128, device=DEV)
    per = max(1, int(8e9 / (16.0 * n * n))) if op == "solve" else 16
    for k0 in range(0, K, per):
        ks = list(range(k0, min(K, k0 + per)))
        two = [[k] + ([L - k] if 0 < k and L - k != k else []) for k in ks]
        if op == "solve":
            V = torch.cat([b for _, b in P.blocks(every, every, s[ks])], 1)
        for a, blk in (enumerate([V]) if op == "solve" else P.blocks(every, every, s[ks])):
            for f, pair in enumerate(two):
                rhs = torch.stack([X[q].conj().resolve_conj() if q != ks[f] else X[q] for q in pair], 1)
                y = torch.linalg.solve(blk[f], rhs) if op == "solve" else blk[f] @ rhs
                for i, q in enumerate(pair):
                    v = y[:, i].conj() if q != ks[f] else y[:, i]
                    Y[q, a:a + len(v)] = v
    return Y.sum(0) if op == "wsum" else Y


def _steps(case, seed, P, every, s, dt, w):
    """The stepping with every operator dense: the states of all steps first,
    then one product per frequency with the columns of all steps and stages."""
    m, N, n = case["stages"], case["steps"], len(every)
    A = _butcher(case)
    lam, E = np.linalg.eig(np.linalg.inv(A))
    Ei = np.linalg.inv(E)
    Q = _vector((N, m, n), seed, dtype=torch.float64)
    F = torch.zeros((N, m, n), dtype=torch.float64, device=DEV)
    for k, sk in enumerate(s):
        cols = torch.zeros((N, m, n), dtype=torch.complex128, device=DEV)
        if k < m:
            e = int(np.argmin(np.abs(lam / dt - sk)))
            t = torch.tensor(Ei[e], device=DEV).to(torch.complex128)
            for i in range(m):
                cols[:, i] = complex(E[i, e]) * torch.einsum("j,njp->np", t, Q.to(torch.complex128))
        else:
            M = np.linalg.inv(np.eye(m) - dt * sk * A)
            u, gr = M.sum(1), torch.tensor(dt * (M @ A)[-1], device=DEV)
            x = torch.zeros(n, dtype=torch.complex128, device=DEV)
            for q in range(N):
                if q > 0:
                    x = complex(u[-1]) * x + (gr[:, None] * Q[q - 1]).sum(0)
                for i in range(m):
                    cols[q, i] = complex(w[k - m] * u[i]) * x
        flat = cols.reshape(N * m, n).T.contiguous()
        for a, blk in P.blocks(every, every, [sk]):
            F.view(N * m, n)[:, a:a + blk.shape[1]] += (blk[0] @ flat).real.T
    return F
