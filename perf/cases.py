"""What the speed of this framework is measured on: the work its users have it do.

A case is a dict of plain values. ``listed()`` holds the fixed ones, ``draw(rng)`` gives more of
the same ranges, ``prepare(case, seed)`` builds what a program has in hand before the call (the
rock image, the domain or the pool), ``run(state)`` is one pass through the public entry points,
``work(case)`` the bytes and operations a pass cannot do without, and ``exact(case, seed)`` the
same outputs from a plain float64 evaluation in torch that shares no code with the framework.

Images are drawn on the GPU from the seed: a thresholded Gaussian random field of correlation
length 4 (the synthetic rock of this repository's benchmark) or overlapping spheres of radius 3
to 6 (its bead pack). A pass of the time-stepping cases is a stretch of steps between two
analyses, then the analysis: the reductions and the fields a program looks at. 200 steps are the
solve server's chunk.
"""
import math

import numpy as np
import torch

from paper_2007_12266_amd import lbm
from paper_2007_12266_amd.inputs import Problem

PRECISION = {"fp64": lbm.FP64, "mixed": lbm.FP32_MIXED, "fp32": lbm.FP32_DEV}
DEV = "cuda" if torch.cuda.is_available() else "cpu"
TAU, ALPHA, BETA, FORCE = 0.7, 0.005, 0.95, 1e-5
RHO_IN, RHO_OUT, RESERVOIR = 1.03, 0.97, 4
GROUP_BYTES = 256 << 20            # the solve server's cache groups
MORPH_DELTA, MORPH_RELAX, MORPH_RADIUS, MORPH_BAND = 0.5, 20, 6, 2.5
ALL_FIELDS, TWO_FIELDS = "phi,rho,ux,uy,uz", "phi,uz"


def _steps(name, scenario, nx, ny, nz, porosity, precision, steps, fields):
    c = {"work": "steps", "scenario": scenario, "nx": nx, "ny": ny, "nz": nz,
         "porosity": porosity, "precision": precision, "steps": steps, "fields": fields}
    return dict(c, name=name) if name else c


def listed():
    return [
        # The smallest domain in use: a 32^3 bead pack with walls in z (the parity problem).
        # Launches and latency decide.
        _steps("spheres32_fp64", "spheres", 32, 32, 32, 0.6, "fp64", 200, ALL_FIELDS),
        # The smallest request of the solve server, in its precision.
        _steps("flow64_mixed", "flow", 64, 64, 64, 0.25, "mixed", 200, ALL_FIELDS),
        # Injection through pressure faces into a plug of rock: ghost and face kernels each step.
        _steps("disp128_fp64", "displacement", 128, 128, 128, 0.2, "fp64", 200, ALL_FIELDS),
        # An uneven sub-volume (rows not a multiple of a wave) in the fastest storage.
        _steps("flow150_fp32", "flow", 150, 107, 121, 0.27, "fp32", 200, ALL_FIELDS),
        # The steady-flow rock.
        _steps("flow256_fp64", "flow", 256, 256, 256, 0.2, "fp64", 200, TWO_FIELDS),
        # A large request of the solve server, in its precision.
        _steps("flow320_mixed", "flow", 320, 320, 320, 0.2, "mixed", 100, TWO_FIELDS),
        # The headline benchmark: displacement in a 512^3 rock.
        _steps("disp512_fp64", "displacement", 512, 512, 512, 0.2, "fp64", 200, TWO_FIELDS),
        # A batch of uneven sub-volumes stepped together, as the batched benchmark draws them.
        {"name": "pool16_mixed", "work": "pool", "members": 16, "lo": 48, "hi": 160, "shapes": 1,
         "precision": "mixed", "steps": 200},
        # Many small volumes together: the pool's tiles are spread over many members.
        {"name": "pool32small_fp32", "work": "pool", "members": 32, "lo": 32, "hi": 72,
         "shapes": 2, "precision": "fp32", "steps": 200},
        # A round of shell aggregation out and back: dilate fluid a, relax, erode it, relax.
        {"name": "morph200_fp64", "work": "morph", "nx": 200, "ny": 200, "nz": 200,
         "porosity": 0.25, "precision": "fp64"},
        # Morphological drainage of a rock image from its inlet (host image in, mask out).
        {"name": "drain256", "work": "drain", "nx": 256, "ny": 256, "nz": 256, "porosity": 0.25,
         "target": 0.5},
        # Distance transform of an image that is on the GPU already.
        {"name": "distance128", "work": "distance", "nx": 128, "ny": 128, "nz": 128,
         "porosity": 0.25},
    ]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _edges(rng, lo, hi):
    base = _log_uniform(rng, lo, hi)
    return [max(24, int(round(base * rng.uniform(0.75, 1.3)))) for _ in range(3)]


def draw(rng):
    kind = rng.choices(["steps", "pool", "morph", "drain", "distance"], [6, 2, 1, 1, 1])[0]
    precision = rng.choice(["fp64", "mixed", "fp32"])
    if kind == "pool":
        lo = int(_log_uniform(rng, 28, 64))
        return {"work": "pool", "members": rng.randint(3, 32), "lo": lo,
                "hi": int(lo * rng.uniform(1.3, 2.5)), "shapes": rng.randrange(1 << 20),
                "precision": precision, "steps": 200}
    porosity = round(rng.uniform(0.15, 0.35), 3)
    if kind in ("drain", "distance"):
        nx, ny, nz = _edges(rng, 40, 260 if kind == "drain" else 118)
        c = {"work": kind, "nx": nx, "ny": ny, "nz": nz, "porosity": porosity}
        return dict(c, target=round(rng.uniform(0.3, 0.7), 3)) if kind == "drain" else c
    if kind == "morph":
        nx, ny, nz = _edges(rng, 40, 200)
        return {"work": "morph", "nx": nx, "ny": ny, "nz": nz, "porosity": porosity,
                "precision": precision}
    scenario = rng.choice(["spheres", "flow", "flow", "displacement"])
    if scenario == "spheres":
        nx, ny, nz = _edges(rng, 28, 80)
        porosity = round(rng.uniform(0.4, 0.65), 3)
    else:
        nx, ny, nz = _edges(rng, 40, 400)
    fields = ALL_FIELDS if nx * ny * nz <= 160 ** 3 else TWO_FIELDS
    c = _steps(None, scenario, nx, ny, nz, porosity, precision, 200, fields)
    most = work([k for k in listed() if k["name"] == "disp512_fp64"][0])["bytes"]
    while work(c)["bytes"] > most:
        c["nx"], c["ny"], c["nz"] = (int(0.9 * c[k]) for k in ("nx", "ny", "nz"))
    return c


# ---- Images, drawn on the GPU ----------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed) & 0x7FFFFFFF)


def _lowest(g, share):
    """Mask of the lowest values of g: a share of them that the seed does not change."""
    flat = g.reshape(-1)
    k = max(1, int(share * flat.numel()))
    at = flat.sort().values[k - 1]
    mask = flat < at
    mask[(flat == at).nonzero().reshape(-1)[: k - int(mask.sum())]] = True
    return mask.reshape(g.shape)


def _rock(nx, ny, nz, porosity, seed, corr=4.0):
    """Pore mask [nz, ny, nx] of a thresholded periodic Gaussian random field."""
    g = torch.randn((nz, ny, nx), generator=_generator(seed), device=DEV)
    s = corr / math.sqrt(2.0)            # the filter's; the field's covariance has length corr
    reach = int(4 * s)
    for axis in range(3):
        out = torch.zeros_like(g)
        for k in range(-reach, reach + 1):
            out.add_(torch.roll(g, k, axis), alpha=math.exp(-0.5 * (k / s) ** 2))
        g = out
    return _lowest(g, porosity)


def _spheres(nx, ny, nz, porosity, seed):
    """Pore mask of overlapping solid spheres of radius 3 to 6, periodic in x and y (the radii
    are scaled together, so that the porosity is the stated one)."""
    mean = 4.0 / 3.0 * math.pi * sum(r ** 3 for r in (3, 4, 5, 6)) / 4
    count = max(1, round(-math.log(porosity) * nx * ny * nz / mean))
    r = torch.rand((count, 4), generator=_generator(seed), device=DEV).cpu().numpy()
    z, y, x = (torch.arange(n, device=DEV) + 0.5 for n in (nz, ny, nx))
    near = torch.full((nz, ny, nx), math.inf, device=DEV)
    for a, b, c, d in r:
        dx, dy = (x - float(a) * nx).abs(), (y - float(b) * ny).abs()
        dx, dy = torch.minimum(dx, nx - dx), torch.minimum(dy, ny - dy)
        dz = z - float(c) * nz
        d2 = (dz * dz)[:, None, None] + (dy * dy)[None, :, None] + (dx * dx)[None, None, :]
        near = torch.minimum(near, d2.sqrt() / (3 + int(4 * d)))
    return _lowest(-near, porosity)


def _image(c, seed):
    """Image, wetting, initial phase and boundaries of one domain, as torch tensors."""
    nx, ny, nz = c["nx"], c["ny"], c["nz"]
    scenario = c.get("scenario", "flow")
    g = _generator(seed + 7)
    d = {"shape": (nz, ny, nx), "affinity": None, "wall": 0.0, "force": FORCE, "faces": False,
         "periodic": (True, True, True)}
    if scenario == "displacement":
        d["pore"] = torch.ones((nz, ny, nx), dtype=torch.bool, device=DEV)
        d["pore"][RESERVOIR:nz - RESERVOIR] = _rock(nx, ny, nz - 2 * RESERVOIR, c["porosity"],
                                                    seed)
        d["phi0"] = -torch.ones((nz, ny, nx), dtype=torch.float64, device=DEV)
        d["phi0"][:RESERVOIR] = 1.0
        d.update(solid=-0.7, wall=-0.7, force=0.0, faces=True, periodic=(True, True, False))
        return d
    if scenario == "spheres":
        d["pore"] = _spheres(nx, ny, nz, c["porosity"], seed)
        d.update(solid=0.5, wall=0.5, periodic=(True, True, False))
    else:
        d["pore"] = _rock(nx, ny, nz, c["porosity"], seed)
        d["solid"] = 0.0
        d["affinity"] = 1.8 * torch.rand((nz, ny, nx), generator=g, device=DEV,
                                         dtype=torch.float64) - 0.9
    ones = torch.rand((nz, ny, nx), generator=g, device=DEV) < 0.5
    d["phi0"] = torch.where(ones, 1.0, -1.0).double()
    return d


def _problem(d):
    host = lambda t: None if t is None else t.cpu().numpy()  # noqa: E731
    return Problem(labels=host(d["pore"].int()), label_kind=np.array([0, 3], dtype=np.int8),
                   label_affinity=np.array([d["solid"], 0.0]), voxel_affinity=host(d["affinity"]),
                   init_phi=host(d["phi0"]), periodic=d["periodic"], tau_a=TAU, tau_b=TAU,
                   alpha=ALPHA, beta=BETA, force=(0.0, 0.0, d["force"]), wall_affinity=d["wall"],
                   bc_z=1 if d["faces"] else 0, rho_in=RHO_IN if d["faces"] else 1.0,
                   rho_out=RHO_OUT if d["faces"] else 1.0)


def _members(c):
    """The shapes of a pool's members: edges, porosity of each."""
    r = np.random.RandomState(c["shapes"])
    return [dict(zip(("nx", "ny", "nz"), (int(e) for e in r.randint(c["lo"], c["hi"] + 1, 3))),
                 porosity=float(r.uniform(0.15, 0.35))) for _ in range(c["members"])]


# ---- The framework's side --------------------------------------------------------------------

def prepare(case, seed):
    kind = case["work"]
    if kind in ("drain", "distance"):
        pore = _rock(case["nx"], case["ny"], case["nz"], case["porosity"], seed).byte()
        if kind == "drain":
            return {"case": case, "pore": pore.cpu().numpy()}
        return {"case": case, "feature": 1 - pore,
                "out": torch.empty(pore.shape, dtype=torch.int32, device=DEV),
                "stream": torch.cuda.current_stream().cuda_stream}
    precision = PRECISION[case["precision"]]
    if kind == "pool":
        pool = lbm.Pool(64 << 30, precision=precision, max_slots=64, chunk_steps=100)
        pool.set_group_bytes(GROUP_BYTES)
        doms = []
        for k, m in enumerate(_members(case)):
            doms.append(lbm.Domain(_problem(_image(m, 1000 * seed + k)), precision=precision))
            pool.admit(doms[-1])
        return {"case": case, "pool": pool, "doms": doms}
    return {"case": case, "dom": lbm.Domain(_problem(_image(case, seed)), precision=precision)}


def _analysis(r):
    return {"sw": np.array([r["sw"]]), "mass": np.array([r["mass_a"], r["mass_b"]]),
            "q": np.array([r["qx"], r["qy"], r["qz"]]), "p": np.array([r["p_a"], r["p_b"]])}


def run(state):
    case = state["case"]
    kind = case["work"]
    if kind == "steps":
        d = state["dom"].step(case["steps"])
        out = _analysis(d.reduce())
        for name in case["fields"].split(","):
            out[name] = d.pore_field(name)
        return out
    if kind == "pool":
        pool = state["pool"].step(case["steps"])
        red = pool.reduce()
        rows = [_analysis(red[k]) for k in sorted(red)]
        out = {k: np.stack([r[k] for r in rows]) for k in rows[0]}
        out["phi"] = [d.pore_field("phi") for d in state["doms"]]
        return out
    if kind == "morph":
        d = state["dom"]
        grow = d.morph(delta=MORPH_DELTA, radius=MORPH_RADIUS, band=MORPH_BAND)
        d.step(MORPH_RELAX)
        shrink = d.morph(delta=-MORPH_DELTA, radius=MORPH_RADIUS, band=MORPH_BAND)
        d.step(MORPH_RELAX)
        volumes = [r[k] for r in (grow, shrink) for k in ("volume_before", "volume_after")]
        return {"volumes": np.array(volumes), "phi": d.pore_field("phi")}
    if kind == "drain":
        nw, r = lbm.prep_drain(state["pore"], periodic=(True, True, False),
                               target_sw=case["target"], inlet=True)
        return {"nw": nw, "found": np.array([r["k"], r["kmax"], r["n_pore"], r["n_nw"]])}
    lbm.prep_distance_noalloc(state["feature"], state["out"], periodic=(False, False, False),
                              wall_axes=7, stream=state["stream"])
    return state["out"]


# ---- What a pass cannot do without -----------------------------------------------------------

def _voxels(c):
    """Pore voxels of a domain, from its porosity."""
    n = c["nx"] * c["ny"] * c["nz"]
    if c.get("scenario") == "displacement":
        return c["porosity"] * n + (1 - c["porosity"]) * c["nx"] * c["ny"] * 2 * RESERVOIR
    return c["porosity"] * n


def work(case):
    """Bytes and operations of one pass. A step reads and writes the state once: 19 populations
    and the 8 numbers that fix the component populations of a voxel. About 600 operations."""
    kind = case["work"]
    if kind == "distance":
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": 5.0 * n, "flops": 40.0 * n}
    if kind == "drain":
        # The distance map of the pore space (1 B in, 4 B out); then, for each of about 8 radii
        # tried, the map read and a count formed; the mask out.
        n = case["nx"] * case["ny"] * case["nz"]
        return {"bytes": (5.0 + 8 * 4.0 + 1.0) * n, "flops": 8 * 40.0 * n}
    f, m = {"fp64": (8, 8), "mixed": (4, 8), "fp32": (4, 4)}[case["precision"]]
    step = 2.0 * (19 * f + 8 * m)
    if kind == "pool":
        n = sum(_voxels(c) for c in _members(case))
        return {"bytes": n * (step * case["steps"] + 8 * m), "flops": 600.0 * n * case["steps"]}
    n = _voxels(case)
    if kind == "morph":
        # The component moments in and out twice, and the steps between.
        return {"bytes": n * (2 * MORPH_RELAX * step + 2 * 2 * 8 * m + 8 * m + 8),
                "flops": 600.0 * 2 * MORPH_RELAX * n}
    reads = 19 * f + 8 * m + 8 * len(case["fields"].split(","))
    return {"bytes": n * (step * case["steps"] + reads), "flops": 600.0 * n * case["steps"]}


# ---- Plain float64 evaluation ----------------------------------------------------------------

XI = [(0, 0, 0), (1, 0, 0), (-1, 0, 0), (0, 1, 0), (0, -1, 0), (0, 0, 1), (0, 0, -1),
      (1, 1, 0), (-1, -1, 0), (1, -1, 0), (-1, 1, 0), (1, 0, 1), (-1, 0, -1), (1, 0, -1),
      (-1, 0, 1), (0, 1, 1), (0, -1, -1), (0, 1, -1), (0, -1, 1)]
OPP = [0] + [q + 1 if q % 2 else q - 1 for q in range(1, 19)]
T19 = [1 / 3] + [1 / 18] * 6 + [1 / 36] * 12
W7 = [1 / 3] + [1 / 9] * 6
CMIN = 1e-10                      # a colour gradient of at most this size counts as zero


def _basis():
    """The D3Q19 moments as rows of polynomials in the velocities."""
    rows = []
    for x, y, z in XI:
        c = x * x + y * y + z * z
        a, w = 3 * x * x - c, y * y - z * z
        rows.append([1, 19 * c - 30, (21 * c * c - 53 * c + 24) / 2, x, (5 * c - 9) * x, y,
                     (5 * c - 9) * y, z, (5 * c - 9) * z, a, (3 * c - 5) * a, w, (3 * c - 5) * w,
                     x * y, y * z, x * z, (y * y - z * z) * x, (z * z - x * x) * y,
                     (x * x - y * y) * z])
    return torch.tensor(rows, dtype=torch.float64, device=DEV).T.contiguous()


class _Exact:
    """The two-fluid model on the pore voxels of one image, populations streamed by pulling."""

    def __init__(self, d):
        nz, ny, nx = d["shape"]
        self.d = d
        pore = d["pore"].reshape(-1)
        v = pore.nonzero().reshape(-1)
        x, y, z = v % nx, v // nx % ny, v // (nx * ny)
        # The library numbers the pores in blocks of 16 rows, each block plane by plane.
        v = v[(((y // 16) * nz + z) * 16 * nx + (y % 16) * nx + x).argsort()]
        x, y, z = v % nx, v // nx % ny, v // (nx * ny)
        self.v, n = v, v.numel()
        index = torch.full((nx * ny * nz,), -1, dtype=torch.int64, device=DEV)
        index[v] = torch.arange(n, device=DEV)
        self.phase = torch.full((nx * ny * nz + 1,), d["wall"], dtype=torch.float64, device=DEV)
        self.phase[:-1] = d["solid"] if d["affinity"] is None else d["affinity"].reshape(-1)
        self.near, self.up, self.wall = [None], [None], [None]
        for q in range(1, 19):
            c, outside, beyond = [], None, None
            for a, (p, size, k) in enumerate(((x, nx, 0), (y, ny, 1), (z, nz, 2))):
                t = p + XI[q][k]
                out = (t < 0) | (t >= size)
                if d["periodic"][a]:
                    t, out = t % size, torch.zeros_like(out)
                elif a == 2 and d["faces"]:
                    beyond, out = out, torch.zeros_like(out)   # the phase mirrors the plane
                    t = torch.where(beyond, p, t)
                c.append(t.clamp(0, size - 1))
                outside = out if outside is None else outside | out
            w = c[0] + nx * (c[1] + ny * c[2])
            self.near.append(torch.where(outside, nx * ny * nz, w))
            to = torch.where(outside if beyond is None else outside | beyond, -1, index[w])
            self.up.append(to.clamp(min=0))      # along q; read through OPP when pulling
            self.wall.append(to < 0)
        self.f = torch.tensor(T19, dtype=torch.float64, device=DEV)[:, None].repeat(1, n)
        p0 = d["phi0"].reshape(-1)[v]
        self.rest((1 + p0) / 2, (1 - p0) / 2)
        self.M = _basis()
        self.Minv = torch.linalg.inv(self.M.cpu()).to(DEV)
        self.z0, self.z1 = (z == 0).nonzero().reshape(-1), (z == nz - 1).nonzero().reshape(-1)

    def rest(self, na, nb):
        w = torch.tensor(W7, dtype=torch.float64, device=DEV)[:, None]
        self.a, self.b, self.fresh = w * na, w * nb, True

    def densities(self):
        na, nb = self.a.sum(0), self.b.sum(0)
        if self.d["faces"] and not self.fresh:
            na[self.z0], nb[self.z0], na[self.z1], nb[self.z1] = 1.0, 0.0, 0.0, 1.0
        return na, nb

    def pull(self, x):
        out = torch.empty_like(x)
        out[0] = x[0]
        for q in range(1, x.shape[0]):
            back = OPP[q]
            out[q] = torch.where(self.wall[back], x[back], x[q][self.up[back]])
        return out

    def step(self):
        na, nb = self.densities()
        n = na + nb
        phi = (na - nb) / n
        self.phase[self.v] = phi
        cx, cy, cz = (torch.zeros_like(phi) for _ in range(3))
        for q in range(1, 19):
            p = self.phase[self.near[q]] * (1.0 if q < 7 else 0.5)
            for c, k in ((cx, 0), (cy, 1), (cz, 2)):
                if XI[q][k]:
                    c += XI[q][k] * p
        size = (cx * cx + cy * cy + cz * cz).sqrt()
        size = torch.where(size > CMIN, size, 0.0)
        inv = torch.where(size > 0, 1.0 / size.clamp(min=CMIN), 0.0)
        nx, ny, nz = cx * inv, cy * inv, cz * inv
        del cx, cy, cz, inv
        rate = 1.0 / TAU                              # both fluids have the same viscosity
        odd = 8.0 * (2.0 - rate) / (8.0 - rate)
        m = self.M @ self.f
        rho, jx, jy, jz = m[0].clone(), m[3].clone(), m[5].clone(), m[7].clone()
        jj, g = jx * jx + jy * jy + jz * jz, ALPHA * size
        a, w = 2 * jx * jx - jy * jy - jz * jz, jy * jy - jz * jz
        eq = {1: -11 * rho + 19 * jj - 19 * g, 2: 3 * rho - 5.5 * jj, 4: -2 / 3 * jx,
              6: -2 / 3 * jy, 8: -2 / 3 * jz, 9: a + g / 2 * (2 * nx * nx - ny * ny - nz * nz),
              10: -a / 2, 11: w + g / 2 * (ny * ny - nz * nz), 12: -w / 2,
              13: jx * jy + g / 2 * nx * ny, 14: jy * jz + g / 2 * ny * nz,
              15: jx * jz + g / 2 * nx * nz}
        for k in range(19):
            if k in (0, 3, 5, 7):
                m[k] = 0.0
            else:
                m[k] = (odd if k in (4, 6, 8, 16, 17, 18) else rate) * (m[k] - eq.get(k, 0.0))
        del eq, a, w, jj
        post = self.f - self.Minv @ m
        del m
        force = self.d["force"]
        for q in range(19):
            if XI[q][2] and force:
                post[q] += T19[q] * 3.0 * XI[q][2] * force
        u = (jx, jy, jz + force / 2)
        seg = BETA * na * nb / n
        a7, b7 = (torch.empty((7, n.numel()), dtype=torch.float64, device=DEV) for _ in "ab")
        for q in range(7):
            eu = 4.5 * sum(XI[q][k] * u[k] for k in range(3))
            en = seg * (XI[q][0] * nx + XI[q][1] * ny + XI[q][2] * nz)
            a7[q], b7[q] = W7[q] * (na * (1 + eu) + en), W7[q] * (nb * (1 + eu) - en)
        self.f, self.a, self.b, self.fresh = self.pull(post), self.pull(a7), self.pull(b7), False
        if self.d["faces"]:
            self.face(self.z0, 1, RHO_IN)
            self.face(self.z1, -1, RHO_OUT)

    def face(self, i, into, rho):
        """The populations that enter through a pressure face (Zou and He)."""
        f = self.f[:, i]
        along = [q for q in range(19) if XI[q][2] == 0]
        s0 = sum(f[q] for q in along)
        tx, ty = (sum(XI[q][k] * f[q] for q in along) for k in (0, 1))
        jz = into * (rho - s0 - 2 * sum(f[q] for q in range(19) if XI[q][2] == -into))
        for q in range(19):
            if XI[q][2] == into:
                self.f[q, i] = (f[OPP[q]] + 6 * T19[q] * XI[q][2] * jz
                                - (XI[q][0] * tx + XI[q][1] * ty) / 2)

    def morph(self, delta):
        """Dilates fluid a by delta voxels; its volume before and after."""
        na, nb = self.densities()
        phi = (na - nb) / (na + nb)
        nz, ny, nx = self.d["shape"]
        fluid = torch.zeros(nx * ny * nz, dtype=torch.bool, device=DEV)
        fluid[self.v] = phi > 0
        fluid = fluid.reshape(nz, ny, nx)
        best = torch.full(fluid.shape, 1 << 20, dtype=torch.int32, device=DEV)
        r = MORPH_RADIUS
        for dz in range(-r, r + 1):
            for dy in range(-r, r + 1):
                for dx in range(-r, r + 1):
                    d2 = dx * dx + dy * dy + dz * dz
                    if 0 < d2 <= r * r:
                        other = torch.roll(fluid, (dz, dy, dx), (0, 1, 2)) != fluid
                        best = torch.where(other & (best > d2), d2, best)
        d2 = best.reshape(-1)[self.v].double()
        far = d2 > r * r
        sign = torch.where(phi > 0, -1.0, 1.0)
        band = phi.abs() < math.tanh(MORPH_BAND * BETA)
        dist = torch.where(far, sign * (r + 0.5), sign * (d2.sqrt() - 0.5))
        p = phi.clamp(-0.999999, 0.999999)
        dist = torch.where(band, -torch.log((1 + p) / (1 - p)) / (2 * BETA), dist)
        e = torch.exp(-2 * BETA * (dist - delta))
        new = torch.where(far & ~band, phi, 2 * e / (1 + e) - 1)
        n = na + nb
        self.rest(n * (1 + new) / 2, n * (1 - new) / 2)
        return int((dist < 0).sum()), int((dist - delta < 0).sum())

    def read(self, names):
        na, nb = self.densities()
        rho = self.f.sum(0)
        phi = (na - nb) / (na + nb)
        u = [sum(XI[q][k] * self.f[q] for q in range(19)) for k in range(3)]
        u[2] = u[2] + self.d["force"] / 2
        a, b = phi > 0, phi < 0
        mean = lambda k: float(rho[k].sum() / 3 / k.sum()) if bool(k.any()) else 0.0  # noqa: E731
        box = float(np.prod(self.d["shape"]))
        out = {"sw": np.array([float(((1 + phi) / 2).mean())]),
               "mass": np.array([float(na.sum()), float(nb.sum())]),
               "q": np.array([float(t.sum()) / box for t in u]),
               "p": np.array([mean(a), mean(b)])}
        fields = {"phi": phi, "rho": rho, "ux": u[0], "uy": u[1], "uz": u[2]}
        out.update({k: fields[k] for k in names})
        return out


def exact(case, seed):
    kind = case["work"]
    if kind in ("drain", "distance"):
        return None                              # whole numbers: held to be the same
    if kind == "pool":
        rows = []
        for k, m in enumerate(_members(case)):
            e = _Exact(_image(m, 1000 * seed + k))
            for _ in range(case["steps"]):
                e.step()
            rows.append(e.read(["phi"]))
        out = {k: np.stack([r[k] for r in rows]) for k in ("sw", "mass", "q", "p")}
        return dict(out, phi=[r["phi"] for r in rows])
    if kind == "steps":
        # About 0.3 us per 1000 voxels and step on the GPU: no value where that is over 20 s.
        if _voxels(case) * case["steps"] > 4e9:
            return None
        e = _Exact(_image(case, seed))
        for _ in range(case["steps"]):
            e.step()
        return e.read(case["fields"].split(","))
    e = _Exact(_image(case, seed))
    volumes = []
    for delta in (MORPH_DELTA, -MORPH_DELTA):
        volumes += e.morph(delta)
        for _ in range(MORPH_RELAX):
            e.step()
    return {"volumes": np.array(volumes), "phi": e.read(["phi"])["phi"]}
