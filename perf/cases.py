"""The work a user of the solver has it do, as cases that can be timed and compared.

A case is one call through a public entry point on a periodic cell with sphere
inclusions.  ``kind`` says which:

* ``operator``   ``Problem.apply_operator_noalloc`` on device tensors (a caller's own
                 solver, serving loops); FP64, with or without macro strain and <sigma>
* ``stiffness``  ``Problem.effective_stiffness``: the six unit loads, C_eff
* ``fields``     ``Problem.solve_device``: displacements and <sigma> in device tensors
* ``stress``     ``Problem.solve`` with displacement and voxel-stress fields on the host
* ``gradient``   ``torch_ops.effective_stiffness`` forward and backward
* ``batch``      ``batch_effective_stiffness``: several cells of uneven size

Geometry: non-overlapping periodic spheres by random sequential addition with a
gap of two voxels, exact signed distances in voxel units, one label per sphere;
positions, radii and (where ``phases`` is "each") the moduli of every inclusion come
from the seed (the operator's cell is one for all seeds, its vectors and strains are not).
"""

import itertools
import math

import numpy as np
import torch

DEV = "cuda:0"
F64 = torch.float64


def listed():
    return [
        # one operator application of the smallest cell of the tests: launch latency
        dict(name="operator 16", kind="operator", n0=16, n1=16, n2=16, spheres=1, contrast=10.0, macro=False,
             discretization="xfem"),
        # residual r(x) with macro strain and <sigma> at the size of the benchmark's cell
        dict(name="operator 128 macro", kind="operator", n0=128, n1=128, n2=128, spheres=40, contrast=10.0,
             macro=True, discretization="xfem"),
        # the smallest solve: every launch and every poll counts
        dict(name="stiffness 16 fp64", kind="stiffness", n0=16, n1=16, n2=16, spheres=1, contrast=10.0,
             precision="fp64", batch=True, discretization="xfem"),
        # a small cell with stiff inclusions in mixed precision
        dict(name="stiffness 64 mixed", kind="stiffness", n0=64, n1=64, n2=64, spheres=10, contrast=100.0,
             precision="mixed", batch=True, discretization="xfem"),
        # the benchmark's workload: 128^3, 40 spheres, contrast 10, six loads, mixed precision
        dict(name="stiffness 128 mixed", kind="stiffness", n0=128, n1=128, n2=128, spheres=40, contrast=10.0,
             precision="mixed", batch=True, discretization="xfem"),
        # the same in plain FP64, one load at a time (the benchmark's comparison path)
        dict(name="stiffness 128 fp64", kind="stiffness", n0=128, n1=128, n2=128, spheres=40, contrast=10.0,
             precision="fp64", batch=False, discretization="xfem"),
        # the largest cell of the benchmark's options
        dict(name="stiffness 256 mixed", kind="stiffness", n0=256, n1=256, n2=256, spheres=120, contrast=20.0,
             precision="mixed", batch=True, discretization="xfem"),
        # the voxel-segmented comparison discretisation, without enrichment
        dict(name="stiffness 96 p1", kind="stiffness", n0=96, n1=96, n2=96, spheres=20, contrast=10.0,
             precision="mixed", batch=True, discretization="p1"),
        # an uneven cell whose axes have other factors than the usual powers of two; fields stay on the device
        dict(name="fields 108x72x54", kind="fields", n0=108, n1=72, n2=54, spheres=12, contrast=10.0, loads=3,
             precision="fp64", discretization="xfem"),
        # local fields of one load for post-processing on the host
        dict(name="stress 64", kind="stress", n0=64, n1=64, n2=64, spheres=10, contrast=10.0, precision="fp64",
             discretization="xfem"),
        # identification of the moduli: C_eff and the gradient of a loss, one material per inclusion
        dict(name="gradient 64", kind="gradient", n0=64, n1=64, n2=64, spheres=24, contrast=20.0, phases="each",
             precision="fp64", discretization="xfem"),
        # several cells of uneven size in one call
        dict(name="batch 32-96", kind="batch", sizes="32,48,64,96", contrast=100.0, precision="mixed",
             discretization="xfem"),
    ]


# even axis lengths with prime factors 2 and 3, as the solver takes them
LENGTHS = (12, 16, 18, 24, 32, 36, 48, 54, 64, 72, 96, 108, 128, 144)


def draw(rng):
    kind = rng.choice(("operator", "stiffness", "stiffness", "fields", "stress", "gradient", "batch"))
    top = dict(operator=144, stiffness=144, fields=128, stress=72, gradient=96, batch=0)[kind]
    contrast = round(10.0 ** rng.uniform(0.7, 2.0), 2)
    precision = rng.choice(("fp64", "mixed"))
    if kind == "batch":
        sizes = [rng.choice((16, 24, 32, 36, 48, 64, 72, 96)) for _ in range(rng.randint(2, 6))]
        return dict(kind=kind, sizes=",".join(map(str, sizes)), contrast=contrast, precision=precision,
                    discretization="xfem")
    base = math.exp(rng.uniform(math.log(14.0), math.log(top)))
    near = [v for v in LENGTHS if v <= top and 0.55 * base <= v <= 1.8 * base]
    # cubes are the usual cells; the others are uneven
    n = [rng.choice(near)] * 3 if rng.random() < 0.4 else [rng.choice(near) for _ in range(3)]
    case = dict(kind=kind, n0=n[0], n1=n[1], n2=n[2], spheres=rng.randint(1, 40), contrast=contrast,
                discretization=rng.choice(("xfem", "xfem", "xfem", "p1")))
    if kind == "operator":
        case.update(macro=rng.random() < 0.5)
        return case
    # local fields are asked for in FP64; C_eff and its gradient in either precision
    case["precision"] = "fp64" if kind in ("fields", "stress", "gradient") else precision
    if kind == "stiffness":
        case["batch"] = rng.random() < 0.7
    if kind == "fields":
        case["loads"] = rng.randint(1, 6)
    if kind == "gradient":
        case.update(phases="each", discretization="xfem")
    return case


# ---------------------------------------------------------------- inputs
def _lame(E, nu):
    return [E * nu / ((1.0 + nu) * (1.0 - 2.0 * nu)), E / (2.0 * (1.0 + nu))]


def _cell(n, spheres, contrast, seed, phases="same"):
    """Level set, labels and Lame pairs (host arrays) of a cell of n voxels."""
    rng = np.random.default_rng([int(seed), *n, int(spheres)])
    ext = np.asarray(n, dtype=np.float64)
    vol = float(np.prod(ext))
    # radii that give about 10 % of volume, at least two voxels and within the cell
    r0 = (0.1 * vol / spheres * 3.0 / (4.0 * math.pi)) ** (1.0 / 3.0)
    r0 = min(max(r0, 2.0), 0.35 * float(ext.min()))
    centers, radii = [], []
    for _ in range(4000):
        if len(radii) == spheres:
            break
        r = r0 * rng.uniform(0.8, 1.2)
        c = rng.uniform(0.0, 1.0, 3) * ext
        if centers:
            d = np.asarray(centers) - c
            d -= ext * np.floor(d / ext + 0.5)
            if np.any(np.sqrt((d * d).sum(1)) < r + np.asarray(radii) + 2.0):
                continue
        centers.append(c)
        radii.append(r)
    L, lab = _levelset(n, centers, radii)
    if phases == "each":
        z = rng.standard_normal((len(radii), 2))
        lame = [_lame(1.0, 0.35)] + [_lame(contrast * math.exp(0.25 * a), min(max(0.22 * math.exp(0.1 * b), 0.05), 0.45))
                                     for a, b in z]
    else:
        lame = [_lame(1.0, 0.3)] + [_lame(contrast, 0.25)] * len(radii)
    return L, lab, np.array(lame)


def _levelset(n, centers, radii):
    ax = [torch.arange(v, dtype=F64, device=DEV) for v in n]
    best = torch.full((n[2], n[1], n[0]), math.inf, dtype=F64, device=DEV)
    lab = torch.zeros(best.shape, dtype=torch.int32, device=DEV)
    for i, (c, r) in enumerate(zip(centers, radii)):
        d2 = []
        for a in range(3):
            d = ax[a] - float(c[a])
            d = d - n[a] * torch.floor(d / n[a] + 0.5)
            d2.append(d * d)
        d = torch.sqrt(d2[2][:, None, None] + d2[1][None, :, None] + d2[0][None, None, :]) - float(r)
        lab.masked_fill_(d < best, i + 1)
        best = torch.minimum(best, d)
    lab.masked_fill_(best >= 0, 0)
    return best.reshape(-1).cpu().numpy(), lab.reshape(-1).cpu().numpy()


def _size(case):
    return (case["n0"], case["n1"], case["n2"])


def _problem(n, cell, case):
    from paper_2601_02172_amd import Problem
    L, lab, lame = cell
    return Problem(n, [float(v) for v in n], L, lab, lame, precision=case.get("precision", "fp64"),
                   batch=case.get("batch", True), discretization=case["discretization"])


def _cell_of(case, seed):
    # the operator's vectors hold the enriched unknowns of the cell: one cell, vectors from the seed
    seed = 0 if case["kind"] == "operator" else seed
    return _cell(_size(case), case["spheres"], case["contrast"], seed, case.get("phases", "same"))


def _cells_of_batch(case, seed):
    sizes = [int(v) for v in case["sizes"].split(",")]
    return [((v, v, v), _cell((v, v, v), 3 + v // 8, case["contrast"], seed * 64 + i)) for i, v in enumerate(sizes)]


def _strains(seed, count):
    """Macro strains of about one per mille in every Mandel component."""
    return np.random.default_rng([int(seed), 7]).standard_normal((count, 6)) * 1e-3


def _state_vector(seed, size):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) + 1)
    return torch.randn(size, dtype=F64, device=DEV, generator=g) * 1e-3


_STREAM = []


def _stream():
    """The one stream of the program (the operator's static work space is shared by all calls on a GPU)."""
    if not _STREAM:
        _STREAM.append(torch.cuda.Stream(device=DEV))
    return _STREAM[0]


def _weights(seed):
    W = np.random.default_rng([int(seed), 11]).standard_normal((6, 6))
    return 0.5 * (W + W.T)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return dict(kind=kind, problems=[_problem(n, c, case) for n, c in _cells_of_batch(case, seed)])
    n = _size(case)
    cell = _cell_of(case, seed)
    p = _problem(n, cell, case)
    s = dict(kind=kind, problem=p)
    if kind == "operator":
        s["x"] = _state_vector(seed, 3 * (p.N + p.nX))
        s["y"] = torch.empty_like(s["x"])
        s["strain"] = torch.tensor(_strains(seed, 1)[0], device=DEV) if case["macro"] else None
        s["avg"] = torch.empty(6, dtype=F64, device=DEV) if case["macro"] else None
        s["stream"] = _stream()
    elif kind == "fields":
        nl = case["loads"]
        s["strain"] = torch.tensor(_strains(seed, nl), device=DEV)
        s["disp"] = torch.empty((nl, 3, p.N), dtype=F64, device=DEV)
        s["avg"] = torch.empty((nl, 6), dtype=F64, device=DEV)
    elif kind == "stress":
        s["strain"] = _strains(seed, 1)
    elif kind == "gradient":
        s["lame"] = torch.tensor(cell[2])
        s["weights"] = torch.tensor(_weights(seed))
    return s


def run(s):
    kind = s["kind"]
    if kind == "batch":
        from paper_2601_02172_amd import batch_effective_stiffness
        return batch_effective_stiffness(s["problems"])
    p = s["problem"]
    if kind == "operator":
        avg = s["avg"]
        p.apply_operator_noalloc(s["x"].data_ptr(), s["y"].data_ptr(),
                                 None if s["strain"] is None else s["strain"].data_ptr(),
                                 None if avg is None else avg.data_ptr(), s["stream"].cuda_stream)
        return dict(y=s["y"]) if avg is None else dict(y=s["y"], avg=avg)
    if kind == "fields":
        p.solve_device(s["strain"].data_ptr(), s["strain"].shape[0], s["disp"].data_ptr(), s["avg"].data_ptr())
        return dict(disp=s["disp"], avg=s["avg"])
    if kind == "stress":
        r = p.solve(s["strain"], disp=True, stress=True)
        return dict(disp=r["disp"], stress=r["stress"], avg=r["avg_stress"])
    if kind == "gradient":
        from paper_2601_02172_amd.torch_ops import effective_stiffness
        lame = s["lame"].clone().requires_grad_(True)
        C = effective_stiffness(lame, p)
        C.backward(s["weights"])
        return dict(c_eff=C.detach(), grad=lame.grad)
    C, _ = p.effective_stiffness()
    return C


# ---------------------------------------------------------------- work
def work(case):
    """Bytes and operations one call cannot do without.

    Operator: the level set, labels, x and the strains are read once and y written
    once.  A solve: per load and CG iteration the fields f, u, d are read and
    written, z = A d is written and read, the half spectrum (as large as a field) is
    written and read twice (the transforms along z need all planes) and d is read by
    the operator: 13 fields of 3 N values.  Iterations: about 80 at contrast 10, growing with the
    square root of the contrast (CG).  Operations: 201 per voxel and application of
    the operator, 2 x 2.5 N log2 N per component for the transforms, 60 per
    frequency for the Green multiply, 12 per value for the updates.
    """
    kind = case["kind"]
    if kind == "operator":
        N = case["n0"] * case["n1"] * case["n2"]
        return dict(bytes=N * (2 * 24 + 4.0), flops=250.0 * N)
    its = 80.0 * math.sqrt(max(case["contrast"], 1.0) / 10.0)
    if case["discretization"] == "p1":
        its *= 0.6
    size = 4.0 if case["precision"] == "mixed" else 8.0
    loads = dict(stress=1, fields=case.get("loads", 1)).get(kind, 6)
    grids = [int(v) ** 3 for v in case["sizes"].split(",")] if kind == "batch" else \
        [case["n0"] * case["n1"] * case["n2"]]
    b = f = 0.0
    for N in grids:
        b += its * loads * 13 * 3 * N * size + N * 12.0
        f += its * loads * N * (201 + 3 * 5.0 * math.log2(N) + 60 + 36)
        if kind == "gradient":
            b += 18.0 * N * 8
            f += N * 6 * 21 * 16.0
    return dict(bytes=b, flops=f)


# ---------------------------------------------------------------- 64-bit reference
# Plain torch on every element of the grid: P1 elements on the six Kuhn tetrahedra of
# each voxel, cut elements by the exact second moments of both sides of the linear
# level set, conjugate gradients with the constant-coefficient preconditioner.
PERMS = list(itertools.permutations(range(3)))
COST = 4.5e8       # voxels x loads x iterations the reference takes in about 20 s


def _moments(L):
    """int lambda_c lambda_d over {L > 0} of a tetrahedron of volume 1/6 with vertex values L (m x 4)."""
    v, order = torch.sort(L, dim=1, descending=True)
    eye = torch.eye(4, dtype=F64, device=L.device)
    npos = (v > 0).sum(1)
    M = torch.zeros((L.shape[0], 4, 4), dtype=F64, device=L.device)

    def point(vv, p, q):
        t = (vv[:, p] / (vv[:, p] - vv[:, q]))[:, None]
        return eye[p] * (1 - t) + eye[q] * t

    def piece(rows):
        B = torch.stack(rows, dim=1)
        s = B.sum(1)
        vol = torch.linalg.det(B).abs() / 120.0
        return vol[:, None, None] * (s[:, :, None] * s[:, None, :] + B.transpose(1, 2) @ B)

    full = (torch.ones((4, 4), dtype=F64, device=L.device) + eye) / 120.0
    for k in (1, 2, 3):
        m = npos == k
        if not bool(m.any()):
            continue
        w = v[m]
        e = [eye[a].expand(w.shape[0], 4) for a in range(4)]
        if k == 1:
            M[m] = piece([e[0], point(w, 0, 1), point(w, 0, 2), point(w, 0, 3)])
        elif k == 2:
            a, b = [e[0], point(w, 0, 2), point(w, 0, 3)], [e[1], point(w, 1, 2), point(w, 1, 3)]
            M[m] = piece([a[0], a[1], a[2], b[0]]) + piece([a[1], a[2], b[0], b[1]]) + piece([a[2], b[0], b[1], b[2]])
        else:
            # the prism between the three positive vertices and the section around the last one
            a, b = [e[0], e[1], e[2]], [point(w, 0, 3), point(w, 1, 3), point(w, 2, 3)]
            M[m] = piece([a[0], a[1], a[2], b[0]]) + piece([a[1], a[2], b[0], b[1]]) + piece([a[2], b[0], b[1], b[2]])
    M[npos == 4] = full
    # back from the sorted to the original vertex order
    back = torch.argsort(order, dim=1)
    M = torch.gather(M, 1, back[:, :, None].expand(-1, 4, 4))
    return torch.gather(M, 2, back[:, None, :].expand(-1, 4, 4))


def _tensor(m):
    """Mandel vector(s) to symmetric 3 x 3."""
    r = math.sqrt(0.5)
    rows = [m[..., 0], m[..., 5] * r, m[..., 4] * r, m[..., 5] * r, m[..., 1], m[..., 3] * r, m[..., 4] * r,
            m[..., 3] * r, m[..., 2]]
    return torch.stack(rows, dim=-1).reshape(*m.shape[:-1], 3, 3)


def _mandel(t):
    r = math.sqrt(2.0)
    return torch.stack([t[..., 0, 0], t[..., 1, 1], t[..., 2, 2], r * t[..., 1, 2], r * t[..., 0, 2],
                        r * t[..., 0, 1]], dim=-1)


def _hooke(eps, lam, mu):
    tr = eps.diagonal(dim1=-2, dim2=-1).sum(-1)
    eye = torch.eye(3, dtype=F64, device=eps.device)
    return (lam * tr)[..., None, None] * eye + (2.0 * mu)[..., None, None] * eps


class _Reference:
    def __init__(self, n, cell, discretization):
        self.n, self.N = n, n[0] * n[1] * n[2]
        L = torch.tensor(cell[0], dtype=F64, device=DEV)
        lab = torch.tensor(cell[1], dtype=torch.int64, device=DEV)
        self.lame = torch.tensor(cell[2], dtype=F64, device=DEV)
        L = torch.where(L.abs() < 1e-6, torch.zeros_like(L), L)
        k, j, i = torch.meshgrid(*[torch.arange(v, device=DEV) for v in (n[2], n[1], n[0])], indexing="ij")
        ijk = [i.reshape(-1), j.reshape(-1), k.reshape(-1)]

        def corner(c):
            a = [(ijk[q] + c[q]) % n[q] for q in range(3)]
            return a[0] + n[0] * (a[1] + n[1] * a[2])

        self.types = []
        p1 = discretization == "p1"
        if p1:
            corners = [corner((x, y, z)) for z in (0, 1) for y in (0, 1) for x in (0, 1)]
            inside = sum(L[c] for c in corners) >= 0
            best = torch.full_like(L, -1.0)
            vox = torch.zeros_like(lab)
            for c in corners:
                a = torch.where((L[c] >= 0) == inside, L[c].abs(), torch.full_like(L, -2.0))
                vox = torch.where(a > best, lab[c], vox)
                best = torch.maximum(best, a)
        for perm in PERMS:
            at, verts, e = [0, 0, 0], [], np.eye(3)
            for s in range(4):
                verts.append(corner(tuple(at)))
                if s < 3:
                    at[perm[s]] += 1
            g = torch.tensor(np.array([-e[perm[0]], e[perm[0]] - e[perm[1]], e[perm[1]] - e[perm[2]], e[perm[2]]]),
                             dtype=F64, device=DEV)
            v = torch.stack(verts, dim=1)
            Lv, lv = L[v], lab[v]
            cut = (Lv > 0).any(1) & (Lv < 0).any(1)
            if p1:
                cut = torch.zeros_like(cut)
            t = dict(v=v, g=g, cut=cut)
            for key, val in (("un", Lv.abs()), ("pos", Lv), ("neg", -Lv)):
                b, m = val[:, 0], lv[:, 0]
                for a in range(1, 4):
                    m = torch.where(val[:, a] > b, lv[:, a], m)
                    b = torch.maximum(b, val[:, a])
                t[key] = vox if p1 and key == "un" else m
            t["iu"] = torch.nonzero(~cut).reshape(-1)
            t["vu"], t["mu"] = v[t["iu"]], t["un"][t["iu"]]
            t["ic"] = torch.nonzero(cut).reshape(-1)
            t["L"] = Lv[t["ic"]]
            self.types.append(t)
        mark = torch.zeros(self.N, dtype=torch.bool, device=DEV)
        for t in self.types:
            mark[t["v"][t["ic"]].reshape(-1)] = True
        self.J = torch.nonzero(mark).reshape(-1)
        self.nX = self.J.numel()
        number = torch.full((self.N,), -1, dtype=torch.int64, device=DEV)
        number[self.J] = torch.arange(self.nX, device=DEV)
        d0 = torch.zeros(self.nX, dtype=F64, device=DEV)
        for t in self.types:
            g, vc, Lc = t["g"], t["v"][t["ic"]], t["L"]
            t["xc"] = number[vc]
            t["vc"] = vc
            t["sides"] = []
            for sg, key in ((1.0, "pos"), (-1.0, "neg")):
                M = _moments(sg * Lc)
                w = Lc.abs() - sg * Lc
                G = w @ g
                t["sides"].append((M, w, G, t[key][t["ic"]]))
                d = (g * g).sum(1)[None] * torch.einsum("mc,md,mcd->m", w, w, M)[:, None]
                d = d + 2.0 * (G @ g.T) * torch.einsum("mc,mca->ma", w, M)
                d = d + (G * G).sum(1)[:, None] * M.diagonal(dim1=1, dim2=2)
                d0.index_add_(0, t["xc"].reshape(-1), d.reshape(-1))
        self.s = d0.rsqrt()

    def strains(self, u, q, eb):
        """Per type: strain of the uncut elements and, per side, of the cut elements' four vertices."""
        for t in self.types:
            g = t["g"]
            H = torch.einsum("mai,ap->mip", u[t["vu"]], g)
            eu = 0.5 * (H + H.transpose(1, 2)) + eb
            ec = []
            if t["ic"].numel():
                H = torch.einsum("mai,ap->mip", u[t["vc"]], g)
                qv = (q * self.s[:, None])[t["xc"]]
                Hq = torch.einsum("mai,ap->mip", qv, g)
                for M, w, G, m in t["sides"]:
                    K = H[:, None] + w[:, :, None, None] * Hq[:, None] + qv[:, :, :, None] * G[:, None, None, :]
                    ec.append(0.5 * (K + K.transpose(2, 3)) + eb)
            yield t, eu, ec

    def apply(self, u, q, eb, stress=False):
        """Residual forces (FE, scaled enriched), volume integral of the stress, voxel stresses."""
        f, fe = torch.zeros_like(u), torch.zeros_like(q)
        total = torch.zeros((3, 3), dtype=F64, device=DEV)
        vox = torch.zeros((self.N, 3, 3), dtype=F64, device=DEV) if stress else None
        lam, mu = self.lame[:, 0], self.lame[:, 1]
        for t, eu, ec in self.strains(u, q, eb):
            g = t["g"]
            s = _hooke(eu, lam[t["mu"]], mu[t["mu"]]) / 6.0
            f.index_add_(0, t["vu"].reshape(-1), torch.einsum("mip,ap->mai", s, g).reshape(-1, 3))
            total += s.sum(0)
            if stress:
                vox.index_add_(0, t["iu"], s)
            for (M, w, G, m), e in zip(t["sides"], ec):
                S = torch.einsum("mcd,mcij->mdij", M, _hooke(e, lam[m][:, None], mu[m][:, None]))
                St, Sw = S.sum(1), torch.einsum("md,mdij->mij", w, S)
                f.index_add_(0, t["vc"].reshape(-1), torch.einsum("mip,ap->mai", St, g).reshape(-1, 3))
                F = torch.einsum("mip,ap->mai", Sw, g) + torch.einsum("maip,mp->mai", S, G)
                F = F * self.s[t["xc"]][:, :, None]
                fe.index_add_(0, t["xc"].reshape(-1), F.reshape(-1, 3))
                total += St.sum(0)
                if stress:
                    vox.index_add_(0, t["ic"], St)
        return f, fe, total, vox

    def symbol(self):
        """Inverse of the multiplier of int grad^s u : grad^s v, zero at the zero frequency."""
        n = self.n
        cols = []
        for c in range(3):
            u = torch.zeros((self.N, 3), dtype=F64, device=DEV)
            u[0, c] = 1.0
            f = torch.zeros_like(u)
            for t in self.types:
                H = torch.einsum("mai,ap->mip", u[t["v"]], t["g"])
                e = 0.5 * (H + H.transpose(1, 2)) / 6.0
                f.index_add_(0, t["v"].reshape(-1), torch.einsum("mip,ap->mai", e, t["g"]).reshape(-1, 3))
            cols.append(torch.fft.fftn(f.reshape(n[2], n[1], n[0], 3), dim=(0, 1, 2)).reshape(-1, 3))
        S = torch.stack(cols, dim=2)
        S[0] = torch.eye(3, dtype=S.dtype, device=DEV)
        # a 3 x 3 inverse by its adjugate
        r = [S[:, i] for i in range(3)]
        adj = torch.stack([torch.linalg.cross(r[1], r[2]), torch.linalg.cross(r[2], r[0]),
                           torch.linalg.cross(r[0], r[1])], dim=2)
        inv = adj / (r[0] * adj[:, :, 0]).sum(1)[:, None, None]
        inv[0] = 0
        return inv

    def solve(self, loads):
        n, inv = self.n, self.symbol()

        def precond(f):
            F = torch.fft.fftn(f.reshape(n[2], n[1], n[0], 3), dim=(0, 1, 2)).reshape(-1, 3, 1)
            return torch.fft.ifftn((inv @ F).reshape(n[2], n[1], n[0], 3), dim=(0, 1, 2)).real.reshape(-1, 3)

        out = []
        zero = torch.zeros((3, 3), dtype=F64, device=DEV)
        for eb in loads:
            E = _tensor(torch.tensor(eb, dtype=F64, device=DEV))
            u = torch.zeros((self.N, 3), dtype=F64, device=DEV)
            q = torch.zeros((self.nX, 3), dtype=F64, device=DEV)
            f, fe, _, _ = self.apply(u, q, E)
            f, fe = -f, -fe
            y = precond(f)
            d, de = y.clone(), fe.clone()
            r2 = float((f * y).sum() + (fe * fe).sum())
            first = r2
            for _ in range(3000):
                if r2 <= 1e-28 * first or r2 == 0.0:
                    break
                z, ze, _, _ = self.apply(d, de, zero)
                a = r2 / float((z * d).sum() + (ze * de).sum())
                u += a * d
                q += a * de
                f -= a * z
                fe -= a * ze
                y = precond(f)
                new = float((f * y).sum() + (fe * fe).sum())
                d = y + (new / r2) * d
                de = fe + (new / r2) * de
                r2 = new
            _, _, total, vox = self.apply(u, q, E, True)
            out.append((E, u, q, _mandel(total / self.N), _mandel(vox)))
        return out

    def gradient(self, solved, W):
        """sum_kl W_kl dC_kl / d(lambda, mu) of every phase, from the six unit-load solutions."""
        W = torch.tensor(W, dtype=F64, device=DEV)
        lam, U = self.lame, [list(self.strains(u, q, E)) for E, u, q, _, _ in solved]
        grad = torch.zeros_like(lam)
        for t in range(6):
            eu = torch.stack([U[k][t][1] for k in range(6)], dim=1)
            tr = eu.diagonal(dim1=-2, dim2=-1).sum(-1)
            parts = [(self.types[t]["mu"], torch.einsum("mk,kl,ml->m", tr, W, tr) / 6.0,
                      torch.einsum("mkij,kl,mlij->m", eu, W, eu) / 3.0)]
            for side in range(len(U[0][t][2])):
                M, _, _, m = self.types[t]["sides"][side]
                e = torch.stack([U[k][t][2][side] for k in range(6)], dim=1)
                tr = e.diagonal(dim1=-2, dim2=-1).sum(-1)
                We = torch.einsum("kl,mlcij->mkcij", W, e)
                parts.append((m, torch.einsum("mkc,mcd,mkd->m", tr, M, We.diagonal(dim1=-2, dim2=-1).sum(-1)),
                              2.0 * torch.einsum("mkcij,mcd,mkdij->m", e, M, We)))
            for m, gl, gm in parts:
                grad[:, 0].index_add_(0, m, gl / self.N)
                grad[:, 1].index_add_(0, m, gm / self.N)
        return grad


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        cells = _cells_of_batch(case, seed)
    else:
        cells = [(_size(case), _cell_of(case, seed))]
    if kind == "operator":
        R = _Reference(*cells[0], case["discretization"])
        x = _state_vector(seed, 3 * (R.N + R.nX))
        u, q = x[:3 * R.N].reshape(3, R.N).T, x[3 * R.N:].reshape(3, R.nX).T
        E = _tensor(torch.tensor(_strains(seed, 1)[0], device=DEV)) if case["macro"] else \
            torch.zeros((3, 3), dtype=F64, device=DEV)
        f, fe, total, _ = R.apply(u.contiguous(), q.contiguous(), E)
        y = torch.cat([f.T.reshape(-1), fe.T.reshape(-1)])
        return dict(y=y, avg=_mandel(total / R.N)) if case["macro"] else dict(y=y)
    loads = _strains(seed, case["loads"] if kind == "fields" else 1) if kind in ("fields", "stress") else np.eye(6)
    its = 80.0 * math.sqrt(max(case["contrast"], 10.0) / 10.0)
    if sum(n[0] * n[1] * n[2] for n, _ in cells) * len(loads) * its > COST:
        return None
    out = []
    for n, cell in cells:
        R = _Reference(n, cell, case["discretization"])
        S = R.solve(loads)
        C = torch.stack([s[3] for s in S], dim=1)
        if kind == "fields":
            return dict(disp=torch.stack([s[1].T for s in S]), avg=torch.stack([s[3] for s in S]))
        if kind == "stress":
            return dict(disp=torch.stack([s[1].T for s in S]), stress=torch.stack([s[4].T for s in S]),
                        avg=torch.stack([s[3] for s in S]))
        if kind == "gradient":
            return dict(c_eff=C, grad=R.gradient(S, _weights(seed)))
        out.append(C)
    return torch.stack(out) if kind == "batch" else out[0]
