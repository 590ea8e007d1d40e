"""Timed workloads of the library, each one pass through its public entry points.

A case names a lattice, a storage precision, a number of sources and one kind
of call:

    apply      Lattice.apply on canonical tensors (layout conversion included)
    resident   A^dagger A applied repeatedly to a field held in the library's
               layout, imported once and exported at the end
    sign       Lattice.sign_apply: sgn(A) b or D_ov b, two-sided Lanczos or Arnoldi
    vjp        Lattice.sign_apply_vjp: result and gradients in b, mu and the links
    autograd   sign_autograd forward and backward, links set on every step
    eig        Lattice.deflation_compute: critical eigentriples

Inputs are seeded: links P_SU3(1 + eps G), complex Gaussian sources.  exact()
gives the same outputs in plain torch at 64 bits where that is affordable.
"""
import json
import math
import os

import numpy as np
import torch

import paper_0810_4228_amd as ovs

MW = -1.5
BC = (1, 1, 1, -1)


def _case(name, kind, dims, precision, nrhs, mu, eps, **options):
    c = {"kind": kind, "lx": dims[0], "ly": dims[1], "lz": dims[2], "lt": dims[3],
         "precision": precision, "nrhs": nrhs, "mu": mu, "eps": eps}
    c.update(options)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: one source on the smallest lattice of the tests;
        # a Python-driven solver or a test makes thousands of these.
        _case("apply_4444_f64_x1", "apply", (4, 4, 4, 4), "f64", 1, 0.3, 0.6, op="Dw"),
        # The operator on tensors at production size, 12 spin-colour sources.
        _case("apply_16x16x16x32_f32_x12", "apply", (16, 16, 16, 32), "f32", 12, 0.4, 0.6,
              op="A"),
        # The same size with the fields kept in the library's layout: a normal-
        # equation or polynomial iteration, where the stencil alone counts.
        _case("resident_16x16x16x32_f32_x12", "resident", (16, 16, 16, 32), "f32", 12, 0.4, 0.6,
              pairs=4),
        # A small deflated solve: 4^4 with eigentriples at hand (quenched
        # studies at this size solve for every source of every configuration).
        _case("sign_4444_f64_x1_deflated", "sign", (4, 4, 4, 4), "f64", 1, 0.3, 0.6, kmax=600,
              tol=1e-8, defl=12),
        # One FP64 source at 8^4 to a tight tolerance, graph replay: the inner
        # solve of an eigenvalue or propagator computation.
        _case("sign_8888_f64_x1_graph", "sign", (8, 8, 8, 8), "f64", 1, 0.3, 0.6, kmax=1000,
              tol=1e-10, graph=True),
        # The overlap operator on five sources of an uneven lattice (plane of
        # 36 sites, no power of two), single precision storage.
        _case("overlap_6x6x10x14_f32_x5", "sign", (6, 6, 10, 14), "f32", 5, 0.2, 0.5, kmax=800,
              tol=1e-5, graph=True, overlap=True),
        # The production solve: 12 sources, 16^3 x 32, FP32 storage, 1e-5.
        _case("sign_16x16x16x32_f32_x12_graph", "sign", (16, 16, 16, 32), "f32", 12, 0.4, 0.6,
              kmax=512, tol=1e-5, graph=True),
        # Two-pass solve (short of memory for the basis) with tolerances on
        # both sides of what FP32 storage holds: an FP32 and an FP64 group.
        _case("sign_16x16x16x16_mixed_x4_twopass", "sign", (16, 16, 16, 16), "f32", 4, 0.2, 0.6,
              kmax=800, tol=1e-5, tol_odd=1e-8, two_pass=True),
        # The comparison method at a fixed number of steps.
        _case("arnoldi_8888_f64_x1", "sign", (8, 8, 8, 8), "f64", 1, 0.3, 0.6, kmax=200,
              method="arnoldi"),
        # Gradients of a fixed-k solve: one source at 8^4, recomputed vectors.
        _case("vjp_8888_f64_x1", "vjp", (8, 8, 8, 8), "f64", 1, 0.3, 0.6, k=200),
        # A step of a force or optimisation program at 16^4 through autograd:
        # links set, forward, backward.
        _case("autograd_16x16x16x16_f64_x1", "autograd", (16, 16, 16, 16), "f64", 1, 0.3, 0.6,
              k=100),
        # Setup of a deflated campaign: critical eigentriples of one lattice.
        _case("eig_4x4x4x8_f64_m8", "eig", (4, 4, 4, 8), "f64", 1, 0.3, 0.6, m=8, tol=1e-8),
    ]


def _volume(c):
    return c["lx"] * c["ly"] * c["lz"] * c["lt"]


def _log_uniform(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _draw_dims(rng, vmin, vmax):
    """Extents (odd ones among them) whose product is about log-uniform in [vmin, vmax]."""
    while True:
        target = _log_uniform(rng, vmin, vmax)
        d = []
        for left in (4, 3, 2, 1):
            mid = (target / math.prod(d)) ** (1.0 / left)
            e = mid * (math.exp(rng.uniform(-0.5, 0.5)) if left > 1 else 1.0)
            d.append(max(2, min(32, round(e))))
        if vmin <= math.prod(d) <= vmax:
            return tuple(d)


def draw(rng):
    kind = rng.choice(["apply", "apply", "resident", "sign", "sign", "sign", "sign", "arnoldi",
                       "vjp", "vjp", "autograd", "eig"])
    mu = rng.choice([0.0, round(rng.uniform(0.05, 0.4), 2)])
    eps = round(rng.uniform(0.4, 0.6), 2)
    if kind == "apply":
        dims = _draw_dims(rng, 16, 16 ** 3 * 32)
        return _case(None, kind, dims, rng.choice(["f64", "f32"]), rng.randint(1, 12), mu, eps,
                     op=rng.choice(["Dw", "Dw_dag", "A", "A_dag"]))
    if kind == "resident":
        dims = _draw_dims(rng, 256, 16 ** 3 * 32)
        return _case(None, kind, dims, rng.choice(["f64", "f32"]), rng.randint(1, 12), mu, eps,
                     pairs=rng.randint(1, 6))
    if kind == "sign":
        dims = _draw_dims(rng, 256, 16 ** 4)
        v = math.prod(dims)
        precision = rng.choice(["f64", "f32"])
        nrhs = rng.randint(1, max(1, min(12, 4 * 16 ** 4 // v)))
        tol = 10.0 ** (-rng.uniform(4.0, 6.0) if precision == "f32" else -rng.uniform(7.0, 10.0))
        return _case(None, kind, dims, precision, nrhs, mu, eps, kmax=min(700, 6 * v), tol=tol,
                     graph=rng.random() < 0.6, overlap=rng.random() < 0.3,
                     two_pass=rng.random() < 0.2,
                     defl=rng.randint(2, 6) if v <= 512 and rng.random() < 0.5 else 0)
    if kind == "arnoldi":
        dims = _draw_dims(rng, 256, 8192)
        return _case(None, "sign", dims, rng.choice(["f64", "f32"]), rng.randint(1, 3), mu, eps,
                     kmax=rng.randint(40, 200), method="arnoldi")
    if kind in ("vjp", "autograd"):
        dims = _draw_dims(rng, 256, 16 ** 4)
        options = {"k": rng.randint(20, 120)}
        if kind == "vjp":
            options["store"] = rng.random() < 0.4
        return _case(None, kind, dims, "f64", rng.randint(1, 2), mu, eps, **options)
    dims = _draw_dims(rng, 256, 512)
    return _case(None, "eig", dims, "f64", 1, max(mu, 0.1), eps, m=rng.randint(3, 8), tol=1e-8)


# ---- inputs -------------------------------------------------------------------


def _su3_project(m):
    """Unitary polar factor (Newton iteration) over the cube root of its determinant."""
    def cofactors(a):
        r0, r1, r2 = a[..., 0, :], a[..., 1, :], a[..., 2, :]
        return torch.stack([torch.linalg.cross(r1, r2), torch.linalg.cross(r2, r0),
                            torch.linalg.cross(r0, r1)], dim=-2)

    for _ in range(40):
        cof = cofactors(m)
        det = (m[..., 0, :] * cof[..., 0, :]).sum(-1)
        m = 0.5 * (m + (cof / det[..., None, None]).conj())  # inverse^dagger = conj(cof / det)
    det = (m[..., 0, :] * cofactors(m)[..., 0, :]).sum(-1)
    return m * torch.exp(-1j * torch.angle(det) / 3.0)[..., None, None]


def _normal(gen, shape):
    g = torch.randn(*shape, 2, dtype=torch.float64, device="cuda", generator=gen)
    return torch.view_as_complex(g) / math.sqrt(2.0)


def _inputs(c, seed):
    """Links [V, 4, 3, 3], sources [nrhs, 12 V] and, for gradients, cotangents."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    v = _volume(c)
    eye = torch.eye(3, dtype=torch.complex128, device="cuda")
    links = _su3_project(eye + c["eps"] * _normal(gen, (v, 4, 3, 3))).contiguous()
    b = _normal(gen, (c["nrhs"], 12 * v))
    chi = _normal(gen, (c["nrhs"], 12 * v)) if c["kind"] in ("vjp", "autograd") else None
    return links, b, chi


def _saved_tuning(dims, nrhs, precision):
    """The committed kernel configuration of a workload, or None (library defaults)."""
    path = os.path.join(os.path.dirname(ovs.__file__), "tuning_mi355x.json")
    with open(path) as fh:
        return json.load(fh).get("%s-%d-%s" % (tuple(dims), nrhs, precision))


def prepare(case, seed):
    c = case
    dims = (c["lx"], c["ly"], c["lz"], c["lt"])
    links, b, chi = _inputs(c, seed)
    lat = ovs.Lattice(dims, bc=BC, precision=c["precision"])
    lat.set_links(links)
    lat.set_params(MW, c["mu"])
    tuning = _saved_tuning(dims, c["nrhs"], c["precision"])
    if tuning:
        lat.set_tuning_raw(c["nrhs"], tuning)
    s = {"case": c, "lat": lat, "b": b, "chi": chi}
    kind = c["kind"]
    if kind == "apply":
        s["out"] = torch.empty_like(b)
    elif kind == "resident":
        s["fields"] = [lat.field_create(c["nrhs"]) for _ in range(2)]
    elif kind == "sign":
        s["out"] = torch.empty_like(b)
        s["defl"] = lat.deflation_compute(c["defl"], tol=1e-10)[0] if c.get("defl") else None
        if c.get("tol"):
            s["tol"] = [c.get("tol_odd", c["tol"]) if j % 2 else c["tol"]
                        for j in range(c["nrhs"])]
    elif kind == "autograd":
        s["args"] = (b.requires_grad_(), torch.tensor(c["mu"], dtype=torch.float64,
                                                      requires_grad=True),
                     links.requires_grad_())
    torch.cuda.synchronize()
    return s


def run(state):
    s, c, lat = state, state["case"], state["lat"]
    kind = c["kind"]
    if kind == "apply":
        return lat.apply(c["op"], s["b"], out=s["out"])
    if kind == "resident":
        f, g = s["fields"]
        f.import_(s["b"])
        for _ in range(c["pairs"]):
            f.apply("A", g)
            g.apply("A_dag", f)
        return f.export()
    if kind == "sign":
        return lat.sign_apply(s["b"], c["kmax"], defl=s["defl"], tol=s.get("tol"),
                              method=c.get("method", "2sl"), two_pass=c.get("two_pass", False),
                              graph=c.get("graph", False), overlap=c.get("overlap", False),
                              out=s["out"])[0]
    if kind == "vjp":
        y, grad_b, grad_mu, grad_u, _, _ = lat.sign_apply_vjp(s["b"], s["chi"], c["k"],
                                                              store_basis=c.get("store", False))
        return y, grad_b, grad_mu, grad_u
    if kind == "autograd":
        b, mu, links = s["args"]
        y = ovs.sign_autograd(lat, b, mu, links, MW, c["k"])
        return (y.detach(),) + torch.autograd.grad(y, (b, mu, links), grad_outputs=s["chi"])
    d, _ = lat.deflation_compute(c["m"], tol=c["tol"])
    lam, right, left, _ = d.get()
    d.close()
    return lam, right, left


# ---- the work of one pass ---------------------------------------------------------


def _steps(c):
    """Krylov steps of a solve: fixed, or about what its tolerance takes (1e-5: 430
    at eps 0.6, mu 0.4; fewer on smoother links and with eigentriples)."""
    if c["kind"] in ("vjp", "autograd"):
        return c["k"]
    if not c.get("tol"):
        return c["kmax"]
    tight = min(c["tol"], c.get("tol_odd", 1.0))
    k = 85.0 * (-math.log10(tight)) * (c["eps"] / 0.6) ** 2 * (0.6 + c["mu"])
    return int(min(c["kmax"], k * (0.8 if c.get("defl") else 1.0)))


def work(case):
    """A Krylov step reads its two current and two previous vectors once, writes the
    next two and applies the operator pair (1368 flops per site and application);
    the result is one more read of the basis, or a second pass over the recurrence.
    The reverse sweep of a gradient reads and writes as much again and applies the
    pair once more, with the outer products of the link force."""
    c = case
    v, n = _volume(c), c["nrhs"]
    es = 8 if c["precision"] == "f32" else 16
    links = 36.0 * es * v
    field, canon = 12.0 * es * v * n, 12.0 * 16 * v * n
    stencil = 1368.0 * v * n
    io = 2 * canon
    kind = c["kind"]
    if kind == "apply":
        return {"bytes": io + links, "flops": stencil}
    if kind == "resident":
        return {"bytes": io + 2 * c["pairs"] * (links + 2 * field), "flops": 2 * c["pairs"] * stencil}
    axpy = 12.0 * v * n * 8  # one complex multiply-add per entry
    if kind == "eig":
        # shift-invert Krylov on both sides: some 2 (m + 20) solves by CG on the
        # normal equations, about 100 steps of two applications each
        applies = 2.0 * (c["m"] + 20) * 100 * 2
        return {"bytes": applies * (links + 2 * field), "flops": applies * (stencil + 3 * axpy)}
    k = _steps(c)
    if c.get("method") == "arnoldi":
        # orthogonalisation: every earlier vector read for the dots and once more
        # for the subtraction, twice
        return {"bytes": io + k * (links + 3 * field) + 2.0 * k * k * field,
                "flops": k * stencil + 2.0 * k * k * axpy}
    step = {"bytes": links + 6 * field, "flops": 2 * stencil + 10 * axpy}
    if kind == "sign":
        last = field if not c.get("two_pass") else links + 4 * field
        return {"bytes": io + k * (step["bytes"] + last),
                "flops": k * (step["flops"] + axpy + (stencil if c.get("two_pass") else 0))}
    forwards = 2 if kind == "autograd" else 1
    force = 4 * 2 * 2 * 9 * 2 * 8.0 * v * n
    return {"bytes": 3 * io + 36 * 16.0 * v + k * (forwards + 1) * step["bytes"],
            "flops": k * ((forwards + 1) * step["flops"] + force)}


# ---- the same in plain torch -------------------------------------------------------


def _gammas():
    s = [[[0, 1], [1, 0]], [[0, -1j], [1j, 0]], [[1, 0], [0, -1]]]
    z, one = np.zeros((2, 2)), np.eye(2)
    g = [np.block([[z, -1j * np.array(a)], [1j * np.array(a), z]]) for a in s]
    return g + [np.block([[z, one], [one, z]])]


class _Plain:
    """The Wilson operator at chemical potential by rolls of whole fields."""

    def __init__(self, c, links):
        self.shape = (c["lt"], c["lz"], c["ly"], c["lx"])
        u = links.reshape(self.shape + (4, 3, 3)).clone()
        u[-1, ..., 3, :, :] *= BC[3]
        self.u = [u[..., nu, :, :].contiguous() for nu in range(4)]
        self.proj = [[torch.tensor(np.eye(4) + sg * g, dtype=torch.complex128, device="cuda")
                      for sg in (1, -1)] for g in _gammas()]
        self.kappa = 1.0 / (8.0 + 2.0 * MW)
        self.mu = c["mu"]

    @staticmethod
    def _spin(p, psi):
        return (p[:, :, None] * psi[..., None, :, :]).sum(-2)

    @staticmethod
    def _colour(u, psi):
        return (u[..., None, :, :] * psi[..., :, None, :]).sum(-1)

    def _dw(self, psi, mu):
        out = psi.clone()
        for nu in range(4):
            ax = 3 - nu
            fwd, bwd = (math.exp(mu), math.exp(-mu)) if nu == 3 else (1.0, 1.0)
            u = self.u[nu]
            out -= self.kappa * fwd * torch.roll(
                self._colour(u, self._spin(self.proj[nu][0], psi)), 1, ax)
            out -= self.kappa * bwd * self._colour(
                u.conj().transpose(-1, -2), self._spin(self.proj[nu][1], torch.roll(psi, -1, ax)))
        return out

    def apply(self, op, x):
        """op on one flat source."""
        psi = x.reshape(self.shape + (4, 3))
        if op == "Dw_dag":
            psi = self.g5(psi)
        psi = self._dw(psi, -self.mu if op.endswith("_dag") else self.mu)
        return (psi if op == "Dw" else self.g5(psi)).reshape(-1)

    @staticmethod
    def g5(psi):
        out = psi.clone()
        out[..., 2:, :] *= -1
        return out


def _sign_first_column(h):
    """sgn(h) e_1 by Newton's iteration with determinant scaling."""
    x, n = h, h.shape[0]
    for _ in range(60):
        inv = np.linalg.inv(x)
        scale = math.exp(-np.linalg.slogdet(x)[1] / n)
        new = 0.5 * (scale * x + inv / scale)
        done = np.linalg.norm(new - x) <= 1e-14 * np.linalg.norm(new)
        x = new
        if done:
            break
    return x[:, 0]


def _krylov_sign(op, b, k):
    """|b| V sgn(V^dagger A V) e_1 on the fully orthogonalised Krylov space of size k."""
    basis = torch.empty(k, b.numel(), dtype=torch.complex128, device="cuda")
    h = torch.zeros(k, k, dtype=torch.complex128, device="cuda")
    norm = torch.linalg.vector_norm(b)
    basis[0] = b / norm
    for j in range(k):
        w = op(basis[j])
        for _ in range(2):
            dots = torch.mv(basis[:j + 1], w.conj()).conj()
            w = w - torch.mv(basis[:j + 1].t(), dots)
            h[:j + 1, j] += dots
        if j + 1 < k:
            h[j + 1, j] = torch.linalg.vector_norm(w)
            basis[j + 1] = w / h[j + 1, j]
    x = torch.from_numpy(_sign_first_column(h.cpu().numpy())).to("cuda")
    return norm * torch.mv(basis.t(), x)


def exact(case, seed):
    c = case
    kind = c["kind"]
    if kind not in ("apply", "resident", "sign"):
        return None
    arnoldi = c.get("method") == "arnoldi"
    if kind == "sign":
        k = c["kmax"] if arnoldi else (500 if c["tol"] >= 1e-6 else 900)
        if 12 * _volume(c) < 2 * k:
            return None
        if _volume(c) * c["nrhs"] > 40000 or c["nrhs"] * (k / 900.0) ** 3 > 1.2:
            return None  # over about 20 seconds
    links, b, _ = _inputs(c, seed)
    op = _Plain(c, links)
    if kind == "apply":
        return torch.stack([op.apply(c["op"], x) for x in b])
    if kind == "resident":
        out = []
        for x in b:
            for _ in range(c["pairs"]):
                x = op.apply("A_dag", op.apply("A", x))
            out.append(x)
        return torch.stack(out)
    out = torch.empty_like(b)
    for r in range(c["nrhs"]):
        y = _krylov_sign(lambda x: op.apply("A", x), b[r], k)
        if c.get("overlap"):
            y = b[r] + op.g5(y.reshape(op.shape + (4, 3))).reshape(-1)
        out[r] = y
    return out
