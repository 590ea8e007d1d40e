"""Kernel variants at the sizes where they can go wrong: edges of their blocks and
tiles, remainders, degenerate entries (GPU)."""
import numpy as np
import pytest

import synth
from gpu_util import rel, say
from oracle import krylov, sign

pytestmark = pytest.mark.gpu

MW = -1.5


@pytest.mark.parametrize("kind", ["random", "ties"])
@pytest.mark.parametrize("k", [1, 2, 15, 16, 17, 18, 63, 64, 65, 66, 80, 128, 129, 130, 193])
def test_inner_sign_tridiag_block_edges(kind, k):
    """sgn(G) e_1 (eq. 1.3) at sizes around the 64-step blocks of the elimination
    and the 16-row blocks of the way back, against the oracle's spectral sign.
    ties: zero diagonal with alternating couplings 1 and 0.4 (even sizes; an odd
    one has a zero eigenvalue), so that the pivot test compares equal moduli at
    the node tau = 1 and meets exact zeros.  The accepted coarse/fine difference
    (3e-7) bounds the coarse rule's error, hence 6e-7."""
    import paper_0810_4228_amd as ovs
    rng = np.random.default_rng(100 + k)
    if kind == "ties":
        if k % 2:
            pytest.skip("odd chains have a zero eigenvalue")
        diag = np.zeros(k, complex)
        c = np.where(np.arange(k) % 2 == 0, 1.0, 0.4)
        sub, sup = c.astype(complex), c.astype(complex)
    else:
        diag = rng.choice([-1.0, 1.0], k) * (1 + 0.3 * rng.random(k)) + 0.2j * rng.standard_normal(k)
        sub = (0.05 + 0.1 * rng.random(k)).astype(complex)
        sup = 0.1 * (rng.standard_normal(k) + 1j * rng.standard_normal(k))
    G = krylov.tridiag(diag, sub[:k - 1].real, sup[:k - 1])
    lat = ovs.Lattice((2, 2, 2, 2))
    x, err, st = lat.inner_sign_tridiag(diag[None], sub[None], sup[None], return_status=True)
    e = rel(x[0], sign.sign_e1(G))
    say(f"inner sign {kind} k={k}: {e:.2e}, estimate {err[0]:.1e}, status {st}")
    assert st == 0
    assert e <= 6e-7


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (3, 2, 5, 4), (4, 4, 4, 4), (5, 3, 7, 3),
                                  (16, 16, 2, 8), (12, 10, 9, 8)])
@pytest.mark.parametrize("nrhs", [1, 3])
def test_one_wave_per_hop_equals_thread_per_site(prec, dims, nrhs):
    """Launches without a set configuration and few sites run one wave per hop;
    the same calls with the one-thread-per-site forms set give the same bits:
    all four operators, and a fixed-k two-sided Lanczos solve (its alpha sums
    the quarters of each 256-site tile, its coefficients follow).  Sizes below,
    at and beyond the 64-site workgroups and 256-site tiles, with remainders,
    and planar tiles (Lx Ly = 256); (12, 10, 9, 8) x 3 exceeds the FP32 limit of
    the operator pair, which then differs from the single operator's form."""
    import torch
    import paper_0810_4228_amd as ovs
    from gpu_util import to_dev
    U = to_dev(synth.random_links(dims, 0.5, seed=41))
    b = to_dev(synth.gaussian_sources(dims, nrhs, seed=42))
    k = min(30, 6 * int(np.prod(dims)))
    out = []
    for cfg in (None, [110, 256, 0, 0, 110, 256, 0, 0]):
        lat = ovs.Lattice(dims, precision=prec)
        lat.set_links(U)
        lat.set_params(MW, 0.3)
        if cfg:
            lat.set_tuning_raw(nrhs, cfg)
        res = [lat.apply(op, b).cpu() for op in ("Dw", "Dw_dag", "A", "A_dag")]
        res.append(lat.sign_apply(b, k)[0].cpu())
        res += [torch.from_numpy(c) for c in lat.last_coefficients(nrhs, k)]
        out.append(res)
        lat.close()
    for x, y in zip(*out):
        assert torch.equal(x, y)


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(2, 2, 2, 2), (3, 2, 5, 4), (5, 3, 7, 3), (12, 10, 9, 8)])
@pytest.mark.parametrize("nrhs", [1, 2, 5])
def test_canonical_apply_forms_agree(prec, dims, nrhs):
    """apply() on canonical tensors gives the same bits by one wave per hop (reads
    and writes them itself), by the staged form (converts the input, writes the
    canonical result, tiles with remainders), by the unstaged one (converts both)
    and by the resident fields' import, application and export; also when the
    output overlaps the input, where the input has to be converted first."""
    import torch
    import paper_0810_4228_amd as ovs
    from gpu_util import to_dev
    U = to_dev(synth.random_links(dims, 0.5, seed=43))
    b = to_dev(synth.gaussian_sources(dims, nrhs, seed=44))
    lat = ovs.Lattice(dims, precision=prec)
    lat.set_links(U)
    lat.set_params(MW, 0.3)
    f, g = lat.field_create(nrhs), lat.field_create(nrhs)
    ref = {}
    for op in ("Dw", "Dw_dag", "A", "A_dag"):
        f.import_(b)
        f.apply(op, g)
        ref[op] = g.export().reshape(b.shape)
        assert torch.equal(lat.apply(op, b), ref[op])
        buf = torch.cat([b.reshape(-1), b.reshape(-1)[:1]])
        n = b.numel()
        lat.apply(op, buf[:n].reshape(b.shape), out=buf[1:].reshape(b.shape))
        assert torch.equal(buf[1:].reshape(b.shape), ref[op])
    for shape in (1110, 110):
        lat.set_tuning_raw(nrhs, [shape, 256, 0, 0, 110, 256, 0, 0])
        for op in ref:
            assert torch.equal(lat.apply(op, b), ref[op])
    f.close()
    g.close()
    lat.close()


@pytest.mark.parametrize("dims,m,tol", [((3, 2, 5, 7), 3, 1e-8), ((4, 4, 8, 8), 2, 1e-8),
                                        ((24, 24, 16, 12), 4, 1e-3)])
def test_eigentriples_both_forms_of_the_inner_solves(dims, m, tol):
    """The deflation eigensolver's inner solves run their stencils with one wave per
    hop up to 1e5 sites (directions formed in the stencil, norms beside it;
    a last workgroup of 18 lanes, and full ones) and in separate launches beyond:
    right and left residuals of the triples, by the operator itself, within the
    requested tolerance (twice it: residuals are relative to |lambda|, whose own
    relative error is below the tolerance)."""
    import torch
    import paper_0810_4228_amd as ovs
    from gpu_util import to_dev
    lat = ovs.Lattice(dims, precision="f64")
    lat.set_links(to_dev(synth.random_links(dims, 0.3, seed=43)))
    lat.set_params(MW, 0.1)
    d, st = lat.deflation_compute(m, tol=tol, max_iter=60)
    lam, R, L, info = d.get()
    assert st == 0
    lam = torch.as_tensor(np.asarray(lam), device=R.device)
    rr = (lat.apply("A", R) - lam[:, None] * R).norm(dim=1) / (lam.abs() * R.norm(dim=1))
    rl = (lat.apply("A_dag", L) - lam.conj()[:, None] * L).norm(dim=1) / (lam.abs() * L.norm(dim=1))
    say(f"eigentriples {dims} m={m}: residuals {float(rr.max()):.1e} {float(rl.max()):.1e}, info {info}")
    assert float(rr.max()) <= 2 * tol and float(rl.max()) <= 2 * tol
    d.close()
    lat.close()


@pytest.mark.parametrize("k", [1, 2, 8, 9, 16, 17, 32, 33, 49])
def test_arnoldi_vector_groups(k):
    """Arnoldi at sizes around the groups of 8 vectors of the dots and of 16 (two in
    turn) of the subtraction, on a field whose last workgroup has a remainder (12 x
    274 entries), two sources, against the oracle: sgn(H) e_1 is accepted at a
    coarse/fine difference quad_err, which bounds the coarse rule's error, and
    orthogonalised twice both bases agree to rounding, hence 2 quad_err + 1e-10."""
    import paper_0810_4228_amd as ovs
    from gpu_util import to_dev
    from oracle import dirac
    dims = (3, 2, 5, 7)
    U = synth.random_links(dims, 0.5, seed=51)
    A = dirac.csr_A(dims, U, MW, 0.3)
    b = synth.gaussian_sources(dims, 2, seed=52)
    lat = ovs.Lattice(dims, precision="f64")
    lat.set_links(to_dev(U))
    lat.set_params(MW, 0.3)
    y, info, st = lat.sign_apply(to_dev(b), k, method="arnoldi")
    for r in range(2):
        e = rel(y.cpu().numpy()[r], krylov.arnoldi_apply(lambda v: A @ v, b[r], k))
        say(f"arnoldi k={k} source {r}: {e:.1e}, quad_err {info[r]['quad_err']:.1e}")
        assert info[r]["k_used"] == k
        assert e <= 2 * info[r]["quad_err"] + 1e-10
    lat.close()


@pytest.mark.parametrize("k", [1, 3, 4, 5, 6, 7, 11, 12, 13, 14, 64, 67, 68, 69, 70, 72, 129])
def test_inner_sign_tridiag_batch_of_steps(k):
    """sgn(T) e_1 by trailing minors, at every residue of k mod 8 (the groups of
    minors that share an exponent and the start of the row blocks), for a batch of
    eight whose matrices end at quadrature steps from 1/4 to 1/64: entries of the
    first row turned to angles d from the imaginary axis, where the difference of the
    rules with steps h and 2 h is about 2 exp(-pi d / h).  The batch runs in several
    launches that share their scratch, with rounds in which some matrices are done;
    every row equals its batch of one (one launch a round) bit for bit.  The accepted
    rule's error is of the order of the squared difference; what remains is rounding:
    the weighted sums (some 7e-14), the minors and the oracle's eigenvectors (each
    some k eps), over the distance d of the nodes from the spectrum: 1e-12 / d."""
    import paper_0810_4228_amd as ovs
    rng = np.random.default_rng(300 + k)
    angle = np.array([1.5, 0.8, 0.4, 0.2, 0.1, 1.5, 0.2, 0.4])
    n = len(angle)
    diag = rng.choice([-1.0, 1.0], (n, k)) * (1 + 0.3 * rng.random((n, k))) \
        + 0.05j * rng.standard_normal((n, k))
    diag[:, 0] = np.exp(1j * (np.pi / 2 - angle))
    sub = (0.05 + 0.05 * rng.random((n, k))).astype(complex)
    sup = 0.03 * (rng.standard_normal((n, k)) + 1j * rng.standard_normal((n, k)))
    lat = ovs.Lattice((2, 2, 2, 2))
    x, err, st = lat.inner_sign_tridiag(diag, sub, sup, return_status=True)
    assert st == 0
    for r in range(n):
        one, err1 = lat.inner_sign_tridiag(diag[r], sub[r], sup[r])
        e = rel(x[r], sign.sign_e1(krylov.tridiag(diag[r], sub[r, :k - 1].real, sup[r, :k - 1])))
        say(f"inner sign k={k} angle {angle[r]}: {e:.1e}, estimate {err[r]:.1e}")
        assert np.array_equal(x[r], one[0]) and err[r] == err1[0]
        assert e <= 10 * err[r] ** 2 + 1e-12 / angle[r]
    lat.close()
