"""Calls whose kernels or buffers are chosen by size, tuning or workspace: every
route is open to the calls that the interface admits, with the same results (GPU)."""
import pytest

import synth
from gpu_util import rel_rows, say, to_dev

pytestmark = pytest.mark.gpu

MW = -1.5


def lattice(dims, prec, U, mu):
    import paper_0810_4228_amd as ovs
    lat = ovs.Lattice(dims, precision=prec)
    lat.set_links(to_dev(U))
    lat.set_params(MW, mu)
    return lat


@pytest.mark.parametrize("two_pass", [False, True])
@pytest.mark.parametrize("nrhs,tight", [(12, 1), (12, 2), (12, 4), (6, 1), (6, 2), (6, 3), (7, 2)])
def test_workspace_of_the_batch_serves_its_fp32_group(nrhs, tight, two_pass):
    """A caller workspace of exactly ovs_workspace_size bytes for the batch: on an
    FP32-storage lattice the group of sources above the FP32 floor runs in it, a
    smaller batch (halves of 5, groups of 3 to 5) whose buffers may not need more
    than the batch's.  Results as on the handle's own memory, bit for bit."""
    import torch
    dims, k = (4, 4, 4, 4), 200
    lat = lattice(dims, "f32", synth.random_links(dims, 0.5, seed=61), 0.3)
    b = to_dev(synth.gaussian_sources(dims, nrhs, seed=62))
    tol = [1e-8] * tight + [1e-4] * (nrhs - tight)
    n = lat.workspace_size(nrhs, k, two_pass=two_pass)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    y, info, st = lat.sign_apply(b, k, tol=tol, two_pass=two_pass, workspace=ws)
    y2, info2, st2 = lat.sign_apply(b, k, tol=tol, two_pass=two_pass)
    say("workspace", nrhs, tight, two_pass, n, st, [i["k_used"] for i in info])
    assert st == st2 and torch.equal(y, y2)
    assert [i["k_used"] for i in info] == [i["k_used"] for i in info2]
    lat.close()


@pytest.mark.parametrize("method,two_pass", [("2sl", False), ("2sl", True), ("arnoldi", False)])
@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_workspace_size_grows_with_the_batch(prec, method, two_pass):
    """ovs_workspace_size does not decrease with the number of sources (batches from
    8 on are two halves), so a workspace sized for a batch holds any part of it."""
    import paper_0810_4228_amd as ovs
    for dims in ((2, 2, 2, 2), (4, 4, 4, 8), (12, 12, 12, 12)):
        lat = ovs.Lattice(dims, precision=prec)
        n = [lat.workspace_size(r, 100, method=method, two_pass=two_pass) for r in range(1, 25)]
        say("workspace sizes", prec, dims, method, two_pass, n[0], n[4], n[5], n[-1])
        assert n == sorted(n)
        lat.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims,nrhs,hops,dual_hops", [
    ((2, 2, 2, 2), 1, True, True), ((4, 4, 6, 6), 3, True, True), ((8, 8, 8, 8), 12, True, True),
    ((12, 12, 12, 12), 5, False, "f64"), ((16, 16, 16, 16), 4, False, False)])
def test_tuning_saved_and_installed_again(prec, dims, nrhs, hops, dual_hops):
    """get_tuning_raw without a set configuration reports the default that runs, one
    wave per hop among them (lanes per site 0, variant 7; batches from 8 on: the
    operator pair of a half), and set_tuning_raw installs it: get, set, get is the
    identity and a solve equals the untuned one bit for bit."""
    import torch
    U = synth.random_links(dims, 0.5, seed=63)
    lat, other = lattice(dims, prec, U, 0.3), lattice(dims, prec, U, 0.3)
    raw = lat.get_tuning_raw(nrhs)
    ex = lat.get_tuning_ex(nrhs)
    say("tuning", prec, dims, nrhs, raw, ex)
    assert (ex["stencil"]["lanes_per_site"] == 0) == hops
    assert (ex["dual"]["variant"] == "one wave per hop") == (dual_hops in (True, prec))
    other.set_tuning_raw(nrhs, raw)
    assert other.get_tuning_raw(nrhs) == raw
    b = to_dev(synth.gaussian_sources(dims, nrhs, seed=64))
    k = 20
    assert torch.equal(lat.apply("A", b), other.apply("A", b))
    assert torch.equal(lat.sign_apply(b, k)[0], other.sign_apply(b, k)[0])
    lat.close()
    other.close()


def test_tuning_of_one_wave_per_hop():
    """What the autotuner chose on a small lattice installs on another handle; set
    for a larger lattice one wave per hop gives the bits of the default forms (FP64
    sums of the operator pair by quarters of a tile, in the same order); fields it
    has no use for are refused."""
    import torch
    import paper_0810_4228_amd as ovs
    U = synth.random_links((4, 4, 4, 4), 0.5, seed=65)
    lat, other = lattice((4, 4, 4, 4), "f64", U, 0.2), lattice((4, 4, 4, 4), "f64", U, 0.2)
    lat.autotune(2)
    raw = lat.get_tuning_raw(2)
    say("autotuned", raw)
    other.set_tuning_raw(2, raw)
    assert other.get_tuning_raw(2) == raw
    good = [100, 64, 0, 0, 172, 512, 0, 0]
    other.set_tuning_raw(2, good)
    assert other.get_tuning_raw(2) == good
    for at, value in ((0, 200), (0, 101), (0, 1100), (1, 256), (2, 40), (3, 1), (4, 272), (4, 171),
                      (4, 180), (4, 102), (6, 40), (7, 2)):
        bad = list(good)
        bad[at] = value
        with pytest.raises(ovs.OvsError) as e:
            other.set_tuning_raw(2, bad)
        assert e.value.status == ovs.OVS_ERR_ARG, bad
        assert other.get_tuning_raw(2) == good
    lat.close()
    other.close()
    for prec in ("f64", "f32"):
        dims = (16, 16, 16, 16)
        U = synth.random_links(dims, 0.5, seed=66)
        b = to_dev(synth.gaussian_sources(dims, 3, seed=67))
        lat, other = lattice(dims, prec, U, 0.2), lattice(dims, prec, U, 0.2)
        other.set_tuning_raw(3, [100, 64, 0, 0, 170, 512, 0, 0])
        for method in ({}, {"two_pass": True}, {"graph": True}, {"persistent": True}):
            assert torch.equal(lat.sign_apply(b, 12, **method)[0], other.sign_apply(b, 12, **method)[0])
        assert torch.equal(lat.apply("A", b), other.apply("A", b))
        lat.close()
        other.close()


def configurations(prec, nrhs):
    """(shape, workgroup, order) of the stencil configurations the autotuner can pick."""
    shapes = [(blk, 1, st) for blk in ((1, 2, 3, 4, 6) if prec == "f32" else (1, 2, 3))
              for st in (0, 1) if st == 0 or blk <= (4 if prec == "f32" else 2)]
    shapes += [(1, g, 0) for g in (2, 4, 8)]
    for blk, g, st in shapes:
        for wg in (64, 128, 256):
            for order in range(8):
                for nt in (0, 1):
                    yield 1000 * st + 100 * blk + 10 * g + nt, wg, order


@pytest.mark.parametrize("prec", ["f64", "f32"])
@pytest.mark.parametrize("dims", [(4, 4, 6, 6), (16, 16, 2, 8), (8, 8, 4, 8)])
def test_every_configuration_on_resident_fields(prec, dims):
    """Every stencil configuration through import, apply and export, and through
    apply on tensors: 1e-14 (FP64) and 1e-6 (FP32 storage) of the oracle for the
    first of each shape, and the same bits by all others and by both routes.  A
    ragged lattice, and planar ones for 256- and 64-site tiles with Lt = 8 (grouped
    block orders), 7 sources (ragged source blocks and windows)."""
    import torch
    from oracle import dirac
    U = synth.random_links(dims, 0.6, seed=68)
    b = synth.gaussian_sources(dims, 7, seed=69)
    lat = lattice(dims, prec, U, 0.3)
    bt = to_dev(b)
    f, g = lat.field_create(7), lat.field_create(7)
    f.import_(bt)
    base = lat.get_tuning_raw(7)
    for op in ("A", "Dw_dag"):
        m = dirac.csr_A(dims, U, MW, 0.3) if op == "A" else dirac.csr_dw(dims, U, MW, 0.3)
        ref = ((m if op == "A" else m.conj().T.tocsr()) @ b.T).T
        first, n = None, 0
        for cfg in configurations(prec, 7):
            lat.set_tuning_raw(7, [cfg[0], cfg[1], 0, cfg[2]] + base[4:])
            f.apply(op, g)
            y = g.export().reshape(bt.shape)
            if first is None:
                first = y
                assert rel_rows(y.cpu().numpy(), ref) <= (1e-14 if prec == "f64" else 1e-6)
            assert torch.equal(y, first), (op, cfg)
            assert torch.equal(lat.apply(op, bt), first), (op, cfg)
            n += 1
        say("resident configurations", prec, dims, op, n)
    f.close()
    g.close()
    lat.close()


@pytest.mark.parametrize("prec", ["f64", "f32"])
def test_apply_obeys_a_set_configuration(prec):
    """apply on tensors runs the configuration that is set, as resident fields do: an
    LDS cap that fits serves both with the same bits, and one that does not fit
    beside the staged tile (FP64 48 KiB, FP32 24 KiB of a CU's 160) is refused by both
    as OVS_ERR_HIP."""
    import torch
    import paper_0810_4228_amd as ovs
    dims = (4, 4, 6, 6)
    lat = lattice(dims, prec, synth.random_links(dims, 0.6, seed=70), 0.3)
    b = to_dev(synth.gaussian_sources(dims, 2, seed=71))
    f, g = lat.field_create(2), lat.field_create(2)
    f.import_(b)
    base = lat.get_tuning_raw(2)
    ref = lat.apply("A", b)
    # caps that fit beside both forms, beside the resident form alone, beside neither
    for cap in (40, 106, 110, 158) if prec == "f64" else (40, 132, 135, 158):
        for wg in (64, 256):
            lat.set_tuning_raw(2, [1110, wg, cap, 0] + base[4:])
            if cap < 158:
                f.apply("A", g)
                assert torch.equal(g.export().reshape(b.shape), ref)
                assert torch.equal(lat.apply("A", b), ref), (cap, wg)
            else:
                for call in (lambda: f.apply("A", g), lambda: lat.apply("A", b)):
                    with pytest.raises(ovs.OvsError) as e:
                        call()
                    assert e.value.status == ovs.OVS_ERR_HIP
    f.close()
    g.close()
    lat.close()


def test_closing_behind_enqueued_calls():
    """Operator calls only enqueue; a workspace that grows, a field or a lattice that
    is closed behind them waits for them: results as with synchronisations between."""
    import torch
    import paper_0810_4228_amd as ovs
    dims = (12, 12, 12, 24)
    U = to_dev(synth.random_links(dims, 0.5, seed=72))
    b = to_dev(synth.gaussian_sources(dims, 8, seed=73))
    out = []
    for wait in (True, False):
        done = []
        with torch.cuda.stream(torch.cuda.Stream()):
            lat = ovs.Lattice(dims, precision="f32")
            lat.set_links(U)
            lat.set_params(MW, 0.2)
            f, g = lat.field_create(8), lat.field_create(8)
            f.import_(b)
            for _ in range(20):
                f.apply("A", g)
                g.apply("A_dag", f)
            done.append(f.export())
            for n in (4, 6, 8):   # staged forms: the scratch fields grow
                done.append(lat.apply("A", b[:n].contiguous()))
                if wait:
                    torch.cuda.synchronize()
            for h in (f, g, lat):
                h.close()
                if wait:
                    torch.cuda.synchronize()
            scrap = torch.full((64 << 20,), 1.0, dtype=torch.float64, device="cuda")
        torch.cuda.synchronize()
        del scrap
        out.append(done)
    for x, y in zip(*out):
        assert torch.isfinite(torch.view_as_real(x)).all() and torch.equal(x, y)
