"""Calls whose kernels or buffers are chosen by size, tuning or workspace: every
route is open to the calls that the interface admits, with the same results (GPU)."""
import pytest

import synth
from gpu_util import say, to_dev

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
