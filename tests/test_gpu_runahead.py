"""The host enqueues layers ahead of the device's stop flag.  How far ahead does not
matter: layers after the stop leave everything as it was, and one launch updates all
matrices with as many workgroups as they fill."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision", ["fp64", "fp32", "split_fp16"])
@pytest.mark.parametrize("n,k", [(2, 1), (16, 3), (33, 1), (130, 2), (257, 3)])
def test_outputs_do_not_depend_on_the_run_ahead(precision, n, k):
    import torch

    import paper_2203_09621_amd as dm
    from workloads import dense_gapped_problem

    p = dense_gapped_problem(n, max(1, n // 2), 0.8, 90 + n, h1="dense", k=k)
    h0, h1 = torch.from_numpy(p.H0).cuda(), [torch.from_numpy(h).cuda() for h in p.H1]
    ref = None
    for ahead in (1, 2, 7, 200):
        try:
            P0, P1s, st = dm.solve(h0, h1, p.nocc, precision=precision, poll_every=ahead)
            out = [t.cpu().numpy() for t in (P0, *P1s)]
            status = 0
        except dm.DmptError as exc:
            out, st, status = [], exc.stats, exc.status
        got = (status, st["layers"], st["d0_layer"], st["sigma"], st["eps1"])
        if ref is None:
            ref = (got, out)
        assert got == ref[0]
        assert all(np.array_equal(a, b) for a, b in zip(out, ref[1]))


# problems that run layer by layer (in the split forms: beyond one workgroup), all of
# which converge
@pytest.mark.parametrize("precision,n,k", [
    ("fp64", 33, 1), ("fp64", 257, 3), ("fp32", 130, 2), ("split_fp16", 97, 2),
    ("split_fp16", 130, 1), ("split_fp16", 257, 3), ("split_bf16", 129, 2)])
def test_converged_layered_solves_do_not_depend_on_the_run_ahead(precision, n, k):
    import torch

    import paper_2203_09621_amd as dm
    from workloads import dense_gapped_problem

    p = dense_gapped_problem(n, n // 2, 0.8, 90 + n, h1="dense", k=k)
    h0, h1 = torch.from_numpy(p.H0).cuda(), [torch.from_numpy(h).cuda() for h in p.H1]
    runs = [dm.solve(h0, h1, p.nocc, precision=precision, poll_every=ahead)
            for ahead in (1, 2, 7, 200)]
    P0, P1s, st = runs[0]
    assert st["converged"] and 10 < st["layers"] < 100
    for Q0, Q1s, su in runs[1:]:
        assert all(su[key] == st[key] for key in ("layers", "d0_layer", "d1_layer", "sigma"))
        assert all(torch.equal(a, b) for a, b in zip([P0, *P1s], [Q0, *Q1s]))
