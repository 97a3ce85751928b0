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
