"""A response that fails leaves nothing behind: the next one on the same context, with
another number of responses and so on other tiles, equals one on a fresh context."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


# direct forms where the tiles of the two calls end at different rows (N = 840 in FP64:
# 864 with one response, 896 with three; N = 720 in FP32: 736 and 768), and split forms
# with one workgroup, 64-row and 128-row tiles
@pytest.mark.parametrize("precision,n,bad,k", [
    ("fp64", 840, 3, 1), ("fp64", 840, 1, 3), ("fp64", 33, 2, 1), ("fp32", 720, 2, 1),
    ("fp32", 720, 1, 2), ("split_fp16", 100, 3, 1), ("split_fp16", 710, 1, 3),
    ("split_bf16", 1290, 3, 1)])
def test_response_after_a_failed_one(precision, n, bad, k):
    import torch

    import paper_2203_09621_amd as dm
    from workloads import dense_gapped_problem

    p = dense_gapped_problem(n, n // 2, 0.8, 700 + n, h1="dense", k=3)
    h0, h1 = torch.from_numpy(p.H0).cuda(), [torch.from_numpy(h).cuda() for h in p.H1]
    nan = h1[0].clone()
    nan[n - 1, n - 1] = float("nan")
    out = [[torch.empty_like(h0) for _ in range(1 + k)] for _ in range(2)]
    fresh = dm.dmpt_init(h0, p.nocc, k_max=3, precision=precision)
    used = dm.dmpt_init(h0, p.nocc, k_max=3, precision=precision)
    try:
        dm.dmpt_response(fresh, h1[:k], P0=out[0][0], P1s=out[0][1:])
        with pytest.raises(dm.DmptError) as exc:
            dm.dmpt_response(used, [nan, *h1[1:bad]])
        assert exc.value.status == -5
        st = dm.dmpt_response(used, h1[:k], P0=out[1][0], P1s=out[1][1:])
    finally:
        dm.dmpt_destroy(fresh)
        dm.dmpt_destroy(used)
    assert all(torch.equal(a, b) for a, b in zip(*out))
    assert np.isfinite(out[1][0].cpu().numpy()).all() and st is not None


@pytest.mark.parametrize("precision", ["split_fp16", "split_bf16"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_statistics_of_a_failed_small_response(precision, value):
    """A problem that runs as one workgroup fails with the statistics of the layer by
    layer path (which per-launch timing keeps)."""
    import torch

    import paper_2203_09621_amd as dm
    from workloads import dense_gapped_problem

    p = dense_gapped_problem(64, 32, 0.8, 31, h1="dense", k=2)
    p.H1[1][5, 5] = value
    got = []
    for timing in (False, True):
        with pytest.raises(dm.DmptError) as exc:
            dm.solve(torch.from_numpy(p.H0).cuda(), [torch.from_numpy(h).cuda() for h in p.H1],
                     p.nocc, precision=precision, timing=timing)
        st = exc.value.stats
        got.append([exc.value.status] + [st[key] for key in (
            "layers", "d0_layer", "d1_layer", "converged", "sigma", "eps1", "epsN", "n_s")])
    assert got[0][0] == -5 and got[0] == got[1]
