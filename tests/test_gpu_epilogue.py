"""The fused epilogue has a path for whole tiles off the diagonal and one for the
rest, in tiles of 128 and of 256 rows and in pairs of tiles.  A problem's outputs are
the same, bit for bit, in whichever launch it runs, and exactly symmetric."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# one tile, tile edges and remainders of either tile size, a pair without a partner
SIZES = [130, 200, 255, 256, 257, 383, 384, 385, 511, 512, 513, 640, 769]


@pytest.mark.parametrize("precision", ["split_fp16", "split_bf16"])
@pytest.mark.parametrize("h1", ["diag", "dense"])
def test_outputs_do_not_depend_on_the_tile(precision, h1):
    import torch

    import paper_2203_09621_amd as dm
    from workloads import dense_gapped_problem

    probs = [dense_gapped_problem(n, max(1, n // 2), 0.6, 300 + n, h1=h1, k=1 + i % 3)
             for i, n in enumerate(SIZES)]
    H0 = [torch.from_numpy(p.H0).cuda() for p in probs]
    H1 = [[torch.from_numpy(h).cuda() for h in p.H1] for p in probs]
    runs = []
    for threshold in (128, 100000):              # every problem in 256-row tiles, in pairs
        b = dm.dmpt_batch_init(SIZES, [p.nocc for p in probs], [p.k for p in probs],
                               precision=precision, tile_threshold=threshold)
        try:
            P0, P1, st, _ = dm.dmpt_batch_response(b, H0, H1)
        finally:
            dm.dmpt_batch_destroy(b)
        runs.append([[P0[i], *P1[i]] for i in range(len(probs))])
    for i, p in enumerate(probs):
        P0, P1s, st = dm.solve(H0[i], H1[i], p.nocc, precision=precision)
        for a, b, c in zip([P0, *P1s], runs[0][i], runs[1][i]):
            assert torch.equal(a, b), (p.N, "256-row tiles")
            assert torch.equal(a, c), (p.N, "pairs")
            assert torch.equal(a, a.T), p.N
            assert np.isfinite(a.cpu().numpy()).all()


# single problems: 64-row tiles with one and with two workgroups per CU, 128-row tiles
# (two sizes beside each change of the rule), against the batch's pairs
@pytest.mark.parametrize("n,k", [(129, 1), (704, 3), (705, 3), (1024, 1), (1025, 1), (1024, 3),
                                 (1100, 3), (1290, 3), (1536, 1), (1537, 1)])
def test_single_problem_tiles_agree(n, k):
    import torch

    import paper_2203_09621_amd as dm
    from workloads import dense_gapped_problem

    p = dense_gapped_problem(n, n // 2, 0.8, 500 + n, h1="diag", k=k)
    H0, H1 = torch.from_numpy(p.H0).cuda(), [torch.from_numpy(h).cuda() for h in p.H1]
    b = dm.dmpt_batch_init([n], [p.nocc], [k], precision="split_fp16", tile_threshold=100000)
    try:
        Q0, Q1, _, _ = dm.dmpt_batch_response(b, [H0], [H1])
    finally:
        dm.dmpt_batch_destroy(b)
    P0, P1s, st = dm.solve(H0, H1, p.nocc, precision="split_fp16")
    assert st["converged"]
    for x, y in zip([P0, *P1s], [Q0[0], *Q1[0]]):
        assert torch.equal(x, y) and torch.equal(x, x.T)
