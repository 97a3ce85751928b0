"""Batches of small and larger problems.  A few small ones run in the larger ones' rounds;
enough of them to save two rounds run as one workgroup each.  Either way every problem
has the results of its own solve, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _run(sizes, precision):
    import torch

    import paper_2203_09621_amd as dm
    from workloads import dense_gapped_problem

    made = {}
    for i, (n, k) in enumerate(sizes):
        if (n, k) not in made:
            p = dense_gapped_problem(n, n // 2, 0.8, 60 + 7 * n + k, h1="diag", k=k)
            made[n, k] = (torch.from_numpy(p.H0).cuda(),
                          [torch.from_numpy(h).cuda() for h in p.H1], p.nocc)
    probs = [made[s] for s in sizes]
    b = dm.dmpt_batch_init([n for n, _ in sizes], [p[2] for p in probs], [k for _, k in sizes],
                           precision=precision, tile_threshold=100000)
    try:
        info = dm.dmpt_batch_info(b)
        P0, P1, st, _ = dm.dmpt_batch_response(b, [p[0] for p in probs], [p[1] for p in probs])
    finally:
        dm.dmpt_batch_destroy(b)
    for i, s in enumerate(sizes):
        if s not in made:
            continue
        h0, h1, nocc = made.pop(s)                         # each problem once
        Q0, Q1, su = dm.solve(h0, h1, nocc, precision=precision)
        assert st[i]["layers"] == su["layers"] and st[i]["d1_layer"] == su["d1_layer"], s
        assert all(torch.equal(x, y) for x, y in zip([P0[i], *P1[i]], [Q0, *Q1])), s
        assert np.isfinite(P0[i].cpu().numpy()).all()
    return info


SMALL = [(5, 1), (16, 2), (20, 3), (33, 3), (40, 1), (64, 3), (90, 1), (90, 2), (96, 3), (128, 1)]


@pytest.mark.parametrize("precision", ["split_fp16", "split_bf16"])
def test_a_few_small_problems_run_with_the_larger_ones(precision):
    sizes = [(200, 2), *SMALL, (300, 1)]
    th, n256, n128 = _run(sizes, precision)
    # pairs of 128-row tiles: 1 + k of a small problem, (1 + k) ceil(T (T + 1) / 4) of a larger
    assert th == 100000 and n256 == 0
    assert n128 >= 3 * 2 + 2 * 3 + sum(1 + k for _, k in SMALL)


def test_many_small_problems_run_as_workgroups():
    sizes = [(200, 2), *SMALL * 30, (300, 1)]              # 870 pairs beside 12
    assert sum(1 + k for _, k in SMALL * 30) > 2 * 256
    th, n256, n128 = _run(sizes, "split_fp16")
    assert th == 100000 and n256 == 0 and n128 < 100
