"""Small problems in the split forms run as one workgroup.  Per-launch timing
keeps the layer-by-layer kernels, so the two paths are compared on the same
inputs: outputs, layers and decisions must be the same, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def dm():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a device"
    import paper_2203_09621_amd as dm
    return dm


def _cuda(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _problem(n, k, h1="dense"):
    from workloads import dense_gapped_problem
    return dense_gapped_problem(n, max(1, n // 2), 0.8, 60 + 7 * n + k, h1=h1, k=k)


def _both(dm, p, precision, **kw):
    h0, h1 = _cuda(p.H0), [_cuda(h) for h in p.H1]
    out = []
    for timing in (False, True):
        try:
            P0, P1s, st = dm.solve(h0, h1, p.nocc, precision=precision, timing=timing, **kw)
            out.append(([t.cpu().numpy() for t in (P0, *P1s)], st, 0))
        except dm.DmptError as exc:
            out.append((None, exc.stats, exc.status))
    return out


# block edges, the largest N of each response count and the first N past it
@pytest.mark.parametrize("precision", ["split_fp16", "split_bf16"])
@pytest.mark.parametrize("n,k", [(2, 1), (31, 3), (32, 1), (33, 2), (64, 1), (64, 3), (65, 2),
                                 (95, 1), (96, 3), (97, 1), (97, 2), (128, 1), (129, 1)])
def test_one_workgroup_equals_layers(dm, precision, n, k):
    (a, sa, ea), (b, sb, eb) = _both(dm, _problem(n, k), precision)
    assert ea == eb == 0
    for x, y in zip(a, b):
        assert np.array_equal(x, y)
    for key in ("layers", "d0_layer", "d1_layer", "sigma", "converged", "eps1", "epsN", "n_s"):
        assert sa[key] == sb[key], key
    assert np.allclose([sa["idem0"], *sa["idem1"]], [sb["idem0"], *sb["idem1"]], rtol=1e-12)


def test_layer_cap_and_nonfinite_input(dm):
    """A capped run ends with the layer cap reported, and a NaN with its status."""
    p = _problem(50, 2)
    (_, sa, ea), (_, sb, eb) = _both(dm, p, "split_fp16", max_layers=7)
    assert ea == eb == -4 and sa["layers"] == sb["layers"] == 7 and sa["sigma"] == sb["sigma"]
    p.H1[1][3, 3] = np.nan
    (_, _, ea), (_, _, eb) = _both(dm, p, "split_fp16")
    assert ea == eb == -5


def test_capped_outputs_hold_the_last_layer(dm):
    import torch
    p = _problem(70, 2)
    h0, h1 = _cuda(p.H0), [_cuda(h) for h in p.H1]
    got = []
    for timing in (False, True):
        P0, P1s = torch.empty_like(h0), [torch.empty_like(h0) for _ in h1]
        ctx = dm.dmpt_init(h0, p.nocc, k_max=2, max_layers=9, timing=timing)
        with pytest.raises(dm.DmptError):
            dm.dmpt_response(ctx, h1, P0, P1s)
        dm.dmpt_destroy(ctx)
        got.append([t.cpu().numpy() for t in (P0, *P1s)])
    assert all(np.array_equal(x, y) for x, y in zip(*got))


@pytest.mark.parametrize("precision", ["split_fp16", "split_bf16"])
def test_batch_of_both_paths_equals_layers(dm, precision):
    """A batch whose small problems (of every configuration, between larger
    ones) run as workgroups: every problem equals its layer-by-layer solve;
    a second response on the same batch repeats it."""
    sizes = [(40, 1), (200, 2), (128, 1), (96, 3), (128, 2), (16, 2), (64, 3), (300, 1), (33, 3),
             (90, 1), (64, 1), (20, 3), (90, 2), (5, 1)]
    probs = [_problem(n, k, "diag") for n, k in sizes]
    b = dm.dmpt_batch_init([p.N for p in probs], [p.nocc for p in probs], [p.k for p in probs],
                           precision=precision)
    H0, H1 = [_cuda(p.H0) for p in probs], [[_cuda(h) for h in p.H1] for p in probs]
    runs = []
    for _ in range(2):
        P0, P1, st, _ = dm.dmpt_batch_response(b, H0, H1)
        runs.append([[t.cpu().numpy() for t in (x, *y)] for x, y in zip(P0, P1)])
    dm.dmpt_batch_destroy(b)
    for i, p in enumerate(probs):
        _, (ref, sst, err) = _both(dm, p, precision)
        assert err == 0 and st[i]["layers"] == sst["layers"] and st[i]["k"] == p.k
        assert st[i]["d0_layer"] == sst["d0_layer"] and st[i]["d1_layer"] == sst["d1_layer"]
        for x, y, z in zip(runs[0][i], runs[1][i], ref):
            assert np.array_equal(x, z) and np.array_equal(y, z), (i, p.N)
