"""Products of non-orthogonal bases read operands without padding where they lie and
write the result in place.  Operands off the 16-byte alignment and results that
overlap Z are copied instead: the values must be the same, bit for bit."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _off(a):
    """A copy of a on the device whose first element is off the 16-byte alignment."""
    import torch
    buf = torch.empty(a.size + 1, dtype=torch.float64, device="cuda")
    v = buf[1:].view(a.shape)
    v.copy_(torch.from_numpy(a))
    assert v.data_ptr() % 16 == 8
    return v


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [1, 31, 127, 128, 129, 384])
def test_copied_and_in_place_operands_agree(n, precision):
    import torch

    import paper_2203_09621_amd as dm
    from workloads import sym_normal

    rng = np.random.default_rng(n)
    z, a = sym_normal(rng, n, 1.0), sym_normal(rng, n, 1.0)
    o = np.eye(n) + 0.2 * a / max(1.0, np.abs(np.linalg.eigvalsh(a)).max())
    zd, ad, od = (torch.from_numpy(v).cuda() for v in (z, a, o))
    ref = dm.dmpt_congruence(_off(z), _off(a), precision=precision)
    assert torch.equal(dm.dmpt_congruence(zd, ad, precision=precision), ref)
    assert torch.equal(zd.cpu(), torch.from_numpy(z)) and torch.equal(ad.cpu(), torch.from_numpy(a))
    assert torch.equal(dm.dmpt_congruence(zd, ad, precision=precision, out=_off(a)), ref)
    za, aa = zd.clone(), ad.clone()
    assert torch.equal(dm.dmpt_congruence(zd, aa, precision=precision, out=aa), ref)
    assert torch.equal(dm.dmpt_congruence(za, ad, precision=precision, out=za), ref)
    buf = torch.zeros(n * n + n, dtype=torch.float64, device="cuda")    # partial overlap with Z
    zv, ov = buf[: n * n].view(n, n), buf[n:].view(n, n)
    zv.copy_(zd)
    assert torch.equal(dm.dmpt_congruence(zv, ad, precision=precision, out=ov), ref)
    tol = 1e-12 if precision == "fp64" else 1e-4
    Z, it, err = dm.dmpt_inverse_factor(od, precision=precision, tol=tol)
    Z2, it2, err2 = dm.dmpt_inverse_factor(_off(o), precision=precision, tol=tol)
    assert it == it2 and err == err2 and torch.equal(Z, Z2)
    assert np.linalg.norm(Z.cpu().numpy() @ o @ Z.cpu().numpy() - np.eye(n)) < 100 * tol
    oo = od.clone()
    assert torch.equal(dm.dmpt_inverse_factor(oo, precision=precision, tol=tol, Z=oo)[0], Z)
