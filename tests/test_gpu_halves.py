"""functional_map hands contiguous evals and lam on by address and everything else through the checked entry
points: strided evals and lam give the same bits, forward and backward, and wrong inputs raise as those do."""
import pytest

pytestmark = pytest.mark.gpu


def _inputs(dev, P=2, n=300, k=20, d=48):
    import torch
    g = torch.Generator(device=dev).manual_seed(3)
    r = lambda *s: torch.randn(*s, generator=g, device=dev)
    evals = (r(2 * P, k).abs() * 20).sort(1).values
    return dict(feat=r(2 * P, n, d).requires_grad_(), phi=r(2 * P, n, k), mass=r(2 * P, n).abs() / n, evals=evals,
                lam=r(P).abs() + 0.01), r(P, k, k)


def _run(a, dC, bwd):
    import torch
    from paper_2604_10377_amd import fmap as F
    C, info = F.functional_map(**a, bwd=bwd)
    dF, = torch.autograd.grad(C, a["feat"], dC)
    return C, info, dF


@pytest.mark.parametrize("bwd", ["stored", "recompute"])
@pytest.mark.parametrize("strided", [("evals",), ("lam",), ("evals", "lam")])
def test_strided_inputs(dev, strided, bwd):
    import torch
    a, dC = _inputs(dev)
    want = _run(a, dC, bwd)
    b = dict(a)
    for name in strided:
        b[name] = torch.stack([a[name], a[name] + 1], -1)[..., 0]
        assert not b[name].is_contiguous()
    if "lam" in strided:  # the checked entry point takes contiguous lam only
        with pytest.raises(ValueError):
            _run(b, dC, bwd)
        return
    for x, y in zip(want, _run(b, dC, bwd)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("change,error", [
    (lambda a: dict(a, evals=a["evals"][:, :-1].contiguous()), ValueError),
    (lambda a: dict(a, evals=a["evals"][:-1]), ValueError),
    (lambda a: dict(a, evals=a["evals"].double()), TypeError),
    (lambda a: dict(a, evals=a["evals"].cpu()), ValueError),
    (lambda a: dict(a, lam=a["lam"].double()), TypeError),
    (lambda a: dict(a, lam=a["lam"][:1]), ValueError),
    (lambda a: dict(a, lam=a["lam"].cpu()), ValueError),
])
def test_wrong_inputs(dev, change, error):
    a, dC = _inputs(dev)
    with pytest.raises(error):
        _run(change(a), dC, "stored")
