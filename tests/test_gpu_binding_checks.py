"""The binding's one-pass argument check on device tensors accepts what the
error-raising pass accepts and refuses what it refuses, with the same error."""
import pytest
import torch

pytestmark = pytest.mark.gpu


def _tensors(**change):
    d = dict(q=torch.zeros((2, 3, 2, 64), dtype=torch.bfloat16, device="cuda"),
             k=torch.zeros((2, 3, 2, 64), dtype=torch.bfloat16, device="cuda"),
             beta=torch.zeros((2, 3, 2), device="cuda"),
             h0=torch.zeros((2, 2, 64, 64), device="cuda"))
    d.update(change)
    return d


@pytest.mark.parametrize("make,error", [
    (lambda d: {}, None),
    (lambda d: dict(k=torch.nn.Parameter(d["k"], requires_grad=False)), None),
    (lambda d: dict(k=None, beta=None, h0=None), None),
    (lambda d: dict(k=d["k"].cpu()), ValueError),
    (lambda d: dict(q=d["q"].cpu()), ValueError),
    (lambda d: dict(k=d["k"].float()), ValueError),
    (lambda d: dict(k=d["k"][0]), ValueError),
    (lambda d: dict(k=d["k"][:, :2].contiguous()), ValueError),
    (lambda d: dict(k=d["k"].transpose(1, 2).contiguous().transpose(1, 2)), ValueError),
    (lambda d: dict(q=d["q"].transpose(1, 2).contiguous().transpose(1, 2)), ValueError),
    (lambda d: dict(k=[0.0]), TypeError),
    (lambda d: dict(beta=d["beta"].double()), ValueError),
    (lambda d: dict(beta=d["beta"][..., None].contiguous()), ValueError),
    (lambda d: dict(h0=d["h0"][:1].contiguous()), ValueError),
    (lambda d: dict(h0=d["h0"].bfloat16()), ValueError),
])
def test_checks_on_device_tensors(make, error):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_2412_06464_amd import gdn
    d = _tensors()
    d.update(make(d))
    check = lambda: gdn._check_tensors(d["q"], rows=(("k", d["k"]),), gates=(("beta", d["beta"]),),
                                       states=(("h0", d["h0"], 64),), nstate=2)
    if error is None:
        check()
    else:
        with pytest.raises(error):
            check()
