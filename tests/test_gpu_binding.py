"""The binding's two ways to a call: the extension module for arguments with nothing to object to, and the checks that say
what is wrong for the others."""
import numpy as np
import pytest
import torch

from paper_2504_03702_amd import binding as ps

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def scan_args(n=3, length=8):
    z = lambda m, dt=torch.int32: torch.zeros(m, dtype=dt, device=DEV)
    kv = torch.arange(n * length, dtype=torch.int32, device=DEV)
    return [kv, torch.full((n,), 40, dtype=torch.int32, device=DEV), n, length, 5, z(n), z(n), z(n), z(2), z(1, torch.float64)]


def test_native_and_checked_ways_give_the_same(monkeypatch):
    ps.load_library()
    assert ps._native is not None
    made = []
    real = ps._made
    monkeypatch.setattr(ps, "_made", lambda name, *a: made.append(real(name, *a)) or made[-1])
    a, b, c = scan_args(), scan_args(), scan_args()
    ps.ps_scaler_scan(*a)
    b[2] = np.int64(3)                                          # an integer the module does not take
    ps.ps_scaler_scan(*b, over_pct=95)
    with torch.cuda.stream(torch.cuda.Stream()):
        torch.cuda.current_stream().wait_stream(torch.cuda.default_stream())
        ps.ps_scaler_scan(*c)
        torch.cuda.synchronize()
    assert made == [True, False, True]
    for x, y, z in zip(a[5:], b[5:], c[5:]):
        assert torch.equal(x, y) and torch.equal(x, z)
    assert a[6].tolist() == [4, 12, 20]


@pytest.mark.parametrize("at,what,error", [
    (0, lambda t: t[:-1], ValueError), (0, lambda t: t.float(), TypeError), (0, lambda t: t.cpu(), TypeError),
    (5, lambda t: torch.zeros(6, dtype=torch.int32, device=DEV)[::2], TypeError), (1, lambda t: None, AttributeError),
    (0, lambda t: t.cpu().numpy(), AttributeError), (4, lambda t: -1, ps.PsError), (4, lambda t: 1.5, Exception),
    (3, lambda t: 1 << 40, Exception), (9, lambda t: t.to(torch.float32), TypeError)])
def test_what_was_refused_stays_refused(at, what, error):
    args = scan_args()
    args[at] = what(args[at])
    with pytest.raises(error):
        ps.ps_scaler_scan(*args)


def test_subclasses_and_parameters_go_through():
    args = scan_args()
    args[0] = torch.nn.Parameter(args[0], requires_grad=False)

    class Mine(torch.Tensor):
        pass

    args[1] = args[1].as_subclass(Mine)
    ps.ps_scaler_scan(*args)
    assert args[6].tolist() == [4, 12, 20]
