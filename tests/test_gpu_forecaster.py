"""GPU parity of ps_forecast (service workload predictor's online phase, paper Sec. 3.2, Alg. 2)
against the fp64 oracle on the same seeded models and histories, through the C ABI."""
import numpy as np
import pytest
import torch

from oracle import forecaster as of
from paper_2504_03702_amd import binding as ps
from paper_2504_03702_amd import workloads as wl

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
TOL = 1e-4          # fp32 recurrence of k + 1 steps against fp64


def run_forecast(x):
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(DEV)
    S = x.hist_p.shape[0]
    out = torch.full((S * 5,), -1.0, dtype=torch.float32, device=DEV)
    ps.ps_forecast(t(x.weights).reshape(-1), x.hidden, t(x.hist_p).reshape(-1), t(x.hist_d).reshape(-1), S, x.k,
                   t(x.mu).reshape(-1), out)
    return out.cpu().numpy().reshape(S, 5).T.astype(np.float64)


@pytest.mark.parametrize("S,H,k", [(1, 1, 1), (3, 8, 4), (8, 32, 12), (5, 64, 24), (130, 17, 9)])
def test_forecasts_and_instance_counts(S, H, k):
    print(f"forecast S={S} H={H} k={k}", flush=True)
    x = wl.make_forecaster_inputs(seed=S + H, n_services=S, hidden=H, k=k)
    got = run_forecast(x)
    ref = of.forecast_services([x.model(s, 0) for s in range(S)], [x.model(s, 1) for s in range(S)],
                               x.hist_p.astype(np.float64), x.hist_d.astype(np.float64),
                               x.mu[:, 0].astype(np.float64), x.mu[:, 1].astype(np.float64), x.mu[:, 2].astype(np.float64))
    scale = np.maximum(np.abs(ref), np.sqrt(np.mean(ref ** 2, axis=1, keepdims=True)))
    err = np.abs(got - ref) / scale
    print(f"  max rel err {err.max():.2e}", flush=True)
    assert err.max() < TOL
    assert np.std(ref[2]) > 0 or S == 1                      # services differ
    if S >= 8:
        # both kinds of second step occur: first forecast inside the history's range (recurrence carried on) and
        # outside it (extended history normalised afresh)
        inside = (ref[0] >= x.hist_p.min(axis=1)) & (ref[0] <= x.hist_p.max(axis=1))
        assert inside.any() and (~inside).any()


def test_argument_checks():
    z = torch.zeros(16, dtype=torch.float32, device=DEV)
    with pytest.raises(ps.PsError) as e:
        load = ps.load_library()
        ps._check(load.ps_forecast(z.data_ptr(), 65, z.data_ptr(), z.data_ptr(), 1, 1, z.data_ptr(), z.data_ptr(), None),
                  "ps_forecast")
    assert e.value.code == -6


@pytest.mark.parametrize("S,H,k", [(2, 2, 70), (4, 31, 5), (9, 32, 1), (3, 33, 65), (2, 63, 48), (600, 64, 3),
                                   (1025, 1, 3), (2047, 4, 3), (2048, 4, 4), (3073, 16, 2), (3074, 32, 1)])
def test_register_tile_edges(S, H, k):
    """Hidden sizes around the register tiles (32, 64; a wavefront holds a quarter of W_mh's rows), histories shorter
    and longer than a wavefront, more services than the chip holds at once, and so many that a wavefront takes a service."""
    x = wl.make_forecaster_inputs(seed=S + H, n_services=S, hidden=H, k=k)
    got = run_forecast(x)
    ref = of.forecast_services([x.model(s, 0) for s in range(S)], [x.model(s, 1) for s in range(S)],
                               x.hist_p.astype(np.float64), x.hist_d.astype(np.float64),
                               x.mu[:, 0].astype(np.float64), x.mu[:, 1].astype(np.float64), x.mu[:, 2].astype(np.float64))
    scale = np.maximum(np.abs(ref), np.sqrt(np.mean(ref ** 2, axis=1, keepdims=True)))
    err = np.abs(got - ref) / scale
    print(f"forecast S={S} H={H} k={k} max rel err {err.max():.2e}", flush=True)
    assert err.max() < TOL


def set_field(x, name, unit, value):
    """Unit `unit` of a vector field of every model of x."""
    at, H = 0, x.hidden
    for f in wl.FORECASTER_FIELDS:
        if f == name:
            x.weights[:, :, at + unit] = value
        at += H * H if f.startswith("W_") else 1 if f == "b_out" else H


# a workgroup a service, of both register tiles, and a wavefront a service
@pytest.mark.parametrize("S,H,k", [(3, 8, 4), (5, 64, 24), (2048, 4, 4)])
def test_gates_held_open_and_shut(S, H, k):
    """Biases that hold a gate open or shut, infinite or so large that the exponent of their exponential overflows:
    sigmoid and tanh saturate, forecasts are the definition's."""
    print(f"forecast saturated S={S} H={H} k={k}", flush=True)
    x = wl.make_forecaster_inputs(seed=S + H, n_services=S, hidden=H, k=k)
    for unit, (name, value) in enumerate([("b_f", np.inf), ("b_i", 3e38), ("b_o", np.inf), ("b_h", -np.inf)]):
        set_field(x, name, unit, value)
    for unit, (name, value) in enumerate([("b_f", -np.inf), ("b_i", -3e38), ("b_o", -np.inf), ("b_h", 3e38)]):
        set_field(x, name, H - 1 - unit, value)
    got = run_forecast(x)
    with np.errstate(over="ignore"):
        ref = of.forecast_services([x.model(s, 0) for s in range(S)], [x.model(s, 1) for s in range(S)],
                                   x.hist_p.astype(np.float64), x.hist_d.astype(np.float64),
                                   x.mu[:, 0].astype(np.float64), x.mu[:, 1].astype(np.float64), x.mu[:, 2].astype(np.float64))
    assert np.isfinite(ref).all() and (ref[:4] > 0).any()
    scale = np.maximum(np.abs(ref), np.sqrt(np.mean(ref ** 2, axis=1, keepdims=True)))
    assert (np.abs(got - ref) / scale).max() < TOL


def test_error_of_the_gates_far_out():
    """A gate's own relative error stays that of an exponential of one unit in the last place however far out the gate is:
    2^-23 for e^-z, 2^-24 for the quotient's rounding and 2^-25 for the products in between, 2.1e-7 in all.  One unit whose
    cell has grown to 20 (tanh 1 to the last bit) and an output gate at z: the forecast is the gate's value."""
    S, k = 1024, 20
    z = np.linspace(-86.0, 86.0, S).astype(np.float32)
    x = wl.make_forecaster_inputs(seed=0, n_services=S, hidden=1, k=k)
    x.weights[:], x.hist_p[:], x.hist_d[:], x.mu[:] = 0, 0, 0, 1
    for name, value in [("b_h", 20.0), ("b_i", 100.0), ("b_f", 100.0), ("b_o", z[:, None]), ("w_out", 1.0)]:
        set_field(x, name, 0, value)
    ref = 1.0 / (1.0 + np.exp(-z.astype(np.float64)))
    err = np.abs(run_forecast(x)[:2] / ref - 1.0)
    print(f"gate error {err.max():.2e}, beyond 20 {err[:, np.abs(z) > 20].max():.2e}", flush=True)
    assert err.max() < 2.1e-7
