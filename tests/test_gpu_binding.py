"""The binding's two ways to a call: the extension module for arguments with nothing to object to, and the checks that say
what is wrong for the others."""
import numpy as np
import pytest
import torch

from paper_2504_03702_amd import binding as ps
from paper_2504_03702_amd import workloads as wl

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


# ---- all seven calls, both ways ------------------------------------------------------------------------------------------
N, INST, HORIZON, LENGTH, WINDOW, HIDDEN, K = 40, 5, 12, 32, 6, 16, 7


def i32(a):
    return torch.from_numpy(np.ascontiguousarray(a, np.int32)).to(DEV)


def z(n, dtype=torch.int32):
    return torch.zeros(n, dtype=dtype, device=DEV)


@pytest.fixture(scope="module")
def model(tmp_models):
    cfg = wl.MODELS["tiny"]
    path = f"{tmp_models}/binding.bin"
    wl.write_model(path, cfg, wl.make_weights(cfg, seed=3))
    return ps.ps_model_load(path, 0)


def call_args(name, model):
    """Arguments of a call, the same every time."""
    rng = np.random.default_rng(5)
    pred, inst, bucket = rng.integers(1, 9, N), rng.integers(0, INST, N), rng.integers(0, HORIZON, N)
    if name == "predict_load":
        b = wl.make_prompts("tiny", seed=1, n_req=6)
        lengths = np.minimum(np.diff(b.offsets), 5 + np.arange(6))
        ws = ps.alloc_workspace(ps.ps_workspace_bytes(model, len(b.token_ids), 6), DEV)
        return [model, i32(b.token_ids), i32(b.offsets), i32(lengths), z(6, torch.float32), z(6), ws, ps.new_status(DEV)]
    if name in ("anticipate", "anticipate_static"):
        args = [i32(pred), i32(inst), i32(bucket), i32(1 + np.arange(INST)), INST, HORIZON, z(INST * HORIZON), z(INST, torch.int64)]
        ws = [ps.alloc_workspace(ps.ps_anticipate_workspace_bytes(N, INST, HORIZON), DEV)] if name == "anticipate" else []
        return args + ws + [ps.new_status(DEV)]
    if name == "lookahead_update":
        ws = ps.alloc_workspace(ps.ps_lookahead_workspace_bytes(N, INST, LENGTH), DEV)
        return [i32(inst), i32(bucket), i32(rng.integers(1, 50, N)), i32(0 * pred), i32(pred), i32(0 * pred + 1), INST, LENGTH,
                z(INST * LENGTH), z(INST, torch.int64), ws, i32(200 + np.arange(INST)), z(INST * LENGTH, torch.float32),
                ps.new_status(DEV)]
    if name == "scaler_scan":
        return [i32(rng.integers(0, 100, INST * LENGTH)), i32(80 + np.arange(INST)), INST, LENGTH, 9, z(INST), z(INST), z(INST), z(2),
                z(1, torch.float64), 90, 20, 40]
    if name == "route":
        return [i32(rng.integers(1, 50, N)), i32(pred), INST, WINDOW, i32(rng.integers(0, 100, INST * WINDOW)), i32(100 + np.arange(INST)),
                i32(rng.integers(0, 9, INST)).long(), i32(rng.integers(0, 9, INST)).long(), z(N), z(N, torch.int64), 70, 2,
                ps.new_status(DEV)]
    f = wl.make_forecaster_inputs(seed=2, n_services=INST, hidden=HIDDEN, k=K)
    t = lambda a: torch.from_numpy(a).to(DEV)
    return [t(f.weights), HIDDEN, t(f.hist_p), t(f.hist_d), INST, K, t(f.mu), z(5 * INST, torch.float32)]


CALLS = ["predict_load", "anticipate", "anticipate_static", "lookahead_update", "scaler_scan", "route", "forecast"]
# tensors whose size nothing checks: what they hold is as long as the caller says
UNSIZED = {"predict_load": {1, 2, 3, 4, 5, 6, 7}, "anticipate": {8, 9}, "anticipate_static": {8}, "lookahead_update": {10, 13},
           "scaler_scan": set(), "route": {12}, "forecast": set()}


def outcome(name, args):
    try:
        getattr(ps, "ps_" + name)(*args)
    except Exception as e:
        return type(e), getattr(e, "code", None)
    torch.cuda.synchronize()
    return [a.cpu() for a in args if isinstance(a, torch.Tensor) and a.dtype != torch.uint8]


def both_ways(monkeypatch, name, model, change=lambda args: None):
    """What a call does by the extension module (or what it hands back) and by ctypes alone; whether the module made it."""
    ps.load_library()
    got, made, real = [], [], ps._made
    for native in (ps._native, None):
        args = call_args(name, model)
        change(args)
        with monkeypatch.context() as m:
            m.setattr(ps, "_native", native)
            m.setattr(ps, "_made", lambda *a: made.append(real(*a)) or made[-1])
            got.append(outcome(name, args))
    return got, made


@pytest.mark.parametrize("name", CALLS)
def test_every_call_gives_the_same_both_ways(monkeypatch, model, name):
    (a, b), made = both_ways(monkeypatch, name, model)
    assert made == [True, False]
    assert isinstance(a, list) and len(a) == len(b)
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    fresh = [t.cpu() for t in call_args(name, model) if isinstance(t, torch.Tensor) and t.dtype != torch.uint8]
    assert any(not torch.equal(x, y) for x, y in zip(a, fresh))        # (something was written)


@pytest.mark.parametrize("name", CALLS)
def test_every_call_without_what_may_be_left_out(monkeypatch, model, name):
    optional = {"predict_load": [3, 7], "anticipate": [3, 7, 9], "anticipate_static": [3, 7, 8], "lookahead_update": [9, 11, 12, 13],
                "route": [12]}.get(name, [])
    def drop(args):
        for i in optional:
            args[i] = None
    (a, b), made = both_ways(monkeypatch, name, model, drop)
    assert made == [True, False]
    assert isinstance(a, list) and all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("name", CALLS)
def test_every_call_refuses_the_same_both_ways(monkeypatch, model, name):
    for at, arg in enumerate(call_args(name, model)):
        if not isinstance(arg, torch.Tensor):
            continue
        wrong = {"type": lambda t: t.to(torch.int16), "place": lambda t: t.cpu()}
        if at not in UNSIZED[name]:
            wrong["size"] = lambda t: torch.cat([t, t[:1]])
        for what, make in wrong.items():
            print(f"{name} argument {at}: {what}", flush=True)
            (a, b), made = both_ways(monkeypatch, name, model, lambda args: args.__setitem__(at, make(args[at])))
            assert made == [False, False] and a == b, (at, what)
            assert a[0] is (ValueError if what == "size" else TypeError), (at, what)
