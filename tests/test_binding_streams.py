"""The binding's stream ordering (CPU only, with stand-ins for torch, its streams and the library):
what waits for what around a call, also one that fails after it enqueued something, and around
the copy into a buffer that an earlier call may still be using."""
import threading
import types

import numpy as np
import pytest

from paper_2308_01957_amd import apx

LOG = []


class Event:
    def record(self, stream):
        self.at = stream
        LOG.append("record " + stream.name)


class Stream:
    def __init__(self, name):
        self.name = name

    def wait_event(self, ev):
        LOG.append("%s waits for %s" % (self.name, ev.at.name))


class Tensor:
    def __init__(self, name, n):
        self.name, self.n = name, n

    def numel(self):
        return self.n

    def data_ptr(self):
        return 1

    def record_stream(self, stream):
        LOG.append("%s used by %s" % (self.name, stream.name))

    def clone(self):
        return Tensor(self.name + " copy", self.n)

    def copy_(self, src):
        LOG.append("caller copies into " + self.name)


@pytest.fixture
def problem(monkeypatch):
    LOG.clear()
    monkeypatch.setattr(apx, "check_buffer", lambda t, *a: t)
    caller = Stream("caller")
    P = object.__new__(apx.Problem)
    cuda = types.SimpleNamespace(current_stream=lambda device: caller, Event=Event, current_device=lambda: 0)
    alloc = lambda *a, **k: Tensor("new", 4)                                        # noqa: E731
    P.torch = types.SimpleNamespace(cuda=cuda, float64="f8", float32="f4", uint8="u1", empty=alloc, zeros=alloc)
    P.device, P.stream, P._events = types.SimpleNamespace(index=0), Stream("library"), threading.local()
    P.n_par, P.n_sub, P.n_pix, P.a_offsets = 4, 1, 4, np.array([0, 16])
    P._theta = P._dev = lambda x, *a: x
    P._prob = P._ctx = None
    P.status = apx.APX_OK

    class Lib:
        def __getattr__(self, name):
            def call(*args):
                LOG.append(name)
                return P.status
            return call

        def apx_status_string(self, status):
            return b"failed"

    P.lib = Lib()
    return P


T = {k: Tensor(k, 4) for k in ("theta", "data", "weight", "F", "z", "u", "seed")}
CALLS = {
    "apx_render": lambda P: P.render(T["theta"]),
    "apx_chi2": lambda P: P.chi2(T["theta"], T["data"], T["weight"]),
    "apx_jacobian": lambda P: P.jacobian(T["theta"]),
    "apx_jtwj": lambda P: P.jtwj(T["theta"], T["data"], T["weight"]),
    "apx_covariance": lambda P: P.covariance(T["theta"], T["data"], T["weight"]),
    "apx_covariance_factor": lambda P: P.covariance_factor(T["theta"], T["data"], T["weight"]),
    "apx_chi2_grad": lambda P: P.chi2_grad(T["theta"], T["data"], T["weight"]),
    "apx_render_vjp": lambda P: P.render_vjp(T["theta"], T["seed"]),
    "apx_lm_init": lambda P: P.lm_init(T["theta"], T["data"], T["weight"]),
    "apx_lm_step": lambda P: P.lm_step(T["data"], T["weight"], T["theta"], Tensor("state", 64)),
    "apx_lm_run": lambda P: P.lm_run(3, T["data"], T["weight"], T["theta"], Tensor("state", 64)),
    "apx_hmc_run": lambda P: P.hmc(T["theta"], T["data"], T["weight"], Tensor("F", 16), 0.1, 2, T["z"], Tensor("u", 1)),
    "apx_nuts_run": lambda P: P.nuts(T["theta"], T["data"], T["weight"], Tensor("F", 16), 0.1, 1, T["z"], Tensor("u", 6)),
    "apx_nuts_warmup": lambda P: P.nuts_warmup(T["theta"], T["data"], T["weight"], Tensor("F", 16), 0.1, 1, 0.8, T["z"],
                                               Tensor("u", 6)),
}


@pytest.mark.parametrize("failing", [False, True], ids=["ok", "error"])
@pytest.mark.parametrize("name", sorted(CALLS))
def test_the_caller_waits_for_every_call(problem, name, failing):
    problem.status = apx.APX_E_HIP if failing else apx.APX_OK
    if failing:
        with pytest.raises(apx.ApxError):
            CALLS[name](problem)
    else:
        CALLS[name](problem)
    at = LOG.index(name)
    assert LOG[at - 1] != name and "library waits for caller" in LOG[:at]
    assert LOG[at + 1:] == ["record library", "caller waits for library"], LOG


def test_a_fit_is_started_again_behind_the_work_on_its_buffers(problem):
    out = Tensor("theta_out", 4)
    problem.lm_init(T["theta"], T["data"], T["weight"], theta_out=out, state_out=Tensor("state", 64))
    copy = LOG.index("caller copies into theta_out")
    assert LOG[:copy] == ["record library", "caller waits for library"], LOG
    assert LOG.index("library waits for caller") > copy
