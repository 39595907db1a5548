"""The native side of the Python binding (csrc/gpp_binding.cpp) against the
package's own argument checks: the same results bit for bit where it takes a
call, and the same answer or error where it declines one."""
import numpy as np
import pytest

from paper_2008_11326_amd import inputs as I
from tests.gpu_helpers import to_device

pytestmark = pytest.mark.gpu

DIMS = I.Dims(7, 2, 130, 5, 3)


class Declines:
    """A native side that declines every call."""

    def __getattr__(self, name):
        return lambda *a: None


@pytest.fixture(scope="module")
def gpp():
    import paper_2008_11326_amd as gpp
    return gpp


@pytest.fixture()
def both(monkeypatch):
    """fn() with the native side, then without it."""
    from paper_2008_11326_amd import _lib

    def run(fn):
        got = fn()
        with monkeypatch.context() as m:
            m.setattr(_lib, "native", lambda: Declines())
            ref = fn()
        return got, ref
    return run


@pytest.fixture(scope="module")
def state():
    return to_device(I.make_problem(DIMS, 71))


def _equal(got, ref):
    assert type(got) is type(ref) and len(got) == len(ref)
    for a, b in zip(got, ref):
        if b is None:
            assert a is None
        else:
            assert a.dtype == b.dtype and a.shape == b.shape
            assert np.array_equal(a.cpu().numpy(), b.cpu().numpy())


def _upstream(torch):
    z = [torch.from_numpy(g).to("cuda:0") for g in
         I.make_upstream_grad(3, np.random.default_rng(5))]
    return dict(grad_achtemp=z[0], grad_asxtemp=z[1])


@pytest.mark.parametrize("call", ["fwd", "fwd_param", "fwd_kept", "noalloc", "qp", "qp_kept",
                                  "bwd", "bwd_some", "batched", "batched_tuples"])
def test_same_results(gpp, both, state, call):
    import torch
    dev = torch.device("cuda:0")
    c = lambda *sh: torch.empty(sh, dtype=torch.complex128, device=dev)
    byte = lambda n: torch.empty(n, dtype=torch.uint8, device=dev)
    fwd_ws = byte(gpp.fwd_workspace_bytes(*DIMS.as_tuple()))
    plan = gpp.Plan([DIMS.as_tuple()] * 3)
    param = dict(state, aqsntemp=torch.nn.Parameter(state["aqsntemp"]))
    fn = {
        "fwd": lambda: gpp.sigma_fwd(**state, nvband=2),
        "fwd_param": lambda: gpp.sigma_fwd(**param, nvband=np.int64(2)),
        "fwd_kept": lambda: gpp.sigma_fwd(**state, nvband=2, out=(c(3), c(3)), workspace=fwd_ws,
                                          stream=torch.cuda.current_stream().cuda_stream),
        "noalloc": lambda: gpp.sigma_fwd_noalloc(**state, nvband=2, out=[c(3), c(3)]),
        "qp": lambda: gpp.sigma_qp(**state, nvband=2, freq_step=0.5),
        "qp_kept": lambda: gpp.sigma_qp(
            **state, nvband=2, freq_step=0.5, energy=0.25, vxc=1, workspace=fwd_ws,
            out=(c(3), c(3), torch.empty(6, dtype=torch.float64, device=dev))),
        "bwd": lambda: gpp.sigma_bwd(**state, nvband=2, **_upstream(torch)),
        "bwd_some": lambda: gpp.sigma_bwd(**state, nvband=2, **_upstream(torch),
                                          want=(False, True, True, False)),
        "batched": lambda: gpp.sigma_batched(plan, [state] * 3),
        "batched_tuples": lambda: gpp.sigma_batched(
            plan, tuple(tuple(state.values()) for _ in range(3)), out=(c(3, 3), c(3, 3))),
    }[call]
    _equal(*both(fn))
    plan.close()


def test_outputs_come_back_as_passed(gpp, state):
    import torch
    out = tuple(torch.empty(3, dtype=torch.complex128, device="cuda:0") for _ in range(2))
    got = gpp.sigma_fwd(**state, nvband=2, out=out)
    assert got[0] is out[0] and got[1] is out[1]


@pytest.mark.parametrize("key", ["aqsmtemp", "aqsntemp", "I_eps_array", "wtilde_array", "vcoul",
                                 "wx_array"])
@pytest.mark.parametrize("change", ["type", "device", "shape", "strides", "conj", "none"])
def test_declined_inputs_meet_the_checks(gpp, both, state, key, change):
    """Every input that is not the plain case is refused as by the checks
    alone: same exception type, same message."""
    import torch
    t = state[key]
    bad = {"type": lambda: t.to(torch.complex64 if t.is_complex() else torch.float32),
           "device": lambda: t.cpu(),
           "shape": lambda: t[..., :-1].contiguous(),
           "strides": lambda: t.repeat_interleave(2, dim=-1)[..., ::2],
           "conj": lambda: t.conj() if t.is_complex() else t[None],
           "none": lambda: None}[change]()
    args = dict(state, **{key: bad})

    def fn():
        try:
            return gpp.sigma_fwd(**args, nvband=2)
        except Exception as e:  # noqa: BLE001 -- compared below
            return type(e), str(e)
    got, ref = both(fn)
    assert isinstance(ref[0], type), "the checks accept this input"
    assert got == ref


def test_library_errors_and_mismatched_states(gpp, both, state):
    import torch
    plan = gpp.Plan([DIMS.as_tuple(), (7, 2, 130, 4, 3)])
    small = torch.empty(16, dtype=torch.uint8, device="cuda:0")

    def err(fn):
        def go():
            with pytest.raises(Exception) as e:
                fn()
            return e.type, str(e.value)
        return go
    for fn in (lambda: gpp.sigma_fwd(**state, nvband=9),
               lambda: gpp.sigma_fwd(**state, nvband=2, workspace=small),
               lambda: gpp.sigma_qp(**state, nvband=2, freq_step=-0.5),
               lambda: gpp.sigma_batched(plan, [state, state]),
               lambda: gpp.sigma_batched(plan, [state])):
        got, ref = both(err(fn))
        assert got == ref
    plan.close()
