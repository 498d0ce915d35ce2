"""The two halves of the Python binding: the native one makes the call, the general one names what is wrong."""
import pytest


def _small(device):
    import torch
    Bt, L, H, P = 2, 8, 4, 3
    c = lambda *s: torch.randn(s, dtype=torch.complex64, device=device)
    f = lambda *s: torch.randn(s, device=device)
    return {"Lambda": -torch.rand(P, dtype=torch.float32, device=device).to(torch.complex64), "B": c(P, H), "C": c(H, P), "D": f(H),
            "log_delta": f(P) - 4, "u": f(Bt, L, H), "is_first": None, "x0": None}


def test_arguments_on_the_cpu_are_refused_by_name():
    from paper_2502_20168_amd import binding as ssm
    with pytest.raises(ValueError, match="Lambda must be a contiguous cuda tensor"):
        ssm.ssm_scan_fwd(**_small("cpu"))


@pytest.mark.gpu
@pytest.mark.parametrize("name,change", [("B", lambda t: t[:, :2]), ("D", lambda t: t.double()), ("u", lambda t: t.transpose(0, 1)),
                                         ("log_delta", lambda t: t.cpu())])
def test_a_wrong_argument_is_named(name, change):
    from paper_2502_20168_amd import binding as ssm
    a = _small("cuda")
    a[name] = change(a[name])
    with pytest.raises((ValueError, ssm.SsmError)):
        ssm.ssm_scan_fwd(**a)


@pytest.mark.gpu
def test_native_and_general_path_agree_and_honour_given_outputs_streams_and_workspaces():
    import torch
    from paper_2502_20168_amd import binding as ssm
    a = _small("cuda")
    ref = ssm.ssm_scan_fwd(**a, profile=True)                    # always the general path
    got = ssm.ssm_scan_fwd(**a)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    out = {"y": torch.empty_like(a["u"])}
    ws = ssm.alloc_workspace(2, 8, 4, 3, False)
    with_stream = ssm.ssm_scan_fwd(**a, out=out, workspace=ws, stream=side)
    own_workspace = ssm.ssm_scan_fwd(**a, stream=side, want_x=False, want_x_last=False)
    torch.cuda.synchronize()
    assert with_stream["y"] is out["y"] and own_workspace["x"] is None and own_workspace["x_last"] is None
    for k in ("y", "x", "x_last"):
        assert torch.equal(got[k], ref[k]) and torch.equal(with_stream[k], ref[k])
    assert torch.equal(own_workspace["y"], ref["y"])
    with pytest.raises(ssm.SsmError) as e:
        ssm.ssm_scan_fwd(**a, workspace=ws[:256])
    assert e.value.code == ssm.SSM_ERR_WORKSPACE


BATCHED = r"""
import sys, types, warnings
sys.path.insert(0, %r)
import torch
from torch._subclasses.fake_tensor import FakeTensorMode
from paper_2502_20168_amd import binding as ssm
warnings.simplefilter("ignore")
Bt, L, H, P, T = 2, 8, 4, 3, 5
with FakeTensorMode(allow_non_fake_inputs=True):
    c = lambda *s: torch.empty(s, dtype=torch.complex64, device="cuda")
    f = lambda *s: torch.empty(s, device="cuda")
    par = [c(P), c(P, H), c(H, P), f(H), f(P)]
    ws = torch.empty(1 << 20, dtype=torch.uint8, device="cuda")
    k = {"workspace": ws, "stream": types.SimpleNamespace(cuda_stream=0)}
    grads = {"du": f(Bt, L, H), "dLambda": c(P), "dB": c(P, H), "dC": c(H, P), "dD": f(H), "dlog_delta": f(P), "dx0": c(Bt, P)}
    calls = {
        "scan_fwd": (f(7, Bt, L, H), lambda u: ssm.ssm_scan_fwd(*par, u, out={"y": f(Bt, L, H), "x": c(Bt, L, P), "x_last": c(Bt, P)}, **k)),
        "scan_bwd": (f(7, Bt, L, H), lambda dy: ssm.ssm_scan_bwd(*par, f(Bt, L, H), None, None, c(Bt, L, P), dy, out=grads, **k)),
        "step": (f(7, Bt, H), lambda u: ssm.ssm_step(ws, par[3], u, P=P, x=c(Bt, P), y=f(Bt, H), stream=k["stream"])),
        "lambda_return": (f(7, T, Bt), lambda r: ssm.ssm_lambda_return(r, f(T, Bt), f(T, Bt), 0.9, 0.9, ret=f(T, Bt), stream=k["stream"])),
        "scan_states": (c(7, Bt, L, P), lambda v: ssm.ssm_scan_states(par[0], v, want_x_last=False, **k)),
        "half_glu_fwd": (f(7, T, H), lambda u: ssm.ssm_half_glu_fwd(u, f(H, H), y=f(T, H), gate=f(T, H), **k)),
        "half_glu_bwd": (f(7, T, H), lambda u: ssm.ssm_half_glu_bwd(u, f(H, H), f(T, H), f(T, H), du=f(T, H), dW=f(H, H), **k)),
    }
    for name, (batch, call) in calls.items():
        print(name, flush=True)
        try:
            torch.func.vmap(call)(batch)
        except RuntimeError as e:
            assert "data pointer" in str(e), e
        else:
            raise AssertionError("not refused")
print("all refused")
"""


def test_a_tensor_without_storage_raises_and_does_not_end_the_interpreter():
    """The data pointer of a batched tensor (torch.func.vmap over a call) cannot be taken: the call raises torch's error."""
    import os, subprocess, sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", BATCHED % root], capture_output=True, text=True, timeout=300)
    assert r.returncode == 0 and r.stdout.strip().endswith("all refused"), (r.returncode, r.stdout, r.stderr[-2000:])


class _NoTruthValue:
    def __bool__(self):
        raise ValueError("neither")


def test_an_error_raised_by_an_option_is_the_callers():
    import types
    import torch
    from torch._subclasses.fake_tensor import FakeTensorMode
    from paper_2502_20168_amd import binding as ssm
    with FakeTensorMode(allow_non_fake_inputs=True):
        a = {k: None if v is None else torch.empty(v.shape, dtype=v.dtype, device="cuda") for k, v in _small("cpu").items()}
        out = {"y": torch.empty(a["u"].shape, device="cuda")}
        with pytest.raises(ValueError, match="neither"):
            ssm.ssm_scan_fwd(**a, want_x=_NoTruthValue(), out=out, workspace=out["y"], stream=types.SimpleNamespace(cuda_stream=0))


@pytest.mark.gpu
def test_an_allocation_that_fails_raises_torchs_error():
    import torch
    from paper_2502_20168_amd import binding as ssm
    r = torch.zeros(64, 1 << 20, device="cuda")                  # 256 MiB
    torch.cuda.empty_cache()
    total = torch.cuda.get_device_properties(0).total_memory
    torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (64 << 20)) / total)
    try:
        with pytest.raises(torch.OutOfMemoryError):
            ssm.ssm_lambda_return(r, r, r, 0.9, 0.9)
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)


def test_without_its_native_half_the_binding_takes_the_general_path(monkeypatch):
    import sys
    import paper_2502_20168_amd as package
    from paper_2502_20168_amd import binding as ssm
    monkeypatch.setattr(ssm, "_native", None)
    monkeypatch.delattr(package, "_ssmbind", raising=False)
    monkeypatch.setitem(sys.modules, "paper_2502_20168_amd._ssmbind", None)      # (its import raises ImportError)
    with pytest.warns(RuntimeWarning, match="native half"), pytest.raises(ValueError, match="Lambda must be a contiguous cuda tensor"):
        ssm.ssm_scan_fwd(**_small("cpu"))
    with pytest.raises(ValueError, match="Lambda must be"):      # said once; every call is served
        ssm.ssm_step_prepare(*(_small("cpu")[k] for k in ("Lambda", "B", "C", "log_delta")))
