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
