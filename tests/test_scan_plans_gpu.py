"""The scan kernels at the edges of plan_scan: whole sequences per workgroup and look-backs over blocks of 256, 512 and 1024 steps,
lanes and chunks that leave a wavefront partly empty, against the float64 recurrence."""
import numpy as np
import pytest

from oracle import ssm_oracle as orc
from paper_2502_20168_amd import binding as ssm
from paper_2502_20168_amd import workloads as wl
from tests.parity_util import TOL_FWD, TOL_GRAD, assert_close, check_workload

pytestmark = pytest.mark.gpu

SHAPES = [
    # Bt, L, P
    (3, 1, 5), (2, 15, 300), (2, 17, 129), (1, 33, 260), (5, 80, 31), (3, 200, 17),    # up to 256 steps: 256 .. 16 states
    (2, 256, 16), (2, 257, 15), (3, 300, 33), (1, 512, 40),                         # whole sequences of 16 states
    (2, 513, 40), (16, 513, 60), (7, 1000, 150), (64, 1024, 9),                       # up to 1024 steps: look-back or whole
    (17, 600, 250), (19, 1000, 256), (49, 1024, 250), (32, 1000, 250),                # more than 256 such workgroups: look-back, the last one whole
    (1, 1025, 20), (2, 5000, 70),                                                     # blocks of 256 steps
    (16, 2040, 64), (2, 20000, 64),                                                   # of 512
    (4, 4000, 250), (1, 60000, 60), (4, 4096, 256),                                   # of 1024
    (12, 2050, 250), (20, 1300, 350),                                                 # of 256 again: many of them
    (3, 3000, 935), (40, 230, 930),                                                   # more than 64 MiB in rows of no whole lines: stores left in the L2
]


def _inputs(Bt, L, P, pr):
    rng = np.random.default_rng(L * 31 + P)
    c = lambda *s: (rng.normal(size=s) + 1j * rng.normal(size=s)).astype(np.complex64)
    Abar = (rng.uniform(0.9, 1.0, P) * np.exp(1j * rng.uniform(0, np.pi, P))).astype(np.complex64)
    return Abar, c(Bt, L, P), c(Bt, L, P), (rng.random((Bt, L)) < pr).astype(np.uint8), c(Bt, P)


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("pr", [0.0, 0.01])
def test_scan_plans(shape, pr):
    import torch
    print(shape, pr, flush=True)
    Bt, L, P = shape
    Abar, v, gx, fl, x0 = _inputs(*shape, pr)
    dA, dv, dg, dfl, dx0 = (torch.from_numpy(a).cuda() for a in (Abar, v, gx, fl, x0))
    x_ref = orc.scan(Abar, v, fl, x0)
    ws = ssm.alloc_workspace(Bt, L, 1, P, True)
    x, xl = ssm.ssm_scan_states(dA, dv, dfl, dx0)
    xs = x_ref.astype(np.complex64)
    chi, dAb, dx = ssm.ssm_scan_states_reverse(dA, dg, torch.from_numpy(xs).cuda(), dfl, dx0, workspace=ws)
    assert ssm.ssm_workspace_status(ws) == ssm.SSM_OK
    assert_close(x.cpu().numpy(), x_ref, TOL_FWD, "x")
    assert_close(xl.cpu().numpy(), x_ref[:, -1], TOL_FWD, "x_last")
    shift = np.zeros_like(fl)
    shift[:, :-1] = fl[:, 1:]                         # the flag of step t+1 cuts the flow into step t
    chi_ref = orc.scan(np.conj(Abar), gx[:, ::-1], shift[:, ::-1])[:, ::-1]
    prev = np.concatenate([x0[:, None, :], xs[:, :-1]], 1).astype(np.complex128)
    assert_close(chi.cpu().numpy(), chi_ref, TOL_FWD, "chi")
    assert_close(dAb.cpu().numpy(), np.sum((1 - fl)[:, :, None] * np.conj(prev) * chi_ref, axis=(0, 1)), TOL_GRAD, "dA_bar")
    assert_close(dx.cpu().numpy(), (1 - fl[:, 0])[:, None] * np.conj(Abar.astype(np.complex128)) * chi_ref[:, 0], TOL_GRAD, "dx0")


# (the forward scan runs in the input projection, up to 4096 steps; longer ones: a scan kernel of several workgroups along time either way)
@pytest.mark.parametrize("shape", [(14, 300, 512, 512), (9, 515, 520, 512), (5, 1500, 512, 512), (5, 1030, 512, 530), (2, 4100, 512, 520), (1, 5003, 530, 512),
                                   (17, 1000, 512, 530), (4, 4200, 512, 530)], ids=str)      # (states past 64 MiB: left in the L2)
def test_scans_that_record_magnitudes(shape):
    """Two planes: the row maxima that the scan kernels (and the forward scan in its product) record scale the products behind them."""
    Bt, L, H, P = shape
    p = ssm.ssm_plan_describe(Bt, L, H, P)
    assert p["planes"] == 2 and p["scans_in_projections"] == 0
    check_workload(wl.custom("maxima", Bt, L, H, P, p_reset=0.01, with_x0=True, seed=29), backward=True)


def test_a_wait_over_blocks_of_1024_steps_gives_up():
    """With no polls every look-back ends at once: reported, and NaN in what depends on it, or right because nobody had to wait."""
    import torch
    Abar, v, _, fl, x0 = _inputs(4, 4000, 250, 0.0)
    dA, dv, dx0 = (torch.from_numpy(a).cuda() for a in (Abar, v, x0))
    ws = ssm.alloc_workspace(4, 4000, 1, 250, False)
    old = ssm.ssm_set_spin_limit(0)
    try:
        x, _ = ssm.ssm_scan_states(dA, dv.clone(), None, dx0, workspace=ws)
        status = ssm.ssm_workspace_status(ws)
    finally:
        ssm.ssm_set_spin_limit(old)
    assert status in (ssm.SSM_OK, ssm.SSM_ERR_SCAN_TIMEOUT)
    if status == ssm.SSM_OK:
        assert_close(x.cpu().numpy(), orc.scan(Abar, v, fl, x0), TOL_FWD, "x")
    else:
        assert bool(torch.isnan(x.real).any())
    x, _ = ssm.ssm_scan_states(dA, dv, None, dx0, workspace=ws)
    assert ssm.ssm_workspace_status(ws) == ssm.SSM_OK and not bool(torch.isnan(x.real).any())
