"""C^H dy that scans its own tiles in reverse on two scaled planes (layers of at least 512 inputs and states, sequences that are no whole tiles)."""
import numpy as np
import pytest

from oracle import ssm_oracle as orc
from paper_2502_20168_amd import binding as ssm
from paper_2502_20168_amd import workloads as wl
from tests.parity_util import TOL_GRAD, rel_errors, run_gpu

pytestmark = pytest.mark.gpu

SHAPES = [(5, 1500, 512, 512), (24, 200, 1024, 512), (300, 13, 512, 530), (1, 4095, 513, 512)]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_tiles_that_wait_for_nobody(shape):
    """With no polls a tile computes the aggregates that have not been published itself, row and overall maxima are gathered once more, and every result is the
    same to the last bit."""
    import torch
    Bt, L, H, P = shape
    print(shape, flush=True)
    assert ssm.ssm_plan_describe(Bt, L, H, P)["planes"] == 2
    d = ssm.to_device(wl.gen_inputs(wl.custom("alone", Bt, L, H, P, p_reset=0.005, with_x0=True, lam_re_lo=0.001, seed=43)))
    par = [d[k] for k in ("Lambda", "B", "C", "D", "log_delta")]
    ws = ssm.alloc_workspace(Bt, L, H, P, True)
    x = ssm.ssm_scan_fwd(*par, d["u"], d["is_first"], d["x0"])["x"]

    def run():
        out = ssm.ssm_scan_bwd(*par, d["u"], d["is_first"], d["x0"], x, d["dy"], workspace=ws)
        assert ssm.ssm_workspace_status(ws) == ssm.SSM_OK
        return out

    want = run()
    old = ssm.ssm_set_spin_limit(0)
    try:
        got = run()
    finally:
        ssm.ssm_set_spin_limit(old)
    again = run()
    for k in want:
        assert torch.equal(got[k], want[k]) and torch.equal(again[k], want[k]), k


@pytest.mark.parametrize("token", [0, 63, 64, 1237, -1], ids=str)
def test_the_largest_state_sets_the_scale_wherever_it_stands(token):
    """One token's dy is 2^20 times as large as the others': were its chi not among the maxima, the planes of chi (a scale for all of it in dBbar, a scale per row
    in du) would overflow.  Rows past the last token and states past the last one: the error bounds of the other gradients hold."""
    print(token, flush=True)
    inp = wl.gen_inputs(wl.custom("spike", 31, 71, 512, 513, p_reset=0.05, with_x0=True, seed=47))
    dy = inp["dy"].reshape(31 * 71, 512)
    dy[token] *= np.float32(2 ** 20)
    ref, got = orc.run_workload(inp, True), run_gpu(inp, True)
    for k in ("du", "dB", "dx0", "dLambda", "dlog_delta"):
        e = rel_errors(got[k], ref[k])[0]
        assert e <= TOL_GRAD, (k, e)
