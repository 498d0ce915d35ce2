"""The forward pass of narrow layers in one launch, at the edges of its tiles and of the rule that chooses it, against the float64 oracle."""
import pytest

from paper_2502_20168_amd import binding as ssm
from paper_2502_20168_amd import workloads as wl
from tests.parity_util import check_workload

pytestmark = pytest.mark.gpu

SHAPES = [
    # Bt, L, H, P
    (1, 1, 4, 2),                                          # the fewest columns and states, one token
    (2, 64, 32, 32), (3, 63, 31, 30), (5, 33, 33, 33),       # full tiles, one row and column less, one more
    (9, 21, 64, 64), (9, 64, 64, 5), (9, 64, 6, 64), (7, 13, 61, 63),    # every pair of tile widths; several sequences per tile
    (64, 1, 40, 20), (65, 1, 40, 20),                        # sequences of one step
    (513, 64, 16, 8), (512, 64, 16, 8), (4, 65, 32, 32), (4, 64, 65, 32), (4, 64, 32, 65), (4, 64, 3, 32), (4, 64, 32, 1),    # either side of the rule
]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("resets,x0", [(0.0, True), (0.1, True), (0.1, False), (1.0, True)])
def test_narrow_layers(shape, resets, x0):
    Bt, L, H, P = shape
    print(shape, resets, x0, flush=True)
    check_workload(wl.custom("narrow", Bt, L, H, P, p_reset=resets, force_first=False, with_x0=x0, seed=17), backward=True)


def test_optional_outputs_and_neighbours():
    """Without the states the outputs are the same to the last bit, and what one sequence holds does not reach its neighbours in the tile."""
    import torch
    a = ssm.to_device(wl.gen_inputs(wl.custom("n", 6, 20, 48, 40, p_reset=0.0, with_x0=True, seed=3)))
    par = (a["Lambda"], a["B"], a["C"], a["D"], a["log_delta"])
    f = ssm.ssm_scan_fwd(*par, a["u"], None, a["x0"])
    g = ssm.ssm_scan_fwd(*par, a["u"], None, a["x0"], want_x=False)
    assert torch.equal(f["y"], g["y"]) and torch.equal(f["x_last"], g["x_last"])
    u = a["u"].clone()
    u[1] = float("nan")
    h = ssm.ssm_scan_fwd(*par, u, None, a["x0"])
    others = [0, 2, 3, 4, 5]
    assert all(torch.equal(h[k][others], f[k][others]) for k in ("y", "x", "x_last")) and torch.isnan(h["y"][1]).all()
