"""The products with packed weights at the sizes where their tiles, chains and packing jobs can go wrong, both passes
against the float64 oracle."""
import pytest

from paper_2502_20168_amd import binding as ssm
from paper_2502_20168_amd import workloads as wl
from tests.parity_util import check_workload

pytestmark = pytest.mark.gpu

SHAPES = [
    # Bt, L, H, P
    (1, 3, 2, 1),          # fewer than four values along every dimension
    (3, 37, 33, 17),       # odd widths: every row, column and K tail
    (2, 65, 127, 65),      # one past a tile in rows and columns
    (5, 77, 96, 40),       # 32-row tiles, columns narrower than a tile
    (16, 64, 256, 256),    # k shared between consumers, reductions beside small products
    (1, 24, 20, 1030),     # more states than a packing job's batch and register rounds
    (1, 24, 1100, 12),     # the same for H
    (90, 100, 40, 70),     # 32 x 64 tiles at many rows: at most 64 columns
    (20, 300, 500, 250),   # 64-row tiles of three planes, ragged
    (24, 200, 1024, 512),  # two planes, separate scans, 128-row tiles beside the reductions
    (8, 128, 96, 512),     # 64-row scanning tiles, chain of two
    (1, 4096, 40, 130),    # 64-row scanning tiles, longest chain, last column tile nearly empty
    (24, 128, 64, 512),    # 128-row scanning tiles forward, 64-row ones in reverse: the smallest such batch
    (48, 128, 40, 512),    # 128-row scanning tiles in reverse: the smallest such batch
    (64, 128, 64, 520),    # 128-row scanning tiles without a chain
    (20, 640, 64, 330),    # 128-row scanning tiles, ten units: more than one run
    (256, 32, 64, 512),    # 128-row scanning tiles of whole sequences
    (128, 64, 64, 512),
    (512, 16, 40, 512),
    (16, 16, 512, 4096),   # 64-row scanning tiles of whole sequences
]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
@pytest.mark.parametrize("resets", [0.0, 0.05])
def test_products(shape, resets):
    Bt, L, H, P = shape
    print(shape, resets, flush=True)
    check_workload(wl.custom("products", Bt, L, H, P, p_reset=resets, force_first=bool(resets), with_x0=True, seed=11), backward=True)


def test_few_tokens_of_the_widest_layers():
    """Two planes without a scan in the tile, at fewer tokens than a tile has rows: only layers this wide get there."""
    p = ssm.ssm_plan_describe(3, 11, 8200, 4100)
    assert p["planes"] == 2 and p["scans_in_projections"] == 0 and p["tile_in"] == 1024 * 64 + 128
    check_workload(wl.custom("wide", 3, 11, 8200, 4100, p_reset=0.05, with_x0=True, seed=13), backward=False)


def test_states_do_not_depend_on_the_tile_of_the_launch():
    """6 x 640 tokens scan in 64-row tiles, 40 x 640 in 128-row ones: the same sequences have the same states to the last bit."""
    import torch
    a = ssm.to_device(wl.gen_inputs(wl.custom("rows", 6, 640, 64, 330, p_reset=0.01, with_x0=True, seed=5)))
    par = (a["Lambda"], a["B"], a["C"], a["D"], a["log_delta"])
    rep = lambda t: torch.cat([t] * 7)[:40].contiguous()
    small = ssm.ssm_scan_fwd(*par, a["u"], a["is_first"], a["x0"])
    big = ssm.ssm_scan_fwd(*par, rep(a["u"]), rep(a["is_first"]), rep(a["x0"]))
    gs = ssm.ssm_scan_bwd(*par, a["u"], a["is_first"], a["x0"], small["x"], a["dy"])
    gb = ssm.ssm_scan_bwd(*par, rep(a["u"]), rep(a["is_first"]), rep(a["x0"]), big["x"], rep(a["dy"]))
    for k in ("x", "x_last"):
        assert torch.equal(big[k][:6], small[k]) and torch.equal(big[k][6:12], small[k]), k
    assert torch.equal(gb["dx0"][:6], gs["dx0"]) and torch.equal(gb["dx0"][6:12], gs["dx0"])
