"""The forward pass of narrow layers in one launch: the S5 block's part of it (GELU(y) stored beside y, the gate's weights packed by workgroups behind the
layer's), launches of many workgroups, and where the rule ends."""
import pytest

from paper_2502_20168_amd import binding as ssm
from paper_2502_20168_amd import workloads as wl
from tests.parity_util import check_workload
from tests.test_block_gpu import test_no_call_writes_outside_its_workspace as check_guards
from tests.test_block_gpu import test_s5_block_matches_oracle_composition as check_block

# every pair of tile widths; several sequences per workgroup and the last one partial; widths that are no multiple of a unit, of a packed group of rows, of 32
BLOCKS = [(2, 64, 32, 32), (3, 63, 31, 30), (5, 33, 33, 33), (9, 21, 64, 64), (65, 1, 40, 20), (9, 64, 6, 64), (9, 64, 64, 5), (7, 13, 61, 63), (1, 1, 4, 2)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape", BLOCKS, ids=["x".join(map(str, s)) for s in BLOCKS])
def test_narrow_blocks(shape):
    """Against the two oracles composed, and the layer's and the gate's own calls to the last bit."""
    print(shape, flush=True)
    assert ssm.ssm_plan_launches(*shape)[0] == 1
    check_block(*shape)


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(3, 63, 31, 30), (65, 1, 40, 20)], ids=str)
def test_narrow_calls_stay_inside_their_workspace(shape):
    print(shape, flush=True)
    check_guards(*shape)


# (Bt, L, H, P), launches of the forward pass: the most workgroups that the rule takes and one more; two rounds of full tiles
EDGES = [((512, 63, 16, 8), 1), ((513, 63, 16, 8), 4), ((2560, 12, 8, 8), 1), ((2561, 12, 8, 8), 4), ((300, 50, 64, 64), 1), ((300, 50, 33, 40), 1)]


@pytest.mark.gpu
@pytest.mark.parametrize("shape,launches", EDGES, ids=["x".join(map(str, s)) for s, _ in EDGES])
def test_many_workgroups(shape, launches):
    Bt, L, H, P = shape
    print(shape, flush=True)
    assert ssm.ssm_plan_launches(*shape)[0] == launches
    check_workload(wl.custom("narrow", Bt, L, H, P, p_reset=0.02, force_first=False, with_x0=True, seed=19), backward=True)


def test_launches_of_the_forward_pass():
    """One in a narrow layer over short sequences on three planes; the number for either pass elsewhere."""
    want = {(1, 1, 4, 2): (1, 4), (4, 64, 64, 64): (1, 4), (126, 64, 64, 64): (1, 4),
            (128, 64, 64, 64): (3, 4),                       # two planes
            (4, 65, 32, 32): (3, 4), (4, 64, 65, 32): (3, 4), (4, 64, 32, 65): (3, 4), (4, 64, 3, 32): (3, 4), (4, 64, 32, 1): (3, 4),
            (512, 63, 16, 8): (1, 5), (513, 63, 16, 8): (4, 5),
            (16, 256, 512, 512): (3, 4), (24, 200, 1024, 512): (3, 4), (1, 5000, 512, 512): (4, 5)}
    assert {s: ssm.ssm_plan_launches(*s) for s in want} == want
    with pytest.raises(ssm.SsmError):
        ssm.ssm_plan_launches(0, 16, 8, 8)
