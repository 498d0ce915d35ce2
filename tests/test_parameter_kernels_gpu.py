"""The parameter kernels (weights and magnitudes before the products, sums and adjoints behind them) at the sizes where their
splits can go wrong, forward and gradient pass against the float64 oracle."""
import pytest

from paper_2502_20168_amd import workloads as wl
from tests.parity_util import check_workload

pytestmark = pytest.mark.gpu

EPILOGUE = [
    # Bt, L, H, P: threads that share out a row (H for dB, 2 P for dC), four columns each, and what is left of the last one
    (1, 70, 1, 1),         # fewer than four columns
    (1, 70, 3, 2),
    (2, 40, 63, 33),       # 16 threads and 16 groups, one column short and two over
    (2, 40, 64, 32),
    (2, 40, 65, 31),
    (1, 130, 129, 63),
    (3, 33, 255, 129),     # 64 and 128 threads
    (3, 33, 257, 127),
    (2, 20, 1023, 514),    # a single group, one and two rounds
    (2, 20, 1025, 513),
    (64, 100, 16, 8),      # many slabs of a small matrix
    (300, 20, 8, 5),       # more partial rows of dAbar than threads
]

PREP = [
    # Bt, L, H, P: column dots and magnitudes of the gradient pass, rows of a slab and columns of a block
    (1, 17, 62, 3),        # three planes: one step and a row, two columns left over
    (5, 79, 67, 12),       # several slabs, the last one short
    (24, 128, 3, 512),     # two planes: fewer than four columns
    (8, 1024, 61, 512),    # one column left over
    (24, 128, 66, 512),    # a second block of two columns
    (40, 100, 515, 513),   # separate scans, ragged widths
    (131, 128, 68, 512),   # slabs of 262 rows: a round of loads and six rows
    (4, 256, 1100, 1040),  # K longer than a packing thread keeps in registers, more states than a batch
]


@pytest.mark.parametrize("shape", PREP, ids=["x".join(map(str, s)) for s in PREP])
def test_launch_in_front_of_the_products(shape):
    print(shape, flush=True)
    check_workload(wl.custom("prep", *shape, p_reset=0.02, with_x0=True, seed=19), backward=True)


@pytest.mark.parametrize("shape", EPILOGUE, ids=["x".join(map(str, s)) for s in EPILOGUE])
def test_sums_behind_the_products(shape):
    print(shape, flush=True)
    check_workload(wl.custom("epilogue", *shape, p_reset=0.05, with_x0=True, seed=17), backward=True)
