"""Small products beside the reductions on 64 x 64 tiles, two workgroups per compute unit: launches of more workgroups than compute units, K loops of the products on
either side of a stage, items of one K tile of 32 tokens and less, and of many, against the float64 oracle."""
import pytest

from paper_2502_20168_amd import binding as ssm
from paper_2502_20168_amd import workloads as wl
from tests.parity_util import check_workload

pytestmark = pytest.mark.gpu

SHAPES = [
    # Bt, L, H, P
    (8, 250, 180, 180), (20, 64, 300, 300),                # 272 to 340 workgroups
    (2, 65, 128, 64), (2, 65, 129, 65), (3, 50, 260, 130),   # products of K = 128, one more, and of more than two stages
    (1, 31, 70, 40), (1, 32, 64, 64), (1, 33, 66, 34),       # fewer tokens than a K tile, one, one more
    (8, 1000, 128, 256),                                   # items of 1000 tokens
    (3, 100, 1000, 1000),                                  # tiles in three columns and more, one slab
    # one workgroup per compute unit, K tiles of 64 tokens: fewer, one more and a half, contractions at the line and beside it, a round of items and one of tiles
    (1, 31, 460, 256), (1, 65, 448, 224), (3, 32, 447, 223), (5, 97, 513, 30), (2, 100, 1024, 512), (32, 250, 128, 225),
]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_small_pairs(shape):
    Bt, L, H, P = shape
    print(shape, flush=True)
    check_workload(wl.custom("pairs", Bt, L, H, P, p_reset=0.03, with_x0=True, seed=23), backward=True)


def test_slabs_are_as_accurate_as_exact_products_summed_in_32_bits():
    """dB and dC of bare products (Abar = 0).  With every product exact, the sum of a slab of 250 tokens is rounded once per 16 of them, 16 times at most, and
    that of eight slabs seven times: 23 roundings of at most 2^-24 of a partial sum, 1.4e-6 at the worst; an average of 2^-25 sqrt(23) = 1.4e-7, of which twice
    is allowed, besides the operands' own error (chi and x are rounded products of 180 terms: 2e-7)."""
    import numpy as np
    from oracle import ssm_oracle as orc
    from tests.parity_util import rel_errors, run_gpu
    inp = wl.gen_inputs(wl.custom("bare", 8, 250, 180, 180, seed=29))
    inp["Lambda"] = np.full(180, -50.0 + 1.0j, np.complex64)
    inp["log_delta"] = np.full(180, 10.0, np.float32)       # Abar underflows to zero
    ref, got = orc.run_workload(inp, True), run_gpu(inp, True)
    errs = {k: rel_errors(got[k], ref[k])[0] for k in ("dB", "dC")}
    print(errs, flush=True)
    assert max(errs.values()) <= 2 * 1.4e-7 + 2e-7, errs
