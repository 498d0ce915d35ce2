"""Host logic that decides what a call launches (no GPU needed): which shapes scan inside the projections,
how many planes, the tiles, K slabs of the reductions and which work items go first.  The decisions are
read back through ssm_plan_describe (include/ssm_measure.h); the expectations are the rules the design
states, evaluated here independently in Python."""
from fractions import Fraction

import pytest

from paper_2502_20168_amd import binding as ssm
from paper_2502_20168_amd import workloads as wl


TILES = ("tile_in", "tile_out", "tile_du")


def _tile(plan, name):
    return divmod(plan[name], 1024)


def _ceil(x, y):
    return -(-x // y)


def test_benchmark_configurations_take_the_paths_the_design_states():
    plans = [ssm.ssm_plan_describe(w.Bt, w.L, w.H, w.P) for w in wl.CONFIGS]
    assert [p["scans_in_projections"] for p in plans] == [0, 0, 1, 1, 1]
    assert [p["planes"] for p in plans] == [3, 3, 2, 2, 2]
    assert [p["products_per_gradient_launch"] for p in plans] == [2, 2, 3, 3, 3]
    # the benchmark shape: four slabs per reduction, in front of du
    assert plans[2]["slabs_dC"] == 4 and plans[2]["slabs_dBbar"] == 4 and plans[2]["slabs_first"] == 1
    assert [_tile(plans[2], k) for k in TILES] == [(128, 128), (64, 128), (64, 128)]
    # 1024 x 16 tokens: the same
    assert plans[4]["slabs_dC"] == 4 and plans[4]["slabs_first"] == 1
    # the small configurations run everything on tiles of 32 rows
    assert all(_tile(p, k)[0] == 32 for p in plans[:2] for k in TILES)


def _expected_tile(T, N, planes, items=0):
    """Rows and columns of the tile of a T x N product without a scan beside `items` work items of reductions."""
    tiles = lambda rows, cols: _ceil(T, rows) * _ceil(N, cols)
    if planes == 3 and N <= 64 and tiles(64, 128) > 128 and items == 0:
        return 32, 64
    if tiles(64, 128) <= 128 and (planes == 3 or items == 0):
        return 32, 128 if tiles(32, 64) + items > 256 else 64 if tiles(32, 32) + items > 128 else 32
    fits = items > 0 and tiles(64, 128) + items > 576 and tiles(128, 128) + items <= 512
    return 128 if planes == 2 and (tiles(128, 128) >= 512 or fits) else 64, 128


@pytest.mark.parametrize("Bt,L,H,P", [(30, 100, 512, 512), (64, 100, 512, 512), (18, 100, 1024, 512), (8, 100, 256, 256),
                                      (16, 1000, 256, 256), (5, 77, 96, 40), (100, 100, 256, 128), (40, 100, 512, 512), (1, 3, 2, 1),
                                      (16, 256, 512, 512), (24, 128, 1024, 512), (64, 128, 64, 256), (128, 256, 512, 512), (256, 16, 96, 512), (300, 100, 40, 70)])
def test_reported_tiles_are_those_of_the_launches(Bt, L, H, P):
    T = Bt * L
    p = ssm.ssm_plan_describe(Bt, L, H, P)
    red = lambda M, N, s, t: _ceil(M, t[0]) * _ceil(N, t[1]) * s
    small = _ceil(T, 128) * _ceil(H, 128) <= 64
    t = (128, 128) if p["planes"] == 2 else (64, 64) if small else (128, 64)
    items = red(2 * P, H, p["slabs_dBbar"], t)
    if p["scans_in_projections"]:
        items += red(H, 2 * P, p["slabs_dC"], t)
        rows = 128 if T // 128 * _ceil(2 * P, 128) >= (192 if L >= 64 else 512) else 64
        assert _tile(p, "tile_in") == (rows, 128)
    elif p["planes"] == 3:
        assert _tile(p, "tile_in") == _expected_tile(T, 2 * P, 3)
    assert _tile(p, "tile_out") == _expected_tile(T, H, p["planes"])
    assert _tile(p, "tile_du") == _expected_tile(T, H, p["planes"], items)


COUNTS = (1, 2, 3, 4, 5, 8, 12, 16, 24, 32, 40, 48, 56, 64)


def _slabs(tiles, T, small=False, fit=None):
    """The count whose number of work items is nearest, in ratio, to 224 (128 beside small products); one two-plane reduction
    beside a product of `fit` columns: at most the largest that leaves 160 items and makes room for 128-row tiles."""
    want, rows = (128, 64) if small else (224, 192)
    allowed = [s for s in COUNTS if s == 1 or T // s >= rows]
    nearest = min(allowed, key=lambda s: (max(Fraction(tiles * s, want), Fraction(want, tiles * s)), s))
    fits = [s for s in allowed if fit and s > 1 and tiles * s >= 160 and _ceil(T, 128) * _ceil(fit, 128) + tiles * s <= 512
            and _ceil(T, 64) * _ceil(fit, 128) + tiles * s > 576]
    return min([nearest] + fits[-1:])


@pytest.mark.parametrize("Bt,L,H,P", [(16, 256, 512, 512), (4, 4096, 256, 256), (1024, 16, 512, 512), (32, 128, 1024, 512),
                                      (256, 64, 256, 256), (8, 1024, 512, 512), (24, 128, 1024, 512), (32, 128, 512, 256), (4, 128, 1024, 1024),
                                      (64, 128, 64, 70)])
def test_slabs_of_the_three_product_launch(Bt, L, H, P):
    T = Bt * L
    p = ssm.ssm_plan_describe(Bt, L, H, P)
    assert p["products_per_gradient_launch"] == 3 and p["scans_in_projections"] == 1
    s = _slabs(2 * _ceil(2 * P, 128) * _ceil(H, 128), T)
    assert p["slabs_dC"] == s and p["slabs_dBbar"] == s
    assert p["slabs_first"] == 1


@pytest.mark.parametrize("Bt,L,H,P", [(64, 100, 512, 512), (16, 1000, 256, 256), (24, 200, 1024, 512), (20, 300, 512, 256),
                                      (10, 1000, 512, 512), (40, 200, 768, 384), (40, 100, 256, 256), (16, 64, 256, 256), (1, 256, 1024, 1024),
                                      (48, 100, 512, 512), (100, 100, 512, 1024),
                                      (8, 128, 64, 256), (5, 77, 96, 40), (1, 3, 2, 1)])
def test_slabs_and_order_of_the_two_product_launches(Bt, L, H, P):
    T = Bt * L
    p = ssm.ssm_plan_describe(Bt, L, H, P)
    assert p["products_per_gradient_launch"] == 2 and p["scans_in_projections"] == 0
    for M, N, K, slabs, first in ((H, 2 * P, H, "slabs_dC", "dC_first"), (2 * P, H, 2 * P, "slabs_dBbar", "dBbar_first")):
        # beside a product of T x N with a K loop of K
        small = _ceil(T, 128) * _ceil(N, 128) <= 64
        tile = (128, 128) if p["planes"] == 2 else (64, 64) if small else (128, 64)
        s = _slabs(_ceil(M, tile[0]) * _ceil(N, tile[1]), T, small, N if p["planes"] == 2 else None)
        assert p[slabs] == s
        assert p[first] == int(not small or _ceil(T, s) > K)


def test_every_plan_is_bounded_and_repeatable():
    import numpy as np
    rng = np.random.Generator(np.random.PCG64(123))
    for _ in range(300):
        Bt, L = int(rng.integers(1, 600)), int(rng.choice([1, 16, 64, 100, 128, 256, 300, 1000, 4096]))
        H, P = int(rng.choice([3, 32, 96, 256, 512, 1024])), int(rng.choice([1, 40, 128, 256, 512]))
        a, b = ssm.ssm_plan_describe(Bt, L, H, P), ssm.ssm_plan_describe(Bt, L, H, P)
        assert a == b
        for k in ("slabs_dC", "slabs_dBbar"):
            assert 1 <= a[k] <= 64 and (a[k] == 1 or -(-Bt * L // a[k]) >= 64)       # a slab keeps at least one K step of 64
        assert a["planes"] in (2, 3) and all(_tile(a, k) in ((32, 32), (32, 64), (32, 128), (64, 128), (128, 128)) for k in TILES)
        assert ssm.ssm_workspace_bytes(Bt, L, H, P, True) > 0 and ssm.ssm_workspace_bytes(Bt, L, H, P, False) > 0


def test_plan_rejects_what_the_library_rejects():
    with pytest.raises(ssm.SsmError):
        ssm.ssm_plan_describe(0, 16, 8, 8)
    with pytest.raises(ssm.SsmError):
        ssm.ssm_plan_describe(1, 16, 1 << 20, 8)


def test_the_binding_loads_torch_before_the_library():
    """A host-only call (no GPU work) must not bind the library to the system's copy of the HIP runtime: torch
    brings its own, and with two copies in the process every later launch on torch's memory fails.  In a fresh
    interpreter, a plan query before any `import torch` leaves torch loaded first."""
    import os, subprocess, sys
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    code = ("import sys; sys.path.insert(0, %r)\n"
            "from paper_2502_20168_amd import binding as ssm\n"
            "assert 'torch' not in sys.modules\n"
            "print(ssm.ssm_plan_describe(16, 256, 512, 512)['planes'])\n"
            "assert 'torch' in sys.modules\n" % root)
    out = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, timeout=300)
    assert out.returncode == 0, out.stderr
    assert out.stdout.strip().splitlines()[-1] == "2"


@pytest.mark.parametrize("Bt,L,H,P", [(238, 1371, 1080, 970), (101, 4072, 662, 736), (207, 3228, 648, 1018), (24, 200, 1024, 512), (20, 300, 500, 250)])
def test_a_workspace_of_the_gradient_pass_holds_the_forward_pass(Bt, L, H, P):
    assert ssm.ssm_workspace_bytes(Bt, L, H, P, False) <= ssm.ssm_workspace_bytes(Bt, L, H, P, True)


@pytest.mark.parametrize("long,short", [((1, 4, 6, 124), (1, 3, 6, 124)), ((3, 4, 286, 5), (3, 3, 286, 5)), ((2, 32, 64, 64), (2, 31, 64, 64)),
                                        ((4, 64, 40, 300), (4, 63, 40, 300)), ((500, 16, 200, 200), (500, 13, 200, 200))])
def test_a_workspace_holds_shorter_sequences_as_well(long, short):
    """Also where the longer ones fill whole tiles, whose rows hand nothing over."""
    for bwd in (False, True):
        assert ssm.ssm_workspace_bytes(*short, bwd) <= ssm.ssm_workspace_bytes(*long, bwd)
        assert ssm.ssm_block_workspace_bytes(*short, bwd) <= ssm.ssm_block_workspace_bytes(*long, bwd)
