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


# Tiles of 32 rows: K around the short stage of 128 k, the long one of 256 and their halves, in either of the two products of a
# step (H, then 2 P), one to three groups of columns, rows that end inside a tile
STEP_SHAPES = [(5, 127, 64), (33, 128, 65), (33, 129, 64), (64, 130, 96), (31, 191, 127), (40, 192, 128), (65, 256, 130), (1, 257, 129), (2, 260, 191),
               (100, 383, 192), (96, 512, 257), (130, 515, 33), (520, 64, 60), (1024, 320, 160), (600, 1030, 40)]


@pytest.mark.parametrize("shape", STEP_SHAPES, ids=["x".join(map(str, s)) for s in STEP_SHAPES])
def test_steps_on_tiles_of_32_rows(shape):
    """Two steps and the adjoint of one against float64: sums of K products of order one, each rounded by 2^-24 of the running sum, and the
    dropped parts of the split below 2^-23 of the terms: 1e-6 of the norm leaves a factor of two or more at K = 1030."""
    import torch
    Bt, H, P = shape
    print(shape, flush=True)
    d = ssm.to_device(wl.gen_inputs(wl.custom("step", Bt, 2, H, P, p_reset=0.3, with_x0=True, seed=23)))
    plan = ssm.ssm_step_prepare(d["Lambda"], d["B"], d["C"], d["log_delta"])
    A, B = (t.to(torch.complex128) for t in ssm.ssm_discretize(d["Lambda"], d["B"], d["log_delta"]))
    C, D = d["C"].to(torch.complex128), d["D"].double()
    x, ref = d["x0"], d["x0"].to(torch.complex128)
    close = lambda got, want: float((got.to(want.dtype) - want).norm() / want.norm()) < 1e-6
    for t in range(2):
        u, first = d["u"][:, t].contiguous(), d["is_first"][:, t].contiguous()
        x, y = ssm.ssm_step(plan, d["D"], u, x, first, P=P)
        ref = u.to(torch.complex128) @ B.T.contiguous() + torch.where(first[:, None] != 0, 0.0, A[None] * ref)
        assert close(x, ref) and close(y, (ref @ C.T.contiguous()).real + D * u.double())
    dy, dx = d["dy"][:, 0].contiguous(), d["x0"]
    gx, du, dxp = ssm.ssm_step_bwd(plan, d["D"], dy, dx, first, P=P)
    g = dy.to(torch.complex128) @ C.conj().contiguous() + dx.to(torch.complex128)
    assert close(gx, g) and close(du, (g @ B.conj().contiguous()).real + D * dy.double())
    assert close(dxp, torch.where(first[:, None] != 0, 0.0, A.conj()[None] * g))


# Three planes: the projections scan the rows of their tiles: sequences that start and end anywhere in a tile, rows past the last token, one tile and
# 64 tiles per sequence (and one step more: a scan kernel), one to many column groups, several workgroups along the columns; 32-row tiles
ROW_SCANS = [(40, 1, 16, 8), (3, 5, 8, 3), (2, 31, 40, 33), (33, 33, 20, 16), (7, 61, 130, 17), (2, 64, 32, 32), (21, 97, 64, 70), (5, 512, 96, 65),
             (3, 1000, 33, 129), (1, 2047, 24, 40), (3, 2048, 20, 36), (1, 2049, 24, 40), (2, 32, 64, 1040), (64, 16, 300, 200), (13, 40, 512, 512),
             # and of 64-row ones
             (30, 100, 256, 256), (9, 997, 70, 140), (3, 4095, 36, 70), (1, 4097, 40, 100), (500, 13, 40, 100), (190, 33, 24, 300), (2001, 3, 16, 129),
             (97, 64, 40, 257), (60, 65, 33, 200), (5, 2049, 40, 33),
             # and, forward, on two planes: rows past the last token, states past the last one, many short sequences, 64 tiles and a step more
             (14, 300, 512, 512), (33, 97, 520, 577), (300, 13, 512, 530), (1, 4095, 512, 512), (1, 4097, 513, 512)]


@pytest.mark.parametrize("shape", ROW_SCANS, ids=["x".join(map(str, s)) for s in ROW_SCANS])
@pytest.mark.parametrize("resets", [0.0, 0.02, 1.0])
def test_scans_on_the_rows_of_tiles(shape, resets):
    Bt, L, H, P = shape
    print(shape, resets, flush=True)
    check_workload(wl.custom("row scans", Bt, L, H, P, p_reset=resets, with_x0=resets < 1.0, lam_re_lo=0.001, seed=31), backward=True)


def test_what_one_sequence_holds_does_not_reach_the_next_in_its_tile():
    """Two of five sequences of 13 steps (three tiles, the last one short) hold values beyond every float: the others come out as
    without them, to the last bit."""
    import torch
    d = ssm.to_device(wl.gen_inputs(wl.custom("inf", 5, 13, 24, 20, p_reset=0.05, with_x0=True, seed=37)))
    par = [d[k] for k in ("Lambda", "B", "C", "D", "log_delta")]
    bad = {k: d[k].clone() for k in ("u", "dy")}
    for k in bad:
        bad[k][1], bad[k][3] = float("inf"), 3e38
    out = []
    for e in (d, bad):
        f = ssm.ssm_scan_fwd(*par, e["u"], d["is_first"], d["x0"])
        b = ssm.ssm_scan_bwd(*par, e["u"], d["is_first"], d["x0"], f["x"], e["dy"])
        out.append([f["y"], f["x"], f["x_last"], b["du"], b["dx0"]])
    assert not bool(torch.isfinite(out[1][0][1]).any())
    for good, got in zip(*out):
        for i in (0, 2, 4):
            assert torch.equal(good[i], got[i])


@pytest.mark.parametrize("shape", [(8, 100, 256, 256), (1, 2047, 24, 40), (2, 64, 32, 32), (20, 300, 500, 250), (9, 997, 70, 140), (3, 4095, 36, 70),
                                   (5, 1500, 512, 512), (24, 200, 1024, 512)], ids=lambda s: "x".join(map(str, s)))
def test_tiles_that_wait_for_nobody(shape):
    """With no polls a tile whose predecessors have not published yet computes their aggregates itself: the same results to the last bit,
    no give-up and no NaN, on 32 and 64 rows, three planes (either direction) and two (forward; the other way a scan kernel may give up)."""
    import torch
    Bt, L, H, P = shape
    print(shape, flush=True)
    d = ssm.to_device(wl.gen_inputs(wl.custom("alone", Bt, L, H, P, p_reset=0.005, with_x0=True, lam_re_lo=0.001, seed=41)))
    par = [d[k] for k in ("Lambda", "B", "C", "D", "log_delta")]
    ws_f, ws_b = ssm.alloc_workspace(Bt, L, H, P, False), ssm.alloc_workspace(Bt, L, H, P, True)
    two_planes = ssm.ssm_plan_describe(Bt, L, H, P)["planes"] == 2

    def run():
        f = ssm.ssm_scan_fwd(*par, d["u"], d["is_first"], d["x0"], workspace=ws_f)
        out = dict(f)
        if not two_planes:
            out.update(ssm.ssm_scan_bwd(*par, d["u"], d["is_first"], d["x0"], f["x"], d["dy"], workspace=ws_b))
            assert ssm.ssm_workspace_status(ws_b) == ssm.SSM_OK
        assert ssm.ssm_workspace_status(ws_f) == ssm.SSM_OK
        return out

    want = run()
    old = ssm.ssm_set_spin_limit(0)
    try:
        got = run()
    finally:
        ssm.ssm_set_spin_limit(old)
    for k in want:
        assert torch.equal(got[k], want[k]), k
    again = run()
    for k in want:
        assert torch.equal(again[k], want[k]), k


def test_row_scans_of_more_workgroups_than_fit_on_four_streams():
    """The header's promise for launches whose tiles wait for one another and are not all resident at once: forward and gradient passes on four
    streams with workspaces of their own, queued together, come out as those alone, to the last bit."""
    import torch
    work = []
    for i, shp in enumerate([(16, 1000, 256, 256), (30, 1000, 512, 512), (100, 100, 256, 200), (3, 2048, 64, 128)]):
        d = ssm.to_device(wl.gen_inputs(wl.custom("streams%d" % i, *shp, p_reset=0.002, with_x0=True, seed=50 + i)))
        work.append((d, ssm.alloc_workspace(*shp, False), ssm.alloc_workspace(*shp, True), torch.cuda.Stream()))

    def run(d, ws_f, ws_b, stream=None):
        par = [d[k] for k in ("Lambda", "B", "C", "D", "log_delta")]
        f = ssm.ssm_scan_fwd(*par, d["u"], d["is_first"], d["x0"], workspace=ws_f, stream=stream)
        b = ssm.ssm_scan_bwd(*par, d["u"], d["is_first"], d["x0"], f["x"], d["dy"], workspace=ws_b, stream=stream)
        return {**f, **b}

    want = [run(*w[:3]) for w in work]
    torch.cuda.synchronize()
    got = []
    for _ in range(6):
        for w in work:
            with torch.cuda.stream(w[3]):
                got.append(run(*w))
    torch.cuda.synchronize()
    for i, g in enumerate(got):
        w = work[i % 4]
        assert ssm.ssm_workspace_status(w[1]) == ssm.SSM_OK and ssm.ssm_workspace_status(w[2]) == ssm.SSM_OK
        for k in g:
            assert torch.equal(g[k], want[i % 4][k]), (i, k)


@pytest.mark.parametrize("shape", [(3, 50, 32, 24), (8, 100, 256, 256), (30, 101, 64, 300)], ids=lambda s: "x".join(map(str, s)))
def test_the_last_saved_state_is_no_factor_of_the_transitions_gradient(shape):
    """x_{t-1} chi_t over the steps there are: what follows the last state does not count, also where the last tile has rows past it."""
    import torch
    Bt, L, H, P = shape
    d = ssm.to_device(wl.gen_inputs(wl.custom("last", Bt, L, H, P, p_reset=0.02, with_x0=True, seed=43)))
    par = [d[k] for k in ("Lambda", "B", "C", "D", "log_delta")]
    x = ssm.ssm_scan_fwd(*par, d["u"], d["is_first"], d["x0"])["x"]
    out = []
    for value in (1.0, float("inf"), float("nan")):
        x[-1, -1] = value
        out.append(ssm.ssm_scan_bwd(*par, d["u"], d["is_first"], d["x0"], x, d["dy"]))
    for o in out[1:]:
        for k in ("du", "dLambda", "dB", "dlog_delta", "dx0"):
            assert torch.equal(o[k], out[0][k]), k
