"""Workspaces of the gradient pass of layers on two planes: nobody asks for room that the shape does not use, and a workspace holds shorter sequences as it does
where every scan is a kernel of its own."""
import pytest

from paper_2502_20168_amd import binding as ssm
from paper_2502_20168_amd import workloads as wl


def _least(shape):
    """The smallest workspace (in whole 256 bytes, the alignment of its arrays) in which the gradient pass runs."""
    lo, hi = 0, ssm.ssm_workspace_bytes(*shape, True) // 256
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (lo, mid) if ssm.ssm_plan_launches(*shape, 256 * mid)[1] else (mid, hi)
    return 256 * hi


def _up(n):
    return -(-n // 256) * 256


@pytest.mark.parametrize("Bt,L,H,P", [(16, 256, 512, 512), (128, 256, 512, 512), (4, 4096, 512, 512)])
def test_scanning_shapes_ask_for_their_own_arrays_only(Bt, L, H, P):
    """Sequences of whole 128-step pieces: chi, two operands in fragment order (two planes of 16 bits, an exponent per row), the slabs, tagged words (two of 8 bytes
    per state and 64 tokens), row maxima, column dots, maxima, rows of dAbar per tile of 64 tokens at most, and 64 KiB for everything per state or per launch."""
    T, p = Bt * L, ssm.ssm_plan_describe(Bt, L, H, P)
    assert p["scans_in_projections"] == 1
    need = T * P * 8 + 2 * (2 * P * H * 4 + (2 * P + H) * 4) + (p["slabs_dC"] + p["slabs_dBbar"]) * 2 * P * H * 4 + T // 64 * P * 24 \
        + T * (-(-H // 64) + -(-2 * P // 128)) * 4
    dots = 512 * H * 4                                       # of dD: at most 512 slabs, and two words per slab and 64 columns
    assert ssm.ssm_workspace_bytes(Bt, L, H, P, True) <= need + dots + dots // 32 + 4 * 65536
    assert _least((Bt, L, H, P)) == _up(ssm.ssm_workspace_bytes(Bt, L, H, P, True))


# the longer ones: more than 64 tiles of 64 tokens (a scan kernel), whole pieces, and other lengths
@pytest.mark.parametrize("long,short", [((24, 4097, 512, 512), 4095), ((24, 4096, 512, 512), 4095), ((16, 1024, 512, 512), 700), ((16, 4097, 512, 512), 1000), ((4, 4097, 700, 530), 4095),
                                        ((24, 4097, 1024, 512), 4095), ((60, 250, 512, 512), 200), ((32, 1000, 513, 600), 250)])
def test_a_workspace_holds_shorter_sequences(long, short):
    Bt, L, H, P = long
    size, s = ssm.ssm_workspace_bytes(*long, True), (Bt, short, H, P)
    assert ssm.ssm_plan_describe(*s)["planes"] == 2
    assert ssm.ssm_plan_launches(*s, size)[1] in (4, 5)
    for bwd in (False, True):
        assert ssm.ssm_workspace_bytes(*s, False) <= ssm.ssm_workspace_bytes(*s, True)


@pytest.mark.parametrize("shape", [(24, 200, 1024, 512), (60, 100, 512, 512), (9, 515, 700, 530), (24, 4095, 512, 512), (300, 200, 700, 1024)])
def test_the_scan_of_rows_takes_little_more_and_less_room_takes_a_scan_kernel(shape):
    full, least = ssm.ssm_workspace_bytes(*shape, True), _least(shape)
    assert least <= full <= 1.025 * least
    assert [ssm.ssm_plan_launches(*shape, n)[1] for n in (full, least, least - 256, 0)] == [4, 4 if least == full else 5, 0, 0]
    assert ssm.ssm_workspace_bytes(*shape, False) <= least


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(60, 100, 512, 512), (9, 700, 512, 1000), (24, 200, 1024, 512), (5, 1500, 512, 512)], ids=lambda s: "x".join(map(str, s)))
def test_the_least_workspace_gives_the_same_gradients(shape):
    """Layer and S5 block in the least room and in full, between guard zones: gradients within 2e-5 of each other's norm (either is within a few 1e-6 of 64 bits; dLambda and
    dlog_delta, sums that cancel, within 2e-4), and the same to the last bit where no scan comes in between (dC, dD, dW)."""
    import torch
    Bt, L, H, P = shape
    print(shape, flush=True)
    d = ssm.to_device(wl.gen_inputs(wl.custom("least", Bt, L, H, P, p_reset=0.01, with_x0=True, seed=53)))
    par = [d[k] for k in ("Lambda", "B", "C", "D", "log_delta")]
    W = torch.from_numpy(wl.gen_half_glu(4, H, seed=7)["W"]).cuda()
    least, full = _least(shape), ssm.ssm_workspace_bytes(*shape, True)
    block = ssm.ssm_block_workspace_bytes(*shape, True)
    assert ssm.ssm_plan_launches(*shape, least)[1] == 5 and least < full

    def run(call, size):
        buf = torch.full((size + 2 * 65536,), 0xA5, dtype=torch.uint8, device="cuda")
        out = call(buf[65536:65536 + size])
        torch.cuda.synchronize()
        assert bool((buf[:65536] == 0xA5).all()) and bool((buf[65536 + size:] == 0xA5).all())
        return out

    x = ssm.ssm_scan_fwd(*par, d["u"], d["is_first"], d["x0"])["x"]
    f = ssm.ssm_block_fwd(*par, W, d["u"], d["is_first"], d["x0"])
    layer = lambda ws: ssm.ssm_scan_bwd(*par, d["u"], d["is_first"], d["x0"], x, d["dy"], workspace=ws)
    gated = lambda ws: ssm.ssm_block_bwd(*par, W, d["u"], d["is_first"], d["x0"], f["x"], f["y"], f["gate"], d["dy"], workspace=ws)
    for call, a, b in ((layer, full, least), (gated, block, block - _up(full) + _up(least))):
        want, got = run(call, a), run(call, b)
        for k in want:
            err = float((got[k] - want[k]).abs().pow(2).sum().sqrt() / want[k].abs().pow(2).sum().sqrt())
            print(k, err, flush=True)
            assert err <= (2e-4 if k in ("dLambda", "dlog_delta") else 2e-5), k
            if k in ("dC", "dD", "dW"):
                assert torch.equal(got[k], want[k]), k
        with pytest.raises(ssm.SsmError):
            call(torch.empty(b - 256, dtype=torch.uint8, device="cuda"))
