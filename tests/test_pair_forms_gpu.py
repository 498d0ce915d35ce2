"""The forms of a small product beside its reductions on 64 x 64 tiles: two workgroups per CU, a CU to each, and items of sixteen wavefronts, on either side of the lines
between them, and how accurately each adds up."""
import numpy as np
import pytest

from paper_2502_20168_amd import binding as ssm
from paper_2502_20168_amd import workloads as wl
from tests.parity_util import check_workload
from tests.test_block_gpu import test_half_glu_matches_oracle as check_gate

pytestmark = pytest.mark.gpu

SHAPES = [
    # Bt, L, H, P; beside du unless stated
    (53, 18, 448, 256), (99, 22, 160, 200), (6, 279, 150, 208),      # one round, sixteen wavefronts: tiles of 32 columns and 64, K and items that end inside a K tile
    (57, 24, 195, 251), (1, 504, 806, 351),                # odd widths; 128 columns
    (297, 12, 235, 100), (22, 89, 512, 160), (11, 699, 128, 160),    # two rounds of tiles beside half as many items; K of a short stage
    (12, 100, 300, 192), (12, 100, 300, 191),              # items of 300 tokens, and K on either side of 384
    (2, 100, 1024, 512), (2, 396, 256, 416),               # items that fill the chip with few tiles behind them; one slot too many
    (3, 187, 991, 294),                                    # a CU to each where C^H dy scans
]


@pytest.mark.parametrize("shape", SHAPES, ids=["x".join(map(str, s)) for s in SHAPES])
def test_forms_of_small_pairs(shape):
    Bt, L, H, P = shape
    print(shape, flush=True)
    check_workload(wl.custom("forms", Bt, L, H, P, p_reset=0.03, with_x0=True, seed=31), backward=True)


@pytest.mark.parametrize("T,H", [(598, 460), (600, 460), (613, 461)])      # items of 299 tokens and of 300; an odd width
def test_forms_beside_the_gates_adjoint(T, H):
    print(T, H, flush=True)
    check_gate(T, H)


# errors of dC and dB on these inputs with the small products of a k step in accumulators of their own, and with all six in one (2-norm): the bound is their geometric mean
@pytest.mark.parametrize("shape,measured", [((8, 250, 180, 180), ((1.18e-7, 2.49e-7), (1.17e-7, 2.48e-7))),             # two workgroups per CU
                                            ((53, 18, 448, 256), ((1.39e-7, 3.39e-7), (1.11e-7, 2.42e-7))),             # a CU to each; sixteen wavefronts
                                            ((22, 89, 512, 160), ((1.60e-7, 3.96e-7), (1.25e-7, 2.84e-7)))], ids=str)
def test_sums_over_tokens_round_once_per_step(shape, measured):
    """Operands that are what the library was given, to the last bit: dC sums dy times the saved states, and with Abar = 0 and a C of ones and zeros chi is dy, so that dB sums dy
    times u over 64.  Their planes are exact and so are the products: what is left is the rounding of the sums."""
    import torch
    Bt, L, H, P = shape
    print(shape, flush=True)
    T, rng = Bt * L, np.random.default_rng(3)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    dy, u = f(T, H), f(T, H)
    x = (f(T, P) + 1j * f(T, P)).astype(np.complex64)
    column = np.arange(P) % H
    C = np.zeros((H, P), np.complex64)
    C[column, np.arange(P)] = 1
    B = (f(P, H) + 1j * f(P, H)).astype(np.complex64)
    d = [torch.from_numpy(a).cuda() for a in (np.full(P, -64, np.complex64), B, C, f(H), np.full(P, 10, np.float32), u.reshape(Bt, L, H),
                                              x.reshape(Bt, L, P), dy.reshape(Bt, L, H))]
    got = ssm.ssm_scan_bwd(*d[:6], None, None, d[6], d[7])
    d64, x64 = dy.astype(np.float64), x.astype(np.complex128)
    want = {"dC": d64.T @ x64.conj(), "dB": d64[:, column].T @ u.astype(np.float64) / 64}
    for k, (apart, together) in zip(("dC", "dB"), measured):
        g = got[k].cpu().numpy()
        error = np.linalg.norm((g if k == "dC" else g.real) - want[k]) / np.linalg.norm(want[k])
        print(k, error, flush=True)
        assert error <= (apart * together) ** 0.5, k
