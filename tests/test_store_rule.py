"""Which results are stored through the L2: the lines of store_rule.h on the host, and passes on the far side of them against the oracle."""
import os
import subprocess

import pytest

from paper_2502_20168_amd import workloads as wl

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

RULE = r"""
#include <cstdio>
#include "store_rule.h"
using namespace ssm;
static int bad = 0;
#define IS(want, ...) do { if ((__VA_ARGS__) != want) { ++bad; printf("line %d: %s\n", __LINE__, #__VA_ARGS__); } } while (0)
int main()
{
    const uintptr_t at = 1 << 20;
    const long MiB = 1 << 20;
    // whole lines at any size
    IS(true, output_through(at, 0, 4096, 2048)); IS(true, output_through(at, at, 1 << 21, 2048)); IS(true, states_through(at, 1 << 21, 512));
    // units that are no 16 aligned bytes: never
    IS(false, output_through(at, 0, 1, 140)); IS(false, output_through(at + 4, 0, 1, 512)); IS(false, output_through(at, at + 8, 1, 512));
    // aligned units, rows of no whole lines: 32 MiB of outputs (both arrays), 64 MiB of states
    IS(true, output_through(at, 0, 32 * MiB / 2000, 2000)); IS(false, output_through(at, 0, 32 * MiB / 2000 + 1, 2000));
    IS(true, output_through(at, at, 16 * MiB / 2000, 2000)); IS(false, output_through(at, at, 16 * MiB / 2000 + 1, 2000));
    IS(true, output_through(at + 16, 0, 16384, 2048)); IS(false, output_through(at + 16, 0, 16385, 2048));
    IS(true, states_through(at, 64 * MiB / 4000, 500)); IS(false, states_through(at, 64 * MiB / 4000 + 1, 500));
    IS(true, states_through(at + 8, 16384, 512)); IS(false, states_through(at + 8, 16385, 512));
    // products beyond 32 bits
    IS(false, output_through(at, 0, 2147483647, 4 * 65535 + 4 - 16)); IS(false, states_through(at, 2147483647, 65535));
    return bad != 0;
}
"""


def test_lines_of_the_rule(tmp_path):
    src, exe = tmp_path / "rule.cpp", tmp_path / "rule"
    src.write_text(RULE)
    subprocess.check_call([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2502_20168_amd", "csrc"), str(src),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


# Just past the lines, rows of no whole lines: states of 64 MiB that the projections scan (rows of 64-token tiles; whole pieces and
# several sequences per tile of 128), with a last tile that is not full; outputs of 32 MiB.
@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(170, 100, 40, 500), (129, 131, 24, 500), (64, 256, 16, 520), (17, 1024, 16, 491), (1032, 16, 16, 530), (170, 100, 500, 4)],
                         ids=str)
def test_stores_left_in_the_l2(shape):
    from parity_util import check_workload
    Bt, L, H, P = shape
    assert Bt * L * P * 8 > 64 << 20 and P % 16 or Bt * L * H * 4 > 32 << 20 and H % 32
    check_workload(wl.custom("far side", Bt, L, H, P, p_reset=0.01, with_x0=True, seed=37), backward=True)
