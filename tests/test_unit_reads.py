"""Every 16-byte request that the producers of a product make for its activations, walked on the host with the functions
that the kernel takes its addresses from: all of them lie inside the activations, or inside the packed weights.  And the
divisions that place a tile, against the processor's."""
import os
import subprocess

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

WALK = r"""
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "pk_units.h"
using namespace ssm;
// The requests of one tile as gemm_pk_tile makes them: PF K tiles at once (four values or more per row), one
// behind the first tile, one for every further tile.
static long walk(const float *A, int M, int K, const char *weights, long weight_bytes, int m0, int rows, int PF)
{
    const PkUnits units(K, K);
    const char *src = units.base(A + (long)m0 * K, weights), *end = reinterpret_cast<const char *>(A + (long)M * K);
    const int nk = (K + PK_BK - 1) / PK_BK;
    long outside = 0;
    auto fetch = [&](int t) {
        for (int r = 0; r < rows; ++r)
            for (int kq = 0; kq < PK_BK; kq += 4) {
                const char *p = src + (units.row(r, M - m0) + units.k(t, kq));
                const bool in_rows = p >= reinterpret_cast<const char *>(A) && p + 16 <= end;
                const bool in_weights = p >= weights && p + 16 <= weights + weight_bytes;
                if (!in_rows && !in_weights) ++outside;
                // a unit that lies inside its row is the one asked for
                const int k = t * PK_BK + kq, row = m0 + r;
                if (row < M && k + 4 <= K && p != reinterpret_cast<const char *>(A + (long)row * K + k)) ++outside;
            }
    };
    if (K >= 4) for (int j = 0; j < PF; ++j) fetch(j);
    fetch(PF);
    for (int kt = 0; kt + 1 < nk; ++kt) fetch(kt + 1 + PF);
    return outside;
}
int main()
{
    long bad = 0;
    for (int K : {1, 2, 3, 4, 5, 6, 7, 8, 31, 60, 61, 63, 64, 65, 67, 127, 130, 200})
        for (int M : {1, 2, 31, 32, 33, 64, 65, 128, 129})
            for (int rows : {32, 64, 128}) {
                // exactly as many bytes as the arguments have (the smallest weights: 32 rows x 64 k, two planes)
                float *A = static_cast<float *>(malloc((size_t)M * K * 4));
                const long wb = 32 * 64 * 2 * 2;
                char *w = static_cast<char *>(malloc(wb));
                for (int m0 = 0; m0 < M; m0 += rows)
                    if (const long n = walk(A, M, K, w, wb, m0, rows, rows == 32 ? 4 : 2)) { bad += n; printf("K %d M %d m0 %d: %ld\n", K, M, m0, n); }
                free(w);
                free(A);
            }
    return bad != 0;
}
"""

DIVIDE = r"""
#include <cstdio>
#include <cstdlib>
#include <initializer_list>
#include "fast_div.h"
int main()
{
    const unsigned top = 0x7fffffffu;
    long bad = 0;
    auto check = [&](unsigned n, unsigned d) { if (n <= top && ssm::FastDiv::by(d)(n) != n / d) { if (!bad++) printf("%u / %u\n", n, d); } };
    srand(1);
    auto any = [&] { return ((unsigned)rand() << 16 ^ (unsigned)rand()) & top; };
    for (int k = 0; k < 200000; ++k) {
        // divisors of any length, and those next to a power of two
        unsigned d = k < 4096 ? k + 1 : any() >> rand() % 31;
        if (k % 3 == 0) d = (1u << k % 31) + (unsigned)(k / 31 % 3) - 1;
        if (d == 0 || d > top) continue;
        const unsigned q = top / d * d, m = any() / d * d;               // multiples and their neighbours
        for (unsigned n : {0u, 1u, d - 1, d, d + 1, m - 1, m, m + d - 1, q - 1, q, top, any()}) check(n, d);
    }
    return bad != 0;
}
"""


def _run(tmp_path, text):
    src, exe = tmp_path / "walk.cpp", tmp_path / "walk"
    src.write_text(text)
    subprocess.check_call([os.environ.get("CXX", "g++"), "-std=c++17", "-O1", "-I", os.path.join(ROOT, "paper_2502_20168_amd", "csrc"), str(src),
                           "-o", str(exe)])
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    assert out.returncode == 0, out.stdout


def test_no_request_leaves_the_activations_or_the_weights(tmp_path):
    _run(tmp_path, WALK)


def test_divisions_by_multiplication_are_exact(tmp_path):
    _run(tmp_path, DIVIDE)
