// Host side of the projection products: which shapes scan inside them, how many K slabs a reduction gets, and
// the launch (instantiations in products2.hip / products3.hip).
#include "ssm_internal.h"
#include "../../include/ssm.h"

namespace ssm {

int gemm_pick_splits(int64_t M, int64_t N, int64_t K, int64_t partner_tiles)
{
    // A long reduction with a small result shares its launch with a product of partner_tiles
    // 128x128 tiles: enough K splits that the two together fill the last round of workgroups
    // on the 256 CUs, keeping at least 256 rows of K per split.
    const int64_t tiles = ((M + 127) / 128) * ((N + 127) / 128);
    const int64_t target = 256 - partner_tiles % 256;
    int64_t s = (target + tiles / 2) / tiles;
    const int64_t maxs = (K + 255) / 256;
    if (s > maxs) s = maxs;
    if (s > 64) s = 64;
    if (s < 1) s = 1;
    return (int)s;
}

// A product over T tokens with N columns that has few 128x128 tiles shares its launch with a K = T
// reduction on 64x64x64 tiles: a quarter of the multiply-adds per workgroup, so that the chain of K
// steps a small shape waits for is short.
// (measured: 16 and 32 leave gains on the table, 128 doubles the step at 40 x 100 tokens, H = P = 256)
constexpr int64_t SMALL_PAIR_ITEMS = 64;
bool gemm_small_pair(int64_t T, int64_t N)
{
    return ((T + 127) / 128) * ((N + 127) / 128) <= SMALL_PAIR_ITEMS;
}

// K splits of an M x N reduction over K rows that shares such a launch with a product of main_M x main_N whose K loop is
// k_main long: work items about as long as that product's (an item takes about 1.5 times as long per row as the product), at
// most two rounds of workgroups in all; where there is room for it in one round, at least 128 rows per item.
int gemm_pick_splits_small(int64_t M, int64_t N, int64_t K, int64_t main_M, int64_t main_N, int64_t k_main)
{
    const int64_t tiles = ((M + 63) / 64) * ((N + 63) / 64);
    const int64_t kt = k_main < 64 ? 64 : k_main;
    int64_t s = (K + k_main / 2) / kt;
    const int64_t room = (512 - ((main_M + 63) / 64) * ((main_N + 63) / 64)) / tiles;
    if (s > room) s = room;
    const int64_t maxs = (K + 63) / 64;
    if (s > maxs) s = maxs;
    const int64_t t64 = ((main_M + 63) / 64) * ((main_N + 127) / 128), items = t64 <= 128 ? ((main_M + 31) / 32) * ((main_N + 127) / 128) : t64;
    int64_t one = (3 * K / 2 + kt / 2) / kt;
    if (one > (256 - items) / tiles) one = (256 - items) / tiles;
    if (one > K / 128) one = K / 128;
    if (s < one) s = one;
    if (s > 64) s = 64;
    if (s < 1) s = 1;
    return (int)s;
}

// List scheduling of nl work items of l K tiles and then ns items of s K tiles on the 256 CUs, as the
// dispatcher hands out workgroups in slot order to CUs as they fall free (a CU's two workgroups share its
// throughput, so a CU is one machine): the K tiles the busiest CU ends up with.  Loads are kept as (level, number of CUs) pairs; a batch of items goes to all CUs of
// the lowest level at once.
int64_t lpt_makespan(int64_t nl, int64_t l, int64_t ns, int64_t s)
{
    constexpr int64_t CUS = 256;
    constexpr int MAXLV = 16;
    int64_t lv[MAXLV], cnt[MAXLV];
    int n = 0;
    const int64_t q = nl / CUS, r = nl % CUS;
    lv[n] = q * l; cnt[n] = CUS - r; ++n;                    // ascending levels
    if (r) { lv[n] = (q + 1) * l; cnt[n] = r; ++n; }
    while (ns > 0) {
        const int64_t k = cnt[0] < ns ? cnt[0] : ns;
        const int64_t target = lv[0] + s;
        ns -= k;
        cnt[0] -= k;
        if (cnt[0] == 0) { for (int i = 1; i < n; ++i) { lv[i - 1] = lv[i]; cnt[i - 1] = cnt[i]; } --n; }
        int pos = 0;
        while (pos < n && lv[pos] < target) ++pos;
        if (pos < n && lv[pos] == target) { cnt[pos] += k; continue; }
        if (n == MAXLV) { lv[n - 1] = lv[n - 1] > target ? lv[n - 1] : target; cnt[n - 1] += k; continue; }   // (never with two item lengths)
        for (int i = n; i > pos; --i) { lv[i] = lv[i - 1]; cnt[i] = cnt[i - 1]; }
        lv[pos] = target; cnt[pos] = k; ++n;
    }
    return lv[n - 1];
}

// K splits of the K = T reductions (red_tiles tiles of 128x128 in all, split_bytes of slabs per split in
// all) that share a launch of 128x128x32 tiles with a product of main_tiles tiles whose K loop is k_main
// long: the count that minimises the busiest CU's K tiles plus what every further set of slabs costs (their
// bytes are written by this launch and read by the parameter epilogue's: measured 1.4 us, about 1.4 K
// tiles, per split of two reductions with 2 MiB slabs).  red_first: the reductions' work items belong in the
// first slots of the launch.  One workgroup per CU: whichever order the schedule model finishes earlier,
// the product first on a tie (measured on ten shapes with separate scan kernels: the model's choice was
// the faster order on every one, by up to 5 % of the step).  Two workgroups per CU: the reductions first
// when their items are at least twice as long as the product's (then a CU holds one of each kind for most
// of the launch instead of ending on single long items; 1024 x 16 tokens, H = P = 512: 0.469 against 0.482 ms).
int gemm_pick_splits_model(int64_t T, int64_t main_tiles, int64_t k_main, int64_t red_tiles, size_t split_bytes, bool two_per_cu,
                           bool &red_first)
{
    static const int cand[] = {1, 2, 3, 4, 5, 6, 8, 10, 12, 16, 24, 32, 48, 64};
    const int64_t a = (k_main + 31) / 32;
    const double per_split = 0.2 + 0.6 * (double)split_bytes / (double)(2 << 20);
    int best = 1;
    double best_cost = -1.0;
    red_first = false;
    for (int sp : cand) {
        if (sp > 1 && sp > T / 256) break;
        const int64_t b = (((T + sp - 1) / sp) + 31) / 32;
        const int64_t m_main = lpt_makespan(main_tiles, a, red_tiles * sp, b), m_red = lpt_makespan(red_tiles * sp, b, main_tiles, a);
        const int64_t m = m_red < m_main ? m_red : m_main;
        const double cost = (double)m + per_split * sp;
        if (best_cost < 0 || cost < best_cost) { best_cost = cost; best = sp; red_first = two_per_cu ? b >= 2 * a : m_red < m_main; }
    }
    return best;
}

// (one reduction of M x N over K rows beside a product of main_tiles tiles, one workgroup per CU)
int gemm_pick_splits_balanced(int64_t M, int64_t N, int64_t K, int64_t main_tiles, int64_t k_main, bool &red_first)
{
    return gemm_pick_splits_model(K, main_tiles, k_main, ((M + 127) / 128) * ((N + 127) / 128), (size_t)M * N * 4, false, red_first);
}

// The projections scan their own output tiles where a sequence is a whole number of 128-step pieces (a bounded chain
// of tiles per sequence) or every 128 tokens are whole sequences of whole 16-step chunks, and there are enough tiles
// (measured with tiles of 128 tokens: from 64 of them on -- a quarter of the CUs -- the scanning tile beats smaller tiles
// plus a scan kernel: +2 % at 64 tiles, +7..13 % at 96-128; no difference at 32-48).
bool gemm_scan_shape_ok(int64_t Bt, int64_t L, int64_t P)
{
    constexpr int64_t PIECE = 128, CHUNK = 16, MIN_TILES = 64;
    const bool chain = L % PIECE == 0 && L <= SCAN_MAX_STEPS;
    const bool whole = L < PIECE && PIECE % L == 0 && L % CHUNK == 0 && (Bt * L) % PIECE == 0;
    if (!chain && !whole) return false;
    const int64_t tiles = (Bt * L / PIECE) * ((2 * P + 127) / 128);
    return tiles >= MIN_TILES && tiles * (PIECE / 64) * 64 <= 0x7fffffffLL;
}

// Two workgroups per CU either way: tiles of 128 tokens (half the weight traffic, half as many scans to set up and hand
// over) from the size on at which they still give every CU two of them.
int gemm_scan_rows(int64_t T, int64_t P) { return (T / 128) * ((2 * P + 127) / 128) >= 512 ? 128 : 64; }

size_t gemm_scan_desc_bytes(int64_t Bt, int64_t L, int64_t P)
{
    if (L <= 64) return 0;                           // a tile holds whole sequences: nothing is handed over
    const int64_t tiles = (Bt * L / 64) * ((2 * P + 127) / 128);
    return (size_t)tiles * 64 * 2 * sizeof(unsigned long long);
}

// Tile tier of an M x N product with `splits` K splits, by rounds of workgroups on the 256 CUs: 0 = 128x128 tiles, 1 =
// 64x128, 2 = 64x64.  Only reported (ssm_plan_describe): how coarse a tile a product of this size can afford.
int gemm_tile_tier(int64_t M, int64_t N, int splits_in)
{
    const int64_t splits = splits_in < 1 ? 1 : splits_in;
    const int64_t r0 = (((M + 127) / 128) * ((N + 127) / 128) * splits + 255) / 256;
    const int64_t r1 = (((M + 63) / 64) * ((N + 127) / 128) * splits + 255) / 256;
    const int64_t r2 = (((M + 63) / 64) * ((N + 63) / 64) * splits + 255) / 256;
    const int64_t c0 = 10 * r0, c1 = 10 * r1, c2 = 6 * r2;
    if (c2 < c0 && c2 < c1) return 2;
    return c1 <= c0 ? 1 : 0;
}

namespace {
bool reduction_ok(const GemmArgs &t, int planes)
{
    return t.A && t.B && t.C && t.M > 0 && t.N > 0 && t.K > 0 && (planes == 3 || (t.amaxA.slots && t.amaxA.n > 0 && t.amaxB.slots && t.amaxB.n > 0));
}
// a scanning epilogue: whole sequences per tile or a chain of tiles, and its buffers
bool scan_args_ok(const GemmArgs &a)
{
    const ScanEpilogue &c = a.scan;
    if (a.planes != 2 || !c.lam || !c.err || c.L <= 0 || a.N != 2 * c.P || a.M % c.L != 0 || (c.rows != 64 && c.rows != 128) || a.M % c.rows != 0) return false;
    const bool chain = c.L % c.rows == 0 && c.L <= SCAN_MAX_STEPS && (c.desc || c.L == 64);
    const bool whole = c.L < c.rows && 64 % c.L == 0 && c.L % (c.rows / 8) == 0;
    return (chain || whole) && (a.epilogue == 7 || (c.xsaved && c.partial));
}
}  // namespace

hipError_t launch_products(const GemmArgs &a, const GemmArgs *b, const GemmArgs *c, bool tn_first, hipStream_t s)
{
    if (a.M <= 0 || a.N <= 0 || a.K <= 0 || !a.A || !a.C || !a.w.frag || (a.planes != 2 && a.planes != 3)) return hipErrorInvalidValue;
    if (a.planes == 2 && (!a.w.exp || !a.amaxA.rows || a.amaxA.row_parts <= 0)) return hipErrorInvalidValue;
    if ((c && !b) || (b && !reduction_ok(*b, a.planes)) || (c && !reduction_ok(*c, a.planes))) return hipErrorInvalidValue;
    switch (a.epilogue) {
    case 0: break;
    case 1: if (!a.diag || !a.E) return hipErrorInvalidValue; break;
    case 2: if (!a.diag || !a.E || a.N % 2) return hipErrorInvalidValue; break;
    case 3: if (!a.E) return hipErrorInvalidValue; break;
    case 4: if (!a.E || !a.E2) return hipErrorInvalidValue; break;
    case 5: if ((a.C2 && !a.diag) || a.N % 2) return hipErrorInvalidValue; break;
    case 6: if (!a.diag || !a.E || !a.C2) return hipErrorInvalidValue; break;
    case 7: case 8: if (!scan_args_ok(a)) return hipErrorInvalidValue; break;
    default: return hipErrorInvalidValue;
    }
    return a.planes == 2 ? products_two_planes(a, b, c, tn_first, s) : products_three_planes(a, b, c, tn_first, s);
}

}  // namespace ssm
