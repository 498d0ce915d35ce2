// Host side of the projection products: which shapes scan inside them, how many K slabs a reduction gets, the tile
// of a product, and the launch (instantiations in products2.hip / products3.hip).
#include "ssm_internal.h"
#include "../../include/ssm.h"

namespace ssm {

// A product over T tokens with N columns that has few 128x128 tiles shares its launch with a K = T
// reduction on 64x64 tiles: a quarter of the multiply-adds per workgroup, so that the chain of K
// steps a small shape waits for is short.
// (forward + gradient pass with 32 instead of 64, 36 shapes of 1000 .. 4000 tokens, H and P 128 .. 512: 3 % faster to 3 %
// slower, 0.1 % slower on the mean; above 64 the product itself has a workgroup per CU)
constexpr int64_t SMALL_PAIR_ITEMS = 64;
bool gemm_small_pair(int64_t T, int64_t N)
{
    return ((T + 127) / 128) * ((N + 127) / 128) <= SMALL_PAIR_ITEMS;
}

// a launch of a two-plane product and `items` work items of reductions fits two workgroups per CU with tiles of 128 rows and
// with 64 does not by far
static bool takes_tall_tiles(int64_t tall, int64_t low, int64_t items) { return low + items > 576 && tall + items <= 512; }

// Reductions of M x N over K rows (`count` of them, with the same number of tiles) that share a launch with a product.
// What a launch of several rounds wants is one work item of the reductions per CU, a few less rather than more, and all of
// them in the first slots: every CU then works on one item from beginning to end while the product's tiles pass through its
// second place.  Beside a small product (64 x 64 tiles)
// half as many, and in front only where an item is the longer chain (more rows than the product's K loop).
// The counts are those that divide 8 or that 8 divides, because then an XCD owns whole slabs or one band of one
// (tn_place), and a few between; the one whose number of items is nearest in ratio; an item keeps at least 192 (64) rows.
// One reduction, two planes: fewer, down to 160 items, where the launch with tiles of 128 rows then fits (4800 tokens, H 1024, P 512: 304 + 192
// workgroups instead of 600 + 256, du beside dBbar 68.5 us against 71; gradient pass, 62 shapes of 2400 .. 11000 tokens: -5 .. +1.5 %, -1.1 % on the mean; the
// gate's 8448 tokens, H 512: 66.6 against 74.5.  With 144 items and fewer +3 .. +30 %; two reductions beside one product -5 .. +9 %, +2 % on the mean).
// dC beside C^H dy that scans its rows: the product keeps its tiles of 64 rows, and the same fewer slabs are still the faster (17 layers for which the counts
// differ, gradient pass: -4.0 .. +0.2 %, -2.1 % on the mean; 24 x 200, 1024, 512 with 2, 3, 4, 5, 8 slabs: 172.1, 168.2, 170.5, 167.8, 173.8 us).
// Measured on 251 launches (every product's reductions at 1000 .. 32768 tokens, H and P from 64 to 1024) against 18 counts in either order:
// the gradient pass is 0.7 % slower than with the best of them on geometric mean, 8 % at worst.  Some (us; this rule, best, same
// count with the product first):
//   one launch of three products   24x128, H 1024, P 512: 129 129 131     16x256, 512, 512: 93.4 93.4 95.2    4x4096, 256, 256: 101 101 102
//   launches of two, two planes    16x1000, 512, 512: 308 308 330
//   launches of two, three planes  20x300, 500, 250: 121 121 130          40x200, 768, 384: 259 259 298
//   beside small products          20x100, 256, 256: 46.7 46.7 50.5       8x128, 256, 256: 39.1 39.1 39.2
// (The launches of two were measured with products that do not scan.  With C^H dy scanning the rows of its tiles beside dC, 17 layers of
// 128 .. 10000 tokens: in the order the other way round forward and gradient pass take 2.5 % less to 10 % more, 1.5 % more on
// geometric mean.)
SlabPlan gemm_plan_slabs(int64_t M, int64_t N, int64_t K, int count, ReductionTile tile, int64_t k_main)
{
    const bool small = tile == REDUCTION_64x64;
    const int64_t tiles = reduction_items(M, N, count, tile), want = small ? 128 : 224, min_rows = small ? 64 : 192;
    // the product beside them: K tokens, as many columns as the reductions
    const int64_t columns = (N + 127) / 128, tall = (K + 127) / 128 * columns, low = (K + 63) / 64 * columns;
    int best = 1, fitting = 0;
    for (int s : {2, 3, 4, 5, 8, 12, 16, 24, 32, 40, 48, 56, 64}) {
        if (K / s < min_rows) break;
        // s is nearer than best: want / (tiles best) > (tiles s) / want
        if (tiles * s <= want || want * want > tiles * best * tiles * s) best = s;
        if (tile == REDUCTION_128x128 && count == 1 && tiles * s >= 160 && takes_tall_tiles(tall, low, tiles * s)) fitting = s;
    }
    if (fitting && fitting < best) best = fitting;
    return {best, !small || (K + best - 1) / best > k_main};
}

// The projections scan their own output tiles where a sequence is a whole number of 128-step pieces (a bounded chain
// of tiles per sequence) or every 128 tokens are whole sequences of whole 16-step chunks, and there are at least 64 tiles of
// 128 tokens.  (From there on the scanning tile with two planes beats a scan kernel and three planes on every shape measured;
// between 32 and 64 tiles it would by 4-20 % too, but those shapes keep the exact split into three planes.)
bool gemm_scan_shape_ok(int64_t Bt, int64_t L, int64_t P)
{
    constexpr int64_t PIECE = 128, CHUNK = 16, MIN_TILES = 64;
    const bool chain = L % PIECE == 0 && L <= SCAN_MAX_STEPS;
    const bool whole = L < PIECE && PIECE % L == 0 && L % CHUNK == 0 && (Bt * L) % PIECE == 0;
    if (!chain && !whole) return false;
    const int64_t tiles = (Bt * L / PIECE) * ((2 * P + 127) / 128);
    return tiles >= MIN_TILES && tiles * (PIECE / 64) * 64 <= 0x7fffffffLL;
}

// Two workgroups per CU either way.  Tiles of 128 tokens have half the weight traffic and half as many scans to set up and hand
// over, tiles of 64 more workgroups.  Time with 128 rows against 64 on 310 shapes, by tiles of 128 tokens x 64 states:
//                               192 tiles      256            384            512 and more
//   L >= 64, forward            -9 .. +2 %     -19 .. +1 %    -27 .. +3 %    -22 .. +1 %    (128 tiles: -1 .. +9 %)
//   L >= 64, gradient pass       0 .. +7 %      -2 .. +6 %    -11 .. +2 %    -11 .. +1 %
//   L < 64, forward              0 .. +4 %       0 .. +2 %     -5 .. +4 %    -10 .. +2 %    (a tile holds whole sequences:
//   L < 64, gradient pass       +2 .. +7 %      +2 .. +7 %      0 .. +3 %     -5 .. +2 %     nothing is handed over)
int gemm_scan_rows(int64_t T, int64_t L, int64_t P, bool reverse)
{
    const int64_t tiles = (T / 128) * ((2 * P + 127) / 128);
    return tiles >= (L < 64 ? 512 : reverse ? 384 : 192) ? 128 : 64;
}

size_t gemm_scan_desc_bytes(int64_t Bt, int64_t L, int64_t P)
{
    if (L <= 64) return 0;                           // a tile holds whole sequences: nothing is handed over
    const int64_t tiles = (Bt * L / 64) * ((2 * P + 127) / 128);
    return (size_t)tiles * 64 * 2 * sizeof(unsigned long long);
}

// Three planes: the input projection and C^H dy scan the rows of the tiles that they take anyway, whatever the sequences' length (up to 64 tiles
// before another one: eight for each of a state's threads): 32 rows in small pairs, else 64.  The launches on tiles of other widths or
// heights keep the scan kernels: at most 32 states and many rows, and the few tokens of layers so wide that the product alone takes 32 rows but not beside reductions.
int gemm_row_scan_rows(int64_t T, int64_t L, int64_t P)
{
    const bool small = gemm_small_pair(T, 2 * P);
    const int rows = small ? 32 : 64;
    if (L > (int64_t)ROW_SCAN_MAX_TILES * rows) return 0;
    return small || (P > 32 && ((T + 63) / 64) * ((2 * P + 127) / 128) > 128) ? rows : 0;
}

size_t gemm_row_scan_desc_bytes(int64_t T, int64_t P, int rows)
{
    return (size_t)((T + rows - 1) / rows) * P * 2 * sizeof(unsigned long long);
}

// The tile of a product.
//   32 rows where 64-row tiles would occupy at most half of the CUs (1024 x 1024 x 512, 128 tiles of 64 x 128: 6.2 us
//     against 7.7; 4096 x 512 x 1024, 256 tiles: 16.7 against 14.5).  What a workgroup then waits for is its chain of
//     dependent matrix instructions (a 32 x 128 x 64 tile of three planes: 24 on one accumulator, 0.55 us), so fewer columns,
//     whose consumers share out k, until there are two workgroups per CU.
//   32 x 64 at any number of rows (three planes) where the result has at most 64 columns, half of a wider tile (16000 tokens, H = 64, P = 256: forward
//     pass 43.6 us against 45.1; the gate's at 16384 tokens, H = 64: 11.7 against 12.4; at 96 columns, and with two planes, the wider tile is faster).
//   128 rows (two planes) where they give every CU two workgroups
//     (32768 x 512 x 1024: 117 us against 122; 4800 x 1024 x 1024, 304 tiles: 47 against 40), and where the launch with its
//     reductions then fits two workgroups per CU and with 64 rows does not by far (gradient pass of 4000 tokens, H = P = 512: 110 against
//     116 us; the gate's, 4096 tokens, H = 1024: 92 against 97, but H = 768, 564 workgroups: 67 against 62).
PkTile product_tile(const GemmArgs &a, const GemmArgs *b, const GemmArgs *c)
{
    if ((a.epilogue >= 7) && a.planes == 2) return {a.scan.rows, 128};
    const auto tiles = [&](int64_t bm, int64_t bn) { return ((a.M + bm - 1) / bm) * ((a.N + bn - 1) / bn); };
    int64_t items = 0;
    for (const GemmArgs *t : {b, c})
        if (t) items += reduction_items(t->M, t->N, t->splits < 1 ? 1 : t->splits, reduction_tile(a.planes, gemm_small_pair(a.M, a.N)));
    if (a.planes == 3 && a.N <= 64 && tiles(64, 128) > 128 && !b && !a.c2_rowmax) return {32, 64};
    // (two planes: no 32-row tiles beside reductions, and none where there are always more tiles but in the widest layers)
    if (tiles(64, 128) <= 128 && (a.planes == 3 || (!b && (a.epilogue == 1 || a.epilogue == 6))))
        return {32, a.c2_rowmax || tiles(32, 64) + items > 256 ? 128 : tiles(32, 32) + items > 128 ? 64 : 32};
    if (a.planes != 2) return {64, 128};
    return {tiles(128, 128) >= 512 || (items > 0 && takes_tall_tiles(tiles(128, 128), tiles(64, 128), items)) ? 128 : 64, 128};
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
    if (!c.lam || !c.err || c.L <= 0 || a.N != 2 * c.P || a.M % c.L != 0 || ((a.epilogue == 8 || a.epilogue == 10) && (!c.xsaved || !c.partial))) return false;
    if (a.epilogue >= 9) return a.planes == 2 && (a.epilogue == 9 || c.amax_out) && c.rows == 64 && c.L <= ROW_SCAN_MAX_TILES * 64 && c.rowmax_out && (c.desc || 64 % c.L == 0);
    if (a.planes == 3) return c.rows > 0 && c.rows == gemm_row_scan_rows(a.M, c.L, c.P) && (c.desc || c.rows % c.L == 0);
    if ((c.rows != 64 && c.rows != 128) || a.M % c.rows != 0) return false;
    const bool chain = c.L % c.rows == 0 && c.L <= SCAN_MAX_STEPS && (c.desc || c.L == 64);
    const bool whole = c.L < c.rows && 64 % c.L == 0 && c.L % (c.rows / 8) == 0;
    return chain || whole;
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
    case 7: case 8: case 9: case 10: if (!scan_args_ok(a)) return hipErrorInvalidValue; break;
    default: return hipErrorInvalidValue;
    }
    return a.planes == 2 ? products_two_planes(a, b, c, tn_first, s) : products_three_planes(a, b, c, tn_first, s);
}

}  // namespace ssm
