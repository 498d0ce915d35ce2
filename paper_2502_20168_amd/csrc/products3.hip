// Products with packed weights on three bf16 planes per operand, and the reductions over tokens that share their
// launches (on 64x64 tiles where the product is small).
#include "gemm_packed.h"

namespace ssm {

hipError_t products_three_planes(const GemmArgs &a, const GemmArgs *b, const GemmArgs *c, bool tn_first, hipStream_t s)
{
    const PkTile t = product_tile(a, b, c);
#define SSM_PK(rows, cols, epi, tnb, wpe) launch_pk_variant<rows, cols, 3, epi, tnb, wpe>(a, b, c, tn_first, s)
#define SSM_SMALL(epi, tnb, wpe) \
    if (t.rows == 32) return t.cols == 32 ? SSM_PK(32, 32, epi, tnb, wpe) : t.cols == 64 ? SSM_PK(32, 64, epi, tnb, wpe) : SSM_PK(32, 128, epi, tnb, wpe)
#define SSM_ALONE(epi) \
    case epi: \
        if (many) return SSM_PK(32, 64, epi, 0, 4); \
        SSM_SMALL(epi, 0, 2); \
        return SSM_PK(64, 128, epi, 0, 4)
    if (!b) {
        // more workgroups than CUs (at most 64 columns, many rows): short stages, two workgroups per CU
        const bool many = t.rows == 32 && t.cols == 64 && (int64_t)((a.M + 31) / 32) * ((a.N + 63) / 64) > 256;
        switch (a.epilogue) {
        SSM_ALONE(0); SSM_ALONE(1); SSM_ALONE(2); SSM_ALONE(3); SSM_ALONE(5); SSM_ALONE(6);
        case 7:
            if (a.scan.rows == 64) return SSM_PK(64, 128, 7, 0, 4);
            SSM_SMALL(7, 0, 2);
            return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
        }
    }
#define SSM_PAIR(epi) \
    case epi: \
        if (!gemm_small_pair(a.M, a.N)) return SSM_PK(64, 128, epi, 96, 4); \
        if (apart) { SSM_SMALL(epi, 64, 2); } \
        SSM_SMALL(epi, 64, 4); \
        return hipErrorInvalidValue            /* (a small pair has at most 128 tiles of 64 x 128: 32 rows) */
    // A small pair whose product contracts 448 and more takes a CU per workgroup, with long stages and reduction tiles of 64 tokens, where the launch fits the chip once, or the
    // tiles or the items alone fill it and the others fit behind them: there two workgroups on a CU do not finish sooner than one behind the other.  Two per
    // CU and one, forward and gradient pass: 254 workgroups (25 x 80, 256, 256) 56.9 and 53.2 us, 250 tiles and 128 items (8 x 1000, 128, 256) 87.2 and 83.3, 56 and 256
    // (2 x 100, 1024, 512) 77.9 and 72.9; but 120 and 150 (20 x 64, 300, 300) 64.7 and 66.8, 190 and 190 (6 x 100, 600, 600) 84.3 and 94.2, and 228 and
    // 140 over 256 (30 x 60, 256, 200) 57.7 and 58.8.
    const int64_t tiles = (int64_t)((a.M + 31) / 32) * ((a.N + t.cols - 1) / t.cols);
    int64_t items = 0;
    for (const GemmArgs *r : {b, c})
        if (r) items += reduction_items(r->M, r->N, r->splits < 1 ? 1 : r->splits, REDUCTION_64x64);
    const bool apart = a.K >= 448 && (tiles + items <= 256 || (tiles + items <= 400 && (tiles >= 240 || items >= 240)));
    switch (a.epilogue) {
    SSM_PAIR(0); SSM_PAIR(1); SSM_PAIR(4); SSM_PAIR(8);
    default: return hipErrorInvalidValue;
    }
#undef SSM_PAIR
#undef SSM_ALONE
#undef SSM_SMALL
#undef SSM_PK
}

}  // namespace ssm
