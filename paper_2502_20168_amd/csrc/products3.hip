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
        if constexpr (epi != 8) { if (form == SIXTEEN) { SSM_SMALL(epi, 65, 4); } } \
        if (form == ALONE) { SSM_SMALL(epi, 64, 2); } \
        SSM_SMALL(epi, 64, 4); \
        return hipErrorInvalidValue            /* (a small pair has at most 128 tiles of 64 x 128: 32 rows) */
    // A small pair: two workgroups per CU, or a CU to each (long stages, K tiles of 64 tokens), the items then by eight wavefronts or by sixteen.  What decides is how many slots
    // of an XCD's CUs its share of the launch takes.  Per cent of the gradient pass against two per CU (eight wavefronts, sixteen), 627 launches of 398 layers:
    //   within one round, by the product's K: below 384 +1.2 +1.6, 384 .. 639 -0.1 +0.1, 640 .. 831 -1.0 -0.2, from 832 on -2.3 -1.2; with items of 300 tokens and more, not much
    //     shorter than K, -2.0 -3.1 (25 x 57, 371, 577: 66.4, 63.7, 60.6 us), but beside a product that scans, whose wavefronts then have 128 registers, -2.6 -2.0;
    //   items that fill the XCD's CUs and a quarter as many tiles behind them -4.3 -3.3 (2 x 100, 1024, 512: 48.6, 46.2, 46.7), at more tiles +5.1 +5.5;
    //   items of half the CUs at most, on their own from beginning to end while the tiles pass in two rounds beside them: where they are at least 1.5 times as long as K -4.3 -6.9, one
    //     of 61 slower (+0.6; 12 x 222, 338, 567: 111.1, 102.5, 95.5), 1.2 .. 1.5 times +1.1 +0.6;
    //   else +8.0 +7.9 (2 x 396, 256, 416, 33 slots beside du: 32.9, 36.4, 37.0).
    enum { SHARED, ALONE, SIXTEEN } form = SHARED;
    if (gemm_small_pair(a.M, a.N)) {
        constexpr int64_t CUS = 32;                                                 // of an XCD
        int64_t items = 0;
        for (const GemmArgs *r : {b, c})
            if (r) items += reduction_items(r->M, r->N, r->splits < 1 ? 1 : r->splits, REDUCTION_64x64);
        const int64_t tiles = (int64_t)((a.M + 31) / 32) * ((a.N + t.cols - 1) / t.cols), t_slots = (tiles + 7) / 8, i_slots = (items + 7) / 8;
        const int64_t tokens = b->splits < 1 ? b->K : (b->K + b->splits - 1) / b->splits;        // of an item
        const bool scans = a.epilogue == 8;
        if (t_slots + i_slots <= CUS)
            form = !scans && a.K >= 384 && tokens >= 300 && 5 * tokens >= 3 * a.K ? SIXTEEN : a.K >= 448 ? ALONE : SHARED;
        else if (i_slots <= CUS && t_slots <= CUS / 4)
            form = a.K >= 448 ? ALONE : SHARED;
        else if (!scans && i_slots <= CUS / 2 && t_slots <= 2 * (CUS - i_slots) && tokens >= 440 && 2 * tokens >= 3 * (int64_t)a.K)
            form = SIXTEEN;
    }
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
