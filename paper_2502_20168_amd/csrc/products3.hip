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
        SSM_SMALL(epi, 64, 4); \
        return hipErrorInvalidValue            /* (a small pair has at most 128 tiles of 64 x 128: 32 rows) */
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
