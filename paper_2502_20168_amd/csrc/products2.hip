// Products with packed weights on two scaled fp16 planes per operand, and the reductions over tokens that share
// their launches.
#include "gemm_packed.h"

namespace ssm {

hipError_t products_two_planes(const GemmArgs &a, const GemmArgs *b, const GemmArgs *c, bool tn_first, hipStream_t s)
{
    const PkTile t = product_tile(a, b, c);
#define SSM_PK(rows, cols, epi, tnb) launch_pk_variant<rows, cols, 2, epi, tnb, (rows) == 32 ? 2 : 4>(a, b, c, tn_first, s)
#define SSM_TALL(epi, tnb) return t.rows <= 64 ? SSM_PK(64, 128, epi, tnb) : SSM_PK(128, 128, epi, tnb)
#define SSM_ALONE(epi) \
    case epi: \
        if (t.rows == 32) return t.cols == 32 ? SSM_PK(32, 32, epi, 0) : t.cols == 64 ? SSM_PK(32, 64, epi, 0) : SSM_PK(32, 128, epi, 0); \
        SSM_TALL(epi, 0)
    if (!b) {
        switch (a.epilogue) {
        SSM_ALONE(1); SSM_ALONE(6);
        case 0: SSM_TALL(0, 0);
        case 3: SSM_TALL(3, 0);
        case 7: SSM_TALL(7, 0);
        case 9: return SSM_PK(64, 128, 9, 0);
        case 8: SSM_TALL(8, 0);
        default: return hipErrorInvalidValue;
        }
    }
    switch (a.epilogue) {
    case 0: SSM_TALL(0, 128);                             // C^H dy with the dC slabs (a separate scan kernel)
    case 10: return SSM_PK(64, 128, 10, 128);             // and its scan
    case 1: SSM_TALL(1, 128);                             // du with the dBbar slabs, and the dC slabs
    case 4: SSM_TALL(4, 128);                             // adjoint of the gate with the dW slabs
    default: return hipErrorInvalidValue;
    }
#undef SSM_ALONE
#undef SSM_TALL
#undef SSM_PK
}

}  // namespace ssm
