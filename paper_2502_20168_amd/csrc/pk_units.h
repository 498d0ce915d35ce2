// Which 16 bytes a producer of a product with packed weights requests for a unit of four consecutive k of a row of the
// activations.  Plain arithmetic, also compiled by the host test that walks every request (tests/test_unit_reads.py).
#pragma once

#ifdef __HIPCC__
#define SSM_UNIT __host__ __device__ __forceinline__
#else
#define SSM_UNIT inline
#endif

namespace ssm {

constexpr int PK_BK = 64;                    // k per K tile

// A unit that reaches over the end of its row (the last K tile of a K that is no multiple of 64, and the requests behind
// the last tile) reads the row's last four values.  A row of fewer than four has no 16 bytes of its own: its values are
// loaded one by one, and the requests that are made all the same, without a branch, go to the first bytes of
// the packed weights (at least 8 KiB), whatever the row and k.
struct PkUnits {
    bool narrow;
    unsigned pitch;                          // bytes from one row to the next
    int klast;                               // the last k that a unit may start at
    SSM_UNIT PkUnits(int K, long lda) : narrow(K < 4), pitch(K < 4 ? 0u : 4u * (unsigned)lda), klast(K < 4 ? 0 : K - 4) {}
    SSM_UNIT const char *base(const float *tile, const void *weights) const
    {
        return narrow ? static_cast<const char *>(weights) : reinterpret_cast<const char *>(tile);
    }
    // byte offsets from the base: of row r of a tile with `rows` rows in all, and of the k that the unit at kq of K tile t reads
    SSM_UNIT unsigned row(int r, int rows) const { return (unsigned)(r < rows ? r : rows - 1) * pitch; }
    SSM_UNIT unsigned k(int t, int kq) const { return 4u * (unsigned)(t * PK_BK + kq < klast ? t * PK_BK + kq : klast); }
};

}  // namespace ssm
