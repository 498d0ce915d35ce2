// Division by a number that the host knows.  Plain arithmetic, also compiled by the host test that compares it with the
// processor's (tests/test_unit_reads.py).
#pragma once

#ifdef __HIPCC__
#define SSM_DIV __host__ __device__ __forceinline__
#else
#define SSM_DIV inline
#endif

namespace ssm {

// floor(n / d), n and d below 2^31, d > 0: n mul >> shift with mul = ceil(2^(31 + l) / d), 2^l >= d (Granlund and Montgomery, 1994).  (Three scalar instructions; the compiler's own
// division by an argument is over twenty, one behind the other, and placing a tile takes five.  No number of rows reaches 2^31, those past the
// last token of a tile included: rows are divided in scans of more than 32 states or of few tokens, and 2^31 rows of 33 states would not fit any memory.)
struct FastDiv {
    unsigned mul, shift;
    static FastDiv by(unsigned d)
    {
        const unsigned l = d > 1 ? 32 - (unsigned)__builtin_clz(d - 1) : 0;
        return {(unsigned)(((1ull << (31 + l)) + d - 1) / d), 31 + l};
    }
    SSM_DIV unsigned operator()(unsigned n) const { return (unsigned)(((unsigned long long)n * mul) >> shift); }
};

}  // namespace ssm
