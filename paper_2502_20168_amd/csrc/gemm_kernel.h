// Operand staging of the projection products and the kernel of the reductions over tokens (gfx950).
//
//   C[m,n] = sum_k A[k,m] * B[k,n],   A, B, C fp32, k = tokens          (dC = dy^T x, dBbar = chi^T u, dW = x1^T dz)
//
// Every fp32 operand value a is split exactly into three bf16 numbers a = a1 + a2 + a3
// (a1 = trunc_bf16(a), a2 = trunc_bf16(a - a1), a3 = a - a1 - a2; 8 + 8 + 8 mantissa bits).  The
// product a*b is then accumulated in fp32 from the six partial products whose weight is at
// least 2^-16 of the leading one (a1b1, a1b2, a2b1, a1b3, a2b2, a3b1); the three dropped ones
// are below 2^-24 |a||b|, i.e. at the level of one fp32 rounding.  Each partial product of two
// bf16 numbers is exact in fp32, so the result has fp32-class accuracy, while the six
// v_mfma_f32_32x32x16_bf16 (32 cycles for 32x32x16 MACs) cost 192 cycles where the fp32 matrix
// instruction needs 512 cycles for the same 32x32x16 block.  Where the largest magnitude of both operands
// is known, two scaled fp16 planes and three products do (see split2_f16).
//
// The split happens once per staged element, between the global load and the LDS store.
#pragma once

#include "gemm_common.h"
#include "lookback.h"

#include <atomic>

namespace ssm {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

struct Split4 { bf16x4 p[3]; };

// four consecutive floats at an address that is only float-aligned (one 16-byte load: global loads need dword alignment)
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));
// Four consecutive values of a row from p, n of which exist (an address that is only float-aligned).
__device__ __forceinline__ float4 load4(const float *p, int n)
{
    if (n >= 4) { const f32x4u v = *reinterpret_cast<const f32x4u *>(p); return make_float4(v.x, v.y, v.z, v.w); }
    return make_float4(n > 0 ? p[0] : 0.f, n > 1 ? p[1] : 0.f, n > 2 ? p[2] : 0.f, 0.f);
}
__device__ __forceinline__ void store4(float *p, float4 v, int n)
{
    if (n >= 4) { const f32x4u w = {v.x, v.y, v.z, v.w}; *reinterpret_cast<f32x4u *>(p) = w; return; }
    if (n > 0) p[0] = v.x;
    if (n > 1) p[1] = v.y;
    if (n > 2) p[2] = v.z;
}

// n of the four values, `at` values behind base (the same for all lanes, at most 2^29 values away)
__device__ __forceinline__ void store4_through(float *base, int at, float4 v, int n)
{
    if (n >= 4) {
        typedef int i32x4 __attribute__((ext_vector_type(4)));
        constexpr int RAW = 0x00020000, SC1 = 16;            // dwords at byte offsets; scope of the device
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i32x4, v), __builtin_amdgcn_make_buffer_rsrc(base, 0, 0x7fffffff, RAW), 4 * at, 0, SC1);
    } else store4(base + at, v, n);
}

// The four values from the sh-th on of a unit that was read sh values early: the rest zeros (sh <= 0: the unit; >= 4: zeros).
// (selections one on top of the other, on lanes: nested ones become branches on lanes, and a loop that has such a branch anywhere is
// rearranged so that its way out meets the way round, where the compiler then waits for loads that it could leave in flight)
__device__ __forceinline__ float4 shift_unit(float4 v, int sh)
{
    const bool one = (sh & 1) != 0 && sh > 0, two = (sh & 2) != 0 && sh > 0, none = sh >= 4;
    v = make_float4(one ? v.y : v.x, one ? v.z : v.y, one ? v.w : v.z, one ? 0.f : v.w);
    v = make_float4(two ? v.z : v.x, two ? v.w : v.y, two ? 0.f : v.z, two ? 0.f : v.w);
    return make_float4(none ? 0.f : v.x, none ? 0.f : v.y, none ? 0.f : v.z, none ? 0.f : v.w);
}

// Exact three-way split of four floats by truncation: a1 = the upper 16 bits of a, a2 = the
// upper 16 bits of a - a1, a3 = a - a1 - a2 (which has at most 8 significant bits left, so its
// upper 16 bits hold it exactly).  Only full-rate integer/float VALU operations are used; two
// bf16 values are packed with one byte permute.
__device__ __forceinline__ void split3_one(float x, unsigned &h, unsigned &m, unsigned &l)
{
    h = __float_as_uint(x) & 0xffff0000u;
    const float r1 = x - __uint_as_float(h);
    m = __float_as_uint(r1) & 0xffff0000u;
    l = __float_as_uint(r1 - __uint_as_float(m));
}
__device__ __forceinline__ Split4 split3_pack(const unsigned (&h)[4], const unsigned (&m)[4], const unsigned (&l)[4])
{
    // bytes 2,3 of the first source become the low half, bytes 2,3 of the second the high half
    union { unsigned u[2]; bf16x4 b; } ph, pm, pl;
    ph.u[0] = __builtin_amdgcn_perm(h[1], h[0], 0x07060302u); ph.u[1] = __builtin_amdgcn_perm(h[3], h[2], 0x07060302u);
    pm.u[0] = __builtin_amdgcn_perm(m[1], m[0], 0x07060302u); pm.u[1] = __builtin_amdgcn_perm(m[3], m[2], 0x07060302u);
    pl.u[0] = __builtin_amdgcn_perm(l[1], l[0], 0x07060302u); pl.u[1] = __builtin_amdgcn_perm(l[3], l[2], 0x07060302u);
    Split4 o;
    o.p[0] = ph.b; o.p[1] = pm.b; o.p[2] = pl.b;
    return o;
}
__device__ __forceinline__ Split4 split3(float4 v)
{
    unsigned h[4], m[4], l[4];
    split3_one(v.x, h[0], m[0], l[0]); split3_one(v.y, h[1], m[1], l[1]);
    split3_one(v.z, h[2], m[2], l[2]); split3_one(v.w, h[3], m[3], l[3]);
    return split3_pack(h, m, l);
}

// Two-plane split into fp16: with the operand (the whole matrix, or one row of it) scaled by a power
// of two so that its largest magnitude lies in [2^14, 2^15), a1 = rn_fp16(s a) and a2 = rn_fp16(s a - a1) (the residual is
// formed exactly by one fused multiply-add).  fp16 keeps 11 significant bits, so
// |s a - a1 - a2| <= 2^-22 |s a| as long as a2 is a normal fp16 number, i.e. for |a| down to 2^-17
// of the largest magnitude; below that the planes act as a fixed-point pair with an absolute error
// of at most 2^-25 (half the spacing of the fp16 subnormals) in scaled units, i.e. 2^-39 of the
// largest magnitude.  The three products a1b1, a1b2, a2b1 (each exact in fp32) then leave a
// relative error of about 3 * 2^-22 per product term at worst -- the level of fp32 rounding -- for
// half the matrix instructions of the three-way bf16 split.  The scale is taken off the
// accumulators before anything is stored.
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ Split4 split2_f16(float4 v, float s)
{
    const f32x2 a = {v.x * s, v.y * s}, b = {v.z * s, v.w * s};
    union { f16x2 h; unsigned u; } ha, hb, la, lb;
    ha.h = __builtin_convertvector(a, f16x2);
    hb.h = __builtin_convertvector(b, f16x2);
    const f32x2 ra = {__builtin_fmaf(v.x, s, -(float)ha.h.x), __builtin_fmaf(v.y, s, -(float)ha.h.y)};
    const f32x2 rb = {__builtin_fmaf(v.z, s, -(float)hb.h.x), __builtin_fmaf(v.w, s, -(float)hb.h.y)};
    la.h = __builtin_convertvector(ra, f16x2);
    lb.h = __builtin_convertvector(rb, f16x2);
    union { unsigned u[2]; bf16x4 b; } p0, p1;       // bf16x4 is only the 8-byte container of the LDS store
    p0.u[0] = ha.u; p0.u[1] = hb.u;
    p1.u[0] = la.u; p1.u[1] = lb.u;
    Split4 o;
    o.p[0] = p0.b; o.p[1] = p1.b; o.p[2] = p1.b;
    return o;
}
// The same values by fused multiply-adds that round to fp16 on the way out, two instructions per element instead of three
// (held opaque, because the compiler otherwise forms the upper half of the first plane twice).  Measured: 32768 x 512 x 1024
// 127.8 -> 121.6 us; in the reductions, whose producers have more waiting to hide, 5 % slower than the other form.
__device__ __forceinline__ Split4 split2_f16_mix(float4 v, float s)
{
    union { f16x2 h; unsigned u; } ha, hb, la, lb;
    ha.h = f16x2{(_Float16)__builtin_fmaf(v.x, s, 0.f), (_Float16)__builtin_fmaf(v.y, s, 0.f)};
    hb.h = f16x2{(_Float16)__builtin_fmaf(v.z, s, 0.f), (_Float16)__builtin_fmaf(v.w, s, 0.f)};
    asm("" : "+v"(ha.u)); asm("" : "+v"(hb.u));
    la.h = f16x2{(_Float16)__builtin_fmaf(v.x, s, -(float)ha.h.x), (_Float16)__builtin_fmaf(v.y, s, -(float)ha.h.y)};
    lb.h = f16x2{(_Float16)__builtin_fmaf(v.z, s, -(float)hb.h.x), (_Float16)__builtin_fmaf(v.w, s, -(float)hb.h.y)};
    union { unsigned u[2]; bf16x4 b; } p0, p1;       // bf16x4 is only the 8-byte container of the LDS store
    p0.u[0] = ha.u; p0.u[1] = hb.u;
    p1.u[0] = la.u; p1.u[1] = lb.u;
    Split4 o;
    o.p[0] = p0.b; o.p[1] = p1.b; o.p[2] = p1.b;
    return o;
}
template <int NPL>
__device__ __forceinline__ Split4 split_planes(float4 v, float s) { return NPL == 3 ? split3(v) : split2_f16(v, s); }

// log2 of the power-of-two scale that brings the largest magnitude of an operand into [2^14, 2^15):
// every lane of the wavefront gets the same value.  The slots hold bit patterns of non-negative
// floats, which order like unsigned integers.  An operand of zeros gets the largest scale (its
// planes are zeros whatever the scale).  Two steps, so that the loads can be issued ahead of other
// memory traffic and waited for behind it: absmax_issue starts eight independent loads per lane (the
// first 512 slots), absmax_log2_scale reduces them (and walks the slots beyond 512, if any).
__device__ __forceinline__ int log2_scale_of(unsigned maxbits);
struct AbsMaxLoads { unsigned w[8]; };
__device__ __forceinline__ AbsMaxLoads absmax_issue(const AbsMax &m, int lane)
{
    AbsMaxLoads r;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int i = lane + 64 * j;
        const unsigned t = m.slots[i < m.n ? i : 0];         // unconditional, so that the loads overlap
        r.w[j] = i < m.n ? t : 0u;
    }
    return r;
}
__device__ __forceinline__ int absmax_log2_scale(const AbsMax &m, const AbsMaxLoads &r, int lane)
{
    unsigned v = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) v = max(v, r.w[j]);
    for (int base = 512; base < m.n; base += 512) {          // more than 512 slots: eight more per lane at a time
        unsigned w[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int i = base + lane + 64 * j;
            const unsigned t = m.slots[i < m.n ? i : 0];
            w[j] = i < m.n ? t : 0u;
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) v = max(v, w[j]);
    }
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, o));
    return log2_scale_of(v);     // (defined below) 14 - floor(log2(maximum)), kept inside the exponent range
}
__device__ __forceinline__ float pow2f(int e) { return __uint_as_float((unsigned)(e + 127) << 23); }   // e in [-127, 127]
__device__ __forceinline__ int log2_scale_of(unsigned maxbits)
{
    const int e = (int)((maxbits >> 23) & 0xffu);
    int f = 268 - e;
    f = f < 1 ? 1 : (f > 254 ? 254 : f);
    return f - 127;
}
// Stages one BK x R fp32 operand tile (R contiguous rows of C's index, k slow): global -> registers (fp32) -> split ->
// NPL LDS planes [k][row] -- the same orientation as in memory, so global loads are whole lines and nothing is
// transposed here; the consumers fetch their fragments with the transposing LDS read.
// A thread handles units of 1 k x 4 rows and writes the four 16-bit values of every plane with one 8-byte store.
// The 64-byte pieces of a k row are permuted (see place) so that a transposing read, which takes one piece of four
// consecutive k, meets every bank once.  (With a k stride of R + 16 halves instead, two k rows shared half their banks:
// the reads of a 128 x 128 x 32 tile took 1.3 us where its matrix instructions take 0.35.)
template <int R, int BK, int NT, int NPL>
struct SplitLoader {
    static constexpr int NV = R * BK / 4 / NT;
    static_assert(NV >= 1 && NV * NT * 4 == R * BK, "tile must be a multiple of the workgroup's float4 loads");
    static constexpr int S = R;                           // stride of k in halves
    static constexpr int PLANE = BK * S;                  // halves per plane
    float4 r[NV];

    // place of 32-row piece c of k row k, in units of 32 halves
    static __device__ __forceinline__ int place(int k, int c) { return R == 128 ? c ^ (k & 3) : c ^ ((k >> 1) & 1); }

    // EDGE 1: the tile hangs over the last row.  A unit past the end reads the operand's last four rows instead (shifted
    // into place where part of it lies inside: the rest only reaches output rows that are never stored), so that it
    // is still one 16-byte load.  EDGE 2: operands of less than four rows, value by value.
    // Rows of k past the end of the range re-read the last one; store() zeroes them.  (No branch around the loads:
    // where paths with different numbers of loads in flight meet, the compiler waits for the larger one, which cost a
    // whole K tile of prefetch distance.)
    // (a uniform base and a 32-bit offset per unit: addresses in full cost as much as half of the split)
    template <int EDGE>
    __device__ __forceinline__ void load(const float *X, long ld, int row0, int rows, int k0, int kend, int tid)
    {
        static_assert(NT % (R / 4) == 0, "a thread keeps its rows");
        const int gr = row0 + 4 * (tid % (R / 4));
        const unsigned gc = 4u * (unsigned)(EDGE == 1 ? min(gr, rows - 4) : gr);
        const int kb = min(k0, kend - 1), kmax = kend - 1 - kb;
        const char *base = reinterpret_cast<const char *>(X + (long)kb * ld);
        const unsigned pitch = 4u * (unsigned)ld;
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const unsigned k = (unsigned)min((tid + i * NT) / (R / 4), kmax);
            if (EDGE == 2) {
                const float *p = reinterpret_cast<const float *>(base + k * pitch);
                r[i] = make_float4(p[min(gr, rows - 1)], p[min(gr + 1, rows - 1)], p[min(gr + 2, rows - 1)], p[min(gr + 3, rows - 1)]);
            } else {
                const f32x4u v = *reinterpret_cast<const f32x4u *>(base + (k * pitch + gc));
                r[i] = make_float4(v.x, v.y, v.z, v.w);
            }
        }
    }
    // EDGE 1: moves the values of a unit that was read early into place: every unit that is partly inside by the same number of values, what lies past the end
    // is any value (five selections per unit; with shift_unit's twelve the du launch of 22 x 512 tokens, H = 675, P = 457 took 203 us, now 181, the gate's 152 and 144)
    __device__ __forceinline__ void shift(int row0, int rows, int tid)
    {
        const bool late = row0 + 4 * (tid % (R / 4)) > rows - 4, one = late && (-rows & 1), two = late && (-rows & 2);
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            float4 &v = r[i];
            v.x = one ? v.y : v.x; v.y = one ? v.z : v.y; v.z = one ? v.w : v.z;
            v.x = two ? v.z : v.x; v.y = two ? v.w : v.y;
        }
    }
    // zeroes what lies past the end of the range in the tile at k0 (its last)
    __device__ __forceinline__ void cut(int k0, int kend, int tid)
    {
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (k0 + (tid + i * NT) / (R / 4) >= kend) r[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }

    // scale: two-plane staging only (a power of two, see split2_f16)
    __device__ __forceinline__ void store(__bf16 *lds, int tid, float scale) const
    {
#pragma unroll
        for (int i = 0; i < NV; ++i) {
            const int idx = tid + i * NT;
            const int k = idx / (R / 4), row = 4 * (idx % (R / 4)), off = k * S + 32 * place(k, row / 32) + row % 32;
            const Split4 sp = split_planes<NPL>(r[i], scale);
#pragma unroll
            for (int s = 0; s < NPL; ++s) *reinterpret_cast<bf16x4 *>(lds + s * PLANE + off) = sp.p[s];
        }
    }

    // Fragment of a 32-row block for one 16-wide k step: lane (li = l % 32, hh = l / 32) gets the 8 values row0 + li,
    // k = kbase + 8 hh .. 8 hh + 7 of a plane by two transposing 8-byte reads.  ds_read_b64_tr_b16 works on groups of
    // 16 lanes: lane i of a group receives element i % 4 of the 8-byte chunks addressed by lanes i / 4, i / 4 + 4,
    // i / 4 + 8, i / 4 + 12 of the group.  With lane sl of a group pointing at [k0 + sl / 4][m0 + 4 (sl % 4)], lane i
    // receives rows m0 + i at k0 .. k0 + 3.
    static __device__ __forceinline__ bf16x8 fragment(const __bf16 *plane, int row0, int kbase, int l)
    {
        typedef short v4s __attribute__((ext_vector_type(4)));
        const int sl = l & 15, grp = l >> 4;
        const __bf16 *p0 = plane + (kbase + 8 * (grp >> 1) + (sl >> 2)) * S + 32 * place(sl >> 2, row0 / 32) + 16 * (grp & 1) + 4 * (sl & 3);
        union { v4s h[2]; bf16x8 v; } u;
        u.h[0] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((v4s __attribute__((address_space(3))) *)(p0));
        u.h[1] = __builtin_amdgcn_ds_read_tr16_b64_v4i16((v4s __attribute__((address_space(3))) *)(p0 + 4 * S));
        return u.v;
    }
};

template <int CTRL>
__device__ __forceinline__ unsigned dpp_move(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}
// max(v, v of lane ^ 16) or max(v, v of lane ^ 32) with the lane-swap instructions of gfx950 (given the
// same register twice, v_permlane16_swap / v_permlane32_swap return it and its copy from the partner row
// or half): no LDS involved
template <int X>
__device__ __forceinline__ unsigned lane_xor_max(unsigned v)
{
    static_assert(X == 16 || X == 32, "rows of 16 lanes or halves of 32");
    if constexpr (X == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return max((unsigned)r[0], (unsigned)r[1]);
    } else {
        const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
        return max((unsigned)r[0], (unsigned)r[1]);
    }
}
// ---------------------------------------------------------------------------------------------
// Wavefront specialisation: a workgroup has four consumer wavefronts (2 x 2) that only read operand fragments from
// LDS and issue MFMAs, and four producer wavefronts that only stage tiles (global load -> split -> LDS).  A producer
// and a consumer share each SIMD, so the VALU work of the split co-executes with the matrix instructions of the other
// wavefront.  Two LDS stages: in iteration kt the producers fill the stage of tile kt+1 while the consumers work
// on tile kt, with one workgroup barrier per K tile.  128 x 128 tiles (three planes 128 x 64), or 64 x 64 where the products of
// the launch are small; two workgroups share a CU, so that one's first loads and stores overlap the other's K loop.
//   Beside small products eight wavefronts of either kind and 64 k per K tile take half as long for an item of 64 x 64, but every workgroup of the launch then has a CU to
// itself, products of eight wavefronts included, and launches of more workgroups than CUs take two rounds.  Gradient pass in that form and with four of either kind, 32 k and two
// workgroups per CU: 20 x 64, 300, 300: 48.0 and 39.4 us; 30 x 60, 256, 200: 40.9 and 33.9; 6 x 100, 600, 600: 64.5 and 55.3.  The lines between the forms: products3.hip.
// ---------------------------------------------------------------------------------------------
constexpr int TN_STAGES = 2;
constexpr int TN_BK = 32;
// Tiles by name: 128 = 128 x 128, 96 = 128 x 64 (three planes: half the registers and three quarters of the LDS of a square
// tile, so that two workgroups share a CU here too), 64 = 64 x 64, 65 = 64 x 64 by eight wavefronts of either kind.
constexpr int tn_rows(int TB) { return TB < 96 ? 64 : 128; }
constexpr int tn_cols(int TB) { return TB == 128 ? 128 : 64; }
constexpr int tn_wavefronts(int TB) { return TB == 65 ? 8 : 4; }
// (stages, two scales)
constexpr size_t tn_lds_bytes(int TB, int NPL, int BK) { return (size_t)TN_STAGES * NPL * BK * (tn_rows(TB) + tn_cols(TB)) * 2 + (NPL == 2 ? 16 : 0); }

template <int TB, int NPL, int EDGE, int BK>
__device__ __forceinline__ void gemm_tn_tile(const GemmDev &g, __bf16 *stages, int m0, int n0, int z, int kbeg, int kend, int tid)
{
    constexpr int TM = tn_rows(TB), TN = tn_cols(TB), NS = TN_STAGES, NC = tn_wavefronts(TB), KG = NC / 4, NP = NC, PT = 64 * NP;
    // K tiles of global loads in flight per producer (128 x 128 tiles: 3, 4 and 6 measured 1-5 % slower)
    constexpr int PF = TB == 65 ? 4 : TB == 64 && BK == TN_BK ? 3 : 2;
    using LA = SplitLoader<TM, BK, PT, NPL>;
    using LB = SplitLoader<TN, BK, PT, NPL>;
    static_assert(NPL == 2 || NPL == 3, "three bf16 planes or two scaled fp16 planes per operand");
    constexpr int STAGE_A = NPL * LA::PLANE, STAGE = STAGE_A + NPL * LB::PLANE;
    // two-plane staging: log2 of the scales of A and B, written by the producers before the first barrier and read by
    // the consumers after the K loop
    int *opexp = reinterpret_cast<int *>(stages + NS * STAGE);
    constexpr int WM = TM / 2, WN = TN / 2, MI = WM / 32, NI = WN / 32;

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nk = (kend - kbeg + BK - 1) / BK;   // (the range is not empty)

    if (wave >= NC) {
        // ------------------------------------------------------------------ producers
        // PF register sets: while tile t is split and stored, the loads of tiles t+1 .. t+PF are in flight
        const int ptid = tid - 64 * NC;
        LA la[PF];
        LB lb[PF];
        auto fetch = [&](int set, int t) {
            la[set].template load<EDGE>(g.A, g.lda, m0, g.M, kbeg + t * BK, kend, ptid);
            lb[set].template load<EDGE>(g.B, g.ldb, n0, g.N, kbeg + t * BK, kend, ptid);
        };
        float sa = 1.f, sb = 1.f;
        AbsMaxLoads ma, mb;
        if constexpr (NPL == 2) {
            if (wave == NC) { ma = absmax_issue(g.amaxA, tid & 63); mb = absmax_issue(g.amaxB, tid & 63); }
        }
#pragma unroll
        for (int j = 0; j < PF; ++j) fetch(j, j);
        if constexpr (NPL == 2) {
            if (wave == NC) {
                const int ea = absmax_log2_scale(g.amaxA, ma, tid & 63), eb = absmax_log2_scale(g.amaxB, mb, tid & 63);
                if ((tid & 63) == 0) { opexp[0] = ea; opexp[1] = eb; }
            }
            __syncthreads();                      // (the consumers wait here as well)
            sa = pow2f(opexp[0]); sb = pow2f(opexp[1]);
        }
        const int ktail = (kend - kbeg) % BK != 0 ? nk - 1 : nk;         // the K tile that hangs over the end of the range
        auto stash = [&](int set, int t) {
            if (t == ktail) {
                la[set].cut(kbeg + t * BK, kend, ptid);
                lb[set].cut(kbeg + t * BK, kend, ptid);
            }
            if constexpr (EDGE == 1) {
                la[set].shift(m0, g.M, ptid);
                lb[set].shift(n0, g.N, ptid);
            }
            __bf16 *st = stages + (t % NS) * STAGE;
            la[set].store(st, ptid, sa);
            lb[set].store(st + STAGE_A, ptid, sb);
        };
        static_assert(NS == 2, "the loop below");
        stash(0, 0);
        fetch(0, PF);
        __syncthreads();
        // step kt stages tile kt + 1 from register set (kt + 1) % PF while the consumers work on tile kt (whole rounds, then
        // what is left: see gemm_pk_tile)
        auto step = [&](int kt, int j) {
            stash((j + 1) % PF, kt + j + 1);
            fetch((j + 1) % PF, kt + j + 1 + PF);
            __syncthreads();
        };
        int kt = 0;
        for (; kt + PF < nk; kt += PF) {
#pragma unroll
            for (int j = 0; j < PF; ++j) step(kt, j);
        }
#pragma unroll
        for (int j = 0; j + 1 < PF; ++j)
            if (kt + j + 1 < nk) step(kt, j);
        __syncthreads();
        if constexpr (KG > 1) __syncthreads();
        return;
    }

    // ---------------------------------------------------------------------- consumers
    const int l = tid & 63;
    const int kg = KG > 1 ? wave / 4 : 0, wm = (KG > 1 ? wave % 4 : wave) / 2, wn = wave % 2;
    const int li = l & 31, hh = l >> 5;
    v16f acc[MI][NI];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    // A single block per wavefront: the five small products of a k step go into two accumulators of their own.  The large one is then rounded once per
    // step instead of six times (errors of sums of exact operands against 64 bits: 0.39 to 0.47 of those in one accumulator, 0.37 to 0.46 where two wavefronts share out the
    // steps), and the chain of dependent matrix instructions is half as long.
    constexpr bool APART = MI == 1 && NI == 1 && NPL == 3;
    v16f small[2];
#pragma unroll
    for (int r = 0; r < 16; ++r) small[0][r] = small[1][r] = 0.f;

    // Software pipeline over the 16-wide k steps: the fragments of step s+1 are requested from LDS before the matrix
    // instructions of step s are issued.  At the last step of a K tile the workgroup barrier comes first: it both
    // releases the stage just read (all its reads have completed, they feed the instructions about to be
    // issued) and guarantees that the next stage is filled.
    constexpr int KS = BK / 16 / KG;              // k steps of a tile per wavefront
    static_assert(KS % 2 == 0, "k steps per tile: even");
    bf16x8 fa[2][MI][NPL], fb[2][NI][NPL];
    auto fetch_frags = [&](int set, int kt, int ks) {
        const __bf16 *st = stages + (kt % NS) * STAGE;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int s = 0; s < NPL; ++s) fa[set][i][s] = LA::fragment(st + s * LA::PLANE, wm * WM + i * 32, (kg * KS + ks) * 16, l);
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int s = 0; s < NPL; ++s) fb[set][j][s] = LB::fragment(st + STAGE_A + s * LB::PLANE, wn * WN + j * 32, (kg * KS + ks) * 16, l);
    };
    // the products of one accumulator keep their order (smallest first); the MI*NI accumulators alternate so that
    // consecutive matrix instructions are independent
    auto multiply = [&](int set) {
        // three planes: a3b1, a2b2, a1b3, a2b1, a1b2, a1b1;  two planes: a2b1, a1b2, a1b1
        constexpr int NPROD = NPL == 3 ? 6 : 3;
        constexpr int PA3[6] = {2, 1, 0, 1, 0, 0}, PB3[6] = {0, 1, 2, 0, 1, 0};
        constexpr int PA2[3] = {1, 0, 0}, PB2[3] = {0, 1, 0};
#pragma unroll
        for (int p = 0; p < NPROD; ++p)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const int pa = NPL == 3 ? PA3[p] : PA2[p % 3], pb = NPL == 3 ? PB3[p] : PB2[p % 3];
                    if constexpr (NPL == 3) {
                        v16f &c = APART && p + 1 < NPROD ? small[p & 1] : acc[i][j];
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[set][i][pa], fb[set][j][pb], c, 0, 0, 0);
                    }
                    else
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fa[set][i][pa]),
                                                                           __builtin_bit_cast(f16x8, fb[set][j][pb]), acc[i][j], 0, 0, 0);
                }
    };
    // issue order of one k step: fragment reads in the shadow of its first matrix instructions (a burst of reads would keep
    // the wavefront from issuing matrix work), so that the last ones hide the latency of the reads behind them
    auto interleave = [&]() {
        constexpr int NREAD = 2 * NPL * (MI + NI), NMFMA = (NPL == 3 ? 6 : 3) * MI * NI, PER = (3 * NREAD + 2 * NMFMA - 1) / (2 * NMFMA);
        static_assert(NREAD % PER == 0, "reads per matrix instruction");
#pragma unroll
        for (int q = 0; q < NREAD / PER; ++q) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, PER, 0);
        }
        __builtin_amdgcn_sched_group_barrier(0x008, NMFMA - NREAD / PER, 0);
    };
    if constexpr (NPL == 2) __syncthreads();      // the producers have put log2 of the scales into opexp
    __syncthreads();
    fetch_frags(0, 0, 0);
    for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            if (ks + 1 < KS) {
                fetch_frags((ks + 1) & 1, kt, ks + 1);
            } else {
                __syncthreads();
                fetch_frags(0, kt + 1, 0);        // past the last tile: a harmless read of a stale stage
            }
            multiply(ks & 1);
            interleave();
        }
    }
    if constexpr (APART) {
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] += small[0][r] + small[1][r];
    }
    if constexpr (KG > 1) {
        static_assert(MI == 1 && NI == 1 && NPL == 3, "one block per wavefront");
        float *part = reinterpret_cast<float *>(stages) + wave % 4 * 1024 + l;
        if (kg == 1) {
#pragma unroll
            for (int r = 0; r < 16; ++r) part[r * 64] = acc[0][0][r];
        }
        __syncthreads();
        if (kg == 1) return;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][0][r] += part[r * 64];
    }
    if constexpr (NPL == 2) {
        // one exponent adjustment per element takes both scales off (exact; their sum can leave the exponent range of
        // a single factor)
        const int st = opexp[0] + opexp[1];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][j][r] = __builtin_ldexpf(acc[i][j][r], -st);
    }
    float *Cz = g.C + (long)z * g.M * g.ldc;
    const bool full = (m0 + TM <= g.M) && (n0 + TN <= g.N);      // no store of this tile needs a bounds check
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int col = n0 + wn * WN + j * 32 + li;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const long row = m0 + wm * WM + i * 32 + 8 * (r / 4) + 4 * hh + (r % 4);
                if (full || (row < g.M && col < g.N)) store_through(Cz + row * g.ldc + col, acc[i][j][r]);
            }
        }
}

// Work item (tile, split) of the workgroup in slot q of XCD x: every XCD owns whole K slabs (or, with fewer than 8
// splits, one contiguous band of the tiles of one slab), so each operand element is fetched from memory once
// instead of once per tile band.
__device__ __forceinline__ void tn_place(const GemmDev &g, int x, int q, int &z, int &tile)
{
    if (g.mode == 0) { z = 0; tile = x * g.nx + q; return; }
    const int n = g.mode == 1 ? q : g.mode == 2 ? x : x * g.nx + q, d = (int)g.by_par(n), rest = n - d * g.par;
    if (g.mode == 1) { z = x + 8 * rest; tile = d; }                              // splits = 8 * par
    else if (g.mode == 2) { z = rest; tile = d * g.nx + q; }                      // 8 = splits * bands of nx tiles, par = splits
    else { z = d; tile = rest; }                                                  // par = tiles
}

template <int TB, int NPL, int BK>
__device__ __forceinline__ void gemm_tn_problem(const GemmDev &g, unsigned char *smem, int x, int q, int tid)
{
    int z, tile;
    tn_place(g, x, q, z, tile);
    if (q >= g.nx || z >= g.splits || tile >= g.ntm * g.ntn) return;
    constexpr int TM = tn_rows(TB), TN = tn_cols(TB);
    const int tm = (int)g.by_ntn(tile), m0 = tm * TM, n0 = (tile - tm * g.ntn) * TN;
    const int kbeg = z * g.kper, kend = min(g.K, kbeg + g.kper);
    __bf16 *stages = reinterpret_cast<__bf16 *>(smem);
    if (kbeg >= kend) {
        // more splits than K tiles: a slab of zeros
        float *Cz = g.C + (long)z * g.M * g.ldc;
        for (int i = tid; i < TM * TN; i += blockDim.x) {
            const int row = m0 + i / TN, col = n0 + i % TN;
            if (row < g.M && col < g.N) Cz[(long)row * g.ldc + col] = 0.f;
        }
    } else if (m0 + TM <= g.M && n0 + TN <= g.N) {
        gemm_tn_tile<TB, NPL, 0, BK>(g, stages, m0, n0, z, kbeg, kend, tid);
    } else if (g.M >= 4 && g.N >= 4) {
        gemm_tn_tile<TB, NPL, 1, BK>(g, stages, m0, n0, z, kbeg, kend, tid);
    } else {
        gemm_tn_tile<TB, NPL, 2, BK>(g, stages, m0, n0, z, kbeg, kend, tid);
    }
}

template <int TB>
inline GemmDev make_tn_dev(const GemmArgs &a)
{
    constexpr int BK = TN_BK;
    GemmDev g{};
    g.A = a.A; g.lda = a.lda; g.B = a.B; g.ldb = a.ldb; g.C = a.C; g.ldc = a.ldc;
    g.M = a.M; g.N = a.N; g.K = a.K;
    const int splits = a.splits < 1 ? 1 : a.splits;
    int kper = (a.K + splits - 1) / splits;
    kper = (kper + BK - 1) / BK * BK;
    g.kper = kper;
    g.ntm = (a.M + tn_rows(TB) - 1) / tn_rows(TB);
    g.ntn = (a.N + tn_cols(TB) - 1) / tn_cols(TB);
    const long ntiles = (long)g.ntm * g.ntn;
    g.splits = splits;
    if (splits == 1) { g.mode = 0; g.par = 1; g.nx = (int)((ntiles + 7) / 8); }
    else if (splits % 8 == 0) { g.mode = 1; g.par = splits / 8; g.nx = (int)(ntiles * g.par); }
    else if (8 % splits == 0) { g.mode = 2; g.par = splits; g.nx = (int)((ntiles * splits + 7) / 8); }
    else { g.mode = 3; g.par = (int)ntiles; g.nx = (int)((ntiles * splits + 7) / 8); }
    g.by_ntn = FastDiv::by(g.ntn); g.by_par = FastDiv::by(g.par);
    g.amaxA = a.amaxA; g.amaxB = a.amaxB;
    return g;
}

// Raises the dynamic LDS limit of a kernel that needs more than 64 KB, once per kernel and device (the attribute belongs
// to the device's copy of the kernel; raising it is idempotent).
constexpr int KERNEL_MAXDEV = 64;
inline hipError_t raise_lds_limit(const void *kern, size_t smem, std::atomic<bool> (&raised)[KERNEL_MAXDEV])
{
    if (smem <= 64 * 1024) return hipSuccess;
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    const bool keep = dev >= 0 && dev < KERNEL_MAXDEV;
    if (keep && raised[dev].load(std::memory_order_acquire)) return hipSuccess;
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)smem);
    if (e == hipSuccess && keep) raised[dev].store(true, std::memory_order_release);
    return e;
}

}  // namespace ssm
