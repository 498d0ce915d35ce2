// Parameter-sized kernels: zero-order-hold discretisation with operand packing for the
// projection GEMMs, the column dot product behind dD, and the adjoint of the discretisation.
// The handful of transcendental evaluations per state run in double precision: they are
// P-sized (a few hundred values), and the (exp(z) - 1)/z quotient cancels badly in fp32 for the
// small |Lambda Delta| that slowly decaying states have.
#include "pack.h"

#include <type_traits>

namespace ssm {

// ---------------------------------------------------------------------------------------------
// partial[s][h] = sum_{t in slab s} a[t,h] * b[t,h]      (dD = sum_t dy_t (.) u_t), and largest magnitudes
// ---------------------------------------------------------------------------------------------
// maximum of v over the wavefront, valid in lane 63 (data-parallel-primitive moves only: inside quads,
// inside rows of 16 lanes, then the last lane of a row broadcast to the following rows)
__device__ __forceinline__ unsigned wave_max_lane63(unsigned v)
{
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0xb1, 0xf, 0xf, false));    // quad_perm [1,0,3,2]
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x4e, 0xf, 0xf, false));    // quad_perm [2,3,0,1]
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x124, 0xf, 0xf, false));   // row_ror:4
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x128, 0xf, 0xf, false));   // row_ror:8
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x142, 0xa, 0xf, false));   // row_bcast:15 into rows 1, 3
    v = max(v, (unsigned)__builtin_amdgcn_update_dpp((int)v, (int)v, 0x143, 0xc, 0xf, false));   // row_bcast:31 into rows 2, 3
    return v;
}

// Four values per lane -> lane l < 4 of every sixteen gets the maximum over the sixteen of value 2 (l & 1) + (l >> 1): two halving
// steps inside the quads (lanes that differ in bit 0, then bit 1, swap the half the other keeps), two rotations.
__device__ __forceinline__ unsigned row16_max4(unsigned v0, unsigned v1, unsigned v2, unsigned v3, int lane)
{
    const bool up0 = lane & 1, up1 = (lane >> 1) & 1;
    const unsigned k0 = up0 ? v2 : v0, s0 = up0 ? v0 : v2, k1 = up0 ? v3 : v1, s1 = up0 ? v1 : v3;
    const unsigned w0 = max(k0, dpp_move<0xb1>(s0)), w1 = max(k1, dpp_move<0xb1>(s1));      // quad_perm [1,0,3,2]
    const unsigned k = up1 ? w1 : w0, sd = up1 ? w0 : w1;
    unsigned v = max(k, dpp_move<0x4e>(sd));                                                // quad_perm [2,3,0,1]
    v = max(v, dpp_move<0x124>(v));                                                         // row_ror:4
    return max(v, dpp_move<0x128>(v));                                                      // row_ror:8
}

// largest bit pattern of the non-negative floats v of a workgroup of NT threads, valid in every thread
template <int NT>
__device__ __forceinline__ unsigned block_absmax(float v)
{
    __shared__ unsigned wmax[NT / 64];
    unsigned u = wave_max_lane63(__float_as_uint(v));
    __syncthreads();                                         // (wmax may still be read from an earlier call)
    if ((threadIdx.x & 63) == 63) wmax[threadIdx.x >> 6] = u;
    __syncthreads();
    u = 0;
#pragma unroll
    for (int w = 0; w < NT / 64; ++w) u = max(u, wmax[w]);
    return u;
}

// partial[slab][64 columns of a block] and, where asked, the largest magnitudes of the pieces of a and b and arow (may be null):
// [colblocks][T], the largest magnitude of a[t, 64 columns of the block] per row t.  Sixteen lanes take a row's 64 columns, 16 bytes
// each, a wavefront four rows, and up to four such steps of both operands are in flight (rows past the slab re-read its last
// one and count as zeros).
template <int NT>
__device__ __forceinline__ void coldot_block(const ColDotArgs &a, int colblock, int slab, unsigned *amax, unsigned *bmax, int slot,
                                             unsigned *arow, float *red)
{
    constexpr int STEP = NT / 16;                            // rows of a step
    const int tid = threadIdx.x, unit = tid & 15;
    const int col = colblock * 64 + 4 * unit, n = a.H - col; // columns of this lane that exist: 4 or more, or none, unless cut
    // (a unit that hangs over the end of its row reads the row's last four values, moved into place once all are on their way; as four
    // requests of one value behind a branch each, the prep launch of 4096 tokens, H = 110, P = 128 took 12.3 us, now 7.4)
    const bool narrow = a.H < 4, cut = a.H % 4 != 0 && colblock * 64 + 64 > a.H;
    const int cc = min(col, a.H - 4);
    const long rows_per = (a.T + a.nslab - 1) / a.nslab;
    const long r0 = slab * rows_per, r1 = min((long)a.T, r0 + rows_per);
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    float ma = 0.f, mb = 0.f;
    unsigned *arow_cb = arow ? arow + (size_t)colblock * a.T : nullptr;
    auto load = [&](const float *p) {
        if (narrow) return make_float4(p[0], p[a.H > 1 ? 1 : 0], p[a.H > 2 ? 2 : 0], 0.f);
        const f32x4u w = *reinterpret_cast<const f32x4u *>(p + cc);
        return make_float4(w.x, w.y, w.z, w.w);
    };
    auto take = [&](long t0, auto steps) {
        constexpr int N = decltype(steps)::value;
        const long t = t0 + tid / 16;
        float4 av[N], bv[N];
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const long r = min(t + j * STEP, r1 - 1) * a.H;
            av[j] = load(a.a + r);
            bv[j] = load(a.b + r);
        }
        if (cut && !narrow) {
#pragma unroll
            for (int j = 0; j < N; ++j) { av[j] = shift_unit(av[j], col - cc); bv[j] = shift_unit(bv[j], col - cc); }
        }
        unsigned rm[4] = {0, 0, 0, 0};
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const bool in = t + j * STEP < r1;
            const bool c0 = in && n > 0, c1 = in && n > 1, c2 = in && n > 2, c3 = in && n > 3;
            const float4 x = make_float4(c0 ? av[j].x : 0.f, c1 ? av[j].y : 0.f, c2 ? av[j].z : 0.f, c3 ? av[j].w : 0.f);
            const float4 y = make_float4(c0 ? bv[j].x : 0.f, c1 ? bv[j].y : 0.f, c2 ? bv[j].z : 0.f, c3 ? bv[j].w : 0.f);
            s = make_float4(fmaf(x.x, y.x, s.x), fmaf(x.y, y.y, s.y), fmaf(x.z, y.z, s.z), fmaf(x.w, y.w, s.w));
            const float mr = fmaxf(fmaxf(fabsf(x.x), fabsf(x.y)), fmaxf(fabsf(x.z), fabsf(x.w)));
            rm[j] = __float_as_uint(mr);
            ma = fmaxf(ma, mr);
            mb = fmaxf(mb, fmaxf(fmaxf(fabsf(y.x), fabsf(y.y)), fmaxf(fabsf(y.z), fabsf(y.w))));
        }
        if (arow_cb) {
            // lane l < 4 of the sixteen gets the row's maximum of step 2 (l & 1) + (l >> 1)
            const unsigned m = row16_max4(rm[0], rm[1], rm[2], rm[3], unit);
            const int j = 2 * (unit & 1) + (unit >> 1);
            if (unit < 4 && j < N && t + j * STEP < r1) arow_cb[t + j * STEP] = m;
        }
    };
    for (long t0 = r0; t0 < r1;) {                           // (uniform)
        if (r1 - t0 > 2 * STEP) { take(t0, std::integral_constant<int, 4>{}); t0 += 4 * STEP; }
        else if (r1 - t0 > STEP) { take(t0, std::integral_constant<int, 2>{}); t0 += 2 * STEP; }
        else { take(t0, std::integral_constant<int, 1>{}); t0 += STEP; }
    }
    // over the four rows of a wavefront, then over the wavefronts in order
#pragma unroll
    for (int o = 16; o <= 32; o *= 2) {
        s.x += __shfl_xor(s.x, o); s.y += __shfl_xor(s.y, o);
        s.z += __shfl_xor(s.z, o); s.w += __shfl_xor(s.w, o);
    }
    if ((tid & 63) < 16) *reinterpret_cast<float4 *>(red + (tid >> 6) * 64 + 4 * unit) = s;
    __syncthreads();
    if (tid < 64 && colblock * 64 + tid < a.H) {
        float sum = 0.f;
#pragma unroll
        for (int w = 0; w < NT / 64; ++w) sum += red[w * 64 + tid];
        a.partial[(long)slab * a.H + colblock * 64 + tid] = sum;
    }
    if (amax) {
        const unsigned ua = block_absmax<NT>(ma), ub = block_absmax<NT>(mb);
        if (tid == 0) { amax[slot] = ua; bmax[slot] = ub; }
    }
}

// slots[row] = largest magnitude of row `row` of x[n / rowlen][rowlen].  A wavefront takes RW rows at a time
// (all their loads in flight before the first reduction): one row each while there are at least as many
// wavefronts as rows, else four -- measured on 4096 cold rows of 512 values: 2.9 us with one row per
// wavefront in 1024 workgroups, 4.7 us with four rows per wavefront in 256.
template <int RW>
__device__ __forceinline__ void absmax_rows_batch(const PrepArgs::Pass &q, size_t row0, size_t rows, int lane)
{
    float m[RW];
#pragma unroll
    for (int r = 0; r < RW; ++r) m[r] = 0.f;
    if (q.vec && q.rowlen <= 512) {
        // up to two float4 per lane and row: 2 RW independent loads
        float4 a[RW][2];
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int i = lane + 64 * h;
                const bool ok = row0 + r < rows && i < q.rowlen / 4;
                const float4 *x4 = reinterpret_cast<const float4 *>(q.x + (ok ? row0 + r : 0) * (size_t)q.rowlen);
                a[r][h] = x4[ok ? i : 0];
            }
        // (held here, or the compiler moves every load into the branch of its selection below, where it is waited for before the next:
        // 16384 rows of 512 values took 11.2 us in the prep launch, now 9.7)
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h) asm volatile("" : "+v"(a[r][h].x), "+v"(a[r][h].y), "+v"(a[r][h].z), "+v"(a[r][h].w));
#pragma unroll
        for (int r = 0; r < RW; ++r)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                if (lane + 64 * h < q.rowlen / 4) m[r] = fmaxf(m[r], fmaxf(fmaxf(fabsf(a[r][h].x), fabsf(a[r][h].y)), fmaxf(fabsf(a[r][h].z), fabsf(a[r][h].w))));
    } else {
#pragma unroll
        for (int r = 0; r < RW; ++r) {
            if (row0 + r >= rows) break;
            const float *x = q.x + (row0 + r) * (size_t)q.rowlen;
            if (q.vec) {
                const float4 *x4 = reinterpret_cast<const float4 *>(x);
                for (int i = lane; i < q.rowlen / 4; i += 64) {
                    const float4 t = x4[i];
                    m[r] = fmaxf(m[r], fmaxf(fmaxf(fabsf(t.x), fabsf(t.y)), fmaxf(fabsf(t.z), fabsf(t.w))));
                }
            } else {
                for (int i = lane; i < q.rowlen; i += 64) m[r] = fmaxf(m[r], fabsf(x[i]));
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RW; ++r) {
        const unsigned u = wave_max_lane63(__float_as_uint(m[r]));
        if (lane == 63 && row0 + r < rows) q.slots[row0 + r] = u;
    }
}
template <int NT>
__device__ __forceinline__ void absmax_rows_block(const PrepArgs::Pass &q, int piece)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const size_t rows = q.n / (size_t)q.rowlen;
    const size_t wid = (size_t)piece * (NT / 64) + wave, nw = (size_t)q.nblocks * (NT / 64);
    if (rows <= nw) {
        if (wid < rows) absmax_rows_batch<1>(q, wid, rows, lane);
    } else {
        for (size_t row0 = wid * 4; row0 < rows; row0 += nw * 4) absmax_rows_batch<4>(q, row0, rows, lane);
    }
}

// slots[piece] = largest magnitude of piece `piece` of x[n] (pieces of whole float4 units when vec)
template <int NT>
__device__ __forceinline__ void absmax_pass_block(const PrepArgs::Pass &q, int piece)
{
    if (q.rowlen > 0) { absmax_rows_block<NT>(q, piece); return; }
    const int tid = threadIdx.x;
    float m = 0.f;
    if (q.vec) {
        const size_t n4 = q.n / 4;
        const float4 *x4 = reinterpret_cast<const float4 *>(q.x);
        size_t i = (size_t)piece * NT + tid;
        const size_t stride = (size_t)q.nblocks * NT;
        for (; i + 7 * stride < n4; i += 8 * stride) {          // eight loads in flight
            float4 v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = x4[i + j * stride];
#pragma unroll
            for (int j = 0; j < 8; ++j)
                m = fmaxf(m, fmaxf(fmaxf(fabsf(v[j].x), fabsf(v[j].y)), fmaxf(fabsf(v[j].z), fabsf(v[j].w))));
        }
        for (; i + 3 * stride < n4; i += 4 * stride) {          // four loads in flight
            const float4 a = x4[i], b = x4[i + stride], c = x4[i + 2 * stride], d = x4[i + 3 * stride];
            m = fmaxf(m, fmaxf(fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))),
                               fmaxf(fmaxf(fabsf(b.x), fabsf(b.y)), fmaxf(fabsf(b.z), fabsf(b.w)))));
            m = fmaxf(m, fmaxf(fmaxf(fmaxf(fabsf(c.x), fabsf(c.y)), fmaxf(fabsf(c.z), fabsf(c.w))),
                               fmaxf(fmaxf(fabsf(d.x), fabsf(d.y)), fmaxf(fabsf(d.z), fabsf(d.w)))));
        }
        for (; i < n4; i += stride) {
            const float4 a = x4[i];
            m = fmaxf(m, fmaxf(fmaxf(fabsf(a.x), fabsf(a.y)), fmaxf(fabsf(a.z), fabsf(a.w))));
        }
    } else {
        for (size_t i = (size_t)piece * NT + tid; i < q.n; i += (size_t)q.nblocks * NT) m = fmaxf(m, fabsf(q.x[i]));
    }
    const unsigned u = block_absmax<NT>(m);
    if (tid == 0) q.slots[piece] = u;
}

__device__ void psi_prime(double zr, double zi, double er, double ei, double &pr, double &pi)
{
    // psi'(z) = (z e^z - e^z + 1)/z^2 = sum_k z^k (k+1)/(k+2)!
    if (zr * zr + zi * zi < 0.25) {
        double tr = 0.5, ti = 0.0;
        pr = 0.5; pi = 0.0;
        // (|z| < 1/2: the terms behind the seventeenth are below 1e-20 of the first; unrolled, so that their coefficients are constants)
#pragma unroll
        for (int k = 1; k < 18; ++k) {
            const double c = (double)(k + 1) / ((double)k * (double)(k + 2));
            const double nr = (tr * zr - ti * zi) * c, ni = (tr * zi + ti * zr) * c;
            tr = nr; ti = ni;
            pr += tr; pi += ti;
        }
    } else {
        // (e^z - psi(z))/z with psi = expm1(z)/z; er, ei = e^z
        const double sh = sin(0.5 * zi);
        const double mr = expm1(zr) * cos(zi) - 2.0 * sh * sh, mi = ei;
        double psr, psi_;
        cdiv(mr, mi, zr, zi, psr, psi_);
        cdiv(er - psr, ei - psi_, zr, zi, pr, pi);
    }
}

__device__ __forceinline__ void adjoint_block(const PackSrc &s, StateAdjoint *out, int blk)
{
    const int p = blk * (int)blockDim.x + (int)threadIdx.x;
    if (p >= s.P) return;
    const float2 L = s.Lambda[p];
    const Zoh z = zoh_discretize(L, s.log_delta[p]);
    double pr, pi;
    psi_prime(z.zr, z.zi, z.lr, z.li, pr, pi);
    const double d = z.delta, Lr = L.x, Li = L.y;
    StateAdjoint o;
    o.ar = d * z.lr; o.ai = d * z.li;                        // Delta Abar
    o.pr = d * d * pr; o.pi = d * d * pi;                    // Delta^2 psi'
    o.mr = d * (Lr * z.lr - Li * z.li); o.mi = d * (Lr * z.li + Li * z.lr);
    o.gr = (float)z.gr; o.gi = (float)z.gi;
    o.pad[0] = o.pad[1] = 0.f;
    out[p] = o;
}

constexpr int PREP_ZERO_UNITS = 2048;        // 16-byte units that a workgroup clears

// Everything that has to be done before the products of a pass, in one launch: the weights of its products in
// fragment order, the column-dot slabs behind dD (gradient pass), the largest magnitudes that scale the planes of
// the activations, and the words to be cleared.  The longest chains of dependent work come first in the grid.
template <int NT>
__global__ void __launch_bounds__(NT, 4) prep_kernel(PrepArgs a)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[pack_lds_bytes(NT)];
    const int blk = blockIdx.x, tid = threadIdx.x;
    const PackSrc src{a.Lambda, a.B, a.C, a.log_delta, a.W, a.P, a.H, a.lam_bar};
    static_assert(PREP_MAX_PACKS == 4, "one load for all");
    const int e0 = a.pack_end[0], e1 = a.pack_end[1], e2 = a.pack_end[2], e3 = a.pack_end[3];
    WsHeader *hdr = a.hdr;
    // (what decides the workgroup's job and what every job reads are requested together, and the job itself next: left to
    // where they are used, the arguments come in five or six trips one behind the other, 1 us of the 3 that a small launch takes)
    asm volatile("" ::"s"(src.Lambda), "s"(src.B), "s"(src.C), "s"(src.log_delta), "s"(src.W), "s"(src.P), "s"(src.H), "s"(src.lam_bar), "s"(e0),
                 "s"(e1), "s"(e2), "s"(e3), "s"(hdr));
    if (a.adj && blk < a.adj_blocks) {
        adjoint_block(src, a.adj, blk);
        return;
    }
    if (blk < e3) {
        const PackJob job = a.pack[(blk >= e0) + (blk >= e1) + (blk >= e2)];
        if (blk == a.adj_blocks && tid == 0 && hdr) { hdr->err = 0; hdr->magic = 0x53534d31u; }
        if (job.planes == 3) pack_dispatch<3, NT>(src, job, blk - job.block0, lds);
        else pack_dispatch<2, NT>(src, job, blk - job.block0, lds);
        return;
    }
    if (a.cd.partial && blk < a.cd_block0 + a.cd_colblocks * a.cd.nslab) {
        const int cb = blk - a.cd_block0;
        coldot_block<NT>(a.cd, cb % a.cd_colblocks, cb / a.cd_colblocks, a.cd_amax, a.cd_bmax, cb, a.cd_arow, reinterpret_cast<float *>(lds));
        return;
    }
    if (a.pass.nblocks > 0 && blk < a.pass.block0 + a.pass.nblocks) {
        absmax_pass_block<NT>(a.pass, blk - a.pass.block0);
        return;
    }
#pragma unroll
    for (int z = 0; z < 2; ++z) {
        if (a.zero[z].nblocks > 0 && blk < a.zero[z].block0 + a.zero[z].nblocks) {
            const size_t i0 = (size_t)(blk - a.zero[z].block0) * PREP_ZERO_UNITS + tid;
#pragma unroll
            for (int k = 0; k < PREP_ZERO_UNITS / NT; ++k) {
                const size_t i = i0 + (size_t)k * NT;
                if (i < a.zero[z].n16) a.zero[z].p[i] = make_uint4(0, 0, 0, 0);
            }
            return;
        }
    }
}

void pack_place(PackJob &j, int block0, int threads)
{
    const int per = pack_lanes(j.kind) * pack_per_lane(j.kind), npad = (j.N + 31) / 32 * 32;
    const int chunks = (j.K + 63) / 64 * 8, rows = threads / pack_lanes(j.kind);
    j.kparts = j.planes == 3 ? (chunks + rows - 1) / rows : 1;
    j.block0 = block0; j.nblocks = (npad + per - 1) / per * j.kparts;
}

hipError_t launch_prep(const PrepArgs &a_in, hipStream_t s)
{
    PrepArgs a = a_in;
    long blocks = 0;
    if (a.npack < 1 || a.npack > PREP_MAX_PACKS) return hipErrorInvalidValue;
    // The gradient pass with two planes: 512 threads, so that a packing workgroup has half as long a chain of chunks per thread
    // (its launch as a whole with 256 and with 512 threads: 8.3 and 7.2 us at 4096 tokens, H = P = 512; 15.1 and 13.9 at 4800, H = 1024,
    // P = 512).  The forward pass gains nothing by it (-3 .. +4 % of its time on twelve shapes): there a pass over the rows of u takes
    // the registers that packing leaves, and starts later with two workgroups per CU than with four.
    const int threads = a.cd.partial && a.pack[0].planes == 2 ? 512 : 256;
    a.adj_blocks = a.adj ? (a.P + threads - 1) / threads : 0;
    blocks = a.adj_blocks;
    for (int i = 0; i < a.npack; ++i) {
        PackJob &j = a.pack[i];
        if (!j.frag || (j.planes != 3 && (j.planes != 2 || !j.exp))) return hipErrorInvalidValue;
        pack_place(j, (int)blocks, threads);
        blocks += j.nblocks;
    }
    for (int i = 0; i < PREP_MAX_PACKS; ++i) a.pack_end[i] = i < a.npack ? a.pack[i].block0 + a.pack[i].nblocks : (int)blocks;
    a.cd_block0 = (int)blocks; a.cd_colblocks = 0;
    if (a.cd.partial) {
        a.cd_colblocks = (a.cd.H + 63) / 64;
        blocks += (long)a.cd_colblocks * a.cd.nslab;
    }
    PrepArgs::Pass &q = a.pass;
    if (q.nblocks > 0) {
        if (!q.x || !q.slots) return hipErrorInvalidValue;
        q.vec = (reinterpret_cast<uintptr_t>(q.x) & 15) == 0 && q.n % 4 == 0 && q.rowlen % 4 == 0;
        if (q.rowlen < 0 || (q.rowlen > 0 && q.n % (size_t)q.rowlen != 0)) return hipErrorInvalidValue;
        q.block0 = (int)blocks;
        blocks += q.nblocks;
    }
    for (PrepArgs::Zero &z : a.zero) {
        z.block0 = (int)blocks;
        z.nblocks = (z.p && z.n16 > 0) ? (int)((z.n16 + PREP_ZERO_UNITS - 1) / PREP_ZERO_UNITS) : 0;
        blocks += z.nblocks;
    }
    if (blocks <= 0 || blocks > 0x7fffffffL) return hipErrorInvalidValue;
    if (threads == 256) hipLaunchKernelGGL(prep_kernel<256>, dim3((unsigned)blocks), dim3(256), 0, s, a);
    else hipLaunchKernelGGL(prep_kernel<512>, dim3((unsigned)blocks), dim3(512), 0, s, a);
    return hipGetLastError();
}

// Workgroup p: Abar_p and, when asked, row p of Bbar as interleaved complex.
__global__ void __launch_bounds__(256) discretize_kernel(const float2 *__restrict__ Lambda, const float2 *__restrict__ B,
                                                         const float *__restrict__ log_delta, int H, float2 *__restrict__ lam_bar,
                                                         float2 *__restrict__ Bbar)
{
    const int p = blockIdx.x;
    const Zoh z = zoh_discretize(Lambda[p], log_delta[p]);
    const float gr = (float)z.gr, gi = (float)z.gi;
    if (threadIdx.x == 0) lam_bar[p] = make_float2((float)z.lr, (float)z.li);
    if (Bbar)
        for (int h = threadIdx.x; h < H; h += 256) {
            const float2 b = B[(long)p * H + h];
            Bbar[(long)p * H + h] = make_float2(gr * b.x - gi * b.y, gr * b.y + gi * b.x);
        }
}

hipError_t launch_discretize(const float2 *Lambda, const float2 *B, const float *log_delta, int P, int H, float2 *lam_bar, float2 *Bbar,
                             hipStream_t s)
{
    hipLaunchKernelGGL(discretize_kernel, dim3((unsigned)P), dim3(256), 0, s, Lambda, B, log_delta, H, lam_bar, Bbar);
    return hipGetLastError();
}

int coldot_slabs(int64_t T, int planes)
{
    // rows of one slab: a round of a workgroup's loads with 256 threads, two with 512 (the prep launch of 4800 tokens, H = 1024, P = 512
    // with 64, 128 and 256 rows: 16.7, 15.5 and 13.9 us; 4096 tokens, 512, 512: 8.4, 7.9 and 7.5)
    const int64_t rows = planes == 2 ? 256 : 64;
    int64_t n = (T + rows - 1) / rows;
    if (n > 64) n = 64;                     // (128 and 256 slabs at 16384 tokens: within 0.5 % either way)
    if (n < 1) n = 1;
    return (int)n;
}

// ---------------------------------------------------------------------------------------------
// Adjoint of the discretisation and final reduction of the split partial sums.
//   workgroups [0, P): state p.   dBbar[p,h] = sum of the K-split slabs (rows 2p, 2p+1);
//       dB[p,h] = conj(g_p) dBbar[p,h];  dg_p = sum_h conj(B[p,h]) dBbar[p,h];
//       dAbar_p = sum of the reverse scan's partial rows;
//       dLambda_p = conj(Delta Abar) dAbar + conj(Delta^2 psi'(z)) dg,   psi(z) = (e^z - 1)/z
//       dlog_delta_p = Delta * Re(conj(Lambda Abar) dAbar + conj(Abar) dg)
//   workgroups [P, P+H): row h of dC = sum of its slabs with the imaginary part negated
//       (dC[h,p] = sum_t dy[t,h] conj(x[t,p])), and dD[h] = sum of the column-dot slabs;
//   workgroups from P+H on: the slabs of another reduction, where there is one.
// The factors of dAbar and dg depend on the parameters alone: the prep launch of the pass computes them (adjoint_block),
// a thread per state beside everything else it does.  Here, in every workgroup of a state, their double-precision
// transcendentals were 2 to 3.4 us in front of sums of 1 to 3 us.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float4 add4(float4 a, float4 b) { return make_float4(a.x + b.x, a.y + b.y, a.z + b.z, a.w + b.w); }

// s[r] = sum over the slabs i, i + step, ... < n of the four values at base + i stride + r pitch, r < R: in the order of the
// slabs, D of them (D R loads) in flight at a time.  A slab past the end re-reads the last one and is not added.
template <int R, int D = 4>
__device__ __forceinline__ void sum_slabs(const float *base, long stride, long pitch, int i, int step, int n, int valid, float4 (&s)[R])
{
#pragma unroll
    for (int r = 0; r < R; ++r) s[r] = make_float4(0.f, 0.f, 0.f, 0.f);
    for (; i < n; i += D * step) {
        float4 v[D][R];
#pragma unroll
        for (int j = 0; j < D; ++j)
#pragma unroll
            for (int r = 0; r < R; ++r) v[j][r] = load4(base + (long)min(i + j * step, n - 1) * stride + r * pitch, valid);
#pragma unroll
        for (int j = 0; j < D; ++j)
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (i + j * step < n) s[r] = add4(s[r], v[j][r]);
    }
}

// Sums of v[0] .. v[3] over the 256 threads of a workgroup in a fixed order; valid in thread 0.  Inside a wavefront lanes that
// differ in bit 5, then bit 4, share out the four sums (seven exchanges of a double instead of twenty-four); red: 16 doubles.
__device__ __forceinline__ double shfl_xor_double(double v, int mask)
{
    int lo = __double2loint(v), hi = __double2hiint(v);
    lo = __shfl_xor(lo, mask); hi = __shfl_xor(hi, mask);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ void block_sum4(double *red, double (&v)[4], int tid)
{
    const int lane = tid & 63;
    const bool up5 = lane & 32, up4 = lane & 16;
    const double a = (up5 ? v[2] : v[0]) + shfl_xor_double(up5 ? v[0] : v[2], 32);
    const double b = (up5 ? v[3] : v[1]) + shfl_xor_double(up5 ? v[1] : v[3], 32);
    double s = (up4 ? b : a) + shfl_xor_double(up4 ? a : b, 16);
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) s += shfl_xor_double(s, o);
    if ((lane & 15) == 0) red[4 * (tid >> 6) + (lane >> 4)] = s;          // lane 0: v[0], 16: v[1], 32: v[2], 48: v[3]
    __syncthreads();
    if (tid == 0) {
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = (red[k] + red[4 + k]) + (red[8 + k] + red[12 + k]);
    }
}

// Bound by the trips to memory of one workgroup: up to P + H = 1280 (96 registers: five per CU) a layer's are all resident at once, and the slabs were written by the launch before.  A
// thread takes four columns of every row it sums in one request; threads that the columns leave over share out the slabs (groups
// of 2^lgB / 2^lgC threads, whose sums meet in LDS in the order of the groups).  First workgroup's start to last one's end, with a
// column per thread and request and the discretisation in front of the sums, and now: 4096 tokens, H = P = 512: 8.3 and 5.3 us;
// 4800 tokens, H = 1024, P = 512: 14.0 and 7.3; 32768 tokens, 512, 512: 11.2 and 7.3; 1024 tokens, 256, 256: 5.3 and 3.6.
// Behind them, started as those end, the gate's dW (a launch of its own: 5.6 us and a boundary, block of 32 x 128, 1024, 512), slab by slab in the
// order of its own call, so nobody shares out slabs: up to 64 of them are as many trips to memory as there are batches in flight, and narrow layers have few
// workgroups.  Eight at a time, and one value per thread up to 128 x 128, instead of four and four: blocks of 4096 tokens, H = P = 64: 57.0 -> 52.3 us, 128:
// 72.1 -> 69.7; 16384, 64: 96.4 -> 92.2, 128: 122.5 -> 117.0.  From H = 200 on four values (16384, 200, 100: 163.9, single ones 166.0); up to four slabs four at a
// time, since a batch reads the last slab again.
constexpr int64_t SINGLE_VALUES = 128 * 128;
__host__ __device__ __forceinline__ bool single_values(int64_t n) { return n <= SINGLE_VALUES; }
__global__ void __launch_bounds__(256) epilogue_kernel(EpilogueArgs a)
{
    __shared__ float4 part[2][256];
    __shared__ double red[16];
    const int tid = threadIdx.x, blk = blockIdx.x;
    const long PH2 = 2L * a.P * a.H;
    if (blk >= a.P + a.H) {
        const long at = (long)(blk - a.P - a.H) * 256 + tid;
        const bool single = single_values(a.also.n);
        const long i = single ? at : 4 * at;
        if (i >= a.also.n) return;
        const int n = single ? 1 : (int)min(a.also.n - i, 4L);
        const float *part = a.also.part + i;
        float4 v[1];
        if (single) sum_slabs<1, 8>(part, a.also.n, 0, 0, 1, a.also.slabs, 1, v);
        else if (a.also.slabs <= 4) sum_slabs<1>(part, a.also.n, 0, 0, 1, a.also.slabs, n, v);
        else sum_slabs<1, 8>(part, a.also.n, 0, 0, 1, a.also.slabs, n, v);
        store4(a.also.out + i, v[0], n);
        return;
    }
    if (blk < a.P) {
        const int p = blk;
        const float2 apart0 = tid < a.npart ? a.dAbar_part[(long)tid * a.P + p] : make_float2(0.f, 0.f);
        const StateAdjoint z = a.adj[p];
        const int units = (a.H + 3) / 4, lg = a.lgB, groups = 256 >> lg, group = tid >> lg, u0 = tid & ((1 << lg) - 1);
        const float *B = reinterpret_cast<const float *>(a.B + (long)p * a.H), *rows = a.dBbar_part + 2L * p * a.H;
        float *dB = reinterpret_cast<float *>(a.dB + (long)p * a.H);
        double sum[4] = {0.0, 0.0, (double)apart0.x, (double)apart0.y};      // dg, dAbar
        auto finish = [&](int u, const float4 (&b)[2], float4 r, float4 i) {
            const int n = 2 * (a.H - 4 * u);                 // floats of B and dB from column 4 u on
            // conj(g) dBbar
            store4(dB + 8 * u, make_float4(z.gr * r.x + z.gi * i.x, z.gr * i.x - z.gi * r.x, z.gr * r.y + z.gi * i.y, z.gr * i.y - z.gi * r.y), n);
            store4(dB + 8 * u + 4, make_float4(z.gr * r.z + z.gi * i.z, z.gr * i.z - z.gi * r.z, z.gr * r.w + z.gi * i.w, z.gr * i.w - z.gi * r.w), n - 4);
            // conj(B) dBbar (columns past the end: zeros)
            const float br[4] = {b[0].x, b[0].z, b[1].x, b[1].z}, bi[4] = {b[0].y, b[0].w, b[1].y, b[1].w};
            const float sr[4] = {r.x, r.y, r.z, r.w}, si[4] = {i.x, i.y, i.z, i.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                sum[0] += (double)br[k] * sr[k] + (double)bi[k] * si[k];
                sum[1] += (double)br[k] * si[k] - (double)bi[k] * sr[k];
            }
        };
        auto unit = [&](int u, float4 (&b)[2], float4 (&v)[2]) {
            const int n = a.H - 4 * u;
            b[0] = load4(B + 8 * u, 2 * n); b[1] = load4(B + 8 * u + 4, 2 * n - 4);
            sum_slabs<2>(rows + 4 * u, PH2, a.H, group, groups, a.nsplit_B, n, v);
        };
        float4 b[2], v[2];
        if (groups == 1) {
            for (int u = u0; u < units; u += 256) { unit(u, b, v); finish(u, b, v[0], v[1]); }
        } else {
            if (u0 < units) { unit(u0, b, v); part[0][tid] = v[0]; part[1][tid] = v[1]; }
            __syncthreads();
            if (group == 0 && u0 < units) {
                for (int g = 1; g < groups; ++g) { v[0] = add4(v[0], part[0][(g << lg) + u0]); v[1] = add4(v[1], part[1][(g << lg) + u0]); }
                finish(u0, b, v[0], v[1]);
            }
        }
        for (long i = tid + 256; i < a.npart; i += 256) {    // dAbar: further partial rows of the reverse scan
            const float2 t = a.dAbar_part[i * a.P + p];
            sum[2] += (double)t.x; sum[3] += (double)t.y;
        }
        block_sum4(red, sum, tid);
        if (tid == 0) {
            const double dgr = sum[0], dgi = sum[1], ar = sum[2], ai = sum[3];
            // conj(Delta Abar) dAbar + conj(Delta^2 psi') dg
            a.dLambda[p] = make_float2((float)((z.ar * ar + z.ai * ai) + (z.pr * dgr + z.pi * dgi)),
                                       (float)((z.ar * ai - z.ai * ar) + (z.pr * dgi - z.pi * dgr)));
            // Delta Re(conj(Lambda Abar) dAbar + conj(Abar) dg)
            a.dlog_delta[p] = (float)((z.mr * ar + z.mi * ai) + (z.ar * dgr + z.ai * dgi));
        }
    } else {
        const int h = blk - a.P;
        const int units = (2 * a.P + 3) / 4, lg = a.lgC, groups = 256 >> lg, group = tid >> lg, u0 = tid & ((1 << lg) - 1);
        const float *row = a.dC_part + (long)h * 2 * a.P;
        float *dC = reinterpret_cast<float *>(a.dC) + (long)h * 2 * a.P;
        double sum[4] = {tid < a.nslab ? (double)a.dD_part[(long)tid * a.H + h] : 0.0, 0.0, 0.0, 0.0};
        auto finish = [&](int u, float4 v) { store4(dC + 4 * u, make_float4(v.x, -v.y, v.z, -v.w), 2 * a.P - 4 * u); };
        float4 v[1];
        if (groups == 1) {
            for (int u = u0; u < units; u += 256) { sum_slabs<1>(row + 4 * u, PH2, 0, 0, 1, a.nsplit_C, 2 * a.P - 4 * u, v); finish(u, v[0]); }
        } else {
            if (u0 < units) { sum_slabs<1>(row + 4 * u0, PH2, 0, group, groups, a.nsplit_C, 2 * a.P - 4 * u0, v); part[0][tid] = v[0]; }
            __syncthreads();
            if (group == 0 && u0 < units) {
                for (int g = 1; g < groups; ++g) v[0] = add4(v[0], part[0][(g << lg) + u0]);
                finish(u0, v[0]);
            }
        }
        for (int sl = tid + 256; sl < a.nslab; sl += 256) sum[0] += (double)a.dD_part[(long)sl * a.H + h];
        block_sum4(red, sum, tid);
        if (tid == 0) a.dD[h] = (float)sum[0];
    }
}

// log2 of the threads that take a row of n columns, four each: 16 to 256
static int column_threads_log2(int n)
{
    int lg = 4;
    while (lg < 8 && (4 << lg) < n) ++lg;
    return lg;
}

hipError_t launch_epilogue(const EpilogueArgs &a_in, hipStream_t s)
{
    EpilogueArgs a = a_in;
    if (!a.adj) return hipErrorInvalidValue;
    a.lgB = column_threads_log2(a.H); a.lgC = column_threads_log2(2 * a.P);
    const int64_t further = !a.also.out ? 0 : single_values(a.also.n) ? (a.also.n + 255) / 256 : (a.also.n + 1023) / 1024;
    if (a.P + a.H + further > 0x7fffffffLL) return hipErrorInvalidValue;
    hipLaunchKernelGGL(epilogue_kernel, dim3((unsigned)(a.P + a.H + further)), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace ssm
