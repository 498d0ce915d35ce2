// Weights of the products: zero-order-hold discretisation, split into planes and fragment order (gfx950).  Run by
// workgroups of the launch in front of the products (prep_kernel, and the element-wise passes of the gate).
#pragma once

#include "gemm_kernel.h"

namespace ssm {

struct Zoh {
    double delta;
    double lr, li;   // Abar = exp(Lambda Delta)
    double gr, gi;   // g = (Abar - 1)/Lambda = Delta * expm1(z)/z
    double zr, zi;   // z = Lambda Delta
};

__device__ __forceinline__ void cdiv(double ar, double ai, double br, double bi, double &qr, double &qi)
{
    const double den = br * br + bi * bi;
    qr = (ar * br + ai * bi) / den;
    qi = (ai * br - ar * bi) / den;
}

__device__ __forceinline__ Zoh zoh_discretize(float2 Lambda, float log_delta)
{
    Zoh o;
    o.delta = exp((double)log_delta);
    o.zr = (double)Lambda.x * o.delta;
    o.zi = (double)Lambda.y * o.delta;
    // e^z and e^z - 1 from expm1(a), sin(b/2) and cos(b/2), z = a + i b: three function evaluations (six, with exp, sin
    // and cos of their own, took longer than the loads of a packing job), and no cancellation in
    // e^z - 1 = expm1(a) cos b - 2 sin^2(b/2) + i e^a sin b
    double sh, ch;
    sincos(0.5 * o.zi, &sh, &ch);
    const double em = expm1(o.zr), ea = em + 1.0, cb = 1.0 - 2.0 * sh * sh, sb = 2.0 * sh * ch;
    o.lr = ea * cb;
    o.li = ea * sb;
    const double er = em * cb - 2.0 * sh * sh, ei = ea * sb;
    if (o.zr == 0.0 && o.zi == 0.0) {
        o.gr = o.delta; o.gi = 0.0;
    } else {
        double qr, qi;
        cdiv(er, ei, o.zr, o.zi, qr, qi);
        o.gr = o.delta * qr; o.gi = o.delta * qi;
    }
    return o;
}

// (Abar, g) rounded, for the packing jobs.  Not inlined: inside their loops its many constants and temporaries took
// the registers of the values in flight, and the transposing job of Bbar spilled (13 us instead of 7).
__device__ __attribute__((noinline)) float4 zoh_rounded(float2 Lambda, float log_delta)
{
    const Zoh z = zoh_discretize(Lambda, log_delta);
    return make_float4((float)z.lr, (float)z.li, (float)z.gr, (float)z.gi);
}

// What the jobs read.
struct PackSrc { const float2 *Lambda, *B, *C; const float *log_delta, *W; int P, H; float2 *lam_bar; };

constexpr int PACK_ZOH_BATCH = 1024;                 // states whose g a transposing job of Bbar keeps in LDS at a time
constexpr size_t PACK_LDS_BYTES = PACK_ZOH_BATCH * 8 + 4 * 16 * 4;

// lanes that share a row of chunks, values of n per lane, chunks per thread that stay in registers
constexpr int pack_lanes(int kind) { return kind == PACK_IN ? 4 : (kind == PACK_WN ? 16 : 8); }
constexpr int pack_per_lane(int kind) { return (kind == PACK_IN || kind == PACK_GX) ? 2 : 1; }
constexpr int pack_kept(int kind) { return pack_per_lane(kind) == 2 ? 2 : 4; }

// A workgroup of 256 threads packs pack_lanes * pack_per_lane consecutive n over the whole (padded) K.  A thread owns
// one n (or the pair re, im of one state) and every (256 / lanes)-th chunk of eight consecutive k: the 16 bytes per
// plane that one lane of a fragment holds, so stores are whole 128-byte lines.  The job is bound by latency: all loads
// of a thread are in flight together and stay in registers between the largest magnitude of every n (its scale, two
// planes) and the split, so that it is one trip to memory (measured at H = P = 512, two trips of dependent chunks
// instead: prep launches of 11.1 and 17.6 us).  A K longer than that is read twice, round by round.
template <int KIND>
__device__ __forceinline__ void pack_block(const PackSrc &s, const PackJob &j, int blk, unsigned char *lds)
{
    constexpr int G = pack_lanes(KIND), V = pack_per_lane(KIND), ROWS = 256 / G, KEPT = pack_kept(KIND), RAW = 8 * V;
    float2 *gz = reinterpret_cast<float2 *>(lds);                                    // [PACK_ZOH_BATCH] g of the states (PACK_DU)
    unsigned *red = reinterpret_cast<unsigned *>(lds + PACK_ZOH_BATCH * 8);          // [4][G * V]
    const int tid = threadIdx.x, nl = tid % G, row = tid / G, lane = tid & 63, wave = tid >> 6;
    const int unit = blk * G + nl;                                                   // state, or n
    const int n0 = unit * V;
    const int nch = (j.K + 63) / 64 * 8;                                             // chunks, padded to whole K tiles
    const int npad = (j.N + 31) / 32 * 32, planes = j.planes;
    const int usrc = min(unit, j.N / V - 1);                                         // (clamped: the values past N are zeroed)
    const bool whole = j.K % 8 == 0;                                                 // no chunk is cut by the end of K

    // raw values of chunk c (clamped into K; what lies outside is zeroed by finish())
    auto fetch = [&](int c, float (&r)[RAW]) {
        const int k = 8 * c;
        if constexpr (KIND == PACK_IN || KIND == PACK_OUT || KIND == PACK_WT) {
            // contiguous in memory: RAW floats from column k (PACK_IN: complex columns)
            const float *src = KIND == PACK_IN ? reinterpret_cast<const float *>(s.B + (long)usrc * s.H)
                                               : (KIND == PACK_OUT ? reinterpret_cast<const float *>(s.C + (long)usrc * s.P) : s.W + (long)usrc * s.H);
            const int last = j.K * V;
            if (whole) {
                const float *q = src + min(k * V, last - RAW);
#pragma unroll
                for (int e = 0; e < RAW; e += 4) {
                    const f32x4u v = *reinterpret_cast<const f32x4u *>(q + e);
                    r[e] = v.x; r[e + 1] = v.y; r[e + 2] = v.z; r[e + 3] = v.w;
                }
            } else {
#pragma unroll
                for (int e = 0; e < RAW; ++e) r[e] = src[min(k * V + e, last - 1)];
            }
        } else if constexpr (KIND == PACK_GX) {
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float2 b = s.C[(long)min(k + e, s.H - 1) * s.P + usrc];
                r[2 * e] = b.x; r[2 * e + 1] = b.y;
            }
        } else if constexpr (KIND == PACK_DU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float2 b = s.B[(long)min(k / 2 + e, s.P - 1) * s.H + usrc];
                r[2 * e] = b.x; r[2 * e + 1] = b.y;
            }
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) r[e] = s.W[(long)min(k + e, s.H - 1) * s.H + usrc];
        }
    };
    float2 g = make_float2(0.f, 0.f);
    int batch = -1;
    // the discretisation behind the values: the thread's own state (PACK_IN), or a batch of states for the whole
    // workgroup (PACK_DU; all threads meet here, the batch index is uniform)
    auto discretize = [&](int b) {
        if constexpr (KIND == PACK_IN) {
            if (batch >= 0) return;
            batch = 0;
            const float4 z = zoh_rounded(s.Lambda[usrc], s.log_delta[usrc]);
            g = make_float2(z.z, z.w);
            if (row == 0 && s.lam_bar && unit < s.P) s.lam_bar[unit] = make_float2(z.x, z.y);
        } else if constexpr (KIND == PACK_DU) {
            if (b == batch) return;
            batch = b;
            __syncthreads();
            const int nb = min(PACK_ZOH_BATCH, s.P - b * PACK_ZOH_BATCH);
            for (int i = tid; i < nb; i += 256) {
                const int p = b * PACK_ZOH_BATCH + i;
                const float4 z = zoh_rounded(s.Lambda[p], s.log_delta[p]);
                gz[i] = make_float2(z.z, z.w);
                if (blk == 0 && s.lam_bar) s.lam_bar[p] = make_float2(z.x, z.y);
            }
            __syncthreads();
        }
    };
    // the eight values of chunk c for each of the thread's n
    auto finish = [&](int c, const float (&r)[RAW], float (&v)[V][8]) {
        float2 q[4];
        if constexpr (KIND == PACK_DU) {
            // (read ahead of the selections below: the compiler would move each read into its branch, and wait 32 times)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                q[e] = gz[(4 * c) % PACK_ZOH_BATCH + e];
                asm volatile("" : "+v"(q[e].x), "+v"(q[e].y));
            }
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            if constexpr (KIND == PACK_IN) {
                v[0][e] = g.x * r[2 * e] - g.y * r[2 * e + 1]; v[V - 1][e] = g.x * r[2 * e + 1] + g.y * r[2 * e];
            } else if constexpr (KIND == PACK_GX) {
                v[0][e] = r[2 * e]; v[V - 1][e] = -r[2 * e + 1];
            } else if constexpr (KIND == PACK_OUT) {
                v[0][e] = (e & 1) ? -r[e] : r[e];
            } else if constexpr (KIND == PACK_DU) {
                v[0][e] = (e & 1) ? q[e / 2].x * r[e] + q[e / 2].y * r[e - 1] : q[e / 2].x * r[e] - q[e / 2].y * r[e + 1];
            } else {
                v[0][e] = r[e];
            }
#pragma unroll
            for (int i = 0; i < V; ++i) v[i][e] = (8 * c + e < j.K && n0 + i < j.N) ? v[i][e] : 0.f;
        }
    };
    float scale[V], m[V];
#pragma unroll
    for (int i = 0; i < V; ++i) { scale[i] = 1.f; m[i] = 0.f; }
    auto take_max = [&](const float (&v)[V][8]) {
#pragma unroll
        for (int i = 0; i < V; ++i)
#pragma unroll
            for (int e = 0; e < 8; ++e) m[i] = fmaxf(m[i], fabsf(v[i][e]));
    };
    auto reduce_max = [&]() {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            unsigned u = __float_as_uint(m[i]);
#pragma unroll
            for (int o = 32; o >= G; o >>= 1) u = max(u, (unsigned)__shfl_xor((int)u, o));
            if (lane < G) red[wave * (G * V) + lane * V + i] = u;
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < V; ++i) {
            unsigned u = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) u = max(u, red[w * (G * V) + nl * V + i]);
            const int e = log2_scale_of(u);
            scale[i] = pow2f(e);
            if (row == 0 && n0 + i < npad) j.exp[n0 + i] = e;
        }
    };
    const int nks = nch / 2;
    auto put = [&](int c, const float (&v)[V][8]) {
        if (n0 >= npad) return;
#pragma unroll
        for (int i = 0; i < V; ++i) {
            const int n = n0 + i;
            const float4 lo = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]), hi = make_float4(v[i][4], v[i][5], v[i][6], v[i][7]);
            uint4 *dst = static_cast<uint4 *>(j.frag) + ((size_t)(n / 32) * nks + c / 2) * (planes * 64) + n % 32 + 32 * (c & 1);
            const Split4 a = planes == 3 ? split3(lo) : split2_f16(lo, scale[i]), b = planes == 3 ? split3(hi) : split2_f16(hi, scale[i]);
#pragma unroll
            for (int q = 0; q < 3; ++q) {
                if (q < planes) {
                    const uint2 x = __builtin_bit_cast(uint2, a.p[q]), y = __builtin_bit_cast(uint2, b.p[q]);
                    dst[q * 64] = make_uint4(x.x, x.y, y.x, y.y);
                }
            }
        }
    };

    // rounds of KEPT chunks per thread; with a single round the values stay in registers between the two passes
    constexpr int ROUND = KEPT * ROWS;
    static_assert(PACK_ZOH_BATCH % (4 * ROUND) == 0, "a round's states lie in one batch");
    const bool single = nch <= ROUND;
    float raw[KEPT][RAW];
    auto fetch_round = [&](int c0) {
#pragma unroll
        for (int t = 0; t < KEPT; ++t) fetch(min(c0 + t * ROWS + row, nch - 1), raw[t]);
    };
    if (planes == 2) {
        for (int c0 = 0; c0 < nch; c0 += ROUND) {
            fetch_round(c0);
            discretize(c0 * 4 / PACK_ZOH_BATCH);
#pragma unroll
            for (int t = 0; t < KEPT; ++t) {
                float v[V][8];
                finish(min(c0 + t * ROWS + row, nch - 1), raw[t], v);
                take_max(v);
            }
        }
        reduce_max();
    }
    for (int c0 = 0; c0 < nch; c0 += ROUND) {
        if (planes != 2 || !single) fetch_round(c0);
        discretize(c0 * 4 / PACK_ZOH_BATCH);
#pragma unroll
        for (int t = 0; t < KEPT; ++t) {
            const int c = c0 + t * ROWS + row;
            if (c < nch) {
                float v[V][8];
                finish(c, raw[t], v);
                put(c, v);
            }
        }
    }
}

__device__ __forceinline__ void pack_dispatch(const PackSrc &s, const PackJob &j, int blk, unsigned char *lds)
{
    switch (j.kind) {
    case PACK_IN: pack_block<PACK_IN>(s, j, blk, lds); break;
    case PACK_OUT: pack_block<PACK_OUT>(s, j, blk, lds); break;
    case PACK_GX: pack_block<PACK_GX>(s, j, blk, lds); break;
    case PACK_DU: pack_block<PACK_DU>(s, j, blk, lds); break;
    case PACK_WN: pack_block<PACK_WN>(s, j, blk, lds); break;
    default: pack_block<PACK_WT>(s, j, blk, lds); break;
    }
}

}  // namespace ssm
