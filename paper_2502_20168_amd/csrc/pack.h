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

// (Abar, g) rounded, for the packing jobs.  Two planes: not inlined, because inside their loops its many constants and temporaries
// took the registers of the values in flight, and the transposing job of Bbar spilled (13 us instead of 7).  Three planes: inlined, so
// that the values are on their way meanwhile (a call waits for all loads first).
template <int PLANES>
__device__ __forceinline__ float4 zoh_rounded(float2 Lambda, float log_delta)
{
    const Zoh z = zoh_discretize(Lambda, log_delta);
    return make_float4((float)z.lr, (float)z.li, (float)z.gr, (float)z.gi);
}
__device__ __attribute__((noinline)) float4 zoh_rounded_call(float2 Lambda, float log_delta) { return zoh_rounded<3>(Lambda, log_delta); }
template <>
__device__ __forceinline__ float4 zoh_rounded<2>(float2 Lambda, float log_delta) { return zoh_rounded_call(Lambda, log_delta); }

struct ZohPair { float4 a, b; };
__device__ __attribute__((noinline)) ZohPair zoh_rounded_pair(float2 La, float da, float2 Lb, float db)
{
    return ZohPair{zoh_rounded<3>(La, da), zoh_rounded<3>(Lb, db)};
}

// What the jobs read.
struct PackSrc { const float2 *Lambda, *B, *C; const float *log_delta, *W; int P, H; float2 *lam_bar; };

constexpr int PACK_ZOH_BATCH = 1024;                 // states whose g a transposing job of Bbar keeps in LDS at a time
constexpr size_t pack_lds_bytes(int threads) { return PACK_ZOH_BATCH * 8 + threads / 64 * 16 * 4; }
constexpr size_t PACK_LDS_BYTES = pack_lds_bytes(256);

// lanes that share a row of chunks, values of n per lane, chunks per thread that stay in registers
constexpr int pack_lanes(int kind) { return kind == PACK_IN ? 4 : (kind == PACK_WN ? 16 : 8); }
constexpr int pack_per_lane(int kind) { return (kind == PACK_IN || kind == PACK_GX) ? 2 : 1; }
constexpr int pack_kept(int kind, int planes) { return planes == 3 ? 1 : pack_per_lane(kind) == 2 ? 2 : 4; }

// A workgroup packs pack_lanes * pack_per_lane consecutive n.  A thread owns one n (or the pair re, im of
// one state) and chunks of eight consecutive k: the 16 bytes per plane that one lane of a fragment holds, so stores are
// whole 128-byte lines.  Up to H = P = 512 the jobs are bound by latency: an empty launch takes 2 us, the discretisation 1.2 us
// and a thread's way through one chunk 0.5 us.
//   Three planes: nothing has to be known about the rest of a row, so a thread has one chunk, and K is shared out over
//     workgroups.  Prep launch of the gradient pass (before, with four chunks per thread, one workgroup per n and all of K; us):
//     1024 x (H 128, P 64) 4.9 -> 4.0, 256 tokens x (256, 512) 9.6 -> 6.6, 512 x (512, 512) 10.0 -> 7.0, 256 x (1024, 1024) 14.2 -> 11.9
//     (41 MB of weights and fragments there).
//   Two planes: every (256 / lanes)-th chunk of the whole K.  All loads of a thread are in flight together and stay in
//     registers between the largest magnitude of every n (its scale) and the split, so that it is one trip to memory
//     (measured at H = P = 512, two trips of dependent chunks instead: prep launches of 11.1 and 17.6 us).
//     A K longer than that is read twice, round by round.
template <int KIND, int PLANES, int NT = 256>
__device__ __forceinline__ void pack_block(const PackSrc &s, const PackJob &j, int wg, unsigned char *lds)
{
    constexpr int G = pack_lanes(KIND), V = pack_per_lane(KIND), ROWS = NT / G, KEPT = pack_kept(KIND, PLANES), RAW = 8 * V;
    constexpr bool SHARED_K = PLANES == 3;
    const int blk = SHARED_K ? wg / j.kparts : wg;
    const int first = SHARED_K ? (wg - blk * j.kparts) * ROWS : 0;                   // the workgroup's first chunk
    float2 *gz = reinterpret_cast<float2 *>(lds);                                    // [PACK_ZOH_BATCH] g of the states (PACK_DU)
    unsigned *red = reinterpret_cast<unsigned *>(lds + PACK_ZOH_BATCH * 8);          // [wavefronts][G * V]
    const int tid = threadIdx.x, nl = tid % G, row = tid / G, lane = tid & 63, wave = tid >> 6;
    const int unit = blk * G + nl;                                                   // state, or n
    const int n0 = unit * V;
    const int nch = (j.K + 63) / 64 * 8;                                             // chunks, padded to whole K tiles
    const int npad = (j.N + 31) / 32 * 32;
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
    // (three planes: the state whose discretisation this thread computes, requested ahead of the values; PACK_DU: of its workgroup's chunks)
    float2 own_lambda;
    float own_delta;
    if constexpr (SHARED_K && (KIND == PACK_IN || KIND == PACK_DU)) {
        const int p = KIND == PACK_IN ? usrc : min(first * 4 + tid, s.P - 1);
        own_lambda = s.Lambda[p]; own_delta = s.log_delta[p];
    }
    // the discretisation behind the values: the thread's own state (PACK_IN), or a batch of states for the whole
    // workgroup (PACK_DU; all threads meet here, the batch index is uniform)
    auto discretize = [&](int b) {
        if constexpr (KIND == PACK_IN) {
            if (batch >= 0) return;
            batch = 0;
            const float4 z = SHARED_K ? zoh_rounded<PLANES>(own_lambda, own_delta) : zoh_rounded<PLANES>(s.Lambda[usrc], s.log_delta[usrc]);
            g = make_float2(z.z, z.w);
            if (row == 0 && first == 0 && s.lam_bar && unit < s.P) s.lam_bar[unit] = make_float2(z.x, z.y);
        } else if constexpr (KIND == PACK_DU && SHARED_K) {
            static_assert(!SHARED_K || ROWS * 4 <= NT, "a state per thread");
            const int p = first * 4 + tid;
            if (tid < ROWS * 4) {
                const float4 z = zoh_rounded<PLANES>(own_lambda, own_delta);
                gz[tid] = make_float2(z.z, z.w);
                if (blk == 0 && s.lam_bar && p < s.P) s.lam_bar[p] = make_float2(z.x, z.y);
            }
            __syncthreads();
        } else if constexpr (KIND == PACK_DU) {
            if (b == batch) return;
            batch = b;
            __syncthreads();
            const int nb = min(PACK_ZOH_BATCH, s.P - b * PACK_ZOH_BATCH);
            auto keep = [&](int i, float4 z) {
                gz[i] = make_float2(z.z, z.w);
                if (blk == 0 && s.lam_bar) s.lam_bar[b * PACK_ZOH_BATCH + i] = make_float2(z.x, z.y);
            };
            const float2 *Lam = s.Lambda + b * PACK_ZOH_BATCH;
            const float *ld = s.log_delta + b * PACK_ZOH_BATCH;
            if (nb <= NT) {
                if (tid < nb) keep(tid, zoh_rounded<PLANES>(Lam[tid], ld[tid]));
            } else {
                for (int i = tid; i < nb; i += 2 * NT) {        // (two chains of double-precision arithmetic at a time)
                    const int k = min(i + NT, nb - 1);
                    const ZohPair z = zoh_rounded_pair(Lam[i], ld[i], Lam[k], ld[k]);
                    keep(i, z.a);
                    if (i + NT < nb) keep(i + NT, z.b);
                }
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
                q[e] = gz[SHARED_K ? 4 * (c - first) + e : (4 * c) % PACK_ZOH_BATCH + e];
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
            for (int w = 0; w < NT / 64; ++w) u = max(u, red[w * (G * V) + nl * V + i]);
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
            uint4 *dst = static_cast<uint4 *>(j.frag) + ((size_t)(n / 32) * nks + c / 2) * (PLANES * 64) + n % 32 + 32 * (c & 1);
            const Split4 a = split_planes<PLANES>(lo, scale[i]), b = split_planes<PLANES>(hi, scale[i]);
#pragma unroll
            for (int q = 0; q < PLANES; ++q) {
                const uint2 x = __builtin_bit_cast(uint2, a.p[q]), y = __builtin_bit_cast(uint2, b.p[q]);
                dst[q * 64] = make_uint4(x.x, x.y, y.x, y.y);
            }
        }
    };

    float raw[KEPT][RAW];
    auto fetch_round = [&](int c0) {
#pragma unroll
        for (int t = 0; t < KEPT; ++t)
            if (t == 0 || c0 + t * ROWS < nch) fetch(min(c0 + t * ROWS + row, nch - 1), raw[t]);
    };
    auto put_round = [&](int c0) {
#pragma unroll
        for (int t = 0; t < KEPT; ++t) {
            const int c = c0 + t * ROWS + row;
            if (c < nch) {
                float v[V][8];
                finish(c, raw[t], v);
                put(c, v);
            }
        }
    };
    if constexpr (SHARED_K) {
        fetch_round(first);
        discretize(0);
        put_round(first);
    } else {
        // rounds of KEPT chunks per thread; with a single round the values stay in registers between the two passes
        constexpr int ROUND = KEPT * ROWS;
        static_assert(PACK_ZOH_BATCH % (4 * ROUND) == 0, "a round's states lie in one batch");
        const bool single = nch <= ROUND;
        for (int c0 = 0; c0 < nch; c0 += ROUND) {
            fetch_round(c0);
            discretize(c0 * 4 / PACK_ZOH_BATCH);
#pragma unroll
            for (int t = 0; t < KEPT; ++t) {
                if (t > 0 && c0 + t * ROWS >= nch) continue;
                float v[V][8];
                finish(min(c0 + t * ROWS + row, nch - 1), raw[t], v);
                take_max(v);
            }
        }
        reduce_max();
        for (int c0 = 0; c0 < nch; c0 += ROUND) {
            if (!single) fetch_round(c0);
            discretize(c0 * 4 / PACK_ZOH_BATCH);
            put_round(c0);
        }
    }
}

template <int PLANES, int NT>
__device__ __forceinline__ void pack_dispatch(const PackSrc &s, const PackJob &j, int wg, unsigned char *lds)
{
    switch (j.kind) {
    case PACK_IN: pack_block<PACK_IN, PLANES, NT>(s, j, wg, lds); break;
    case PACK_OUT: pack_block<PACK_OUT, PLANES, NT>(s, j, wg, lds); break;
    case PACK_GX: pack_block<PACK_GX, PLANES, NT>(s, j, wg, lds); break;
    case PACK_DU: pack_block<PACK_DU, PLANES, NT>(s, j, wg, lds); break;
    case PACK_WN: pack_block<PACK_WN, PLANES, NT>(s, j, wg, lds); break;
    default: pack_block<PACK_WT, PLANES, NT>(s, j, wg, lds); break;
    }
}

}  // namespace ssm
