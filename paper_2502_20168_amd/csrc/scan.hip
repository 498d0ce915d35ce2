// Resettable scan over the sequence dimension, forward and reverse time (gfx950).
//
// What is computed: the inclusive scan of Eq. 4 over the elements (Abar, Bbar u_k, reset flag)
// of Eq. 9 under the operator of Eq. 10.  For a diagonal Abar the products are element-wise, so
// every (sequence, state) pair is an independent lane.  Partial results are combined with that operator:
//   1. a thread walks SCAN_E consecutive steps held in registers (loads are coalesced over the
//      state index: neighbouring threads own neighbouring states of the same step);
//   2. the chunks of a wavefront exchange their (product, state) aggregates between lanes, the wavefronts of a
//      workgroup through LDS;
//   3. a workgroup holds whole sequences, or (plan_scan) 1024, 512 or 256 steps of one: several workgroups along time
//      exchange aggregates through descriptors in global memory with a decoupled look-back: each publishes its own aggregate
//      before it waits for anything, then fetches the aggregates of the earlier workgroups of its group (one per thread, all in
//      flight at once) plus the inclusive state that closes the previous group.
// With a look-back, logical time-block ids come from an atomic ticket per chain, so a workgroup only ever waits
// for workgroups that started before it, and every wait is bounded by spin_limit.
//
// The reverse scan runs the same operator over reversed time with conj(Abar):
//   chi_t = gx_t + [not is_first_{t+1}] conj(Abar) chi_{t+1}
// and additionally reduces dAbar += [not is_first_t] conj(x_{t-1}) chi_t.
#include "ssm_internal.h"
#include "lookback.h"

#include <type_traits>

namespace ssm {

// Abar^(16 * cy) for cy a power of two, in double so that the power itself adds no error
__device__ __forceinline__ float2 pow_block(float2 lam, int cy)
{
    double r = lam.x, i = lam.y;
    for (int n = 1; n < SCAN_E * cy; n *= 2) {
        const double nr = r * r - i * i, ni = 2.0 * r * i;
        r = nr; i = ni;
    }
    return make_float2((float)r, (float)i);
}

// v[e], e < 16, per lane -> the maximum over the 16 lanes of a group (lanes 16g .. 16g+15) of
// v[group16_index(lane)]: halving exchanges between lanes that differ in bit 0, 1, 2, 3.
__device__ __forceinline__ unsigned group16_max(unsigned (&v)[16], int lane)
{
#pragma unroll
    for (int bit = 0; bit < 4; ++bit) {
        const int n = 8 >> bit;
        // (bitwise: a selection between array elements becomes one between their addresses, and the array goes to scratch)
        const unsigned up = 0u - ((unsigned)(lane >> bit) & 1u);
#pragma unroll
        for (int k = 0; k < n; ++k) {
            const unsigned x = (v[k] ^ v[k + n]) & up, keep = v[k] ^ x, send = v[k + n] ^ x;
            v[k] = max(keep, (unsigned)__shfl_xor((int)send, 1 << bit));
        }
    }
    return v[0];
}
__device__ __forceinline__ int group16_index(int lane) { return 8 * (lane & 1) + 4 * ((lane >> 1) & 1) + 2 * ((lane >> 2) & 1) + ((lane >> 3) & 1); }
__device__ __forceinline__ float2 shfl_up2(float2 v, int d) { return make_float2(__shfl_up(v.x, d), __shfl_up(v.y, d)); }

// MAXOUT: the kernel also records the largest magnitude of every token row of its output (atomic maxima
// into a.rowmax_out, zero on entry: the product that consumes the output stages every token under its own
// scale) and of the whole output (a.amax_out, ABSMAX_SLOTS slots, zero on entry).
// THROUGH: the states are stored through the L2 (store_through); see store_rule.h.
template <bool REV, bool MAXOUT, bool THROUGH>
__global__ void __launch_bounds__(MAXOUT ? 256 : SCAN_MAX_THREADS) scan_kernel(ScanArgs a)
{
    constexpr int E = SCAN_E;
    constexpr int THREADS = MAXOUT ? 256 : SCAN_MAX_THREADS;
    __shared__ float2 sA[THREADS];                   // (level 2: one per wavefront and lane; level 3: one per thread)
    __shared__ float2 sS[THREADS];
    __shared__ float2 sX[MAXOUT ? 256 : 16];
    __shared__ unsigned s_tb;

    const int tid = threadIdx.x;
    // A chain = the workgroups along time of one sequence and group of states.  (Scalar values all of them, by multiplications: as divisions by lanes they
    // were 0.2 us in front of the first loads.)  Time index slowest: all first-in-time workgroups start before any second-in-time one.
    const int nchains = a.nPX * a.Bt;
    int tb = (int)a.by_chains(blockIdx.x);
    const int chain = (int)blockIdx.x - tb * nchains, b = (int)a.by_nPX(chain), px = chain - b * a.nPX;
    const int lane = tid & (a.pxb - 1), chunk = tid >> a.lg_pxb;
    const int p = px * a.pxb + lane, pc = min(p, a.P - 1);       // pc, sc below: a valid state and step for every thread
    float2 lam = a.lam[pc];
    if (a.nTB > 1) {
        // One ticket counter per chain: the i-th workgroup of a chain to start takes time block i, so its predecessors along
        // time have started before it.
        if (tid == 0) s_tb = atomicAdd(a.ticket + (size_t)chain * SCAN_TICKET_STRIDE, 1u);
        __syncthreads();
        tb = __builtin_amdgcn_readfirstlane((int)s_tb);
    } else {
        // no cross-workgroup wait can happen: mark the workspace header as clean
        if (blockIdx.x == 0 && tid == 0) { a.err[0] = 0; a.err[1] = 0x53534d31u; }
    }
    const bool active = p < a.P;
    const int L = a.L;
    const int s0 = (tb * a.cy + chunk) * E;          // first logical step of this thread
    const int len = max(0, min(E, L - s0));
    const long rowbase = (long)b * L;
    // every thread of the wavefront (MAXOUT: of the workgroup) owns E steps of a valid state: no guards needed
    const bool full = MAXOUT ? ((tb + 1) * a.cy * E <= L) && ((px + 1) * a.pxb <= a.P) : __builtin_amdgcn_ballot_w64(len == E && active) == ~0ull;
    const int stride = REV ? -a.P : a.P;                         // elements between consecutive logical steps
    const int sc = min(s0, L - 1);
    const long first = (rowbase + (REV ? (L - 1 - sc) : sc)) * a.P + pc;      // element of logical step s0
    const bool ends = len > 0 && s0 + len == L;                  // the thread owns the last logical step
    // state that flows into the sequence (with a look-back, into its first workgroup: level 3)
    float2 Xin = make_float2(0.f, 0.f);
    if (!MAXOUT && a.nTB == 1 && !REV && a.x0 && active) Xin = a.x0[(long)b * a.P + p];

    if (REV) lam.y = -lam.y;

    // logical step s <-> time t: forward t = s, reverse t = L-1-s.
    // Steps past the end of the sequence re-read the last valid one.  They (and lanes past P) are computed on and never
    // stored: nothing follows them, so no state depends on them.  (Guards around every load and step made the launches with
    // a ragged end wait for one step after the other: 4800 x 512, L = 200: 20.7 us forward, 23.4 reverse.)
    float2 val[E];
    float2 xp[REV ? E : 1];
    {
        const float2 *src = a.in + first;
        if (full) {
#pragma unroll
            for (int e = 0; e < E; ++e) val[e] = src[e * stride];
        } else {
            const int lim = max(len - 1, 0) * stride;
#pragma unroll
            for (int e = 0; e < E; ++e) val[e] = src[REV ? max(e * stride, lim) : min(e * stride, lim)];
        }
        if constexpr (REV) {
            // state before each step: x[t-1]; only the very last logical step has t = 0
            const int row = L - 2 - sc;                          // t - 1 of step s0
            const float2 *xs = a.xsaved + (rowbase + max(row, 0)) * a.P + pc;
            const int xlim = max(min(len - 1, row), 0) * stride;
            float2 xfirst = make_float2(0.f, 0.f);
            if (a.x0 && ends && active) xfirst = a.x0[(long)b * a.P + p];
            if (full) {
#pragma unroll
                for (int e = 0; e < E - 1; ++e) xp[e] = xs[e * stride];
                xp[E - 1] = xs[max((E - 1) * stride, xlim)];
                xp[E - 1] = make_float2(ends ? xfirst.x : xp[E - 1].x, ends ? xfirst.y : xp[E - 1].y);
            } else {
#pragma unroll
                for (int e = 0; e < E; ++e) xp[e] = xs[max(e * stride, xlim)];
#pragma unroll
                for (int e = 0; e < E; ++e) {
                    const bool t0 = s0 + e == L - 1;
                    xp[e] = make_float2(t0 ? xfirst.x : xp[e].x, t0 ? xfirst.y : xp[e].y);
                }
            }
        }
    }

    // flags of the thread's steps as a bit mask (bit e = is_first at the time of logical step s0+e)
    unsigned fmask = 0;
    if (a.is_first && len > 0) {
        const int tlo = REV ? (L - s0 - len) : s0;             // lowest time index of the chunk
        const uint8_t *fp = a.is_first + rowbase + tlo;
        if (len == E) {
            typedef unsigned u32x4u __attribute__((ext_vector_type(4), aligned(1)));
            const u32x4u w = *reinterpret_cast<const u32x4u *>(fp);
            const unsigned ww[4] = {w.x, w.y, w.z, w.w};
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const unsigned f = ((ww[j >> 2] >> (8 * (j & 3))) & 0xffu) != 0;
                fmask |= f << (REV ? (E - 1 - j) : j);
            }
        } else {
            unsigned f[E];
#pragma unroll
            for (int e = 0; e < E; ++e) f[e] = fp[REV ? max(len - 1 - e, 0) : min(e, len - 1)];
#pragma unroll
            for (int e = 0; e < E; ++e) fmask |= (unsigned)(f[e] != 0 && e < len) << e;
        }
    }
    // rmask bit e: the incoming state of logical step s0+e is dropped.
    // forward: the step's own flag.  reverse: the flag that cuts chi_{t+1} -> chi_t is
    // is_first[t+1], i.e. the flag of the previous logical step.
    unsigned rmask = fmask;
    const unsigned mmask = fmask;                               // reverse only: is_first at the step itself
    if (REV) {
        rmask = fmask << 1;
        if (a.is_first && len > 0 && s0 > 0) rmask |= (unsigned)(a.is_first[rowbase + (L - s0)] != 0);
    }
    // wavefront-uniform: no flag anywhere in the steps of this wavefront -> plain recurrence
    const bool plain = (__builtin_amdgcn_ballot_w64((rmask | mmask) != 0) == 0);

    // ---- level 1, first pass: aggregate of the thread's steps for zero incoming state
    float2 A = make_float2(1.f, 0.f), S = make_float2(0.f, 0.f);
    static_assert(E == 16, "Abar^E below is four squarings");
    if (plain) {
#pragma unroll
        for (int e = 0; e < E; ++e) S = cfma(lam, S, val[e]);
    } else {
        // branch-free: a reset zeroes the multiplier of that step
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const bool r = (rmask >> e) & 1u;
            const float2 le = make_float2(r ? 0.f : lam.x, r ? 0.f : lam.y);
            S = cfma(le, S, val[e]);
        }
    }
    // (up to 64 chunks multiply their Abar^E: rounded once, or the states behind them lose what four rounded squarings lose, 64 times
    // over: 4 x 4096 x 256 with slow decay, error against 64 bits 5.9e-6 of the norm with blocks of 1024 steps, 2.2e-6 with 256)
    float2 l2;
    if constexpr (MAXOUT) {                                      // (at most 16 chunks)
        l2 = cmul(lam, lam);
        l2 = cmul(l2, l2); l2 = cmul(l2, l2); l2 = cmul(l2, l2);
    } else {
        l2 = pow_block(lam, 1);
    }
    A = (rmask & 0xffffu) ? make_float2(0.f, 0.f) : l2;

    // ---- level 2: exclusive combine over the earlier chunks of this workgroup: between the lanes of a wavefront that hold the
    // same state (in log2 steps), then over the earlier groups of chunks (wavefronts; chunks, where one fills a wavefront) in LDS
    const bool several = a.pxb < 64;                 // chunks of a state in one wavefront
    const int wl = tid & 63, group = several ? tid >> 6 : chunk, ngroup = several ? (a.cy * a.pxb + 63) >> 6 : a.cy;
    // (MAXOUT: chunk by chunk in LDS, the incoming state by way of sX, and the sum of dAbar over the chunks as well.  Its registers hold the
    // maxima too: with the exchanges the reverse one needs 134 of them where it needs 118, one wavefront of a SIMD fewer, and takes 34.0 us
    // where it takes 28.6: 30 x 300 x 512)
    float2 Aex = make_float2(1.f, 0.f), Sex = make_float2(0.f, 0.f);
    if constexpr (MAXOUT) {
        sA[tid] = A;
        sS[tid] = S;
        __syncthreads();
        for (int j = 0; j < chunk; ++j) {
            const float2 Aj = sA[j * a.pxb + lane], Sj = sS[j * a.pxb + lane];
            Sex = cfma(Aj, Sex, Sj);
            Aex = cmul(Aj, Aex);
        }
    } else {
        float2 Ai = A, Si = S;
        for (int d = a.pxb; d < 64; d *= 2) {
            const float2 Au = shfl_up2(Ai, d), Su = shfl_up2(Si, d);
            const float2 nS = cfma(Ai, Su, Si), nA = cmul(Ai, Au);
            Si = make_float2(wl >= d ? nS.x : Si.x, wl >= d ? nS.y : Si.y);
            Ai = make_float2(wl >= d ? nA.x : Ai.x, wl >= d ? nA.y : Ai.y);
        }
        if (several) {
            const float2 Au = shfl_up2(Ai, a.pxb), Su = shfl_up2(Si, a.pxb);
            Aex = make_float2(wl >= a.pxb ? Au.x : 1.f, wl >= a.pxb ? Au.y : 0.f);
            Sex = make_float2(wl >= a.pxb ? Su.x : 0.f, wl >= a.pxb ? Su.y : 0.f);
        }
        if (!several || wl >= 64 - a.pxb) { sA[group * a.pxb + lane] = Ai; sS[group * a.pxb + lane] = Si; }
        __syncthreads();
        float2 Ap = make_float2(1.f, 0.f), Sp = make_float2(0.f, 0.f);
        // (three aggregates are read at a time: one by one, every step of the chain waits for LDS)
        for (int g0 = 0; g0 < group; g0 += 3) {
            float2 Ac[3], Sc[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const int i = min(g0 + c, group - 1) * a.pxb + lane;
                Ac[c] = sA[i]; Sc[c] = sS[i];
                asm volatile("" : "+v"(Ac[c].x), "+v"(Ac[c].y), "+v"(Sc[c].x), "+v"(Sc[c].y));
            }
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const bool use = g0 + c < group;
                const float2 nS = cfma(Ac[c], Sp, Sc[c]), nA = cmul(Ac[c], Ap);
                Sp = make_float2(use ? nS.x : Sp.x, use ? nS.y : Sp.y);
                Ap = make_float2(use ? nA.x : Ap.x, use ? nA.y : Ap.y);
            }
        }
        Sex = cfma(Aex, Sp, Sex);
        Aex = cmul(Aex, Ap);
    }

    // ---- level 3: incoming state of the workgroup.
    // Workgroups along time form groups of G = cy.  The incoming state is always evaluated in
    // one canonical order, whatever the timing: start from the inclusive state of the last
    // workgroup of the previous group (x0 / zero for the first group) and fold the aggregates of
    // the earlier workgroups of the own group over it.  Results are therefore bitwise
    // reproducible.  Every workgroup publishes its aggregate before it waits for anything; the
    // last workgroup of a group also publishes its inclusive state.  Every predecessor covers
    // exactly cy*E steps, so its transition product is Abar^(cy*E) or zero (tag 2).
    const int G = a.cy;
    const int sg0 = (tb / G) * G;
    const bool lastchunk = (chunk == a.cy - 1);
    const size_t desc_stride = (size_t)nchains * a.pxb;          // descriptors per time block
    ScanDesc *mine = a.desc + (((size_t)tb * nchains + chain) * a.pxb + lane);
    float2 Ablk = make_float2(0.f, 0.f), Sblk = make_float2(0.f, 0.f);
    if (lastchunk) {
        Ablk = cmul(A, Aex);
        Sblk = cfma(A, Sex, S);
        if (a.nTB > 1 && tb + 1 < a.nTB) {
            const unsigned tag = (Ablk.x == 0.f && Ablk.y == 0.f) ? 2u : 1u;
            publish_word(&mine->agg[0], Sblk.x, tag);
            publish_word(&mine->agg[1], Sblk.y, tag);
        }
        if ((MAXOUT || a.nTB > 1) && sg0 == 0 && !REV && a.x0 && active) Xin = a.x0[(long)b * a.P + p];
    }
    if (tb > 0) {                                    // uniform over the workgroup
        __syncthreads();                             // level 2 has finished reading sA / sS
        // thread (lane, chunk) fetches the aggregate of workgroup sg0 + chunk of this lane
        float2 Aj = make_float2(1.f, 0.f), Sj = make_float2(0.f, 0.f);
        const int j = sg0 + chunk;
        if (j < tb) {
            const ScanDesc *pred = mine - (size_t)(tb - j) * desc_stride;
            const float2 power = pow_block(lam, a.cy);           // (before the wait, not behind it)
            unsigned tag = 0;
            if (!wait_pair(pred->agg, 1u, a.spin_limit, Sj, tag)) {
                // gave up: flag it, hand on NaN (the states that depend on the missing aggregate become
                // NaN, so the failure cannot pass as data) and finish anyway
                atomicOr(a.err, 1u);
                Sj = make_float2(__builtin_nanf(""), __builtin_nanf(""));
                Aj = make_float2(0.f, 0.f);
            } else {
                Aj = make_float2(tag == 2u ? 0.f : power.x, tag == 2u ? 0.f : power.y);
            }
        }
        sA[tid] = Aj;
        sS[tid] = Sj;
        if (lastchunk && sg0 > 0) {
            const ScanDesc *pred = mine - (size_t)(tb - sg0 + 1) * desc_stride;
            unsigned tag = 0;
            float2 incl;
            if (!wait_pair(pred->incl, 3u, a.spin_limit, incl, tag)) {
                atomicOr(a.err, 1u);
                Xin = make_float2(__builtin_nanf(""), __builtin_nanf(""));
            } else {
                Xin = incl;
            }
        }
        __syncthreads();
        if (lastchunk) {
            const int n = tb - sg0;
            // (five aggregates are read at a time: one by one, every step of the chain waits for LDS)
            for (int c0 = 0; c0 < n; c0 += 5) {
                float2 Ac[5], Sc[5];
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    const int i = min(c0 + c, n - 1) * a.pxb + lane;
                    Ac[c] = sA[i]; Sc[c] = sS[i];
                    asm volatile("" : "+v"(Ac[c].x), "+v"(Ac[c].y), "+v"(Sc[c].x), "+v"(Sc[c].y));
                }
#pragma unroll
                for (int c = 0; c < 5; ++c) {
                    const float2 nX = cfma(Ac[c], Xin, Sc[c]);
                    Xin = make_float2(c0 + c < n ? nX.x : Xin.x, c0 + c < n ? nX.y : Xin.y);
                }
            }
        }
    }
    if (lastchunk) {
        if (a.nTB > 1 && tb + 1 < a.nTB && (tb + 1) % G == 0) {
            const float2 incl = cfma(Ablk, Xin, Sblk);
            publish_word(&mine->incl[0], incl.x, 3u);
            publish_word(&mine->incl[1], incl.y, 3u);
        }
        if (MAXOUT || a.nTB > 1) sX[lane] = Xin;
    }
    if (MAXOUT || a.nTB > 1) {                                 // uniform
        __syncthreads();
        Xin = sX[lane];
    }

    // ---- level 1, second pass: the states themselves
    float2 xs = cfma(Aex, Xin, Sex);
    float2 acc = make_float2(0.f, 0.f);
    unsigned rm[MAXOUT ? E : 1];                     // MAXOUT: magnitude of the value stored at step e
    float2 xend = make_float2(0.f, 0.f);             // state of the last logical step
    float2 *dst = a.out + first;
    auto second_pass = [&](auto all_steps, auto no_resets) {
        constexpr bool FULL = decltype(all_steps)::value, PLAIN = decltype(no_resets)::value;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const bool r = !PLAIN && ((rmask >> e) & 1u), valid = FULL || (e < len && active);
            const float2 le = make_float2(r ? 0.f : lam.x, r ? 0.f : lam.y);
            xs = cfma(le, xs, val[e]);
            if (valid) {
                if constexpr (THROUGH) store_through(dst + e * stride, xs);
                else dst[e * stride] = xs;
            }
            if constexpr (MAXOUT) rm[e] = valid ? __float_as_uint(fmaxf(fabsf(xs.x), fabsf(xs.y))) : 0u;
            if constexpr (REV) {
                // conj(x_{t-1}) * chi_t
                const bool m = !valid || (!PLAIN && ((mmask >> e) & 1u));
                const float2 q = make_float2(m ? 0.f : xp[e].x, m ? 0.f : xp[e].y);
                acc.x = fmaf(q.x, xs.x, fmaf(q.y, xs.y, acc.x));
                acc.y = fmaf(q.x, xs.y, fmaf(-q.y, xs.x, acc.y));
            }
            if (!FULL || e == E - 1) { const bool end = s0 + e == L - 1; xend = make_float2(end ? xs.x : xend.x, end ? xs.y : xend.y); }
        }
    };
    // (uniform per wavefront)
    if (full && plain) second_pass(std::true_type{}, std::true_type{});
    else if (full) second_pass(std::true_type{}, std::false_type{});
    else second_pass(std::false_type{}, std::false_type{});
    if (ends && active) {
        if constexpr (REV) {
            if (a.dx0) a.dx0[(long)b * a.P + p] = ((mmask >> (len - 1)) & 1u) ? make_float2(0.f, 0.f) : cmul(lam, xend);
        } else {
            if (a.x_last) a.x_last[(long)b * a.P + p] = xend;
        }
    }

    if constexpr (MAXOUT) {
        // a group of 16 lanes holds 16 neighbouring states of the same 16 steps: one atomic per step and group
        unsigned all = 0;
#pragma unroll
        for (int e = 0; e < E; ++e) all = max(all, rm[e]);
        const unsigned m = group16_max(rm, tid);
        const int e = group16_index(tid);
        if (e < len) {
            const int t = REV ? (L - 1 - (s0 + e)) : (s0 + e);
            atomicMax(a.rowmax_out + rowbase + t, m);
        }
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) all = max(all, (unsigned)__shfl_xor((int)all, o));
        if ((tid & 63) == 0) atomicMax(a.amax_out + (blockIdx.x * 4 + (tid >> 6)) % ABSMAX_SLOTS, all);
    }
    if (REV) {
        // sum the chunks' contributions to dAbar; one partial row per (sequence, workgroup in time)
        const int parts = MAXOUT ? a.cy : ngroup;
        if constexpr (MAXOUT) {
            sA[tid] = acc;
        } else {
            for (int d = a.pxb; d < 64; d *= 2) {
                acc.x += __shfl_xor(acc.x, d);
                acc.y += __shfl_xor(acc.y, d);
            }
            __syncthreads();                         // level 2 has finished reading sA
            if (!several || wl < a.pxb) sA[group * a.pxb + lane] = acc;
        }
        __syncthreads();
        if (tid < a.pxb && active) {
            float2 sum = make_float2(0.f, 0.f);
            for (int j = 0; j < parts; ++j) {
                sum.x += sA[j * a.pxb + lane].x;
                sum.y += sA[j * a.pxb + lane].y;
            }
            a.partial[((size_t)b * a.nTB + tb) * a.P + p] = sum;
        }
    }
}

// Chunks and states of a workgroup.  16 states are one 128-byte line of a step.
//   up to 256 steps: about 256 threads, as many states as that leaves for whole sequences;
//   up to 512 steps: whole sequences of 16 states; up to 1024 as well where there are 64 such workgroups, and either one per CU at most, or up to three rounds of them
//   that leave no more than three tenths of the chip's threads idle (one of 1024 threads has a CU to itself, so nothing overlaps its loads and stores: what is saved is
//   the clearing launch).  Forward and reverse call with a look-back and with whole sequences: 10 x 520 x 400: 44.3 and 36.5;
//   12 x 1024 x 1024: 171 and 165; 8 x 700 x 640: 61.1 and 64.2; 100 x 600 x 200: 193 and 199; 28 x 1024 x 768: 322 and 330;
//   else a look-back, over blocks of 256 steps; of 1024 or 512 where that makes 192 to 384 of them, about one per CU (with more of
//   them, small workgroups that overlap are better: 5 x 3000 x 700: 47.8 us with 256 steps, 53.1 with 1024) and the last one
//   does not leave more than a tenth of all idle (16 x 2100 x 64: 13.4 and 14.9).
//   Scans that record magnitudes (records): 256 steps at most, since the maxima and the saved states together do not fit the registers of
//   1024 threads (gradient pass with larger workgroups: 8 x 700, H = 512, P = 640 166.9 -> 173.6 us).
// Bytes and trips to memory bound all of them.  With 256 steps to a workgroup at every length, and a look-back above (us, scan-level entry points,
// forward and reverse, now behind the arrow):  20 x 300 x 250: 17.8 -> 14.1, 22.7 -> 19.5    10 x 500 x 300: 16.5 -> 12.9, 21.2 -> 17.7
//   1 x 300 x 64: 9.2 -> 6.3, 12.2 -> 9.4    16 x 1000 x 512: 26.8 -> 25.9, 39.9 -> 40.1
//   4 x 4096 x 256: 17.0 -> 16.2, 26.1 -> 26.3    2 x 20000 x 64: 21.4 -> 17.6, 28.8 -> 24.4    1 x 60000 x 64: 39.0 -> 18.8, 49.4 -> 28.4
// (whole sequences of 4096 steps, four states to a workgroup of 1024 threads: 4 x 4096 x 256 16.5 and 28.0, 1 x 4096 x 64 14.7 and 20.8)
ScanPlan plan_scan(int64_t Bt, int64_t L, int64_t P, bool records)
{
    ScanPlan pl;
    const int64_t chunks = (L + SCAN_E - 1) / SCAN_E, chains = (P + 15) / 16 * Bt;
    pl.pxb = 16;
    if (records) {
        pl.cy = 1;
        while (pl.cy < 16 && pl.cy < chunks) pl.cy *= 2;
        pl.pxb = 256 / pl.cy;
    } else if (chunks <= 16) {
        pl.pxb = 256;
        while (pl.pxb > 16 && (pl.pxb * chunks > 256 || pl.pxb / 2 >= P)) pl.pxb /= 2;
        pl.cy = (int)chunks;
    } else if (chunks <= 32 || (chunks <= 64 && chains >= 64 && (chains <= 256 || (chains <= 768 && chains * chunks * 10 >= (chains + 255) / 256 * 256 * 64 * 7)))) {
        pl.cy = (int)chunks;
    } else {
        pl.cy = 16;
        for (int cy : {32, 64}) {
            const int64_t blocks = (chunks + cy - 1) / cy;
            if (blocks > 1 && chains * blocks >= 192 && chains * blocks <= 384 && blocks * cy * 10 <= chunks * 11) pl.cy = cy;
        }
    }
    pl.nPX = (int)((P + pl.pxb - 1) / pl.pxb);
    pl.nTB = (int)((chunks + pl.cy - 1) / pl.cy);
    pl.nblocks = (int64_t)pl.nPX * Bt * pl.nTB;
    // look-back scratch: ticket counters (one per chain, 64 bytes apart) followed by descriptors
    pl.ticket_bytes = pl.nTB > 1 ? (size_t)pl.nPX * Bt * SCAN_TICKET_STRIDE * sizeof(uint32_t) : 0;
    pl.desc_bytes = pl.nTB > 1 ? (size_t)pl.nblocks * pl.pxb * sizeof(ScanDesc) : 0;
    pl.partial_elems = (size_t)Bt * pl.nTB * P;
    return pl;
}

hipError_t launch_scan(const ScanArgs &a_in, bool reverse, hipStream_t s)
{
    ScanArgs a = a_in;
    const int64_t nblocks = (int64_t)a.nPX * a.Bt * a.nTB;
    if (nblocks <= 0 || nblocks > 0x7fffffffLL || a.pxb < 16 || a.pxb > 256 || (a.pxb & (a.pxb - 1)) || a.cy < 1) return hipErrorInvalidValue;
    // a look-back: a thread per (state, workgroup of a group), blocks of a power of two of chunks
    if (a.nTB > 1 ? a.pxb != 16 || (a.cy != 16 && a.cy != 32 && a.cy != 64) : (int64_t)a.cy * SCAN_E < a.L) return hipErrorInvalidValue;
    const int64_t threads = ((int64_t)a.pxb * a.cy + 63) / 64 * 64;
    a.by_chains = FastDiv::by((unsigned)((int64_t)a.nPX * a.Bt)); a.by_nPX = FastDiv::by((unsigned)a.nPX);
    a.lg_pxb = __builtin_ctz((unsigned)a.pxb);
    const bool maxout = a.rowmax_out != nullptr;
    if (threads > (maxout ? 256 : SCAN_MAX_THREADS) || (maxout && !a.amax_out)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)nblocks), block((unsigned)threads);
    const bool through = states_through(reinterpret_cast<uintptr_t>(a.out), (int64_t)a.Bt * a.L, a.P);
    const auto launch = [&](auto rev, auto max) {
        constexpr bool R = decltype(rev)::value, M = decltype(max)::value;
        if (through) hipLaunchKernelGGL((scan_kernel<R, M, true>), grid, block, 0, s, a);
        else hipLaunchKernelGGL((scan_kernel<R, M, false>), grid, block, 0, s, a);
    };
    if (reverse && maxout) launch(std::true_type{}, std::true_type{});
    else if (reverse) launch(std::true_type{}, std::false_type{});
    else if (maxout) launch(std::false_type{}, std::true_type{});
    else launch(std::false_type{}, std::false_type{});
    return hipGetLastError();
}

// zeroes the header and the 16-byte words of the ticket counters + descriptors that follow it
__global__ void __launch_bounds__(256) clear_kernel(WsHeader *hdr, uint4 *desc, size_t n16)
{
    const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
    if (i == 0) {
        hdr->err = 0; hdr->magic = 0x53534d31u;
    }
    for (size_t j = i; j < n16; j += (size_t)gridDim.x * 256) desc[j] = make_uint4(0, 0, 0, 0);
}

hipError_t launch_clear(WsHeader *hdr, void *scratch, size_t scratch_bytes, hipStream_t s)
{
    const size_t n16 = scratch_bytes / 16;
    uint4 *desc = static_cast<uint4 *>(scratch);
    size_t blocks = (n16 + 255) / 256;
    if (blocks < 1) blocks = 1;
    if (blocks > 1024) blocks = 1024;
    hipLaunchKernelGGL(clear_kernel, dim3((unsigned)blocks), dim3(256), 0, s, hdr, desc, n16);
    return hipGetLastError();
}

// out[p] = sum_i partial[i * P + p] in one fixed order: a workgroup owns 64 states, its four wavefronts
// take the rows i = w, w + 4, ... (eight loads in flight each), and the four sums are added in order.
__global__ void __launch_bounds__(256) reduce_partials_kernel(const float2 *__restrict__ partial, long n, long P,
                                                              float2 *__restrict__ out)
{
    __shared__ float2 part[4][64];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const long p = (long)blockIdx.x * 64 + l;
    float2 s = make_float2(0.f, 0.f);
    if (p < P) {
        long i = w;
        for (; i + 28 < n; i += 32) {
            float2 v[8];
#pragma unroll
            for (int k = 0; k < 8; ++k) v[k] = partial[(i + 4 * k) * P + p];
#pragma unroll
            for (int k = 0; k < 8; ++k) { s.x += v[k].x; s.y += v[k].y; }
        }
        for (; i < n; i += 4) { const float2 v = partial[i * P + p]; s.x += v.x; s.y += v.y; }
    }
    part[w][l] = s;
    __syncthreads();
    if (w == 0 && p < P) {
        float2 t = part[0][l];
#pragma unroll
        for (int k = 1; k < 4; ++k) { t.x += part[k][l].x; t.y += part[k][l].y; }
        out[p] = t;
    }
}

hipError_t launch_reduce_partials(const float2 *partial, int64_t n, int64_t P, float2 *out, hipStream_t s)
{
    hipLaunchKernelGGL(reduce_partials_kernel, dim3((unsigned)((P + 63) / 64)), dim3(256), 0, s,
                       partial, (long)n, (long)P, out);
    return hipGetLastError();
}

}  // namespace ssm
