// Products of fp32 activations with packed weights (gfx950):
//
//   C[m,n] = f( sum_k A[m,k] W(n,k) ),   A [M, K] fp32 with k contiguous, rows = tokens
//
// on the 16-bit matrix cores with both operands split into planes: two fp16 planes of the operand scaled by a
// power of two (NPL = 2: every token row and every weight row n has its own scale) or three bf16 planes
// (NPL = 3, exact); see split2_f16 / split3 in gemm_kernel.h.
//
// The weights are split once per call, by the prep launch, into fragment order: the 16 bytes that lane l needs for a
// 32 x 16 block of W are at frag[((n / 32) (Kp / 16) + k / 16) NPL + plane][l].  A consumer wavefront therefore loads its
// fragments from the L2 straight into registers, one fully coalesced 1 KiB load each, PFB k steps ahead, and only the
// activations pass through producers and LDS.  What bounded the kernel that staged both operands through LDS was
// the LDS itself: per 128x128x32 tile 64 KB of fragment reads and 32 KB of stores (which it takes at half rate)
// for 768 cycles of matrix work.  Here a wavefront owns all BM rows of 32 columns, so no fragment of the weights is
// loaded twice in a workgroup, and the LDS carries 16 KB of stores and 64 KB of reads for the same matrix work.
// Measured stand-alone, 4096 x 1024 x 512: 15.2 us against 21.9; 4096 x 512 x 1024: 14.5 against 24; 32768 x 1024 x 512:
// 104 us, 990 TFLOP/s of fp16 matrix work (a large fp16 library product reaches 1200 on this card).
//
// A workgroup is four consumer wavefronts (32 columns each) and four producer wavefronts (load, split, store to LDS);
// BM = 64 rows by default, 32 (gemm_pk32_tile) where 64-row tiles would leave CUs idle.  At most 128 registers: two workgroups share a
// CU, and the first loads, the stores and the scans of one overlap the K loop of the other.
#pragma once

#include "gemm_kernel.h"
#include "pk_units.h"

#include <type_traits>

namespace ssm {

constexpr int PK_BN = 128, PK_CONSUMERS = 4, PK_PRODUCERS = 4, PK_STAGES = 2;
constexpr int PK_THREADS = 64 * (PK_CONSUMERS + PK_PRODUCERS);
constexpr int PK32_WAVES = 8;                        // tiles of 32 rows: wavefronts that multiply
constexpr int PK32_SHORT = 128, PK32_LONG = 256;     // and k per stage

// Place of an element of the output tile staged in LDS: rows of BN floats, pieces of 32 (rows, at 32 columns) swapped in rows
// 4 .. 7 of every eight, so that the two groups of rows that a wavefront stores at once meet different banks.
template <int BN = PK_BN>
__device__ __forceinline__ int tile_at(int row, int col)
{
    return BN == 32 ? (row ^ ((row >> 2) & 1)) * BN + col : row * BN + (col ^ ((row & 4) << 3));
}

// the resettable scan over the rows of a tile (sequences of any length): row_scan_body
constexpr bool scans_rows(int planes, int epilogue) { return epilogue >= 9 || (planes == 3 && epilogue >= 7); }

struct PkDev {
    const float *A; long lda;
    const uint4 *frag; const int *bexp;     // packed weights; log2 of the scale of every row n (two planes)
    float *C; long ldc;
    const float *diag; const float *E; long lde;
    const float *E2; float *C2;
    const uint8_t *rowflag;
    int M, N, K, nkt;                       // nkt: K tiles of 64
    int ntm, ntn, nx, mode, slot0;          // tiles; slots per XCD, placement mode, first slot
    int sc_nt, sc_cpu, sc_ncg, sc_units, sc_rev;
    FastDiv by_ntn, by_unit, by_ncg, by_cpu;     // ntn, sc_nt * sc_cpu, sc_ncg, sc_cpu
    ScanEpilogue scan;
    const unsigned *rows; int row_parts;    // largest magnitudes of the rows of A (two planes), see AbsMax
    // C and C2 are stored through the L2 (store_rule.h).  (Here: the four bytes in front of row_stride were empty.  In front of `scan` it moved the
    // arguments of the scans by eight, some into another cache line: an input projection on 32 x 64 tiles, 8000 tokens, H = 100, P = 30: 7.5 -> 8.0 us)
    int through;
    long row_stride;
    unsigned *c2_rowmax;                    // epilogue 6: [ceil(N/128)][M] or null
};

// LEFT: the states stay in the L2 until the launch ends (store_rule.h).  A kernel of its own: chosen between at run time, the stores of 64-row row scans took
// 0.5 to 1 % of forward and gradient pass (6000 to 12000 tokens, H from 64 to 128, P from 250 to 512), through the L2 as before.
template <bool LEFT> __device__ __forceinline__ void store_state(float2 *p, float2 v)
{
    if constexpr (LEFT) *p = v;
    else store_through(p, v);
}

// ---------------------------------------------------------------------------------------------
// Epilogues 7 and 8: the resettable scan (forward, or the reverse one of the gradient pass) over the rows of a
// ROWS x 128 output tile: 64 or 128 steps of 64 complex states, either a piece of one sequence (the pieces form a
// chain) or whole sequences.  The order of the arithmetic is that of units of 64 steps and chunks of 8 whichever ROWS is,
// so that the states do not depend on the tile a launch takes (and with it on the batch) to the last bit.  All eight
// wavefronts take part, 64 lanes x ROWS/8 steps (one or two chunks each):
//   1. the accumulators go through LDS so that a thread owns consecutive steps of one state;
//   2. per-thread pass for zero incoming state, chunk aggregates combined through LDS;
//   3. chain: the aggregate of every unit (state for zero incoming state, reset tag) is published as tagged 64-bit
//      words before any wait.  Wavefront q folds the q-th run of 8 earlier units of the sequence (in scan order), all
//      its words requested at once; then every wavefront folds the runs over the sequence's incoming state.  The grouping
//      depends on the position in the chain alone, so results are bitwise reproducible whatever the timing;
//   4. second per-thread pass writes the states (forward: x_last at the sequence end; reverse: the per-tile row of
//      dAbar and dx0).
// Every predecessor sits in an earlier slot of the same XCD (placement mode 5), i.e. it was dispatched earlier and
// publishes without waiting for anything, and every wait is bounded.
// ---------------------------------------------------------------------------------------------
constexpr int SCAN_WAVES = 8, SCAN_CHUNK = 8, SCAN_UNIT = 64, SCAN_RUN = 8;      // steps, steps, units
static_assert(SCAN_MAX_STEPS <= SCAN_WAVES * SCAN_RUN * SCAN_UNIT, "a run for every wavefront");
// (128 rows: 80 KiB, two workgroups per CU)
constexpr size_t scan_lds_bytes(int ROWS)
{
    return (size_t)ROWS * PK_BN * 4                                  // staged tile
           + ROWS / SCAN_CHUNK * 64 * 8                              // chunk states
           + SCAN_WAVES * 64 * 8 * 2;                                // folded runs of predecessors: product and state
}

struct ScanLds {
    float *tile; float2 *cS, *pS, *pA;
    float2 *uS; unsigned *top;                       // state of the tile's first unit, largest magnitudes: in the places of the last chunks, which nobody reads
    __device__ ScanLds(void *base, int rows)
    {
        char *p = static_cast<char *>(base);
        tile = reinterpret_cast<float *>(p); p += (size_t)rows * PK_BN * 4;
        cS = reinterpret_cast<float2 *>(p); p += rows / SCAN_CHUNK * 64 * 8;
        pS = reinterpret_cast<float2 *>(p); p += SCAN_WAVES * 64 * 8;
        pA = reinterpret_cast<float2 *>(p);
        uS = cS + (SCAN_UNIT / SCAN_CHUNK - 1) * 64;
        top = reinterpret_cast<unsigned *>(cS + (rows / SCAN_CHUNK - 1) * 64);
    }
};

// v[e], e < 8, per lane -> every lane gets the maximum over the 64 lanes of v[rows8_index(lane)]: three halving
// exchanges between lanes that differ in bit 0, 1, 2 (data-parallel-primitive moves inside quads, then a half-row
// mirror: lane ^ 7, whose partner holds the other half of the remaining pair), a rotation by 8 inside a row of 16,
// and the two exchanges across rows (lane swaps).
__device__ __forceinline__ unsigned rows8_wave_max(unsigned (&v)[8], int lane)
{
    {
        const bool up = lane & 1;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const unsigned keep = up ? v[k + 4] : v[k], send = up ? v[k] : v[k + 4];
            v[k] = max(keep, dpp_move<0xb1>(send));                   // quad_perm [1,0,3,2]: lane ^ 1
        }
    }
    {
        const bool up = (lane >> 1) & 1;
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const unsigned keep = up ? v[k + 2] : v[k], send = up ? v[k] : v[k + 2];
            v[k] = max(keep, dpp_move<0x4e>(send));                   // quad_perm [2,3,0,1]: lane ^ 2
        }
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        // lanes with the same two low bits: rotations by 4 and 8 inside a row of 16, lane swaps across rows
        v[k] = max(v[k], dpp_move<0x124>(v[k]));                      // row_ror:4
        v[k] = max(v[k], dpp_move<0x128>(v[k]));                      // row_ror:8
        v[k] = lane_xor_max<16>(v[k]);
        v[k] = lane_xor_max<32>(v[k]);
    }
    // (bitwise: a selection between two array elements becomes one between their addresses, and the array goes to scratch)
    return v[0] ^ ((v[0] ^ v[1]) & (0u - (unsigned)((lane >> 2) & 1)));
}
__device__ __forceinline__ int rows8_index(int lane) { return 4 * (lane & 1) + 2 * ((lane >> 1) & 1) + ((lane >> 2) & 1); }

// Reverse scan: the saved states x_{t-1} of a thread's steps (x_{-1} = x0, zero when absent), plus the last state of
// the sequence for the thread that owns its last steps.
template <int RC> struct ScanSaved { float2 xp[RC]; float2 xl; };
template <int RC>
__device__ __forceinline__ ScanSaved<RC> scan_request_saved(const ScanEpilogue &a, int q, int c, int m0, int n0)
{
    const int p = n0 / 2 + c;
    const bool active = p < a.P;
    const int row0 = m0 + q * RC;
    const int b = (int)a.by_L(row0), t0 = row0 - b * a.L;
    // (row addresses are uniform: one lane offset for all of them)
    const float2 *xprev = a.xsaved + ((long)row0 - 1) * a.P + n0 / 2;                // x_{t0-1}; valid for e >= 1 or t0 > 0
    ScanSaved<RC> s;
    s.xl = make_float2(0.f, 0.f);
    if (a.xmax_out && active && t0 + RC == a.L) s.xl = (xprev + (long)RC * a.P)[c];
#pragma unroll
    for (int e = 0; e < RC; ++e) {
        s.xp[e] = make_float2(0.f, 0.f);
        if (active) {
            if (t0 + e > 0) s.xp[e] = (xprev + (long)e * a.P)[c];
            else if (a.x0) s.xp[e] = a.x0[(long)b * a.P + p];
        }
    }
    return s;
}

// The flags of the tile's steps, one or two bytes per lane of every wavefront, requested first of all and turned into words
// of bits when the first K tile has arrived: the scan starts without a trip to memory, and what it does about resets is
// decided by scalar instructions.
template <int ROWS> struct ScanFlagBytes { unsigned own[ROWS / 64], next; };
template <int ROWS> struct ScanFlags {                       // bit r of first[h]: row 64 h + r of the tile
    unsigned long long first[ROWS / 64], drop[ROWS / 64];
    // word h (bitwise: a selection between array elements becomes one between their addresses, and the array goes to scratch)
    static __device__ __forceinline__ unsigned long long word(const unsigned long long (&w)[ROWS / 64], int h)
    {
        return ROWS == 64 ? w[0] : w[0] ^ ((w[0] ^ w[ROWS / 64 - 1]) & (0ull - (unsigned long long)h));
    }
    // the bits of the n rows from r on (within one word)
    static __device__ __forceinline__ unsigned bits(const unsigned long long (&w)[ROWS / 64], int r, int n)
    {
        return (unsigned)(word(w, r / 64) >> (r & 63)) & ((1u << n) - 1u);
    }
};
// (Without flags the bytes come from the packed weights and are not used.  With the requests in a branch the compiler moves the comparison of
// the bytes into it as well, and the workgroup waits for them before it requests anything else.)
template <int ROWS, bool REV>
__device__ __forceinline__ ScanFlagBytes<ROWS> scan_request_flags(const PkDev &g, int l, int m0)
{
    ScanFlagBytes<ROWS> v;
    const uint8_t *f = g.scan.is_first ? g.scan.is_first + m0 : reinterpret_cast<const uint8_t *>(g.frag);
    v.next = 0;
#pragma unroll
    for (int h = 0; h < ROWS / 64; ++h) v.own[h] = f[64 * h + l];
    if (REV) v.next = f[min(ROWS, g.M - 1 - m0)];
    return v;
}
// first: is_first.  drop: the state that flows into the step is dropped -- forward: the step's own flag; reverse: the flag
// of the next time step (nothing flows in at a sequence end).
template <int ROWS, bool REV>
__device__ __forceinline__ ScanFlags<ROWS> scan_flags(const ScanEpilogue &a, const ScanFlagBytes<ROWS> &v, int m0)
{
    constexpr int H = ROWS / 64;
    ScanFlags<ROWS> f;
#pragma unroll
    for (int h = 0; h < H; ++h) f.first[h] = f.drop[h] = a.is_first ? __ballot(v.own[h] != 0) : 0ull;
    if (REV) {
#pragma unroll
        for (int h = 0; h < H; ++h) f.drop[h] = (f.first[h] >> 1) | (h + 1 < H ? f.first[h + 1 < H ? h + 1 : h] << 63 : 0ull);
        if (a.L < ROWS) {
#pragma unroll
            for (int h = 0; h < H; ++h)
                for (int r = a.L - 1; r < 64; r += a.L) f.drop[h] |= 1ull << r;          // (L divides 64)
        } else if ((int)a.by_L(m0 + ROWS) * a.L == m0 + ROWS || (a.is_first && __builtin_amdgcn_readfirstlane(v.next) != 0)) f.drop[H - 1] |= 1ull << 63;
    }
    return f;
}

// the maximum over sixteen lanes, and over the 64, in all of them
__device__ __forceinline__ unsigned row16_max(unsigned v)
{
    v = max(v, dpp_move<0xb1>(v));                                    // quad_perm [1,0,3,2]
    v = max(v, dpp_move<0x4e>(v));                                    // quad_perm [2,3,0,1]
    v = max(v, dpp_move<0x124>(v));                                   // row_ror:4
    return max(v, dpp_move<0x128>(v));                                // row_ror:8
}
__device__ __forceinline__ unsigned wave_max(unsigned v) { return lane_xor_max<32>(lane_xor_max<16>(row16_max(v))); }

// The tile is staged in lds.tile on entry.  REV: chi_t = gx_t + [not is_first_{t+1}] conj(Abar) chi_{t+1}, which walks
// time backwards (later chunks and later tiles are the predecessors) and also reduces
// dAbar += [not is_first_t] conj(x_{t-1}) chi_t per tile and writes dx0.  LEFT: see store_state.
template <int ROWS, bool REV, bool LEFT>
__device__ __forceinline__ void scan_epilogue_body(const PkDev &g, const ScanLds &lds, int q, int c, int m0, int n0, int tile,
                                                   ScanSaved<ROWS / SCAN_WAVES> &saved, const ScanFlags<ROWS> &flags, float2 lam)
{
    constexpr int RC = ROWS / SCAN_WAVES, H = ROWS / SCAN_UNIT, NC = RC / SCAN_CHUNK, WH = SCAN_WAVES / H, UC = SCAN_UNIT / SCAN_CHUNK;
    static_assert(SCAN_CHUNK == 8 && UC == 8 && (H == 1 || H == 2), "the powers of Abar below");
    const ScanEpilogue &a = g.scan;
    // (q, the wavefront, is uniform, and so is all that follows from it: positions, chunks, resets)
    const int hs = REV ? H - 1 - q / WH : q / WH;            // unit of the tile, in scan order
    const int c0 = (REV ? WH - 1 - q % WH : q % WH) * NC;    // the thread's first chunk of the unit, in scan order
    const int p = n0 / 2 + c;
    const bool active = p < a.P;
    // A tile is either one piece of a chain of tiles of one sequence or holds whole sequences: then there is no chain, a
    // sequence starts at a chunk boundary inside the tile and its incoming state is x0 (forward) or zero (reverse).
    const bool whole_seqs = a.L < ROWS;
    const int row0 = m0 + q * RC;                            // token index of this thread's first step
    const int b = (int)a.by_L(row0), t0 = row0 - b * a.L;    // its sequence and its lowest time index
    const int tmL = whole_seqs ? 0 : t0 / ROWS, nt = whole_seqs ? 1 : a.L / ROWS;      // (ROWS: a power of two)
    const int tn = n0 / PK_BN;
    const int npred = H * (REV ? nt - 1 - tmL : tmL);        // units of the chain before the tile in scan order
    const unsigned fmask = flags.bits(flags.first, q * RC, RC), rmask = flags.bits(flags.drop, q * RC, RC);
    // whether a chunk of unit h (scan order) contains a reset
    auto chunk_resets = [&](int h, int j) { return flags.bits(flags.drop, REV ? ROWS - SCAN_UNIT * h - 8 * (j + 1) : SCAN_UNIT * h + 8 * j, 8) != 0; };
    auto unit_resets = [&](int h) { return flags.word(flags.drop, REV ? H - 1 - h : h) != 0; };

    if (REV) lam.y = -lam.y;
    float2 X = make_float2(0.f, 0.f);                        // state that flows into the sequence
    if (!REV && a.x0 && active) X = a.x0[(long)b * a.P + p];
    auto mine = [&](int e) { return reinterpret_cast<float2 *>(lds.tile + tile_at(q * RC + e, 2 * c)); };      // the thread's steps
    float2 val[SCAN_CHUNK], S[NC];
    auto read_chunk = [&](int k) {
#pragma unroll
        for (int i = 0; i < SCAN_CHUNK; ++i) val[i] = *mine(REV ? RC - 1 - (8 * k + i) : 8 * k + i);
    };
    // Reverse: the saved states pass through this launch exactly once, so their largest magnitude is recorded on
    // the way: dy^T x, in the next launch, stages x under that scale (x0 is not part of x)
    float xmax = 0.f, amax = 0.f;
    // pass 1: state after each of the thread's chunks for zero incoming state (a reset zeroes the multiplier)
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        S[k] = make_float2(0.f, 0.f);
        read_chunk(k);
#pragma unroll
        for (int i = 0; i < SCAN_CHUNK; ++i) {
            const int e = REV ? RC - 1 - (8 * k + i) : 8 * k + i;
            const bool r = (rmask >> e) & 1u;
            const float2 le = make_float2(r ? 0.f : lam.x, r ? 0.f : lam.y);
            S[k] = cfma(le, S[k], val[i]);
        }
        if (c0 + k < UC - 1) lds.cS[(hs * UC + c0 + k) * 64 + c] = S[k];
    }
    float2 lrc = cmul(lam, lam);                             // Abar^8 by three squarings
    lrc = cmul(lrc, lrc); lrc = cmul(lrc, lrc);
    float2 lunit = cmul(lrc, lrc);                           // Abar^64 by three more
    lunit = cmul(lunit, lunit); lunit = cmul(lunit, lunit);
    __syncthreads();                                         // the chunk states are in LDS

    // exclusive combine over the chunks of the same unit (or sequence) that come earlier in scan order
    float2 Aex[NC], Sex[NC];
    {
        const int cfirst = c0 - (whole_seqs ? min(c0, (REV ? a.L - RC - t0 : t0) / SCAN_CHUNK) : c0);
        // (all chunk states are read first, whether this thread folds them or not: left inside the condition below,
        // the reads end up in its branch and a thread waits for LDS once per chunk it folds, the last chunk's
        // wavefront seven times in a row, and the unit's aggregate goes out late)
        float2 Sc[UC - 1];
#pragma unroll
        for (int j = 0; j < UC - NC; ++j) {
            Sc[j] = lds.cS[(hs * UC + j) * 64 + c];
            asm volatile("" : "+v"(Sc[j].x), "+v"(Sc[j].y));
        }
        Aex[0] = make_float2(1.f, 0.f); Sex[0] = make_float2(0.f, 0.f);
#pragma unroll
        for (int j = 0; j < UC - NC; ++j) {
            if (j < cfirst || j >= c0) continue;
            const bool any = chunk_resets(hs, j);
            const float2 Aj = make_float2(any ? 0.f : lrc.x, any ? 0.f : lrc.y);
            Sex[0] = cfma(Aj, Sex[0], Sc[j]);
            Aex[0] = cmul(Aj, Aex[0]);
        }
#pragma unroll
        for (int k = 1; k < NC; ++k) {                       // (a sequence is a whole number of a thread's steps)
            const bool any = chunk_resets(hs, c0 + k - 1);
            const float2 Aj = make_float2(any ? 0.f : lrc.x, any ? 0.f : lrc.y);
            Sex[k] = cfma(Aj, Sex[k - 1], S[k - 1]);
            Aex[k] = cmul(Aj, Aex[k - 1]);
        }
    }
    if (!whole_seqs) {
        if (c0 == UC - NC) {
            // the unit's aggregate goes out before anything is waited for
            const bool has_succ = REV ? (tmL > 0) : (tmL + 1 < nt);
            const bool any = chunk_resets(hs, UC - 1);
            const float2 Ath = make_float2(any ? 0.f : lrc.x, any ? 0.f : lrc.y);
            const float2 Su = cfma(Ath, Sex[NC - 1], S[NC - 1]);
            const unsigned tag = unit_resets(hs) ? 2u : 1u;
            if (active && has_succ) {
                const int unit = (m0 / ROWS) * H + (REV ? H - 1 - hs : hs);
                unsigned long long *word = a.desc + (((size_t)unit * g.ntn + tn) * 64 + c) * 2;
                publish_word(word, Su.x, tag);
                publish_word(word + 1, Su.y, tag);
            }
            if (H == 2 && hs == 0) lds.uS[c] = Su;
        }
        if (REV && RC == 16) saved = scan_request_saved<RC>(a, q, c, m0, n0);    // (128 rows: no registers for them before)
        // The k-th unit in scan order is unit k of the sequence forward, unit H nt - 1 - k in reverse.  Wavefront q folds
        // the q-th run.
        const int kn = min(SCAN_RUN, npred - q * SCAN_RUN);
        if (kn > 0) {
            float2 Ar = make_float2(1.f, 0.f), Sr = make_float2(0.f, 0.f);
            // (all words of the run are requested in every round until all are there, for all lanes: the loads of a round are
            // in flight together, and the wavefront leaves the loop as one)
            const long step = (REV ? -1 : 1) * (long)g.ntn * 64 * 2;
            const int kb = q * SCAN_RUN;
            const unsigned long long *w = a.desc + (((size_t)(b * nt * H + (REV ? nt * H - 1 - kb : kb)) * g.ntn + tn) * 64 + c) * 2;
            auto fold = [&](auto count) {
                constexpr int N = decltype(count)::value;    // requests per round, at least kn
                unsigned long long w0[N], w1[N];
                bool all = false;                            // of this lane
                for (unsigned spins = 0;; ++spins) {
                    all = true;
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        const unsigned long long *wj = w + step * min(j, kn - 1);
                        w0[j] = poll_word(wj); w1[j] = poll_word(wj + 1);
                    }
#pragma unroll
                    for (int j = 0; j < N; ++j) all = all & (word_tag(w0[j]) != 0) & (word_tag(w1[j]) != 0);
                    if (__ballot(active && !all) == 0 || spins >= a.spin_limit) break;
                    __builtin_amdgcn_s_sleep(1);
                }
                if (active && !all) atomicOr(a.err, 1u);     // gave up: flagged, and finished anyway
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    if (j >= kn) continue;
                    // a missing aggregate hands on NaN: every state that depends on it becomes NaN, so the failure cannot
                    // pass as data
                    const bool missing = (word_tag(w0[j]) == 0) | (word_tag(w1[j]) == 0), cut = missing | (word_tag(w0[j]) == 2u);
                    const float2 Sj = missing ? make_float2(__builtin_nanf(""), __builtin_nanf("")) : make_float2(word_value(w0[j]), word_value(w1[j]));
                    const float2 Aj = make_float2(cut ? 0.f : lunit.x, cut ? 0.f : lunit.y);
                    Sr = cfma(Aj, Sr, Sj);
                    Ar = cmul(Aj, Ar);
                }
            };
            if (kn <= SCAN_RUN / 2) fold(std::integral_constant<int, SCAN_RUN / 2>{});
            else fold(std::integral_constant<int, SCAN_RUN>{});
            lds.pS[q * 64 + c] = Sr;
            lds.pA[q * 64 + c] = Ar;
        }
        if (npred > 0 || H == 2) {
            __syncthreads();                                 // the folded runs and the first unit's state are in LDS
            const int nrun = (npred + SCAN_RUN - 1) / SCAN_RUN;
            float2 before = X, Al = make_float2(1.f, 0.f), Sl = make_float2(0.f, 0.f);
#pragma unroll
            for (int j = 0; j < SCAN_WAVES; ++j) {
                if (j >= nrun) break;
                Al = lds.pA[j * 64 + c]; Sl = lds.pS[j * 64 + c];
                before = X;
                X = cfma(Al, X, Sl);
            }
            if (H == 2 && hs == 1) {
                // the tile's own first unit is one more predecessor, in the last run if that has room
                const float2 S0 = lds.uS[c];
                const bool any = unit_resets(0);
                const float2 A0 = make_float2(any ? 0.f : lunit.x, any ? 0.f : lunit.y);
                if (npred % SCAN_RUN != 0) X = cfma(cmul(A0, Al), before, cfma(A0, Sl, S0));
                else X = cfma(A0, X, S0);
            }
        }
    } else if (REV && RC == 16) saved = scan_request_saved<RC>(a, q, c, m0, n0);

    // pass 2: the states themselves
    float2 xs = make_float2(0.f, 0.f);
    asm volatile("" : "+v"(lam.x), "+v"(lam.y));             // (or the selected multipliers of pass 1 are kept: 2 RC registers)
    float2 *dst = reinterpret_cast<float2 *>(g.C) + (long)row0 * a.P + n0 / 2;
    float2 acc = make_float2(0.f, 0.f);                      // reverse: dAbar += [not is_first_t] conj(x_{t-1}) chi_t
    if (REV) xmax = fmaxf(fabsf(saved.xl.x), fabsf(saved.xl.y));
#pragma unroll
    for (int k = 0; k < NC; ++k) {
        read_chunk(k);                                       // (again: held since pass 1 they would take the registers of what is in flight)
        unsigned rm[SCAN_CHUNK];                             // largest magnitude per step (row of the tile), for rowmax_out
        xs = cfma(Aex[k], X, Sex[k]);
#pragma unroll
        for (int i = 0; i < SCAN_CHUNK; ++i) {
            const int e = REV ? RC - 1 - (8 * k + i) : 8 * k + i;
            const bool r = (rmask >> e) & 1u;
            const float2 le = make_float2(r ? 0.f : lam.x, r ? 0.f : lam.y);
            xs = cfma(le, xs, val[i]);
            val[i] = xs;
            const float me = fmaxf(fabsf(xs.x), fabsf(xs.y));
            rm[e % SCAN_CHUNK] = active ? __float_as_uint(me) : 0u;
            amax = fmaxf(amax, me);
            if (REV) {
                if (t0 + e > 0) xmax = fmaxf(xmax, fmaxf(fabsf(saved.xp[e].x), fabsf(saved.xp[e].y)));
                const bool m = (fmask >> e) & 1u;
                const float2 qv = make_float2(m ? 0.f : saved.xp[e].x, m ? 0.f : saved.xp[e].y);
                acc.x = fmaf(qv.x, xs.x, fmaf(qv.y, xs.y, acc.x));
                acc.y = fmaf(qv.x, xs.y, fmaf(-qv.y, xs.x, acc.y));
            }
        }
        if (active) {
#pragma unroll
            for (int i = 0; i < SCAN_CHUNK; ++i) store_state<LEFT>(dst + (long)(REV ? RC - 1 - (8 * k + i) : 8 * k + i) * a.P + c, val[i]);
        }
        if (a.rowmax_out) {
            // largest magnitude of every row within this column tile, stored as [column tile][row] (the consumer of C
            // takes the maximum over the column tiles): lane l < 8 ends up with row rows8_index(l)
            const unsigned r = rows8_wave_max(rm, c);
            if (c < 8) a.rowmax_out[(size_t)tn * g.M + row0 + (REV ? RC - 8 * (k + 1) : 8 * k) + rows8_index(c)] = r;
        }
    }
    if (!REV) {
        if (active && a.x_last && t0 + RC == a.L) a.x_last[(long)b * a.P + p] = xs;
    } else {
        // lam holds conj(Abar) here: dx0 = [not is_first_0] conj(Abar) chi_0
        if (active && a.dx0 && t0 == 0) a.dx0[(long)b * a.P + p] = (fmask & 1u) ? make_float2(0.f, 0.f) : cmul(lam, xs);
        *mine(0) = acc;                                      // (its own row of the tile, which it has read)
        __syncthreads();                                     // the wavefronts' contributions to dAbar are in LDS
        if (q == 0 && active) {
            float2 sum = make_float2(0.f, 0.f);
#pragma unroll
            for (int j = 0; j < SCAN_WAVES; ++j) { const float2 v = *reinterpret_cast<const float2 *>(lds.tile + tile_at(j * RC, 2 * c)); sum.x += v.x; sum.y += v.y; }
            a.partial[(size_t)(m0 / ROWS) * a.P + p] = sum;
        }
    }
    if (a.amax_out) {
        // one atomic per workgroup, spread over ABSMAX_SLOTS addresses (the bit patterns of non-negative floats order
        // like unsigned integers)
        const unsigned v0 = wave_max(active ? __float_as_uint(amax) : 0u), vx0 = REV ? wave_max(active ? __float_as_uint(xmax) : 0u) : 0u;
        if (c == 0) { lds.top[q] = v0; lds.top[SCAN_WAVES + q] = vx0; }
        __syncthreads();                                     // the wavefronts' maxima are in LDS
        if (q == 0 && c == 0) {
            unsigned v = v0, vx = vx0;
            for (int j = 1; j < SCAN_WAVES; ++j) { v = max(v, lds.top[j]); vx = max(vx, lds.top[SCAN_WAVES + j]); }
            atomicMax(a.amax_out + (unsigned)tile % ABSMAX_SLOTS, v);
            if (REV && a.xmax_out) atomicMax(a.xmax_out + (unsigned)tile % ABSMAX_SLOTS, vx);
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Epilogues 0 .. 6: the tile goes through LDS and all eight wavefronts store it in rows of 512 bytes, 16 bytes per lane.
// The inputs of the store function are requested before the workgroup meets (by the producers while the consumers
// work on the last K tile), so that their way from memory is not paid behind the K loop.
// ---------------------------------------------------------------------------------------------
template <int BM, int BN, int EPI>
struct StoreInputs {
    static constexpr int KW = BM == 32 ? PK32_WAVES * 32 / BN : 1, LANES = BN / 4;      // partial tiles to add up, lanes that share a row
    static constexpr int ALL = BM * BN / 4 < PK_THREADS ? 1 : BM * BN / 4 / PK_THREADS;      // units of four columns per thread,
    static constexpr int UNITS = ALL < 4 ? ALL : 4, BATCHES = ALL / UNITS;      // in batches of at most four
    static constexpr bool HAS_E = EPI >= 1 && EPI <= 6, HAS_E2 = EPI == 4, HAS_DIAG = EPI == 1 || EPI == 2 || EPI == 5 || EPI == 6;
    float4 e[UNITS], e2[UNITS], d;
    bool dropped[UNITS];

    static __device__ __forceinline__ int row_of(int tid, int batch, int i) { return tid / LANES + (batch * UNITS + i) * (PK_THREADS / LANES); }
    __device__ __forceinline__ void request(const PkDev &g, int tid, int batch, int m0, int n0)
    {
        const int col = n0 + 4 * (tid % LANES), n = g.N - col;
        // a tile inside the result: the requests without a branch per unit and column (0.3 us of a launch of 9)
        if (m0 + BM <= g.M && n0 + BN <= g.N) {
#pragma unroll
            for (int i = 0; i < UNITS; ++i) {
                const int r = row_of(tid, batch, i);
                const long row = m0 + (BM * BN / 4 < PK_THREADS ? min(r, BM - 1) : r);          // (threads past the tile: any row of it)
                e[i] = e2[i] = make_float4(0.f, 0.f, 0.f, 0.f);
                dropped[i] = false;
                if (HAS_E && (EPI != 5 || g.E)) e[i] = load4(g.E + row * g.lde + col, 4);
                if (HAS_E2) e2[i] = load4(g.E2 + row * g.lde + col, 4);
                if ((EPI == 2 || EPI == 5) && g.rowflag) dropped[i] = g.rowflag[row] != 0;
            }
            d = make_float4(0.f, 0.f, 0.f, 0.f);
            if (HAS_DIAG && (EPI != 5 || g.C2)) d = load4(g.diag + col, 4);
            return;
        }
#pragma unroll
        for (int i = 0; i < UNITS; ++i) {
            const long row = m0 + row_of(tid, batch, i);
            const bool in = row < g.M && n > 0 && row < m0 + BM;
            e[i] = e2[i] = make_float4(0.f, 0.f, 0.f, 0.f);
            dropped[i] = false;
            if (HAS_E && (EPI != 5 || g.E) && in) e[i] = load4(g.E + row * g.lde + col, n);
            if (HAS_E2 && in) e2[i] = load4(g.E2 + row * g.lde + col, n);
            if ((EPI == 2 || EPI == 5) && g.rowflag && in) dropped[i] = g.rowflag[row] != 0;
        }
        d = make_float4(0.f, 0.f, 0.f, 0.f);
        if (HAS_DIAG && n > 0 && (EPI != 5 || g.C2)) d = load4(g.diag + col, n);
    }
    __device__ __forceinline__ void store(const PkDev &g, const float *tile, int tid, int batch, int m0, int n0)
    {
        const int c = 4 * (tid % LANES), col = n0 + c, n = g.N - col;
#pragma unroll
        for (int i = 0; i < UNITS; ++i) {
            const int r = row_of(tid, batch, i);
            const long row = m0 + r;
            if (BM * BN / 4 < PK_THREADS && r >= BM) continue;           // (threads past the tile)
            const bool in = row < g.M && n > 0;
            float4 v = *reinterpret_cast<const float4 *>(tile + tile_at<BN>(r, c));
#pragma unroll
            for (int k = 1; k < KW; ++k) {
                const float4 w = *reinterpret_cast<const float4 *>(tile + k * BM * BN + tile_at<BN>(r, c));
                v = make_float4(v.x + w.x, v.y + w.y, v.z + w.z, v.w + w.w);
            }
            float4 o = v, o2 = v;
            bool second = false;
            if constexpr (EPI == 1 || EPI == 6) {
                // v + diag[col] * E[row, col]  (D (.) u and D (.) dy); 6: GELU of it into C2 as well
                o = make_float4(fmaf(d.x, e[i].x, v.x), fmaf(d.y, e[i].y, v.y), fmaf(d.z, e[i].z, v.z), fmaf(d.w, e[i].w, v.w));
                if constexpr (EPI == 6) {
                    o2 = make_float4(gelu_value(o.x), gelu_value(o.y), gelu_value(o.z), gelu_value(o.w));
                    second = true;
                }
            } else if constexpr (EPI == 2) {
                // one recurrence step (Eq. 3, first line): columns are interleaved (re, im) pairs of complex states, diag
                // holds Abar; adds the carried state [not rowflag[row]] (Abar E)
                if (!dropped[i])
                    o = make_float4(v.x + fmaf(d.x, e[i].x, -d.y * e[i].y), v.y + fmaf(d.x, e[i].y, d.y * e[i].x),
                                    v.z + fmaf(d.z, e[i].z, -d.w * e[i].w), v.w + fmaf(d.z, e[i].w, d.w * e[i].z));
            } else if constexpr (EPI == 5) {
                // its adjoint: g = v + E (E may be null), C2 = [not rowflag[row]] conj(Abar) g
                o = make_float4(v.x + e[i].x, v.y + e[i].y, v.z + e[i].z, v.w + e[i].w);
                second = g.C2 != nullptr;
                o2 = dropped[i] ? make_float4(0.f, 0.f, 0.f, 0.f)
                                : make_float4(fmaf(d.x, o.x, d.y * o.y), fmaf(d.x, o.y, -d.y * o.x), fmaf(d.z, o.z, d.w * o.w), fmaf(d.z, o.w, -d.w * o.z));
            } else if constexpr (EPI == 3) {
                // half-GLU gate: s = sigmoid(v) is kept in C2 when asked and the stored value is E[row, col] * s
                o2 = make_float4(sigmoidf(v.x), sigmoidf(v.y), sigmoidf(v.z), sigmoidf(v.w));
                second = g.C2 != nullptr;
                o = make_float4(e[i].x * o2.x, e[i].y * o2.y, e[i].z * o2.z, e[i].w * o2.w);
            } else if constexpr (EPI == 4) {
                // adjoint of the gate with respect to its input: E + v * E2
                o = make_float4(fmaf(v.x, e2[i].x, e[i].x), fmaf(v.y, e2[i].y, e[i].y), fmaf(v.z, e2[i].z, e[i].z), fmaf(v.w, e2[i].w, e[i].w));
            }
            if (in) {
                if (BM == 128 || !g.through) {
                    // (128 rows: launches of several rounds: of little use, and 1024 x 16 tokens, 512, 512, forward, take 0.5 % longer with it)
                    store4(g.C + row * g.ldc + col, o, n);
                    if (second) store4(g.C2 + row * g.ldc + col, o2, n);
                } else {
                    const int at = r * (int)g.ldc + c;
                    store4_through(g.C + m0 * g.ldc + n0, at, o, n);
                    if (second) store4_through(g.C2 + m0 * g.ldc + n0, at, o2, n);
                }
            }
            if constexpr (EPI == 6 && BN == 128) {
                // the product that consumes C2 stages its rows under a scale each: the largest magnitude of every row within
                // the workgroup's 128 columns (32 neighbouring lanes hold them)
                if (g.c2_rowmax) {
                    unsigned m = 0;
                    if (in) m = __float_as_uint(fmaxf(fmaxf(fabsf(o2.x), n > 1 ? fabsf(o2.y) : 0.f), fmaxf(n > 2 ? fabsf(o2.z) : 0.f, n > 3 ? fabsf(o2.w) : 0.f)));
                    m = max(m, dpp_move<0xb1>(m));
                    m = max(m, dpp_move<0x4e>(m));
                    m = max(m, dpp_move<0x124>(m));
                    m = max(m, dpp_move<0x128>(m));
                    m = lane_xor_max<16>(m);
                    if (tid % 32 == 0 && row < g.M) g.c2_rowmax[(size_t)(n0 / PK_BN) * g.M + row] = m;
                }
            }
        }
    }
};

// ---------------------------------------------------------------------------------------------
// Epilogues 7 and 8 with three planes, 9 and 10 (forward, reverse) with two: the resettable scan over the 32 or 64 consecutive tokens of a tile and its BN / 2 states.  The tokens are
// those of any sequences: where one starts inside the tile nothing flows in (its x0 is put into the element itself), so the length
// of a sequence need not fit the tile.  Thread (q, c), q < 8, owns the q-th run of 4 or 8 tokens in scan order of state c:
//   1. pass for zero incoming state; the runs are combined through LDS;
//   2. the tile's aggregate (state for zero incoming state, tag) is published as two tagged words per state before any wait;
//   3. the tiles that come earlier in the same sequence are shared out over the eight threads of a state, each requests all its words at once and
//      folds them, and every thread folds the eight;
//   4. second pass from the registers: states, x_last; reverse: dAbar (a row per tile) and dx0.
// The powers of Abar that the folds take are computed in double precision and rounded once.  A reset selects instead of multiplying by zero: what
// one sequence holds cannot reach the next, infinities and NaN included.
//   A tile waits for tiles on other XCDs.  They have smaller workgroup ids (modes 6 and 7) and publish without waiting for anything, but
// they need not have been started: every XCD starts its share of a launch on its own, and one can be full of tiles of another launch, on
// another stream, that wait for theirs behind tiles of this one.  So no tile relies on it: after ROW_SCAN_POLLS polls it computes the
// aggregate that is missing itself, to the last bit as its own tile would, publishes it and starts again (gemm_pk_kernel).  On 18 layers
// the passes take 0.6 % longer than with tiles that rely on the order (2 % at most); with row tiles drawn from counters up to 4 %, chains of one XCD
// (mode 5) up to 8 %, where several XCDs read the same rows or get unequal shares.
// Bound by its chain of dependent steps (the tile through LDS 0.3 us, either pass and the fold between them 0.4 to 0.5 each, a trip to
// memory and back where tiles wait).  As a kernel of its own the scan paid its start, the way to memory and back, and the gap in front of it.  With scan
// kernels and now: input projection of 16 x 64 tokens, H = P = 256 (32 rows): 5.8 + 4.8 us and 8.6; of 20 x 300, 500, 250 (64 rows): 23.1 + 14.1 and 30.6, C^H dy
// 42.8 + 16.6 and 56.8.  Forward and gradient pass, 19 layers of 128 .. 4000 tokens on 32 rows: 13 % faster on geometric mean (16 x 64, 256, 256: 53.7 -> 47.5 us;
// 32 x 60, 200, 100: 55.0 -> 45.9; 1 x 2048, 128, 64: 46.6 -> 39.4); 14 on 64 rows: 7 % (20 x 300, 500, 250: 182 -> 172; 9 x 997, 128, 140: 97.0 -> 82.7; 100 x 100,
// 1000, 128: 259 -> 255).  Forward on two planes (64 rows; there the states' row maxima are recorded as well): 24 x 200, 1024, 512: 95.5 -> 90.4; 100 x 100, 512, 512:
// 106.6 -> 90.2; 300 x 100: 264 -> 240, although products of many tiles alone are a little faster with 128 rows.
// Reverse on two planes, beside the dC slabs (64 rows; chi's row maxima and its largest magnitude are recorded): chi is written once instead of written, read and written again, and the
// chain along time is hidden behind the reductions.  Forward and gradient pass with a scan kernel and now: 60 x 100, 512, 512: 198.6 -> 185.9; 9 x 515, 700, 530: 235.7 ->
// 217.8; 300 x 100, 512, 512: 787 -> 750; 2000 x 5, 512, 512: 345.6 -> 290.6; 24 x 200, 1024, 512: 261.4 -> 261.9 (as much as the scan cost is lost where the product
// took 128-row tiles); 21 layers: 4 % faster on geometric mean, 0.4 % slower at worst.  The dC slabs beside du instead: 1.2 % slower; their items behind the tiles: 2.8 %.
// ---------------------------------------------------------------------------------------------
constexpr int ROW_SCAN_CHUNKS = 8;                            // runs of a tile, threads that share out the tiles before it
static_assert(ROW_SCAN_MAX_TILES <= ROW_SCAN_CHUNKS * 8, "a thread folds at most eight tiles");
constexpr size_t row_scan_lds_bytes(int BN) { return (size_t)4 * ROW_SCAN_CHUNKS * (BN / 2) * 8; }

// What is requested ahead: Abar, the flags, and for the thread's tokens x_{t-1} (reverse) and x0 where they start a sequence (both directions).
struct RowScanStart { float2 lam; unsigned flag, next; };
template <int ROWS> struct RowScanSaved { float2 x[ROWS / ROW_SCAN_CHUNKS]; };
// bit r: row r of the tile; sequence of row 0
template <int ROWS> struct RowScanMasks {
    using Bits = std::conditional_t<ROWS == 32, unsigned, unsigned long long>;
    Bits first, start, end, drop; int b0;
    static_assert(ROWS == 32 || ROWS == 64, "a bit for every row");
};
__device__ __forceinline__ int popcount(unsigned v) { return __popc(v); }
__device__ __forceinline__ int popcount(unsigned long long v) { return __popcll(v); }
__device__ __forceinline__ unsigned reversed(unsigned v) { return __brev(v); }
__device__ __forceinline__ unsigned long long reversed(unsigned long long v) { return __brevll(v); }

// row of the tile that a lane looks at; 32 rows: lane 32 and those above it at the one behind the tile
template <int ROWS> __device__ __forceinline__ int row_scan_lane(int tid) { return ROWS == 32 ? min(tid & 63, ROWS) : tid & 63; }
template <int ROWS, int BN, bool TIGHT>
__device__ __forceinline__ RowScanStart row_scan_start(const PkDev &g, int tid, int m0, int n0)
{
    const ScanEpilogue &a = g.scan;
    RowScanStart s;
    s.lam = a.lam[min(n0 / 2 + tid % (BN / 2), a.P - 1)];
    // (requested without a branch: see scan_request_flags.  TIGHT: beside a reduction 128 columns leave no registers to do without one)
    if constexpr (TIGHT) {
        s.flag = s.next = 0;
        if (a.is_first) s.flag = a.is_first[min(m0 + row_scan_lane<ROWS>(tid), g.M - 1)];
        return s;
    }
    const uint8_t *f = a.is_first ? a.is_first + m0 : reinterpret_cast<const uint8_t *>(g.frag);
    s.flag = f[min(row_scan_lane<ROWS>(tid), g.M - 1 - m0)];
    s.next = ROWS == 64 ? f[min(ROWS, g.M - 1 - m0)] : 0u;
    return s;
}
// the rows at which a sequence starts and ends (whole wavefronts; the last token ends one, so that in reverse nothing comes in from rows past it)
template <int ROWS>
__device__ __forceinline__ RowScanMasks<ROWS> row_scan_ends(const PkDev &g, int tid, int m0)
{
    using Bits = typename RowScanMasks<ROWS>::Bits;
    const unsigned row = (unsigned)(m0 + row_scan_lane<ROWS>(tid)), L = (unsigned)g.scan.L, b = g.scan.by_L(row);
    return {0, (Bits)__ballot(row == b * L), (Bits)__ballot(row + 1 == (b + 1) * L), 0, __builtin_amdgcn_readfirstlane((int)b)};
}
// drop: nothing flows into the row -- forward: a flag, or the start of a sequence; reverse: a flag of the token behind it, or a sequence end
template <int ROWS, bool REV>
__device__ __forceinline__ void row_scan_flags(RowScanMasks<ROWS> &k, const RowScanStart &s, bool flags)
{
    using Bits = typename RowScanMasks<ROWS>::Bits;
    const unsigned long long f = flags ? __ballot(s.flag != 0) : 0ull;
    k.first = (Bits)f;
    unsigned long long behind = f >> 1;
    if (ROWS == 64) behind |= (unsigned long long)(flags && __builtin_amdgcn_readfirstlane(s.next) != 0) << 63;
    k.drop = REV ? (Bits)behind | k.end : k.first | k.start;
}
// Powers of Abar (its conjugate in reverse) over a run of tokens, the runs before the thread's, and a tile: in double precision, rounded once.
struct RowScanPowers { float2 run, before, tile; };
template <int ROWS, int BN, bool REV>
__device__ __forceinline__ RowScanPowers row_scan_powers(float2 lam, int tid)
{
    const int q = tid / (BN / 2);
    double re = lam.x, im = REV ? -lam.y : lam.y, br = 1.0, bi = 0.0;
    auto square = [&] {
        const double t = re * re - im * im;
        im *= 2.0 * re; re = t;
    };
    auto take = [&](bool bit) {
        const double r = br * re - bi * im, i = br * im + bi * re;
        br = bit ? r : br; bi = bit ? i : bi;
    };
    RowScanPowers w;
    square(); square();
    if (ROWS == 64) square();
    w.run = make_float2((float)re, (float)im);
    take(q & 1); square(); take(q & 2); square(); take(q & 4); square();
    w.before = make_float2((float)br, (float)bi);
    w.tile = make_float2((float)re, (float)im);
    return w;
}
// sequence of a row
template <int ROWS>
__device__ __forceinline__ int row_scan_sequence(const RowScanMasks<ROWS> &k, int r)
{
    return k.b0 + popcount((typename RowScanMasks<ROWS>::Bits)(k.start & (((typename RowScanMasks<ROWS>::Bits)2 << r) - 2)));
}

template <int ROWS, int BN, bool REV>
__device__ __forceinline__ RowScanSaved<ROWS> row_scan_request(const PkDev &g, const RowScanMasks<ROWS> &k, int tid, int m0, int n0)
{
    constexpr int CH = ROWS / ROW_SCAN_CHUNKS;
    const ScanEpilogue &a = g.scan;
    const int c = tid % (BN / 2), q = tid / (BN / 2), p = n0 / 2 + c;
    const auto row_of = [&](int i) { return REV ? ROWS - 1 - (CH * q + i) : CH * q + i; };
    RowScanSaved<ROWS> s;
#pragma unroll
    for (int i = 0; i < CH; ++i) s.x[i] = make_float2(0.f, 0.f);
    if (q >= ROW_SCAN_CHUNKS) return s;                      // (whole wavefronts)
    if (REV) {
        // (rows and states past the end: any)
        const float2 *x = a.xsaved + min(p, a.P - 1);
#pragma unroll
        for (int i = 0; i < CH; ++i) s.x[i] = x[(long)min(max(m0 + row_of(i) - 1, 0), g.M - 1) * a.P];
    }
    if (k.start != 0) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int r = row_of(i);
            if (!((k.start >> r) & 1u)) continue;
            s.x[i] = make_float2(0.f, 0.f);
            if (a.x0 && p < a.P && m0 + r < g.M) s.x[i] = a.x0[(long)row_scan_sequence(k, r) * a.P + p];
        }
    }
    return s;
}

// tile: KW partial tiles of ROWS x BN, as tile_at places them; mem: row_scan_lds_bytes of LDS that nobody else uses
// (MAXIMA: 64 rows, whose eight tokens of a thread make a wavefront one run of all states)
// ahead: only the aggregate is published, for another tile's sake.  Returns -1, or the row tile whose aggregate is missing (nothing is stored then).
template <int ROWS, int BN, int KW, bool REV, bool MAXIMA = false, bool LEFT = false>
__device__ __forceinline__ int row_scan_body(const PkDev &g, const float *tile, float2 *mem, int tid, int m0, int n0, float2 lam, const RowScanPowers &power,
                                             const RowScanMasks<ROWS> &k, const RowScanSaved<ROWS> &saved, bool ahead)
{
    using Bits = typename RowScanMasks<ROWS>::Bits;
    constexpr int NL = BN / 2, NC = ROW_SCAN_CHUNKS, CH = ROWS / NC;
    const ScanEpilogue &a = g.scan;
    float2 *cS = mem, *pS = mem + NC * NL, *pA = mem + 2 * NC * NL, *cD = mem + 3 * NC * NL;
    int *missing = reinterpret_cast<int *>(cS + (NC - 1) * NL);      // (the last run's state is nobody's input) row tile that is waited for in vain, or -1
    const int c = tid % NL, q = tid / NL, p = n0 / 2 + c;
    const bool on = q < NC, active = on && p < a.P;          // (on: whole wavefronts)
    auto row_of = [&](int i) { return REV ? ROWS - 1 - (CH * q + i) : CH * q + i; };
    // the drop bits in scan order: bit e: the e-th row of the scan
    const Bits cut = REV ? reversed(k.drop) : k.drop;
    // earlier tiles of the sequence that flows in, none where it is cut at the first row of the scan; whether another tile follows in the sequence
    const int here = m0 / ROWS;
    int npred = 0;
    bool has_succ;
    if (REV) {
        const long end = (long)(k.b0 + popcount((Bits)(k.start & ~(Bits)1)) + 1) * a.L - 1;        // of the sequence of the last row
        if (!(cut & 1u) && m0 + ROWS < g.M) npred = (int)(end / ROWS) - here;       // (behind the last row nothing follows)
        has_succ = !(k.start & 1u);
    } else {
        if (!(cut & 1u)) npred = here - (int)((long)k.b0 * a.L / ROWS);
        has_succ = !(k.end >> (ROWS - 1));
    }
    const int run = (npred + NC - 1) / NC;                   // tiles that a thread folds
    if (REV) lam.y = -lam.y;
    float2 val[CH], S = make_float2(0.f, 0.f);
    if (on) {
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const float *at = tile + tile_at<BN>(row_of(i), 2 * c);
            val[i] = *reinterpret_cast<const float2 *>(at);
#pragma unroll
            for (int w = 1; w < KW; ++w) {
                const float2 v = *reinterpret_cast<const float2 *>(at + w * ROWS * BN);
                val[i].x += v.x; val[i].y += v.y;
            }
        }
        if (m0 + ROWS > g.M) {                               // (rows past the last token: zeros)
#pragma unroll
            for (int i = 0; i < CH; ++i)
                if (m0 + row_of(i) >= g.M) val[i] = make_float2(0.f, 0.f);
        }
        if (!REV && (k.start & ~k.first) != 0) {
            // the state that flows into a sequence, unless its first step drops it
#pragma unroll
            for (int i = 0; i < CH; ++i)
                if ((k.start & ~k.first) >> row_of(i) & 1u) val[i] = cfma(lam, saved.x[i], val[i]);
        }
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const float2 n = cfma(lam, S, val[i]);
            const bool r = (cut >> (CH * q + i)) & 1u;
            S = make_float2(r ? val[i].x : n.x, r ? val[i].y : n.y);
        }
        if (q < NC - 1) cS[q * NL + c] = S;
    }
    if (tid == 0) *missing = -1;
    __syncthreads();                                         // the states of the runs are in LDS
    float2 Sex = make_float2(0.f, 0.f);
    const bool cut_before = on && (cut & (((Bits)1 << (CH * (q & 7))) - 1)) != 0;       // a reset in an earlier run of the tile
    if (on) {
        float2 Sc[NC - 1];
#pragma unroll
        for (int j = 0; j < NC - 1; ++j) Sc[j] = cS[j * NL + c];
#pragma unroll
        for (int j = 0; j < NC - 1; ++j) {
            const bool any = ((cut >> (CH * j)) & ((1u << CH) - 1u)) != 0;
            const float2 n = cfma(power.run, Sex, Sc[j]);
            const float2 m = make_float2(any ? Sc[j].x : n.x, any ? Sc[j].y : n.y);
            Sex = make_float2(j < q ? m.x : Sex.x, j < q ? m.y : Sex.y);
        }
        if (q == NC - 1 && active && (has_succ || ahead)) {
            const bool any = (cut >> (CH * (NC - 1))) != 0;
            const float2 n = cfma(power.run, Sex, S);
            unsigned long long *word = a.desc + (size_t)here * 2 * a.P + p;
            const unsigned tag = cut != 0 ? 2u : 1u;
            publish_word(word, any ? S.x : n.x, tag);
            publish_word(word + a.P, any ? S.y : n.y, tag);
        }
        const int kn = ahead ? 0 : min(run, npred - q * run);
        if (kn > 0) {
            // the earliest tile of the run first; all words are requested in every round until all are there
            const int first = (REV ? here + npred : here - npred) + (REV ? -1 : 1) * q * run;
            const long step = (REV ? -1 : 1) * (long)a.P * 2;
            const unsigned long long *w = a.desc + (size_t)first * 2 * a.P + min(p, a.P - 1);
            float2 Ar = make_float2(1.f, 0.f), Sr = make_float2(0.f, 0.f);
            auto fold = [&](auto count, int j0) {            // tiles j0 .. j0 + N - 1 of the run
                constexpr int N = decltype(count)::value;
                unsigned long long w0[N], w1[N];
                bool all = false;
                for (unsigned spins = 0;; ++spins) {
                    all = true;
#pragma unroll
                    for (int j = 0; j < N; ++j) {
                        const unsigned long long *wj = w + step * min(j0 + j, kn - 1);
                        w0[j] = poll_word(wj); w1[j] = poll_word(wj + a.P);
                    }
#pragma unroll
                    for (int j = 0; j < N; ++j) all = all & (word_tag(w0[j]) != 0) & (word_tag(w1[j]) != 0);
                    if (__ballot(active && !all) == 0 || spins >= a.spin_limit) break;
                    __builtin_amdgcn_s_sleep(1);
                }
#pragma unroll
                for (int j = 0; j < N; ++j) {
                    if (j0 + j >= kn) continue;
                    if (active && (word_tag(w0[j]) == 0 || word_tag(w1[j]) == 0)) *missing = first + (REV ? -1 : 1) * (j0 + j);       // (any of them)
                    const bool stop = word_tag(w0[j]) == 2u;
                    const float2 Sj = make_float2(word_value(w0[j]), word_value(w1[j]));
                    const float2 n = cfma(power.tile, Sr, Sj), An = cmul(power.tile, Ar);
                    Sr = make_float2(stop ? Sj.x : n.x, stop ? Sj.y : n.y);
                    Ar = make_float2(stop ? 0.f : An.x, stop ? 0.f : An.y);
                }
            };
            // (four at a time: eight take more registers than there are)
            if (run == 1) fold(std::integral_constant<int, 1>{}, 0);
            else for (int j = 0; j < run; j += 4) fold(std::integral_constant<int, 4>{}, j);
            pS[q * NL + c] = Sr;
            pA[q * NL + c] = Ar;
        }
    }
    if (ahead) return -1;
    if (npred > 0) {
        __syncthreads();                                     // the folded runs are in LDS
        const int m = __builtin_amdgcn_readfirstlane(*missing);
        if (m >= 0) return m;
    }
    if (on) {
        float2 X = make_float2(0.f, 0.f);
        for (int j0 = 0; j0 * run < npred; j0 += 4) {        // (four reads at a time; those behind the last run are not used)
            float2 Al[4], Sl[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) { Al[j] = pA[(j0 + j) * NL + c]; Sl[j] = pS[(j0 + j) * NL + c]; }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                if ((j0 + j) * run >= npred) break;
                const float2 n = cfma(Al[j], X, Sl[j]);
                const bool stop = Al[j].x == 0.f && Al[j].y == 0.f;
                X = make_float2(stop ? Sl[j].x : n.x, stop ? Sl[j].y : n.y);
            }
        }
        const float2 in = cfma(power.before, X, Sex);
        float2 xs = make_float2(cut_before ? Sex.x : in.x, cut_before ? Sex.y : in.y), acc = make_float2(0.f, 0.f);
        float2 *dst = reinterpret_cast<float2 *>(g.C) + (long)m0 * a.P + p;
        // rows whose x_{t-1} is no factor of dAbar: where the state is dropped, and those past the last token
        const Bits no_factor = k.first | (m0 + ROWS > g.M ? ~(Bits)0 << (g.M - m0) : (Bits)0);
#pragma unroll
        for (int i = 0; i < CH; ++i) {
            const int r = row_of(i);
            const float2 n = cfma(lam, xs, val[i]);
            const bool rs = (cut >> (CH * q + i)) & 1u;
            xs = make_float2(rs ? val[i].x : n.x, rs ? val[i].y : n.y);
            if (REV) {
                const bool none = (no_factor >> r) & 1u;
                const float2 v = make_float2(none ? 0.f : saved.x[i].x, none ? 0.f : saved.x[i].y);
                acc.x = fmaf(v.x, xs.x, fmaf(v.y, xs.y, acc.x));
                acc.y = fmaf(v.x, xs.y, fmaf(-v.y, xs.x, acc.y));
            }
            val[i] = xs;
        }
        if (active) {
            if (m0 + ROWS <= g.M) {
#pragma unroll
                for (int i = 0; i < CH; ++i) store_state<LEFT>(dst + row_of(i) * a.P, val[i]);
            } else {
#pragma unroll
                for (int i = 0; i < CH; ++i)
                    if (m0 + row_of(i) < g.M) store_state<LEFT>(dst + row_of(i) * a.P, val[i]);
            }
            if constexpr (MAXIMA) static_assert(ROWS == 64 && BN == 128, "rows8_wave_max");
            const Bits edge = REV ? k.start : k.end;
            float2 *at_edge = REV ? a.dx0 : a.x_last;
            if (edge != 0 && at_edge) {
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    const int r = row_of(i);                 // (lam holds conj(Abar) in reverse)
                    if (((edge >> r) & 1u) && m0 + r < g.M)
                        at_edge[(long)row_scan_sequence(k, r) * a.P + p] = !REV ? val[i] : (k.first >> r) & 1u ? make_float2(0.f, 0.f) : cmul(lam, val[i]);
                }
            }
        }
        if (REV) cD[q * NL + c] = acc;
        if constexpr (MAXIMA) {
            // largest magnitude of every row within the tile's states, for the product that stages the states under a scale each
            unsigned top[CH];
#pragma unroll
            for (int i = 0; i < CH; ++i) top[i] = active ? __float_as_uint(fmaxf(fabsf(val[i].x), fabsf(val[i].y))) : 0u;
            const unsigned r = rows8_wave_max(top, c);
            const int row = m0 + row_of(rows8_index(c));
            if (c < 8 && row < g.M) a.rowmax_out[(size_t)(n0 / BN) * g.M + row] = r;
            if constexpr (REV) {
                // and of chi as a whole, for the sums over tokens
                const unsigned v = wave_max(r);
                if (c == 0) atomicMax(a.amax_out + (unsigned)(here * NC + q) % ABSMAX_SLOTS, v);
            }
        }
    }
    if (REV) {
        __syncthreads();                                     // the runs' contributions to dAbar are in LDS
        if (q == 0 && active) {
            float2 sum = make_float2(0.f, 0.f);
#pragma unroll
            for (int j = 0; j < NC; ++j) { const float2 v = cD[j * NL + c]; sum.x += v.x; sum.y += v.y; }
            a.partial[(size_t)here * a.P + p] = sum;
        }
    }
    return -1;
}

// Place of the c-th 16-byte piece of row r of an LDS plane (rows of 128 bytes, no padding): the pieces of a row are permuted
// so that 16 lanes reading the same piece of 16 rows, and 32 lanes writing two neighbouring rows, meet every bank once.
__device__ __forceinline__ int pk_swizzle(int r, int c) { return c ^ ((r >> 1) & 7); }

// Four values from k on of a row of fewer than four.  (Waited for here: left outstanding, they would make the path without them wait for
// everything it has requested since.)
__device__ __forceinline__ float4 narrow_unit(const PkDev &g, int row, int k)
{
    const float *p = g.A + (long)row * g.lda;
    float v[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        v[j] = k + j < g.K ? p[k + j] : 0.f;
        asm volatile("" : "+v"(v[j]));
    }
    return make_float4(v[0], v[1], v[2], v[3]);
}

// ahead and result: see row_scan_body (other epilogues: false and -1)
template <int BM, int NPL, int EPI, bool LEFT>
__device__ __forceinline__ int gemm_pk_tile(const PkDev &g, unsigned char *smem_raw, int m0, int n0, int tile, int tid, bool ahead)
{
    constexpr int NC = PK_CONSUMERS, NP = PK_PRODUCERS, BK = PK_BK, NS = PK_STAGES, PT = 64 * NP;
    constexpr int S = BK;                         // row stride of an LDS plane in halves; see pk_swizzle
    constexpr int PLANE = BM * S, STAGE = NPL * PLANE;
    constexpr int MI = BM / 32, KS = BK / 16;
    static_assert(PK_BN == 32 * NC && (BM == 64 || BM == 128), "32 columns per consumer");
    constexpr bool SCANS = (EPI == 7 || EPI == 8) && NPL == 2, ROW_SCANS = scans_rows(NPL, EPI), REVERSE = EPI == 8 || EPI == 10;
    constexpr int RC = SCANS ? BM / SCAN_WAVES : 8, FR = SCANS ? BM : 64;      // (scans)
    static_assert(!SCANS || BM >= 64, "scanning tiles have 64 or 128 rows");
    // k steps of the weights in flight: what 128 registers hold
    constexpr int PFB = (NPL == 3 && MI == 2) || MI == 4 ? 2 : 4;
    static_assert(MI <= 2 || NPL == 2, "128 rows of three planes do not fit the registers");
    __bf16 *stages = reinterpret_cast<__bf16 *>(smem_raw);
    int *rowexp = reinterpret_cast<int *>(stages + NS * STAGE);      // [BM] log2 of the scale of every row (two planes)

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63;
    const int nk = g.nkt;
    ScanSaved<RC> saved;
    ScanFlagBytes<FR> flag_bytes;
    ScanFlags<FR> flags;
    float2 lam;                                              // Abar of the lane's state
    StoreInputs<BM, PK_BN, EPI> in;
    if constexpr (SCANS) flag_bytes = scan_request_flags<FR, EPI == 8>(g, l, m0);
    RowScanStart row_scan;
    RowScanMasks<64> row_masks;
    RowScanSaved<64> row_saved;
    static_assert(!ROW_SCANS || BM == 64, "rows of the masks");
    if constexpr (ROW_SCANS) {
        row_scan = row_scan_start<64, PK_BN, false>(g, tid, m0, n0);
        row_masks = row_scan_ends<64>(g, tid, m0);
    }

    if (wave >= NC) {
        // ------------------------------------------------------------------ producers
        // a thread stages NV units of 1 row x 4 k per K tile; PF K tiles of loads in flight
        constexpr int NV = BM * BK / 4 / PT, PF = 2;
        static_assert(NV * PT * 4 == BM * BK, "tile must be a multiple of the producers' units");
        const int pt = tid - 64 * NC;
        const int kq = 4 * (pt % (BK / 4)), r0 = pt / (BK / 4);
        constexpr int RSTEP = PT / (BK / 4);
        static_assert(RSTEP % 16 == 0, "the swizzle of a thread's rows is one");
        // (a uniform base and a 32-bit offset per unit; rows past M: never stored)
        const PkUnits units(g.K, g.lda);
        const char *src = units.base(g.A + (long)m0 * g.lda, g.frag);
        unsigned row_at[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) row_at[i] = units.row(r0 + i * RSTEP, g.M - m0);
        float4 r[PF][NV];
        // Nothing is read past a row (see PkUnits); stash() puts the values of a unit that was read early into place.  No branch
        // around the loads: where paths with different numbers of loads in flight meet, the compiler waits
        // for the larger one, which cost a whole K tile of prefetch distance.
        auto fetch = [&](int set, int t) {
            const unsigned k = units.k(t, kq);
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const f32x4u v = *reinterpret_cast<const f32x4u *>(src + (row_at[i] + k));
                r[set][i] = make_float4(v.x, v.y, v.z, v.w);
            }
        };
        float sc[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i) sc[i] = 1.f;
        // Two planes: the 16 lanes that stage a row gather the words of its largest magnitude among them, and one of them
        // hands log2 of the scale to the consumers (which read it behind the K loop).
        unsigned rw[NV];
        if constexpr (NPL == 2) {
            // (the words of all rows together; a loop over further ones only where there are some)
            const auto words = [&](int j, auto take) {
                const unsigned *w = g.rows + m0 + (long)min(j, g.row_parts - 1) * g.row_stride;
#pragma unroll
                for (int i = 0; i < NV; ++i) take(i, w[min(r0 + i * RSTEP, g.M - 1 - m0)]);
            };
            words(kq / 4, [&](int i, unsigned v) { rw[i] = v; });
            for (int j = 16; j < g.row_parts; j += 16) words(j + kq / 4, [&](int i, unsigned v) { rw[i] = max(rw[i], v); });
        }
        const bool narrow = units.narrow;
#pragma unroll
        for (int j = 0; j < PF; ++j) fetch(j, j);
        if (narrow) {
#pragma unroll
            for (int i = 0; i < NV; ++i) r[0][i] = narrow_unit(g, m0 + min(r0 + i * RSTEP, g.M - 1 - m0), kq);
        }
        if constexpr (NPL == 2) {
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                unsigned v = rw[i];
                v = max(v, dpp_move<0xb1>(v));                        // quad_perm [1,0,3,2]
                v = max(v, dpp_move<0x4e>(v));                        // quad_perm [2,3,0,1]
                v = max(v, dpp_move<0x124>(v));                       // row_ror:4
                v = max(v, dpp_move<0x128>(v));                       // row_ror:8
                const int e = log2_scale_of(v);
                sc[i] = pow2f(e);
                if (kq == 0) rowexp[r0 + i * RSTEP] = e;
            }
        }
        const int ktail = (g.K % BK != 0 && !narrow) ? nk - 1 : nk;      // the K tile that hangs over
        auto stash = [&](int set, int t) {
            if (t == ktail) {
                const int sh = t * BK + kq - units.klast;              // > 0: the unit was read sh values early; >= 4: it lies past the row
#pragma unroll
                for (int i = 0; i < NV; ++i) r[set][i] = shift_unit(r[set][i], sh);
            }
            __bf16 *st = stages + (t % NS) * STAGE + r0 * S + 8 * pk_swizzle(r0, kq / 8) + kq % 8;      // (RSTEP rows on: the same)
#pragma unroll
            for (int i = 0; i < NV; ++i) {
                const Split4 sp = NPL == 3 ? split3(r[set][i]) : split2_f16_mix(r[set][i], sc[i]);
#pragma unroll
                for (int p = 0; p < NPL; ++p) *reinterpret_cast<bf16x4 *>(st + p * PLANE + i * RSTEP * S) = sp.p[p];
            }
        };
        static_assert(NS == 2, "the loop below");
        stash(0, 0);
        fetch(0, PF);
        __syncthreads();
        if constexpr (SCANS) flags = scan_flags<FR, EPI == 8>(g.scan, flag_bytes, m0);
        // step kt stages tile kt + 1 from register set (kt + 1) % PF while the consumers work on tile kt.  (Whole rounds, then what
        // is left: a loop with a second way out is rearranged so that its ways out meet the way round, where the compiler then waits
        // for loads that it could leave in flight.)
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
        if constexpr (SCANS) lam = g.scan.lam[min(n0 / 2 + l, g.scan.P - 1)];
        if constexpr (SCANS && EPI == 8 && MI < 4) saved = scan_request_saved<RC>(g.scan, wave, l, m0, n0);
        if constexpr (ROW_SCANS) row_saved = row_scan_request<64, PK_BN, REVERSE>(g, row_masks, tid, m0, n0);
        else if constexpr (!SCANS) in.request(g, tid, 0, m0, n0);
        __syncthreads();                             // barriers 1 and 2, see below
        __syncthreads();
    } else {
        // ------------------------------------------------------------------ consumers
        const int li = l & 31, hh = l >> 5;
        const bool work = n0 + wave * 32 < g.N;       // (a wavefront whose 32 columns lie past N only attends the barriers)
        v16f acc[MI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][r] = 0.f;
        const int nks = nk * KS;
        const uint4 *bp = g.frag + (size_t)(work ? n0 / 32 + wave : 0) * nks * (NPL * 64) + l;
        int frag_at[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) frag_at[ks] = li * S + 8 * pk_swizzle(li, 2 * ks + hh);
        uint4 fb[PFB][NPL];
        constexpr int MG = 2, NG = MI / MG;         // row fragments per step of the loop below, steps per k step
        bf16x8 fa[2][MG][NPL];
        auto load_weights = [&](int set, int s) {
#pragma unroll
            for (int p = 0; p < NPL; ++p) fb[set][p] = bp[(size_t)s * (NPL * 64) + p * 64];
        };
        auto load_rows = [&](int set, int kt, int ks, int ig) {
            const __bf16 *st = stages + (kt % NS) * STAGE + frag_at[ks];
#pragma unroll
            for (int i = 0; i < MG; ++i)
#pragma unroll
                for (int p = 0; p < NPL; ++p) fa[set][i][p] = *reinterpret_cast<const bf16x8 *>(st + p * PLANE + (ig * MG + i) * 32 * S);
        };
        // the products of one accumulator keep their order (smallest first): a3b1, a2b2, a1b3, a2b1, a1b2, a1b1 with
        // three planes, a2b1, a1b2, a1b1 with two
        auto multiply = [&](int sa, int sb, int ig) {
            constexpr int NPROD = NPL == 3 ? 6 : 3;
            constexpr int PA3[6] = {2, 1, 0, 1, 0, 0}, PB3[6] = {0, 1, 2, 0, 1, 0};
            constexpr int PA2[3] = {1, 0, 0}, PB2[3] = {0, 1, 0};
#pragma unroll
            for (int p = 0; p < NPROD; ++p)
#pragma unroll
                for (int i = 0; i < MG; ++i) {
                    v16f &c = acc[ig * MG + i];
                    if constexpr (NPL == 3)
                        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[sa][i][PA3[p]], __builtin_bit_cast(bf16x8, fb[sb][PB3[p]]), c, 0, 0, 0);
                    else
                        c = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fa[sa][i][PA2[p % 3]]),
                                                                   __builtin_bit_cast(f16x8, fb[sb][PB2[p % 3]]), c, 0, 0, 0);
                }
        };
        int eb = 0;                                   // log2 of the scale of this lane's weight row
        if (work) {
#pragma unroll
            for (int s = 0; s < PFB; ++s) load_weights(s, s);
            if constexpr (NPL == 2) eb = g.bexp[n0 + wave * 32 + li];
        }
        __syncthreads();
        if constexpr (SCANS) flags = scan_flags<FR, EPI == 8>(g.scan, flag_bytes, m0);
        if (work) {
            load_rows(0, 0, 0, 0);
            for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
                for (int st = 0; st < KS * NG; ++st) {
                    // the row fragments of the next step are requested before the matrix instructions of this one; at the
                    // last step of a K tile the workgroup barrier comes first: it releases the stage just read and
                    // guarantees that the next one is filled
                    const int ks = st / NG, ig = st % NG, set = ks % PFB, rs = st & 1;
                    if (st + 1 < KS * NG) load_rows(rs ^ 1, kt, (st + 1) / NG, (st + 1) % NG);
                    else {
                        __syncthreads();
                        load_rows(rs ^ 1, kt + 1, 0, 0);   // past the last tile: a harmless read of a stale stage
                    }
                    multiply(rs, set, ig);
                    if (ig == NG - 1) load_weights(set, min(kt + (ks + PFB) / KS, nk - 1) * KS + (ks + PFB) % KS);
                    // issue order: an LDS read in the shadow of each of the first matrix instructions, the loads of the
                    // weights behind the last
                    constexpr int NREAD = NPL * MG, NMFMA = (NPL == 3 ? 6 : 3) * MG;
#pragma unroll
                    for (int z = 0; z < NREAD; ++z) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    }
                    __builtin_amdgcn_sched_group_barrier(0x008, NMFMA - NREAD, 0);
                    if (ig == NG - 1) __builtin_amdgcn_sched_group_barrier(0x020, NPL, 0);
                }
            }
        } else {
            for (int kt = 0; kt < nk; ++kt) __syncthreads();
        }

        auto row_of = [&](int i, int r) { return i * 32 + 8 * (r / 4) + 4 * hh + (r % 4); };     // row inside the tile
        if constexpr (NPL == 2) {
            // the power of two that takes both operand scales off again (their sum can leave the exponent range of a
            // single factor: one exponent adjustment per element, exact like a multiplication by the power)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[i][r] = __builtin_ldexpf(acc[i][r], -(rowexp[row_of(i, r)] + eb));
        }
        if constexpr (SCANS) lam = g.scan.lam[min(n0 / 2 + l, g.scan.P - 1)];
        // (at 128 rows the accumulators leave no registers for the inputs before they are staged)
        if constexpr (SCANS && EPI == 8 && MI < 4) saved = scan_request_saved<RC>(g.scan, wave, l, m0, n0);
        if constexpr (ROW_SCANS) row_saved = row_scan_request<64, PK_BN, REVERSE>(g, row_masks, tid, m0, n0);
        else if constexpr (!SCANS && MI < 4) in.request(g, tid, 0, m0, n0);
        __syncthreads();                                 // barrier 1: every wavefront has left the K loop, LDS is free
        float *out = reinterpret_cast<float *>(smem_raw);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) out[tile_at(row_of(i, r), wave * 32 + li)] = acc[i][r];
        if constexpr (!SCANS && MI == 4) in.request(g, tid, 0, m0, n0);
        __syncthreads();                                 // barrier 2: the tile is staged
    }

    // (producers and consumers together: one copy of the code)
    if constexpr (SCANS) scan_epilogue_body<FR, EPI == 8, LEFT>(g, ScanLds(smem_raw, FR), wave, l, m0, n0, tile, saved, flags, lam);
    else if constexpr (ROW_SCANS) {
        row_scan_flags<64, REVERSE>(row_masks, row_scan, g.scan.is_first != nullptr);
        const RowScanPowers power = row_scan_powers<64, PK_BN, REVERSE>(row_scan.lam, tid);
        return row_scan_body<64, PK_BN, 1, REVERSE, EPI >= 9, LEFT>(g, reinterpret_cast<const float *>(smem_raw), reinterpret_cast<float2 *>(smem_raw + BM * PK_BN * 4), tid,
                                                               m0, n0, row_scan.lam, power, row_masks, row_saved, ahead);
    } else {
#pragma unroll
        for (int batch = 0; batch < in.BATCHES; ++batch) {
            if (batch > 0) in.request(g, tid, batch, m0, n0);
            in.store(g, reinterpret_cast<const float *>(smem_raw), tid, batch, m0, n0);
        }
    }
    return -1;
}

// Tiles of 32 rows: launches that leave a workgroup a CU to itself (beside reductions also two to a CU, on short stages: products3.hip), whose time is a chain of dependent steps rather than
// throughput.  All eight wavefronts load, split and multiply.  A stage is 256 k of all rows, double-buffered in LDS, with one meeting of the
// workgroup per stage; wavefronts that share 32 columns take every KW-th k step, and their partial tiles are added up as they are stored.
//   The two wavefronts of a SIMD do the same thing at the same time, so what is not interleaved in each of them does not overlap: the
// split of the next stage goes on in pieces of four instructions behind the matrix instructions, which wait for one another, and a unit's
// registers are requested again (two stages ahead) as soon as it is stored.  The workgroup meets before the last k step of a stage, whose fragments
// are in registers by then, so that the first fragments of the next stage come in its shadow.
// Bound by what the L2 hands a CU (64 columns of three planes: 512 bytes per k, 125 bytes per ns) and by the matrix cores at the
// clock that such a launch gets (1.7 - 1.9 GHz).  Launches, first start to last end, with four wavefronts that staged 64 k at a time for four that
// multiplied, and now: 1024 x 512 x 1024: 9.4 and 8.5 us; 256 x 512 x 1024: 8.2 and 6.1; 64 x 512 x 1024: 7.2 and 4.9.
//   A wait counts the requests made behind the one it is for.  So that the compiler finds the same order in every round of the loop, the
// first stage stands in front of it, the loop has a single way out, and there is no branch on lanes in it.
// AHEAD: k steps of the weights in flight: four; two beside a reduction, where wavefronts have 128 registers (short stages
// of at most 64 columns: four there too).  No variant spills.  With four on short stages of 128 columns, and the places of all eight
// steps of a stage kept, those beside a reduction spilled up to 14: forward and gradient pass of 32 x 60 tokens, H = 100, P = 200:
// 55.0 -> 51.4 us; 16 x 64, 128, 256: 42.0 -> 39.8; 16 x 64, 256, 256: 47.2 -> 46.8.
template <int BN, int NPL, int EPI, int KC, int AHEAD>
__device__ __forceinline__ int gemm_pk32_tile(const PkDev &g, unsigned char *smem_raw, int m0, int n0, int tid, bool ahead)
{
    constexpr int BM = 32, S = KC, PLANE = BM * S, STAGE = NPL * PLANE, KS = KC / 16;
    constexpr int CG = BN / 32, KW = PK32_WAVES / CG, KSW = KS / KW;         // column groups, wavefronts per group, k steps per wavefront and stage
    constexpr int PFB = KSW < AHEAD ? KSW : AHEAD;
    constexpr int RL = 32, NR = 2, NV = NR * (KC / 128);                     // lanes that share 128 k of a row, rows and units of a thread
    static_assert(PK_THREADS / RL * NR == BM && (KC == 128 || KC == 256) && KSW % PFB == 0, "units, register sets");
    __bf16 *stages = reinterpret_cast<__bf16 *>(smem_raw);
    int *rowexp = reinterpret_cast<int *>(stages + 2 * STAGE);               // [BM] log2 of the scale of every row (two planes)
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, li = l & 31, hh = l >> 5;
    const int cg = wave % CG, kw = wave / CG;
    const int nks = g.nkt * (PK_BK / 16), nst = (nks + KS - 1) / KS;         // k steps; stages
    // piece c (16 bytes) of row r: permuted so that sixteen lanes that read the same piece of sixteen rows meet every bank once
    auto place = [](int r, int c) { return r * S + 8 * (c ^ (r & 15)); };
    constexpr bool SCANS = EPI == 7 || EPI == 8;
    RowScanStart scan;
    RowScanMasks<BM> masks;
    RowScanSaved<BM> saved;
    RowScanPowers power;
    // (beside a reduction, whose wavefronts have 128 registers, the states before the last stage)
    constexpr bool EARLY = AHEAD == 4, TIGHT = !EARLY && BN == 128;
    if constexpr (SCANS) {
        scan = row_scan_start<BM, BN, TIGHT>(g, tid, m0, n0);
        masks = row_scan_ends<BM>(g, tid, m0);
        if constexpr (EARLY) saved = row_scan_request<BM, BN, EPI == 8>(g, masks, tid, m0, n0);
    }

    // ---- the rows (a unit that hangs over the end of its row reads the row's last four values, see PkUnits)
    const int kl = tid % RL, kq = 4 * kl, r0 = tid / RL;                     // units 0 and 1: rows r0 and r0 + 16; 2 and 3: 128 k on
    const PkUnits units(g.K, g.lda);
    const char *src = units.base(g.A + (long)m0 * g.lda, g.frag);
    unsigned row_at[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) row_at[i] = units.row(r0 + 16 * i, g.M - m0);
    float4 r[NV];
    auto k_of = [&](int i, int t) { return t * KC + 128 * (i / NR) + kq; };
    auto fetch = [&](int i, int t) {                                         // unit i of stage t
        const f32x4u v = *reinterpret_cast<const f32x4u *>(src + (row_at[i % NR] + units.k(0, k_of(i, t))));
        r[i] = make_float4(v.x, v.y, v.z, v.w);
    };
    const bool narrow = units.narrow;
#pragma unroll
    for (int i = 0; i < NV; ++i) fetch(i, 0);
    if (narrow) {
#pragma unroll
        for (int i = 0; i < NR; ++i) r[i] = narrow_unit(g, m0 + min(r0 + 16 * i, g.M - 1 - m0), kq);
    }
    unsigned rw[NR];
    if constexpr (NPL == 2) {
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const unsigned *w = g.rows + min(m0 + r0 + 16 * i, g.M - 1);
            rw[i] = w[(long)min(kl, g.row_parts - 1) * g.row_stride];
            for (int j = kl + RL; j < g.row_parts; j += RL) rw[i] = max(rw[i], w[(long)j * g.row_stride]);
        }
    }
    // ---- the weights: k step j of this wavefront is step kw + KW j of the product
    const bool work = n0 + cg * 32 < g.N;           // (a wavefront whose 32 columns lie past N multiplies the first ones and stores nothing)
    const uint4 *bp = g.frag + (size_t)(work ? n0 / 32 + cg : 0) * nks * (NPL * 64);       // (a uniform address per step, the lane as its offset)
    uint4 fb[PFB][NPL];
    auto load_weights = [&](int set, int j) {
        const uint4 *q = bp + (size_t)min(kw + KW * j, nks - 1) * (NPL * 64);
#pragma unroll
        for (int p = 0; p < NPL; ++p) fb[set][p] = q[p * 64 + l];
    };
    int eb = 0;                                     // log2 of the scale of this lane's weight row
    if constexpr (NPL == 2) { if (work) eb = g.bexp[n0 + cg * 32 + li]; }
#pragma unroll
    for (int j = 0; j < PFB; ++j) load_weights(j, j);

    float sc[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        sc[i] = 1.f;
        if constexpr (NPL == 2) {
            const int e = log2_scale_of(lane_xor_max<16>(row16_max(rw[i])));
            sc[i] = pow2f(e);
            if (kl == 0) rowexp[r0 + 16 * i] = e;
        }
    }
    const bool cut = g.K % KC != 0 && !narrow;
    // units of stage t that hang over: moved into place, zeros past the end of the row
    auto shift = [&](int t) {
#pragma unroll
        for (int i = 0; i < NV; ++i) r[i] = shift_unit(r[i], k_of(i, t) - units.klast);
    };
    // The split of a thread's units in pieces: three planes: an element (four instructions), or a unit's six packed words and their
    // stores; two planes: a unit.
    constexpr int PER_UNIT = NPL == 3 ? 5 : 1, PIECES = NV * PER_UNIT;
    unsigned h[4], m[4], lo[4];
    auto piece = [&](__bf16 *st, int k) {
        const int i = k / PER_UNIT, e = k % PER_UNIT;
        if (NPL == 3 && e < 4) {
            const float x = e == 0 ? r[i].x : e == 1 ? r[i].y : e == 2 ? r[i].z : r[i].w;
            split3_one(x, h[e], m[e], lo[e]);
        } else {
            const Split4 sp = NPL == 3 ? split3_pack(h, m, lo) : split2_f16_mix(r[i], sc[i % NR]);
            __bf16 *at = st + place(r0, kq / 8) + kq % 8 + 16 * (i % NR) * S + 128 * (i / NR);        // (16 rows or 128 k on: the same permutation)
#pragma unroll
            for (int p = 0; p < NPL; ++p) *reinterpret_cast<bf16x4 *>(at + p * PLANE) = sp.p[p];
        }
    };
    v16f acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    // Fragment of a k step of the stage in LDS: row li, k = 16 ks + 8 hh ..  Its piece is 2 (kw + KW j) + hh, and 2 kw + hh < 2 KW, a
    // power of two: step j's place is step 0's with bits of j flipped.  (Beside a reduction, where there are no registers to keep the
    // places of eight steps in, they are flipped at every step.)
    const int frag0 = place(li, 2 * kw + hh);
    int frag_at[KSW];
#pragma unroll
    for (int j = 0; j < KSW; ++j) frag_at[j] = frag0 ^ 16 * KW * j;
    bf16x8 fa[2][NPL];
    auto load_rows = [&](int set, const __bf16 *st, int j) {
        int at = frag_at[j];
        if constexpr (AHEAD == 2 && KSW == 8) asm volatile("v_xor_b32 %0, %1, %2" : "=v"(at) : "i"(16 * KW * j), "v"(frag0));
#pragma unroll
        for (int p = 0; p < NPL; ++p) fa[set][p] = *reinterpret_cast<const bf16x8 *>(st + p * PLANE + at);
    };
    // product q of a k step, smallest first (the order of gemm_pk_tile)
    constexpr int NPROD = NPL == 3 ? 6 : 3;
    auto multiply = [&](int sa, int sb, int q) {
        constexpr int PA3[6] = {2, 1, 0, 1, 0, 0}, PB3[6] = {0, 1, 2, 0, 1, 0};
        constexpr int PA2[3] = {1, 0, 0}, PB2[3] = {0, 1, 0};
        if constexpr (NPL == 3)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[sa][PA3[q]], __builtin_bit_cast(bf16x8, fb[sb][PB3[q]]), acc, 0, 0, 0);
        else
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, fa[sa][PA2[q % 3]]),
                                                         __builtin_bit_cast(f16x8, fb[sb][PB2[q % 3]]), acc, 0, 0, 0);
    };
    // pieces [k0, k1) of what goes to st, those behind matrix instruction n of m
    auto pieces_behind = [&](__bf16 *st, int k0, int k1, int n, int m, int refill) {
#pragma unroll
        for (int k = 0; k < PIECES; ++k)
            if (k >= k0 + (n * (k1 - k0) + m - 1) / m && k < k0 + ((n + 1) * (k1 - k0) + m - 1) / m) {
                piece(st, k);
                if (k % PER_UNIT == PER_UNIT - 1) fetch(k / PER_UNIT, refill);
            }
    };
    // Multiplies stage t from k step JB on, whose fragments are in registers, and puts stage t + 1 into the other half of LDS.
    auto stage = [&](int t, auto from) {
        constexpr int JB = decltype(from)::value, NM = (KSW - 1 - JB) * NPROD;     // matrix instructions in front of the meeting
        const __bf16 *cur = stages + (t & 1) * STAGE;
        __bf16 *next = stages + ((t & 1) ^ 1) * STAGE;
        if (cut && t + 2 == nst) shift(t + 1);
        if constexpr (NM == 0) pieces_behind(next, 0, PIECES, 0, 1, t + 2);
#pragma unroll
        for (int j = JB; j < KSW; ++j) {
            if (j + 1 < KSW) load_rows((j + 1) & 1, cur, j + 1);
            else {
                __syncthreads();
                load_rows(0, next, 0);
            }
#pragma unroll
            for (int q = 0; q < NPROD; ++q) {
                multiply(j & 1, j % PFB, q);
                if (j + 1 < KSW) pieces_behind(next, 0, PIECES, (j - JB) * NPROD + q, NM > 0 ? NM : 1, t + 2);
                __builtin_amdgcn_sched_barrier(0);
            }
            load_weights(j % PFB, t * KSW + j + PFB);
        }
    };
    // the last stage: no further one, and no k steps past the end
    auto last = [&](auto from) {
        constexpr int JB = decltype(from)::value;
        const __bf16 *cur = stages + ((nst - 1) & 1) * STAGE;
#pragma unroll
        for (int j = JB; j < KSW; ++j) {
            if (j + 1 < KSW) load_rows((j + 1) & 1, cur, j + 1);
            if ((nst - 1) * KS + KW * j + kw < nks) {
#pragma unroll
                for (int q = 0; q < NPROD; ++q) multiply(j & 1, j % PFB, q);
            }
            if (j + PFB < KSW) load_weights(j % PFB, (nst - 1) * KSW + j + PFB);
        }
    };
    // The first stage in halves, so that 128 k are multiplied while the other 128 are split (K is longer than 128 there); not beside a
    // reduction, where the further copies of the code take more registers than a wavefront has.
    constexpr bool HALVES = KC == 256 && AHEAD == 4;
    constexpr int HALF_STAGE = HALVES ? PIECES / 2 : PIECES;
    StoreInputs<BM, BN, EPI> in;
    auto request = [&] {
        if constexpr (SCANS) {
            row_scan_flags<BM, EPI == 8>(masks, scan, TIGHT || g.scan.is_first != nullptr);
            if constexpr (EARLY) power = row_scan_powers<BM, BN, EPI == 8>(scan.lam, tid);
            else saved = row_scan_request<BM, BN, EPI == 8>(g, masks, tid, m0, n0);
        } else in.request(g, tid, 0, m0, n0);
    };
    if (cut && nst == 1) shift(0);
#pragma unroll
    for (int k = 0; k < HALF_STAGE; ++k) pieces_behind(stages, k, k + 1, 0, 1, 1);
    __syncthreads();
    load_rows(0, stages, 0);
    if constexpr (!HALVES) {
        if constexpr (KSW % 2 == 0) {                     // (a single k step per wavefront and stage: only where one stage is all)
            if (nst > 1) stage(0, std::integral_constant<int, 0>{});
            for (int t = 1; t + 1 < nst; ++t) stage(t, std::integral_constant<int, 0>{});
        }
        request();
        last(std::integral_constant<int, 0>{});
    } else {
        constexpr int JB = KSW / 2;
#pragma unroll
        for (int j = 0; j < JB; ++j) {
            if (j + 1 < JB) load_rows((j + 1) & 1, stages, j + 1);
#pragma unroll
            for (int q = 0; q < NPROD; ++q) {
                multiply(j & 1, j % PFB, q);
                pieces_behind(stages, HALF_STAGE, PIECES, j * NPROD + q, JB * NPROD, 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            load_weights(j % PFB, j + PFB);
        }
        __syncthreads();
        load_rows(JB & 1, stages, JB);
        if (nst == 1) {
            request();
            last(std::integral_constant<int, JB>{});
        } else {
            stage(0, std::integral_constant<int, JB>{});
            for (int t = 1; t + 1 < nst; ++t) stage(t, std::integral_constant<int, 0>{});
            request();
            last(std::integral_constant<int, 0>{});
        }
    }
    if constexpr (NPL == 2) {
        // (see gemm_pk_tile)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[e] = __builtin_ldexpf(acc[e], -(rowexp[8 * (e / 4) + 4 * hh + (e % 4)] + eb));
    }
    constexpr bool HALF = PK32_WAVES * 1024 * 4 <= STAGE * 2;                    // the parts fit the half of the stages that nobody reads any more
    static_assert(HALF || PK32_WAVES * 1024 * 4 <= 2 * STAGE * 2, "or all of them");
    if constexpr (!HALF) __syncthreads();
    float *out = reinterpret_cast<float *>(stages + (HALF ? (nst & 1) * STAGE : 0));
#pragma unroll
    for (int e = 0; e < 16; ++e) out[kw * BM * BN + tile_at<BN>(8 * (e / 4) + 4 * hh + (e % 4), cg * 32 + li)] = acc[e];
    __syncthreads();
    if constexpr (SCANS) {
        constexpr int FREE = (HALF ? STAGE : 2 * STAGE) * 2 - PK32_WAVES * 1024 * 4;        // bytes of LDS behind the parts
        static_assert(FREE >= (int)row_scan_lds_bytes(BN), "what the scan keeps there");
        if constexpr (!EARLY) power = row_scan_powers<BM, BN, EPI == 8>(scan.lam, tid);
        return row_scan_body<BM, BN, KW, EPI == 8>(g, out, reinterpret_cast<float2 *>(out + PK32_WAVES * 1024), tid, m0, n0, scan.lam, power, masks, saved, ahead);
    } else {
        static_assert(in.BATCHES == 1, "a unit or two per thread");
        in.store(g, out, tid, 0, m0, n0);
    }
    return -1;
}

// Tile of the workgroup in slot q of XCD x (workgroup ids are dealt round-robin to the 8 XCDs, each with its own L2):
//   mode 0: XCD x owns the contiguous band of tiles [x nx, (x+1) nx), so it reads its band of A and the weights once
//           into its own L2;
//   mode 5 (scan epilogues): a unit = the tiles of one sequence and one group of column tiles, time-major; units are dealt
//           to the XCDs, so a tile only ever waits for tiles in earlier slots of its own XCD, which were dispatched
//           before it;
//   modes 6 and 7 (scans of rows): row tiles in the order of the scan, so that predecessors have smaller workgroup ids.  6: the
//           column tiles of a row tile go to different XCDs, so that few row tiles occupy all of them; 7: to one, which then reads the rows once (the
//           row tile before it belongs to the XCD before that, or to the last one in an earlier round of slots).
__device__ __forceinline__ int pk_place(const PkDev &g, int x, int q)
{
    if (g.mode == 0) return x * g.nx + q;
    if (g.mode == 6 || g.mode == 7) {
        const int n = 8 * q + x;
        const int m = g.mode == 6 ? n : q, d = (int)g.by_ntn(m), tn = m - d * g.ntn, r = g.mode == 6 ? d : 8 * d + x;       // row tile in scan order
        return r < g.ntm ? (g.sc_rev ? g.ntm - 1 - r : r) * g.ntn + tn : g.ntm * g.ntn;
    }
    const int per_unit = g.sc_nt * g.sc_cpu;
    const int u = (int)g.by_unit(q), uid = x + 8 * u, r = q - u * per_unit;
    const int b = (int)g.by_ncg(uid), cg = uid - b * g.sc_ncg;
    const int tslot = (int)g.by_cpu(r), tn = cg * g.sc_cpu + r - tslot * g.sc_cpu;      // time-ordered slot; the reverse scan starts at the sequence end
    const int tmL = g.sc_rev ? g.sc_nt - 1 - tslot : tslot;
    return (uid < g.sc_units && tn < g.ntn) ? (b * g.sc_nt + tmL) * g.ntn + tn : g.ntm * g.ntn;
}

// kc: k per stage
constexpr size_t pk_lds_bytes(int BM, int BN, int NPL, int epi, int kc)
{
    const bool scans = (epi == 7 || epi == 8) && NPL == 2, row_scans = BM == 64 && (epi >= 7) && !scans;
    const size_t st = (size_t)PK_STAGES * NPL * BM * kc * 2 + (size_t)BM * 4;          // stages and scales
    const size_t tile = (size_t)BM * BN * 4 * (BM == 32 ? PK32_WAVES * 32 / BN : 1);           // the staged tile (or its parts)
    const size_t ep = scans ? scan_lds_bytes(BM) : row_scans ? tile + row_scan_lds_bytes(BN) : tile;
    return ep > st ? ep : st;
}

// One launch carries a product with packed weights and up to two K = T reductions (TNB > 0: their tile is
// that of this name; absent ones have no slots).  Every problem owns a contiguous range of the slots of every XCD.
// (a reduction may have more wavefronts than a product; the surplus leaves a product's workgroup at once)
constexpr int pk_threads(int TNB) { return TNB > 0 ? 128 * tn_wavefronts(TNB) : PK_THREADS; }
constexpr int pk_tn_bk(int TNB, int WPE) { return TNB == 65 || WPE == 2 ? 2 * TN_BK : TN_BK; }

// A pointer that was read as a word: to global memory.  (The compiler knows that of the kernel's arguments themselves.  A load from an address that it does not
// know it of counts against LDS as well as memory, and every wait for one is a wait for all.)
template <class T> __device__ __forceinline__ void in_global(T *&p)
{
    auto q = (T __attribute__((address_space(1))) *)p;
    asm("" : "+s"(q));
    p = (T *)q;
}
__device__ __forceinline__ void in_global(PkDev &g)
{
    in_global(g.A); in_global(g.frag); in_global(g.bexp); in_global(g.C); in_global(g.rows);
    ScanEpilogue &a = g.scan;
    in_global(a.lam); in_global(a.is_first); in_global(a.x0); in_global(a.x_last); in_global(a.xsaved); in_global(a.partial);
    in_global(a.dx0); in_global(a.desc); in_global(a.err); in_global(a.rowmax_out); in_global(a.amax_out);
}

__device__ __forceinline__ void in_global(GemmDev &g)
{
    in_global(g.A); in_global(g.B); in_global(g.C); in_global(g.amaxA.slots); in_global(g.amaxB.slots);
}

template <int BM, int BN, int NPL, int EPI, int TNB, int WPE, bool LEFT>
__global__ void __launch_bounds__(pk_threads(TNB), WPE) gemm_pk_kernel(PkDev g, GemmDev t0, GemmDev t1)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    const int x = blockIdx.x % 8, q = blockIdx.x / 8, tid = threadIdx.x;
    if (TNB == 0 || (q >= g.slot0 && q < g.slot0 + g.nx)) {
        // (what the way to the first loads needs is requested together: left to where they are used, the arguments come in four or five trips)
        // (a scan beside a reduction has no registers to keep them in)
        if constexpr (EPI < 7 || TNB == 0)
            asm volatile("" ::"s"(g.A), "s"(g.lda), "s"(g.frag), "s"(g.bexp), "s"(g.rows), "s"(g.row_parts), "s"(g.row_stride), "s"(g.M), "s"(g.N), "s"(g.K), "s"(g.nkt),
                         "s"(g.ntm), "s"(g.ntn), "s"(g.nx), "s"(g.mode), "s"(g.slot0), "s"(g.by_ntn.mul), "s"(g.by_ntn.shift));
        if constexpr (EPI >= 7 && TNB == 0)
            asm volatile("" ::"s"(g.scan.is_first), "s"(g.scan.lam), "s"(g.scan.L), "s"(g.scan.P), "s"(g.scan.by_L.mul), "s"(g.scan.by_L.shift), "s"(g.sc_rev), "s"(g.sc_nt),
                         "s"(g.sc_cpu), "s"(g.sc_ncg), "s"(g.sc_units), "s"(g.by_unit.mul), "s"(g.by_unit.shift), "s"(g.by_ncg.mul), "s"(g.by_ncg.shift),
                         "s"(g.by_cpu.mul), "s"(g.by_cpu.shift));
        // (only scans are placed otherwise than in mode 0: left to run time, every product has the code of all modes on its way to the first loads)
        const int tile = EPI < 7 ? x * g.nx + q - g.slot0 : pk_place(g, x, q - g.slot0);
        if (tile >= g.ntm * g.ntn || tid >= PK_THREADS) return;
        const int tm = (int)g.by_ntn(tile), tn = tile - tm * g.ntn;
        auto run = [&](const PkDev &g, int tm, int tid, bool ahead) {
            if constexpr (BM == 32 && BN == 64 && WPE == 4 && TNB == 0) return gemm_pk32_tile<BN, NPL, EPI, PK32_SHORT, 4>(g, smem_raw, tm * BM, tn * BN, tid, ahead);
            else if constexpr (BM == 32) {
                // (two to a CU beside reductions: long stages only where 32 columns have a single k step per wavefront and short stage; beside items of sixteen wavefronts, whose
                // launches leave a workgroup a CU too, long ones with the registers of two)
                constexpr bool ALONE = TNB == 0 || WPE == 2, LONG = ALONE || TNB == 65 || BN == 32;
                if (!LONG || g.K <= PK32_SHORT) return gemm_pk32_tile<BN, NPL, EPI, PK32_SHORT, ALONE || BN < 128 ? 4 : 2>(g, smem_raw, tm * BM, tn * BN, tid, ahead);
                if constexpr (LONG) return gemm_pk32_tile<BN, NPL, EPI, PK32_LONG, ALONE ? 4 : 2>(g, smem_raw, tm * BM, tn * BN, tid, ahead);
            } else return gemm_pk_tile<BM, NPL, EPI, LEFT>(g, smem_raw, tm * BM, tn * BN, tile, tid, ahead);
        };
        const int missing = __builtin_amdgcn_readfirstlane(run(g, tm, tid, false));
        if constexpr (scans_rows(NPL, EPI)) {
            if (__builtin_expect(missing >= 0, 0)) {
                // The aggregate of row tile `missing`, then this tile again, until none is missing.  (At most two rounds per tile of the
                // sequence; the bound on them only keeps a mistake from hanging.)  A copy of the code for itself: in a loop nothing may stay
                // in registers from one round to the next, the arguments included, which every tile would pay for (16 layers: 0.2 %).
                auto args = (const unsigned long long __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr();
                for (int m = missing, rounds = 0;; ++rounds) {
                    __syncthreads();                         // LDS is free
                    int id = tid;
                    asm volatile("" : "+v"(id), "+s"(m), "+s"(args));
                    static_assert(sizeof(PkDev) % 8 == 0, "whole words, the first of the arguments");
                    union { unsigned long long w[sizeof(PkDev) / 8]; PkDev g; } own;
#pragma unroll
                    for (size_t i = 0; i < sizeof(PkDev) / 8; ++i) own.w[i] = args[i];
                    in_global(own.g);
                    const int next = __builtin_amdgcn_readfirstlane(run(own.g, m, id, m != tm));
                    if (next < 0 && m == tm) break;
                    if (rounds > 4 * ROW_SCAN_MAX_TILES) { atomicOr(own.g.scan.err, 1u); break; }
                    m = next < 0 ? tm : next;
                }
            }
        }
    } else if constexpr (TNB > 0) {
        // (one copy of the code for both, whose arguments are read as words: with a copy each, whose loops do not fit the instruction cache together,
        // and choosing between the two structs would put them on the stack)
        const bool second = q < t0.slot0 || q >= t0.slot0 + t0.nx;
        static_assert(sizeof(PkDev) % 8 == 0 && sizeof(GemmDev) % 8 == 0, "whole words, one behind the other");
        auto args = (const unsigned long long __attribute__((address_space(4))) *)__builtin_amdgcn_kernarg_segment_ptr() + (sizeof(PkDev) + (second ? sizeof(GemmDev) : 0)) / 8;
        union { unsigned long long w[sizeof(GemmDev) / 8]; GemmDev t; } own;
#pragma unroll
        for (size_t i = 0; i < sizeof(GemmDev) / 8; ++i) own.w[i] = args[i];
        in_global(own.t);
        gemm_tn_problem<TNB, NPL, pk_tn_bk(TNB, WPE)>(own.t, smem_raw, x, q - own.t.slot0, tid);
    }
}

template <int BM, int BN>
inline PkDev make_pk_dev(const GemmArgs &a)
{
    PkDev g{};
    g.A = a.A; g.lda = a.lda; g.frag = static_cast<const uint4 *>(a.w.frag); g.bexp = a.w.exp; g.C = a.C; g.ldc = a.ldc;
    g.diag = a.diag; g.E = a.E; g.lde = a.lde; g.E2 = a.E2; g.C2 = a.C2; g.rowflag = a.rowflag;
    g.M = a.M; g.N = a.N; g.K = a.K; g.nkt = (a.K + PK_BK - 1) / PK_BK;
    g.ntm = (a.M + BM - 1) / BM; g.ntn = (a.N + BN - 1) / BN;
    const long ntiles = (long)g.ntm * g.ntn;
    g.nx = (int)((ntiles + 7) / 8); g.mode = 0; g.slot0 = 0;
    g.by_ntn = FastDiv::by(g.ntn);
    g.scan = a.scan;
    if (a.scan.L > 0) g.scan.by_L = FastDiv::by(a.scan.L);
    g.rows = a.amaxA.rows; g.row_parts = a.amaxA.row_parts; g.row_stride = a.amaxA.row_stride;
    g.c2_rowmax = a.c2_rowmax;
    const auto address = [](const void *p) { return reinterpret_cast<uintptr_t>(p); };
    g.through = a.epilogue >= 7 ? states_through(address(a.C), a.M, a.scan.P) : output_through(address(a.C), address(a.C2), a.M, 4 * a.ldc);
    if (scans_rows(a.planes, a.epilogue)) {
        g.sc_rev = a.epilogue == 8 || a.epilogue == 10;
        // (mode 7 from 64 row tiles on, where the XCDs get as many within 1/8: 14 shapes of 3000 .. 30000 tokens, gradient pass: 1.6 % faster on geometric
        // mean, 16 x 1000, 256, 256: 201.4 -> 194.9 us, 20 x 300, 500, 250: 171.2 -> 169.1, none slower by more than runs of one side differ)
        g.mode = BM == 64 && g.ntm >= 64 ? 7 : 6;
        if (g.mode == 7) g.nx = (g.ntm + 7) / 8 * g.ntn;
    } else if ((a.epilogue == 7 || a.epilogue == 8) && a.scan.L >= BM) {
        g.sc_rev = a.epilogue == 8;
        const int nseq = a.M / a.scan.L;
        g.sc_nt = a.scan.L / BM;
        int ncg = nseq >= 8 ? 1 : (8 + nseq - 1) / nseq;
        if (ncg > g.ntn) ncg = g.ntn;
        g.sc_ncg = ncg;
        g.sc_cpu = (g.ntn + ncg - 1) / ncg;
        g.sc_units = nseq * ncg;
        g.mode = 5;
        g.nx = ((g.sc_units + 7) / 8) * g.sc_nt * g.sc_cpu;
        g.by_unit = FastDiv::by(g.sc_nt * g.sc_cpu); g.by_ncg = FastDiv::by(g.sc_ncg); g.by_cpu = FastDiv::by(g.sc_cpu);
    }
    return g;
}

// t0, t1: the reductions of the launch (null: none; t1 only with t0); tn_first: their work items take the first slots.
template <int BM, int BN, int NPL, int EPI, int TNB, int WPE>
hipError_t launch_pk_variant(const GemmArgs &a, const GemmArgs *b, const GemmArgs *c, bool tn_first, hipStream_t s)
{
    if ((TNB > 0) != (b != nullptr) || (c && !b)) return hipErrorInvalidValue;
    PkDev g = make_pk_dev<BM, BN>(a);
    GemmDev t[2]{};
    long slots = 0;
    if (!tn_first) { g.slot0 = 0; slots = g.nx; }
    if constexpr (TNB > 0) {
        const GemmArgs *tn[2] = {b, c};
        for (int i = 0; i < 2; ++i) {
            if (tn[i]) t[i] = make_tn_dev<TNB>(*tn[i]);
            t[i].slot0 = (int)slots;
            slots += t[i].nx;
        }
    }
    if (tn_first) { g.slot0 = (int)slots; slots += g.nx; }
    constexpr size_t tnl = TNB > 0 ? tn_lds_bytes(TNB, NPL, pk_tn_bk(TNB, WPE)) : 0;
    constexpr size_t pk = pk_lds_bytes(BM, BN, NPL, EPI, BM == 32 ? PK32_LONG : PK_BK);
    constexpr size_t pk_short = BM == 32 ? pk_lds_bytes(BM, BN, NPL, EPI, PK32_SHORT) : pk;
    constexpr size_t most = pk > tnl ? pk : tnl;
    const size_t smem = BM == 32 && ((BN >= 64 && WPE == 4 && TNB != 65) || a.K <= PK32_SHORT) ? (pk_short > tnl ? pk_short : tnl) : most;
    if (slots <= 0 || slots > 0x7fffffffL / 8) return hipErrorInvalidValue;
    const auto launch = [&](auto left) -> hipError_t {
        auto kern = gemm_pk_kernel<BM, BN, NPL, EPI, TNB, WPE, decltype(left)::value>;
        static std::atomic<bool> raised[KERNEL_MAXDEV];
        const hipError_t e = raise_lds_limit(reinterpret_cast<const void *>(kern), most, raised);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kern, dim3((unsigned)(8 * slots)), dim3(pk_threads(TNB)), smem, s, g, t[0], t[1]);
        return hipGetLastError();
    };
    // (scans on smaller tiles: launches of at most 4 MiB of states on 32 rows, 32 MiB in the chains of 64)
    if constexpr (EPI >= 7 && (BM == 128 || (BM == 64 && scans_rows(NPL, EPI))))
        if (!g.through) return launch(std::true_type{});
    return launch(std::false_type{});
}

}  // namespace ssm
