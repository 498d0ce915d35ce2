// The forward pass of narrow layers (at most 64 columns and 64 states) over short sequences (at most 64 steps) in one launch.
//
// A workgroup takes as many whole sequences as 64 tokens hold, so nothing passes between workgroups: no words to clear, no packed weights, no
// launch in front of or behind another.  Everything it reads is requested at once, in whole lines, split once into three bf16 planes and kept in LDS:
// input projection (32 x 32 blocks of u Bbar^T, a wavefront each), the resettable scan (eight threads per state, eight tokens each), output
// projection (K = 2P in two halves), D (.) u.
//   Such a layer is bound by latency: as prep, input projection with its scan and output projection it was three launches of 3.5 to 6.6 us, each a
// trip to memory and back, and the host took as long to submit them (2.4 us each) as they took to run.  Time per C call, one behind the other: 2 x 64 tokens, H = P = 32: 13.1 -> 5.6 us
// (by the clock inside: arguments and requests 0.6, discretisation 0.7 while the values come, planes 0.6, products 0.4 and 0.6, scan 1.5, stores 0.4 and the start
// and end of a launch); 16 x 64, 64, 64: 13.0 -> 8.0; 128 x 33, 64, 64: 14.5 -> 8.1; 1500 x 7, 64, 64: 17.7 -> 8.8; 500 x 60, 64, 64: 29.3 -> 16.6.  With every operand
// requested by the lanes of its fragment instead of in whole lines the first two took 6.6 and 12.5.  Errors against 64 bits: 0.87 to 1.03 of what they were.
#include "pack.h"

namespace ssm {

namespace {
constexpr int NF_ROWS = 64, NF_THREADS = 512, NF_RUNS = 8, NF_RUN = NF_ROWS / NF_RUNS;

// place of an element of a tile of BN columns: pieces of 32 (rows, at 32 columns) swapped in rows 4 .. 7 of every eight, which a wavefront stores together with
// rows 0 .. 3
template <int BN> __device__ __forceinline__ int nf_at(int row, int col)
{
    return BN == 32 ? (row ^ ((row >> 2) & 1)) * BN + col : row * BN + (col ^ ((row & 4) << 3));
}

// Four values of a row of n >= 4 that starts at `row`, from k on, its last four past its end: all requests of a workgroup without a branch, so that they are in
// flight together.
__device__ __forceinline__ float4 request(const float *base, unsigned row, int k, int n)
{
    const f32x4u v = *reinterpret_cast<const f32x4u *>(reinterpret_cast<const char *>(base) + 4 * (row + (unsigned)min(k, n - 4)));
    return make_float4(v.x, v.y, v.z, v.w);
}
// what was requested, moved into place: zeros past the end
__device__ __forceinline__ void into_place(float4 &v, int k, int n) { v = shift_unit(v, k - min(k, n - 4)); }
// (or the compiler moves a request into the branch of its first use, where it is waited for before the next)
__device__ __forceinline__ void hold(float4 &v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }

// An operand in LDS: three planes of ROWS x K 16-bit values, the 16-byte pieces of a row permuted so that the rows of a fragment meet different banks.
template <int ROWS, int K>
struct PlanesLds {
    __bf16 *p;
    __device__ __forceinline__ __bf16 *at(int row, int k) const { return p + row * K + 8 * ((k / 8) ^ ((row / (128 / K > 0 ? 128 / K : 1)) & (K / 8 - 1))) + k % 8; }
    __device__ __forceinline__ void put(int row, int k, float4 v) const
    {
        const Split4 s = split3(v);
#pragma unroll
        for (int q = 0; q < 3; ++q) *reinterpret_cast<bf16x4 *>(at(row, k) + q * ROWS * K) = s.p[q];
    }
    __device__ __forceinline__ void put(int row, int k, float2 v) const
    {
        unsigned h[2], m[2], l[2];
        split3_one(v.x, h[0], m[0], l[0]); split3_one(v.y, h[1], m[1], l[1]);
        unsigned *o = reinterpret_cast<unsigned *>(at(row, k));
        o[0] = __builtin_amdgcn_perm(h[1], h[0], 0x07060302u);
        o[ROWS * K / 2] = __builtin_amdgcn_perm(m[1], m[0], 0x07060302u);
        o[ROWS * K] = __builtin_amdgcn_perm(l[1], l[0], 0x07060302u);
    }
    __device__ __forceinline__ bf16x8 get(int row, int k, int q) const { return *reinterpret_cast<const bf16x8 *>(at(row, k) + q * ROWS * K); }
};

// The product of a lane's rows over N steps of K from k on: the six products of the planes, smallest first, each over all steps (step by step the small
// products of the later steps would be added to the large ones of the earlier: up to 1.15 times the error).
template <int N, class A, class B>
__device__ __forceinline__ v16f multiply(const A &a, int arow, const B &b, int brow, int k)
{
    constexpr int PA[6] = {2, 1, 0, 1, 0, 0}, PB[6] = {0, 1, 2, 0, 1, 0};
    bf16x8 fa[N][3], fb[N][3];
#pragma unroll
    for (int s = 0; s < N; ++s)
#pragma unroll
        for (int q = 2; q >= 0; --q) { fa[s][q] = a.get(arow, k + 16 * s, q); fb[s][2 - q] = b.get(brow, k + 16 * s, 2 - q); }
    v16f c;
#pragma unroll
    for (int i = 0; i < 16; ++i) c[i] = 0.f;
#pragma unroll
    for (int q = 0; q < 6; ++q)
#pragma unroll
        for (int s = 0; s < N; ++s) c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[s][PA[q]], fb[s][PB[q]], c, 0, 0, 0);
    return c;
}
}  // namespace

// KH: steps of 16 columns (2: up to 32, 4: up to 64); KP: the same of states
template <int KH, int KP>
__global__ void __launch_bounds__(NF_THREADS, 2) narrow_fwd_kernel(NarrowFwd a)
{
    constexpr int HC = 16 * KH, PC = 16 * KP, UW = HC / 4;   // columns and states that the tiles hold, units of a row of u
    constexpr int NU = NF_ROWS * UW / NF_THREADS, NB = PC * UW / NF_THREADS > 0 ? PC * UW / NF_THREADS : 1, NC = HC * PC / 2 / NF_THREADS;    // units of a thread
    __shared__ __attribute__((aligned(16))) __bf16 us[3 * NF_ROWS * HC], cs[3 * HC * 2 * PC], bx[3 * 2 * PC * (HC > NF_ROWS ? HC : NF_ROWS)];
    __shared__ __attribute__((aligned(16))) float vt[NF_ROWS * (PC > HC ? 2 * PC : 2 * HC)];
    __shared__ float2 runs[NF_RUNS * PC], g_of[PC];
    __shared__ float4 lam_of[PC];                            // Abar and Abar^8
    static_assert(sizeof(vt) >= pack_lds_bytes(NF_THREADS), "the packing job");
    // (all arguments that the requests need come in one trip)
    asm volatile("" ::"s"(a.Lambda), "s"(a.B), "s"(a.C), "s"(a.D), "s"(a.log_delta), "s"(a.u), "s"(a.is_first), "s"(a.x0), "s"(a.Bt), "s"(a.L), "s"(a.H), "s"(a.P), "s"(a.seqs),
                 "s"(a.layer_blocks), "s"(a.by_L.mul), "s"(a.by_L.shift));
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l = tid & 63, li = l & 31, hh = l >> 5;
    if ((int)blockIdx.x >= a.layer_blocks) {
        const PackSrc src{nullptr, nullptr, nullptr, nullptr, a.W, a.P, a.H, nullptr};
        pack_block<PACK_WN, 3, NF_THREADS>(src, a.pack, blockIdx.x - a.layer_blocks, reinterpret_cast<unsigned char *>(vt));
        return;
    }
    const PlanesLds<NF_ROWS, HC> U{us};
    const PlanesLds<2 * PC, HC> Bb{bx};
    const PlanesLds<HC, 2 * PC> Cp{cs};
    const PlanesLds<NF_ROWS, 2 * PC> X{bx};                  // (in the place of Bbar, which nobody reads any more)
    float *pt = vt;                                          // the halves of y, in the place of the elements of the scan
    const int H = a.H, P = a.P, L = a.L;
    const int seq0 = blockIdx.x * a.seqs, rows = min(a.seqs, a.Bt - seq0) * L;       // its first sequence, its tokens
    const long m0 = (long)seq0 * L;

    // ---- requests
    const bool cut_h = H != HC, cut_p = P != PC;             // rows that end before the steps of K do
    const int col = 4 * (tid % UW), row0 = tid / UW;         // units of u, of Bbar (four complex columns of a state) and of y
    constexpr int RSTEP = NF_THREADS / UW;
    const int ccol = 4 * (tid % (PC / 2)), crow = tid / (PC / 2);        // units of C
    constexpr int CSTEP = NF_THREADS / (PC / 2);
    const float *u0 = a.u + m0 * H;                          // (uniform; 32-bit offsets from there)
    const int p_own = min(l, P - 1);
    const float2 Lambda = a.Lambda[p_own];
    const float log_delta = a.log_delta[p_own];
    float4 u[NU], b[NB][2], w[NC];
#pragma unroll
    for (int j = 0; j < NU; ++j) u[j] = request(u0, min(row0 + j * RSTEP, rows - 1) * H, col, H);
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < 2; ++i) b[j][i] = request(reinterpret_cast<const float *>(a.B), 2 * min(row0 + j * RSTEP, P - 1) * H, 2 * col + 4 * i, 2 * H);
#pragma unroll
    for (int j = 0; j < NC; ++j) w[j] = request(reinterpret_cast<const float *>(a.C), 2 * min(crow + j * CSTEP, H - 1) * P, ccol, 2 * P);
    float4 d = request(a.D, 0, col, H);
    // the flags, and where sequences start and end (lane l: row l)
    const int r = min(l, rows - 1), seq = (int)a.by_L(r), step = r - seq * L;
    const unsigned flag = (a.is_first ? a.is_first + m0 : reinterpret_cast<const uint8_t *>(a.u))[r];       // (without flags: any byte, not used)
    const unsigned long long start = __ballot(step == 0 && l < rows), end = __ballot(step == L - 1 && l < rows);
    auto sequence = [&](int row) { return seq0 + __popcll(start & ((2ull << row) - 2ull)); };
    const int c = l, q = wave, r0 = NF_RUN * q;              // of the scan: state, run, its first row
    const bool active = c < P;
    float2 x0[NF_RUN];
#pragma unroll
    for (int i = 0; i < NF_RUN; ++i) x0[i] = make_float2(0.f, 0.f);
    if (a.x0 && (start >> r0 & 0xffu) != 0) {
#pragma unroll
        for (int i = 0; i < NF_RUN; ++i)
            if (start >> (r0 + i) & 1u) x0[i] = (a.x0 + (long)sequence(r0 + i) * P)[min(c, P - 1)];
    }

    // ---- the operands in planes; the discretisation by the first wavefront
    if (wave == 0) {
        const float4 z = zoh_rounded<3>(Lambda, log_delta);
        double pr = z.x, pi = z.y;                           // Abar^8 in double precision, rounded once
#pragma unroll
        for (int i = 0; i < 3; ++i) { const double re = pr * pr - pi * pi; pi *= 2.0 * pr; pr = re; }
        static_assert(NF_RUN == 8, "three squarings");
        if (l < PC) { lam_of[l] = make_float4(z.x, z.y, (float)pr, (float)pi); g_of[l] = make_float2(z.z, z.w); }
    }
#pragma unroll
    for (int j = 0; j < NU; ++j) hold(u[j]);
#pragma unroll
    for (int j = 0; j < NB; ++j) { hold(b[j][0]); hold(b[j][1]); }
#pragma unroll
    for (int j = 0; j < NC; ++j) hold(w[j]);
    hold(d);
    if (cut_h) {
#pragma unroll
        for (int j = 0; j < NU; ++j) into_place(u[j], col, H);
#pragma unroll
        for (int j = 0; j < NB; ++j) { into_place(b[j][0], 2 * col, 2 * H); into_place(b[j][1], 2 * col + 4, 2 * H); }
        into_place(d, col, H);
    }
    if (cut_p) {
#pragma unroll
        for (int j = 0; j < NC; ++j) into_place(w[j], ccol, 2 * P);
    }
#pragma unroll
    for (int j = 0; j < NU; ++j) U.put(row0 + j * RSTEP, col, u[j]);
#pragma unroll
    for (int j = 0; j < NC; ++j) Cp.put(crow + j * CSTEP, ccol, make_float4(w[j].x, -w[j].y, w[j].z, -w[j].w));
    __syncthreads();                                         // g is in LDS
#pragma unroll
    for (int j = 0; j < NB; ++j) {
        const int p = row0 + j * RSTEP;
        if (p >= PC) continue;                               // (whole wavefronts)
        const float2 g = g_of[p];
        const float4 s = b[j][0], t = b[j][1];
        Bb.put(2 * p, col, make_float4(g.x * s.x - g.y * s.y, g.x * s.z - g.y * s.w, g.x * t.x - g.y * t.y, g.x * t.z - g.y * t.w));
        Bb.put(2 * p + 1, col, make_float4(g.x * s.y + g.y * s.x, g.x * s.w + g.y * s.z, g.x * t.y + g.y * t.x, g.x * t.w + g.y * t.z));
    }
    const unsigned long long first = a.is_first ? __ballot(flag != 0 && l < rows) : 0ull, cut = first | start;
    __syncthreads();                                         // the operands are in LDS
    // ---- input projection: a block of 32 rows and 32 columns per wavefront
    const int rb = 32 * (wave & 1);
    if (wave >> 1 < PC / 16) {
        const int n = 32 * (wave >> 1) + li;
        const v16f acc = multiply<KH>(U, rb + li, Bb, n, 8 * hh);
#pragma unroll
        for (int i = 0; i < 16; ++i) vt[nf_at<2 * PC>(rb + 8 * (i / 4) + 4 * hh + i % 4, n)] = acc[i];
    }
    __syncthreads();                                         // the elements of the scan are in LDS
    // ---- the scan
    const int cc = min(c, PC - 1);
    const float4 power = lam_of[cc];
    const float2 lam = make_float2(power.x, power.y), lam8 = make_float2(power.z, power.w);
    float2 val[NF_RUN], S = make_float2(0.f, 0.f);
#pragma unroll
    for (int i = 0; i < NF_RUN; ++i) val[i] = *reinterpret_cast<const float2 *>(vt + nf_at<2 * PC>(r0 + i, 2 * cc));
#pragma unroll
    for (int i = 0; i < NF_RUN; ++i) {
        const bool in = r0 + i < rows && active;             // (rows past the last token, states past the last: zeros)
        val[i] = make_float2(in ? val[i].x : 0.f, in ? val[i].y : 0.f);
        // the state that flows into a sequence, unless its first step drops it
        if (((start & ~first) >> (r0 + i)) & 1u) val[i] = cfma(lam, x0[i], val[i]);
    }
#pragma unroll
    for (int i = 0; i < NF_RUN; ++i) {
        const float2 n = cfma(lam, S, val[i]);
        const bool drop = cut >> (r0 + i) & 1u;
        S = make_float2(drop ? val[i].x : n.x, drop ? val[i].y : n.y);
    }
    if (c < PC) runs[q * PC + c] = S;
    __syncthreads();                                         // the states of the runs are in LDS
    float2 xs = make_float2(0.f, 0.f), Sj[NF_RUNS - 1];
#pragma unroll
    for (int j = 0; j < NF_RUNS - 1; ++j) Sj[j] = runs[j * PC + cc];
#pragma unroll
    for (int j = 0; j < NF_RUNS - 1; ++j) {
        if (j >= q) break;                                   // (uniform)
        const float2 n = cfma(lam8, xs, Sj[j]);
        const bool any = (cut >> (NF_RUN * j) & 0xffu) != 0;
        xs = make_float2(any ? Sj[j].x : n.x, any ? Sj[j].y : n.y);
    }
#pragma unroll
    for (int i = 0; i < NF_RUN; ++i) {
        const float2 n = cfma(lam, xs, val[i]);
        const bool drop = cut >> (r0 + i) & 1u;
        xs = make_float2(drop ? val[i].x : n.x, drop ? val[i].y : n.y);
        val[i] = xs;
    }
    if (c < PC) {
#pragma unroll
        for (int i = 0; i < NF_RUN; ++i) X.put(r0 + i, 2 * c, val[i]);
    }
    __syncthreads();                                         // the states are in LDS
    // ---- output projection: row block wave % 2, columns 32 (wave / 2 % 2) .., half wave / 4 of K
    const int kh = wave >> 2, n2 = 32 * (wave >> 1 & 1) + li;
    if ((wave >> 1 & 1) < HC / 32) {
        const v16f acc = multiply<KP>(X, rb + li, Cp, n2, PC * kh + 8 * hh);
#pragma unroll
        for (int i = 0; i < 16; ++i) pt[kh * NF_ROWS * HC + nf_at<HC>(rb + 8 * (i / 4) + 4 * hh + i % 4, n2)] = acc[i];
    }
    if (active) {
        if (a.x) {
            float2 *dst = a.x + (m0 + r0) * P + c;
#pragma unroll
            for (int i = 0; i < NF_RUN; ++i)
                if (r0 + i < rows) store_through(dst + i * P, val[i]);
        }
        if (a.x_last && (end >> r0 & 0xffu) != 0) {
#pragma unroll
            for (int i = 0; i < NF_RUN; ++i)
                if (end >> (r0 + i) & 1u) a.x_last[(long)sequence(r0 + i) * P + c] = val[i];
        }
    }
    __syncthreads();                                         // both halves of the product are in LDS
    const int nc = H - col;
#pragma unroll
    for (int j = 0; j < NU; ++j) {
        const int row = row0 + j * RSTEP;
        if (row >= rows || nc <= 0) continue;
        const float4 v = *reinterpret_cast<const float4 *>(pt + nf_at<HC>(row, col)), t = *reinterpret_cast<const float4 *>(pt + NF_ROWS * HC + nf_at<HC>(row, col));
        u[j] = make_float4(fmaf(d.x, u[j].x, v.x + t.x), fmaf(d.y, u[j].y, v.y + t.y), fmaf(d.z, u[j].z, v.z + t.z), fmaf(d.w, u[j].w, v.w + t.w));
        store4(a.y + (m0 + row) * H + col, u[j], nc);
    }
    if (a.gelu_y) {
#pragma unroll 1
        for (int j = 0; j < NU; ++j) {
            const int row = row0 + j * RSTEP;
            if (row >= rows || nc <= 0) continue;
            const float4 o = j == 0 ? u[0] : u[NU - 1];
            store4(a.gelu_y + (m0 + row) * H + col, make_float4(gelu_value(o.x), gelu_value(o.y), gelu_value(o.z), gelu_value(o.w)), nc);
        }
    }
    if (blockIdx.x == 0 && tid == 0) { a.hdr->err = 0; a.hdr->magic = 0x53534d31u; }
}

hipError_t launch_narrow_fwd(const NarrowFwd &in, hipStream_t s)
{
    NarrowFwd a = in;
    if (!a.Lambda || !a.B || !a.C || !a.D || !a.log_delta || !a.u || !a.y || !a.hdr || a.Bt <= 0 || a.L <= 0 || a.L > NF_ROWS || a.H < 4 || a.P < 2 || a.H > NARROW_MAX || a.P > NARROW_MAX ||
        (a.W && (!a.pack.frag || a.pack.planes != 3 || a.pack.kind != PACK_WN)))
        return hipErrorInvalidValue;
    a.seqs = NF_ROWS / a.L;
    a.by_L = FastDiv::by(a.L);
    a.layer_blocks = (a.Bt + a.seqs - 1) / a.seqs;
    long blocks = a.layer_blocks;
    if (a.W) {
        pack_place(a.pack, 0, NF_THREADS);
        blocks += a.pack.nblocks;
    }
    if (blocks > 0x7fffffffL) return hipErrorInvalidValue;
    const auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(NF_THREADS), 0, s, a);
        return hipGetLastError();
    };
    if (a.H <= 32) return a.P <= 32 ? launch(narrow_fwd_kernel<2, 2>) : launch(narrow_fwd_kernel<2, 4>);
    return a.P <= 32 ? launch(narrow_fwd_kernel<4, 2>) : launch(narrow_fwd_kernel<4, 4>);
}

}  // namespace ssm
