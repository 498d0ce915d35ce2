// Operations around the SSM layer (gfx950): the bootstrapped lambda-return of the actor-critic
// section and the half-GLU gate of the S5 sequence layer (appendix), with their adjoints.
#include "../../include/ssm.h"
#include "pack.h"

#include <type_traits>

namespace ssm {
namespace {

constexpr size_t ALIGN = 256;
inline size_t up(size_t n) { return (n + ALIGN - 1) / ALIGN * ALIGN; }
inline bool misaligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }
#define HIP_TRY(expr) do { if ((expr) != hipSuccess) return SSM_ERR_HIP; } while (0)

// ---------------------------------------------------------------------------------------------
// lambda-return:  V_t = r_t + gamma c_t ((1 - lambda) v_t + lambda V_{t+1}),  V_T = v_T.
// Time-major arrays [T, N]; one thread per trajectory walks time backwards.  Neighbouring
// threads read neighbouring trajectories of the same step, so every access is one coalesced
// row segment; the only serial dependency is one fused multiply-add per step.
// At 65536 trajectories a SIMD has a single wavefront, so a launch lasts as long as that one's trips to memory and its
// instructions one behind the other: the loads of eight steps are in flight together (then of four, two, one), and an address is a
// uniform row and the thread as its offset.  With a 64-bit address per value and four steps in flight (forward) or what the
// compiler made of a plain loop (adjoint), and now: 16 steps of 65536 trajectories 3.96 and 3.74 us, adjoint 6.16 and 5.25; 64 of 2048: 5.8
// and 4.8, 12.3 and 6.6.  (Sixteen steps in flight: 3.8 and 5.5 us at the first; workgroups of 256: the same within 2 %, slower at few trajectories.)
// ---------------------------------------------------------------------------------------------
constexpr int LAMBDA_STEPS = 8, LAMBDA_THREADS = 64;      // (and what is left of the steps in batches of four, two, one)
__global__ void __launch_bounds__(LAMBDA_THREADS) lambda_return_kernel(const float *__restrict__ r, const float *__restrict__ c,
                                                                       const float *__restrict__ v, float gamma, float lam,
                                                                       long T, long N, float *__restrict__ ret)
{
    // (rows from the workgroup's first trajectory on: a uniform address and the thread as its offset)
    const long n0 = (long)blockIdx.x * LAMBDA_THREADS;
    const unsigned n = threadIdx.x;
    if (n0 + n >= N) return;
    r += n0; c += n0; v += n0; ret += n0;
    const float gl = gamma * lam, g1 = gamma * (1.f - lam);
    float V = (v + (T - 1) * N)[n];
    (ret + (T - 1) * N)[n] = V;
    long t = T - 2;
    auto steps = [&](auto count) {
        constexpr int S = decltype(count)::value;
        for (; t >= S - 1; t -= S) {
            float rr[S], cc[S], vv[S];
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const long o = (t - j) * N;
                rr[j] = (r + o)[n]; cc[j] = (c + o)[n]; vv[j] = (v + o)[n];
            }
#pragma unroll
            for (int j = 0; j < S; ++j) {
                // r + c (g1 v) + (c gl) V
                V = fmaf(cc[j] * gl, V, fmaf(cc[j], g1 * vv[j], rr[j]));
                (ret + (t - j) * N)[n] = V;
            }
        }
    };
    steps(std::integral_constant<int, LAMBDA_STEPS>{});
    steps(std::integral_constant<int, 4>{});
    steps(std::integral_constant<int, 2>{});
    steps(std::integral_constant<int, 1>{});
}

// Adjoint: G_t = dret_t + gamma lambda c_{t-1} G_{t-1} walks time forwards;
// dr_t = G_t, dc_t = G_t gamma ((1-lambda) v_t + lambda V_{t+1}), dv_t = G_t gamma c_t (1-lambda) for t < T-1;
// the last step has dv = G and no reward / continue gradient.
__global__ void __launch_bounds__(LAMBDA_THREADS) lambda_return_bwd_kernel(const float *__restrict__ c, const float *__restrict__ v,
                                                                           const float *__restrict__ ret, const float *__restrict__ dret,
                                                                           float gamma, float lam, long T, long N,
                                                                           float *__restrict__ dr, float *__restrict__ dc,
                                                                           float *__restrict__ dv)
{
    const long n0 = (long)blockIdx.x * LAMBDA_THREADS;
    const unsigned n = threadIdx.x;
    if (n0 + n >= N) return;
    c += n0; v += n0; ret += n0; dret += n0; dr += n0; dc += n0; dv += n0;
    const float gl = gamma * lam, g1 = gamma * (1.f - lam);
    float G = 0.f, cprev = 0.f;
    long t = 0;
    auto steps = [&](auto count) {
        constexpr int S = decltype(count)::value;
        for (; t + S < T; t += S) {
            float cc[S], vv[S], rt[S], dd[S];
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const long o = (t + j) * N;
                cc[j] = (c + o)[n]; vv[j] = (v + o)[n]; rt[j] = (ret + o + N)[n]; dd[j] = (dret + o)[n];
            }
#pragma unroll
            for (int j = 0; j < S; ++j) {
                const long o = (t + j) * N;
                G = fmaf(gl * cprev, G, dd[j]);
                (dr + o)[n] = G;
                (dc + o)[n] = G * fmaf(gl, rt[j], g1 * vv[j]);
                (dv + o)[n] = G * (g1 * cc[j]);
                cprev = cc[j];
            }
        }
    };
    steps(std::integral_constant<int, LAMBDA_STEPS>{});
    steps(std::integral_constant<int, 4>{});
    steps(std::integral_constant<int, 2>{});
    steps(std::integral_constant<int, 1>{});
    const long o = (T - 1) * N;
    G = fmaf(gl * cprev, G, (dret + o)[n]);
    (dr + o)[n] = 0.f;
    (dc + o)[n] = 0.f;
    (dv + o)[n] = G;
}

// ---------------------------------------------------------------------------------------------
// half-GLU:  x1 = GELU(u),  y = u (.) sigmoid(x1 W).
// The element-wise halves run as small streaming kernels (float4 per thread); the products run
// on the projection GEMM with the gate fused into its store (epilogues 3 and 4).
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ float gelu_exact(float x) { return gelu_value(x); }

// Every element-wise pass also packs W for the product behind it, in workgroups of its own at the head of the grid.
__global__ void __launch_bounds__(256) gelu_kernel(const float4 *__restrict__ u, float4 *__restrict__ x1, long n4,
                                                   const float *__restrict__ ut, float *__restrict__ x1t, long n, PackSrc src, PackJob w)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[PACK_LDS_BYTES];
    if ((int)blockIdx.x < w.nblocks) { pack_block<PACK_WN, 3>(src, w, blockIdx.x, lds); return; }
    const long i = (long)(blockIdx.x - w.nblocks) * 256 + threadIdx.x;
    if (i < n4) {
        const float4 a = u[i];
        x1[i] = make_float4(gelu_exact(a.x), gelu_exact(a.y), gelu_exact(a.z), gelu_exact(a.w));
    }
    const long j = 4 * n4 + i;                           // the up to three elements past the last float4
    if (i < 4 && j < n) x1t[j] = gelu_exact(ut[j]);
}

// One pass over the inputs of the gate's adjoint (s = the gate saved by the forward call): x1 = GELU(u) and
// dz = dy u s (1 - s), the operands of the two products, and the two terms that the store of dz W^T needs,
// ds = dy s and gd = GELU'(u) (du = ds + (dz W^T) gd): formed here, where u, s and dy pass anyway, they cost
// that store two loads per value and no error function.
__global__ void __launch_bounds__(256) gate_bwd_prep_kernel(const float *__restrict__ u, const float *__restrict__ s,
                                                            const float *__restrict__ dy, float *__restrict__ x1,
                                                            float *__restrict__ dz, float *__restrict__ ds,
                                                            float *__restrict__ gd, long n, PackSrc src, PackJob w)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[PACK_LDS_BYTES];
    if ((int)blockIdx.x < w.nblocks) { pack_block<PACK_WT, 3>(src, w, blockIdx.x, lds); return; }
    const long i0 = ((long)(blockIdx.x - w.nblocks) * 256 + threadIdx.x) * 4;
    if (i0 + 4 <= n) {
        const float4 a = *reinterpret_cast<const float4 *>(u + i0);
        const float4 g = *reinterpret_cast<const float4 *>(s + i0);
        const float4 d = *reinterpret_cast<const float4 *>(dy + i0);
        *reinterpret_cast<float4 *>(x1 + i0) =
            make_float4(gelu_exact(a.x), gelu_exact(a.y), gelu_exact(a.z), gelu_exact(a.w));
        *reinterpret_cast<float4 *>(dz + i0) =
            make_float4(d.x * a.x * (g.x * (1.f - g.x)), d.y * a.y * (g.y * (1.f - g.y)),
                        d.z * a.z * (g.z * (1.f - g.z)), d.w * a.w * (g.w * (1.f - g.w)));
        *reinterpret_cast<float4 *>(ds + i0) = make_float4(d.x * g.x, d.y * g.y, d.z * g.z, d.w * g.w);
        *reinterpret_cast<float4 *>(gd + i0) =
            make_float4(gelu_derivative(a.x), gelu_derivative(a.y), gelu_derivative(a.z), gelu_derivative(a.w));
    } else {
        for (long i = i0; i < n; ++i) {
            x1[i] = gelu_exact(u[i]);
            dz[i] = dy[i] * u[i] * (s[i] * (1.f - s[i]));
            ds[i] = dy[i] * s[i];
            gd[i] = gelu_derivative(u[i]);
        }
    }
}

// The same two passes for widths that are multiples of 64, where the products behind them stage their
// operands as two scaled fp16 planes (three matrix instructions per k block instead of six): they also
// measure the largest magnitudes that scale those planes -- of every token row of the product's first
// operand in pieces of 64 columns (rowmax[piece][row]; 16 neighbouring lanes hold one piece), of a whole
// operand per workgroup (slots[workgroup]).
__device__ __forceinline__ unsigned abs_bits4(float4 v)
{
    return __float_as_uint(fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
}
__device__ __forceinline__ unsigned max16(unsigned v)
{
#pragma unroll
    for (int o = 8; o > 0; o >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, o));
    return v;
}
// maximum over the 256 threads of the workgroup, valid in thread 0 (red: 4 words of LDS)
__device__ __forceinline__ unsigned block_max(unsigned v, unsigned *red)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = max(v, (unsigned)__shfl_xor((int)v, o));
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    return max(max(red[0], red[1]), max(red[2], red[3]));
}
__global__ void __launch_bounds__(256) gelu_max_kernel(const float4 *__restrict__ u, float4 *__restrict__ x1, long n4,
                                                       int H, long T, unsigned *__restrict__ rowmax, PackSrc src, PackJob w)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[PACK_LDS_BYTES];
    if ((int)blockIdx.x < w.nblocks) {                   // (first in the grid: their chains of loads start at once)
        pack_block<PACK_WN, 2>(src, w, blockIdx.x, lds);
        return;
    }
    const long i = (long)(blockIdx.x - w.nblocks) * 256 + threadIdx.x;
    unsigned m = 0;
    if (i < n4) {                                        // (n4 is a multiple of 16: a row piece is in or out as a whole)
        const float4 a = u[i];
        const float4 g = make_float4(gelu_exact(a.x), gelu_exact(a.y), gelu_exact(a.z), gelu_exact(a.w));
        x1[i] = g;
        m = abs_bits4(g);
    }
    m = max16(m);
    if ((threadIdx.x & 15) == 0 && i < n4) {
        const long e0 = i * 4, row = e0 / H;
        rowmax[(size_t)((e0 - row * H) / 64) * T + row] = m;
    }
}

__global__ void __launch_bounds__(256) gate_bwd_prep_max_kernel(const float *__restrict__ u, const float *__restrict__ s,
                                                                const float *__restrict__ dy, float *__restrict__ x1,
                                                                float *__restrict__ dz, float *__restrict__ ds,
                                                                float *__restrict__ gd, long n, int H, long T,
                                                                unsigned *__restrict__ dz_rowmax,
                                                                unsigned *__restrict__ x1_slots, unsigned *__restrict__ dz_slots,
                                                                PackSrc src, PackJob w)
{
    __shared__ __attribute__((aligned(16))) unsigned char lds[PACK_LDS_BYTES];
    unsigned *red = reinterpret_cast<unsigned *>(lds);
    if ((int)blockIdx.x < w.nblocks) {
        pack_block<PACK_WT, 2>(src, w, blockIdx.x, lds);
        return;
    }
    const int b = (int)blockIdx.x - w.nblocks, main_blocks = (int)gridDim.x - w.nblocks;
    const long stride = (long)main_blocks * 1024;
    unsigned mx = 0, mz = 0;
    for (long base = ((long)b * 256 + threadIdx.x) * 4; base < n; base += 4 * stride) {
        // the inputs of four pieces first, so that their loads are in flight together
        float4 a[4], g[4], d[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const long i0 = base + k * stride;
            if (i0 < n) {
                a[k] = *reinterpret_cast<const float4 *>(u + i0);
                g[k] = *reinterpret_cast<const float4 *>(s + i0);
                d[k] = *reinterpret_cast<const float4 *>(dy + i0);
            }
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const long i0 = base + k * stride;
            if (i0 < n) {                                // (n is a multiple of 64: the 16 lanes of a piece stay together)
                const float4 xo = make_float4(gelu_exact(a[k].x), gelu_exact(a[k].y), gelu_exact(a[k].z), gelu_exact(a[k].w));
                const float4 zo = make_float4(d[k].x * a[k].x * (g[k].x * (1.f - g[k].x)), d[k].y * a[k].y * (g[k].y * (1.f - g[k].y)),
                                              d[k].z * a[k].z * (g[k].z * (1.f - g[k].z)), d[k].w * a[k].w * (g[k].w * (1.f - g[k].w)));
                *reinterpret_cast<float4 *>(x1 + i0) = xo;
                *reinterpret_cast<float4 *>(dz + i0) = zo;
                *reinterpret_cast<float4 *>(ds + i0) = make_float4(d[k].x * g[k].x, d[k].y * g[k].y, d[k].z * g[k].z, d[k].w * g[k].w);
                *reinterpret_cast<float4 *>(gd + i0) =
                    make_float4(gelu_derivative(a[k].x), gelu_derivative(a[k].y), gelu_derivative(a[k].z), gelu_derivative(a[k].w));
                const unsigned bz = abs_bits4(zo);
                mx = max(mx, abs_bits4(xo)); mz = max(mz, bz);
                const unsigned piece = max16(bz);
                if ((threadIdx.x & 15) == 0) {
                    const long row = i0 / H;
                    dz_rowmax[(size_t)((i0 - row * H) / 64) * T + row] = piece;
                }
            }
        }
    }
    mx = block_max(mx, red);
    __syncthreads();
    mz = block_max(mz, red);
    if (threadIdx.x == 0) { x1_slots[b] = mx; dz_slots[b] = mz; }
}

// fixed-order sum of the K-split slabs of a product
__global__ void __launch_bounds__(256) sum_slabs_kernel(const float *__restrict__ part, long n, int nslab,
                                                        float *__restrict__ out)
{
    const long i = (long)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    // (up to eight loads in flight: one slab at a time, a sum over many slabs of a small matrix is that many trips to memory in a row:
    // 4096 tokens, H = 64, 64 slabs: the gate's gradient pass 29.1 us, now 15.1)
    float acc = 0.f;
    int z = 0;
    const float *p = part + i;
    auto batch = [&](auto count) {
        constexpr int N = decltype(count)::value;
        for (; z + N <= nslab; z += N, p += N * n) {
            float v[N];
#pragma unroll
            for (int j = 0; j < N; ++j) v[j] = p[j * n];
#pragma unroll
            for (int j = 0; j < N; ++j) acc += v[j];
        }
    };
    batch(std::integral_constant<int, 8>{});
    batch(std::integral_constant<int, 4>{});
    batch(std::integral_constant<int, 1>{});
    out[i] = acc;
}

constexpr int GLU_MAX_SLOTS = 512;      // workgroups of the element-wise pass that report a maximum each
struct GluLayout {
    size_t x1, dz, ds, gd, dWpart, wfrag, wexp, total; int splits, planes;
    // widths that are multiples of 64: two scaled fp16 planes per operand, with their largest magnitudes
    bool two_planes; size_t rowmax, slots; int row_parts, main_blocks;
    bool dw_first;             // gradient pass, one launch for dz W^T and the slabs of x1^T dz: dW's work items first
};

bool make_glu_layout(int64_t T, int64_t H, bool bwd, GluLayout &o)
{
    if (T <= 0 || H <= 0 || H > SSM_MAX_WIDTH || T > SSM_MAX_TOKENS || T > SSM_MAX_ELEMS / H) return false;
    size_t off = 0;
    o.x1 = off; off += up((size_t)T * H * 4);
    o.dz = o.ds = o.gd = o.dWpart = 0; o.splits = 1;
    o.two_planes = gate_two_planes_shape(T, H);
    // gradient pass: both products wait for the same element-wise pass and share one launch
    o.planes = o.two_planes ? 2 : 3; o.dw_first = false;
    o.wfrag = off; off += up(packed_frag_bytes(H, H, o.planes));
    o.wexp = off; off += up((size_t)(H + 31) / 32 * 32 * 4);
    if (bwd) {
        o.dz = off; off += up((size_t)T * H * 4);
        o.ds = off; off += up((size_t)T * H * 4);
        o.gd = off; off += up((size_t)T * H * 4);
        const SlabPlan dW = gemm_plan_slabs(H, H, T, 1, reduction_tile(o.planes, gemm_small_pair(T, H)), H);
        o.splits = dW.slabs; o.dw_first = dW.first;
    }
    if (bwd) { o.dWpart = off; off += up((size_t)o.splits * H * H * 4); }
    o.rowmax = o.slots = 0; o.row_parts = o.main_blocks = 0;
    if (o.two_planes) {
        o.row_parts = (int)(H / 64);
        const int64_t blocks = (T * H / 4 + 255) / 256;
        o.main_blocks = (int)(bwd ? (blocks < GLU_MAX_SLOTS ? blocks : GLU_MAX_SLOTS) : blocks);
        o.rowmax = off; off += up((size_t)o.row_parts * T * 4);
        o.slots = off; off += up((size_t)(2 * GLU_MAX_SLOTS) * 4);     // x1, dz
    }
    o.total = off;
    return true;
}

PackJob glu_pack(char *ws, const GluLayout &lo, int64_t H, int kind)
{
    PackJob j{};
    j.kind = kind; j.N = j.K = (int)H; j.planes = lo.planes;
    j.frag = ws + lo.wfrag; j.exp = reinterpret_cast<int *>(ws + lo.wexp);
    pack_place(j, 0);
    return j;
}
PackSrc glu_source(const float *W, int64_t H)
{
    PackSrc s{};
    s.W = W; s.H = (int)H;
    return s;
}

}  // namespace

int half_glu_backward(const float *u, const float *W, const float *gate, const float *dy, int64_t T, int64_t H, float *du, float *dW,
                      void *workspace, size_t ws_bytes, hipStream_t s, SlabSum *dW_slabs)
{
    if (!u || !W || !gate || !dy || !du || !dW) return SSM_ERR_INVALID_ARG;
    if (T <= 0 || H <= 0) return SSM_ERR_INVALID_ARG;
    GluLayout lo;
    if (!make_glu_layout(T, H, true, lo)) return SSM_ERR_UNSUPPORTED;
    if (misaligned(u, 16) || misaligned(W, 4) || misaligned(gate, 16) || misaligned(dy, 16) || misaligned(du, 4) ||
        misaligned(dW, 4))
        return SSM_ERR_INVALID_ARG;
    if (!workspace || misaligned(workspace, ALIGN) || ws_bytes < lo.total) return SSM_ERR_WORKSPACE;
    char *ws = static_cast<char *>(workspace);
    float *x1 = reinterpret_cast<float *>(ws + lo.x1);
    float *dz = reinterpret_cast<float *>(ws + lo.dz);
    float *ds = reinterpret_cast<float *>(ws + lo.ds), *gd = reinterpret_cast<float *>(ws + lo.gd);
    float *dWpart = reinterpret_cast<float *>(ws + lo.dWpart);
    const long n = (long)T * H;
    unsigned *rowmax = reinterpret_cast<unsigned *>(ws + lo.rowmax);
    unsigned *x1_slots = reinterpret_cast<unsigned *>(ws + lo.slots), *dz_slots = x1_slots + GLU_MAX_SLOTS;
    const PackJob w = glu_pack(ws, lo, H, PACK_WT);
    if (lo.two_planes) {
        hipLaunchKernelGGL(gate_bwd_prep_max_kernel, dim3((unsigned)(lo.main_blocks + w.nblocks)), dim3(256), 0, s, u, gate, dy,
                           x1, dz, ds, gd, n, (int)H, (long)T, rowmax, x1_slots, dz_slots, glu_source(W, H), w);
    } else {
        hipLaunchKernelGGL(gate_bwd_prep_kernel, dim3((unsigned)(((n + 3) / 4 + 255) / 256 + w.nblocks)), dim3(256), 0, s, u, gate, dy, x1,
                           dz, ds, gd, n, glu_source(W, H), w);
    }
    HIP_TRY(hipGetLastError());
    // du[t, i] = ds[t, i] + gd[t, i] sum_j dz[t, j] W[i, j]
    GemmArgs g{};
    g.A = dz; g.lda = H; g.w = PackedW{w.frag, w.exp}; g.planes = lo.planes;
    g.C = du; g.ldc = H; g.E = ds; g.E2 = gd; g.lde = H; g.epilogue = 4;
    g.M = (int)T; g.N = (int)H; g.K = (int)H;
    if (lo.two_planes) g.amaxA = AbsMax{nullptr, 0, rowmax, lo.row_parts, (long)T};
    // dW[i, j] = sum_t x1[t, i] dz[t, j]: reduction over tokens in K slabs (same launch), then a fixed-order sum
    GemmArgs h{};
    h.A = x1; h.lda = H;
    h.B = dz; h.ldb = H;
    h.C = dWpart; h.ldc = H;
    h.M = (int)H; h.N = (int)H; h.K = (int)T; h.splits = lo.splits;
    if (lo.two_planes) { h.amaxA = AbsMax{x1_slots, lo.main_blocks, nullptr, 0, 0}; h.amaxB = AbsMax{dz_slots, lo.main_blocks, nullptr, 0, 0}; }
    HIP_TRY(launch_products(g, &h, nullptr, lo.dw_first, s));
    const long nw = (long)H * H;
    if (dW_slabs) {
        *dW_slabs = SlabSum{dWpart, dW, nw, lo.splits};
        return SSM_OK;
    }
    hipLaunchKernelGGL(sum_slabs_kernel, dim3((unsigned)((nw + 255) / 256)), dim3(256), 0, s, dWpart, nw, lo.splits, dW);
    HIP_TRY(hipGetLastError());
    return SSM_OK;
}

}  // namespace ssm

using namespace ssm;

extern "C" {

ssm_status ssm_lambda_return(const float *reward, const float *cont, const float *value, float gamma,
                             float lambda, int64_t T, int64_t N, float *ret, void *stream)
{
    if (!reward || !cont || !value || !ret) return SSM_ERR_INVALID_ARG;
    if (T <= 0 || N <= 0) return SSM_ERR_INVALID_ARG;
    if (T > SSM_MAX_TOKENS || N > SSM_MAX_TOKENS || T > SSM_MAX_ELEMS / N) return SSM_ERR_UNSUPPORTED;
    if (misaligned(reward, 4) || misaligned(cont, 4) || misaligned(value, 4) || misaligned(ret, 4))
        return SSM_ERR_INVALID_ARG;
    const unsigned blocks = (unsigned)((N + LAMBDA_THREADS - 1) / LAMBDA_THREADS);
    hipLaunchKernelGGL(lambda_return_kernel, dim3(blocks), dim3(LAMBDA_THREADS), 0, static_cast<hipStream_t>(stream),
                       reward, cont, value, gamma, lambda, (long)T, (long)N, ret);
    HIP_TRY(hipGetLastError());
    return SSM_OK;
}

ssm_status ssm_lambda_return_bwd(const float *cont, const float *value, const float *ret, const float *dret,
                                 float gamma, float lambda, int64_t T, int64_t N,
                                 float *dreward, float *dcont, float *dvalue, void *stream)
{
    if (!cont || !value || !ret || !dret || !dreward || !dcont || !dvalue) return SSM_ERR_INVALID_ARG;
    if (T <= 0 || N <= 0) return SSM_ERR_INVALID_ARG;
    if (T > SSM_MAX_TOKENS || N > SSM_MAX_TOKENS || T > SSM_MAX_ELEMS / N) return SSM_ERR_UNSUPPORTED;
    if (misaligned(cont, 4) || misaligned(value, 4) || misaligned(ret, 4) || misaligned(dret, 4) ||
        misaligned(dreward, 4) || misaligned(dcont, 4) || misaligned(dvalue, 4))
        return SSM_ERR_INVALID_ARG;
    const unsigned blocks = (unsigned)((N + LAMBDA_THREADS - 1) / LAMBDA_THREADS);
    hipLaunchKernelGGL(lambda_return_bwd_kernel, dim3(blocks), dim3(LAMBDA_THREADS), 0, static_cast<hipStream_t>(stream),
                       cont, value, ret, dret, gamma, lambda, (long)T, (long)N, dreward, dcont, dvalue);
    HIP_TRY(hipGetLastError());
    return SSM_OK;
}

size_t ssm_half_glu_workspace_bytes(int64_t T, int64_t H, int want_bwd)
{
    GluLayout lo;
    return make_glu_layout(T, H, want_bwd != 0, lo) ? lo.total : 0;
}

ssm_status ssm_half_glu_fwd(const float *u, const float *W, int64_t T, int64_t H, float *y, float *gate,
                            void *workspace, size_t ws_bytes, void *stream)
{
    if (!u || !W || !y) return SSM_ERR_INVALID_ARG;
    if (T <= 0 || H <= 0) return SSM_ERR_INVALID_ARG;
    GluLayout lo;
    if (!make_glu_layout(T, H, false, lo)) return SSM_ERR_UNSUPPORTED;
    if (misaligned(u, 16) || misaligned(W, 4) || misaligned(y, 4) || misaligned(gate, 4)) return SSM_ERR_INVALID_ARG;
    if (!workspace || misaligned(workspace, ALIGN) || ws_bytes < lo.total) return SSM_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    float *x1 = reinterpret_cast<float *>(ws + lo.x1);
    const long n = (long)T * H, n4 = n / 4;
    unsigned *rowmax = reinterpret_cast<unsigned *>(ws + lo.rowmax);
    const PackJob w = glu_pack(ws, lo, H, PACK_WN);
    if (lo.two_planes) {
        hipLaunchKernelGGL(gelu_max_kernel, dim3((unsigned)(lo.main_blocks + w.nblocks)), dim3(256), 0, s,
                           reinterpret_cast<const float4 *>(u), reinterpret_cast<float4 *>(x1), n4, (int)H, (long)T, rowmax,
                           glu_source(W, H), w);
    } else {
        const long threads = n4 > 4 ? n4 : 4;
        hipLaunchKernelGGL(gelu_kernel, dim3((unsigned)((threads + 255) / 256 + w.nblocks)), dim3(256), 0, s,
                           reinterpret_cast<const float4 *>(u), reinterpret_cast<float4 *>(x1), n4, u, x1, n, glu_source(W, H), w);
    }
    HIP_TRY(hipGetLastError());
    // y[t, j] = u[t, j] sigmoid(sum_i x1[t, i] W[i, j])
    GemmArgs g{};
    g.A = x1; g.lda = H; g.w = PackedW{w.frag, w.exp}; g.planes = lo.planes;
    g.C = y; g.ldc = H; g.E = u; g.lde = H; g.C2 = gate; g.epilogue = 3;
    g.M = (int)T; g.N = (int)H; g.K = (int)H;
    if (lo.two_planes) g.amaxA = AbsMax{nullptr, 0, rowmax, lo.row_parts, (long)T};
    HIP_TRY(launch_product(g, s));
    return SSM_OK;
}

ssm_status ssm_half_glu_bwd(const float *u, const float *W, const float *gate, const float *dy,
                            int64_t T, int64_t H, float *du, float *dW,
                            void *workspace, size_t ws_bytes, void *stream)
{
    return static_cast<ssm_status>(half_glu_backward(u, W, gate, dy, T, H, du, dW, workspace, ws_bytes, static_cast<hipStream_t>(stream), nullptr));
}

}  // extern "C"
