// Internal declarations shared by the translation units of libssmscan (gfx950 only).
// Nothing here is part of the C ABI; see include/ssm.h for that.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "fast_div.h"
#include "store_rule.h"

namespace ssm {

// ---------------------------------------------------------------------------------------------
// Projection products.  Two kinds:
//   a product of activations with packed weights, C[m,n] = f(sum_k A[m,k] W(n,k))  (gemm_packed.h).  f:
//     epilogue 0: none; 1: + diag[n] * E[m,n]; 2: + [not rowflag[m]] * (Abar (.) E)[m,n] with diag = Abar as
//     interleaved complex and the columns of C and E interleaved (re, im) pairs (one recurrence step);
//     3: C = E (.) sigmoid(product), sigmoid kept in C2 when non-null (half-GLU gate);
//     4: C = E + product (.) E2 (adjoint of the gate with respect to its input: E = dy (.) s, E2 = GELU'(u));
//     5: C = product + E (E may be null), C2 = [not rowflag[m]] conj(Abar) (.) C with diag = Abar and complex
//        (re, im) column pairs (adjoint of one recurrence step);
//     6: as 1, and C2 = GELU(C) (output projection that feeds the half-GLU gate);
//     7: the resettable scan over the rows of the output tile (see ScanEpilogue): C = states;
//     8: the reverse-time scan of the gradient pass over the rows of the output tile: C = chi;
//     9, 10: as 7 and 8 with two planes and sequences of any length;
//   a reduction over tokens, C[m,n] = sum_k A[k,m] B[k,n]  (gemm_kernel.h).  splits > 1: split z covers a
//     contiguous K range and writes its own slab C + z*M*ldc; the caller reduces the slabs.
// ---------------------------------------------------------------------------------------------
// Largest magnitude of a matrix, kept as n bit patterns of non-negative floats whose maximum it is
// (written by the kernel that produced the matrix, or by a pass over it), or, for a matrix whose
// rows are tokens, per row: rows[j * row_stride + r], j < row_parts, are patterns whose maximum is the
// largest magnitude of row r.  A product whose two operands both carry one may stage them as two
// scaled fp16 planes (see gemm_kernel.h); per-row maxima (k-contiguous A operand only) give
// every row its own scale.
constexpr int ABSMAX_SLOTS = 512;            // slots of a maximum that is gathered with atomics
struct AbsMax {
    const unsigned *slots; int n;            // slots == nullptr and rows == nullptr: not known
    const unsigned *rows; int row_parts; long row_stride;
};

// Epilogue 7 of a product with packed weights: the resettable scan (Eq. 4 with the elements of Eq. 9 and the
// operator of Eq. 10) over the rows of the output tile itself, so that the input projection stores the states x
// directly and Bbar u never goes to memory.  Rows are tokens (Bt sequences of L steps), columns (re, im) pairs of P
// states.
constexpr int SCAN_MAX_STEPS = 4096;         // longest sequence
constexpr int ROW_SCAN_MAX_TILES = 64;       // scans of rows: tiles of a sequence that come before another one
constexpr uint32_t ROW_SCAN_POLLS = 256;     // polls after which a tile computes the aggregate that it waits for itself: a few times as long as a launch takes
struct ScanEpilogue {
    const float2 *lam;            // [P] Abar
    const uint8_t *is_first;      // [Bt*L] or null
    const float2 *x0;             // [Bt, P] or null
    float2 *x_last;               // [Bt, P] or null (forward)
    const float2 *xsaved;         // [Bt, L, P] states of the forward pass (reverse, epilogues 8 and 10)
    float2 *partial;              // [ceil(Bt * L / rows), P] per-tile rows of dAbar (reverse)
    float2 *dx0;                  // [Bt, P] or null (reverse)
    unsigned long long *desc;     // [M / 64 * ceil(N/128) * 64][2] tagged aggregate words, scans of rows: [ceil(M / rows)][2][P]; zero on entry
    unsigned *err;                // set when a bounded wait gives up
    unsigned *amax_out;           // [ABSMAX_SLOTS] or null (epilogue 10: not): atomic maximum of the magnitudes stored to C, zero on entry
    unsigned *xmax_out;           // [ABSMAX_SLOTS] or null (epilogue 8, with amax_out): atomic maximum of the magnitudes of xsaved
    unsigned *rowmax_out;         // [ceil(N/128), M] or null: per column tile and row, the largest magnitude stored to C
    int L, P;
    FastDiv by_L;                 // set by the launch
    int rows;                     // tokens per tile: gemm_scan_rows, three planes: gemm_row_scan_rows
    unsigned spin_limit;
};

// Weights in fragment order, split into planes (see gemm_packed.h); exp: log2 of the scale of every row n (two planes).
struct PackedW { const void *frag; const int *exp; };
// bytes of the fragments of N x K weights
inline size_t packed_frag_bytes(int64_t N, int64_t K, int planes) { return (size_t)((N + 31) / 32 * 32) * (size_t)((K + 63) / 64 * 64) * 2 * planes; }

struct GemmArgs {
    const float *A; int64_t lda;
    const float *B; int64_t ldb;                     // reductions
    PackedW w; int planes;                           // products with packed weights: 2 or 3 planes per operand
    float *C; int64_t ldc;
    const float *diag; const float *E; int64_t lde;
    int epilogue; const uint8_t *rowflag;
    const float *E2; float *C2;                      // epilogues 3, 4, 6 (gate), pitch lde / ldc; 5
    int M, N, K, splits;
    ScanEpilogue scan;                               // epilogues 7 to 10
    AbsMax amaxA, amaxB;                             // largest magnitudes of A (products: of its rows) and B when known
    unsigned *c2_rowmax;                             // epilogue 6: [ceil(N/128)][M] words, the largest magnitude of every
                                                     // row of C2 per piece of 128 columns; or null
};
// The gate's products stage two scaled fp16 planes per operand (and the passes before them measure the
// largest magnitudes) at widths that are multiples of 64 from 512 on, with enough tokens (against three planes, forward +
// gradient pass: -7 % at 4096 tokens, H = 512, -17 % at 16384; -24 % at 4096, H = 1024.  Below the line, two planes against
// three: +27 % at 2048 tokens, H = 256, where the passes cost more than the shorter K loops save, -3 % at 16384; +12 % at
// 1024, H = 512, -4 % at 2048 and -11 % at 3000, where the exact three planes are kept)
inline bool gate_two_planes_shape(int64_t T, int64_t H) { return H % 64 == 0 && H >= 512 && ((T + 63) / 64) * ((H + 127) / 128) >= 200; }
// the input projection (epilogue 7) and C^H dy (epilogue 8, the reverse scan of the gradient pass) scan
// their own output tiles at this shape
bool gemm_scan_shape_ok(int64_t Bt, int64_t L, int64_t P);
// tokens per scanning tile at such a shape: 64 or 128
int gemm_scan_rows(int64_t T, int64_t L, int64_t P, bool reverse);
// bytes of tagged words epilogues 7 and 8 need (zeroed before the launch)
size_t gemm_scan_desc_bytes(int64_t Bt, int64_t L, int64_t P);
// the same products scan the rows of their tiles, sequences of any length (epilogues 7 and 8 with three planes, 9 and 10 on 64 rows with two): tokens per tile with
// three planes, 32 or 64, 0 where they do not; and the bytes of tagged words
int gemm_row_scan_rows(int64_t T, int64_t L, int64_t P);
size_t gemm_row_scan_desc_bytes(int64_t T, int64_t P, int rows);
// One launch: a product with packed weights and up to two reductions over tokens whose inputs are ready at the same
// time (b, c: null when absent; c only with b).  tn_first: the reductions' work items take the first slots.
hipError_t launch_products(const GemmArgs &a, const GemmArgs *b, const GemmArgs *c, bool tn_first, hipStream_t s);
inline hipError_t launch_product(const GemmArgs &a, hipStream_t s) { return launch_products(a, nullptr, nullptr, false, s); }
// the instantiations with two and three planes
hipError_t products_two_planes(const GemmArgs &a, const GemmArgs *b, const GemmArgs *c, bool tn_first, hipStream_t s);
hipError_t products_three_planes(const GemmArgs &a, const GemmArgs *b, const GemmArgs *c, bool tn_first, hipStream_t s);
// the tile of the product of a launch (arguments as for launch_products; of a, M, N, planes, epilogue, scan.rows and
// c2_rowmax count, of the reductions M, N and splits)
struct PkTile { int rows, cols; };
PkTile product_tile(const GemmArgs &a, const GemmArgs *b, const GemmArgs *c);
// a product over T tokens with N columns has so few tiles that the reduction in its launch runs on 64x64 tiles
bool gemm_small_pair(int64_t T, int64_t N);
// Tiles of the reductions of a launch: beside small products, beside other products on three planes, on two planes.
enum ReductionTile { REDUCTION_64x64 = 64, REDUCTION_128x64 = 96, REDUCTION_128x128 = 128 };
inline ReductionTile reduction_tile(int planes, bool small) { return planes == 2 ? REDUCTION_128x128 : small ? REDUCTION_64x64 : REDUCTION_128x64; }
// K slabs of `count` reductions of M x N over K rows that share a launch with a product whose K loop is k_main long, and
// whether their work items take the first slots
struct SlabPlan { int slabs; bool first; };
inline int64_t reduction_items(int64_t M, int64_t N, int slabs, ReductionTile tile)
{
    const int64_t tm = tile == REDUCTION_64x64 ? 64 : 128, tn = tile == REDUCTION_128x128 ? 128 : 64;
    return ((M + tm - 1) / tm) * ((N + tn - 1) / tn) * slabs;
}
SlabPlan gemm_plan_slabs(int64_t M, int64_t N, int64_t K, int count, ReductionTile tile, int64_t k_main);

// ---------------------------------------------------------------------------------------------
// Resettable scan over the sequence dimension (forward and reverse time).
// One thread owns SCAN_E consecutive steps of one (sequence, state) lane; a workgroup is laid out as cy chunks x pxb lanes and so
// covers cy*SCAN_E steps of pxb states: whole sequences, or a part of longer ones, whose workgroups along time hand their
// running state forward through descriptors in global memory (decoupled look-back).
// ---------------------------------------------------------------------------------------------
constexpr int SCAN_E = 16;
constexpr int SCAN_MAX_THREADS = 1024;
constexpr int SCAN_TICKET_STRIDE = 16;   // uint32 slots between the ticket counters of two chains

struct ScanDesc {            // one per (workgroup, lane); 32 bytes; every word = (float << 32) | tag
    unsigned long long agg[2];   // re, im of the state at the end of the workgroup's steps for zero
                                 // incoming state; tag 1 = no reset among the steps, tag 2 = reset
    unsigned long long incl[2];  // re, im of that state with the incoming state included; tag 3
};

struct ScanPlan {
    int pxb, cy;             // lanes and chunks per workgroup
    int nPX, nTB;            // workgroups along the state and the time dimension
    int64_t nblocks;         // nPX * Bt * nTB
    size_t ticket_bytes;     // per-chain ticket counters, 0 when nTB == 1
    size_t desc_bytes;       // 0 when nTB == 1
    size_t partial_elems;    // Bt * nTB * P complex partial sums of the reverse scan
};
// records: the scans also record the magnitudes of their output (ScanArgs::rowmax_out)
ScanPlan plan_scan(int64_t Bt, int64_t L, int64_t P, bool records);

struct WsHeader {            // first 256 bytes of every workspace
    uint32_t err, magic;
};

struct ScanArgs {
    const float2 *in;        // v (forward) or gx (reverse), [Bt,L,P]
    float2 *out;             // x (forward) or chi (reverse); may alias `in`
    const float2 *lam;       // A_bar [P]
    const uint8_t *is_first; // [Bt,L] or null
    const float2 *x0;        // [Bt,P] or null
    float2 *x_last;          // forward only, or null
    const float2 *xsaved;    // reverse only: states x [Bt,L,P]
    float2 *partial;         // reverse only: [Bt*nTB, P]
    float2 *dx0;             // reverse only, or null
    ScanDesc *desc;
    uint32_t *ticket;        // per-chain counters, SCAN_TICKET_STRIDE apart (nTB > 1 only)
    uint32_t *err;           // &WsHeader::err (the magic word follows it)
    int Bt, L, P, pxb, cy, nPX, nTB;
    FastDiv by_chains, by_nPX; int lg_pxb;       // nPX * Bt, nPX; log2 of pxb (set by the launch)
    uint32_t spin_limit;
    unsigned *rowmax_out;    // [Bt*L] or null: atomic maximum of the magnitudes of every token row of `out`, zero on entry
    unsigned *amax_out;      // [ABSMAX_SLOTS] (with rowmax_out): atomic maximum of the magnitudes of `out`, zero on entry
};
hipError_t launch_scan(const ScanArgs &a, bool reverse, hipStream_t s);
// workspace layout of the scan-level entry points: header, ticket counters, descriptors, partial rows
struct ScanOnlyLayout { ScanPlan plan; size_t hdr, ticket, desc, dApart, total; };
int make_scan_layout(int64_t Bt, int64_t L, int64_t P, bool rev, ScanOnlyLayout &o);   // returns an ssm_status
// body of ssm_scan_states (returns an ssm_status); workspace may be any 256-byte aligned device memory
int scan_states_forward(const void *A_bar, void *v, const uint8_t *is_first, const void *x0, int64_t Bt, int64_t L,
                        int64_t P, void *x_last, void *workspace, size_t ws_bytes, hipStream_t s);
uint32_t scan_spin_limit();
uint32_t scan_set_spin_limit(uint32_t polls);
// zeroes the header and `scratch_bytes` (a multiple of 16) of ticket counters + descriptors
hipError_t launch_clear(WsHeader *hdr, void *scratch, size_t scratch_bytes, hipStream_t s);
// out[p] = sum_i partial[i*P + p]
hipError_t launch_reduce_partials(const float2 *partial, int64_t n, int64_t P, float2 *out, hipStream_t s);

// ---------------------------------------------------------------------------------------------
// Parameter-sized kernels
// ---------------------------------------------------------------------------------------------
struct ColDotArgs {          // partial[s][h] = sum over the rows of slab s of a[t,h] * b[t,h]
    const float *a; const float *b; int64_t T; int H; int nslab; float *partial;
};
int coldot_slabs(int64_t T, int planes);

// Weights of one product for the prep launch to split and put into fragment order (see gemm_packed.h):
//   PACK_IN   n = 2p+c, k = h:  Bbar                     (input projection)
//   PACK_OUT  n = h, k = 2p+c:  (Re C, -Im C)             (output projection)
//   PACK_GX   n = 2p+c, k = h:  (Re C, -Im C) transposed  (C^H dy)
//   PACK_DU   n = h, k = 2p+c:  Bbar transposed           (Re(Bbar^H chi))
//   PACK_WN   n = j, k = i:     W[i, j]                   (gate)
//   PACK_WT   n = i, k = j:     W[i, j]                   (adjoint of the gate)
enum PackKind { PACK_IN, PACK_OUT, PACK_GX, PACK_DU, PACK_WN, PACK_WT };
struct PackJob { int kind, N, K, planes; void *frag; int *exp; int block0, nblocks, kparts; };   // the last three set by the launch
void pack_place(PackJob &j, int block0, int threads = 256);     // workgroups that a job takes, from block0 on; three planes: parts that K is shared out in

// Factors of the adjoint of the discretisation of one state, all they need being the parameters: dLambda = conj(a) dAbar + conj(p) dg,
// dlog_delta = Re(conj(m) dAbar + conj(a) dg), dB = conj(g) dBbar.
struct alignas(16) StateAdjoint { double ar, ai, pr, pi, mr, mi; float gr, gi, pad[2]; };

constexpr int PREP_MAX_PACKS = 4;
struct PrepArgs {
    const float2 *Lambda; const float2 *B; const float2 *C; const float *log_delta; const float *W;
    int P, H;
    float2 *lam_bar;         // [P], written by the PACK_IN or the PACK_DU job
    WsHeader *hdr;           // cleared when non-null
    int pack_end[PREP_MAX_PACKS]; int npack;     // first workgroup behind every job (set by launch_prep); jobs: at least one
    PackJob pack[PREP_MAX_PACKS];
    StateAdjoint *adj; int adj_blocks;           // [P] or null (gradient pass); its workgroups, the first of the grid (set by launch_prep)
    ColDotArgs cd;           // cd.partial non-null: the launch also computes the column-dot slabs
    int cd_block0, cd_colblocks;                 // set by launch_prep
    struct Zero { uint4 *p; size_t n16; int block0, nblocks; } zero[2];   // regions to clear in the same launch (block ranges set by it)
    // largest magnitudes for the two-plane fp16 staging of the products (all may be null):
    unsigned *cd_amax, *cd_bmax;   // [cd.nslab * ceil(cd.H/64)]: of the pieces of cd.a and cd.b
    unsigned *cd_arow;       // [ceil(cd.H/64)][cd.T]: of every row of cd.a within a block of 64 columns
    struct Pass { const float *x; size_t n; unsigned *slots; int nblocks, block0, vec, rowlen; } pass;
                             // rowlen == 0: slots[nblocks] of nblocks pieces of x[n]; rowlen > 0: slots[n / rowlen],
                             // one per row of rowlen values; block0 and vec set by launch_prep
};
constexpr int PREP_PASS_BLOCKS = 256;        // pieces of a pass that measures one maximum per piece
constexpr int PREP_ROW_PASS_BLOCKS = 1024;   // workgroups of a pass that measures one maximum per row
hipError_t launch_prep(const PrepArgs &a, hipStream_t s);
// ssm_discretize: Abar [P] and, when asked, Bbar [P, H] as interleaved complex
hipError_t launch_discretize(const float2 *Lambda, const float2 *B, const float *log_delta, int P, int H, float2 *lam_bar, float2 *Bbar,
                             hipStream_t s);

// The forward pass of a narrow layer in one launch (narrow.hip).
constexpr int NARROW_MAX = 64;               // columns, states, and steps
struct NarrowFwd {
    const float2 *Lambda, *B, *C; const float *D, *log_delta, *u; const uint8_t *is_first; const float2 *x0;
    float *y; float2 *x, *x_last;            // x, x_last: or null
    float *gelu_y;                           // GELU(y), or null
    WsHeader *hdr;
    int Bt, L, H, P;
    const float *W; PackJob pack;            // the gate's weights, put into fragment order beside it, or null
    int seqs, layer_blocks; FastDiv by_L;    // sequences of a workgroup; workgroups of the layer (set by the launch)
};
// (Its requests take units of four values: rows of at least that many.  Against the other launches of the forward pass 1.2 to 2.8 times as fast.  Up to 512 workgroups, and on
// three planes only: the range in which the errors were compared, not where it stops paying.  Beyond: 128 x 64 tokens, 64, 64 (two planes) 16.0 us and 8.4; 256 x 32: 14.7, 8.5;
// 512 x 64, 32, 32: 22.2, 8.0; 600 x 50, 64, 64 (600 workgroups): 29.3, 22.8; 2000 x 50, 32, 32: 47.4, 25.8.)
inline bool narrow_fwd_shape(int64_t Bt, int64_t L, int64_t H, int64_t P)
{
    return H >= 4 && P >= 2 && H <= NARROW_MAX && P <= NARROW_MAX && L <= NARROW_MAX && (Bt + NARROW_MAX / L - 1) / (NARROW_MAX / L) <= 512;
}
hipError_t launch_narrow_fwd(const NarrowFwd &a, hipStream_t s);

// out[i] = sum of slabs of n values each, in their order; out == nullptr: nothing to sum
struct SlabSum { const float *part; float *out; int64_t n; int slabs; };

struct EpilogueArgs {
    const float2 *B; const StateAdjoint *adj; int P, H;
    const float *dBbar_part; int nsplit_B;   // [nsplit_B][2P][H]
    const float *dC_part; int nsplit_C;      // [nsplit_C][H][2P]  (sum_t dy x_re, sum_t dy x_im)
    const float2 *dAbar_part; int64_t npart; // [npart][P]
    const float *dD_part; int nslab;         // [nslab][H]
    float2 *dLambda; float2 *dB; float2 *dC; float *dD; float *dlog_delta;
    SlabSum also;                            // of another reduction, in the same launch
    int lgB, lgC;                            // set by launch_epilogue
};
hipError_t launch_epilogue(const EpilogueArgs &a, hipStream_t s);
// body of ssm_half_glu_bwd (returns an ssm_status); dW_slabs non-null: the slabs of dW are left to a later launch, which is handed over
int half_glu_backward(const float *u, const float *W, const float *gate, const float *dy, int64_t T, int64_t H, float *du, float *dW,
                      void *workspace, size_t ws_bytes, hipStream_t s, SlabSum *dW_slabs);

}  // namespace ssm
