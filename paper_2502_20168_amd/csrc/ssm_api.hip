// Host side of libssmscan: argument validation, workspace layout and the kernel sequences of
// the forward and the gradient pass.  See include/ssm.h for the contract of every entry point.
#include "../../include/ssm.h"
#include "../../include/ssm_measure.h"
#include "ssm_internal.h"

#include <algorithm>
#include <atomic>
#include <vector>

using namespace ssm;

namespace ssm {

namespace {
constexpr size_t WS_ALIGN = 256;
inline size_t up256(size_t v) { return (v + WS_ALIGN - 1) / WS_ALIGN * WS_ALIGN; }
inline bool off_align(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }
}  // namespace

int make_scan_layout(int64_t Bt, int64_t L, int64_t P, bool rev, ScanOnlyLayout &o)
{
    if (Bt <= 0 || L <= 0 || P <= 0) return SSM_ERR_INVALID_ARG;
    if (P > SSM_MAX_WIDTH) return SSM_ERR_UNSUPPORTED;
    if (Bt > SSM_MAX_TOKENS || L > SSM_MAX_TOKENS || Bt > SSM_MAX_TOKENS / L) return SSM_ERR_UNSUPPORTED;
    if (Bt * L > SSM_MAX_ELEMS / (2 * P)) return SSM_ERR_UNSUPPORTED;
    o.plan = plan_scan(Bt, L, P, false);
    if (o.plan.nblocks > 0x7fffffffLL) return SSM_ERR_UNSUPPORTED;
    size_t off = 0;
    o.hdr = off; off += up256(sizeof(WsHeader));
    o.ticket = off; off += up256(o.plan.ticket_bytes);
    o.desc = off; off += up256(o.plan.desc_bytes);
    o.dApart = off; if (rev) off += up256(o.plan.partial_elems * 8);
    o.total = off;
    return SSM_OK;
}

// ssm_scan_states on a caller's workspace, or on the built-in scratch of the no-allocation entry point
int scan_states_forward(const void *A_bar, void *v, const uint8_t *is_first, const void *x0, int64_t Bt, int64_t L,
                        int64_t P, void *x_last, void *workspace, size_t ws_bytes, hipStream_t s)
{
    if (!A_bar || !v) return SSM_ERR_INVALID_ARG;
    ScanOnlyLayout lo;
    const int st = make_scan_layout(Bt, L, P, false, lo);
    if (st != SSM_OK) return st;
    if (off_align(A_bar, 8) || off_align(v, 8) || off_align(x0, 8) || off_align(x_last, 8)) return SSM_ERR_INVALID_ARG;
    if (!workspace || off_align(workspace, WS_ALIGN) || ws_bytes < lo.total) return SSM_ERR_WORKSPACE;
    char *ws = static_cast<char *>(workspace);
    WsHeader *hdr = reinterpret_cast<WsHeader *>(ws + lo.hdr);
    ScanDesc *desc = reinterpret_cast<ScanDesc *>(ws + lo.desc);
    if (lo.plan.nTB > 1 &&
        launch_clear(hdr, ws + lo.ticket, lo.desc + up256(lo.plan.desc_bytes) - lo.ticket, s) != hipSuccess)
        return SSM_ERR_HIP;
    ScanArgs sa{};
    sa.in = static_cast<const float2 *>(v); sa.out = static_cast<float2 *>(v);
    sa.lam = static_cast<const float2 *>(A_bar); sa.is_first = is_first;
    sa.x0 = static_cast<const float2 *>(x0); sa.x_last = static_cast<float2 *>(x_last);
    sa.desc = desc; sa.ticket = reinterpret_cast<uint32_t *>(ws + lo.ticket); sa.err = &hdr->err;
    sa.Bt = (int)Bt; sa.L = (int)L; sa.P = (int)P;
    sa.pxb = lo.plan.pxb; sa.cy = lo.plan.cy; sa.nPX = lo.plan.nPX; sa.nTB = lo.plan.nTB;
    sa.spin_limit = scan_spin_limit();
    return launch_scan(sa, false, s) == hipSuccess ? SSM_OK : SSM_ERR_HIP;
}

// upper bound on the polls of one cross-workgroup wait (each poll sleeps ~128 clocks); the only
// process-wide setting of the library, changed through ssm_set_spin_limit (a test hook)
static std::atomic<uint32_t> g_spin_limit{1u << 20};
uint32_t scan_spin_limit() { return g_spin_limit.load(std::memory_order_relaxed); }
uint32_t scan_set_spin_limit(uint32_t polls) { return g_spin_limit.exchange(polls, std::memory_order_relaxed); }

}  // namespace ssm

namespace {

constexpr size_t ALIGN = 256;
inline size_t up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }

// weights of one product in fragment order, and the exponents of their rows (two planes)
struct PackedLayout { size_t frag, exp; int N, K; };
void add_packed(size_t &off, PackedLayout &o, int64_t N, int64_t K, int planes)
{
    o.N = (int)N; o.K = (int)K;
    o.frag = off; off += up(packed_frag_bytes(N, K, planes));
    o.exp = off; off += up((size_t)(N + 31) / 32 * 32 * 4);
}
PackJob pack_job(char *base, const PackedLayout &l, int kind, int planes)
{
    PackJob j{};
    j.kind = kind; j.N = l.N; j.K = l.K; j.planes = planes;
    j.frag = base + l.frag; j.exp = reinterpret_cast<int *>(base + l.exp);
    return j;
}
PackedW packed(const char *base, const PackedLayout &l) { return PackedW{base + l.frag, reinterpret_cast<const int *>(base + l.exp)}; }

struct Layout {
    ScanPlan plan;
    int nslab;
    // slabs of dC = dy^T x and dBbar = chi^T u.  Scanning shapes: both in the launch of Re(Bbar^H chi) (dC waits there for
    // the largest magnitude of the saved states, which the reverse scan records on its way); otherwise dC shares the
    // launch of C^H dy.
    SlabPlan dC, dB;
    // sequences of no whole 128-step pieces, products of more than 64 tiles: two scaled fp16 planes there too, the projections scan the rows of their tiles and
    // record the largest magnitude of every row of x and chi; the scans of sequences of more than 64 tiles in a kernel of their own (which records
    // them with atomics).  The prep launch measures the rest
    bool planes2_unfused;
    int planes;              // per operand of every product
    int row_scan;            // tokens per tile of the input projection and of C^H dy, which scan them (no scan kernel), or 0
    PackedLayout w_in, w_out;          // forward: Bbar and C
    PackedLayout w_gx, w_du;           // gradient pass: both transposed
    size_t hdr, lam, adj, xbuf, chi, ticket, desc, dCpart, dBpart, dApart, dDpart, fdesc, fdesc_bytes, total;
    // largest magnitudes of the operands of the products (shapes whose projections scan their own tiles):
    // amax_atomic: 2 x ABSMAX_SLOTS words gathered with atomics, directly before fdesc so that one range is
    // cleared; amax_slots: PREP_PASS_BLOCKS and 2 x amax_cd words of the passes
    size_t amax_atomic, amax_slots; int amax_cd;
    // per-row maxima of the operands whose rows are tokens: rowmax (u forward: [T]; dy gradient pass: [ceil(H/64), T]) and
    // rowpart [ceil(2P/128), T] (x forward, chi gradient pass: one word per column tile of the scanning projection)
    size_t rowmax, rowpart; int row_parts;
};

ssm_status check_dims(int64_t Bt, int64_t L, int64_t H, int64_t P)
{
    if (Bt <= 0 || L <= 0 || H <= 0 || P <= 0) return SSM_ERR_INVALID_ARG;
    if (H > SSM_MAX_WIDTH || P > SSM_MAX_WIDTH) return SSM_ERR_UNSUPPORTED;
    if (Bt > SSM_MAX_TOKENS || L > SSM_MAX_TOKENS || Bt > SSM_MAX_TOKENS / L) return SSM_ERR_UNSUPPORTED;
    const int64_t w = H > 2 * P ? H : 2 * P;
    if (Bt * L > SSM_MAX_ELEMS / w) return SSM_ERR_UNSUPPORTED;
    return SSM_OK;
}

// rows = false: a scan kernel in the gradient pass on two planes also where C^H dy could scan the rows of its tiles
ssm_status make_layout(int64_t Bt, int64_t L, int64_t H, int64_t P, bool bwd, Layout &o, bool rows = true)
{
    ssm_status st = check_dims(Bt, L, H, P);
    if (st != SSM_OK) return st;
    const size_t T = (size_t)Bt * L;
    // (forward + gradient pass with three planes instead, 20 shapes of H, P >= 512 at 3200 .. 16000 tokens: 17 % slower at
    // 32 x 100 tokens, H = P = 512, 28-56 % at the others.  With a shorter contraction two planes would be faster as well, by
    // 4-29 % from 4800 tokens on (nothing at 32 x 100, H = P = 256); those shapes keep the exact split into three planes,
    // which holds every element to its own last bit whatever else its row or matrix holds)
    const bool fused = gemm_scan_shape_ok(Bt, L, P);
    o.planes2_unfused = !fused && !gemm_small_pair((int64_t)T, 2 * P) && !gemm_small_pair((int64_t)T, H) && H >= 512 && P >= 512;
    o.planes = fused || o.planes2_unfused ? 2 : 3;
    o.row_scan = o.planes == 3 ? gemm_row_scan_rows((int64_t)T, L, P) : o.planes2_unfused && (rows || !bwd) && L <= 64 * ROW_SCAN_MAX_TILES ? 64 : 0;
    o.nslab = coldot_slabs((int64_t)T, o.planes);
    o.plan = plan_scan(Bt, L, P, o.planes2_unfused);
    if (o.plan.nblocks > 0x7fffffffLL) return SSM_ERR_UNSUPPORTED;
    size_t off = 0;
    o.hdr = off; off += up(sizeof(WsHeader));
    o.lam = off; off += up((size_t)P * 8);
    o.ticket = off; if (!o.row_scan) off += up(o.plan.ticket_bytes);       // tickets and descriptors are contiguous
    o.desc = off; if (!o.row_scan) off += up(o.plan.desc_bytes);
    o.adj = o.xbuf = o.chi = o.dCpart = o.dBpart = o.dApart = o.dDpart = o.fdesc = o.fdesc_bytes = 0;
    size_t dA_elems = o.plan.partial_elems;
    o.amax_atomic = o.amax_slots = o.rowmax = o.rowpart = 0; o.amax_cd = o.row_parts = 0;
    if (o.planes2_unfused) {
        o.amax_atomic = off; off += 2 * ABSMAX_SLOTS * 4;            // chi / x (atomic slots of the scan kernels)
        o.row_parts = o.row_scan ? (int)((2 * P + 127) / 128) : 1;
        o.rowpart = off; off += up(T * (size_t)o.row_parts * 4);     // rows of x / chi, directly behind: one range is cleared (scan kernels)
        o.amax_cd = o.nslab * (int)((H + 63) / 64);
        o.amax_slots = off; off += up((size_t)(PREP_PASS_BLOCKS + 2 * o.amax_cd) * 4);
        o.rowmax = off; off += up(T * (size_t)((H + 63) / 64) * 4);
    }
    if (fused) {                                     // tagged words of a projection that scans its own output
        static_assert(ABSMAX_SLOTS * 4 % ALIGN == 0, "the atomic slots and the tagged words are cleared as one range");
        o.amax_atomic = off; off += 2 * ABSMAX_SLOTS * 4;            // chi, then the saved states (gradient pass)
        o.fdesc_bytes = gemm_scan_desc_bytes(Bt, L, P);
        o.fdesc = off; off += up(o.fdesc_bytes);
        o.amax_cd = o.nslab * (int)((H + 63) / 64);
        o.amax_slots = off; off += up((size_t)(PREP_PASS_BLOCKS + 2 * o.amax_cd) * 4);
        o.row_parts = (int)((2 * P + 127) / 128);
        o.rowmax = off; off += up(T * (size_t)((H + 63) / 64) * 4);
        o.rowpart = off; off += up(T * (size_t)o.row_parts * 4);
        const size_t per_tile = (size_t)(Bt * L / gemm_scan_rows(Bt * L, L, P, true)) * P;  // one dAbar row per scanning tile
        if (per_tile > dA_elems) dA_elems = per_tile;
    }
    size_t shared_words = 0;         // in the place of the dBbar slabs, which are written in the launch after the scan
    if (o.row_scan) {
        // (reserved also where a tile holds whole sequences and nothing is handed over, so that a workspace holds shorter sequences as well)
        const size_t words = gemm_row_scan_desc_bytes((int64_t)T, P, o.row_scan);
        if (bwd && o.planes == 2) shared_words = words;
        else { o.fdesc = off; off += up(words); }
        o.fdesc_bytes = o.row_scan % L == 0 ? 0 : words;
        dA_elems = (T + o.row_scan - 1) / o.row_scan * P;
    }
    if (fused) {
        o.dC = o.dB = gemm_plan_slabs(2 * P, H, (int64_t)T, 2, REDUCTION_128x128, 2 * P);
    } else {
        o.dC = gemm_plan_slabs(H, 2 * P, (int64_t)T, 1, reduction_tile(o.planes, gemm_small_pair((int64_t)T, 2 * P)), H);
        o.dB = gemm_plan_slabs(2 * P, H, (int64_t)T, 1, reduction_tile(o.planes, gemm_small_pair((int64_t)T, H)), 2 * P);
    }
    if (!bwd) {
        add_packed(off, o.w_in, 2 * P, H, o.planes);
        add_packed(off, o.w_out, H, 2 * P, o.planes);
        o.xbuf = off; off += up(T * P * 8);
    } else {
        add_packed(off, o.w_gx, 2 * P, H, o.planes);
        add_packed(off, o.w_du, H, 2 * P, o.planes);
        o.chi = off; off += up(T * P * 8);
        o.dCpart = off; off += up((size_t)o.dC.slabs * 2 * P * H * 4);
        o.dBpart = off; off += up(std::max((size_t)o.dB.slabs * 2 * P * H * 4, shared_words));
        if (shared_words) o.fdesc = o.dBpart;
        o.dApart = off; off += up(dA_elems * 8);
        o.dDpart = off; off += up((size_t)o.nslab * H * 4);
        o.adj = off; off += up((size_t)P * sizeof(StateAdjoint));
    }
    o.total = off;
    if (bwd && o.planes2_unfused) {
        // a workspace of the gradient pass holds the forward pass as well, whose row maxima can be more (a word per column tile)
        Layout fwd;
        st = make_layout(Bt, L, H, P, false, fwd);
        if (st != SSM_OK) return st;
        o.total = std::max(o.total, fwd.total);
    }
    if (bwd && o.planes2_unfused && o.row_scan) {
        // (never less than with a scan kernel, so that a workspace holds as many shorter sequences: see gradient_layout)
        Layout kernel;
        st = make_layout(Bt, L, H, P, true, kernel, false);
        if (st != SSM_OK) return st;
        o.total = std::max(o.total, kernel.total);
    }
    return SSM_OK;
}

// The gradient pass in a workspace of ws_bytes.  On two planes the scan of rows takes up to 2.4 % more than a scan kernel, 0.2 % at the median of 1300 shapes (16
// bytes per state and 64 tokens that find no room among the dBbar slabs, 8 of dAbar, a row maximum per 128 columns).  A workspace that holds the scan kernel's form only, say
// one of 24 x 4096 steps, 512, 512, whose caller goes on with 24 x 4095, runs that: 60 x 100 tokens, 512, 512: 136 us instead of 121.
ssm_status gradient_layout(int64_t Bt, int64_t L, int64_t H, int64_t P, size_t ws_bytes, Layout &o)
{
    const ssm_status st = make_layout(Bt, L, H, P, true, o);
    return st == SSM_OK && ws_bytes < o.total && o.planes2_unfused && o.row_scan ? make_layout(Bt, L, H, P, true, o, false) : st;
}

// pieces of the pass that measures the largest magnitude of n floats (each workgroup takes whole
// rounds of 512 float4 units)
inline int pass_pieces(size_t n)
{
    const size_t rounds = (n / 4 + 512 * 4 - 1) / (512 * 4);
    return (int)(rounds < 1 ? 1 : (rounds > (size_t)PREP_PASS_BLOCKS ? (size_t)PREP_PASS_BLOCKS : rounds));
}

// workgroups of the pass that measures the largest magnitude of every row: a row per wavefront (four
// wavefronts per workgroup) while that stays within the limit, else four rows per wavefront at a time
inline int row_pass_blocks(size_t rows)
{
    const size_t b = (rows + 3) / 4;
    return (int)(b < 1 ? 1 : (b > (size_t)PREP_ROW_PASS_BLOCKS ? (size_t)PREP_ROW_PASS_BLOCKS : b));
}

inline bool misaligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) & (a - 1)) != 0; }

inline uint32_t spin_limit() { return scan_spin_limit(); }

// Records an event on the stream around every stage when timing is requested.
struct StageTimer {
    hipStream_t s;
    std::vector<hipEvent_t> ev;
    bool ok = true;
    explicit StageTimer(hipStream_t st) : s(st) {}
    void mark()
    {
        hipEvent_t e;
        if (hipEventCreate(&e) != hipSuccess) { ok = false; return; }
        if (hipEventRecord(e, s) != hipSuccess) ok = false;
        ev.push_back(e);
    }
    bool finish(float *ms, int n)
    {
        if (hipStreamSynchronize(s) != hipSuccess) ok = false;
        for (int i = 0; i < n; ++i) {
            ms[i] = 0.f;
            if (ok && i + 1 < (int)ev.size() && hipEventElapsedTime(&ms[i], ev[i], ev[i + 1]) != hipSuccess) ok = false;
        }
        for (hipEvent_t e : ev) (void)hipEventDestroy(e);
        ev.clear();
        return ok;
    }
};
#define MARK() do { if (timer) timer->mark(); } while (0)
#define HIP_TRY(expr) do { if ((expr) != hipSuccess) return SSM_ERR_HIP; } while (0)

// What a pass needs cleared, in its prep launch: the words that gather maxima with atomics and, directly behind them, the
// tagged words of the scanning projections or the row maxima of the recording scan kernels; the ticket counters and
// descriptors of scan kernels with several workgroups along time.
void zero_ranges(PrepArgs &pa, const Layout &lo, char *ws, bool fused, size_t T)
{
    if (lo.planes == 2 && !lo.row_scan) {
        pa.zero[0].p = reinterpret_cast<uint4 *>(ws + lo.amax_atomic);
        pa.zero[0].n16 = (2 * ABSMAX_SLOTS * 4 + (fused ? lo.fdesc_bytes : up(T * 4))) / 16;
    }
    if (lo.row_scan) {
        pa.zero[0].p = reinterpret_cast<uint4 *>(ws + lo.fdesc);
        pa.zero[0].n16 = lo.fdesc_bytes / 16;
        if (lo.planes == 2 && lo.chi) {                  // the gradient pass: the largest magnitude of chi
            pa.zero[1].p = reinterpret_cast<uint4 *>(ws + lo.amax_atomic);
            pa.zero[1].n16 = ABSMAX_SLOTS * 4 / 16;
        }
    }
    if (!fused && !lo.row_scan && lo.plan.nTB > 1) {
        pa.zero[1].p = reinterpret_cast<uint4 *>(ws + lo.ticket);
        pa.zero[1].n16 = (lo.desc + up(lo.plan.desc_bytes) - lo.ticket) / 16;
    }
}

// a narrow layer over short sequences
inline bool fwd_is_one_launch(const Layout &lo, int64_t Bt, int64_t L, int64_t H, int64_t P) { return lo.planes == 3 && narrow_fwd_shape(Bt, L, H, P); }

// The S5 block: the layer's forward pass prepares the gate's product on its way -- W goes into fragment order in the
// prep launch, and with two planes the rows of GELU(y) are measured where the output projection stores it.
struct GatePrep { unsigned *x1_rowmax; const float *W; PackJob w; };

ssm_status run_fwd(const ssm_c64 *Lambda, const ssm_c64 *B, const ssm_c64 *C, const float *D,
                   const float *log_delta, const float *u, const uint8_t *is_first, const ssm_c64 *x0,
                   int64_t Bt, int64_t L, int64_t H, int64_t P, float *y, ssm_c64 *x, ssm_c64 *x_last,
                   void *workspace, size_t ws_bytes, hipStream_t s, StageTimer *timer, float *gelu_y = nullptr,
                   const GatePrep *gate = nullptr)
{
    if (!Lambda || !B || !C || !D || !log_delta || !u || !y) return SSM_ERR_INVALID_ARG;
    Layout lo;
    ssm_status st = make_layout(Bt, L, H, P, false, lo);
    if (st != SSM_OK) return st;
    if (misaligned(Lambda, 8) || misaligned(B, 8) || misaligned(C, 8) || misaligned(D, 4) ||
        misaligned(log_delta, 4) || misaligned(u, 4) || misaligned(y, 4) || misaligned(x, 8) ||
        misaligned(x0, 8) || misaligned(x_last, 8))
        return SSM_ERR_INVALID_ARG;
    if (!workspace || misaligned(workspace, ALIGN) || ws_bytes < lo.total) return SSM_ERR_WORKSPACE;

    char *ws = static_cast<char *>(workspace);
    WsHeader *hdr = reinterpret_cast<WsHeader *>(ws + lo.hdr);
    float2 *lam = reinterpret_cast<float2 *>(ws + lo.lam);
    ScanDesc *desc = reinterpret_cast<ScanDesc *>(ws + lo.desc);
    float2 *xs = x ? reinterpret_cast<float2 *>(x) : reinterpret_cast<float2 *>(ws + lo.xbuf);
    const int T = (int)(Bt * L);

    if (fwd_is_one_launch(lo, Bt, L, H, P)) {
        MARK();
        NarrowFwd n{};
        n.Lambda = reinterpret_cast<const float2 *>(Lambda); n.B = reinterpret_cast<const float2 *>(B); n.C = reinterpret_cast<const float2 *>(C);
        n.D = D; n.log_delta = log_delta; n.u = u; n.is_first = is_first; n.x0 = reinterpret_cast<const float2 *>(x0);
        n.y = y; n.x = reinterpret_cast<float2 *>(x); n.x_last = reinterpret_cast<float2 *>(x_last); n.gelu_y = gelu_y; n.hdr = hdr;
        n.Bt = (int)Bt; n.L = (int)L; n.H = (int)H; n.P = (int)P;
        if (gate) { n.W = gate->W; n.pack = gate->w; }
        HIP_TRY(launch_narrow_fwd(n, s));
        for (int i = 0; i < SSM_FWD_STAGES; ++i) MARK();
        return SSM_OK;
    }

    // Two planes, sequences of whole 128-step pieces (fused), and sequences of other lengths (lo.row_scan): the input projection scans its own
    // output tile and stores the states directly (no scan kernel, Bbar u never goes to memory).
    const bool fused = gemm_scan_shape_ok(Bt, L, P);
    MARK();
    PrepArgs pa{};
    pa.Lambda = reinterpret_cast<const float2 *>(Lambda); pa.B = reinterpret_cast<const float2 *>(B);
    pa.C = reinterpret_cast<const float2 *>(C); pa.log_delta = log_delta;
    pa.P = (int)P; pa.H = (int)H; pa.lam_bar = lam; pa.hdr = hdr;
    pa.pack[0] = pack_job(ws, lo.w_in, PACK_IN, lo.planes);
    pa.pack[1] = pack_job(ws, lo.w_out, PACK_OUT, lo.planes);
    pa.npack = 2;
    zero_ranges(pa, lo, ws, fused, (size_t)T);
    // two scaled fp16 planes per operand: every operand of the two products brings its largest magnitude
    const bool two_planes = lo.planes == 2;
    unsigned *rowmax = reinterpret_cast<unsigned *>(ws + lo.rowmax), *rowpart = reinterpret_cast<unsigned *>(ws + lo.rowpart);
    if (two_planes) {
        // u and x enter their products with tokens as rows: every token gets its own scale
        pa.pass.x = u; pa.pass.n = (size_t)T * H; pa.pass.slots = rowmax; pa.pass.rowlen = (int)H;
        pa.pass.nblocks = row_pass_blocks((size_t)T);
    }
    if (gate) { pa.W = gate->W; pa.pack[pa.npack++] = gate->w; }
    HIP_TRY(launch_prep(pa, s));
    MARK();

    // v[t, 2p+c] = sum_h u[t,h] * Bbar_ri[2p+c, h]      (second scan-element component, Eq. 6)
    GemmArgs g1{};
    g1.A = u; g1.lda = H; g1.w = packed(ws, lo.w_in); g1.planes = lo.planes;
    g1.C = reinterpret_cast<float *>(xs); g1.ldc = 2 * P;
    g1.M = T; g1.N = (int)(2 * P); g1.K = (int)H;
    if (two_planes) g1.amaxA = AbsMax{nullptr, 0, rowmax, 1, T};
    if (fused || lo.row_scan) {
        g1.epilogue = fused || !two_planes ? 7 : 9;
        g1.scan.lam = lam; g1.scan.is_first = is_first;
        g1.scan.x0 = reinterpret_cast<const float2 *>(x0); g1.scan.x_last = reinterpret_cast<float2 *>(x_last);
        g1.scan.desc = reinterpret_cast<unsigned long long *>(ws + lo.fdesc); g1.scan.err = &hdr->err;
        g1.scan.L = (int)L; g1.scan.P = (int)P;
        g1.scan.rows = fused ? gemm_scan_rows(T, L, P, false) : lo.row_scan; g1.scan.spin_limit = fused ? spin_limit() : std::min(spin_limit(), ROW_SCAN_POLLS);
        if (two_planes) g1.scan.rowmax_out = rowpart;        // of the states, for the output projection
    }
    HIP_TRY(launch_product(g1, s));
    MARK();

    if (!fused && !lo.row_scan) {
        ScanArgs sa{};
        sa.in = xs; sa.out = xs; sa.lam = lam; sa.is_first = is_first;
        sa.x0 = reinterpret_cast<const float2 *>(x0); sa.x_last = reinterpret_cast<float2 *>(x_last);
        sa.desc = desc; sa.ticket = reinterpret_cast<uint32_t *>(ws + lo.ticket); sa.err = &hdr->err;
        sa.Bt = (int)Bt; sa.L = (int)L; sa.P = (int)P;
        sa.pxb = lo.plan.pxb; sa.cy = lo.plan.cy; sa.nPX = lo.plan.nPX; sa.nTB = lo.plan.nTB;
        sa.spin_limit = spin_limit();
        if (two_planes) {                                    // rows of the states, for the output projection
            sa.rowmax_out = rowpart;
            sa.amax_out = reinterpret_cast<unsigned *>(ws + lo.amax_atomic) + ABSMAX_SLOTS;
        }
        HIP_TRY(launch_scan(sa, false, s));
    }
    MARK();

    // y[t,h] = sum_p (Re C[h,p] x_re - Im C[h,p] x_im) + D[h] u[t,h]       (Eq. 3, second line)
    GemmArgs g2{};
    g2.A = reinterpret_cast<const float *>(xs); g2.lda = 2 * P; g2.w = packed(ws, lo.w_out); g2.planes = lo.planes;
    g2.M = T; g2.N = (int)H; g2.K = (int)(2 * P);
    if (two_planes) g2.amaxA = AbsMax{nullptr, 0, rowpart, lo.row_parts, T};
    g2.C = y; g2.ldc = H; g2.diag = D; g2.E = u; g2.lde = H; g2.epilogue = 1;
    if (gelu_y) { g2.epilogue = 6; g2.C2 = gelu_y; }       // the S5 block: GELU(y) for the gate, same store
    if (gelu_y && gate) g2.c2_rowmax = gate->x1_rowmax;
    HIP_TRY(launch_product(g2, s));
    MARK();
    return SSM_OK;
}

ssm_status run_bwd(const ssm_c64 *Lambda, const ssm_c64 *B, const ssm_c64 *C, const float *D,
                   const float *log_delta, const float *u, const uint8_t *is_first, const ssm_c64 *x0,
                   int64_t Bt, int64_t L, int64_t H, int64_t P, const ssm_c64 *x, const float *dy,
                   float *du, ssm_c64 *dLambda, ssm_c64 *dB, ssm_c64 *dC, float *dD, float *dlog_delta,
                   ssm_c64 *dx0, void *workspace, size_t ws_bytes, hipStream_t s, StageTimer *timer, const SlabSum &also = {})
{
    if (!Lambda || !B || !C || !D || !log_delta || !u || !x || !dy || !du || !dLambda || !dB || !dC ||
        !dD || !dlog_delta)
        return SSM_ERR_INVALID_ARG;
    Layout lo;
    ssm_status st = gradient_layout(Bt, L, H, P, ws_bytes, lo);
    if (st != SSM_OK) return st;
    if (misaligned(Lambda, 8) || misaligned(B, 8) || misaligned(C, 8) || misaligned(D, 4) ||
        misaligned(log_delta, 4) || misaligned(u, 4) || misaligned(x, 8) || misaligned(dy, 4) ||
        misaligned(du, 4) || misaligned(dLambda, 8) || misaligned(dB, 8) || misaligned(dC, 8) ||
        misaligned(dD, 4) || misaligned(dlog_delta, 4) || misaligned(dx0, 8) || misaligned(x0, 8))
        return SSM_ERR_INVALID_ARG;
    if (!workspace || misaligned(workspace, ALIGN) || ws_bytes < lo.total) return SSM_ERR_WORKSPACE;

    char *ws = static_cast<char *>(workspace);
    WsHeader *hdr = reinterpret_cast<WsHeader *>(ws + lo.hdr);
    float2 *lam = reinterpret_cast<float2 *>(ws + lo.lam);
    ScanDesc *desc = reinterpret_cast<ScanDesc *>(ws + lo.desc);
    float2 *chi = reinterpret_cast<float2 *>(ws + lo.chi);
    float *dCpart = reinterpret_cast<float *>(ws + lo.dCpart);
    float *dBpart = reinterpret_cast<float *>(ws + lo.dBpart);
    float2 *dApart = reinterpret_cast<float2 *>(ws + lo.dApart);
    float *dDpart = reinterpret_cast<float *>(ws + lo.dDpart);
    const int T = (int)(Bt * L);
    const float *xf = reinterpret_cast<const float *>(x);

    // The same shapes, and other lengths (lo.row_scan): C^H dy runs the reverse scan on its own output tile (chi stored directly, dAbar rows per tile, no scan kernel).
    const bool fused = gemm_scan_shape_ok(Bt, L, P);
    MARK();
    PrepArgs pa{};
    pa.Lambda = reinterpret_cast<const float2 *>(Lambda); pa.B = reinterpret_cast<const float2 *>(B);
    pa.C = reinterpret_cast<const float2 *>(C); pa.log_delta = log_delta;
    pa.P = (int)P; pa.H = (int)H; pa.lam_bar = lam; pa.hdr = hdr;
    pa.pack[0] = pack_job(ws, lo.w_du, PACK_DU, lo.planes);
    pa.pack[1] = pack_job(ws, lo.w_gx, PACK_GX, lo.planes);
    pa.npack = 2;
    zero_ranges(pa, lo, ws, fused, (size_t)T);
    pa.adj = reinterpret_cast<StateAdjoint *>(ws + lo.adj);
    // dD slabs: sum_t dy[t,h] u[t,h] over row slabs, in the same launch
    pa.cd.a = dy; pa.cd.b = u; pa.cd.T = T; pa.cd.H = (int)H; pa.cd.nslab = lo.nslab; pa.cd.partial = dDpart;
    // two scaled fp16 planes per operand: dy and u are measured where dD reads them, chi and the saved
    // states where the reverse scan stores / reads them
    const bool two_planes = lo.planes == 2;
    const bool x_pass = lo.planes2_unfused;       // the largest magnitude of the saved states from a pass of the prep launch
    unsigned *am_atomic = reinterpret_cast<unsigned *>(ws + lo.amax_atomic), *am_xsaved = am_atomic + ABSMAX_SLOTS;
    unsigned *am_pass = reinterpret_cast<unsigned *>(ws + lo.amax_slots);
    unsigned *am_dy = am_pass + PREP_PASS_BLOCKS, *am_u = am_dy + lo.amax_cd;
    unsigned *rowmax = reinterpret_cast<unsigned *>(ws + lo.rowmax), *rowpart = reinterpret_cast<unsigned *>(ws + lo.rowpart);
    const int x_pieces = pass_pieces((size_t)T * 2 * P);
    if (two_planes) {
        pa.cd_amax = am_dy; pa.cd_bmax = am_u;
        pa.cd_arow = rowmax;                 // [ceil(H/64)][T]: rows of dy, measured where the dD column dots read it
        if (x_pass) { pa.pass.x = xf; pa.pass.n = (size_t)T * 2 * P; pa.pass.slots = am_pass; pa.pass.nblocks = x_pieces; }
    }
    // dy and chi enter C^H dy and Bbar^H chi with tokens as rows (a scale per token); the sums over tokens
    // (dC, dBbar) take one scale per matrix
    const AbsMax mx_dy{am_dy, lo.amax_cd, nullptr, 0, 0}, mx_u{am_u, lo.amax_cd, nullptr, 0, 0},
                 mx_x{x_pass ? am_pass : am_xsaved, x_pass ? x_pieces : ABSMAX_SLOTS, nullptr, 0, 0},
                 mx_chi{am_atomic, ABSMAX_SLOTS, nullptr, 0, 0},
                 mx_dy_rows{nullptr, 0, rowmax, (int)((H + 63) / 64), T}, mx_chi_rows{nullptr, 0, rowpart, lo.row_parts, T};
    HIP_TRY(launch_prep(pa, s));
    MARK();

    // gx[t, 2p+c] = sum_h dy[t,h] * Cc[h, 2p+c]           (C^H dy_t)
    GemmArgs g3{};
    g3.A = dy; g3.lda = H; g3.w = packed(ws, lo.w_gx); g3.planes = lo.planes;
    g3.C = reinterpret_cast<float *>(chi); g3.ldc = 2 * P;
    g3.M = T; g3.N = (int)(2 * P); g3.K = (int)H;
    // dC slabs: [h, 2p+c] = sum_t dy[t,h] * x[t, 2p+c]
    GemmArgs g4{};
    g4.A = dy; g4.lda = H;
    g4.B = xf; g4.ldb = 2 * P;
    g4.C = dCpart; g4.ldc = 2 * P;
    g4.M = (int)H; g4.N = (int)(2 * P); g4.K = T; g4.splits = lo.dC.slabs;
    if (two_planes) { g3.amaxA = mx_dy_rows; g4.amaxA = mx_dy; g4.amaxB = mx_x; }
    if (fused || lo.row_scan) {
        // the product scans its own tiles; with two planes and fused the dC slabs wait for the next launch, where the largest
        // magnitude of the saved states (recorded here, as the scan reads them) is known
        g3.epilogue = two_planes && !fused ? 10 : 8;
        g3.scan.lam = lam; g3.scan.is_first = is_first;
        g3.scan.x0 = reinterpret_cast<const float2 *>(x0);
        g3.scan.xsaved = reinterpret_cast<const float2 *>(x); g3.scan.partial = dApart;
        g3.scan.dx0 = reinterpret_cast<float2 *>(dx0);
        g3.scan.desc = reinterpret_cast<unsigned long long *>(ws + lo.fdesc); g3.scan.err = &hdr->err;
        g3.scan.L = (int)L; g3.scan.P = (int)P;
        g3.scan.rows = fused ? gemm_scan_rows(T, L, P, true) : lo.row_scan; g3.scan.spin_limit = fused ? spin_limit() : std::min(spin_limit(), ROW_SCAN_POLLS);
        if (two_planes) { g3.scan.amax_out = am_atomic; g3.scan.xmax_out = fused ? am_xsaved : nullptr; g3.scan.rowmax_out = rowpart; }
    }
    // (otherwise dC needs only dy and the saved states: it shares the launch)
    HIP_TRY(fused ? launch_product(g3, s) : launch_products(g3, &g4, nullptr, lo.dC.first, s));
    MARK();

    if (!fused && !lo.row_scan) {
        ScanArgs sa{};
        sa.in = chi; sa.out = chi; sa.lam = lam; sa.is_first = is_first;
        sa.x0 = reinterpret_cast<const float2 *>(x0);
        sa.xsaved = reinterpret_cast<const float2 *>(x); sa.partial = dApart;
        sa.dx0 = reinterpret_cast<float2 *>(dx0);
        sa.desc = desc; sa.ticket = reinterpret_cast<uint32_t *>(ws + lo.ticket); sa.err = &hdr->err;
        sa.Bt = (int)Bt; sa.L = (int)L; sa.P = (int)P;
        sa.pxb = lo.plan.pxb; sa.cy = lo.plan.cy; sa.nPX = lo.plan.nPX; sa.nTB = lo.plan.nTB;
        sa.spin_limit = spin_limit();
        if (two_planes) { sa.rowmax_out = rowpart; sa.amax_out = am_atomic; }      // rows of chi for du, all of chi for dBbar
        HIP_TRY(launch_scan(sa, true, s));
    }
    MARK();

    // du[t,h] = sum_{p,c} chi[t, 2p+c] * Bbar_ri[2p+c, h] + D[h] dy[t,h]      (Re(Bbar^H chi) + D dy)
    GemmArgs g5{};
    g5.A = reinterpret_cast<const float *>(chi); g5.lda = 2 * P; g5.w = packed(ws, lo.w_du); g5.planes = lo.planes;
    g5.C = du; g5.ldc = H; g5.diag = D; g5.E = dy; g5.lde = H; g5.epilogue = 1;
    g5.M = T; g5.N = (int)H; g5.K = (int)(2 * P);
    // dBbar slabs: [2p+c, h] = sum_t chi[t, 2p+c] * u[t,h]   (same launch)
    GemmArgs g6{};
    g6.A = reinterpret_cast<const float *>(chi); g6.lda = 2 * P;
    g6.B = u; g6.ldb = H;
    g6.C = dBpart; g6.ldc = H;
    g6.M = (int)(2 * P); g6.N = (int)H; g6.K = T; g6.splits = lo.dB.slabs;
    if (two_planes) { g5.amaxA = mx_chi_rows; g6.amaxA = mx_chi; g6.amaxB = mx_u; }
    // three products in one launch where the dC slabs had to wait for the largest magnitude of the saved states
    HIP_TRY(launch_products(g5, &g6, fused ? &g4 : nullptr, lo.dB.first, s));
    MARK();
    MARK();

    EpilogueArgs ea{};
    ea.B = reinterpret_cast<const float2 *>(B); ea.adj = pa.adj; ea.P = (int)P; ea.H = (int)H;
    ea.dBbar_part = dBpart; ea.nsplit_B = lo.dB.slabs;
    ea.dC_part = dCpart; ea.nsplit_C = lo.dC.slabs;
    ea.dAbar_part = dApart;
    ea.npart = fused ? Bt * L / gemm_scan_rows(T, L, P, true) : lo.row_scan ? (Bt * L + lo.row_scan - 1) / lo.row_scan : (int64_t)Bt * lo.plan.nTB;
    ea.dD_part = dDpart; ea.nslab = lo.nslab;
    ea.dLambda = reinterpret_cast<float2 *>(dLambda); ea.dB = reinterpret_cast<float2 *>(dB);
    ea.dC = reinterpret_cast<float2 *>(dC); ea.dD = dD; ea.dlog_delta = dlog_delta;
    ea.also = also;
    HIP_TRY(launch_epilogue(ea, s));
    MARK();
    return SSM_OK;
}

}  // namespace

extern "C" {

const char *ssm_strerror(int status)
{
    switch (status) {
    case SSM_OK: return "ok";
    case SSM_ERR_INVALID_ARG: return "invalid argument (null required pointer, non-positive dimension or misaligned array)";
    case SSM_ERR_WORKSPACE: return "workspace missing, misaligned or smaller than ssm_workspace_bytes()";
    case SSM_ERR_UNSUPPORTED: return "dimension beyond the supported limits";
    case SSM_ERR_HIP: return "HIP runtime call or kernel launch failed";
    case SSM_ERR_SCAN_TIMEOUT: return "a bounded cross-workgroup wait in the scan gave up; outputs invalid";
    case SSM_ERR_SCRATCH_LIMIT: return "shape needs more than the built-in scratch of the no-allocation entry point";
    default: return "unknown status";
    }
}

int ssm_version(void) { return 200; }

uint32_t ssm_set_spin_limit(uint32_t polls)
{
    return scan_set_spin_limit(polls);
}

size_t ssm_workspace_bytes(int64_t Bt, int64_t L, int64_t H, int64_t P, int want_bwd)
{
    Layout lo;
    if (make_layout(Bt, L, H, P, want_bwd != 0, lo) != SSM_OK) return 0;
    return lo.total;
}

ssm_status ssm_discretize(const ssm_c64 *Lambda, const ssm_c64 *B, const float *log_delta,
                          int64_t P, int64_t H, ssm_c64 *A_bar, ssm_c64 *B_bar, void *stream)
{
    if (!Lambda || !log_delta || !A_bar || (B_bar && !B)) return SSM_ERR_INVALID_ARG;
    if (P <= 0 || H <= 0) return SSM_ERR_INVALID_ARG;
    if (P > SSM_MAX_WIDTH || H > SSM_MAX_WIDTH) return SSM_ERR_UNSUPPORTED;
    if (misaligned(Lambda, 8) || misaligned(B, 8) || misaligned(log_delta, 4) || misaligned(A_bar, 8) ||
        misaligned(B_bar, 8))
        return SSM_ERR_INVALID_ARG;
    HIP_TRY(launch_discretize(reinterpret_cast<const float2 *>(Lambda), reinterpret_cast<const float2 *>(B), log_delta, (int)P, (int)H,
                              reinterpret_cast<float2 *>(A_bar), reinterpret_cast<float2 *>(B_bar), static_cast<hipStream_t>(stream)));
    return SSM_OK;
}

ssm_status ssm_scan_fwd(const ssm_c64 *Lambda, const ssm_c64 *B, const ssm_c64 *C, const float *D,
                        const float *log_delta, const float *u, const uint8_t *is_first,
                        const ssm_c64 *x0, int64_t Bt, int64_t L, int64_t H, int64_t P,
                        float *y, ssm_c64 *x, ssm_c64 *x_last, void *workspace, size_t ws_bytes, void *stream)
{
    return run_fwd(Lambda, B, C, D, log_delta, u, is_first, x0, Bt, L, H, P, y, x, x_last, workspace,
                   ws_bytes, static_cast<hipStream_t>(stream), nullptr);
}

ssm_status ssm_scan_bwd(const ssm_c64 *Lambda, const ssm_c64 *B, const ssm_c64 *C, const float *D,
                        const float *log_delta, const float *u, const uint8_t *is_first,
                        const ssm_c64 *x0, int64_t Bt, int64_t L, int64_t H, int64_t P,
                        const ssm_c64 *x, const float *dy, float *du, ssm_c64 *dLambda, ssm_c64 *dB,
                        ssm_c64 *dC, float *dD, float *dlog_delta, ssm_c64 *dx0,
                        void *workspace, size_t ws_bytes, void *stream)
{
    return run_bwd(Lambda, B, C, D, log_delta, u, is_first, x0, Bt, L, H, P, x, dy, du, dLambda, dB, dC,
                   dD, dlog_delta, dx0, workspace, ws_bytes, static_cast<hipStream_t>(stream), nullptr);
}

ssm_status ssm_scan_fwd_profiled(const ssm_c64 *Lambda, const ssm_c64 *B, const ssm_c64 *C,
                                 const float *D, const float *log_delta, const float *u,
                                 const uint8_t *is_first, const ssm_c64 *x0,
                                 int64_t Bt, int64_t L, int64_t H, int64_t P,
                                 float *y, ssm_c64 *x, ssm_c64 *x_last,
                                 void *workspace, size_t ws_bytes, void *stream, float *stage_ms)
{
    if (!stage_ms) return SSM_ERR_INVALID_ARG;
    StageTimer timer(static_cast<hipStream_t>(stream));
    ssm_status st = run_fwd(Lambda, B, C, D, log_delta, u, is_first, x0, Bt, L, H, P, y, x, x_last,
                            workspace, ws_bytes, static_cast<hipStream_t>(stream), &timer);
    const bool ok = timer.finish(stage_ms, SSM_FWD_STAGES);
    if (st != SSM_OK) return st;
    return ok ? SSM_OK : SSM_ERR_HIP;
}

ssm_status ssm_scan_bwd_profiled(const ssm_c64 *Lambda, const ssm_c64 *B, const ssm_c64 *C,
                                 const float *D, const float *log_delta, const float *u,
                                 const uint8_t *is_first, const ssm_c64 *x0,
                                 int64_t Bt, int64_t L, int64_t H, int64_t P,
                                 const ssm_c64 *x, const float *dy,
                                 float *du, ssm_c64 *dLambda, ssm_c64 *dB, ssm_c64 *dC, float *dD,
                                 float *dlog_delta, ssm_c64 *dx0,
                                 void *workspace, size_t ws_bytes, void *stream, float *stage_ms)
{
    if (!stage_ms) return SSM_ERR_INVALID_ARG;
    StageTimer timer(static_cast<hipStream_t>(stream));
    ssm_status st = run_bwd(Lambda, B, C, D, log_delta, u, is_first, x0, Bt, L, H, P, x, dy, du, dLambda,
                            dB, dC, dD, dlog_delta, dx0, workspace, ws_bytes,
                            static_cast<hipStream_t>(stream), &timer);
    const bool ok = timer.finish(stage_ms, SSM_BWD_STAGES);
    if (st != SSM_OK) return st;
    return ok ? SSM_OK : SSM_ERR_HIP;
}

ssm_status ssm_plan_describe(int64_t Bt, int64_t L, int64_t H, int64_t P, int32_t *out)
{
    if (!out) return SSM_ERR_INVALID_ARG;
    Layout lo;
    ssm_status st = make_layout(Bt, L, H, P, true, lo);
    if (st != SSM_OK) return st;
    const bool fused = gemm_scan_shape_ok(Bt, L, P);
    const int64_t T = Bt * L;
    out[0] = fused ? 1 : 0;
    out[1] = lo.planes;
    out[2] = lo.dC.slabs; out[3] = lo.dB.slabs;
    out[4] = fused ? 3 : 2;
    out[5] = fused && lo.dB.first;
    out[6] = !fused && lo.dC.first; out[7] = !fused && lo.dB.first;
    // the tiles of the input and the output projection and of du
    GemmArgs in{}, o{}, du{}, dC{}, dB{};
    in.planes = o.planes = du.planes = lo.planes;
    in.M = o.M = du.M = (int)T; in.N = (int)(2 * P); o.N = du.N = (int)H;
    Layout fwd;
    st = make_layout(Bt, L, H, P, false, fwd);
    if (st != SSM_OK) return st;
    in.epilogue = fused ? 7 : fwd.row_scan ? (lo.planes == 2 ? 9 : 7) : 0;
    in.scan.rows = fused ? gemm_scan_rows(T, L, P, false) : fwd.row_scan;
    o.epilogue = du.epilogue = 1;
    dC.M = (int)H; dC.N = (int)(2 * P); dC.splits = lo.dC.slabs;
    dB.M = (int)(2 * P); dB.N = (int)H; dB.splits = lo.dB.slabs;
    const auto tile = [](PkTile t) { return t.rows * 1024 + t.cols; };
    out[8] = tile(product_tile(in, nullptr, nullptr));
    out[9] = tile(product_tile(o, nullptr, nullptr));
    out[10] = tile(product_tile(du, &dB, fused ? &dC : nullptr));
    out[11] = lo.plan.nTB;
    return SSM_OK;
}

ssm_status ssm_plan_launches(int64_t Bt, int64_t L, int64_t H, int64_t P, size_t ws_bytes, int32_t *out)
{
    if (!out) return SSM_ERR_INVALID_ARG;
    const bool fused = gemm_scan_shape_ok(Bt, L, P);
    Layout lo;
    ssm_status st = make_layout(Bt, L, H, P, false, lo);
    if (st != SSM_OK) return st;
    out[0] = fwd_is_one_launch(lo, Bt, L, H, P) ? 1 : fused || lo.row_scan ? 3 : 4;
    st = gradient_layout(Bt, L, H, P, ws_bytes, lo);
    if (st != SSM_OK) return st;
    out[1] = ws_bytes < lo.total ? 0 : fused || lo.row_scan ? 4 : 5;
    return SSM_OK;
}

ssm_status ssm_scan_states(const ssm_c64 *A_bar, ssm_c64 *v, const uint8_t *is_first,
                           const ssm_c64 *x0, int64_t Bt, int64_t L, int64_t P, ssm_c64 *x_last,
                           void *workspace, size_t ws_bytes, void *stream)
{
    return (ssm_status)scan_states_forward(A_bar, v, is_first, x0, Bt, L, P, x_last, workspace, ws_bytes,
                                           static_cast<hipStream_t>(stream));
}

ssm_status ssm_scan_states_reverse(const ssm_c64 *A_bar, ssm_c64 *gx, const ssm_c64 *x,
                                   const uint8_t *is_first, const ssm_c64 *x0,
                                   int64_t Bt, int64_t L, int64_t P, ssm_c64 *dA_bar, ssm_c64 *dx0,
                                   void *workspace, size_t ws_bytes, void *stream)
{
    if (!A_bar || !gx || !x || !dA_bar) return SSM_ERR_INVALID_ARG;
    ScanOnlyLayout lo;
    ssm_status st = (ssm_status)make_scan_layout(Bt, L, P, true, lo);
    if (st != SSM_OK) return st;
    if (misaligned(A_bar, 8) || misaligned(gx, 8) || misaligned(x, 8) || misaligned(x0, 8) ||
        misaligned(dA_bar, 8) || misaligned(dx0, 8))
        return SSM_ERR_INVALID_ARG;
    if (!workspace || misaligned(workspace, ALIGN) || ws_bytes < lo.total) return SSM_ERR_WORKSPACE;
    hipStream_t s = static_cast<hipStream_t>(stream);
    char *ws = static_cast<char *>(workspace);
    WsHeader *hdr = reinterpret_cast<WsHeader *>(ws + lo.hdr);
    ScanDesc *desc = reinterpret_cast<ScanDesc *>(ws + lo.desc);
    float2 *dApart = reinterpret_cast<float2 *>(ws + lo.dApart);
    if (lo.plan.nTB > 1)
        HIP_TRY(launch_clear(hdr, ws + lo.ticket, lo.desc + up(lo.plan.desc_bytes) - lo.ticket, s));
    ScanArgs sa{};
    sa.in = reinterpret_cast<const float2 *>(gx); sa.out = reinterpret_cast<float2 *>(gx);
    sa.lam = reinterpret_cast<const float2 *>(A_bar); sa.is_first = is_first;
    sa.x0 = reinterpret_cast<const float2 *>(x0);
    sa.xsaved = reinterpret_cast<const float2 *>(x); sa.partial = dApart;
    sa.dx0 = reinterpret_cast<float2 *>(dx0);
    sa.desc = desc; sa.ticket = reinterpret_cast<uint32_t *>(ws + lo.ticket); sa.err = &hdr->err;
    sa.Bt = (int)Bt; sa.L = (int)L; sa.P = (int)P;
    sa.pxb = lo.plan.pxb; sa.cy = lo.plan.cy; sa.nPX = lo.plan.nPX; sa.nTB = lo.plan.nTB;
    sa.spin_limit = spin_limit();
    HIP_TRY(launch_scan(sa, true, s));
    HIP_TRY(launch_reduce_partials(dApart, (int64_t)Bt * lo.plan.nTB, P,
                                   reinterpret_cast<float2 *>(dA_bar), s));
    return SSM_OK;
}

namespace {
constexpr int STEP_PLANES = 3;
struct StepPlan { size_t lam, total; PackedLayout in, out, gx, du; };
bool make_step_plan(int64_t H, int64_t P, StepPlan &o)
{
    if (H <= 0 || P <= 0 || H > SSM_MAX_WIDTH || P > SSM_MAX_WIDTH) return false;
    size_t off = 0;
    o.lam = off; off += up((size_t)P * 8);
    add_packed(off, o.in, 2 * P, H, STEP_PLANES);
    add_packed(off, o.out, H, 2 * P, STEP_PLANES);
    add_packed(off, o.gx, 2 * P, H, STEP_PLANES);
    add_packed(off, o.du, H, 2 * P, STEP_PLANES);
    o.total = off;
    return true;
}
}  // namespace

size_t ssm_step_plan_bytes(int64_t H, int64_t P)
{
    StepPlan pl;
    return make_step_plan(H, P, pl) ? pl.total : 0;
}

ssm_status ssm_step_prepare(const ssm_c64 *Lambda, const ssm_c64 *B, const ssm_c64 *C,
                            const float *log_delta, int64_t H, int64_t P,
                            void *plan, size_t plan_bytes, void *stream)
{
    if (!Lambda || !B || !C || !log_delta) return SSM_ERR_INVALID_ARG;
    if (H <= 0 || P <= 0) return SSM_ERR_INVALID_ARG;
    StepPlan pl;
    if (!make_step_plan(H, P, pl)) return SSM_ERR_UNSUPPORTED;
    if (misaligned(Lambda, 8) || misaligned(B, 8) || misaligned(C, 8) || misaligned(log_delta, 4))
        return SSM_ERR_INVALID_ARG;
    if (!plan || misaligned(plan, ALIGN) || plan_bytes < pl.total) return SSM_ERR_WORKSPACE;
    char *pb = static_cast<char *>(plan);
    PrepArgs pa{};
    pa.Lambda = reinterpret_cast<const float2 *>(Lambda); pa.B = reinterpret_cast<const float2 *>(B);
    pa.C = reinterpret_cast<const float2 *>(C); pa.log_delta = log_delta;
    pa.P = (int)P; pa.H = (int)H;
    pa.lam_bar = reinterpret_cast<float2 *>(pb + pl.lam);
    pa.pack[0] = pack_job(pb, pl.du, PACK_DU, STEP_PLANES);
    pa.pack[1] = pack_job(pb, pl.in, PACK_IN, STEP_PLANES);
    pa.pack[2] = pack_job(pb, pl.out, PACK_OUT, STEP_PLANES);
    pa.pack[3] = pack_job(pb, pl.gx, PACK_GX, STEP_PLANES);
    pa.npack = 4;
    HIP_TRY(launch_prep(pa, static_cast<hipStream_t>(stream)));
    return SSM_OK;
}

ssm_status ssm_step(const void *plan, size_t plan_bytes, const float *D, const float *u,
                    const ssm_c64 *x_prev, const uint8_t *is_first, int64_t Bt, int64_t H, int64_t P,
                    ssm_c64 *x, float *y, void *stream)
{
    if (!D || !u || !x || !y) return SSM_ERR_INVALID_ARG;
    ssm_status st = check_dims(Bt, 1, H, P);
    if (st != SSM_OK) return st;
    StepPlan pl;
    if (!make_step_plan(H, P, pl)) return SSM_ERR_UNSUPPORTED;
    if (misaligned(D, 4) || misaligned(u, 4) || misaligned(x_prev, 8) || misaligned(x, 8) || misaligned(y, 4) ||
        (x_prev && x_prev == x))
        return SSM_ERR_INVALID_ARG;
    if (!plan || misaligned(plan, ALIGN) || plan_bytes < pl.total) return SSM_ERR_WORKSPACE;
    const char *pb = static_cast<const char *>(plan);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // x = Bbar u (+ Abar (.) x_prev where the sequence continues)          (Eq. 3, first line)
    GemmArgs g1{};
    g1.A = u; g1.lda = H; g1.w = packed(pb, pl.in); g1.planes = STEP_PLANES;
    g1.C = reinterpret_cast<float *>(x); g1.ldc = 2 * P;
    g1.M = (int)Bt; g1.N = (int)(2 * P); g1.K = (int)H;
    if (x_prev) {
        g1.epilogue = 2;
        g1.diag = reinterpret_cast<const float *>(pb + pl.lam);
        g1.E = reinterpret_cast<const float *>(x_prev); g1.lde = 2 * P;
        g1.rowflag = is_first;
    }
    HIP_TRY(launch_product(g1, s));
    // y = Re(C x) + D (.) u                                                 (Eq. 3, second line)
    GemmArgs g2{};
    g2.A = reinterpret_cast<const float *>(x); g2.lda = 2 * P; g2.w = packed(pb, pl.out); g2.planes = STEP_PLANES;
    g2.C = y; g2.ldc = H; g2.diag = D; g2.E = u; g2.lde = H; g2.epilogue = 1;
    g2.M = (int)Bt; g2.N = (int)H; g2.K = (int)(2 * P);
    HIP_TRY(launch_product(g2, s));
    return SSM_OK;
}

ssm_status ssm_step_bwd(const void *plan, size_t plan_bytes, const float *D, const float *dy,
                        const ssm_c64 *dx, const uint8_t *is_first, int64_t Bt, int64_t H, int64_t P,
                        ssm_c64 *gx, float *du, ssm_c64 *dx_prev, void *stream)
{
    if (!D || !dy || !gx || !du) return SSM_ERR_INVALID_ARG;
    ssm_status st = check_dims(Bt, 1, H, P);
    if (st != SSM_OK) return st;
    StepPlan pl;
    if (!make_step_plan(H, P, pl)) return SSM_ERR_UNSUPPORTED;
    if (misaligned(D, 4) || misaligned(dy, 4) || misaligned(dx, 8) || misaligned(gx, 8) || misaligned(du, 4) ||
        misaligned(dx_prev, 8) || (dx && (dx == gx || dx == dx_prev)) || (dx_prev && dx_prev == gx))
        return SSM_ERR_INVALID_ARG;
    if (!plan || misaligned(plan, ALIGN) || plan_bytes < pl.total) return SSM_ERR_WORKSPACE;
    const char *pb = static_cast<const char *>(plan);
    hipStream_t s = static_cast<hipStream_t>(stream);
    // gx = C^H dy + dx;  dx_prev = [not is_first] conj(Abar) (.) gx
    GemmArgs g1{};
    g1.A = dy; g1.lda = H; g1.w = packed(pb, pl.gx); g1.planes = STEP_PLANES;
    g1.C = reinterpret_cast<float *>(gx); g1.ldc = 2 * P;
    g1.E = reinterpret_cast<const float *>(dx); g1.lde = 2 * P;
    g1.C2 = reinterpret_cast<float *>(dx_prev);
    g1.diag = reinterpret_cast<const float *>(pb + pl.lam); g1.rowflag = is_first; g1.epilogue = 5;
    g1.M = (int)Bt; g1.N = (int)(2 * P); g1.K = (int)H;
    HIP_TRY(launch_product(g1, s));
    // du = Re(Bbar^H gx) + D (.) dy
    GemmArgs g2{};
    g2.A = reinterpret_cast<const float *>(gx); g2.lda = 2 * P; g2.w = packed(pb, pl.du); g2.planes = STEP_PLANES;
    g2.C = du; g2.ldc = H; g2.diag = D; g2.E = dy; g2.lde = H; g2.epilogue = 1;
    g2.M = (int)Bt; g2.N = (int)H; g2.K = (int)(2 * P);
    HIP_TRY(launch_product(g2, s));
    return SSM_OK;
}

namespace {
struct BlockLayout {
    size_t ssm, x1, glu, dypre, total;
    // forward: the gate's W in fragment order; with two planes the rows of GELU(y) in pieces of 128 columns
    int gate_planes, row_parts; PackedLayout w; size_t x1_rowmax;
};
bool make_block_layout(int64_t Bt, int64_t L, int64_t H, int64_t P, bool bwd, BlockLayout &o, bool rows = true)
{
    Layout lo;
    if (make_layout(Bt, L, H, P, bwd, lo, rows) != SSM_OK) return false;
    const size_t TH = up((size_t)Bt * L * H * 4);
    size_t off = 0;
    o.ssm = off; off += up(lo.total);
    o.x1 = o.glu = o.dypre = 0;
    o.gate_planes = gate_two_planes_shape(Bt * L, H) ? 2 : 3; o.row_parts = (int)((H + 127) / 128); o.x1_rowmax = 0;
    if (!bwd) {
        o.x1 = off; off += TH;
        add_packed(off, o.w, H, H, o.gate_planes);
        if (o.gate_planes == 2) { o.x1_rowmax = off; off += up((size_t)o.row_parts * Bt * L * 4); }
    } else {
        const size_t g = ssm_half_glu_workspace_bytes(Bt * L, H, 1);
        if (g == 0) return false;
        o.glu = off; off += up(g);
        o.dypre = off; off += TH;
    }
    o.total = off;
    return true;
}
}  // namespace

size_t ssm_block_workspace_bytes(int64_t Bt, int64_t L, int64_t H, int64_t P, int want_bwd)
{
    BlockLayout bl;
    return make_block_layout(Bt, L, H, P, want_bwd != 0, bl) ? bl.total : 0;
}

ssm_status ssm_block_fwd(const ssm_c64 *Lambda, const ssm_c64 *B, const ssm_c64 *C, const float *D,
                         const float *log_delta, const float *W, const float *u, const uint8_t *is_first,
                         const ssm_c64 *x0, int64_t Bt, int64_t L, int64_t H, int64_t P,
                         float *y, float *out, float *gate, ssm_c64 *x, ssm_c64 *x_last,
                         void *workspace, size_t ws_bytes, void *stream)
{
    if (!W || !out || !y) return SSM_ERR_INVALID_ARG;
    ssm_status st = check_dims(Bt, L, H, P);
    if (st != SSM_OK) return st;
    BlockLayout bl;
    if (!make_block_layout(Bt, L, H, P, false, bl)) return SSM_ERR_UNSUPPORTED;
    if (misaligned(W, 4) || misaligned(out, 4) || misaligned(gate, 4)) return SSM_ERR_INVALID_ARG;
    if (!workspace || misaligned(workspace, ALIGN) || ws_bytes < bl.total) return SSM_ERR_WORKSPACE;
    char *ws = static_cast<char *>(workspace);
    hipStream_t s = static_cast<hipStream_t>(stream);
    float *x1 = reinterpret_cast<float *>(ws + bl.x1);
    // the layer; its output projection also stores x1 = GELU(y)
    GatePrep gp{bl.gate_planes == 2 ? reinterpret_cast<unsigned *>(ws + bl.x1_rowmax) : nullptr, W, pack_job(ws, bl.w, PACK_WN, bl.gate_planes)};
    st = run_fwd(Lambda, B, C, D, log_delta, u, is_first, x0, Bt, L, H, P, y, x, x_last, ws + bl.ssm, bl.x1 - bl.ssm, s,
                 nullptr, x1, &gp);
    if (st != SSM_OK) return st;
    // out[t, j] = y[t, j] sigmoid(sum_i x1[t, i] W[i, j])
    GemmArgs g{};
    g.A = x1; g.lda = H; g.w = packed(ws, bl.w); g.planes = bl.gate_planes;
    g.C = out; g.ldc = H; g.E = y; g.lde = H; g.C2 = gate; g.epilogue = 3;
    g.M = (int)(Bt * L); g.N = (int)H; g.K = (int)H;
    if (bl.gate_planes == 2) g.amaxA = AbsMax{nullptr, 0, gp.x1_rowmax, bl.row_parts, (long)(Bt * L)};
    HIP_TRY(launch_product(g, s));
    return SSM_OK;
}

ssm_status ssm_block_bwd(const ssm_c64 *Lambda, const ssm_c64 *B, const ssm_c64 *C, const float *D,
                         const float *log_delta, const float *W, const float *u, const uint8_t *is_first,
                         const ssm_c64 *x0, int64_t Bt, int64_t L, int64_t H, int64_t P,
                         const ssm_c64 *x, const float *y, const float *gate, const float *dout,
                         float *du, ssm_c64 *dLambda, ssm_c64 *dB, ssm_c64 *dC, float *dD, float *dlog_delta,
                         ssm_c64 *dx0, float *dW, void *workspace, size_t ws_bytes, void *stream)
{
    if (!W || !y || !gate || !dout || !dW) return SSM_ERR_INVALID_ARG;
    ssm_status st = check_dims(Bt, L, H, P);
    if (st != SSM_OK) return st;
    BlockLayout bl;
    if (!make_block_layout(Bt, L, H, P, true, bl)) return SSM_ERR_UNSUPPORTED;
    // (the layer's part may be what its form with a scan kernel takes: see gradient_layout)
    if (ws_bytes < bl.total && !make_block_layout(Bt, L, H, P, true, bl, false)) return SSM_ERR_UNSUPPORTED;
    if (!workspace || misaligned(workspace, ALIGN) || ws_bytes < bl.total) return SSM_ERR_WORKSPACE;
    char *ws = static_cast<char *>(workspace);
    float *dypre = reinterpret_cast<float *>(ws + bl.dypre);
    // the gate's adjoint turns dout into the gradient of the layer's output, then the layer's own pass
    // (whose last launch also sums up the slabs of dW)
    SlabSum dW_slabs{};
    hipStream_t s = static_cast<hipStream_t>(stream);
    st = static_cast<ssm_status>(half_glu_backward(y, W, gate, dout, Bt * L, H, dypre, dW, ws + bl.glu, bl.dypre - bl.glu, s, &dW_slabs));
    if (st != SSM_OK) return st;
    return run_bwd(Lambda, B, C, D, log_delta, u, is_first, x0, Bt, L, H, P, x, dypre, du, dLambda, dB, dC, dD,
                   dlog_delta, dx0, ws + bl.ssm, bl.glu - bl.ssm, s, nullptr, dW_slabs);
}

ssm_status ssm_workspace_status(const void *workspace, void *stream)
{
    if (!workspace) return SSM_ERR_WORKSPACE;
    HIP_TRY(hipStreamSynchronize(static_cast<hipStream_t>(stream)));
    WsHeader h{};
    HIP_TRY(hipMemcpy(&h, workspace, sizeof(h), hipMemcpyDeviceToHost));
    if (h.magic != 0x53534d31u) return SSM_ERR_INVALID_ARG;   // no call has used this workspace
    return h.err ? SSM_ERR_SCAN_TIMEOUT : SSM_OK;
}

}  // extern "C"
