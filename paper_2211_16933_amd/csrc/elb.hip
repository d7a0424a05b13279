// C ABI of the FDLB solver (include/elb.h): context set-up, workspace layout and the
// launch sequence of the RK3 step on gfx950.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <fstream>
#include <initializer_list>
#include <map>
#include <mutex>
#include <sstream>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/elb.h"
#include "closure_kernels.h"
#include "host_math.h"
#include "readout_kernels.h"
#include "stage_table.h"
#include "state_kernels.h"

using namespace elb;

namespace {

const int kSupportedQ[] = {8, 12, 16, 20, 24, 32, 40, 48, 64, 96, 200};

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

struct Layout {
    size_t p, btd, bpd, bpf, sq, rsq, rec, cref, gref, ref, rows, check, oldref, flag, seedb, psi[3], U[3], out, cons, amp;
    // learned closure (params.closure = 1)
    size_t corr, rows5, mparams, mwb, mnorm, pc, proj, outside, sx, sy;
    // chi_RET-FM (params.chi_mode = ELB_CHI_RETFM): ball-average weights
    size_t chiw;
    size_t tables;
    size_t total;
};

// sigma / dx of chi_RET-FM: sigma = E_l l with l = kn kn_length
double fm_ratio(const elb_params *p) { return p->denseness * p->kn * p->kn_length / (p->length / p->nx); }

// dynamic LDS of the chi_RET-FM stage kernel (phase R): weights, densities, chi and ln chi
size_t fm_lds_bytes(int J, int rows) { return sizeof(double) * (size_t)(4 * J + 1 + 3 * rows); }

// half-width J of the ball-average stencil, -1 for chi_SET
int fm_reach(const elb_params *p)
{
    if (p->chi_mode != ELB_CHI_RETFM) return -1;
    double S = fm_ratio(p);
    return S > 0.0 ? (int)std::ceil(S) + 1 : 0;
}

int padded_q(int q) { return (q + 15) / 16 * 16; }

int elem_size(int precision) { return precision == ELB_FP64 ? 8 : 4; }

Layout make_layout(int nx, int Q, int N, int precision, int closure, int chi_reach)
{
    Layout L{};
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align256(o + bytes); return at; };
    L.p = take(sizeof(double) * Q);
    const int QP = padded_q(Q);
    (void)N;
    L.btd = take(sizeof(double) * (size_t)QP * QP);
    L.bpd = take(sizeof(double) * (size_t)QP * QP);
    L.bpf = take(sizeof(float) * (size_t)QP * QP);
    L.sq = take(sizeof(double) * (QP + 2));
    L.rsq = take(sizeof(double) * (QP + 2));
    L.rec = take(sizeof(double) * 2 * QP);
    L.chiw = chi_reach >= 0 ? take(sizeof(double) * (2 * (size_t)chi_reach + 1)) : o;
    L.tables = o;  // up to here uploaded at creation
    // uploaded together when a state is set: reference tables, then the fields n, u, T (and a
    // place for the check of distributions)
    L.cref = take(sizeof(double) * (QP + 3 * (size_t)Q + 3 * (size_t)nx + 1));
    L.gref = L.cref + sizeof(double) * QP;
    L.ref = L.gref + sizeof(double) * Q;
    L.rows = L.ref + sizeof(double) * 2 * Q;
    L.check = take(sizeof(StateCheck) * CHECK_BLOCKS);
    L.oldref = take(sizeof(double) * 2 * Q);
    L.seedb = take(sizeof(unsigned));
    size_t lvl = (size_t)(nx + 2 * NG) * 2 * Q * elem_size(precision);
    for (int s = 0; s < 3; ++s) L.psi[s] = take(lvl);
    size_t ul = precision == ELB_FP32_MIXED ? sizeof(double) * 3 * (size_t)(nx + 2 * NG) : 0;
    for (int s = 0; s < 3; ++s) L.U[s] = take(ul);
    // the moment fields and, right behind them, the failure flag: one copy brings both
    L.out = take(sizeof(double) * (5 * (size_t)nx + 2));
    L.flag = L.out + sizeof(double) * 5 * (size_t)nx;
    L.cons = take(sizeof(double) * 3 * (size_t)nx);
    L.amp = take(sizeof(double) * 3);
    if (closure) {
        L.corr = take((size_t)elem_size(precision) * nx * Q);
        L.rows5 = take(sizeof(double) * 5 * (size_t)(nx + 2 * NG));
        L.mparams = take(sizeof(float) * MLP_PARAMS);
        L.mwb = take(sizeof(unsigned short) * MLP_PARAMS);
        L.mnorm = take(sizeof(float) * MLP_NORM);
        L.pc = take(sizeof(double) * MLP_OUT * MLP_OUT);
        L.proj = take(sizeof(double) * MLP_OUT * MAXQP);
        L.outside = take(sizeof(unsigned long long));
        L.sx = take(sizeof(float) * MLP_IN * (size_t)nx);
        L.sy = take(sizeof(float) * MLP_OUT * (size_t)nx);
    }
    L.total = o;
    return L;
}

// reason of the last failed elb_create, elb_derived or elb_workspace_bytes on this thread
// (none of them leaves a context to hold it)
thread_local std::string g_create_error;

bool q_supported(int q)
{
    for (int v : kSupportedQ)
        if (v == q) return true;
    return false;
}

}  // namespace

// Pinned host memory that the small uploads and downloads of a context (or of a batch, whose
// contexts share one stream) go through: taken piece by piece, given back as a whole once the
// stream has been waited for.  Reserved when the context or batch is created (the first use of a
// new one costs 0.1 to 0.3 ms), at most STAGE_MAX bytes.  What the buffer does not hold as a whole is
// copied directly.  Measured, us per copy with its wait, to the host, directly / through the
// buffer: 16 KB 22 / 15, 64 KB 12 / 13, 256 KB 20 / 20; in two pieces 384 KB 26 / 35, 512 KB 32 / 40.
// The caller's array makes no difference when its pages are mapped, copied before or not; pages
// touched for the first time add 0.15 to 0.25 us per KB on either way.
constexpr size_t STAGE_MIN = size_t(1) << 14, STAGE_MAX = size_t(1) << 18;

// Pinned buffers pass from closed contexts to new ones: freeing one would wait for every stream of
// the device, and contexts are independent.  At most PINNED_MAX bytes are ever taken (64 of the
// largest buffers in use at once); contexts beyond them copy from pageable memory.  The buffers
// that wait for reuse stay until the process ends.
constexpr size_t PINNED_MAX = size_t(1) << 24;
// Before the bytes that are taken piece by piece lies the failure flag that a kernel leaves for the host.
constexpr size_t STAGE_HEAD = 256;

struct PinnedBuffer {
    char *p = nullptr;
    size_t cap = 0;  // without the head
    int device = -1;
};

class PinnedPool {
public:
    // a buffer of at least `cap` bytes for the current device (p == NULL: none)
    PinnedBuffer take(size_t cap)
    {
        PinnedBuffer b;
        if (hipGetDevice(&b.device) != hipSuccess) {
            (void)hipGetLastError();
            return b;
        }
        std::lock_guard<std::mutex> lk(mu_);
        int best = -1;
        for (int i = 0; i < nfree_; ++i)
            if (free_[i].device == b.device && free_[i].cap >= cap && (best < 0 || free_[i].cap < free_[best].cap)) best = i;
        if (best >= 0) {
            b = free_[best];
            free_[best] = free_[--nfree_];
            return b;
        }
        if (taken_ + cap > PINNED_MAX) return b;
        if (hipHostMalloc(reinterpret_cast<void **>(&b.p), STAGE_HEAD + cap, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            b.p = nullptr;
            return b;
        }
        b.cap = cap;
        taken_ += cap;
        std::memset(b.p, 0, STAGE_HEAD + cap);  // first touch
        return b;
    }
    // no enqueued copy or kernel may still use it
    void give(const PinnedBuffer &b)
    {
        std::lock_guard<std::mutex> lk(mu_);
        free_[nfree_++] = b;
    }

private:
    std::mutex mu_;
    PinnedBuffer free_[PINNED_MAX / STAGE_MIN];  // a place for every buffer there can be
    int nfree_ = 0;
    size_t taken_ = 0;
};

// never destroyed: contexts may be closed while the process ends
PinnedPool &pinned_pool()
{
    static PinnedPool *pool = new PinnedPool();
    return *pool;
}

struct HostStage {
    PinnedBuffer buf;
    size_t used = 0;
    // the stream of its copies has been waited for (buf.p = NULL: without success, so that the
    // buffer must not be used again)
    ~HostStage() { if (buf.p) pinned_pool().give(buf); }
    size_t cap() const { return buf.p ? buf.cap : 0; }
    int *flag() const { return reinterpret_cast<int *>(buf.p); }
    // a buffer of `n` bytes within the limits above (none: everything is copied directly)
    void reserve(size_t n)
    {
        size_t want = STAGE_MIN;
        while (want < n && want < STAGE_MAX) want *= 2;
        buf = pinned_pool().take(want);
    }
    // n bytes that no enqueued copy uses; NULL: more than the buffer holds
    char *take(size_t n, hipStream_t st)
    {
        n = align256(n);
        if (n > cap()) return nullptr;
        if (used + n > cap()) {
            if (hipStreamSynchronize(st) != hipSuccess) return nullptr;
            used = 0;
        }
        char *at = buf.p + STAGE_HEAD + used;
        used += n;
        return at;
    }
};

struct elb_ctx {
    elb_params P;
    int Q = 0, N = 0;
    double dx = 0, dt = 0, b = 0, mu_ref = 0, eta0 = 0, chi0 = 0;
    hipStream_t stream = nullptr;
    char *ws = nullptr;
    Layout L{};
    HostStage own_stage;
    HostStage *stage = &own_stage;  // a batch's contexts share the batch's
    std::vector<double> p, w, Btd;
    // deviation storage (FP32): reference state and its per-column distribution
    double n_ref = 0, u_ref = 0, T_ref = 1;
    std::vector<double> ref;     // phi_ref (Q) then theta_ref (Q); zero for FP64 storage
    double ref_sum[6] = {0, 0, 0, 0, 0, 0};
    bool has_state = false;
    bool closure_on = false;     // learned correction applied in every stage
    bool closure_fused = true;   // evaluated inside the stage kernel (else two kernels before it)
    const StageKernel *kernel = nullptr;     // the stage kernel's tile shape for this problem
    const StageKernel *kernel_cl = nullptr;  // and with the learned closure inside (closure = 1)
    int fm_J = -1;               // chi_RET-FM: stencil half-width of the ball average
    std::vector<double> fm_w;    // and its weights
    // a captured chunk of GRAPH_STEPS steps (elb_step), replayed on `stream`; dropped when
    // the captured kernel arguments change (new reference state, closure switched)
    bool use_graph = false;
    hipStream_t cap_stream = nullptr;
    hipGraph_t graph_def = nullptr;
    hipGraphExec_t graph = nullptr;

    ~elb_ctx()
    {
        if (graph) (void)hipGraphExecDestroy(graph);
        if (graph_def) (void)hipGraphDestroy(graph_def);
        if (cap_stream) (void)hipStreamDestroy(cap_stream);
    }
    int64_t steps = 0;
    // stochastic rounding of the FP32 stores: stage launches since the state was set (the
    // stream of launch j is j); while a graph is captured, launches take their offset in the
    // graph and read the base that is set before each replay
    mutable uint32_t launches = 0;
    mutable bool capturing = false;
    mutable uint32_t cap_seed = 0;
    std::string err;

    template <typename T>
    T *dev(size_t off) const { return reinterpret_cast<T *>(ws + off); }
};

namespace {

int fail(elb_ctx *c, int code, const char *fmt, ...)
{
    if (c) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        c->err = buf;
    }
    return code;
}

int hip_check(elb_ctx *c, hipError_t e, const char *what)
{
    if (e != hipSuccess) return fail(c, ELB_EHIP, "%s: %s", what, hipGetErrorString(e));
    return ELB_OK;
}

// Validates p and fills the derived quantities; returns ELB_OK or an error code with a
// message in *msg.
int derive(const elb_params *p, int *N, double *dx, double *dt, double *b, double *mu_ref,
           double *eta0, double *chi0, std::vector<double> *nodes, std::string *msg)
{
    if (!p) { *msg = "params is NULL"; return ELB_EINVAL; }
    if (p->nx < 8) { *msg = "nx must be >= 8"; return ELB_EINVAL; }
    // cell indices, tile starts and grid sizes are 32-bit
    if (p->nx > (1 << 30)) { *msg = "nx must be <= 2^30"; return ELB_EINVAL; }
    if (p->q < 7) { *msg = "q must be >= 7 (Shakhov needs moments up to order 6)"; return ELB_EINVAL; }
    if (!q_supported(p->q)) { *msg = "q not among the compiled values (elb_supported_q)"; return ELB_EUNSUPPORTED; }
    int n = p->n_herm == 0 ? p->q - 1 : p->n_herm;
    if (n < 6 || n > p->q - 1) { *msg = "n_herm must be 0 or in [6, q-1]"; return ELB_EINVAL; }
    if (!(p->length > 0) || !std::isfinite(p->length) || !std::isfinite(p->x0)) { *msg = "length must be finite and > 0"; return ELB_EINVAL; }
    if (!(p->denseness >= 0) || !std::isfinite(p->denseness)) { *msg = "denseness must be finite and >= 0"; return ELB_EINVAL; }
    if (!(p->kn > 0) || !(p->kn_length > 0) || !(p->n_ref > 0) || !std::isfinite(p->kn) ||
        !std::isfinite(p->kn_length) || !std::isfinite(p->n_ref)) { *msg = "kn, kn_length, n_ref must be finite and > 0"; return ELB_EINVAL; }
    // the contact value diverges at eta = 1; E_l(eta=0.49) ~ 127
    if (p->denseness > 100.0) { *msg = "denseness above the range of chi_SET used here"; return ELB_EINVAL; }
    if (p->pr_mode != ELB_PR_CONST && p->pr_mode != ELB_PR_ENSKOG) { *msg = "bad pr_mode"; return ELB_EINVAL; }
    if (p->pr_mode == ELB_PR_CONST && !(p->pr > 0 && p->pr <= 10)) { *msg = "pr must be in (0, 10]"; return ELB_EINVAL; }
    if (p->bc != ELB_BC_PERIODIC && p->bc != ELB_BC_EQUILIBRIUM) { *msg = "bad bc"; return ELB_EINVAL; }
    if (p->precision != ELB_FP64 && p->precision != ELB_FP32 && p->precision != ELB_FP32_MIXED) { *msg = "bad precision"; return ELB_EINVAL; }
    if (p->closure != 0 && p->closure != 1) { *msg = "closure must be 0 or 1"; return ELB_EINVAL; }
    if (p->closure && p->q > MLP_OUT) { *msg = "the learned closure supports q <= 16"; return ELB_EUNSUPPORTED; }
    if (p->chi_mode != ELB_CHI_SET && p->chi_mode != ELB_CHI_RETFM) { *msg = "bad chi_mode"; return ELB_EINVAL; }
    if (p->moment_fixup != 0 && p->moment_fixup != 1) { *msg = "moment_fixup must be 0 or 1"; return ELB_EINVAL; }
    if (p->moment_fixup && p->precision != ELB_FP32_MIXED) { *msg = "moment_fixup needs ELB_FP32_MIXED"; return ELB_EINVAL; }
    if (p->chi_mode == ELB_CHI_RETFM) {
        if (p->closure) { *msg = "the learned closure takes chi_SET only"; return ELB_EUNSUPPORTED; }
        if (!(fm_ratio(p) <= 128.0)) { *msg = "chi_RET-FM needs sigma / dx <= 128"; return ELB_EUNSUPPORTED; }
    }
    if (p->bc == ELB_BC_EQUILIBRIUM) {
        const double *g[2] = {p->ghost_left, p->ghost_right};
        for (auto s : g)
            if (!(s[0] > 0) || !(s[2] > 0) || !std::isfinite(s[0]) || !std::isfinite(s[1]) || !std::isfinite(s[2])) {
                *msg = "ghost states need finite n > 0, T > 0";
                return ELB_EINVAL;
            }
    }
    std::vector<double> pk(p->q);
    if (gauss_hermite_nodes(p->q, pk.data()) != 0) { *msg = "quadrature failed"; return ELB_EINVAL; }
    double pmax = pk.back();
    *N = n;
    *dx = p->length / p->nx;
    if (p->dt > 0) {
        if (!std::isfinite(p->dt)) { *msg = "dt must be finite"; return ELB_EINVAL; }
        *dt = p->dt;
    } else {
        if (!(p->cfl > 0 && p->cfl <= 1.0)) { *msg = "cfl must be in (0, 1] when dt <= 0"; return ELB_EINVAL; }
        *dt = p->cfl * (*dx) / pmax;
    }
    if (*dt * pmax / *dx > 1.0 + 1e-12) { *msg = "dt violates CFL <= 1 for the largest node"; return ELB_EINVAL; }
    map_units(p->denseness, p->kn, p->kn_length, p->n_ref, b, mu_ref, eta0, chi0);
    if (nodes) *nodes = pk;
    return ELB_OK;
}

double host_tau(const elb_ctx *c, double n, double T)
{
    double eta = 0.25 * c->b * n;
    double chi = chi_set(eta);
    double y = c->b * n * chi;
    const double cm = (4.0 / 25.0) * (1.0 + 12.0 / M_PI);
    return c->mu_ref * (1.0 + 0.8 * y + cm * y * y) / (n * chi * std::sqrt(T));
}

// SSP-RK3 weights of level n and of the right-hand side, per stage
const double RK_AN[3] = {0.0, 0.75, 1.0 / 3.0}, RK_AL[3] = {1.0, 0.25, 2.0 / 3.0};

StageTable stage_table(int precision, int fixup)
{
    switch (precision) {
        case ELB_FP64: return stage_table_f64();
        case ELB_FP32: return stage_table_f32();
        default: return fixup ? stage_table_fixup() : stage_table_mixed();
    }
}

// bytes a context uploads to set a state, and downloads as moments; with the learned closure also a
// projection table and a sample, which go through the buffer one after the other
size_t stage_bytes(const elb_params *p)
{
    const size_t nx = p->nx;
    const size_t n = std::max(align256(sizeof(double) * (padded_q(p->q) + 3 * (size_t)p->q + 3 * nx)),
                              align256(sizeof(double) * (5 * nx + 2)));
    if (!p->closure) return n;
    return std::max(n, align256(sizeof(double) * MAXQP * MLP_OUT) + align256(sizeof(float) * MLP_IN * nx) +
                           align256(sizeof(float) * p->q * nx));
}

// The stage kernel of a problem: its first compiled tile whose number of blocks is at most the
// tile's cap (stage_kernels.hip has the caps and what they were measured on).
const StageKernel *pick_stage(const elb_params *p, int ret, int closure)
{
    const StageTable t = stage_table(p->precision, p->moment_fixup);
    for (int i = 0; i < t.stages; ++i) {
        const StageKernel *k = &t.stage[i];
        if (k->q == p->q && k->ret == ret && k->closure == closure && (p->nx + k->cells() - 1) / k->cells() <= k->cap)
            return k;
    }
    return nullptr;  // not reached: the last tile of a Q takes any number of blocks
}

template <typename R>
void launch_stage_t(const elb_ctx *c, int s_in, int s_out, double an, double aL)
{
    StageArgs<R> a{};
    a.psi_s = c->dev<R>(c->L.psi[s_in]);
    a.psi_n = c->dev<R>(c->L.psi[0]);
    a.psi_out = c->dev<R>(c->L.psi[s_out]);
    a.U_s = c->dev<double>(c->L.U[s_in]);
    a.U_n = c->dev<double>(c->L.U[0]);
    a.U_out = c->dev<double>(c->L.U[s_out]);
    a.p = c->dev<double>(c->L.p);
    a.Bt = (sizeof(R) == 8) ? (const R *)c->dev<double>(c->L.bpd) : (const R *)c->dev<float>(c->L.bpf);
    a.cref = c->dev<double>(c->L.cref);
    a.gref = c->dev<double>(c->L.gref);
    a.rec = c->dev<double>(c->L.rec);
    a.w = c->dev<double>(c->L.btd);  // row l = 0 of the Hermite matrix: w_k He_0 = w_k
    a.flag = c->dev<int>(c->L.flag);
    a.nx = c->P.nx;
    a.N = c->N;
    a.periodic = c->P.bc == ELB_BC_PERIODIC;
    a.pr_enskog = c->P.pr_mode == ELB_PR_ENSKOG;
    a.b = c->b;
    a.pr = c->P.pr;
    a.inv_dx = 1.0 / c->dx;
    a.inv_mu = 1.0 / c->mu_ref;
    a.a_n = an;
    a.w_rhs = aL * c->dt;
    a.w_flux = aL * c->dt / (6.0 * c->dx);
    a.T_ref = c->T_ref;
    for (int m = 0; m < 6; ++m) a.ref_sum[m] = c->ref_sum[m];
    const bool fused = c->closure_on && c->closure_fused;
    a.corr = c->closure_on && !fused ? c->dev<R>(c->L.corr) : nullptr;
    if (fused) {
        a.mwb = c->dev<unsigned short>(c->L.mwb);
        a.mparams = c->dev<float>(c->L.mparams);
        a.mnorm = c->dev<float>(c->L.mnorm);
        a.mpc = c->dev<double>(c->L.pc);
        a.cl_denseness = c->P.denseness;
        a.cl_log10kn = std::log10(c->P.kn);
        a.outside = c->dev<unsigned long long>(c->L.outside);
    }
    a.fm_w = c->fm_J >= 0 ? c->dev<double>(c->L.chiw) : nullptr;
    a.fm_J = c->fm_J;
    if (c->capturing) {
        a.seed = c->cap_seed++;
        a.seed_base = c->dev<unsigned>(c->L.seedb);
    } else {
        a.seed = c->launches++;
        a.seed_base = nullptr;
    }
    const StageKernel *k = fused ? c->kernel_cl : c->kernel;
    const int blocks = (c->P.nx + k->cells() - 1) / k->cells();
    k->launch(&a, blocks, k->ret ? fm_lds_bytes(c->fm_J, k->rows) : 0, c->stream);
}

// Moments of every row of level s (ghost or wrapped halo rows included) into rows5.
void launch_closure_rows(const elb_ctx *c, int s)
{
    int nx = c->P.nx, R = nx + 2 * NG;
    const double *U = c->P.precision == ELB_FP32_MIXED ? c->dev<double>(c->L.U[s]) : nullptr;
    int periodic = c->P.bc == ELB_BC_PERIODIC;
    if (c->P.precision == ELB_FP64)
        hipLaunchKernelGGL(k_closure_rows<double>, dim3((R + 255) / 256), dim3(256), 0, c->stream,
                           c->dev<double>(c->L.psi[s]), c->dev<double>(c->L.ref), U, c->dev<double>(c->L.p), nx, c->Q,
                           periodic, c->dev<double>(c->L.rows5));
    else
        hipLaunchKernelGGL(k_closure_rows<float>, dim3((R + 255) / 256), dim3(256), 0, c->stream,
                           c->dev<float>(c->L.psi[s]), c->dev<double>(c->L.ref), U, c->dev<double>(c->L.p), nx, c->Q,
                           periodic, c->dev<double>(c->L.rows5));
}

ClosureConst closure_const(const elb_ctx *c)
{
    ClosureConst cc;
    cc.dx = c->dx;
    cc.b = c->b;
    cc.mu_ref = c->mu_ref;
    cc.denseness = c->P.denseness;
    cc.log10kn = std::log10(c->P.kn);
    return cc;
}

void launch_stage(const elb_ctx *c, int s_in, int s_out, double an, double aL)
{
    if (c->closure_on && !c->closure_fused) {
        // separate form: correction of L[phi] for the stage input, then the stage adds it
        launch_closure_rows(c, s_in);
        int nx = c->P.nx;
        dim3 grid((nx + MLP_ROWS - 1) / MLP_ROWS);
        if (c->P.precision == ELB_FP64)
            hipLaunchKernelGGL(k_closure_apply<double>, grid, dim3(256), 0, c->stream,
                               c->dev<unsigned short>(c->L.mwb), c->dev<float>(c->L.mparams),
                               c->dev<float>(c->L.mnorm), c->dev<double>(c->L.pc), c->dev<double>(c->L.rows5),
                               closure_const(c), nx, c->Q, c->dev<double>(c->L.corr),
                               c->dev<unsigned long long>(c->L.outside));
        else
            hipLaunchKernelGGL(k_closure_apply<float>, grid, dim3(256), 0, c->stream,
                               c->dev<unsigned short>(c->L.mwb), c->dev<float>(c->L.mparams),
                               c->dev<float>(c->L.mnorm), c->dev<double>(c->L.pc), c->dev<double>(c->L.rows5),
                               closure_const(c), nx, c->Q, c->dev<float>(c->L.corr),
                               c->dev<unsigned long long>(c->L.outside));
    }
    if (c->P.precision == ELB_FP64) launch_stage_t<double>(c, s_in, s_out, an, aL);
    else launch_stage_t<float>(c, s_in, s_out, an, aL);
}

// Drops the captured step graph of a context (after draining its stream).
void drop_ctx_graph(elb_ctx *c)
{
    if (!c->graph && !c->graph_def) return;
    (void)hipStreamSynchronize(c->stream);
    if (c->graph) (void)hipGraphExecDestroy(c->graph);
    if (c->graph_def) (void)hipGraphDestroy(c->graph_def);
    c->graph = nullptr;
    c->graph_def = nullptr;
}

// Reference equilibrium of the deviation storage (FP32 modes): the mean state (n_r, u_r,
// T_r) of the given cells; phi_ref_k = n_r g_k(u_r, T_r), theta_ref_k = 2 T_r phi_ref_k, the
// coefficients n_r c_l(u_r, T_r) and the FP64 reference sums.  FP64 storage: all zero.  Writes
// the tables as they are uploaded: cref [QP], gref [Q], ref [2Q].
void make_reference(elb_ctx *c, double n_r, double u_r, double T_r, double *tables)
{
    drop_ctx_graph(c);  // the stage arguments carry the reference sums
    int Q = c->Q, QP = padded_q(Q), N = c->N;
    double *cref = tables, *gref = tables + QP;
    std::fill(tables, tables + QP + 3 * (size_t)Q, 0.0);
    c->ref.assign(2 * Q, 0.0);
    for (int m = 0; m < 6; ++m) c->ref_sum[m] = 0.0;
    c->n_ref = n_r; c->u_ref = u_r; c->T_ref = T_r;
    if (c->P.precision == ELB_FP64) return;
    std::vector<double> cc(QP, 0.0);
    cc[0] = 1.0;
    if (N >= 1) cc[1] = u_r;
    for (int l = 1; l < N; ++l)
        cc[l + 1] = (u_r * cc[l] + (T_r - 1.0) * std::sqrt((double)l) * cc[l - 1]) / std::sqrt((double)(l + 1));
    for (int l = 0; l <= N; ++l) cref[l] = n_r * cc[l];
    for (int l = 0; l <= N; ++l)
        for (int k = 0; k < Q; ++k) gref[k] += c->Btd[(size_t)l * QP + k] * cref[l];
    for (int k = 0; k < Q; ++k) {
        c->ref[k] = gref[k];
        c->ref[Q + k] = 2.0 * T_r * gref[k];
    }
    std::copy(c->ref.begin(), c->ref.end(), tables + QP + Q);
    for (int k = 0; k < Q; ++k) {
        double pk = c->p[k];
        c->ref_sum[0] += c->ref[k];
        c->ref_sum[1] += pk * c->ref[k];
        c->ref_sum[2] += pk * pk * c->ref[k];
        c->ref_sum[3] += pk * pk * pk * c->ref[k];
        c->ref_sum[4] += c->ref[Q + k];
        c->ref_sum[5] += pk * c->ref[Q + k];
    }
}

// A copy between the pinned buffer and the workspace.  Up to 16 KB the runtime copies with a kernel,
// about 3 us in the stream, beyond with a DMA engine, 11 us and more: up to 32 KB go in two pieces
// (two reads of 24 and 16 KB, with the kernel before them and the wait, 27 and 37 us; of 48 and 32 KB in
// pieces 34 and whole 38 us, 96 and 64 KB 74 and 42).
constexpr size_t PINNED_SMALL = size_t(1) << 15;

hipError_t copy_pinned(void *dst, const void *src, size_t bytes, hipMemcpyKind kind, hipStream_t st)
{
    const size_t step = bytes <= PINNED_SMALL ? PINNED_SMALL / 2 : bytes;
    hipError_t e = hipSuccess;
    for (size_t at = 0; at < bytes && e == hipSuccess; at += step)
        e = hipMemcpyAsync((char *)dst + at, (const char *)src + at, std::min(step, bytes - at), kind, st);
    return e;
}

// Copies `bytes` from the host to the workspace in stream order: through the pinned buffer when it
// holds them, else from the caller's memory.  The source may change after the return; with
// wait = false only after the stream has been waited for.
int upload(elb_ctx *c, size_t off, const void *src, size_t bytes, bool wait = true)
{
    char *st = c->stage->take(bytes, c->stream);
    if (st) {
        std::memcpy(st, src, bytes);
        return hip_check(c, copy_pinned(c->dev<char>(off), st, bytes, hipMemcpyHostToDevice, c->stream), "copy to the device");
    }
    hipError_t e = hipMemcpyAsync(c->dev<char>(off), src, bytes, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess && wait) e = hipStreamSynchronize(c->stream);
    return hip_check(c, e, "copy to the device");
}

// Refuses a call whose stream is being captured.  A small state goes up through the pinned buffer
// without a wait, which a capture would take in: the call would report a state that is not set,
// and a replay would upload whatever the buffer holds by then.
int not_captured(elb_ctx *c)
{
    hipStreamCaptureStatus st = hipStreamCaptureStatusNone;
    const int rc = hip_check(c, hipStreamIsCapturing(c->stream, &st), "stream query");
    if (rc) return rc;
    return st == hipStreamCaptureStatusNone ? ELB_OK : fail(c, ELB_EHIP, "a state cannot be set while the stream is captured");
}

// make_reference and its upload.
int set_reference(elb_ctx *c, double n_r, double u_r, double T_r)
{
    std::vector<double> tables(padded_q(c->Q) + 3 * (size_t)c->Q);
    make_reference(c, n_r, u_r, T_r, tables.data());
    return upload(c, c->L.cref, tables.data(), sizeof(double) * tables.size());
}

// Sets level 0 and the ghost rows of every level to the equilibrium of the fields n, u, T held
// in the `rows` buffer, and clears the failure flag.
int init_levels(elb_ctx *c)
{
    InitArgs a{};
    for (int s = 0; s < 3; ++s) {
        a.psi[s] = c->ws + c->L.psi[s];
        a.U[s] = c->P.precision == ELB_FP32_MIXED ? c->dev<double>(c->L.U[s]) : nullptr;
    }
    a.fields = c->dev<double>(c->L.rows);
    a.Bt = c->dev<double>(c->L.btd);
    a.sq = c->dev<double>(c->L.sq);
    a.rsq = c->dev<double>(c->L.rsq);
    a.ref = c->dev<double>(c->L.ref);
    a.flag = c->dev<int>(c->L.flag);
    for (int j = 0; j < 3; ++j) {
        a.ghost[0][j] = c->P.ghost_left[j];
        a.ghost[1][j] = c->P.ghost_right[j];
    }
    a.nx = c->P.nx;
    a.Q = c->Q;
    a.QP = padded_q(c->Q);
    a.N = c->N;
    a.periodic = c->P.bc == ELB_BC_PERIODIC;
    const size_t R = (size_t)c->P.nx + 2 * NG;
    const bool f64 = c->P.precision == ELB_FP64;
    if ((double)R * c->Q * c->N >= INIT_TILES) {
        const int rows = init_rows(c->Q);
        const dim3 grid((unsigned)((R + rows - 1) / rows));
        const size_t lds = sizeof(double) * (size_t)rows * (c->N + 1);
        if (f64) hipLaunchKernelGGL(k_init_tiles<double>, grid, dim3(INIT_THREADS), lds, c->stream, a, rows);
        else hipLaunchKernelGGL(k_init_tiles<float>, grid, dim3(INIT_THREADS), lds, c->stream, a, rows);
    } else {
        const dim3 grid((unsigned)((R * c->Q + INIT_THREADS - 1) / INIT_THREADS));
        if (f64) hipLaunchKernelGGL(k_init_equilibrium<double>, grid, dim3(INIT_THREADS), 0, c->stream, a);
        else hipLaunchKernelGGL(k_init_equilibrium<float>, grid, dim3(INIT_THREADS), 0, c->stream, a);
    }
    return hip_check(c, hipGetLastError(), "init kernel launch");
}

// `o`: n, u, T, q, Pxx [nx] each, in device or pinned memory, then the failure flag.
int run_moments(elb_ctx *c, double *o, bool conserved = false)
{
    const int nx = c->P.nx, Q = c->Q;
    const int threads = 256;
    const double *U = c->P.precision == ELB_FP32_MIXED ? c->dev<double>(c->L.U[0]) : nullptr;
    double *cons = conserved ? c->dev<double>(c->L.cons) : nullptr;
    const int *flag = c->dev<int>(c->L.flag);
    for (int first = 0; first < nx; first += MOM_CELLS) {  // nx <= 2^30
        // MOM_LANES threads per cell
        const unsigned blocks = (unsigned)(((size_t)std::min(nx - first, MOM_CELLS) * MOM_LANES + threads - 1) / threads);
        if (c->P.precision == ELB_FP64)
            hipLaunchKernelGGL(k_moments<double>, dim3(blocks), dim3(threads), 0, c->stream, c->dev<double>(c->L.psi[0]),
                               c->dev<double>(c->L.ref), U, c->dev<double>(c->L.p), nx, Q, first, o, flag, cons);
        else
            hipLaunchKernelGGL(k_moments<float>, dim3(blocks), dim3(threads), 0, c->stream, c->dev<float>(c->L.psi[0]),
                               c->dev<double>(c->L.ref), U, c->dev<double>(c->L.p), nx, Q, first, o, flag, cons);
    }
    return hip_check(c, hipGetLastError(), "moments kernel launch");
}

// Copies pieces of the workspace to the host (dst = NULL: not wanted) and waits for the stream:
// small ones (PINNED_SMALL) through the pinned buffer, as many as it holds with one wait; larger
// ones that it holds through it one by one; others directly.  Larger ones with one wait, or
// through the buffer and directly by turns, were slower: moments of 16384 cells 95 us one by one,
// 102 with two of the five in flight; samples of 2000 cells (96 and 64 KB) 99 and 123.
struct Piece {
    void *dst;
    size_t off, bytes;
};

int download(elb_ctx *c, std::initializer_list<Piece> pieces)
{
    char *st[6] = {};
    hipError_t e = hipSuccess;
    auto wait = [&]() {
        if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
        int i = 0;
        for (const Piece &p : pieces) {
            if (st[i] && e == hipSuccess) std::memcpy(p.dst, st[i], p.bytes);
            st[i++] = nullptr;
        }
        c->stage->used = 0;  // the stream has been waited for
    };
    int i = 0;
    bool pending = false;
    for (const Piece &p : pieces) {
        char *&at = st[i++];
        if (!p.dst || e != hipSuccess) continue;
        const size_t n = align256(p.bytes);
        if (n <= c->stage->cap() && c->stage->used + n > c->stage->cap()) wait();
        if (n <= c->stage->cap()) at = c->stage->take(n, c->stream);
        if (e == hipSuccess)
            e = at ? copy_pinned(at, c->dev<char>(p.off), p.bytes, hipMemcpyDeviceToHost, c->stream)
                   : hipMemcpyAsync(p.dst, c->dev<char>(p.off), p.bytes, hipMemcpyDeviceToHost, c->stream);
        pending = !(at && p.bytes > PINNED_SMALL);
        if (!pending) wait();
    }
    if (pending) wait();
    return hip_check(c, e, "copy to the host");
}

// Offsets of the FP64 planes phi, theta [nx][Q] in the interiors of levels 1 and 2 (FP64 storage:
// both in level 1's), which the next stage writes before anything reads them.
void dist_planes(const elb_ctx *c, size_t at[2])
{
    const size_t skip = (size_t)NG * 2 * c->Q * elem_size(c->P.precision);
    at[0] = c->L.psi[1] + skip;
    at[1] = c->P.precision == ELB_FP64 ? at[0] + sizeof(double) * (size_t)c->P.nx * c->Q : c->L.psi[2] + skip;
}

int flag_status(elb_ctx *c, int flag)
{
    if (flag) return fail(c, ELB_ENONFINITE, "a cell reached n <= 0, T <= 0 or non-finite moments");
    return ELB_OK;
}

int check_flag(elb_ctx *c)
{
    int flag = 0;
    int rc = download(c, {{&flag, c->L.flag, sizeof flag}});
    return rc ? rc : flag_status(c, flag);
}

}  // namespace

extern "C" {

int elb_supported_q(int32_t *out, int32_t cap)
{
    int n = (int)(sizeof kSupportedQ / sizeof kSupportedQ[0]);
    for (int i = 0; i < n && i < cap && out; ++i) out[i] = kSupportedQ[i];
    return n;
}

int elb_quadrature(int32_t q, double *nodes, double *weights)
{
    if (q < 1 || q > 256 || !nodes || !weights) return ELB_EINVAL;
    return gauss_hermite(q, nodes, weights) == 0 ? ELB_OK : ELB_EINVAL;
}

int elb_derived(const elb_params *p, double out[7])
{
    if (!out) return ELB_EINVAL;
    int N;
    double dx, dt, b, mu, eta0, chi0;
    std::string msg;
    int rc = derive(p, &N, &dx, &dt, &b, &mu, &eta0, &chi0, nullptr, &msg);
    if (rc) { g_create_error = msg; return rc; }
    out[0] = dx; out[1] = dt; out[2] = b; out[3] = mu; out[4] = eta0; out[5] = chi0; out[6] = N;
    return ELB_OK;
}

int64_t elb_workspace_bytes(const elb_params *p)
{
    int N;
    double dx, dt, b, mu, eta0, chi0;
    std::string msg;
    if (derive(p, &N, &dx, &dt, &b, &mu, &eta0, &chi0, nullptr, &msg)) { g_create_error = msg; return -1; }
    return (int64_t)make_layout(p->nx, p->q, N, p->precision, p->closure, fm_reach(p)).total;
}

}  // extern "C"

namespace {

// The stage kernel's copy of Bt, packed per MFMA lane (phase C of the stage kernel).  Where the
// projection splits by the parity of l over the positive nodes (in halves of KD):
//   Bp[par][tn][lane][ks] = Bt[2 ((lane / 16) KS + ks) + par][Q/2 + 16 tn + lane % 16],
// otherwise Bp[tn][lane][ks] = Bt[(lane / 16) KS + ks][16 tn + lane % 16] (KD = QP); KS = KD / 4.
// Both fill at most QP x QP values (zero outside the table).
template <typename R>
void pack_projection(const std::vector<double> &Bt, int Q, int elem, R *out)
{
    const int QP = padded_q(Q), QH = Q / 2;
    const bool split = split_projection(Q, elem);
    const int KD = split ? padded_q(QH) : QP, KS = KD / 4, TN = KD / 16, NP = split ? 2 : 1;
    for (int par = 0; par < NP; ++par)
        for (int tn = 0; tn < TN; ++tn)
            for (int ln = 0; ln < 64; ++ln)
                for (int ks = 0; ks < KS; ++ks) {
                    const int kk = ln >> 4, cl = tn * 16 + (ln & 15);
                    const int l = split ? 2 * (kk * KS + ks) + par : kk * KS + ks;
                    const int k = split ? QH + cl : cl;
                    out[(((size_t)par * TN + tn) * 64 + ln) * KS + ks] =
                        (R)(l < QP && k < QP ? Bt[(size_t)l * QP + k] : 0.0);
                }
}

// elb_create; `stage` is the pinned buffer of the batch that the context belongs to, or NULL.
int create_ctx(const elb_params *p, void *dev_workspace, int64_t workspace_bytes, void *hip_stream, HostStage *stage,
               elb_ctx **out)
{
    if (!out) return ELB_EINVAL;
    *out = nullptr;
    g_create_error = "";
    elb_ctx *c = new (std::nothrow) elb_ctx();
    if (!c) { g_create_error = "host allocation failed"; return ELB_ENOMEM; }
    std::string msg;
    int rc = derive(p, &c->N, &c->dx, &c->dt, &c->b, &c->mu_ref, &c->eta0, &c->chi0, &c->p, &msg);
    if (rc) { g_create_error = msg; delete c; return rc; }
    c->P = *p;
    c->Q = p->q;
    c->L = make_layout(p->nx, p->q, c->N, p->precision, p->closure, fm_reach(p));
    if (!dev_workspace || workspace_bytes < (int64_t)c->L.total) { g_create_error = "workspace missing or too small"; delete c; return ELB_ENOMEM; }
    if (((uintptr_t)dev_workspace) & 255) { g_create_error = "workspace not 256-byte aligned"; delete c; return ELB_EINVAL; }
    c->ws = (char *)dev_workspace;
    c->stream = (hipStream_t)hip_stream;
    c->kernel = pick_stage(p, fm_reach(p) >= 0, 0);
    if (p->closure) c->kernel_cl = pick_stage(p, 0, 1);
    int Q = c->Q, N = c->N;
    c->w.resize(Q);
    gauss_hermite(Q, c->p.data(), c->w.data());
    // Bt[l][k] = w_k h_l(p_k), h_l = He_l / sqrt(l!), zero-padded to QP x QP
    const int QP = padded_q(Q);
    c->Btd.assign((size_t)QP * QP, 0.0);
    std::vector<double> h(Q + 2);
    for (int k = 0; k < Q; ++k) {
        hermite_orthonormal(N, c->p[k], h.data());
        for (int l = 0; l <= N; ++l) c->Btd[(size_t)l * QP + k] = c->w[k] * h[l];
    }
    // every table in an image of its part of the workspace, uploaded at once
    std::vector<double> image(c->L.tables / sizeof(double), 0.0);
    auto table = [&](size_t off) { return image.data() + off / sizeof(double); };
    std::copy(c->p.begin(), c->p.end(), table(c->L.p));
    std::copy(c->Btd.begin(), c->Btd.end(), table(c->L.btd));
    pack_projection(c->Btd, Q, sizeof(double), table(c->L.bpd));
    pack_projection(c->Btd, Q, sizeof(float), reinterpret_cast<float *>(table(c->L.bpf)));
    double *sq = table(c->L.sq), *rsq = table(c->L.rsq), *rec = table(c->L.rec);
    for (int l = 0; l < QP + 2; ++l) {
        sq[l] = std::sqrt((double)l);
        rsq[l] = l ? 1.0 / std::sqrt((double)l) : 0.0;
    }
    for (int l = 0; l < QP; ++l) {
        rec[l] = l ? 1.0 / std::sqrt((double)l) : 0.0;
        rec[QP + l] = std::sqrt((double)l / (double)(l + 1));
    }
    if (p->chi_mode == ELB_CHI_RETFM) {
        c->fm_J = fm_weights(fm_ratio(p), c->fm_w);
        std::copy(c->fm_w.begin(), c->fm_w.end(), table(c->L.chiw));
    }
    hipError_t e = hipMemcpyAsync(c->ws, image.data(), c->L.tables, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->dev<int>(c->L.flag), 0, sizeof(int) * 4, c->stream);
    if (e == hipSuccess && p->closure)
        e = hipMemsetAsync(c->dev<unsigned long long>(c->L.outside), 0, sizeof(unsigned long long), c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) {
        g_create_error = std::string("table upload: ") + hipGetErrorString(e);
        delete c;
        return ELB_EHIP;
    }
    if (stage) c->stage = stage;
    else c->own_stage.reserve(stage_bytes(p));
    if (set_reference(c, 1.0, 0.0, 1.0) != ELB_OK) {
        g_create_error = c->err;
        if (hipStreamSynchronize(c->stream) != hipSuccess) c->own_stage.buf.p = nullptr;
        delete c;
        return ELB_EHIP;
    }
    *out = c;
    return ELB_OK;
}

}  // namespace

extern "C" {

int elb_create(const elb_params *p, void *dev_workspace, int64_t workspace_bytes, void *hip_stream, elb_ctx **out)
{
    return create_ctx(p, dev_workspace, workspace_bytes, hip_stream, nullptr, out);
}

int elb_set_state_moments(elb_ctx *c, const double *n, const double *u, const double *T)
{
    if (!c) return ELB_EINVAL;
    if (!n || !u || !T) return fail(c, ELB_EINVAL, "NULL input array");
    if (int rc = not_captured(c)) return rc;
    const int nx = c->P.nx;
    const size_t nb = sizeof(double) * nx, tables = sizeof(double) * (padded_q(c->Q) + 3 * (size_t)c->Q);
    // the reference tables and the fields in one upload; fields too large for the pinned
    // buffer are copied from the caller's arrays
    char *up = c->stage->take(tables + 3 * nb, c->stream);
    const bool staged = up != nullptr;
    if (staged) {
        std::memcpy(up + tables, n, nb);
        std::memcpy(up + tables + nb, u, nb);
        std::memcpy(up + tables + 2 * nb, T, nb);
    }
    const double *src[3] = {n, u, T};
    auto upload_fields = [&]() {
        if (staged)
            return hip_check(c, hipMemcpyAsync(c->dev<char>(c->L.rows), up + tables, 3 * nb, hipMemcpyHostToDevice, c->stream),
                             "rows copy");
        for (int f = 0; f < 3; ++f)
            if (int rc = upload(c, c->L.rows + f * nb, src[f], nb)) return rc;
        return (int)ELB_OK;
    };
    // Every cell is checked, and the smallest tau found, before the state is touched (the
    // `rows` buffer is not part of it): on the host for few cells, on the GPU for many.  The
    // host takes about 15 ns per cell (a square root and two divisions for tau), the GPU about
    // 20 us more of launch and wait.  Meanwhile the host adds up the mean state, whose order
    // of summation fixes the bits of the FP32 modes.
    StateCheck sum{};
    double sn = 0, su = 0, sT = 0;
    auto mean_state = [&]() {
        if (c->P.precision == ELB_FP64) return;  // FP64 storage has no reference state
        double a = 0, b = 0, d = 0;              // (in registers)
        for (int i = 0; i < nx; ++i) { a += n[i]; b += u[i]; d += T[i]; }
        sn = a; su = b; sT = d;
    };
    const bool on_gpu = nx > CHECK_HOST_CELLS;
    if (on_gpu) {
        int rc = upload_fields();
        if (rc) return rc;
        const int blocks = std::min(CHECK_BLOCKS, (nx + CHECK_THREADS - 1) / CHECK_THREADS);
        hipLaunchKernelGGL(k_check_state, dim3(blocks), dim3(CHECK_THREADS), 0, c->stream, c->dev<double>(c->L.rows), nx, c->b,
                           c->mu_ref, c->dev<StateCheck>(c->L.check));
        rc = hip_check(c, hipGetLastError(), "check kernel launch");
        if (rc) return rc;
        mean_state();
        StateCheck part[CHECK_BLOCKS];
        rc = download(c, {{part, c->L.check, sizeof(StateCheck) * blocks}});
        if (rc) return rc;
        sum = part[0];
        for (int i = 1; i < blocks; ++i) sum.add(part[i]);
    } else {
        sum.clear();
        for (int i = 0; i < nx; ++i) sum.cell(i, n[i], u[i], T[i], c->b, c->mu_ref);
        mean_state();
    }
    if (sum.bad < (unsigned)nx && sum.bad <= sum.dense)
        return fail(c, ELB_EINVAL, "cell %u: need finite n > 0, T > 0", sum.bad);
    if (sum.dense < (unsigned)nx) return fail(c, ELB_EINVAL, "cell %u: reduced density eta >= 0.99", sum.dense);
    double min_tau = sum.min_tau;
    if (c->P.bc == ELB_BC_EQUILIBRIUM)
        for (const double *g : {c->P.ghost_left, c->P.ghost_right}) min_tau = std::fmin(min_tau, host_tau(c, g[0], g[2]));
    if (c->dt > 2.5 * min_tau)
        return fail(c, ELB_EINVAL, "dt = %g exceeds the RK3 stability limit 2.5 min tau = %g", c->dt, 2.5 * min_tau);
    const double n_r = sn / nx, u_r = su / nx, T_r = sT / nx;
    int rc;
    if (on_gpu || !staged) {
        rc = set_reference(c, n_r, u_r, T_r);
        if (!rc && !on_gpu) rc = upload_fields();
    } else {
        make_reference(c, n_r, u_r, T_r, reinterpret_cast<double *>(up));
        rc = hip_check(c, hipMemcpyAsync(c->dev<char>(c->L.cref), up, tables + 3 * nb, hipMemcpyHostToDevice, c->stream),
                       "state upload");
    }
    if (!rc) rc = init_levels(c);
    if (rc) return rc;
    c->has_state = true;
    c->steps = 0;
    c->launches = 0;
    return ELB_OK;
}

int elb_set_state_dist(elb_ctx *c, const double *phi, const double *theta)
{
    if (!c) return ELB_EINVAL;
    if (!phi || !theta) return fail(c, ELB_EINVAL, "NULL input array");
    if (int rc = not_captured(c)) return rc;
    const int nx = c->P.nx, Q = c->Q, R = nx + 2 * NG;
    const bool f64 = c->P.precision == ELB_FP64;
    const size_t n = (size_t)nx * Q;
    // the planes into the interiors of levels 1 and 2; nothing else changes before they pass
    size_t at[2];
    dist_planes(c, at);
    int rc = upload(c, at[0], phi, sizeof(double) * n, false);
    if (!rc) rc = upload(c, at[1], theta, sizeof(double) * n, false);
    double *dphi = c->dev<double>(at[0]), *dtheta = c->dev<double>(at[1]);
    // behind the cells' sums, so that one copy brings both
    const size_t bad_at = c->L.rows + sizeof(double) * 3 * nx;
    int *bad = c->dev<int>(bad_at), nonfinite = 0;
    if (!rc) rc = hip_check(c, hipMemsetAsync(bad, 0, sizeof(int), c->stream), "check reset");
    if (rc) {
        (void)hipStreamSynchronize(c->stream);  // the planes may still be read
        return rc;
    }
    double mean[3] = {};
    if (f64) {
        // theta follows phi
        hipLaunchKernelGGL(k_all_finite, dim3((unsigned)std::min<size_t>(2048, (2 * n + 255) / 256)), dim3(256), 0, c->stream,
                           (const double *)dphi, 2 * n, bad);
        rc = download(c, {{&nonfinite, bad_at, sizeof nonfinite}});
        if (!rc) rc = hip_check(c, hipGetLastError(), "check kernel launch");
        if (rc) return rc;
        if (nonfinite) return fail(c, ELB_EINVAL, "non-finite distribution value");
    } else {
        // reference of the deviation storage: mean primitive state of the given cells, whose sum
        // runs over the cells in order
        hipLaunchKernelGGL(k_dist_sums, dim3((nx + SUM_CELLS - 1) / SUM_CELLS), dim3(SUM_CELLS), 0, c->stream,
                           (const double *)dphi, (const double *)dtheta, c->dev<double>(c->L.p), nx, Q, c->dev<double>(c->L.rows), bad);
        std::vector<double> f(3 * (size_t)nx + 1);
        rc = download(c, {{f.data(), c->L.rows, sizeof(double) * f.size()}});
        if (!rc) rc = hip_check(c, hipGetLastError(), "sum kernel launch");
        if (rc) return rc;
        std::memcpy(&nonfinite, &f[3 * (size_t)nx], sizeof nonfinite);
        if (nonfinite) return fail(c, ELB_EINVAL, "non-finite distribution value");
        double sn = 0, su = 0, sT = 0;
        for (int i = 0; i < nx; ++i) { sn += f[i]; su += f[(size_t)nx + i]; sT += f[2 * (size_t)nx + i]; }
        if (!(sn > 0) || !(sT > 0) || !std::isfinite(su)) return fail(c, ELB_EINVAL, "distributions with non-positive mean density or temperature");
        mean[0] = sn / nx; mean[1] = su / nx; mean[2] = sT / nx;
    }
    // the values are taken from here on
    if (!c->has_state && c->P.bc == ELB_BC_EQUILIBRIUM) {
        // ghost rows need the equilibrium of the end states: set them from a uniform state
        // first (which leaves the interiors of levels 1 and 2, and with them the planes, alone)
        std::vector<double> gn(nx, c->P.ghost_left[0]), gu(nx, c->P.ghost_left[1]), gT(nx, c->P.ghost_left[2]);
        rc = elb_set_state_moments(c, gn.data(), gu.data(), gT.data());
        if (rc) return rc;
    }
    if (!f64) {
        const std::vector<double> old_ref = c->ref;
        rc = set_reference(c, mean[0], mean[1], mean[2]);
        if (!rc) rc = upload(c, c->L.oldref, old_ref.data(), sizeof(double) * old_ref.size());
        if (rc) return rc;
    }
    // ghost rows (kept from the current state) move to the new reference
    const dim3 grid = plane_grid((size_t)R * Q);
    if (f64)
        hipLaunchKernelGGL(k_dist_pack<double>, grid, dim3(PLANE_THREADS), 0, c->stream, (const double *)dphi, (const double *)dtheta,
                           c->dev<double>(c->L.ref), (const double *)nullptr, nx, Q, c->dev<double>(c->L.psi[0]),
                           c->dev<double>(c->L.psi[1]), c->dev<double>(c->L.psi[2]), c->dev<int>(c->L.flag));
    else
        hipLaunchKernelGGL(k_dist_pack<float>, grid, dim3(PLANE_THREADS), 0, c->stream, (const double *)dphi, (const double *)dtheta,
                           c->dev<double>(c->L.ref), c->has_state ? c->dev<double>(c->L.oldref) : (const double *)nullptr, nx, Q,
                           c->dev<float>(c->L.psi[0]), c->dev<float>(c->L.psi[1]), c->dev<float>(c->L.psi[2]),
                           c->dev<int>(c->L.flag));
    if (c->P.precision == ELB_FP32_MIXED) {
        // conserved densities of the stored (FP32) distributions, summed in FP64
        const LevelU lu = {{c->dev<double>(c->L.U[0]), c->dev<double>(c->L.U[1]), c->dev<double>(c->L.U[2])}};
        hipLaunchKernelGGL(k_conserved_from_psi<float>, dim3((R + 63) / 64), dim3(64), 0, c->stream,
                           c->dev<float>(c->L.psi[0]), c->dev<double>(c->L.ref), lu, c->dev<double>(c->L.p), R, Q);
    }
    rc = hip_check(c, hipGetLastError(), "distribution launch");
    if (rc) return rc;
    c->has_state = true;
    c->steps = 0;
    c->launches = 0;
    return ELB_OK;
}

}  // extern "C"

namespace {

void launch_steps(elb_ctx *c, int64_t nsteps)
{
    // stage s: psi_out = a_n psi + (1 - a_n) psi^(s) + a_L dt L[psi^(s)]
    for (int64_t s = 0; s < nsteps; ++s) {
        launch_stage(c, 0, 1, RK_AN[0], RK_AL[0]);  // psi1 = psi + dt L[psi]
        launch_stage(c, 1, 2, RK_AN[1], RK_AL[1]);  // psi2 = 3/4 psi + 1/4 psi1 + 1/4 dt L[psi1]
        launch_stage(c, 2, 0, RK_AN[2], RK_AL[2]);  // psi' = 1/3 psi + 2/3 psi2 + 2/3 dt L[psi2]
    }
}

constexpr int64_t GRAPH_STEPS = 50;

// Captures GRAPH_STEPS steps of the context on its private capture stream.
int capture_ctx_graph(elb_ctx *c)
{
    drop_ctx_graph(c);
    if (!c->cap_stream) {
        hipError_t e = hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking);
        if (e != hipSuccess) return fail(c, ELB_EHIP, "capture stream: %s", hipGetErrorString(e));
    }
    hipError_t e = hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return fail(c, ELB_EHIP, "begin capture: %s", hipGetErrorString(e));
    hipStream_t own = c->stream;
    c->stream = c->cap_stream;  // launch_stage enqueues on c->stream
    c->capturing = true;
    c->cap_seed = 0;
    launch_steps(c, GRAPH_STEPS);
    c->capturing = false;
    c->stream = own;
    e = hipStreamEndCapture(c->cap_stream, &c->graph_def);
    if (e != hipSuccess) return fail(c, ELB_EHIP, "end capture: %s", hipGetErrorString(e));
    e = hipGraphInstantiate(&c->graph, c->graph_def, nullptr, nullptr, 0);
    if (e != hipSuccess) { drop_ctx_graph(c); return fail(c, ELB_EHIP, "graph instantiate: %s", hipGetErrorString(e)); }
    return ELB_OK;
}

}  // namespace

extern "C" {

int elb_step(elb_ctx *c, int64_t nsteps)
{
    if (!c) return ELB_EINVAL;
    if (!c->has_state) return fail(c, ELB_ESTATE, "no state set");
    if (nsteps < 0) return fail(c, ELB_EINVAL, "nsteps < 0");
    int64_t done = 0;
    if (c->use_graph && nsteps >= GRAPH_STEPS) {
        if (!c->graph) {
            int rc = capture_ctx_graph(c);
            if (rc) return rc;
        }
        for (; nsteps - done >= GRAPH_STEPS; done += GRAPH_STEPS) {
            if (c->P.precision != ELB_FP64)  // FP64 stores are not dithered
                hipLaunchKernelGGL(k_set_seed, dim3(1), dim3(64), 0, c->stream, c->dev<unsigned>(c->L.seedb),
                                   c->launches);
            hipError_t e = hipGraphLaunch(c->graph, c->stream);
            if (e != hipSuccess) return fail(c, ELB_EHIP, "graph launch: %s", hipGetErrorString(e));
            c->launches += 3 * GRAPH_STEPS;
        }
    }
    launch_steps(c, nsteps - done);
    c->steps += nsteps;
    return hip_check(c, hipGetLastError(), "stage launch");
}

int elb_set_graph(elb_ctx *c, int32_t enabled)
{
    if (!c) return ELB_EINVAL;
    c->use_graph = enabled != 0;
    if (!c->use_graph) drop_ctx_graph(c);
    return ELB_OK;
}

int elb_get_moments(elb_ctx *c, double *n, double *u, double *T, double *qx, double *pxx)
{
    if (!c) return ELB_EINVAL;
    if (!c->has_state) return fail(c, ELB_ESTATE, "no state set");
    const size_t nx = c->P.nx;
    double *dst[5] = {n, u, T, qx, pxx};
    // Few cells: the kernel writes the fields and the flag into the pinned buffer itself, which
    // saves the copy (about 5 us); more: one copy when the buffer holds them, else field by field
    const size_t bytes = sizeof(double) * (5 * nx + 2);
    char *st = c->stage->take(bytes, c->stream);
    const bool direct = st && nx <= MOM_DIRECT;
    double *o = direct ? reinterpret_cast<double *>(st) : c->dev<double>(c->L.out);
    int rc = run_moments(c, o);
    if (rc) return rc;
    if (st) {
        if (!direct)
            rc = hip_check(c, hipMemcpyAsync(st, o, bytes, hipMemcpyDeviceToHost, c->stream), "moments copy");
        if (!rc) rc = hip_check(c, hipStreamSynchronize(c->stream), "stream sync");
        if (rc) return rc;
        c->stage->used = 0;
        for (int f = 0; f < 5; ++f)
            if (dst[f]) std::memcpy(dst[f], st + sizeof(double) * f * nx, sizeof(double) * nx);
        int flag;
        std::memcpy(&flag, st + sizeof(double) * 5 * nx, sizeof flag);
        return flag_status(c, flag);
    }
    int flag = 0;
    const size_t at = c->L.out, nb = sizeof(double) * nx;
    rc = download(c, {{dst[0], at, nb}, {dst[1], at + nb, nb}, {dst[2], at + 2 * nb, nb}, {dst[3], at + 3 * nb, nb},
                      {dst[4], at + 4 * nb, nb}, {&flag, c->L.flag, sizeof flag}});
    return rc ? rc : flag_status(c, flag);
}

int elb_get_amplitudes(elb_ctx *c, double k, double out[2])
{
    if (!c) return ELB_EINVAL;
    if (!out || !std::isfinite(k)) return fail(c, ELB_EINVAL, "NULL output or non-finite k");
    if (!c->has_state) return fail(c, ELB_ESTATE, "no state set");
    const int nx = c->P.nx, Q = c->Q;
    // the kernel writes the three numbers into the pinned buffer itself
    char *st = c->stage->take(3 * sizeof(double), c->stream);
    double *amp = st ? reinterpret_cast<double *>(st) : c->dev<double>(c->L.amp);
    const int *flag = c->dev<int>(c->L.flag);
    const double *U = c->P.precision == ELB_FP32_MIXED ? c->dev<double>(c->L.U[0]) : nullptr;
    const double *dens = c->dev<double>(c->L.out);
    // With bookkeeping, and for few cells, one kernel forms the densities and projects them;
    // else the moment kernel spreads the cells over the chip first.  The line: the one block
    // takes about 0.8 us per 64 cells and 16 nodes, the extra launch 6 us.
    const bool direct = U || (size_t)nx * ((Q + MOM_LANES - 1) / MOM_LANES) <= AMP_DIRECT;
    if (!direct) {
        int rc = run_moments(c, c->dev<double>(c->L.out));
        if (rc) return rc;
    }
    if (U || !direct)
        hipLaunchKernelGGL((k_amplitudes<double, true>), dim3(1), dim3(AMP_THREADS), 0, c->stream, (const double *)nullptr,
                           (const double *)nullptr, U ? U + 3 * NG : dens, U ? 3 : 1, nx, Q, c->P.x0, c->dx, k, flag, amp);
    else if (c->P.precision == ELB_FP64)
        hipLaunchKernelGGL((k_amplitudes<double, false>), dim3(1), dim3(AMP_THREADS), 0, c->stream,
                           c->dev<double>(c->L.psi[0]), c->dev<double>(c->L.ref), (const double *)nullptr, 0, nx, Q, c->P.x0, c->dx,
                           k, flag, amp);
    else
        hipLaunchKernelGGL((k_amplitudes<float, false>), dim3(1), dim3(AMP_THREADS), 0, c->stream,
                           c->dev<float>(c->L.psi[0]), c->dev<double>(c->L.ref), (const double *)nullptr, 0, nx, Q, c->P.x0, c->dx,
                           k, flag, amp);
    int rc = hip_check(c, hipGetLastError(), "amplitude kernel launch");
    if (rc) return rc;
    double v[3];
    if (st) {
        rc = hip_check(c, hipStreamSynchronize(c->stream), "stream sync");
        std::memcpy(v, st, sizeof v);
        c->stage->used = 0;
    } else {
        rc = download(c, {{v, c->L.amp, sizeof v}});
    }
    if (rc) return rc;
    out[0] = v[0];
    out[1] = v[1];
    return flag_status(c, v[2] != 0.0);
}

int elb_get_dist(elb_ctx *c, double *phi, double *theta)
{
    if (!c) return ELB_EINVAL;
    if (!c->has_state) return fail(c, ELB_ESTATE, "no state set");
    const int nx = c->P.nx, Q = c->Q;
    const size_t n = (size_t)nx * Q;
    size_t at[2];
    dist_planes(c, at);
    const dim3 grid = plane_grid(n);
    if (c->P.precision == ELB_FP64)
        hipLaunchKernelGGL(k_dist_planes<double>, grid, dim3(PLANE_THREADS), 0, c->stream, c->dev<double>(c->L.psi[0]),
                           c->dev<double>(c->L.ref), nx, Q, c->dev<double>(at[0]), c->dev<double>(at[1]), c->dev<int>(c->L.flag),
                           c->stage->flag());
    else
        hipLaunchKernelGGL(k_dist_planes<float>, grid, dim3(PLANE_THREADS), 0, c->stream, c->dev<float>(c->L.psi[0]),
                           c->dev<double>(c->L.ref), nx, Q, c->dev<double>(at[0]), c->dev<double>(at[1]), c->dev<int>(c->L.flag),
                           c->stage->flag());
    int rc = hip_check(c, hipGetLastError(), "dist kernel launch");
    if (!rc) rc = download(c, {{phi, at[0], sizeof(double) * n}, {theta, at[1], sizeof(double) * n}});
    if (rc) return rc;
    return c->stage->flag() ? flag_status(c, *c->stage->flag()) : check_flag(c);
}

int elb_get_conserved(elb_ctx *c, double out[3])
{
    if (!c || !out) return ELB_EINVAL;
    if (!c->has_state) return fail(c, ELB_ESTATE, "no state set");
    int rc = run_moments(c, c->dev<double>(c->L.out), true);
    if (rc) return rc;
    int nx = c->P.nx;
    std::vector<double> cons(3 * (size_t)nx);
    rc = hip_check(c, hipMemcpyAsync(cons.data(), c->dev<double>(c->L.cons), sizeof(double) * cons.size(),
                                     hipMemcpyDeviceToHost, c->stream), "conserved copy");
    if (rc) return rc;
    rc = check_flag(c);
    if (rc) return rc;
    double m = 0, j = 0, e = 0;
    for (int i = 0; i < nx; ++i) { m += cons[3 * i]; j += cons[3 * i + 1]; e += cons[3 * i + 2]; }
    out[0] = m * c->dx; out[1] = j * c->dx; out[2] = e * c->dx;
    return ELB_OK;
}

int elb_get_time(const elb_ctx *c, double *dt, int64_t *steps)
{
    if (!c) return ELB_EINVAL;
    if (dt) *dt = c->dt;
    if (steps) *steps = c->steps;
    return ELB_OK;
}

const char *elb_last_error(const elb_ctx *c)
{
    if (!c) return g_create_error.c_str();
    return c->err.c_str();
}

int elb_destroy(elb_ctx *c)
{
    if (!c) return ELB_EINVAL;
    hipError_t e = hipStreamSynchronize(c->stream);
    if (e != hipSuccess) c->own_stage.buf.p = nullptr;
    delete c;
    return e == hipSuccess ? ELB_OK : ELB_EHIP;
}

}  // extern "C"

// ======================================================================================
// Batches: many independent problems (own nx, Q, physics, boundaries, time step) stepped
// together.  Each instance keeps the state layout of a single context in its own slice of
// the batch workspace; one kernel launch per stage and per group of instances sharing Q and
// tile shape covers every (instance, tile) item of the group, and a chunk of steps is
// captured once in a HIP graph and replayed.
// ======================================================================================
namespace {

std::vector<const BatchKernel *> batch_variants(int q, int precision, int ret)
{
    std::vector<const BatchKernel *> v;
    const StageTable t = stage_table(precision, 0);
    for (int i = 0; i < t.batches; ++i)
        if (t.batch[i].q == q && t.batch[i].ret == ret) v.push_back(&t.batch[i]);
    return v;
}

struct BatchGroup {
    int q = 0, ret = 0;                       // node count; chi_RET-FM (1) or chi_SET (0)
    int fm_J = 0;                             // chi_RET-FM: largest stencil half-width
    std::vector<int> inst;                    // instances of this Q and chi mode
    std::vector<const BatchKernel *> variants;
    std::vector<int2 *> d_items;              // per variant, in the workspace
    std::vector<int> nitems;                  // per variant
    std::vector<int> grid;                    // per variant
    int chosen = 0;
    std::string key;                          // tuner cache key
};

}  // namespace

struct elb_batch {
    int count = 0, precision = 0;
    HostStage stage;  // shared by the contexts (one stream)
    hipStream_t stream = nullptr;
    char *ws = nullptr;
    InstDesc *d_inst = nullptr;
    std::vector<elb_ctx *> ctx;
    std::vector<BatchGroup> groups;
    hipStream_t cap_stream = nullptr;  // private stream used only to capture the graph
    // capture only: side streams and events that fork the Q groups into parallel branches of the
    // graph, each through all steps of the chunk, and join them at its end
    std::vector<hipStream_t> side;
    hipEvent_t ev_fork = nullptr;
    std::vector<hipEvent_t> ev_join;
    hipGraphExec_t graph = nullptr;
    hipGraph_t graph_def = nullptr;
    int64_t graph_steps = 0;
    int use_graph = 1;
    // stochastic rounding stream of the FP32 stores, as for a single context: stage launches
    // since a state was last set; captured launches read the base set before each replay
    uint32_t launches = 0;
    bool capturing = false;
    uint32_t cap_seed = 0;
    unsigned *seed_dev = nullptr;
    std::string err;
};

namespace {

int bfail(elb_batch *b, int code, const char *fmt, ...)
{
    if (b) {
        char buf[512];
        va_list ap;
        va_start(ap, fmt);
        vsnprintf(buf, sizeof buf, fmt, ap);
        va_end(ap);
        b->err = buf;
    }
    return code;
}

struct BatchLayout {
    size_t inst = 0, items = 0, seedb = 0, total = 0;
    std::vector<size_t> ctx;        // per instance
    std::vector<size_t> item_off;   // per (group, variant), in order of group creation
};

int inst_ret(const elb_params &p) { return p.chi_mode == ELB_CHI_RETFM ? 1 : 0; }

// groups: one per (Q, chi mode) among the instances, ascending
std::vector<std::pair<int, int>> batch_specs(const elb_params *p, int count)
{
    std::vector<std::pair<int, int>> v;
    for (int i = 0; i < count; ++i) {
        std::pair<int, int> k(p[i].q, inst_ret(p[i]));
        if (std::find(v.begin(), v.end(), k) == v.end()) v.push_back(k);
    }
    std::sort(v.begin(), v.end());
    return v;
}

// dynamic LDS of a group's launch (the chi_RET-FM phase of the stage kernel)
size_t group_lds(const BatchGroup &g, int v) { return g.ret ? fm_lds_bytes(g.fm_J, g.variants[v]->rows) : 0; }

int batch_layout(const elb_params *p, int count, BatchLayout *L, std::string *msg)
{
    if (!p || count < 1) { *msg = "need at least one instance"; return ELB_EINVAL; }
    for (int i = 0; i < count; ++i) {
        if (p[i].precision != p[0].precision) { *msg = "all instances of a batch share the precision"; return ELB_EINVAL; }
        if (batch_variants(p[i].q, p[i].precision, inst_ret(p[i])).empty()) { *msg = "q not compiled for batches"; return ELB_EUNSUPPORTED; }
        if (p[i].closure) { *msg = "batches do not carry the learned closure"; return ELB_EUNSUPPORTED; }
        if (p[i].moment_fixup) { *msg = "batches do not carry the moment fix-up"; return ELB_EUNSUPPORTED; }
    }
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align256(o + bytes); return at; };
    L->inst = take(sizeof(InstDesc) * count);
    L->seedb = take(sizeof(unsigned));
    for (auto spec : batch_specs(p, count))
        for (const BatchKernel *k : batch_variants(spec.first, p[0].precision, spec.second)) {
            size_t n = 0;
            for (int i = 0; i < count; ++i)
                if (p[i].q == spec.first && inst_ret(p[i]) == spec.second)
                    n += (p[i].nx + k->cells() - 1) / k->cells();
            L->item_off.push_back(take(sizeof(int2) * n));
        }
    L->ctx.resize(count);
    for (int i = 0; i < count; ++i) {
        int64_t b = elb_workspace_bytes(&p[i]);
        if (b < 0) {
            int N; double dx, dt, bb, mu, e0, c0;
            int rc = derive(&p[i], &N, &dx, &dt, &bb, &mu, &e0, &c0, nullptr, msg);
            *msg = "instance " + std::to_string(i) + ": " + *msg;
            return rc ? rc : ELB_EINVAL;
        }
        L->ctx[i] = take((size_t)b);
    }
    L->total = o;
    return ELB_OK;
}

// Device descriptor of an instance from its context.
InstDesc describe(const elb_ctx *c)
{
    InstDesc d{};
    for (int s = 0; s < 3; ++s) {
        d.psi[s] = c->ws + c->L.psi[s];
        d.U[s] = c->dev<double>(c->L.U[s]);
    }
    d.p = c->dev<double>(c->L.p);
    d.cref = c->dev<double>(c->L.cref);
    d.gref = c->dev<double>(c->L.gref);
    d.rec = c->dev<double>(c->L.rec);
    d.w = c->dev<double>(c->L.btd);  // row l = 0 of the Hermite matrix: w_k
    d.Bt = c->P.precision == ELB_FP64 ? (const void *)c->dev<double>(c->L.bpd) : (const void *)c->dev<float>(c->L.bpf);
    d.flag = c->dev<int>(c->L.flag);
    d.nx = c->P.nx;
    d.N = c->N;
    d.periodic = c->P.bc == ELB_BC_PERIODIC;
    d.pr_enskog = c->P.pr_mode == ELB_PR_ENSKOG;
    d.b = c->b;
    d.pr = c->P.pr;
    d.inv_dx = 1.0 / c->dx;
    d.inv_mu = 1.0 / c->mu_ref;
    for (int s = 0; s < 3; ++s) {
        d.w_rhs[s] = RK_AL[s] * c->dt;
        d.w_flux[s] = RK_AL[s] * c->dt / (6.0 * c->dx);
    }
    d.T_ref = c->T_ref;
    for (int m = 0; m < 6; ++m) d.ref_sum[m] = c->ref_sum[m];
    d.fm_w = c->fm_J >= 0 ? c->dev<double>(c->L.chiw) : nullptr;
    d.fm_J = c->fm_J;
    return d;
}

// Device descriptor of instance i.  A captured graph reads the descriptors from device memory
// and stays valid.
int upload_descriptor(elb_batch *b, int i)
{
    const InstDesc d = describe(b->ctx[i]);
    char *up = b->stage.take(sizeof d, b->stream);
    if (up) std::memcpy(up, &d, sizeof d);
    hipError_t e = hipMemcpyAsync(b->d_inst + i, up ? (const void *)up : &d, sizeof d, hipMemcpyHostToDevice, b->stream);
    if (e == hipSuccess && !up) e = hipStreamSynchronize(b->stream);
    if (e != hipSuccess) return bfail(b, ELB_EHIP, "descriptor upload: %s", hipGetErrorString(e));
    return ELB_OK;
}

void drop_graph(elb_batch *b)
{
    if (b->graph) (void)hipGraphExecDestroy(b->graph);
    if (b->graph_def) (void)hipGraphDestroy(b->graph_def);
    b->graph = nullptr;
    b->graph_def = nullptr;
    b->graph_steps = 0;
}

// Stage `s` (0, 1, 2) of one group on stream st.
void enqueue_stage(elb_batch *b, const BatchGroup &g, hipStream_t st, int s, uint32_t seed)
{
    const int v = g.chosen;
    BatchStage bs{};
    bs.inst = b->d_inst;
    bs.items = g.d_items[v];
    bs.nitems = g.nitems[v];
    bs.s_in = s;
    bs.s_out = (s + 1) % 3;
    bs.a_n = RK_AN[s];
    bs.seed = seed;
    bs.seed_base = b->capturing ? b->seed_dev : nullptr;
    g.variants[v]->launch(bs, g.grid[v], group_lds(g, v), st);
}

// nsteps steps of every group.  With fork (graph capture), groups 1.. run on side streams that
// wait for the start on st and are joined back into st at the end, so the captured graph holds
// them as parallel branches.  The groups share nothing that is written, so a branch runs through
// all its steps: joined after every stage, each stage waited for its slowest group's last
// blocks (128 problems of 4 node counts, 150 stages and the readout: 14.5 ms, 13.0 without).
void enqueue_steps(elb_batch *b, hipStream_t st, int64_t nsteps, bool fork)
{
    const size_t G = b->groups.size();
    const uint32_t seed0 = b->capturing ? b->cap_seed : b->launches;
    if (fork && G > 1 && b->side.size() + 1 >= G) {
        (void)hipEventRecord(b->ev_fork, st);
        for (size_t gi = 0; gi < G; ++gi) {
            hipStream_t gs = gi ? b->side[gi - 1] : st;
            if (gi) (void)hipStreamWaitEvent(gs, b->ev_fork, 0);
            for (int64_t j = 0; j < 3 * nsteps; ++j)
                enqueue_stage(b, b->groups[gi], gs, (int)(j % 3), seed0 + (uint32_t)j);
            if (gi) (void)hipEventRecord(b->ev_join[gi - 1], gs);
        }
        for (size_t gi = 1; gi < G; ++gi) (void)hipStreamWaitEvent(st, b->ev_join[gi - 1], 0);
    } else {
        for (int64_t j = 0; j < 3 * nsteps; ++j)
            for (const auto &g : b->groups) enqueue_stage(b, g, st, (int)(j % 3), seed0 + (uint32_t)j);
    }
    (b->capturing ? b->cap_seed : b->launches) = seed0 + (uint32_t)(3 * nsteps);
}

// The graph is captured on the batch's private stream (the caller's stream may be the
// legacy default stream, which cannot be captured) and launched on the caller's stream.
int capture_graph(elb_batch *b, int64_t steps)
{
    drop_graph(b);
    if (!b->cap_stream) {
        hipError_t e = hipStreamCreateWithFlags(&b->cap_stream, hipStreamNonBlocking);
        if (e != hipSuccess) return bfail(b, ELB_EHIP, "capture stream: %s", hipGetErrorString(e));
    }
    while (b->side.size() + 1 < b->groups.size()) {
        hipStream_t sd = nullptr;
        hipEvent_t ev = nullptr;
        hipError_t e = hipStreamCreateWithFlags(&sd, hipStreamNonBlocking);
        if (e == hipSuccess) b->side.push_back(sd);
        if (e == hipSuccess) e = hipEventCreateWithFlags(&ev, hipEventDisableTiming);
        if (e == hipSuccess) b->ev_join.push_back(ev);
        if (e != hipSuccess) return bfail(b, ELB_EHIP, "side stream: %s", hipGetErrorString(e));
    }
    if (!b->ev_fork) {
        hipError_t e = hipEventCreateWithFlags(&b->ev_fork, hipEventDisableTiming);
        if (e != hipSuccess) return bfail(b, ELB_EHIP, "fork event: %s", hipGetErrorString(e));
    }
    hipError_t e = hipStreamBeginCapture(b->cap_stream, hipStreamCaptureModeThreadLocal);
    if (e != hipSuccess) return bfail(b, ELB_EHIP, "begin capture: %s", hipGetErrorString(e));
    b->capturing = true;
    b->cap_seed = 0;
    enqueue_steps(b, b->cap_stream, steps, true);
    b->capturing = false;
    e = hipStreamEndCapture(b->cap_stream, &b->graph_def);
    if (e != hipSuccess) return bfail(b, ELB_EHIP, "end capture: %s", hipGetErrorString(e));
    e = hipGraphInstantiate(&b->graph, b->graph_def, nullptr, nullptr, 0);
    if (e != hipSuccess) { drop_graph(b); return bfail(b, ELB_EHIP, "graph instantiate: %s", hipGetErrorString(e)); }
    b->graph_steps = steps;
    return ELB_OK;
}

std::string read_file(const char *path)
{
    std::ifstream f(path);
    if (!f) return std::string();
    std::stringstream ss;
    ss << f.rdbuf();
    return ss.str();
}

// The tuner cache is a JSON object {"key": variant_index, ...} with one key per group:
// "<arch>/<precision>/q<Q>/cells<2^k bucket of the group's cell count>".
std::map<std::string, int> parse_cache(const std::string &txt)
{
    std::map<std::string, int> m;
    size_t pos = 0;
    while ((pos = txt.find('"', pos)) != std::string::npos) {
        size_t end = txt.find('"', pos + 1);
        if (end == std::string::npos) break;
        std::string key = txt.substr(pos + 1, end - pos - 1);
        size_t colon = txt.find(':', end);
        if (colon == std::string::npos) break;
        m[key] = std::atoi(txt.c_str() + colon + 1);
        pos = txt.find_first_of(",}", colon);
        if (pos == std::string::npos) break;
    }
    return m;
}

void write_cache(const char *path, const std::map<std::string, int> &m)
{
    std::ofstream f(path);
    f << "{\n";
    size_t i = 0;
    for (const auto &kv : m) f << "  \"" << kv.first << "\": " << kv.second << (++i < m.size() ? ",\n" : "\n");
    f << "}\n";
}

}  // namespace

extern "C" {

// Reason the last failed elb_batch_create or elb_batch_workspace_bytes on this thread failed.
thread_local std::string g_batch_create_error;

int64_t elb_batch_workspace_bytes(const elb_params *params, int32_t count)
{
    BatchLayout L;
    std::string msg;
    if (batch_layout(params, count, &L, &msg)) { g_batch_create_error = msg; return -1; }
    return (int64_t)L.total;
}

int elb_batch_create(const elb_params *params, int32_t count, void *dev_workspace, int64_t workspace_bytes,
                     void *hip_stream, elb_batch **out)
{
    if (!out) return ELB_EINVAL;
    *out = nullptr;
    BatchLayout L;
    std::string msg;
    int rc = batch_layout(params, count, &L, &msg);
    if (rc) { g_batch_create_error = msg; return rc; }
    if (!dev_workspace || workspace_bytes < (int64_t)L.total) {
        g_batch_create_error = "workspace missing or too small";
        return ELB_ENOMEM;
    }
    if (((uintptr_t)dev_workspace) & 255) {
        g_batch_create_error = "workspace not 256-byte aligned";
        return ELB_EINVAL;
    }
    elb_batch *b = new (std::nothrow) elb_batch();
    if (!b) { g_batch_create_error = "host allocation failed"; return ELB_ENOMEM; }
    b->count = count;
    b->precision = params[0].precision;
    b->stream = (hipStream_t)hip_stream;
    b->ws = (char *)dev_workspace;
    b->d_inst = reinterpret_cast<InstDesc *>(b->ws + L.inst);
    b->seed_dev = reinterpret_cast<unsigned *>(b->ws + L.seedb);
    b->ctx.assign(count, nullptr);
    size_t moved = 0;  // room for the uploads of several instances
    for (int i = 0; i < count; ++i) moved = std::min(STAGE_MAX, moved + stage_bytes(&params[i]));
    b->stage.reserve(moved);
    for (int i = 0; i < count; ++i) {
        int64_t bytes = elb_workspace_bytes(&params[i]);
        rc = create_ctx(&params[i], b->ws + L.ctx[i], bytes, hip_stream, &b->stage, &b->ctx[i]);
        if (rc) {
            g_batch_create_error = "instance " + std::to_string(i) + ": " + elb_last_error(nullptr);
            for (auto c : b->ctx) if (c) elb_destroy(c);
            delete b;
            return rc;
        }
    }
    size_t vi = 0;
    for (auto spec : batch_specs(params, count)) {
        BatchGroup g;
        const int q = spec.first;
        g.q = q;
        g.ret = spec.second;
        for (int i = 0; i < count; ++i)
            if (params[i].q == q && inst_ret(params[i]) == g.ret) {
                g.inst.push_back(i);
                g.fm_J = std::max(g.fm_J, b->ctx[i]->fm_J);
            }
        g.variants = batch_variants(q, b->precision, g.ret);
        int64_t cells = 0;
        for (int i : g.inst) cells += params[i].nx;
        int bucket = 0;
        while ((int64_t(1) << (bucket + 1)) <= cells) ++bucket;
        g.key = "gfx950/" + std::to_string(b->precision) + "/q" + std::to_string(q) + (g.ret ? "/ret" : "") +
                "/cells2^" + std::to_string(bucket);
        for (const BatchKernel *k : g.variants) {
            std::vector<int2> items;
            for (int i : g.inst) {
                int tiles = (params[i].nx + k->cells() - 1) / k->cells();
                for (int t = 0; t < tiles; ++t) items.push_back(make_int2(i, t));
            }
            int2 *d = reinterpret_cast<int2 *>(b->ws + L.item_off[vi++]);
            hipError_t e = hipMemcpyAsync(d, items.data(), sizeof(int2) * items.size(), hipMemcpyHostToDevice, b->stream);
            if (e != hipSuccess) {
                g_batch_create_error = std::string("item upload: ") + hipGetErrorString(e);
                elb_batch_destroy(b);
                return ELB_EHIP;
            }
            g.d_items.push_back(d);
            g.nitems.push_back((int)items.size());
            g.grid.push_back((int)items.size());  // one block per (instance, tile) item
        }
        // before any tuning: the smallest tile whose items fit its cap, as for a single problem;
        // else the large-problem tile
        for (int v = 1, cells_v = INT_MAX; v < (int)g.variants.size(); ++v)
            if (g.variants[v]->cap != INT_MAX && g.nitems[v] <= g.variants[v]->cap && g.variants[v]->cells() < cells_v) {
                g.chosen = v;
                cells_v = g.variants[v]->cells();
            }
        b->groups.push_back(g);
    }
    if (hipError_t e = hipStreamSynchronize(b->stream); e != hipSuccess) {
        g_batch_create_error = std::string("item upload: ") + hipGetErrorString(e);
        elb_batch_destroy(b);
        return ELB_EHIP;
    }
    *out = b;
    return ELB_OK;
}

int elb_batch_set_state_moments(elb_batch *b, int32_t inst, const double *n, const double *u, const double *T)
{
    if (!b) return ELB_EINVAL;
    if (inst < 0 || inst >= b->count) return bfail(b, ELB_EINVAL, "instance %d out of range", inst);
    int rc = elb_set_state_moments(b->ctx[inst], n, u, T);
    if (rc) return bfail(b, rc, "instance %d: %s", inst, elb_last_error(b->ctx[inst]));
    b->launches = 0;
    return upload_descriptor(b, inst);
}

int elb_batch_step(elb_batch *b, int64_t nsteps)
{
    if (!b) return ELB_EINVAL;
    if (nsteps < 0) return bfail(b, ELB_EINVAL, "nsteps < 0");
    for (int i = 0; i < b->count; ++i)
        if (!b->ctx[i]->has_state) return bfail(b, ELB_ESTATE, "instance %d has no state", i);
    int64_t done = 0;
    if (b->use_graph && nsteps > 0) {
        const int64_t chunk = std::min<int64_t>(nsteps, 50);
        if (b->graph_steps != chunk) {
            int rc = capture_graph(b, chunk);
            if (rc) return rc;
        }
        while (nsteps - done >= chunk) {
            if (b->precision != ELB_FP64)  // FP64 stores are not dithered
                hipLaunchKernelGGL(k_set_seed, dim3(1), dim3(64), 0, b->stream, b->seed_dev, b->launches);
            hipError_t e = hipGraphLaunch(b->graph, b->stream);
            if (e != hipSuccess) return bfail(b, ELB_EHIP, "graph launch: %s", hipGetErrorString(e));
            done += chunk;
            b->launches += (uint32_t)(3 * chunk);
        }
    }
    enqueue_steps(b, b->stream, nsteps - done, false);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return bfail(b, ELB_EHIP, "stage launch: %s", hipGetErrorString(e));
    for (auto c : b->ctx) c->steps += nsteps;
    return ELB_OK;
}

int elb_batch_set_graph(elb_batch *b, int32_t enabled)
{
    if (!b) return ELB_EINVAL;
    b->use_graph = enabled ? 1 : 0;
    if (!enabled) drop_graph(b);
    return ELB_OK;
}

int elb_batch_get_moments(elb_batch *b, int32_t inst, double *n, double *u, double *T, double *qx, double *pxx)
{
    if (!b) return ELB_EINVAL;
    if (inst < 0 || inst >= b->count) return bfail(b, ELB_EINVAL, "instance %d out of range", inst);
    int rc = elb_get_moments(b->ctx[inst], n, u, T, qx, pxx);
    if (rc) return bfail(b, rc, "instance %d: %s", inst, elb_last_error(b->ctx[inst]));
    return ELB_OK;
}

int elb_batch_get_amplitudes(elb_batch *b, int32_t inst, double k, double out[2])
{
    if (!b) return ELB_EINVAL;
    if (inst < 0 || inst >= b->count) return bfail(b, ELB_EINVAL, "instance %d out of range", inst);
    int rc = elb_get_amplitudes(b->ctx[inst], k, out);
    if (rc) return bfail(b, rc, "instance %d: %s", inst, elb_last_error(b->ctx[inst]));
    return ELB_OK;
}

int elb_batch_get_dist(elb_batch *b, int32_t inst, double *phi, double *theta)
{
    if (!b) return ELB_EINVAL;
    if (inst < 0 || inst >= b->count) return bfail(b, ELB_EINVAL, "instance %d out of range", inst);
    int rc = elb_get_dist(b->ctx[inst], phi, theta);
    if (rc) return bfail(b, rc, "instance %d: %s", inst, elb_last_error(b->ctx[inst]));
    return ELB_OK;
}

int elb_batch_tune(elb_batch *b, const char *cache_path, int32_t force)
{
    if (!b) return ELB_EINVAL;
    for (int i = 0; i < b->count; ++i)
        if (!b->ctx[i]->has_state) return bfail(b, ELB_ESTATE, "instance %d has no state", i);
    std::map<std::string, int> cache;
    if (cache_path) cache = parse_cache(read_file(cache_path));
    drop_graph(b);
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) {
        if (e0) (void)hipEventDestroy(e0);
        return bfail(b, ELB_EHIP, "tuning: event creation failed");
    }
    bool changed = false;
    for (auto &g : b->groups) {
        auto it = cache.find(g.key);
        if (!force && it != cache.end() && it->second >= 0 && it->second < (int)g.variants.size()) {
            g.chosen = it->second;
            continue;
        }
        float best = 1e30f;
        int best_v = 0;
        for (int v = 0; v < (int)g.variants.size(); ++v) {
            // stage 1 only (reads level 0, writes level 1): the state is left unchanged
            BatchStage bs{};
            bs.inst = b->d_inst;
            bs.items = g.d_items[v];
            bs.nitems = g.nitems[v];
            bs.s_in = 0;
            bs.s_out = 1;
            bs.a_n = RK_AN[0];
            g.variants[v]->launch(bs, g.grid[v], group_lds(g, v), b->stream);  // warm-up
            float tmin = 1e30f;
            for (int rep = 0; rep < 5; ++rep) {
                (void)hipEventRecord(e0, b->stream);
                g.variants[v]->launch(bs, g.grid[v], group_lds(g, v), b->stream);
                (void)hipEventRecord(e1, b->stream);
                (void)hipEventSynchronize(e1);
                float ms = 1e30f;  // a failed timing never wins; the error is reported below
                if (hipEventElapsedTime(&ms, e0, e1) != hipSuccess) ms = 1e30f;
                tmin = std::min(tmin, ms);
            }
            if (tmin < best) { best = tmin; best_v = v; }
        }
        g.chosen = best_v;
        cache[g.key] = best_v;
        changed = true;
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return bfail(b, ELB_EHIP, "tuning: %s", hipGetErrorString(e));
    if (cache_path && changed) write_cache(cache_path, cache);  // only choices from clean timings
    return ELB_OK;
}

int elb_batch_groups(const elb_batch *b, int32_t *q, int32_t *strips, int32_t *strip_len, int32_t *items, int32_t cap)
{
    if (!b) return ELB_EINVAL;
    int n = (int)b->groups.size();
    for (int i = 0; i < n && i < cap; ++i) {
        const auto &g = b->groups[i];
        const BatchKernel *k = g.variants[g.chosen];
        if (q) q[i] = g.q;
        if (strips) strips[i] = k->S;
        if (strip_len) strip_len[i] = k->L;
        if (items) items[i] = g.nitems[g.chosen];
    }
    return n;
}

const char *elb_batch_last_error(const elb_batch *b)
{
    if (!b) return g_batch_create_error.c_str();
    return b->err.c_str();
}

int elb_batch_destroy(elb_batch *b)
{
    if (!b) return ELB_EINVAL;
    if (hipStreamSynchronize(b->stream) != hipSuccess) b->stage.buf.p = nullptr;
    drop_graph(b);
    if (b->cap_stream) (void)hipStreamDestroy(b->cap_stream);
    for (auto sd : b->side) (void)hipStreamDestroy(sd);
    for (auto ev : b->ev_join) (void)hipEventDestroy(ev);
    if (b->ev_fork) (void)hipEventDestroy(b->ev_fork);
    for (auto c : b->ctx)
        if (c) elb_destroy(c);
    delete b;
    return ELB_OK;
}

}  // extern "C"

// ======================================================================================
// Learned closure: training kernels, samples and the corrected step
// ======================================================================================
namespace {

struct MlpWs {
    size_t a0, a0t, at, g4t, gt, z, dz, part, lpart, total;
    size_t lstride;  // elements from layer to layer of at and gt
    int nblk_w, nblk_l;
};

// Tiles of 16 rows per block of the training forward: as many as leave 1024 blocks (four per CU),
// up to 8, so that the weights are read from L2 once for all of them.  us with 1 / 2 / 4 / 8 tiles:
// 16384 rows 8.9 / 8.8 / 10.8 / 17, 32768 14.8 / 12.1 / 13.1 / 18, 65536 23 / 20 / 18 / 23,
// 131072 40 / 31 / 30 / 28, 4194304 1507 / 1375 / 1289 / 1241 (16: 1242).
int forward_tiles(int64_t batch)
{
    const int64_t t = batch / TRAIN_ROWS / 1024;
    return t >= 8 ? 8 : t >= 4 ? 4 : t >= 2 ? 2 : 1;
}

MlpWs mlp_ws(int64_t batch)
{
    MlpWs w{};
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t at = o; o = align256(o + bytes); return at; };
    w.nblk_w = (int)((batch + WGRAD_ROWS - 1) / WGRAD_ROWS);
    w.nblk_l = (int)std::min<int64_t>(256, (batch * MLP_OUT + 255) / 256);
    // transposed bf16 operands of the weight gradients, in whole chunks
    const size_t rows = (size_t)w.nblk_w * WGRAD_ROWS;
    w.lstride = rows * MLP_H;
    w.a0 = take(sizeof(unsigned short) * MLP_K1 * (size_t)batch);
    w.a0t = take(sizeof(unsigned short) * MLP_K1 * rows);
    w.at = take(sizeof(unsigned short) * 3 * w.lstride);
    w.g4t = take(sizeof(unsigned short) * MLP_OUT * rows);
    w.gt = take(sizeof(unsigned short) * 3 * w.lstride);
    w.z = take(sizeof(float) * 3 * MLP_H * (size_t)batch);
    w.dz = take(sizeof(float) * 3 * MLP_H * (size_t)batch);
    w.part = take(sizeof(float) * MLP_PARAMS * (size_t)w.nblk_w);
    w.lpart = take(sizeof(double) * 256);
    w.total = o;
    return w;
}

const int64_t kMaxBatch = int64_t(1) << 24;

unsigned short host_bf16(float f)
{
    unsigned int u;
    std::memcpy(&u, &f, 4);
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (unsigned short)(u >> 16);
}

// Pi[j][k] = w_j sum_{l < q_to} h_l(p_j) h_l(P_k), h_l = He_l / sqrt(l!): student values with
// the teacher's Hermite moments 0..q_to-1.
int projection_host(int q_from, int q_to, double *P)
{
    if (q_from < 1 || q_from > 256 || q_to < 1 || q_to > q_from) return ELB_EINVAL;
    std::vector<double> pT(q_from), wT(q_from), ps(q_to), wsv(q_to), hT((size_t)q_from * q_to), hs(q_to);
    if (gauss_hermite(q_from, pT.data(), wT.data()) || gauss_hermite(q_to, ps.data(), wsv.data())) return ELB_EINVAL;
    std::vector<double> h(q_to + 2);
    for (int k = 0; k < q_from; ++k) {
        hermite_orthonormal(q_to - 1, pT[k], h.data());
        for (int l = 0; l < q_to; ++l) hT[(size_t)k * q_to + l] = h[l];
    }
    for (int j = 0; j < q_to; ++j) {
        hermite_orthonormal(q_to - 1, ps[j], h.data());
        for (int k = 0; k < q_from; ++k) {
            double s = 0.0;
            for (int l = 0; l < q_to; ++l) s += h[l] * hT[(size_t)k * q_to + l];
            P[(size_t)j * q_from + k] = wsv[j] * s;
        }
    }
    return ELB_OK;
}

// Lam[k][j] = W_k sum_{l < q_from} h_l(P_k) h_l(p_j): the values on the q_to nodes P_k
// (weights W_k) of the Hermite series that carries the moments 0..q_from-1 of a state on the
// q_from nodes p_j; the left inverse of projection_host(q_to, q_from).
int lift_host(int q_from, int q_to, double *Lam)
{
    if (q_from < 1 || q_from > 256 || q_to < q_from || q_to > 256) return ELB_EINVAL;
    std::vector<double> ps(q_from), wsv(q_from), pT(q_to), wT(q_to), hs((size_t)q_from * q_from);
    if (gauss_hermite(q_from, ps.data(), wsv.data()) || gauss_hermite(q_to, pT.data(), wT.data())) return ELB_EINVAL;
    std::vector<double> h(q_from + 2);
    for (int j = 0; j < q_from; ++j) {
        hermite_orthonormal(q_from - 1, ps[j], h.data());
        for (int l = 0; l < q_from; ++l) hs[(size_t)j * q_from + l] = h[l];
    }
    for (int k = 0; k < q_to; ++k) {
        hermite_orthonormal(q_from - 1, pT[k], h.data());
        for (int j = 0; j < q_from; ++j) {
            double acc = 0.0;
            for (int l = 0; l < q_from; ++l) acc += h[l] * hs[(size_t)j * q_from + l];
            Lam[(size_t)k * q_from + j] = wT[k] * acc;
        }
    }
    return ELB_OK;
}

// psi + L[psi] of level 0, without the learned correction, into level 1 (interior rows) of an
// FP64 context: one stage with a_n = 0, a_s = 1, a_L = 1 and dt = 1.
int rhs_stage(elb_ctx *c)
{
    const double dt = c->dt;
    const bool on = c->closure_on;
    const uint32_t launches = c->launches;
    c->dt = 1.0;
    c->closure_on = false;
    launch_stage(c, 0, 1, 0.0, 1.0);
    c->dt = dt;
    c->closure_on = on;
    c->launches = launches;
    return hip_check(c, hipGetLastError(), "rhs launch");
}

// f(std::integral_constant<int, q>) for the student node counts
template <typename F>
void with_student_q(int q, F f)
{
    switch (q) {
        case 8: f(std::integral_constant<int, 8>{}); break;
        case 12: f(std::integral_constant<int, 12>{}); break;
        default: f(std::integral_constant<int, 16>{}); break;  // closure contexts have q <= 16
    }
}

// Allocation-free loss: the per-block partial sums of k_mlp_loss live in a file-scope device
// array instead of the caller's workspace.  Every GPU the library runs on holds its own copy
// of `scratch` until the process ends.  In host code the name is only a stand-in for the
// symbol; kernels get the device address that hipGetSymbolAddress returns for the current
// device, looked up once per device and kept.
constexpr int kScratchDoubles = 256;  // k_mlp_loss launches at most 256 blocks
__device__ __align__(256) double scratch[kScratchDoubles];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_addr[kMaxDevices] = {};

int scratch_address(double **out, std::string *msg)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0) { *msg = "no current HIP device"; return ELB_EHIP; }
    if (dev >= kMaxDevices) { *msg = "device ordinal beyond 63"; return ELB_EUNSUPPORTED; }
    std::lock_guard<std::mutex> lk(g_scratch_mu);
    if (!g_scratch_addr[dev]) {
        void *ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            *msg = std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e);
            return ELB_EHIP;
        }
        g_scratch_addr[dev] = static_cast<double *>(ptr);
    }
    *out = g_scratch_addr[dev];
    return ELB_OK;
}

}  // namespace

extern "C" {

int64_t elb_mlp_param_count(void) { return MLP_PARAMS; }
int64_t elb_mlp_norm_count(void) { return MLP_NORM; }

int64_t elb_mlp_workspace_bytes(int64_t batch)
{
    if (batch < 1 || batch > kMaxBatch) return -1;
    return (int64_t)mlp_ws(batch).total;
}

int elb_mlp_round(const float *params, uint16_t *wb, void *stream)
{
    if (!params || !wb) return ELB_EINVAL;
    hipLaunchKernelGGL(k_round_bf16, dim3((MLP_PARAMS + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       params, (unsigned short *)wb, MLP_PARAMS);
    return hipGetLastError() == hipSuccess ? ELB_OK : ELB_EHIP;
}

int elb_mlp_forward(const float *params, const uint16_t *wb, const float *norm, const float *x,
                    const int32_t *index, int64_t batch, float *y, void *ws, void *stream)
{
    if (!params || !wb || !norm || !x || !y || !ws || batch < 1 || batch > kMaxBatch) return ELB_EINVAL;
    MlpWs w = mlp_ws(batch);
    char *base = (char *)ws;
    const int tiles = forward_tiles(batch), rows = tiles * TRAIN_ROWS;
    hipLaunchKernelGGL(k_mlp_forward, dim3((unsigned)((batch + rows - 1) / rows)), dim3(256), 0,
                       (hipStream_t)stream, (const unsigned short *)wb, params, norm, x, (const int *)index,
                       (int)batch, tiles, y, (unsigned short *)(base + w.a0), (float *)(base + w.z));
    return hipGetLastError() == hipSuccess ? ELB_OK : ELB_EHIP;
}

int elb_mlp_loss(const float *y, const float *t, const int32_t *index, const float *norm, int64_t batch,
                 int32_t q_out, float *dy, double *loss, void *ws, void *stream)
{
    if (!y || !t || !norm || !dy || !loss || !ws || batch < 1 || batch > kMaxBatch || q_out < 1 ||
        q_out > MLP_OUT)
        return ELB_EINVAL;
    MlpWs w = mlp_ws(batch);
    double *lp = (double *)((char *)ws + w.lpart);
    hipLaunchKernelGGL(k_mlp_loss, dim3(w.nblk_l), dim3(256), 0, (hipStream_t)stream, y, t, (const int *)index,
                       norm, (int)batch, q_out, dy, lp);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, (hipStream_t)stream, lp, w.nblk_l,
                       1.0 / ((double)batch * q_out), loss);
    return hipGetLastError() == hipSuccess ? ELB_OK : ELB_EHIP;
}

int elb_mlp_loss_noalloc(const float *y, const float *t, const int32_t *index, const float *norm,
                         int64_t batch, int32_t q_out, float *dy, double *loss, void *stream)
{
    if (!y || !t || !norm || !dy || !loss) {
        g_create_error = "elb_mlp_loss_noalloc: y, t, norm, dy and loss must be non-NULL";
        return ELB_EINVAL;
    }
    if (batch < 1 || batch > kMaxBatch || q_out < 1 || q_out > MLP_OUT) {
        g_create_error = "elb_mlp_loss_noalloc: batch must be in [1, 2^24] and q_out in [1, 16]";
        return ELB_EINVAL;
    }
    // one partial sum per block; the grid is capped so that they fit the scratch array
    const int nblk = (int)std::min<int64_t>(kScratchDoubles, (batch * MLP_OUT + 255) / 256);
    double *lp = nullptr;
    std::string msg;
    if (int rc = scratch_address(&lp, &msg)) {
        g_create_error = "elb_mlp_loss_noalloc: " + msg;
        return rc;
    }
    hipLaunchKernelGGL(k_mlp_loss, dim3(nblk), dim3(256), 0, (hipStream_t)stream, y, t, (const int *)index,
                       norm, (int)batch, q_out, dy, lp);
    hipLaunchKernelGGL(k_sum_partials, dim3(1), dim3(256), 0, (hipStream_t)stream, lp, nblk,
                       1.0 / ((double)batch * q_out), loss);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) {
        g_create_error = std::string("elb_mlp_loss_noalloc: ") + hipGetErrorString(e);
        return ELB_EHIP;
    }
    return ELB_OK;
}

int elb_mlp_backward(const uint16_t *wb, const float *dy, int64_t batch, float *grad, void *ws, void *stream)
{
    if (!wb || !dy || !grad || !ws || batch < 1 || batch > kMaxBatch) return ELB_EINVAL;
    MlpWs w = mlp_ws(batch);
    char *base = (char *)ws;
    hipStream_t st = (hipStream_t)stream;
    const float *z = (const float *)(base + w.z);
    float *dz = (float *)(base + w.dz);
    unsigned short *gt = (unsigned short *)(base + w.gt), *g4t = (unsigned short *)(base + w.g4t);
    hipLaunchKernelGGL(k_mlp_backward, dim3((unsigned)((batch + TRAIN_ROWS - 1) / TRAIN_ROWS)), dim3(256), 0, st,
                       (const unsigned short *)wb, dy, z, (const unsigned short *)(base + w.a0), (int)batch, dz, gt,
                       (unsigned short *)(base + w.at), w.lstride, g4t, (unsigned short *)(base + w.a0t));
    hipLaunchKernelGGL(k_mlp_wgrad, dim3(w.nblk_w, 4), dim3(WGRAD_THREADS), 0, st, dy, (const float *)dz,
                       (const unsigned short *)gt, w.lstride, (const unsigned short *)g4t,
                       (const unsigned short *)(base + w.a0t), (const unsigned short *)(base + w.at), w.lstride, (int)batch,
                       (float *)(base + w.part));
    hipLaunchKernelGGL(k_mlp_reduce, dim3((MLP_PARAMS + 63) / 64), dim3(64), 0, st,
                       (const float *)(base + w.part), w.nblk_w, grad);
    return hipGetLastError() == hipSuccess ? ELB_OK : ELB_EHIP;
}

int elb_mlp_adam(float *params, uint16_t *wb, float *m, float *v, const float *grad, int64_t step, float lr,
                 float beta1, float beta2, float eps, void *stream)
{
    if (!params || !wb || !m || !v || !grad || step < 1 || !(lr > 0) || !(beta1 >= 0 && beta1 < 1) ||
        !(beta2 >= 0 && beta2 < 1) || !(eps > 0))
        return ELB_EINVAL;
    float c1 = (float)(1.0 - std::pow((double)beta1, (double)step));
    float c2 = (float)(1.0 - std::pow((double)beta2, (double)step));
    hipLaunchKernelGGL(k_mlp_adam, dim3((MLP_PARAMS + 255) / 256), dim3(256), 0, (hipStream_t)stream, params,
                       (unsigned short *)wb, m, v, grad, MLP_PARAMS, lr, beta1, beta2, eps, c1, c2);
    return hipGetLastError() == hipSuccess ? ELB_OK : ELB_EHIP;
}

int elb_mlp_normaliser(const float *x, int64_t n, int32_t dim, double margin, float *mean, float *std_,
                       float *lo, float *hi)
{
    if (!x || n < 1 || dim < 1 || !mean || !std_ || !(margin >= 0)) return ELB_EINVAL;
    for (int c = 0; c < dim; ++c) {
        double s = 0.0, s2 = 0.0;
        for (int64_t i = 0; i < n; ++i) {
            double v = x[i * dim + c];
            if (!std::isfinite(v)) return ELB_EINVAL;
            s += v;
        }
        double mu = s / (double)n;
        for (int64_t i = 0; i < n; ++i) {
            double d = x[i * dim + c] - mu;
            s2 += d * d;
        }
        double sd = std::sqrt(s2 / (double)n);
        if (!(sd > 1e-12 * std::fmax(1.0, std::fabs(mu)))) sd = 1.0;
        mean[c] = (float)mu;
        std_[c] = (float)sd;
        if (lo && hi) {
            double mn = 1e300, mx = -1e300;
            for (int64_t i = 0; i < n; ++i) {
                double v = ((double)x[i * dim + c] - mean[c]) / std_[c];
                mn = std::fmin(mn, v);
                mx = std::fmax(mx, v);
            }
            double w = margin * (mx - mn);
            lo[c] = (float)(mn - w);
            hi[c] = (float)(mx + w);
        }
    }
    return ELB_OK;
}

int elb_projection(int32_t q_from, int32_t q_to, double *P)
{
    if (!P) return ELB_EINVAL;
    return projection_host(q_from, q_to, P);
}

int elb_lift(int32_t q_from, int32_t q_to, double *L)
{
    if (!L) return ELB_EINVAL;
    return lift_host(q_from, q_to, L);
}

int elb_closure_lift(elb_ctx *student, elb_ctx *teacher)
{
    if (!student || !teacher) return ELB_EINVAL;
    elb_ctx *s = student, *t = teacher;
    if (!t->has_state || !s->has_state) return fail(t, ELB_ESTATE, "teacher and student need a state");
    if (t->P.precision != ELB_FP64 || s->P.precision != ELB_FP64) return fail(t, ELB_EINVAL, "the lift needs FP64 contexts");
    if (!s->P.closure) return fail(t, ELB_EINVAL, "the student must be created with closure = 1");
    if (t->P.nx != s->P.nx || t->P.bc != s->P.bc || t->P.length != s->P.length || s->Q > t->Q)
        return fail(t, ELB_EINVAL, "teacher and student differ in grid or boundaries, or q_student > q_teacher");
    if (t->stream != s->stream) return fail(t, ELB_EINVAL, "teacher and student must share a stream");
    const int nx = s->P.nx, QT = t->Q, QS = s->Q;
    std::vector<double> Lam((size_t)QT * QS);
    int rc = lift_host(QS, QT, Lam.data());
    if (rc) return fail(t, rc, "lift");
    hipStream_t st = s->stream;
    double *dL = s->dev<double>(s->L.proj);  // QT x QS <= 208 x 16 fits the projection buffer
    rc = upload(s, s->L.proj, Lam.data(), sizeof(double) * Lam.size());
    if (rc) return fail(t, rc, "lift: %s", s->err.c_str());
    drop_ctx_graph(t);
    const double *sp = s->dev<double>(s->L.psi[0]) + (size_t)NG * 2 * QS;
    double *tp = t->dev<double>(t->L.psi[0]) + (size_t)NG * 2 * QT;
    with_student_q(QS, [&](auto q) {
        hipLaunchKernelGGL(k_lift_rows<decltype(q)::value>, dim3((nx + LIFT_ROWS - 1) / LIFT_ROWS, 2), dim3((QT + 63) / 64 * 64), 0,
                           st, (const double *)dL, sp, QT, tp, nx);
    });
    rc = hip_check(t, hipGetLastError(), "lift launch");
    if (rc) return rc;
    rc = hip_check(t, hipStreamSynchronize(st), "lift");
    if (rc) return rc;
    t->steps = 0;
    t->launches = 0;
    return ELB_OK;
}

int elb_rhs(elb_ctx *c, double *phi_rhs, double *theta_rhs)
{
    if (!c) return ELB_EINVAL;
    if (!c->has_state) return fail(c, ELB_ESTATE, "no state set");
    if (c->P.precision != ELB_FP64) return fail(c, ELB_EINVAL, "elb_rhs needs an FP64 context");
    int rc = rhs_stage(c);
    if (rc) return rc;
    const int nx = c->P.nx, Q = c->Q;
    const size_t n = (size_t)nx * Q, in = sizeof(double) * (size_t)NG * 2 * Q;
    // the two planes fill the interior of level 2
    double *planes = c->dev<double>(c->L.psi[2] + in);
    hipLaunchKernelGGL(k_rhs_planes, plane_grid(n), dim3(PLANE_THREADS), 0, c->stream,
                       (const double *)c->dev<double>(c->L.psi[1] + in), (const double *)c->dev<double>(c->L.psi[0] + in), nx, Q,
                       planes, planes + n);
    rc = hip_check(c, hipGetLastError(), "rhs launch");
    if (!rc) rc = check_flag(c);
    if (rc) return rc;
    const size_t at = c->L.psi[2] + in, nb = sizeof(double) * n;
    return download(c, {{phi_rhs, at, nb}, {theta_rhs, at + nb, nb}});
}

int elb_closure_sample(elb_ctx *teacher, elb_ctx *student, float *x, float *y)
{
    if (!teacher || !student || !x || !y) return ELB_EINVAL;
    elb_ctx *t = teacher, *s = student;
    if (!t->has_state || !s->has_state) return fail(s, ELB_ESTATE, "teacher and student need a state");
    if (t->P.precision != ELB_FP64 || s->P.precision != ELB_FP64) return fail(s, ELB_EINVAL, "sampling needs FP64 contexts");
    if (!s->P.closure) return fail(s, ELB_EINVAL, "the student must be created with closure = 1");
    if (t->P.nx != s->P.nx || t->P.bc != s->P.bc || t->P.length != s->P.length || s->Q > t->Q)
        return fail(s, ELB_EINVAL, "teacher and student differ in grid or boundaries, or q_student > q_teacher");
    if (t->stream != s->stream) return fail(s, ELB_EINVAL, "teacher and student must share a stream");
    const int nx = s->P.nx, QT = t->Q, QS = s->Q;
    std::vector<double> P((size_t)QS * QT), Pt((size_t)QT * MLP_OUT, 0.0);
    int rc = projection_host(QT, QS, P.data());
    if (rc) return fail(s, rc, "projection");
    for (int j = 0; j < QS; ++j)
        for (int k = 0; k < QT; ++k) Pt[(size_t)k * MLP_OUT + j] = P[(size_t)j * QT + k];
    hipStream_t st = s->stream;
    double *dP = s->dev<double>(s->L.proj);
    rc = upload(s, s->L.proj, Pt.data(), sizeof(double) * Pt.size());
    if (rc) return rc;
    rc = rhs_stage(t);                                         // psi_T + L_T into teacher level 1
    if (rc) return fail(s, rc, "teacher rhs: %s", t->err.c_str());
    const size_t offT = (size_t)NG * 2 * QT, offS = (size_t)NG * 2 * QS;
    const double *tp0 = t->dev<double>(t->L.psi[0]) + offT, *tp1 = t->dev<double>(t->L.psi[1]) + offT;
    double *sp = s->dev<double>(s->L.psi[0]) + offS, *Lt = s->dev<double>(s->L.psi[2]) + offS;
    with_student_q(QS, [&](auto q) {
        hipLaunchKernelGGL(k_project_rows<decltype(q)::value>, dim3((nx + PROJ_THREADS - 1) / PROJ_THREADS, 3),
                           dim3(PROJ_THREADS), 0, st, (const double *)dP, tp0, tp1, QT, sp, Lt, nx);
    });
    rc = hip_check(s, hipGetLastError(), "projection launch");
    if (!rc) rc = rhs_stage(s);                                // and of the projected state
    if (rc) return rc;
    launch_closure_rows(s, 0);
    hipLaunchKernelGGL(k_closure_sample, dim3((nx + 255) / 256), dim3(256), 0, st, s->dev<double>(s->L.rows5),
                       closure_const(s), nx, QS, (const double *)Lt, (const double *)(s->dev<double>(s->L.psi[1]) + offS),
                       (const double *)sp, 2 * QS, s->dev<float>(s->L.sx), s->dev<float>(s->L.sy));
    rc = hip_check(s, hipGetLastError(), "sample launch");
    if (!rc) rc = download(s, {{x, s->L.sx, sizeof(float) * MLP_IN * (size_t)nx}, {y, s->L.sy, sizeof(float) * QS * (size_t)nx}});
    if (rc) return rc;
    rc = check_flag(t);
    if (rc) return fail(s, rc, "teacher: %s", t->err.c_str());
    return check_flag(s);
}

int elb_set_closure(elb_ctx *c, const float *params, const float *norm, int32_t enabled)
{
    if (!c) return ELB_EINVAL;
    if (!c->P.closure) return fail(c, ELB_EINVAL, "context created with closure = 0");
    drop_ctx_graph(c);  // the closure kernels are part of a captured step
    if (enabled < 0 || enabled > 2) return fail(c, ELB_EINVAL, "enabled must be 0, 1 or 2");
    if (!enabled) { c->closure_on = false; return ELB_OK; }
    if (!params || !norm) return fail(c, ELB_EINVAL, "NULL parameters");
    for (int j = 0; j < MLP_PARAMS; ++j)
        if (!std::isfinite(params[j])) return fail(c, ELB_EINVAL, "non-finite parameter %d", j);
    for (int j = 0; j < MLP_NORM; ++j)
        if (std::isnan(norm[j])) return fail(c, ELB_EINVAL, "NaN in the normalisation block");
    for (int j = 0; j < MLP_IN; ++j)
        if (!(norm[NRM_IN_STD + j] > 0) || !std::isfinite(norm[NRM_IN_MEAN + j]))
            return fail(c, ELB_EINVAL, "input std must be > 0");
    for (int j = 0; j < c->Q; ++j)
        if (!(norm[NRM_OUT_STD + j] > 0) || !std::isfinite(norm[NRM_OUT_MEAN + j]))
            return fail(c, ELB_EINVAL, "output std must be > 0");
    std::vector<unsigned short> wb(MLP_PARAMS);
    for (int j = 0; j < MLP_PARAMS; ++j) wb[j] = host_bf16(params[j]);
    // conservative projector I - V (V^T V)^{-1} V^T, V = [1, p, p^2] on the student nodes
    const int Q = c->Q;
    double G[3][3] = {{0}}, Gi[3][3];
    for (int k = 0; k < Q; ++k) {
        double v[3] = {1.0, c->p[k], c->p[k] * c->p[k]};
        for (int a = 0; a < 3; ++a)
            for (int b = 0; b < 3; ++b) G[a][b] += v[a] * v[b];
    }
    double det = G[0][0] * (G[1][1] * G[2][2] - G[1][2] * G[2][1]) - G[0][1] * (G[1][0] * G[2][2] - G[1][2] * G[2][0]) +
                 G[0][2] * (G[1][0] * G[2][1] - G[1][1] * G[2][0]);
    for (int a = 0; a < 3; ++a)
        for (int b = 0; b < 3; ++b) {
            int a1 = (b + 1) % 3, a2 = (b + 2) % 3, b1 = (a + 1) % 3, b2 = (a + 2) % 3;
            Gi[a][b] = (G[a1][b1] * G[a2][b2] - G[a1][b2] * G[a2][b1]) / det;
        }
    std::vector<double> pc(MLP_OUT * MLP_OUT, 0.0);
    for (int i = 0; i < Q; ++i)
        for (int j = 0; j < Q; ++j) {
            double vi[3] = {1.0, c->p[i], c->p[i] * c->p[i]}, vj[3] = {1.0, c->p[j], c->p[j] * c->p[j]};
            double s = 0.0;
            for (int a = 0; a < 3; ++a)
                for (int b = 0; b < 3; ++b) s += vi[a] * Gi[a][b] * vj[b];
            pc[i * MLP_OUT + j] = (i == j ? 1.0 : 0.0) - s;
        }
    hipError_t e = hipMemcpyAsync(c->dev<float>(c->L.mparams), params, sizeof(float) * MLP_PARAMS, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(c->dev<unsigned short>(c->L.mwb), wb.data(), sizeof(unsigned short) * MLP_PARAMS, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(c->dev<float>(c->L.mnorm), norm, sizeof(float) * MLP_NORM, hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(c->dev<double>(c->L.pc), pc.data(), sizeof(double) * pc.size(), hipMemcpyHostToDevice, c->stream);
    if (e == hipSuccess) e = hipMemsetAsync(c->dev<unsigned long long>(c->L.outside), 0, sizeof(unsigned long long), c->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(c->stream);
    int rc = hip_check(c, e, "closure upload");
    if (rc) return rc;
    c->closure_on = true;
    c->closure_fused = enabled == 1;
    return ELB_OK;
}

int elb_closure_outside(elb_ctx *c, int64_t *count, int32_t reset)
{
    if (!c || !count) return ELB_EINVAL;
    if (!c->P.closure) return fail(c, ELB_EINVAL, "context created with closure = 0");
    unsigned long long v = 0;
    int rc = hip_check(c, hipMemcpyAsync(&v, c->dev<unsigned long long>(c->L.outside), sizeof v, hipMemcpyDeviceToHost, c->stream), "counter copy");
    if (!rc && reset) rc = hip_check(c, hipMemsetAsync(c->dev<unsigned long long>(c->L.outside), 0, sizeof v, c->stream), "counter reset");
    if (!rc) rc = hip_check(c, hipStreamSynchronize(c->stream), "stream sync");
    if (rc) return rc;
    *count = (int64_t)v;
    return ELB_OK;
}

}  // extern "C"
