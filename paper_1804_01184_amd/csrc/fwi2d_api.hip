// C ABI of libfwi2d: plans, workspace layout and the time-stepping schedule
// (forward sweep with checkpoints, then per segment a recompute that stores
// the pressure history followed by the adjoint sweep).
#include "../../include/fwi2d.h"
#include "fwi2d_internal.h"

#include <algorithm>
#include <cstdarg>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

using namespace fwi;

namespace {

thread_local std::string g_err;

fwi_status fail(fwi_status s, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
fwi_status fail(fwi_status s, const char *fmt, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(buf, sizeof buf, fmt, ap);
    va_end(ap);
    g_err = buf;
    return s;
}

constexpr size_t kAlign = 256;
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
inline long long align64(long long v) { return (v + 63) / 64 * 64; }
// the smallest band height giving as many bands of Nz rows as H does: a
// launch of a few rounds of waves lasts about as long as its tallest band
inline int balanced_rows(long long Nz, int H)
{
    const long long bands = (Nz + H - 1) / H;
    return (int)((Nz + bands - 1) / bands);
}

// Stability limit of the fourth-order staggered leapfrog scheme in 2-D:
// vmax dt sqrt(1/dx^2 + 1/dz^2) (|c1| + |c2|) <= 1.
double stability_number(const fwi_grid &g)
{
    return g.vmax * g.dt * std::sqrt(1.0 / (g.dx * g.dx) + 1.0 / (g.dz * g.dz)) *
           (9.0 / 8.0 + 1.0 / 24.0);
}

}  // namespace

struct fwi_plan {
    fwi_grid grid;
    int S, nrec, per_shot;
    int Spad;   // shots of a batched launch: S padded to whole shot groups
    int mode, k, nseg;
    Sweep sweep;   // batched decomposition (band rows, shots per group)
    bool two_step = false;   // forward sweeps use the two-step kernel
    Sweep sweep2;            // its decomposition
    bool samp_nodes = false; // its intermediate level, when only sampled, is
                             // kept at the receiver nodes alone
    bool adj2 = false;       // adjoint sweeps use the two-step kernel
    Sweep sweep_a2;          // its decomposition, with shot groups of its own
    int adj_list = 0;        // listed nodes of the strip adjoints (0: they do not add R^T r)
    int samp_list = 0;       // listed nodes of the two-step forward kernel
    // tile kernels (several steps per launch, state in registers)
    struct TileRun {   // most steps per launch and the axes of its tiles
        int T = 0;
        TileAxis x{}, z{};
    };
    struct Tiles {
        bool on = false;    // the sweeps of a gradient
        bool fwd = false;   // a forward sweep by itself
        TileRun call, keep, adj;   // forward call; forward and adjoint sweeps of a gradient
        int levels = 0;            // of the forward call's sampling buffer
    } tile;
    int device;
    Geo geo;
    long long SS, ST;  // per-shot floats of a state record / a store record
    // Geometry tables.  The plan holds no device memory: every call that
    // needs them copies the host image `blob` into its workspace and builds
    // the damping tables there (TabOff: byte offsets in the workspace's
    // table region).
    struct TabOff {
        size_t pml, zpad, st;                            // built on the device
        size_t sij, sw, ri, rw, in, is, ip, ir, iw, win; // copied from blob
        size_t swin, rnode, rptr, irc, aln, alc, alp, slc, slp;   // copied from blob
        size_t blob;                                     // offset of blob's image
        size_t bytes;                                    // size of the region
    } to{};
    std::vector<char> blob;
    hipEvent_t blob_ev = nullptr;   // recorded after the last copy of blob
    int inj_nodes = 0;
    std::vector<int> shot_node_ptr;  // [S+1] node range of each shot
    std::vector<int2> h_src_ij;
    std::vector<float4> h_src_w;
    // per-launch event timing (instrumentation)
    bool timing = false;
    struct Mark {
        int cls;
        hipEvent_t a, b;
    };
    std::vector<Mark> marks;
    std::vector<hipEvent_t> spare;
    fwi_timing acc{};
    // workspace holding the state kept by fwi_forward_keep (null: none)
    void *kept_ws = nullptr;
};

namespace {

hipEvent_t take_event(fwi_plan *p)
{
    hipEvent_t e = nullptr;
    if (!p->spare.empty()) {
        e = p->spare.back();
        p->spare.pop_back();
    } else if (hipEventCreate(&e) != hipSuccess) {
        e = nullptr;
    }
    return e;
}

// Brackets the launches issued in its scope with events when timing is on.
// With by_launch, the events are not recorded here: the caller hands them
// (b, e) to a launch that stamps them with its dispatch's start and end.
struct Timed {
    fwi_plan *p;
    hipStream_t st;
    int cls;
    bool by_launch;
    hipEvent_t b = nullptr, e = nullptr;
    Timed(fwi_plan *p_, hipStream_t st_, int cls_, bool by_launch_ = false)
        : p(p_), st(st_), cls(cls_), by_launch(by_launch_)
    {
        if (!p->timing)
            return;
        b = take_event(p);
        e = take_event(p);
        if (!b || !e) {
            b = e = nullptr;
            return;
        }
        if (!by_launch)
            (void)hipEventRecord(b, st);
    }
    ~Timed()
    {
        if (!b || !e)
            return;
        if (!by_launch)
            (void)hipEventRecord(e, st);
        p->marks.push_back({cls, b, e});
    }
};

// Folds the recorded marks into the per-class sums.
fwi_status collect_marks(fwi_plan *p)
{
    for (auto &m : p->marks) {
        float ms = 0.0f;
        if (hipEventSynchronize(m.b) != hipSuccess ||
            hipEventElapsedTime(&ms, m.a, m.b) != hipSuccess)
            return FWI_EDEVICE;
        p->acc.launches[m.cls] += 1;
        p->acc.ms[m.cls] += ms;
        p->spare.push_back(m.a);
        p->spare.push_back(m.b);
    }
    p->marks.clear();
    return FWI_OK;
}

struct Layout {
    size_t tab;   // geometry and damping tables (FWI_OP_FORWARD / FWI_OP_GRADIENT)
    size_t Kphys, rhophys, Kpad, bx, bz, Q;
    size_t work[2], lam[2];
    size_t ckpt, store, gpart, fold, traces, resid, partials;
    size_t mid;   // p^{n+1} of a two-step launch outside the stored history
    size_t injacc;   // R^T r of up to stage_steps steps per injection node (batched adjoint)
    size_t nodes;    // p^{n+1} at the receiver nodes (two-step forward, level only sampled)
    size_t hist;     // levels to sample (tile forward without a kept history)
    size_t total;
};

int batch_of(const fwi_plan *p) { return p->mode == FWI_EXEC_PLAIN ? 1 : p->Spad; }
// partial gradients of a backward sweep
int partials_of(const fwi_plan *p)
{
    return p->mode == FWI_EXEC_PLAIN ? 1
           : p->tile.on              ? p->S
           : p->adj2                 ? p->sweep_a2.ngroups
                                     : p->sweep.ngroups;
}

// Steps of R^T r staged at a time for the batched adjoints (even): 64, fewer where
// the sums of a dense acquisition's nodes would take more than 256 MB (a receiver
// on every node of 64 shots of 1081 x 1081 would stage 23 GB).
constexpr int kStageSteps = 64;
int stage_steps(const fwi_plan *p)
{
    const long long nodes = std::max(1, std::max(p->inj_nodes, p->adj_list));
    return (int)std::max(2LL, std::min<long long>(kStageSteps, (1LL << 26) / nodes / 2 * 2));
}

Layout layout(const fwi_plan *p, int op)
{
    Layout L{};
    size_t off = 0;
    // every array is followed by at least 64 spare bytes (the batched
    // kernels may read a few bytes past a field and discard them); arrays of
    // 8 MB and more start on 2 MB boundaries (huge-page boundaries of a 2
    // MB-aligned workspace).  Measured on MI355X on one and the same device
    // buffer, the sweeps take the same time (within 0.2 %) with 256-byte
    // starts: the boundaries cost at most a few MB and buy nothing measurable
    auto take = [&](size_t floats) {
        const size_t bytes = floats * sizeof(float) + 64;
        off = align_up(off, bytes >= (8u << 20) ? (size_t)2 << 20 : kAlign);
        size_t o = off;
        off = align_up(off + bytes, kAlign);
        return o;
    };
    const Geo &g = p->geo;
    long long nphys = (long long)g.nz * g.nx;
    long long ntr = (long long)p->S * p->nrec * p->grid.nt;
    int B = batch_of(p);
    if (op == FWI_OP_MISFIT) {
        L.partials = take(misfit_blocks(ntr));
        L.total = off;
        return L;
    }
    L.tab = off;
    off = align_up(off + p->to.bytes + 64, kAlign);
    L.Kphys = take(nphys);
    L.rhophys = take(nphys);
    // K, bx, bz as one block (the batched kernels address them from K)
    L.Kpad = take(3 * g.N);
    L.bx = L.Kpad + g.N * sizeof(float);
    L.bz = L.Kpad + 2 * g.N * sizeof(float);
    L.Q = take((size_t)p->S * p->grid.nt);
    L.work[0] = take((size_t)B * p->SS);
    L.work[1] = take((size_t)B * p->SS);
    if (p->tile.fwd && op == FWI_OP_FORWARD)
        L.hist = take((size_t)p->tile.levels * p->S * align64(g.N));
    if (p->two_step)
        L.mid = take((size_t)B * p->ST);
    if (p->samp_nodes)
        L.nodes = take((size_t)std::max(p->samp_list, 1));
    if (op == FWI_OP_GRADIENT) {
        L.lam[0] = take((size_t)B * p->SS);
        L.lam[1] = take((size_t)B * p->SS);
        L.ckpt = take((size_t)(p->nseg - 1) * B * p->SS);
        L.store = take((size_t)(p->k + 1) * B * p->ST);
        L.gpart = take((size_t)partials_of(p) * 3 * g.N);
        L.fold = take(2 * (size_t)g.N);
        L.traces = take(ntr);
        L.resid = take(ntr);
        L.partials = take(misfit_blocks(ntr));
        if (p->mode != FWI_EXEC_PLAIN)
            L.injacc = take((size_t)std::max(std::max(p->inj_nodes, p->adj_list), 1) *
                                std::min(stage_steps(p), p->grid.nt) + 64);
    }
    L.total = off;
    if (op == FWI_OP_GRADIENT)   // a gradient workspace also serves a forward call
        L.total = std::max(L.total, layout(p, FWI_OP_FORWARD).total);
    return L;
}

// Pointers into a workspace for one batch of shots.
struct State {
    Fld vx, vz, p, pz;
};

State state_at(float *base, const fwi_plan *pl)
{
    const Geo &g = pl->geo;
    State s;
    s.vx = {base, pl->SS};
    s.vz = {base + g.N, pl->SS};
    s.p = {base + 2 * g.N, pl->SS};
    s.pz = {base + 3 * g.N, pl->SS};
    return s;
}

// Device addresses of the plan's tables in a workspace.
struct DevTabs {
    float *pml = nullptr, *zpad = nullptr;
    SweepTables *sweep_tabs = nullptr;
    int2 *src_ij = nullptr;
    float4 *src_w = nullptr;
    long long *rec_idx = nullptr;
    float4 *rec_w = nullptr;
    long long *inj_node = nullptr;
    int *inj_shot = nullptr, *inj_cptr = nullptr, *inj_crec = nullptr;
    float *inj_cw = nullptr;
    unsigned *inj_win = nullptr;   // strip adjoint: [Spad][Nz + 2 kZPad][strips]
    int *al_node = nullptr, *al_col = nullptr, *al_ptr = nullptr;   // its node list
    unsigned *samp_win = nullptr;  // two-step forward: [S][Nz][strips]
    int *sl_col = nullptr, *sl_ptr = nullptr;   // its node list
    int4 *rec_node = nullptr;      // [S][nrec]: node index of each bilinear corner
    int *inj_rowptr = nullptr;     // tile adjoint: [S][Nz + 1] first node of each row
    unsigned *inj_rc = nullptr;    // tile adjoint: row << 16 | column of each node
};

struct Ctx {
    fwi_plan *pl;
    hipStream_t st;
    char *ws;
    Layout L;
    DevTabs tb;
    Pml t;
    Mdl m;
    float *f(size_t off) const { return (float *)(ws + off); }
};

Pml pml_tables(const fwi_plan *p, const float *b)
{
    const Geo &g = p->geo;
    Pml t;
    t.ax = b;
    t.bx = b + g.Nx;
    t.ahx = b + 2 * g.Nx;
    t.bhx = b + 3 * g.Nx;
    const float *z = b + 4 * g.Nx;
    t.az = z;
    t.bz = z + g.Nz;
    t.ahz = z + 2 * g.Nz;
    t.bhz = z + 3 * g.Nz;
    return t;
}

// Copies the pressure and its absorbing-layer split of `nb` shots.
__global__ void k_copy_p(Fld dp, Fld dpz, Fld sp, Fld spz, long long N, long long Npml, int nb)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long per = N + Npml;
    long long total = per * nb;
    long long stride = (long long)gridDim.x * blockDim.x;
    for (; i < total; i += stride) {
        int s = (int)(i / per);
        long long r = i - (long long)s * per;
        if (r < N)
            dp.shot(s)[r] = sp.shot(s)[r];
        else
            dpz.shot(s)[r - N] = spz.shot(s)[r - N];
    }
}

void copy_p(const Ctx &c, Fld dp, Fld dpz, Fld sp, Fld spz, int nb)
{
    const Geo &g = c.pl->geo;
    long long total = (g.N + g.Npml) * nb;
    unsigned blocks = (unsigned)std::min<long long>((total + 255) / 256, 8192);
    Timed tm(c.pl, c.st, FWI_KC_OTHER);
    hipLaunchKernelGGL(k_copy_p, dim3(blocks), dim3(256), 0, c.st, dp, dpz, sp, spz, g.N, g.Npml,
                       nb);
}

// Source / receiver tables of shots [s0, s0 + nb).
Src src_of(const Ctx &c, int s0)
{
    Src s;
    s.ij = c.tb.src_ij + s0;
    s.w = c.tb.src_w + s0;
    s.Q = c.f(c.L.Q) + (size_t)s0 * c.pl->grid.nt;
    s.nt = c.pl->grid.nt;
    return s;
}

Rec rec_of(const Ctx &c, int s0)
{
    Rec r;
    r.idx = c.tb.rec_idx + (size_t)s0 * c.pl->nrec;
    r.w = c.tb.rec_w + (size_t)s0 * c.pl->nrec;
    r.nrec = c.pl->nrec;
    return r;
}

Inj inj_of(const Ctx &c, int s0, int nb)
{
    const fwi_plan *p = c.pl;
    int a = p->shot_node_ptr[s0], b = p->shot_node_ptr[s0 + nb];
    Inj in;
    in.node = c.tb.inj_node + a;
    in.shot = c.tb.inj_shot + a;
    in.cptr = c.tb.inj_cptr + a;
    in.crec = c.tb.inj_crec;
    in.cw = c.tb.inj_cw;
    in.nnodes = b - a;
    return in;
}

// Real (not padding) shots among [s0, s0 + nb).
int real_shots(const fwi_plan *p, int s0, int nb) { return std::max(0, std::min(nb, p->S - s0)); }

// Record descriptor of a batch: `f` is the first field of the record, the
// record spans `floats` floats from there.
Recd recd(const Fld &f, long long floats)
{
    return Recd{f.p, (unsigned)(f.ss * sizeof(float)), (unsigned)(floats * sizeof(float))};
}

// One forward step n -> n+1 for shots [s0, s0+nb) from `in` to `out`.
void step_fwd(const Ctx &c, int s0, int nb, const State &in, const State &out, int n)
{
    const fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    Src src = src_of(c, s0);
    if (p->mode == FWI_EXEC_PLAIN) {
        {
            Timed tm(c.pl, c.st, FWI_KC_PLAIN_VEL);
            launch_plain_vel(g, c.t, c.m, in.vx.p, in.vz.p, out.vx.p, out.vz.p, in.p.p, c.st);
        }
        Timed tm(c.pl, c.st, FWI_KC_PLAIN_PRES);
        launch_plain_pres(g, c.t, c.m, out.vx.p, out.vz.p, in.p.p, in.pz.p, out.p.p, out.pz.p,
                          p->h_src_ij[s0], p->h_src_w[s0], src.Q, n, c.st);
    } else {
        // velocity records: vx then vz; pressure records: p then its split,
        // N floats apart in state records and store slots alike
        FwdStep a;
        a.vin = recd(in.vx, 2 * g.N);
        a.pin = recd(in.p, g.N + g.Npml);
        a.vout = recd(out.vx, 2 * g.N);
        a.pout = recd(out.p, g.N + g.Npml);
        a.Q = src.Q;
        a.n = n;
        Timed tm(c.pl, c.st, FWI_KC_FWD_STEP, true);
        launch_fused_fwd(g, c.tb.pml, c.m.K, c.tb.sweep_tabs, p->S, p->sweep, a, c.st, tm.b,
                         tm.e);
    }
}

// Two forward steps n -> n+2 for shots [s0, s0+nb) (batched only): `mid`
// (a pressure record: p, then its split N floats later) receives p^{n+1},
// `out` the state at n+2; out's velocities must not be in's.
void step_fwd2(const Ctx &c, int s0, int nb, const State &in, Fld mid, const State &out, int n,
               int midw = 0)
{
    const fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    (void)nb;
    FwdStep2 a;
    a.vin = recd(in.vx, 2 * g.N);
    a.pin = recd(in.p, g.N + g.Npml);
    a.vout = recd(out.vx, 2 * g.N);
    a.pout = recd(out.p, g.N + g.Npml);
    a.pmid = recd(mid, g.N + g.Npml);
    a.zpad = c.tb.zpad;
    a.Q = src_of(c, s0).Q;
    a.nodes = midw == 1 ? c.f(c.L.nodes) : nullptr;
    a.nwin = c.tb.samp_win;
    a.nptr = c.tb.sl_ptr;
    a.ncol = c.tb.sl_col;
    a.midw = midw;
    a.n = n;
    Timed tm(c.pl, c.st, FWI_KC_FWD_PAIR, true);
    launch_fused_fwd2(g, c.tb.pml, c.m.K, c.tb.sweep_tabs, p->S, p->sweep2, a, c.st, tm.b, tm.e);
}

// One plain adjoint step n of shot s0: injects R^T r^n into `in`, then writes
// the adjoint state of step n into `out` and accumulates the sensitivities
// into gpart.  pn, pn1 (and splits): pressure levels n and n+1.
void step_adj_plain(const Ctx &c, int s0, const State &in, const State &out, Fld pn, Fld pzn,
                    Fld pn1, Fld pzn1, const float *resid, float *gpart, int n)
{
    const fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    {
        Timed tm(c.pl, c.st, FWI_KC_INJECT);
        launch_inject(g, inj_of(c, s0, 1), resid, p->nrec, p->grid.nt, n, in.p, s0, c.st);
    }
    {
        Timed tm(c.pl, c.st, FWI_KC_PLAIN_ADJ_A);
        launch_plain_adj_a(g, c.t, c.m, in.vx.p, in.vz.p, out.vx.p, out.vz.p, in.p.p, in.pz.p,
                           pn.p, pzn.p, pn1.p, pzn1.p, gpart, gpart + g.N, gpart + 2 * g.N, c.st);
    }
    Timed tm(c.pl, c.st, FWI_KC_PLAIN_ADJ_B);
    launch_plain_adj_b(g, c.t, c.m, out.vx.p, out.vz.p, in.p.p, in.pz.p, out.p.p, out.pz.p, c.st);
}

AdjNodes nodes_of(const Ctx &c)
{
    return AdjNodes{c.pl->adj_list ? c.tb.inj_win : nullptr, c.tb.al_ptr, c.tb.al_col};
}

// Batched adjoint step m: pm holds p^m, injv R^T r^{m-1} per node.
void step_adj(const Ctx &c, const State &in, const State &out, Fld pm, const float *injv,
              float *gpart)
{
    const fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    AdjStep a;   // adjoint records: lvx, lvz, lpx, lpz
    a.lin = recd(in.vx, 3 * g.N + g.Npml);
    a.lout = recd(out.vx, 3 * g.N + g.Npml);
    a.pn = recd(pm, g.N);
    a.nd = nodes_of(c);
    a.injv = injv;
    a.gpart = gpart;
    {
        Timed tm(c.pl, c.st, FWI_KC_ADJ_STEP, true);
        launch_fused_adj(g, c.tb.pml, c.m.K, p->sweep, a, c.st, tm.b, tm.e);
    }
    if (!a.nd.win) {
        Timed tm(c.pl, c.st, FWI_KC_INJECT);
        launch_inject_post(g, inj_of(c, 0, p->S), injv, p->sweep.spg, out.p, pm, c.m.K, gpart,
                           c.st);
    }
}

// Batched adjoint steps m, m-1: pm1 holds p^{m-1}, the next level of the
// store p^m; injA, injB: R^T r^{m-1}, R^T r^{m-2} per node (injB may be null).
void step_adj2(const Ctx &c, const State &in, const State &out, Fld pm1, const float *injA,
               const float *injB, float *gpart)
{
    const fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    AdjStep2 a;
    a.lin = recd(in.vx, 3 * g.N + g.Npml);
    a.lout = recd(out.vx, 3 * g.N + g.Npml);
    a.pm1 = recd(pm1, g.N);
    a.lvl = (unsigned)((size_t)p->Spad * p->ST * sizeof(float));   // (below 2 GiB: plan creation)
    a.gpart = gpart;
    a.zpad = c.tb.zpad;
    a.nd = nodes_of(c);
    a.injA = injA;
    a.injB = injB;
    Timed tm(c.pl, c.st, FWI_KC_ADJ_PAIR, true);
    launch_fused_adj2(g, c.tb.pml, c.m.K, p->sweep_a2, a, c.st, tm.b, tm.e);
}

void zero_state(const Ctx &c, float *base, int nb)
{
    Timed tm(c.pl, c.st, FWI_KC_OTHER);
    launch_fill(base, (long long)nb * c.pl->SS, 0.0f, c.st);
}

// Forward sweep over all steps for shots [s0, s0+nb).  With `keep`, the
// states at multiples of k go to checkpoint slots and the pressure of the
// last segment to the store (slot m holds p at step nlast + m).  `traces`
// (may be null) receives the receiver samples of these shots.
void sweep_forward(const Ctx &c, int s0, int nb, bool keep, float *traces)
{
    const fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    const int nt = p->grid.nt, k = p->k;
    const int nlast = (p->nseg - 1) * k;
    State w[2] = {state_at(c.f(c.L.work[0]), p), state_at(c.f(c.L.work[1]), p)};
    zero_state(c, c.f(c.L.work[0]), nb);
    State cur = w[0];
    int cw = 0;  // work buffer holding cur's velocities (-1: a checkpoint slot)
    Rec rec = rec_of(c, s0);
    float *slot0 = c.f(c.L.store);
    auto slot_p = [&](int level) {   // store slot of a level >= nlast
        float *b = slot0 + (size_t)(level - nlast) * nb * p->ST;
        return std::make_pair(Fld{b, p->ST}, Fld{b + g.N, p->ST});
    };
    // levels kept as full states (checkpoints, and the level the stored
    // history starts from)
    auto full_state = [&](int level) { return keep && level % k == 0 && level <= nlast; };
    // target of level n+1 for a step from a state whose velocities are in
    // work buffer cw
    auto target = [&](int n, int cw_in, int &cw_out) {
        const int nw = cw_in == 0 ? 1 : 0;
        State out = w[nw];
        cw_out = nw;
        if (keep && n >= nlast) {
            auto sl = slot_p(n + 1);
            out.p = sl.first;
            out.pz = sl.second;
        } else if (full_state(n + 1)) {
            out = state_at(c.f(c.L.ckpt) + (size_t)((n + 1) / k - 1) * nb * p->SS, p);
            cw_out = -1;
        }
        return out;
    };
    // samples of levels in the store are taken in one launch at the end
    auto sample = [&](const State &st, int n) {
        if (!traces || (keep && n >= nlast))
            return;
        Timed tm(c.pl, c.st, FWI_KC_SAMPLE);
        launch_sample(g, st.p, st.pz, rec, real_shots(p, s0, nb), traces, nt, n, c.st);
    };
    for (int n = 0; n < nt;) {
        if (keep && n == nlast) {
            auto sl = slot_p(nlast);
            copy_p(c, sl.first, sl.second, cur.p, cur.pz, nb);
        }
        if (p->two_step && n + 1 < nt && !full_state(n + 1)) {
            // two steps: level n+1 only as pressure (history slot or scratch)
            std::pair<Fld, Fld> mid;
            // level n+1 outside the stored history is only sampled: where
            // the node tables exist, just its receiver nodes are kept (or
            // nothing, without traces)
            int midw = 0;
            if (keep && n + 1 > nlast) {
                mid = slot_p(n + 1);
            } else {
                mid = {Fld{c.f(c.L.mid), p->ST}, Fld{c.f(c.L.mid) + g.N, p->ST}};
                if (p->samp_nodes)
                    midw = traces ? 1 : 2;
            }
            int cw2;
            State out = target(n + 1, cw, cw2);
            if (cw2 == cw)   // velocities of n+2 must not overwrite those of n
                cw2 = -1;
            step_fwd2(c, s0, nb, cur, mid.first, out, n, midw);
            if (midw == 1) {
                Timed tm(c.pl, c.st, FWI_KC_SAMPLE);
                launch_sample_nodes(c.f(c.L.nodes), c.tb.rec_node + (size_t)s0 * p->nrec,
                                    rec.w, p->nrec, real_shots(p, s0, nb), traces, nt, n, c.st);
            } else {
                State ms = cur;
                ms.p = mid.first;
                ms.pz = mid.second;
                sample(ms, n);
            }
            sample(out, n + 1);
            cur = out;
            cw = cw2;
            n += 2;
        } else {
            int cw1;
            State out = target(n, cw, cw1);
            step_fwd(c, s0, nb, cur, out, n);
            sample(out, n);
            cur = out;
            cw = cw1;
            n += 1;
        }
    }
    if (traces && keep) {
        Timed tm(c.pl, c.st, FWI_KC_SAMPLE);
        launch_sample_hist(g, slot_p(nlast + 1).first.p, (long long)nb * p->ST, p->ST, rec,
                           real_shots(p, s0, nb), traces, nt, nlast, nt - nlast, c.st);
    }
}

// Backward sweep for shots [s0, s0+nb) after sweep_forward(keep = true).
void sweep_backward(const Ctx &c, int s0, int nb, const float *resid, float *gpart)
{
    const fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    const int nt = p->grid.nt, k = p->k;
    float *store = c.f(c.L.store);
    auto slot = [&](int m) {
        float *b = store + (size_t)m * nb * p->ST;
        return std::make_pair(Fld{b, p->ST}, Fld{b + g.N, p->ST});
    };
    State lam[2] = {state_at(c.f(c.L.lam[0]), p), state_at(c.f(c.L.lam[1]), p)};
    zero_state(c, c.f(c.L.lam[0]), nb);
    int li = 0;
    // batched: next adjoint step; R^T r^n of levels n = top .. staged lie in
    // injv, an even number of them at a time
    const int stage = stage_steps(p);
    int m = nt, top = -1, staged = nt;
    float *injv = c.f(c.L.injacc);
    const Inj inj = inj_of(c, 0, p->S);
    const int *list = p->adj_list ? c.tb.al_node : nullptr;
    const int nlist = list ? p->adj_list : inj.nnodes;
    for (int sg = p->nseg - 1; sg >= 0; --sg) {
        int n0 = sg * k, n1 = std::min(n0 + k, nt);
        if (sg != p->nseg - 1) {
            // recompute the segment from its checkpoint, keeping the pressure
            State w[2] = {state_at(c.f(c.L.work[0]), p), state_at(c.f(c.L.work[1]), p)};
            State cur;
            int cw;
            if (n0 == 0) {
                zero_state(c, c.f(c.L.work[0]), nb);
                cur = w[0];
                cw = 0;
            } else {
                cur = state_at(c.f(c.L.ckpt) + (size_t)(n0 / k - 1) * nb * p->SS, p);
                cw = -1;
            }
            auto s0p = slot(0);
            copy_p(c, s0p.first, s0p.second, cur.p, cur.pz, nb);
            for (int n = n0; n < n1;) {
                int nw = cw == 0 ? 1 : 0;
                State out = w[nw];
                if (p->two_step && n + 1 < n1) {
                    auto sm = slot(n + 1 - n0), sl = slot(n + 2 - n0);
                    out.p = sl.first;
                    out.pz = sl.second;
                    step_fwd2(c, s0, nb, cur, sm.first, out, n);
                    n += 2;
                } else {
                    auto sl = slot(n + 1 - n0);
                    out.p = sl.first;
                    out.pz = sl.second;
                    step_fwd(c, s0, nb, cur, out, n);
                    n += 1;
                }
                cur = out;
                cw = nw;
            }
        }
        if (p->mode == FWI_EXEC_PLAIN) {
            for (int n = n1 - 1; n >= n0; --n) {
                auto a = slot(n - n0), b = slot(n + 1 - n0);
                step_adj_plain(c, s0, lam[li], lam[li ^ 1], a.first, a.second, b.first, b.second,
                               resid, gpart, n);
                li ^= 1;
            }
            continue;
        }
        // adjoint steps m down to n0+1, where the two-step kernel is on in
        // pairs: a pair may reach into the next segment by one step, whose
        // level n0 is slot 0 (step 0, of level 0, adds nothing)
        while (m > n0) {
            if (m - 1 < staged) {
                staged = m - std::min(stage, m);
                top = m - 1;
                Timed tm(c.pl, c.st, FWI_KC_INJECT);
                launch_inject_stage(inj, list, nlist, resid, p->nrec, nt, top, top - staged + 1,
                                    injv, c.st);
            }
            const float *va = injv + (size_t)(top - (m - 1)) * nlist;
            if (p->adj2) {
                step_adj2(c, lam[li], lam[li ^ 1], slot(m - 1 - n0).first, va,
                          m > 1 ? va + nlist : nullptr, gpart);
                m -= 2;
            } else {
                step_adj(c, lam[li], lam[li ^ 1], slot(m - n0).first, va, gpart);
                m -= 1;
            }
            li ^= 1;
        }
    }
}

// ------------------------------------------------------------ tile sweeps

Recd tile_rec(const fwi_plan *p, float *base)
{
    return Recd{base, (unsigned)(p->SS * sizeof(float)),
                (unsigned)((3 * p->geo.N + p->geo.Npml) * sizeof(float))};
}

// Forward steps n0 .. n1-1 of every shot from the state record batch `cur`;
// p^{n0+1} .. p^{n1} go to hist (unless null).  The last state is written to
// `last`, or to a work buffer if that is null; returns where it is.
float *tile_steps_fwd(const Ctx &c, const fwi_plan::TileRun &run, float *cur, int n0, int n1,
                      float *hist, long long lvl, long long ss, float *last)
{
    const fwi_plan *p = c.pl;
    float *w0 = c.f(c.L.work[0]), *w1 = c.f(c.L.work[1]);
    for (int n = n0; n < n1;) {
        const int t = std::min(run.T, n1 - n);
        float *out = n + t == n1 && last ? last : (cur == w0 ? w1 : w0);
        FwdTile a;
        a.in = tile_rec(p, cur);
        a.out = tile_rec(p, out);
        a.hist = hist ? hist + (size_t)(n - n0) * lvl : nullptr;
        a.lvl = lvl;
        a.ss = ss;
        a.Q = c.f(c.L.Q);
        a.src_ij = (const int *)c.tb.src_ij;
        a.src_w = (const float *)c.tb.src_w;
        a.n = n;
        a.nt = p->grid.nt;
        a.T = t;
        a.S = p->S;
        a.x = run.x;
        a.z = run.z;
        Timed tm(c.pl, c.st, FWI_KC_FWD_STEP, true);
        launch_tile_fwd(p->geo, c.tb.pml, c.tb.zpad, c.m.K, a, c.st, tm.b, tm.e);
        cur = out;
        n += t;
    }
    return cur;
}

// sweep_forward with the tile kernels: every level is written (to the store,
// segment after segment, or to the sampling buffer) and sampled in runs.
void tile_forward(const Ctx &c, bool keep, float *traces)
{
    const fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    const int nt = p->grid.nt, B = batch_of(p);
    float *cur = c.f(c.L.work[0]);
    zero_state(c, cur, B);
    const int run = keep ? p->k : p->tile.levels;
    const long long ss = keep ? p->ST : align64(g.N);
    const long long lvl = keep ? (long long)B * p->ST : (long long)p->S * ss;
    float *hist = keep ? c.f(c.L.store) + lvl : c.f(c.L.hist);
    for (int n0 = 0; n0 < nt; n0 += run) {
        const int n1 = std::min(n0 + run, nt);
        float *ck = keep && n1 < nt ? c.f(c.L.ckpt) + (size_t)(n0 / run) * B * p->SS : nullptr;
        cur = tile_steps_fwd(c, keep ? p->tile.keep : p->tile.call, cur, n0, n1,
                             traces || n1 == nt ? hist : nullptr, lvl, ss, ck);
        if (traces) {
            Timed tm(c.pl, c.st, FWI_KC_SAMPLE);
            launch_sample_hist(g, hist, lvl, ss, rec_of(c, 0), p->S, traces, nt, n0, n1 - n0,
                               c.st);
        }
    }
}

// sweep_backward with the tile kernels, after tile_forward(keep = true).
void tile_backward(const Ctx &c, const float *resid, float *gpart)
{
    const fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    const int nt = p->grid.nt, k = p->k, B = batch_of(p);
    const long long lvl = (long long)B * p->ST;
    float *store = c.f(c.L.store), *injv = c.f(c.L.injacc);
    float *lam[2] = {c.f(c.L.lam[0]), c.f(c.L.lam[1])};
    const Inj inj = inj_of(c, 0, p->S);
    zero_state(c, lam[0], B);
    int li = 0;
    for (int sg = p->nseg - 1; sg >= 0; --sg) {
        const int n0 = sg * k, n1 = std::min(n0 + k, nt);
        if (sg != p->nseg - 1) {
            // recompute the segment from its checkpoint, keeping the pressure
            float *cur = c.f(c.L.work[0]);
            if (n0 == 0)
                zero_state(c, cur, B);
            else
                cur = c.f(c.L.ckpt) + (size_t)(sg - 1) * B * p->SS;
            tile_steps_fwd(c, p->tile.keep, cur, n0, n1, store + lvl, lvl, p->ST, nullptr);
        }
        // adjoint steps m = n1 .. n0+1; step m takes p^m and adds R^T r^{m-1}
        for (int m = n1; m > n0;) {
            const int cnt = std::min(stage_steps(p), m - n0);
            {
                Timed tm(c.pl, c.st, FWI_KC_INJECT);
                launch_inject_stage(inj, nullptr, inj.nnodes, resid, p->nrec, nt, m - 1, cnt, injv,
                                    c.st);
            }
            for (int j = 0; j < cnt;) {
                const int t = std::min(p->tile.adj.T, cnt - j);
                AdjTile a;
                a.in = tile_rec(p, lam[li]);
                a.out = tile_rec(p, lam[li ^ 1]);
                a.hist = store + (size_t)(m - j - n0) * lvl;
                a.lvl = lvl;
                a.ss = p->ST;
                a.injv = injv + (size_t)j * inj.nnodes;
                a.rowptr = c.tb.inj_rowptr;
                a.injrc = c.tb.inj_rc;
                a.nnodes = inj.nnodes;
                a.gpart = gpart;
                a.T = t;
                a.S = p->S;
                a.x = p->tile.adj.x;
                a.z = p->tile.adj.z;
                Timed tm(c.pl, c.st, FWI_KC_ADJ_STEP, true);
                launch_tile_adj(g, c.tb.pml, c.tb.zpad, c.m.K, a, c.st, tm.b, tm.e);
                li ^= 1;
                j += t;
            }
            m -= cnt;
        }
    }
}

fwi_status check_call(const fwi_plan *p, void *ws, size_t ws_bytes, int op)
{
    if (!p)
        return fail(FWI_EINVAL, "plan is NULL");
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != p->device)
        return fail(FWI_ESTATE, "current device %d differs from the plan's device %d", dev,
                    p->device);
    size_t need = layout(p, op).total;
    if (need > 0) {
        if (!ws)
            return fail(FWI_EWORKSPACE, "workspace is NULL (needs %zu bytes)", need);
        if ((uintptr_t)ws % kAlign)
            return fail(FWI_EWORKSPACE, "workspace not %zu-byte aligned", kAlign);
        if (ws_bytes < need)
            return fail(FWI_EWORKSPACE, "workspace of %zu bytes, needs %zu", ws_bytes, need);
    }
    return FWI_OK;
}

fwi_status launched(const char *what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return fail(FWI_EDEVICE, "%s: %s", what, hipGetErrorString(e));
    return FWI_OK;
}

bool valid_param(int p) { return p >= FWI_K_RHO && p <= FWI_INVK_INVRHO; }

Ctx make_ctx(fwi_plan *p, void *ws, void *stream, int op)
{
    Ctx c;
    c.pl = p;
    c.st = (hipStream_t)stream;
    c.ws = (char *)ws;
    c.L = layout(p, op);
    if (op != FWI_OP_MISFIT) {
        char *b = c.ws + c.L.tab;
        const fwi_plan::TabOff &o = p->to;
        c.tb.pml = (float *)(b + o.pml);
        c.tb.zpad = (float *)(b + o.zpad);
        c.tb.sweep_tabs = (SweepTables *)(b + o.st);
        c.tb.src_ij = (int2 *)(b + o.sij);
        c.tb.src_w = (float4 *)(b + o.sw);
        c.tb.rec_idx = (long long *)(b + o.ri);
        c.tb.rec_w = (float4 *)(b + o.rw);
        c.tb.inj_node = (long long *)(b + o.in);
        c.tb.inj_shot = (int *)(b + o.is);
        c.tb.inj_cptr = (int *)(b + o.ip);
        c.tb.inj_crec = (int *)(b + o.ir);
        c.tb.inj_cw = (float *)(b + o.iw);
        c.tb.inj_win = (unsigned *)(b + o.win);
        c.tb.al_node = (int *)(b + o.aln);
        c.tb.al_col = (int *)(b + o.alc);
        c.tb.al_ptr = (int *)(b + o.alp);
        c.tb.sl_col = (int *)(b + o.slc);
        c.tb.sl_ptr = (int *)(b + o.slp);
        c.tb.samp_win = (unsigned *)(b + o.swin);
        c.tb.rec_node = (int4 *)(b + o.rnode);
        c.tb.inj_rowptr = (int *)(b + o.rptr);
        c.tb.inj_rc = (unsigned *)(b + o.irc);
        c.t = pml_tables(p, c.tb.pml);
    }
    c.m.K = c.f(c.L.Kpad);
    c.m.bx = c.f(c.L.bx);
    c.m.bz = c.f(c.L.bz);
    return c;
}

__global__ void k_sweep_tables(SweepTables *T, const int2 *ij, const float4 *w, int nt)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        T->src_ij = ij;
        T->src_w = w;
        T->nt = nt;
    }
}

// Puts the plan's tables into the call's workspace: the geometry tables
// copied from the plan's host image (immutable while the plan lives, so the
// copy may complete after this returns), the damping tables and the
// source-table record of the batched kernels built on the device.
void upload_tables(const Ctx &c)
{
    fwi_plan *p = c.pl;
    const fwi_grid &G = p->grid;
    Timed tm(c.pl, c.st, FWI_KC_OTHER);
    (void)hipMemcpyAsync(c.ws + c.L.tab + p->to.blob, p->blob.data(), p->blob.size(),
                         hipMemcpyHostToDevice, c.st);
    // the plan keeps blob until this copy has run (fwi_plan_destroy)
    if (!p->blob_ev)
        (void)hipEventCreateWithFlags(&p->blob_ev, hipEventDisableTiming);
    if (p->blob_ev)
        (void)hipEventRecord(p->blob_ev, c.st);
    launch_pml_tables(p->geo, G.vmax, G.npml > 0 ? G.pml_r : 0.5, G.dx, G.dz, G.dt, c.tb.pml,
                      c.st);
    launch_ztab_pad(p->geo, c.tb.pml, c.tb.zpad, c.st);
    hipLaunchKernelGGL(k_sweep_tables, dim3(1), dim3(64), 0, c.st, c.tb.sweep_tabs,
                       (const int2 *)c.tb.src_ij, (const float4 *)c.tb.src_w, G.nt);
}

void prepare(const Ctx &c, int param, const float *m1, const float *m2, const float *wavelet)
{
    const fwi_plan *p = c.pl;
    upload_tables(c);
    Timed tm(c.pl, c.st, FWI_KC_OTHER);
    launch_prep_model(p->geo, param, m1, m2, c.f(c.L.Kphys), c.f(c.L.rhophys), c.f(c.L.Kpad),
                      c.f(c.L.bx), c.f(c.L.bz), c.st);
    launch_cumulative_wavelet(wavelet, p->per_shot, p->S, p->grid.nt, (float)p->grid.dt,
                              c.f(c.L.Q), c.st);
}

// Backward half of the gradient: zero the partial sensitivities, sweep
// backward from the kept forward state (batched) or per shot (plain, which
// redoes each shot's forward sweep first), finalize.
fwi_status run_backward(const Ctx &c, int param, const float *m1, const float *m2,
                        const float *res, float *g1, float *g2)
{
    fwi_plan *p = c.pl;
    const Geo &g = p->geo;
    float *gpart = c.f(c.L.gpart);
    int G = partials_of(p);
    {
        Timed tm(p, c.st, FWI_KC_OTHER);
        launch_fill(gpart, (long long)G * 3 * g.N, 0.0f, c.st);
    }
    if (p->mode == FWI_EXEC_PLAIN) {
        for (int s = 0; s < p->S; ++s) {
            sweep_forward(c, s, 1, true, nullptr);
            sweep_backward(c, s, 1, res, gpart);
        }
    } else if (p->tile.on) {
        tile_backward(c, res, gpart);
    } else {
        sweep_backward(c, 0, p->Spad, res, gpart);
    }
    {
        Timed tm(p, c.st, FWI_KC_OTHER);
        launch_finalize(g, param, m1, m2, c.m.bx, c.m.bz, gpart, G, c.f(c.L.fold), g1, g2, c.st);
    }
    return launched("gradient");
}

// Misfit gradient (observed given, J written) or adjoint for a given
// adjoint source (adj_src given).
fwi_status run_gradient(fwi_plan *p, int param, const float *m1, const float *m2,
                        const float *wavelet, const float *observed, const float *adj_src,
                        float *J, float *g1, float *g2, float *traces, void *ws, void *stream)
{
    if (p->kept_ws == ws)
        p->kept_ws = nullptr;
    Ctx c = make_ctx(p, ws, stream, FWI_OP_GRADIENT);
    prepare(c, param, m1, m2, wavelet);
    float *tr = traces ? traces : c.f(c.L.traces);
    long long per_shot = (long long)p->nrec * p->grid.nt;
    long long ntr = per_shot * p->S;
    float *resid = c.f(c.L.resid);
    float *partials = c.f(c.L.partials);
    if (p->mode == FWI_EXEC_PLAIN) {
        // shot after shot: forward keeping its history, its residual, its
        // backward sweep; J over all shots at the end
        const Geo &g = p->geo;
        float *gpart = c.f(c.L.gpart);
        {
            Timed tm(p, c.st, FWI_KC_OTHER);
            launch_fill(gpart, 3 * g.N, 0.0f, c.st);
        }
        for (int s = 0; s < p->S; ++s) {
            const float *res = adj_src;
            sweep_forward(c, s, 1, true, observed ? tr + s * per_shot : nullptr);
            if (observed) {
                Timed tm(p, c.st, FWI_KC_OTHER);
                launch_misfit(tr + s * per_shot, observed + s * per_shot, resid + s * per_shot,
                              per_shot, partials, misfit_blocks(per_shot), J, c.st);
                res = resid;
            }
            sweep_backward(c, s, 1, res, gpart);
        }
        if (observed) {
            Timed tm(p, c.st, FWI_KC_OTHER);
            launch_misfit(tr, observed, nullptr, ntr, partials, misfit_blocks(ntr), J, c.st);
        }
        {
            Timed tm(p, c.st, FWI_KC_OTHER);
            launch_finalize(g, param, m1, m2, c.m.bx, c.m.bz, gpart, 1, c.f(c.L.fold), g1, g2,
                            c.st);
        }
        return launched("gradient");
    }
    if (p->tile.on)
        tile_forward(c, true, observed ? tr : nullptr);
    else
        sweep_forward(c, 0, p->Spad, true, observed ? tr : nullptr);
    const float *res = adj_src;
    if (observed) {
        Timed tm(p, c.st, FWI_KC_OTHER);
        launch_misfit(tr, observed, resid, ntr, partials, misfit_blocks(ntr), J, c.st);
        res = resid;
    }
    return run_backward(c, param, m1, m2, res, g1, g2);
}

}  // namespace

namespace {

// Whether the whole pressure history of `shots` shots of a sweep is kept by
// default: plain (one shot) up to 64 GiB, batched up to half the device memory.
bool history_fits(const fwi_plan *p, int shots)
{
    const double bytes = (double)(p->grid.nt + 1) * shots * p->ST * sizeof(float);
    double budget = 64.0 * (1ull << 30);
    if (p->mode != FWI_EXEC_PLAIN) {
        size_t free_b = 0, total_b = 0;
        budget = hipMemGetInfo(&free_b, &total_b) == hipSuccess ? 0.5 * (double)total_b : 0.0;
        (void)hipGetLastError();
    }
    return bytes <= budget;
}

// n tiles of `span` nodes over an axis of `len`, overlapping enough that each
// owned node lies `halo` or more from the inner edges of its tile; n = 0 if
// the span is too short.
TileAxis tile_axis(int len, int span, int halo)
{
    if (len <= span)
        return {1, len, 0, halo};
    const int last = len - span, most = span - 2 * halo;
    if (most < 1)
        return {0, len, 0, halo};
    for (int n = 2;; ++n) {
        int gap = 0, prev = 0;
        for (int k = 1; k < n; ++k) {
            const int f = k * last / (n - 1);
            gap = std::max(gap, f - prev);
            prev = f;
        }
        if (gap <= most)
            return {n, len, last, halo};
    }
}

// Tile kernels or strip kernels, and the steps per tile launch.
//
// A tile launch of T steps costs, with one 64 x 64 tile a workgroup on 256
// compute units (MI355X, us; sides of 101 to 541 padded nodes, 1 to 32 shots,
// T 2 to 8, within about 10%):
//   forward  3 + rounds of two workgroups a unit (11 + 1.9 T), a half round
//            (6.3 + 1.15 T)
//   adjoint  2.5 + rounds of one workgroup a unit (7.5 + 1.95 T)
// plus about 3.2 between launches: the load and the store of the tile, then
// the arithmetic of its T steps.  More steps spread the first over more time
// but shrink the owned part of a tile (64 - 6 T nodes a side), so T grows until
// the tiles no longer fit one round.  The strip kernels take 24.5 us a step for
// both sweeps of a gradient while the launch is what bounds them and about 14.5
// + 9.8 per million nodes (all shots) beyond, a forward sweep by itself 13.5 and
// 9.2 + 3.3.  So the tiles win up to about two million nodes, and for a forward
// sweep up to three and a half (us a step, tiles and strips; gradient: 3 shots
// of 156 x 327 7.4 and 23.1; 12 of 281 x 281 19.4 and 26.5; 12 of 253 x 419 22.0
// and 30.1; 7 of 537 x 599, 2.3 million, 40.1 and 35.0; 13 of 413 x 531, 2.9
// million, 46.5 and 42.8; forward: 8.0 and 14.2 for the second, 14.9 and 15.8 for
// the fourth, 17.2 and 17.5 for the fifth).
//
// Launches end at checkpoints and after the last step, so the run between them
// counts (and about 8 us for its sampling and staging launches, with checkpoints);
// the strip kernels' pairs cross checkpoints in the adjoint.  Checkpoints on every
// step, a tile launch and its overlap for one step: 8 shots of 241 x 241, 120 steps,
// 7.8 ms, strips 4.9; 10 of 381 x 381 13.6 and 7.3, every second step 7.6 and 6.4,
// every third 5.6 and 6.3.
//
// A plan that sets any part of the decomposition keeps the strip kernels.
fwi_plan::Tiles choose_tiles(const fwi_plan *p, const fwi_exec &ex)
{
    fwi_plan::Tiles t;
    const Geo &g = p->geo;
    if (ex.mode != FWI_EXEC_BATCHED || ex.band_rows || ex.shots_per_group || ex.lane_cols ||
        ex.two_step || ex.two_step_band_rows || ex.two_step_shots_per_group ||
        ex.two_step_lane_cols || ex.adj_two_step || ex.adj_two_step_band_rows ||
        ex.adj_two_step_lane_cols || g.Nz > 32767 || g.Nx > 32767)
        return t;
    const double nodes = (double)g.N * p->S;
    if (nodes > 4e6)
        return t;
    // us a step of a sweep in runs of `len` steps, by launches of at most T
    auto cost = [&](const fwi_plan::TileRun &r, bool adj, int len) {
        const long long h = ((long long)r.x.n * r.z.n * p->S + 255) / 256;
        auto launch = [&](int n) {
            return adj ? 5.7 + (double)h * (7.5 + 1.95 * n)
                       : 6.2 + (double)(h / 2) * (11 + 1.9 * n) + (double)(h % 2) * (6.3 + 1.15 * n);
        };
        const int full = len / r.T, rest = len % r.T;
        return (full * launch(r.T) + (rest ? launch(rest) : 0.0)) / len;
    };
    auto choose = [&](bool adj, int len, fwi_plan::TileRun &best) {
        double least = 1e30;
        for (int T = 1; T <= std::min(8, len); ++T) {
            const fwi_plan::TileRun r = {T, tile_axis(g.Nx, kTileX, 3 * T),
                                         tile_axis(g.Nz, kTileZ, 3 * T)};
            if (!r.x.n || !r.z.n)
                continue;
            const double us = cost(r, adj, len);
            if (us < least) {
                least = us;
                best = r;
            }
        }
        return least;
    };
    const double strips_f = std::max(13.5, 9.2 + 3.3e-6 * nodes);
    const double strips = std::max(24.5, 14.5 + 9.8e-6 * nodes) + (p->nseg > 1 ? strips_f : 0.0);
    const double f = choose(false, p->k, t.keep), a = choose(true, std::min(p->k, kStageSteps), t.adj);
    t.on = (p->nseg > 1 ? 2.0 * f + a + 8.0 / p->k : f + a) < strips;
    t.fwd = choose(false, p->grid.nt, t.call) < strips_f || t.on;
    // levels that a forward call buffers for sampling: about 64 MB, whole
    // launches
    const double level = (double)p->S * (double)align64(g.N) * sizeof(float);
    const int lv = (int)std::min(64.0, std::max(8.0, 64e6 / level));
    t.levels = std::max(1, lv / std::max(t.call.T, 1) * t.call.T);
    return t;
}

}  // namespace

// ------------------------------------------------------- static misfit scratch
//
// The partial sums of fwi_misfit_noalloc live in this file-scope device
// array: one copy per GPU, created with the code object and held until the
// process ends.  On the host, `scratch` names a stand-in, not device memory,
// so host code never hands it to a kernel: the first call on a device looks
// up that device's address once (with the device current) and every call
// passes the address it found.

constexpr int kScratchFloats = 2048;   // misfit partial sums (8 KiB)
static __device__ __align__(256) float scratch[kScratchFloats];

namespace {

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;

// Host tables of destroyed plans whose last copy into a workspace was still
// queued, with the event that marks its completion.
struct Retired {
    std::vector<char> blob;
    hipEvent_t ev;
};
std::mutex g_retired_mu;
std::vector<Retired> g_retired;

void sweep_retired()
{
    std::lock_guard<std::mutex> lock(g_retired_mu);
    for (size_t k = 0; k < g_retired.size();) {
        if (hipEventQuery(g_retired[k].ev) == hipErrorNotReady) {
            ++k;
            continue;
        }
        (void)hipEventDestroy(g_retired[k].ev);
        g_retired[k] = std::move(g_retired.back());
        g_retired.pop_back();
    }
    (void)hipGetLastError();
}
float *g_scratch_ptr[kMaxDevices];

// Address of `scratch` on the current device.
fwi_status scratch_on_current_device(float **out)
{
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices)
        return fail(FWI_EDEVICE, "no usable current HIP device (%d)", dev);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void *ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return fail(FWI_EDEVICE, "address of the static scratch on device %d: %s", dev,
                        hipGetErrorString(e));
        }
        g_scratch_ptr[dev] = (float *)ptr;
    }
    *out = g_scratch_ptr[dev];
    return FWI_OK;
}

}  // namespace

// ------------------------------------------------------------------ C ABI

extern "C" {

const char *fwi_status_str(fwi_status s)
{
    switch (s) {
    case FWI_OK: return "ok";
    case FWI_EINVAL: return "invalid argument";
    case FWI_ENOMEM: return "out of memory";
    case FWI_EDEVICE: return "device error";
    case FWI_EUNSTABLE: return "time step above the stability limit";
    case FWI_ENONFINITE: return "non-finite value";
    case FWI_ESTATE: return "bad state";
    case FWI_EWORKSPACE: return "bad workspace";
    }
    return "unknown status";
}

const char *fwi_last_error(void) { return g_err.c_str(); }

fwi_status fwi_plan_create(const fwi_grid *grid, const fwi_acq *acq, const fwi_exec *exec,
                           fwi_plan **out)
{
    if (!grid || !acq || !out)
        return fail(FWI_EINVAL, "NULL argument");
    *out = nullptr;
    const fwi_grid &G = *grid;
    if (G.nz < 5 || G.nx < 5 || G.npml < 0 || G.nt < 1)
        return fail(FWI_EINVAL, "grid sizes nz=%d nx=%d npml=%d nt=%d out of range", G.nz, G.nx,
                    G.npml, G.nt);
    if (!(G.dx > 0) || !(G.dz > 0) || !(G.dt > 0) || !(G.vmax > 0) || !std::isfinite(G.dx) ||
        !std::isfinite(G.dz) || !std::isfinite(G.dt) || !std::isfinite(G.vmax))
        return fail(FWI_EINVAL, "dx, dz, dt and vmax must be positive and finite");
    if (G.npml > 0 && !(G.pml_r > 0 && G.pml_r < 1))
        return fail(FWI_EINVAL, "pml_r must lie in (0, 1)");
    long long Nz = G.nz + 2LL * G.npml, Nx = G.nx + 2LL * G.npml;
    if (Nz * Nx > (1LL << 31) - 1)
        return fail(FWI_EINVAL, "padded grid too large");
    double sn = stability_number(G);
    if (sn > 1.0)
        return fail(FWI_EUNSTABLE, "vmax dt sqrt(1/dx^2+1/dz^2)(9/8+1/24) = %.4f > 1", sn);
    if (acq->nshots < 1 || acq->nrec < 1 || !acq->src_xz || !acq->rec_xz)
        return fail(FWI_EINVAL, "need at least one shot and one receiver with positions");
    fwi_exec ex{FWI_EXEC_BATCHED, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
    if (exec)
        ex = *exec;
    if (ex.mode != FWI_EXEC_BATCHED && ex.mode != FWI_EXEC_PLAIN)
        return fail(FWI_EINVAL, "unknown exec mode %d", ex.mode);
    if (ex.band_rows != 0 && (ex.band_rows < 4 || ex.band_rows > 4096))
        return fail(FWI_EINVAL, "band_rows %d out of range (4..4096)", ex.band_rows);
    if (ex.shots_per_group < 0 || ex.lane_cols < 0 ||
        (ex.shots_per_group != 0 && ex.lane_cols != 0 &&
         !fused_supported(ex.shots_per_group, ex.lane_cols)) ||
        (ex.shots_per_group != 0 && ex.lane_cols == 0 &&
         !fused_supported(ex.shots_per_group, 1)) ||
        (ex.lane_cols != 0 && ex.shots_per_group == 0 && !fused_supported(1, ex.lane_cols)))
        return fail(FWI_EINVAL, "shots_per_group %d with lane_cols %d not supported",
                    ex.shots_per_group, ex.lane_cols);
    if (ex.ckpt_every < 0)
        return fail(FWI_EINVAL, "ckpt_every out of range");
    if (ex.two_step < 0 || ex.two_step > 2)
        return fail(FWI_EINVAL, "two_step %d out of range (0, 1, 2)", ex.two_step);
    if (ex.two_step_band_rows != 0 && (ex.two_step_band_rows < 4 || ex.two_step_band_rows > 4096))
        return fail(FWI_EINVAL, "two_step_band_rows %d out of range (4..4096)",
                    ex.two_step_band_rows);
    {
        const int s2 = ex.two_step_shots_per_group, c2 = ex.two_step_lane_cols;
        if (s2 < 0 || c2 < 0 || !fused2_supported(s2 ? s2 : 1, c2 ? c2 : 1))
            return fail(FWI_EINVAL, "two-step kernel: shots_per_group %d with lane_cols %d not "
                        "supported", s2, c2);
    }
    if (ex.adj_two_step < 0 || ex.adj_two_step > 2)
        return fail(FWI_EINVAL, "adj_two_step %d out of range (0, 1, 2)", ex.adj_two_step);
    if (ex.adj_two_step_band_rows != 0 &&
        (ex.adj_two_step_band_rows < 4 || ex.adj_two_step_band_rows > 4096))
        return fail(FWI_EINVAL, "adj_two_step_band_rows %d out of range (4..4096)",
                    ex.adj_two_step_band_rows);
    if (ex.adj_two_step_lane_cols < 0 || ex.adj_two_step_lane_cols > 2)
        return fail(FWI_EINVAL, "adj_two_step_lane_cols %d not supported (1, 2)",
                    ex.adj_two_step_lane_cols);

    sweep_retired();
    fwi_plan *p = new fwi_plan();
    p->grid = G;
    p->S = acq->nshots;
    p->nrec = acq->nrec;
    p->per_shot = acq->wavelet_per_shot ? 1 : 0;
    p->mode = ex.mode;
    Geo &g = p->geo;
    g.Nz = (int)Nz;
    g.Nx = (int)Nx;
    g.npml = G.npml;
    g.nz = G.nz;
    g.nx = G.nx;
    g.rdx = (float)(1.0 / G.dx);
    g.rdz = (float)(1.0 / G.dz);
    g.dt = (float)G.dt;
    g.N = Nz * Nx;
    g.Npml = 2LL * G.npml * Nx + (Nz - 2LL * G.npml) * 2 * G.npml;
    // record strides 4 KB longer than the records, so that consecutive
    // shots' fields do not fall on the same offsets modulo large powers of
    // two (measured on MI355X: no change in the sweeps' time either way)
    p->SS = align64(3 * g.N + g.Npml) + 1024;
    p->ST = align64(g.N + g.Npml) + 1024;
    {
        // Defaults, from the autotuner's measurements on MI355X over padded
        // grids of 281 to 2081 nodes a side with 8 to 64 shots.
        //
        // Band heights of the two-step forward kernel: a launch of W equal
        // waves, R of which the device holds at once, runs about ceil(W / R)
        // rounds, each as long as one band (H rows plus the 6 rows of the
        // two-step halo).  Among the heights the autotuner tries, the smallest
        // ceil(W / R) (H + 6) wins, ties going to the taller band; the choices
        // come within 10% of the measured best.
        auto resident = [](int sg, int cl) {
            const int r = resident_waves2(sg, cl);
            return r > 0 ? r : 2048;   // two waves per SIMD of 256 compute units
        };
        auto pick_rows = [&](int Sp, int sg, int cl, int R, const int *cand, int nc) {
            int best = 0;
            long long best_cost = 0;
            for (int i = 0; i < nc; ++i) {
                const int H = balanced_rows(Nz, (int)std::min<long long>(cand[i], Nz));
                const long long W = sweep_of(g, Sp, H, sg, cl, 2).nwaves;
                const long long cost = (W + R - 1) / R * (H + 6);
                if (best == 0 || cost < best_cost || (cost == best_cost && H > best)) {
                    best = H;
                    best_cost = cost;
                }
            }
            return best;
        };
        // Shots per wave and band height of the two-step adjoint: a row of a
        // workgroup takes kRowUs[n - 1] us where a compute unit runs n
        // workgroups at once (measured on a whole MI355X, 256 compute units, at one
        // column per lane; wider lanes are taken in proportion); with more workgroups than run
        // at once their rounds overlap, and each full round takes kRoundUs.  A
        // band takes kStart rows more (its halo and the start of its windows),
        // and taller bands lose some of the cache lines that the groups of a
        // band share.  With more shots a wave moves fewer bytes (the model and
        // the partial gradient once for all) but fewer waves run.  Over thirty
        // sizes of 121 x 585 to 2081 x 2081 padded nodes with 3 to 64 shots,
        // against the best of all heights and groups measured, the choice takes
        // 1.002 times as long on average and 1.03 at most (with the rounds one
        // after the other 1.04 and 1.21): 64 shots of 1081 x 1081 (4 shots a
        // wave, 91 rows) 897 us, 2 shots 1005; 32 of 2081 x 2081 (4, 64) 1585,
        // best 1553, 2 shots 1748; 40 of 481 x 481 (2, 20) 167, 1 shot 172, 4
        // shots 185; 13 of 413 x 531 (1, 20) 57, 2 shots 67.  (Taken before the
        // receiver nodes of a row were added at once: 1 to 6 % less since on these.)
        // Shots that only fill up a group cost the forward sweeps too.
        auto adj_cost = [&](int sg, int cl, int H) {
            static const double kRowUs[3][4] = {
                {1.14, 1.49, 1.94, 2.36}, {2.1, 2.4, 3.08, 0}, {3.14, 3.76, 0, 0}};
            static const double kRoundUs[3] = {2.68, 3.18, 3.8}, kStart[3] = {10.4, 9.5, 9.9};
            const int i = sg == 1 ? 0 : sg == 2 ? 1 : 2, most = sg == 1 ? 4 : sg == 2 ? 3 : 2;
            const long long b =
                std::max(1LL, (sweep_of(g, p->S, H, sg, cl, 2).nwaves + 1023LL) / 1024);
            const double us = b <= most ? kRowUs[i][b - 1] : kRoundUs[i] * (double)b / most;
            const double pad = (double)((p->S + sg - 1) / sg * sg) / p->S;
            return us * cl * (H + kStart[i]) * (1.0 + H / 590.0) * (1.0 + 0.87 * (pad - 1.0));
        };
        static const int kRowsAdj2[] = {12, 16, 20, 24, 32, 48, 64, 96, 128, 160, 192};
        auto adj_rows = [&](int sg, int cl, double &cost) {
            int best = 0;
            for (int cand : kRowsAdj2) {
                const int H = ex.adj_two_step_band_rows
                                  ? ex.adj_two_step_band_rows
                                  : balanced_rows(Nz, (int)std::min<long long>(cand, Nz));
                const double c = adj_cost(sg, cl, H);
                if (best == 0 || c < cost) {
                    best = H;
                    cost = c;
                }
            }
            return best;
        };
        static const int kRowsFwd2[] = {12, 14, 16, 18, 20, 22, 24, 26, 28, 30, 32, 34, 36,
                                        40, 44, 48, 52, 56, 60, 64, 68, 72, 76, 80, 88, 96};
        // the batched kernels address a shot group's records, the model and
        // a partial gradient with 32-bit byte offsets below 2^31
        const long long lim = (1LL << 31) - 64LL * Nx;
        // the two-step adjoint addresses a group's pressure levels (consecutive
        // store levels, the padded shots' ST floats apart) through one buffer
        // resource.  It reads two; the bound is that of three, so that the
        // plans accepted with adj_two_step = 2 stay the same.
        auto adj2_fits = [&](int sg) {
            const long long Sp = (p->S + sg - 1) / sg * sg;
            return (2LL * Sp + sg) * p->ST * 4 < lim;
        };
        const bool adj2_wanted =
            p->mode != FWI_EXEC_PLAIN && ex.adj_two_step != 1 && adj2_fits(2);
        const int ca = ex.adj_two_step_lane_cols ? ex.adj_two_step_lane_cols : 1;
        // Shot groups of the one-step kernels: with the two-step adjoint (they
        // then only run what a forward segment leaves over) two shots a wave,
        // or one when even 16-row bands of two-shot waves number fewer than
        // two per SIMD of 256 compute units; without it up to four.  One column
        // per lane.
        int spg = ex.shots_per_group, cols = ex.lane_cols;
        if (spg == 0) {
            if (adj2_wanted) {
                spg = p->S >= 2 && sweep_of(g, p->S, 16, 2, ca, 2).nwaves >= 2048 ? 2 : 1;
            } else {
                spg = p->S >= 4 ? 4 : (p->S >= 2 ? 2 : 1);
            }
            if (cols != 0 && !fused_supported(spg, cols))
                spg = 1;
        }
        if (cols == 0)
            cols = 1;
        int H = ex.band_rows;
        if (H == 0) {
            Sweep one = sweep_of(g, p->S, (int)Nz, spg, cols);
            long long per_band = (long long)one.nstrips * one.ngroups;
            long long bands = std::max<long long>(1, (4096 + per_band - 1) / per_band);
            H = balanced_rows(Nz, (int)std::min<long long>(64, std::max<long long>(
                                      8, (Nz + bands - 1) / bands)));
        }
        // shot groups of the two-step adjoint: those of the one-step kernels
        // where the caller set them, else by its cost, leaving out groups whose
        // padding shots would cost the plan its whole pressure history
        const auto padded = [&](int sg) { return (p->S + sg - 1) / sg * sg; };
        const bool kept = ex.ckpt_every == 0 && history_fits(p, padded(spg));
        int spg_a = spg;
        if (ex.shots_per_group == 0 && adj2_wanted && adj2_supported(spg, ca)) {
            double best = 0.0;
            for (int sg = 1; sg <= 4; sg *= 2) {
                double c = 0.0;
                if (sg > p->S || !adj2_supported(sg, ca) || !adj2_fits(sg) ||
                    (long long)sg * p->SS * 4 >= lim ||
                    (kept && !history_fits(p, padded(std::max(spg, sg)))))
                    continue;
                (void)adj_rows(sg, ca, c);
                if (best == 0.0 || c < best) {
                    spg_a = sg;
                    best = c;
                }
            }
        }
        const int fill = std::max(spg, spg_a);   // (powers of two)
        p->Spad = p->mode == FWI_EXEC_PLAIN ? p->S : padded(fill);
        p->sweep = sweep_of(g, p->Spad, H, spg, cols);
        // two-step forward kernel over the same padded shots: two columns
        // per lane; two shots a wave from 800 padded columns up, else one
        // (and one if the padded count is odd)
        const int cols2 = ex.two_step_lane_cols ? ex.two_step_lane_cols : 2;
        int spg2 = ex.two_step_shots_per_group;
        if (spg2 == 0) {
            spg2 = Nx >= 800 && p->Spad % 2 == 0 ? 2 : 1;
            if (!fused2_supported(spg2, cols2))
                spg2 = 1;
        }
        int H2 = ex.two_step_band_rows;
        if (H2 == 0)
            H2 = pick_rows(p->Spad, spg2, cols2, resident(spg2, cols2), kRowsFwd2,
                           (int)(sizeof kRowsFwd2 / sizeof kRowsFwd2[0]));
        p->sweep2 = sweep_of(g, p->Spad, H2, spg2, cols2, 2);
        p->two_step = p->mode != FWI_EXEC_PLAIN && ex.two_step != 1 && p->Spad % spg2 == 0 &&
                      (long long)spg2 * p->SS * 4 < lim;
        const bool a2ok = p->mode != FWI_EXEC_PLAIN && adj2_supported(spg, ca);
        if (ex.adj_two_step == 2 && !a2ok) {
            delete p;
            return fail(FWI_EINVAL, "two-step adjoint: shots_per_group %d with lane_cols %d not "
                        "supported (or plain mode)", spg, ca);
        }
        const bool a2fits = adj2_fits(spg);
        if (ex.adj_two_step == 2 && a2ok && !a2fits) {
            delete p;
            return fail(FWI_EINVAL, "two-step adjoint: three pressure levels of %d shots exceed "
                        "2 GiB", p->Spad);
        }
        // (a call of one step has no pair to make: a gradient of 10 shots of 381 x 381
        // takes 140 us with the one-step launch, 151 with a pair)
        p->adj2 = ex.adj_two_step != 1 && a2ok && a2fits && (G.nt > 1 || ex.adj_two_step == 2);
        int Ha = ex.adj_two_step_band_rows;
        if (Ha == 0) {
            double c = 0.0;
            Ha = adj_rows(spg_a, ca, c);
        }
        p->sweep_a2 = sweep_of(g, p->Spad, Ha, spg_a, ca, 2);
        if (p->mode != FWI_EXEC_PLAIN &&
            ((long long)spg * p->SS * 4 >= lim || 3 * g.N * 4 >= lim)) {
            delete p;
            return fail(FWI_EINVAL, "grid of %lld cells too large for %d shots per group "
                        "(records of a group must stay below 2 GiB)", (long long)g.N, spg);
        }
    }
    {
        // checkpoint interval: with ckpt_every = 0 the whole pressure history
        // is kept when it fits, so the backward sweep needs no recompute; else
        // every ceil(sqrt(nt)) steps
        int k = ex.ckpt_every > 0 ? ex.ckpt_every : (int)std::ceil(std::sqrt((double)G.nt));
        if (ex.ckpt_every == 0 && history_fits(p, batch_of(p)))
            k = G.nt;
        p->k = std::max(1, std::min(k, G.nt));
        p->nseg = (G.nt + p->k - 1) / p->k;
    }
    p->tile = choose_tiles(p, ex);

    // geometry: bilinear cell and weights of every source and receiver
    const int S = p->S, nr = p->nrec;
    std::vector<long long> rec_idx((size_t)S * nr);
    std::vector<float4> rec_w((size_t)S * nr);
    p->h_src_ij.resize(S);
    p->h_src_w.resize(S);
    auto locate = [&](double x, double z, int &i, int &j, double w[4]) -> bool {
        double fx = x / G.dx, fz = z / G.dz;
        if (!std::isfinite(fx) || !std::isfinite(fz))
            return false;
        double jf = std::floor(fx), iff = std::floor(fz);
        if (iff < 0 || jf < 0 || iff > G.nz - 2 || jf > G.nx - 2)
            return false;
        double tx = fx - jf, tz = fz - iff;
        i = (int)iff + G.npml;
        j = (int)jf + G.npml;
        w[0] = (1 - tx) * (1 - tz);
        w[1] = tx * (1 - tz);
        w[2] = (1 - tx) * tz;
        w[3] = tx * tz;
        return true;
    };
    const double h2 = G.dx * G.dz;
    for (int s = 0; s < S; ++s) {
        int i, j;
        double w[4];
        if (!locate(acq->src_xz[2 * s], acq->src_xz[2 * s + 1], i, j, w)) {
            delete p;
            return fail(FWI_EINVAL, "source %d at (%g, %g) m is not inside the physical grid", s,
                        acq->src_xz[2 * s], acq->src_xz[2 * s + 1]);
        }
        p->h_src_ij[s] = make_int2(i, j);
        p->h_src_w[s] = make_float4((float)(w[0] / h2), (float)(w[1] / h2), (float)(w[2] / h2),
                                    (float)(w[3] / h2));
        for (int r = 0; r < nr; ++r) {
            const double *xz = acq->rec_xz + 2 * ((size_t)s * nr + r);
            if (!locate(xz[0], xz[1], i, j, w)) {
                delete p;
                return fail(FWI_EINVAL, "receiver %d of shot %d at (%g, %g) m is not inside the "
                            "physical grid", r, s, xz[0], xz[1]);
            }
            rec_idx[(size_t)s * nr + r] = (long long)i * g.Nx + j;
            rec_w[(size_t)s * nr + r] = make_float4((float)w[0], (float)w[1], (float)w[2],
                                                    (float)w[3]);
        }
    }
    // adjoint injection: per shot, the nodes touched by receivers (ascending
    // node) with their (receiver, weight) contributions in receiver order
    std::vector<long long> inj_node;
    std::vector<int> inj_shot, inj_cptr, inj_crec;
    std::vector<float> inj_cw;
    p->shot_node_ptr.assign(S + 1, 0);
    struct Touch {   // (a receiver touches a node once)
        long long node;
        int rec;
        float w;
    };
    std::vector<Touch> touch;
    for (int s = 0; s < S; ++s) {
        touch.clear();
        for (int r = 0; r < nr; ++r) {
            long long c = rec_idx[(size_t)s * nr + r];
            float4 w = rec_w[(size_t)s * nr + r];
            long long cs[4] = {c, c + 1, c + g.Nx, c + g.Nx + 1};
            float ws[4] = {w.x, w.y, w.z, w.w};
            for (int q = 0; q < 4; ++q)
                if (ws[q] != 0.0f)
                    touch.push_back({cs[q], r, ws[q]});
        }
        std::sort(touch.begin(), touch.end(), [](const Touch &a, const Touch &b) {
            return a.node != b.node ? a.node < b.node : a.rec < b.rec;
        });
        for (const Touch &t : touch) {
            if ((int)inj_node.size() == p->shot_node_ptr[s] || inj_node.back() != t.node) {
                inj_node.push_back(t.node);
                inj_shot.push_back(s);
                inj_cptr.push_back((int)inj_crec.size());
            }
            inj_crec.push_back(t.rec);
            inj_cw.push_back(t.w);
        }
        p->shot_node_ptr[s + 1] = (int)inj_node.size();
    }
    inj_cptr.push_back((int)inj_crec.size());
    p->inj_nodes = (int)inj_node.size();
    // where each row's nodes begin (they lie in row order), and every node's
    // column
    std::vector<int> inj_rowptr((size_t)S * (g.Nz + 1)), inj_col(inj_node.size());
    for (size_t k = 0; k < inj_node.size(); ++k)
        inj_col[k] = (int)(inj_node[k] % g.Nx);
    for (int s = 0; s < S; ++s) {
        int k = p->shot_node_ptr[s];
        for (int i = 0; i <= g.Nz; ++i) {
            while (k < p->shot_node_ptr[s + 1] && inj_node[k] < (long long)i * g.Nx)
                ++k;
            inj_rowptr[(size_t)s * (g.Nz + 1) + i] = k;
        }
    }
    std::vector<unsigned> inj_rc;
    if (p->tile.on) {
        inj_rc.resize(inj_node.size());
        for (size_t k = 0; k < inj_node.size(); ++k)
            inj_rc[k] = ((unsigned)(inj_node[k] / g.Nx) << 16) | (unsigned)inj_col[k];
    }
    // Nodes listed by shot, strip and row, those of a strip being the ones
    // whose columns lie in [strip W - reach, strip W - reach + width): for
    // every row and strip the packed range (first << 9 | count; width <= 256)
    // counted from the strip's first node, rows offset by `pad` in a table of
    // `rows` rows a shot.  False if a strip holds more nodes than that packs.
    auto list_nodes = [&](int nstrips, int W, int reach, int width, int shots, int rows, int pad,
                          std::vector<unsigned> &win, std::vector<int> &ptr,
                          std::vector<int> &node, std::vector<int> &col) {
        win.assign((size_t)shots * rows * nstrips, 0u);
        ptr.assign((size_t)shots * nstrips, 0);
        std::vector<int> full;   // rows that hold nodes
        for (int s = 0; s < S; ++s) {
            const int *rp = &inj_rowptr[(size_t)s * (g.Nz + 1)];
            full.clear();
            for (int i = 0; i < g.Nz; ++i)
                if (rp[i] != rp[i + 1])
                    full.push_back(i);
            for (int st = 0; st < nstrips; ++st) {
                const int base = (int)node.size();
                ptr[(size_t)s * nstrips + st] = base;
                const int lo = st * W - reach;
                for (int i : full) {
                    const auto r0 = inj_col.begin() + rp[i], r1 = inj_col.begin() + rp[i + 1];
                    if (*(r1 - 1) < lo || *r0 >= lo + width)
                        continue;
                    const auto c0 = std::lower_bound(r0, r1, lo);
                    const auto c1 = std::lower_bound(c0, r1, lo + width);
                    if (c0 == c1)
                        continue;
                    const size_t first = node.size() - (size_t)base;
                    if (first >= (1u << 23) || node.size() > (1u << 30))
                        return false;
                    win[((size_t)s * rows + pad + i) * nstrips + st] =
                        ((unsigned)first << 9) | (unsigned)(c1 - c0);
                    for (auto c = c0; c != c1; ++c) {
                        node.push_back((int)(c - inj_col.begin()));
                        col.push_back(*c);
                    }
                }
            }
        }
        return true;
    };
    // strip adjoint: the strip's window (its output columns and halo)
    std::vector<unsigned> inj_win;
    std::vector<int> al_node, al_col, al_ptr;
    if (p->mode != FWI_EXEC_PLAIN && !p->tile.on) {
        const Sweep &sa = p->adj2 ? p->sweep_a2 : p->sweep;
        const int reach = p->adj2 ? 6 : 3;
        const int halo = (reach + sa.cols - 1) / sa.cols * sa.cols;
        if (list_nodes(sa.nstrips, strip_cols(sa.cols, p->adj2 ? 2 : 1), halo, 64 * sa.cols,
                       p->Spad, g.Nz + 2 * kZPad, kZPad, inj_win, al_ptr, al_node, al_col)) {
            p->adj_list = (int)al_node.size();
        } else {   // one-step adjoint, R^T r added by launches of its own
            p->adj2 = false;
            inj_win.clear();
            al_ptr.clear();
            al_node.clear();
            al_col.clear();
        }
        al_col.resize(al_col.size() + 64, -1);   // (runs of 64 are read)
    }
    // two-step forward, whose intermediate level, when only sampled, is kept at
    // the receiver nodes: the columns the strip owns; and for every receiver
    // the listed nodes of its four bilinear corners (-1 where the weight is
    // zero, which has no node)
    std::vector<unsigned> samp_win;
    std::vector<int> sl_node, sl_col, sl_ptr;
    std::vector<int4> rec_node;
    if (p->two_step && !p->tile.on) {
        const Sweep &s2 = p->sweep2;
        const int W = strip_cols(s2.cols, 2);
        p->samp_nodes =
            list_nodes(s2.nstrips, W, 0, W, S, g.Nz, 0, samp_win, sl_ptr, sl_node, sl_col);
        if (p->samp_nodes) {
            p->samp_list = (int)sl_node.size();   // every node once
            std::vector<int> at(inj_node.size());
            for (size_t l = 0; l < sl_node.size(); ++l)
                at[sl_node[l]] = (int)l;
            rec_node.resize((size_t)S * nr);
            for (int s = 0; s < S; ++s) {
                const auto b0 = inj_node.begin() + p->shot_node_ptr[s];
                const auto b1 = inj_node.begin() + p->shot_node_ptr[s + 1];
                for (int r = 0; r < nr; ++r) {
                    const long long c = rec_idx[(size_t)s * nr + r];
                    const float4 w = rec_w[(size_t)s * nr + r];
                    const long long cs[4] = {c, c + 1, c + g.Nx, c + g.Nx + 1};
                    const float ws[4] = {w.x, w.y, w.z, w.w};
                    int q4[4];
                    for (int q = 0; q < 4; ++q) {
                        q4[q] = -1;
                        if (ws[q] != 0.0f)
                            q4[q] = at[std::lower_bound(b0, b1, cs[q]) - inj_node.begin()];
                    }
                    rec_node[(size_t)s * nr + r] = make_int4(q4[0], q4[1], q4[2], q4[3]);
                }
            }
        } else {
            samp_win.clear();
            sl_ptr.clear();
            sl_col.clear();
        }
        sl_col.resize(sl_col.size() + 64, -1);
    }
    if (!p->tile.on)
        inj_rowptr.clear();

    if (hipGetDevice(&p->device) != hipSuccess) {
        delete p;
        return fail(FWI_EDEVICE, "no HIP device");
    }
    // the tables' layout in a workspace's table region: the damping tables
    // and the batched kernels' source-table record are built there by each
    // call, the rest is copied from the host image `blob`
    size_t off = 0;
    auto take = [&](size_t bytes) {
        size_t o = off;
        off = align_up(off + std::max<size_t>(bytes, 1), kAlign);
        return o;
    };
    fwi_plan::TabOff &o = p->to;
    o.pml = take(sizeof(float) * (4 * g.Nx + 4 * g.Nz));
    o.zpad = take(sizeof(float) * 4 * (g.Nz + 2 * kZPad));
    o.st = take(sizeof(SweepTables));
    o.blob = off;
    o.sij = take(sizeof(int2) * S);
    o.sw = take(sizeof(float4) * S);
    o.ri = take(sizeof(long long) * rec_idx.size());
    o.rw = take(sizeof(float4) * rec_w.size());
    o.in = take(sizeof(long long) * inj_node.size());
    o.is = take(sizeof(int) * inj_shot.size());
    o.ip = take(sizeof(int) * inj_cptr.size());
    o.ir = take(sizeof(int) * inj_crec.size());
    o.iw = take(sizeof(float) * inj_cw.size());
    o.win = take(sizeof(unsigned) * inj_win.size());
    o.aln = take(sizeof(int) * al_node.size());
    o.alc = take(sizeof(int) * al_col.size());
    o.alp = take(sizeof(int) * al_ptr.size());
    o.slc = take(sizeof(int) * sl_col.size());
    o.slp = take(sizeof(int) * sl_ptr.size());
    o.swin = take(sizeof(unsigned) * samp_win.size());
    o.rnode = take(sizeof(int4) * rec_node.size());
    o.rptr = take(sizeof(int) * inj_rowptr.size());
    o.irc = take(sizeof(unsigned) * inj_rc.size());
    o.bytes = off;
    try {
        p->blob.assign(off - o.blob, 0);
    } catch (const std::bad_alloc &) {
        delete p;
        return fail(FWI_ENOMEM, "host allocation of %zu bytes for plan tables failed",
                    off - o.blob);
    }
    auto put = [&](size_t at, const void *src, size_t bytes) {
        if (bytes)
            std::memcpy(p->blob.data() + (at - o.blob), src, bytes);
    };
    put(o.sij, p->h_src_ij.data(), sizeof(int2) * S);
    put(o.sw, p->h_src_w.data(), sizeof(float4) * S);
    put(o.ri, rec_idx.data(), sizeof(long long) * rec_idx.size());
    put(o.rw, rec_w.data(), sizeof(float4) * rec_w.size());
    put(o.in, inj_node.data(), sizeof(long long) * inj_node.size());
    put(o.is, inj_shot.data(), sizeof(int) * inj_shot.size());
    put(o.ip, inj_cptr.data(), sizeof(int) * inj_cptr.size());
    put(o.ir, inj_crec.data(), sizeof(int) * inj_crec.size());
    put(o.iw, inj_cw.data(), sizeof(float) * inj_cw.size());
    put(o.win, inj_win.data(), sizeof(unsigned) * inj_win.size());
    put(o.aln, al_node.data(), sizeof(int) * al_node.size());
    put(o.alc, al_col.data(), sizeof(int) * al_col.size());
    put(o.alp, al_ptr.data(), sizeof(int) * al_ptr.size());
    put(o.slc, sl_col.data(), sizeof(int) * sl_col.size());
    put(o.slp, sl_ptr.data(), sizeof(int) * sl_ptr.size());
    put(o.swin, samp_win.data(), sizeof(unsigned) * samp_win.size());
    put(o.rnode, rec_node.data(), sizeof(int4) * rec_node.size());
    put(o.rptr, inj_rowptr.data(), sizeof(int) * inj_rowptr.size());
    put(o.irc, inj_rc.data(), sizeof(unsigned) * inj_rc.size());
    *out = p;
    return FWI_OK;
}

void fwi_plan_destroy(fwi_plan *p)
{
    if (!p)
        return;
    (void)collect_marks(p);
    for (hipEvent_t e : p->spare)
        (void)hipEventDestroy(e);
    sweep_retired();
    if (p->blob_ev && hipEventQuery(p->blob_ev) == hipErrorNotReady) {
        // a copy of the tables may still be queued: keep them until it ran
        std::lock_guard<std::mutex> lock(g_retired_mu);
        g_retired.push_back({std::move(p->blob), p->blob_ev});
    } else if (p->blob_ev) {
        (void)hipEventDestroy(p->blob_ev);
    }
    (void)hipGetLastError();
    delete p;
}

fwi_status fwi_plan_get_info(const fwi_plan *p, fwi_plan_info *info)
{
    if (!p || !info)
        return fail(FWI_EINVAL, "NULL argument");
    info->Nz = p->geo.Nz;
    info->Nx = p->geo.Nx;
    info->ckpt_every = p->k;
    info->segments = p->nseg;
    info->band_rows = p->sweep.H;
    info->shots_per_group = p->mode == FWI_EXEC_PLAIN ? 1 : p->sweep.spg;
    info->lane_cols = p->mode == FWI_EXEC_PLAIN ? 1 : p->sweep.cols;
    info->two_step = p->two_step ? 1 : 0;
    info->two_step_band_rows = p->sweep2.H;
    info->two_step_shots_per_group = p->sweep2.spg;
    info->two_step_lane_cols = p->sweep2.cols;
    info->adj_two_step = p->adj2 ? 1 : 0;
    info->adj_two_step_band_rows = p->sweep_a2.H;
    info->adj_two_step_lane_cols = p->sweep_a2.cols;
    info->shot_groups = p->mode == FWI_EXEC_PLAIN ? 1 : (p->S + p->sweep.spg - 1) / p->sweep.spg;
    info->mode = p->mode;
    info->device = p->device;
    info->pml_cells = p->geo.Npml;
    info->cfl = p->grid.vmax * p->grid.dt / std::min(p->grid.dx, p->grid.dz);
    return FWI_OK;
}

size_t fwi_workspace_bytes(const fwi_plan *p, int32_t op)
{
    if (!p || op < FWI_OP_FORWARD || op > FWI_OP_GRADIENT)
        return 0;
    return layout(p, op).total;
}

fwi_status fwi_forward(fwi_plan *p, int32_t param, const float *m1, const float *m2,
                       const float *wavelet, float *traces, void *ws, size_t ws_bytes,
                       void *stream)
{
    fwi_status st = check_call(p, ws, ws_bytes, FWI_OP_FORWARD);
    if (st != FWI_OK)
        return st;
    if (!valid_param(param) || !m1 || !m2 || !wavelet || !traces)
        return fail(FWI_EINVAL, "bad parameterization or NULL array");
    if (p->kept_ws == ws)
        p->kept_ws = nullptr;
    Ctx c = make_ctx(p, ws, stream, FWI_OP_FORWARD);
    prepare(c, param, m1, m2, wavelet);
    long long per_shot = (long long)p->nrec * p->grid.nt;
    if (p->mode == FWI_EXEC_PLAIN) {
        for (int s = 0; s < p->S; ++s)
            sweep_forward(c, s, 1, false, traces + s * per_shot);
    } else if (p->tile.fwd) {
        tile_forward(c, false, traces);
    } else {
        sweep_forward(c, 0, p->Spad, false, traces);
    }
    return launched("forward");
}

fwi_status fwi_misfit(fwi_plan *p, const float *traces, const float *observed, float *residual,
                      float *J, void *ws, size_t ws_bytes, void *stream)
{
    fwi_status st = check_call(p, ws, ws_bytes, FWI_OP_MISFIT);
    if (st != FWI_OK)
        return st;
    if (!traces || !observed || !J)
        return fail(FWI_EINVAL, "NULL array");
    long long n = (long long)p->S * p->nrec * p->grid.nt;
    Layout L = layout(p, FWI_OP_MISFIT);
    {
        Timed tm(p, (hipStream_t)stream, FWI_KC_OTHER);
        launch_misfit(traces, observed, residual, n, (float *)((char *)ws + L.partials),
                      misfit_blocks(n), J, (hipStream_t)stream);
    }
    return launched("misfit");
}

fwi_status fwi_misfit_noalloc(fwi_plan *p, const float *traces, const float *observed,
                              float *residual, float *J, void *stream)
{
    if (!p)
        return fail(FWI_EINVAL, "plan is NULL");
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev != p->device)
        return fail(FWI_ESTATE, "current device %d differs from the plan's device %d", dev,
                    p->device);
    if (!traces || !observed || !J)
        return fail(FWI_EINVAL, "NULL array");
    long long n = (long long)p->S * p->nrec * p->grid.nt;
    const int nb = misfit_blocks(n);
    if (nb > kScratchFloats)
        return fail(FWI_EINVAL, "misfit of %lld samples needs %d partial sums; the static "
                    "scratch holds %d", n, nb, kScratchFloats);
    float *part = nullptr;
    fwi_status st = scratch_on_current_device(&part);
    if (st != FWI_OK)
        return st;
    // every partial sum is written by its block before the final sum reads
    // it, so nothing left from an earlier call needs clearing
    launch_misfit(traces, observed, residual, n, part, nb, J, (hipStream_t)stream);
    return launched("misfit_noalloc");
}

fwi_status fwi_misfit_weighted(fwi_plan *p, const float *traces, const float *observed,
                               const float *weights, float *residual, float *J, void *ws,
                               size_t ws_bytes, void *stream)
{
    fwi_status st = check_call(p, ws, ws_bytes, FWI_OP_MISFIT);
    if (st != FWI_OK)
        return st;
    if (!traces || !observed || !weights || !J)
        return fail(FWI_EINVAL, "NULL array");
    long long n = (long long)p->S * p->nrec * p->grid.nt;
    Layout L = layout(p, FWI_OP_MISFIT);
    {
        Timed tm(p, (hipStream_t)stream, FWI_KC_OTHER);
        launch_misfit(traces, observed, residual, n, (float *)((char *)ws + L.partials),
                      misfit_blocks(n), J, (hipStream_t)stream, weights, p->grid.nt);
    }
    return launched("misfit_weighted");
}

fwi_status fwi_gradient(fwi_plan *p, int32_t param, const float *m1, const float *m2,
                        const float *wavelet, const float *observed, float *J, float *g1,
                        float *g2, float *traces, void *ws, size_t ws_bytes, void *stream)
{
    fwi_status st = check_call(p, ws, ws_bytes, FWI_OP_GRADIENT);
    if (st != FWI_OK)
        return st;
    if (!valid_param(param) || !m1 || !m2 || !wavelet || !observed || !J || !g1 || !g2)
        return fail(FWI_EINVAL, "bad parameterization or NULL array");
    return run_gradient(p, param, m1, m2, wavelet, observed, nullptr, J, g1, g2, traces, ws,
                        stream);
}

fwi_status fwi_adjoint(fwi_plan *p, int32_t param, const float *m1, const float *m2,
                       const float *wavelet, const float *adj_src, float *g1, float *g2,
                       void *ws, size_t ws_bytes, void *stream)
{
    fwi_status st = check_call(p, ws, ws_bytes, FWI_OP_GRADIENT);
    if (st != FWI_OK)
        return st;
    if (!valid_param(param) || !m1 || !m2 || !wavelet || !adj_src || !g1 || !g2)
        return fail(FWI_EINVAL, "bad parameterization or NULL array");
    return run_gradient(p, param, m1, m2, wavelet, nullptr, adj_src, nullptr, g1, g2, nullptr,
                        ws, stream);
}

fwi_status fwi_forward_keep(fwi_plan *p, int32_t param, const float *m1, const float *m2,
                            const float *wavelet, float *traces, void *ws, size_t ws_bytes,
                            void *stream)
{
    fwi_status st = check_call(p, ws, ws_bytes, FWI_OP_GRADIENT);
    if (st != FWI_OK)
        return st;
    if (!valid_param(param) || !m1 || !m2 || !wavelet || !traces)
        return fail(FWI_EINVAL, "bad parameterization or NULL array");
    Ctx c = make_ctx(p, ws, stream, FWI_OP_GRADIENT);
    prepare(c, param, m1, m2, wavelet);
    long long per_shot = (long long)p->nrec * p->grid.nt;
    if (p->mode == FWI_EXEC_PLAIN) {
        for (int s = 0; s < p->S; ++s)
            sweep_forward(c, s, 1, false, traces + s * per_shot);
    } else if (p->tile.on) {
        tile_forward(c, true, traces);
    } else {
        sweep_forward(c, 0, p->Spad, true, traces);
    }
    p->kept_ws = ws;
    return launched("forward_keep");
}

fwi_status fwi_adjoint_kept(fwi_plan *p, int32_t param, const float *m1, const float *m2,
                            const float *wavelet, const float *adj_src, float *g1, float *g2,
                            void *ws, size_t ws_bytes, void *stream)
{
    fwi_status st = check_call(p, ws, ws_bytes, FWI_OP_GRADIENT);
    if (st != FWI_OK)
        return st;
    if (!valid_param(param) || !m1 || !m2 || !wavelet || !adj_src || !g1 || !g2)
        return fail(FWI_EINVAL, "bad parameterization or NULL array");
    if (p->kept_ws != ws)
        return fail(FWI_ESTATE, "no forward state kept on this workspace");
    p->kept_ws = nullptr;
    Ctx c = make_ctx(p, ws, stream, FWI_OP_GRADIENT);
    return run_backward(c, param, m1, m2, adj_src, g1, g2);
}

fwi_status fwi_model_convert(int32_t from, int32_t to, int64_t n, const float *a1,
                             const float *a2, float *b1, float *b2, void *stream)
{
    if (!valid_param(from) || !valid_param(to) || n < 0 || (n > 0 && (!a1 || !a2 || !b1 || !b2)))
        return fail(FWI_EINVAL, "bad parameterization, size or NULL array");
    if (n == 0)
        return FWI_OK;
    launch_convert(from, to, n, a1, a2, b1, b2, (hipStream_t)stream);
    return launched("model_convert");
}

fwi_status fwi_chain_rule(int32_t param, int64_t n, const float *m1, const float *m2,
                          const float *gK, const float *grho, float *g1, float *g2, void *stream)
{
    if (!valid_param(param) || n < 0 ||
        (n > 0 && (!m1 || !m2 || !gK || !grho || !g1 || !g2)))
        return fail(FWI_EINVAL, "bad parameterization, size or NULL array");
    if (n == 0)
        return FWI_OK;
    launch_chain_rule(param, n, m1, m2, gK, grho, g1, g2, (hipStream_t)stream);
    return launched("chain_rule");
}

fwi_status fwi_contrast_scale(int64_t n, const float *m0, float *g, void *stream)
{
    if (n < 0 || (n > 0 && (!m0 || !g)))
        return fail(FWI_EINVAL, "bad size or NULL array");
    if (n == 0)
        return FWI_OK;
    launch_contrast_scale(n, m0, g, (hipStream_t)stream);
    return launched("contrast_scale");
}

fwi_status fwi_descent_direction(int64_t n, const float *m0, const float *g, const float *mask,
                                 float *d, void *stream)
{
    if (n < 0 || (n > 0 && (!m0 || !g || !d)))
        return fail(FWI_EINVAL, "bad size or NULL array");
    if (n == 0)
        return FWI_OK;
    launch_descent_dir(n, m0, g, mask, d, (hipStream_t)stream);
    return launched("descent_direction");
}

fwi_status fwi_descent_apply(int64_t n, const float *m, const float *m0, const float *d,
                             float alpha, float *out, void *stream)
{
    if (n < 0 || (n > 0 && (!m || !m0 || !d || !out)))
        return fail(FWI_EINVAL, "bad size or NULL array");
    if (!std::isfinite(alpha))
        return fail(FWI_ENONFINITE, "step length is not finite");
    if (n == 0)
        return FWI_OK;
    launch_descent_apply(n, m, m0, d, alpha, out, (hipStream_t)stream);
    return launched("descent_apply");
}

fwi_status fwi_descent_norms(int64_t n, const float *a, const float *b, float *out, void *stream)
{
    if (n < 0 || !out || (n > 0 && !a))
        return fail(FWI_EINVAL, "bad size or NULL array");
    launch_norms2(n, a, b, out, (hipStream_t)stream);
    return launched("descent_norms");
}

// ------------------------------------------------------------------ born
namespace {

bool born_sizes_ok(int F, int S, int R, int C)
{
    return F >= 0 && S >= 0 && R >= 0 && C >= 0 && F <= 65535 && S <= 65535 * 64 &&
           (long long)S * R < (1LL << 31);
}

bool born_media_ok(double K0, double rho0)
{
    return std::isfinite(K0) && std::isfinite(rho0) && K0 > 0.0 && rho0 > 0.0;
}

struct BornWs {
    size_t data, grad, misfit, total;
};

BornWs born_ws(int F, int S, int R, int C)
{
    BornSplit b = born_data_split(F, S, R, C);
    BornWs w;
    w.data = align_up((size_t)b.nsplit * F * S * R * 2 * sizeof(float), kAlign);
    w.grad = born_grad_wt_offset(b, C) + align_up(born_grad_wt_bytes(b, F, R), kAlign);
    w.misfit = align_up((size_t)misfit_blocks(2LL * F * S * R) * sizeof(float), kAlign);
    w.total = std::max(w.data, std::max(w.grad, w.misfit));
    return w;
}

fwi_status born_work_ok(void *work, size_t bytes, size_t need)
{
    if (need == 0)
        return FWI_OK;
    if (!work || ((uintptr_t)work % kAlign) != 0 || bytes < need)
        return fail(FWI_EWORKSPACE, "workspace needs %zu bytes, 256-byte aligned (got %zu)",
                    need, work ? bytes : (size_t)0);
    return FWI_OK;
}

}  // namespace

fwi_status fwi_born_green(int32_t F, const float *omega, int32_t C, const float *cells,
                          int32_t P, const float *pts, double K0, double rho0, float *G,
                          float *Gx, float *Gz, void *stream)
{
    if (F < 0 || C < 0 || P < 0)
        return fail(FWI_EINVAL, "negative size");
    if (!born_media_ok(K0, rho0))
        return fail(FWI_EINVAL, "K0 and rho0 must be positive and finite");
    if ((Gx == nullptr) != (Gz == nullptr))
        return fail(FWI_EINVAL, "Gx and Gz must both be given or both be NULL");
    const long long n = (long long)F * C * P;
    if (n == 0)
        return FWI_OK;
    if (!omega || !cells || !pts || !G)
        return fail(FWI_EINVAL, "NULL array");
    launch_born_green(F, C, P, omega, cells, pts, K0, rho0, G, Gx, Gz, (hipStream_t)stream);
    return launched("born_green");
}

size_t fwi_born_workspace_bytes(int32_t F, int32_t S, int32_t R, int32_t C)
{
    if (!born_sizes_ok(F, S, R, C))
        return 0;
    return born_ws(F, S, R, C).total;
}

fwi_status fwi_born_data(int32_t F, const float *omega, const float *spec, int32_t S,
                         int32_t R, int32_t C, double K0, double rho0, double dA,
                         const float *xiK, const float *xiR, const float *Gs, const float *Gsx,
                         const float *Gsz, const float *Gr, const float *Grx, const float *Grz,
                         const float *Gd, float *d, void *work, size_t work_bytes,
                         void *stream)
{
    if (!born_sizes_ok(F, S, R, C))
        return fail(FWI_EINVAL, "bad sizes (negative, F > 65535, S > 4194240 or S R >= 2^31)");
    if (!born_media_ok(K0, rho0) || !std::isfinite(dA) || dA <= 0.0)
        return fail(FWI_EINVAL, "K0, rho0 and dA must be positive and finite");
    if ((long long)F * S * R == 0)
        return FWI_OK;
    if (!omega || !spec || !d)
        return fail(FWI_EINVAL, "NULL array");
    if (C > 0 && (!xiK || !xiR || !Gs || !Gsx || !Gsz || !Gr || !Grx || !Grz))
        return fail(FWI_EINVAL, "NULL contrast or table");
    BornWs w = born_ws(F, S, R, C);
    fwi_status st = born_work_ok(work, work_bytes, w.data);
    if (st != FWI_OK)
        return st;
    launch_born_data(born_data_split(F, S, R, C), F, S, R, C, omega, spec, K0, rho0, dA, xiK,
                     xiR, Gs, Gsx, Gsz, Gr, Grx, Grz, Gd, d, (float *)work,
                     (hipStream_t)stream);
    return launched("born_data");
}

fwi_status fwi_born_misfit(int64_t n, const float *d, const float *q, float *resid, float *J,
                           void *work, size_t work_bytes, void *stream)
{
    if (n < 0 || !J || (n > 0 && (!d || !q)))
        return fail(FWI_EINVAL, "bad size or NULL array");
    if (n > (1LL << 40))
        return fail(FWI_EINVAL, "n too large");
    const size_t need = align_up((size_t)misfit_blocks(2 * n) * sizeof(float), kAlign);
    fwi_status st = born_work_ok(work, work_bytes, need);
    if (st != FWI_OK)
        return st;
    launch_misfit(d, q, resid, 2 * n, (float *)work, misfit_blocks(2 * n), J,
                  (hipStream_t)stream);
    return launched("born_misfit");
}

fwi_status fwi_born_gradient(int32_t F, const float *omega, const float *spec, int32_t S,
                             int32_t R, int32_t C, double K0, double rho0, double dA,
                             const float *resid, const float *Gs, const float *Gsx,
                             const float *Gsz, const float *Gr, const float *Grx,
                             const float *Grz, float *gK, float *gR, void *work,
                             size_t work_bytes, void *stream)
{
    if (!born_sizes_ok(F, S, R, C))
        return fail(FWI_EINVAL, "bad sizes (negative, F > 65535, S > 4194240 or S R >= 2^31)");
    if (!born_media_ok(K0, rho0) || !std::isfinite(dA) || dA <= 0.0)
        return fail(FWI_EINVAL, "K0, rho0 and dA must be positive and finite");
    if (C == 0)
        return FWI_OK;
    if (!gK || !gR)
        return fail(FWI_EINVAL, "NULL gradient array");
    const bool any = (long long)F * S * R > 0;
    if (any && (!omega || !spec || !resid || !Gs || !Gsx || !Gsz || !Gr || !Grx || !Grz))
        return fail(FWI_EINVAL, "NULL array");
    BornWs w = born_ws(F, S, R, C);
    fwi_status st = born_work_ok(work, work_bytes, any ? w.grad : 0);
    if (st != FWI_OK)
        return st;
    launch_born_gradient(born_data_split(F, S, R, C), F, S, R, C, omega, spec, K0, rho0, dA,
                         resid, Gs, Gsx, Gsz, Gr, Grx, Grz, gK, gR, (float *)work,
                         (hipStream_t)stream);
    return launched("born_gradient");
}

fwi_status fwi_born_contrasts(int32_t scheme, int32_t param, int64_t n, const float *xa,
                              const float *xb, float *xiK, float *xiR, void *stream)
{
    if ((scheme != 1 && scheme != 2) || !valid_param(param) || n < 0 ||
        (n > 0 && (!xa || !xb || !xiK || !xiR)))
        return fail(FWI_EINVAL, "bad scheme, parameterization, size or NULL array");
    launch_born_contrasts(scheme, param, n, xa, xb, xiK, xiR, (hipStream_t)stream);
    return launched("born_contrasts");
}

fwi_status fwi_born_chain(int32_t scheme, int32_t param, int64_t n, const float *xa,
                          const float *xb, const float *gK, const float *gR, float *ga,
                          float *gb, void *stream)
{
    if ((scheme != 1 && scheme != 2) || !valid_param(param) || n < 0 ||
        (n > 0 && (!gK || !gR || !ga || !gb || (scheme == 2 && (!xa || !xb)))))
        return fail(FWI_EINVAL, "bad scheme, parameterization, size or NULL array");
    launch_born_chain(scheme, param, n, xa, xb, gK, gR, ga, gb, (hipStream_t)stream);
    return launched("born_chain");
}

fwi_status fwi_born_hessian(int32_t F, const float *omega, const float *spec, int32_t S,
                            int32_t R, double K0, double rho0, const float *Gs,
                            const float *Gsx, const float *Gsz, const float *Gr,
                            const float *Grx, const float *Grz, int32_t param, float *H,
                            void *stream)
{
    if (!born_sizes_ok(F, S, R, 1) || !valid_param(param) || !H)
        return fail(FWI_EINVAL, "bad sizes, parameterization or NULL output");
    if (!born_media_ok(K0, rho0))
        return fail(FWI_EINVAL, "K0 and rho0 must be positive and finite");
    if ((long long)F * S * R > 0 &&
        (!omega || !spec || !Gs || !Gsx || !Gsz || !Gr || !Grx || !Grz))
        return fail(FWI_EINVAL, "NULL array");
    launch_born_hessian(F, S, R, omega, spec, K0, rho0, Gs, Gsx, Gsz, Gr, Grx, Grz, param, H,
                        (hipStream_t)stream);
    return launched("born_hessian");
}

fwi_status fwi_timing_enable(fwi_plan *p, int32_t enable)
{
    if (!p)
        return fail(FWI_EINVAL, "plan is NULL");
    if (collect_marks(p) != FWI_OK)
        return fail(FWI_EDEVICE, "waiting for timing events failed");
    p->timing = enable != 0;
    p->acc = fwi_timing{};
    return FWI_OK;
}

fwi_status fwi_timing_read(fwi_plan *p, fwi_timing *out, int32_t reset)
{
    if (!p || !out)
        return fail(FWI_EINVAL, "NULL argument");
    if (collect_marks(p) != FWI_OK)
        return fail(FWI_EDEVICE, "waiting for timing events failed");
    *out = p->acc;
    if (reset)
        p->acc = fwi_timing{};
    return FWI_OK;
}

fwi_status fwi_sync(void *stream)
{
    hipError_t e = hipStreamSynchronize((hipStream_t)stream);
    if (e == hipSuccess)
        e = hipGetLastError();
    if (e != hipSuccess)
        return fail(FWI_EDEVICE, "%s", hipGetErrorString(e));
    return FWI_OK;
}

}  // extern "C"
