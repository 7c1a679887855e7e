// Host runtime and C ABI of libflavorpic (see include/fpic.h).
//
// A context is a batch of one simulation: every 1D entry point runs the same
// segmented kernels over a table of (simulation, tile, direction group)
// work items.  The runtime carves the caller's workspace, uploads the small
// per-simulation tables, builds the work tables (cost-sorted for the step,
// contiguous per simulation for per-simulation calls), and captures one and
// K RK4 steps into hipGraphs on a private stream; fpic_step replays them on
// the caller's stream.  Kernels read the step number from device memory, so
// the captured graphs stay valid as time advances.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "fpic.h"
#include "fpic_internal.h"
#include "fpic_3d.h"
#include "fpic_diag.h"

using namespace fpic;

namespace {
thread_local std::string g_err;
}  // namespace

int fpic::fail(int code, const std::string &msg)
{
    g_err = msg;
    return code;
}

namespace {

#define HIPCHECK(x)                                                                     \
    do {                                                                                \
        hipError_t e_ = (x);                                                            \
        if (e_ != hipSuccess)                                                           \
            return fail(FPIC_EHIP, std::string(#x) + ": " + hipGetErrorString(e_));    \
    } while (0)

size_t align_up(size_t x) { return (x + 255) & ~size_t(255); }

struct Carver {
    size_t off = 0;
    size_t take(size_t bytes)
    {
        off = align_up(off);
        size_t o = off;
        off += bytes;
        return o;
    }
};

constexpr int kRedBlocks = 256;  // blocks of the diagnostic reductions
constexpr int kFailed = 63;      // word of the pinned buffer: a step launch failed
constexpr unsigned long long kArriveRule = ~0ull;
// Contexts whose waves have one direction each, in at most one workgroup per
// CU, run whole steps in one launch (fpic_1d_steps.h), if a tile has at most
// kMaxStepGroups direction groups: every workgroup sums all groups' partials
// of its tile in every stage.  us per step, one launch per stage and
// reduction (the faster slope form) against whole steps: 32 cells x 26
// directions 66 -> 38, 200 x 92 (12 groups) 81 -> 57, 777 x 92 quadratic (12)
// 108 -> 76, 512 x 128 (16) 79 -> 65, 2048 x 64 (8) 87 -> 67; but 256 x 378
// (48) 95 -> 103.
constexpr int64_t kMaxStepParticles = (int64_t)kMaxStepWgs * MAX_WAVES * TILE;
constexpr int kMaxStepGroups = 24;
constexpr int kStepsPerLaunch = 512;

// Sizes and offsets of one simulation inside the workspace.
struct SimPlan {
    int ncell = 0, ndir = 0, ntile = 0, ngroup = 0, dpw = 0;
    int64_t np = 0;
    size_t o_tab = 0, o_Y = 0, o_K1 = 0, o_K2 = 0, o_K3 = 0, o_G0 = 0, o_G1 = 0, o_G2 = 0, o_G3 = 0;
    size_t o_part = 0, o_edge = 0, o_part2 = 0, o_edge2 = 0, o_step = 0;
};

struct Plan {
    int nsim = 0, waves = 0, max_dpw = 0, spg = 0, shape = 1;
    bool nt = false;  // streaming cache policy in the stage kernels
    int rk = 2;       // slopes formed again: 2 k1 and k2, 1 k1, 0 none
    std::vector<SimPlan> sims;
    size_t o_desc = 0, o_work = 0, o_red = 0, o_scratch = 0, o_bar = 0, total = 0;
    int nwork = 0, nred = 0;
    bool steps = false;  // small enough for whole steps in one launch
};

int validate_1d(const fpic_config &c, int idx)
{
    char buf[256];
    auto bad = [&](const char *what) {
        std::snprintf(buf, sizeof buf, "config %d: %s", idx, what);
        return fail(FPIC_EINVAL, buf);
    };
    if (c.ncell[0] < 1 || c.ncell[1] < 1 || c.ncell[2] < 1)
        return bad("cell counts must be >= 1");
    if (c.ndir < 1)
        return bad("ndir must be >= 1");
    if (!c.dirs || !c.N || !c.Nbar)
        return bad("dirs, N and Nbar must be non-null host arrays");
    if (c.shape_order != 1 && c.shape_order != 2)
        return fail(FPIC_EUNSUPPORTED,
                    "shape_order must be 1 (linear, cloud in cell) or 2 (quadratic)");
    for (int a = 0; a < 3; ++a)
        if (!(c.dx[a] > 0.0) || !std::isfinite(c.dx[a]))
            return bad("cell widths must be positive and finite");
    if (!(c.dt > 0.0) || !std::isfinite(c.dt))
        return bad("dt must be positive and finite");
    if ((int64_t)c.ncell[0] * c.ncell[1] * c.ncell[2] > (int64_t)1 << 30)
        return bad("too many cells");
    double hmax = 0.0;
    for (int i = 0; i < 18; ++i) {
        if (!std::isfinite(c.hvac[i]))
            return bad("hvac has a non-finite entry");
        hmax = std::max(hmax, std::fabs(c.hvac[i]));
    }
    for (int a = 0; a < 3; ++a)
        if (!std::isfinite(c.vmat[a]))
            return bad("vmat has a non-finite entry");
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < 3; ++j) {
            const double re = c.hvac[2 * (3 * i + j)], im = c.hvac[2 * (3 * i + j) + 1];
            const double rt = c.hvac[2 * (3 * j + i)], it = c.hvac[2 * (3 * j + i) + 1];
            if (std::fabs(re - rt) + std::fabs(im + it) > 1e-12 * (1.0 + hmax))
                return bad("hvac is not Hermitian");
        }
    double vmax[3] = {0, 0, 0};
    for (int d = 0; d < c.ndir; ++d) {
        const double *v = c.dirs + 3 * d;
        const double n2 = v[0] * v[0] + v[1] * v[1] + v[2] * v[2];
        if (!std::isfinite(n2) || std::fabs(n2 - 1.0) > 1e-9)
            return bad("directions must be unit vectors");
        if (!std::isfinite(c.N[d]) || !std::isfinite(c.Nbar[d]))
            return bad("weights must be finite");
        for (int a = 0; a < 3; ++a)
            vmax[a] = std::max(vmax[a], std::fabs(v[a]));
    }
    for (int a = 0; a < 3; ++a)
        if (c.ncell[a] > 1 && 0.5 * c.dt * vmax[a] / c.dx[a] >= 1.0 - 1e-9)
            return fail(FPIC_EUNSUPPORTED,
                        "dt too large: a particle may cross a whole cell within one "
                        "Runge-Kutta stage (need dt/2 * max|Omega| < dx)");
    return FPIC_OK;
}

bool is_1d(const fpic_config &c) { return c.ncell[0] == 1 && c.ncell[1] == 1; }

// The launch shape where the caller leaves it open (waves or dpw zero).  A
// workgroup stages its grid tiles and sums its waves' deposits once, about as
// long as 1.5 directions take (2.5 in workgroups of up to 4 waves), and each of
// its waves sweeps dpw directions; the chip holds 8 waves per CU (the stage
// kernels use 211-254 registers), so a launch takes ceil(workgroups / slots)
// rounds of dpw and that.  The shape with the fewest is taken: up to one
// workgroup of 8 waves on each of the 256 CUs (of this chip; not asked of the
// device, since a plan and its workspace are the same on any), then longer
// waves.  Against 4 waves and about 1024 workgroups, us per step: 2048 x 378
// 285 -> 202, 1000 x 378 209 -> 137, 4096 x 128 239 -> 164, 512 x 128 90 -> 81,
// 777 x 92 quadratic 147 -> 116, 5000 x 378 565 -> 467, 24 boxes of 11.5 M
// particles 3958 -> 3094 (those measured fastest in a sweep of 1-8 waves and
// 1-24 directions).  Workgroups of 4 waves stage twice as many tiles per CU
// (219 us for the 2048 x 378 box) and pay where their smaller granularity saves
// a round.  A single box gets at most the workgroups (and partial sums) of the
// caller's waves, or 4, in about 1024 of them: fpic_step_noalloc's fixed
// scratch, which takes the same shape, holds every box up to the size its limit
// states.  With several directions a wave given, 4 waves are taken: 8 make
// fewer workgroups of longer waves (us per step, 4 against 8: 200 x 92 with 4
// directions 170, 230; 512 x 128 with 4 117, 139, with 12 236, 291; 2048 x 378
// with 12 268, 308, with 4 293, 284), and from 51 directions a wave on those of
// a quadratic box pass the LDS.
void choose_shape(int nsim, const fpic_config *cfgs, int &waves, int &dpw)
{
    constexpr int kCus = 256;
    const bool w_open = waves == 0, d_open = dpw == 0;
    int64_t most = INT64_MAX;
    if (dpw > 1) {
        waves = w_open ? 4 : waves;
        return;
    }
    double best = 1e300;
    int bw = w_open ? 4 : waves, bd = dpw;
    if (d_open) {
        const int64_t ntile = (cfgs[0].ncell[2] + TILE - 1) / TILE, nd = cfgs[0].ndir, target = 1024 * bw;
        bd = (int)std::max<int64_t>(1, std::min<int64_t>(64, (ntile * nd + target - 1) / target));
        if (nsim == 1)
            most = ntile * ((nd + (int64_t)bw * bd - 1) / ((int64_t)bw * bd));
    }
    for (int w : {8, 4}) {
        if (!w_open && w == 4)
            break;  // the caller's waves, once
        const int wv = w_open ? w : waves;
        for (int d : {1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 32}) {
            if (!d_open && d > 1)
                break;  // the caller's dpw, once
            const int dp = d_open ? d : dpw;
            int64_t wg = 0;
            for (int i = 0; i < nsim; ++i) {
                const int64_t dpg = (int64_t)wv * std::min(dp, cfgs[i].ndir);
                wg += (int64_t)((cfgs[i].ncell[2] + TILE - 1) / TILE) * ((cfgs[i].ndir + dpg - 1) / dpg);
            }
            const int64_t slots = (int64_t)kCus * 8 / wv;
            const double fixed = wv >= 8 ? 1.5 : 2.5;
            const double cost = (double)((wg + slots - 1) / slots) * (dp + fixed);
            if (wg <= most && cost < best) {
                best = cost;
                bw = wv;
                bd = dp;
            }
        }
    }
    waves = bw;
    dpw = bd;
}

// external_state: the state array is the caller's (no room for it in the
// workspace); used by the entry point that allocates nothing.
int make_plan(int nsim, const fpic_config *cfgs, const fpic_tuning *tune, Plan &P,
              bool external_state = false)
{
    if (nsim < 1 || !cfgs)
        return fail(FPIC_EINVAL, "need at least one configuration");
    for (int i = 0; i < nsim; ++i) {
        int rc = validate_1d(cfgs[i], i);
        if (rc)
            return rc;
        if (!is_1d(cfgs[i]))
            return fail(FPIC_EINVAL, "batches hold 1D boxes only (ncell = {1, 1, nz})");
        if (cfgs[i].shape_order != cfgs[0].shape_order)
            return fail(FPIC_EINVAL, "the boxes of a batch must share one shape_order");
    }
    P = Plan();
    P.nsim = nsim;
    P.shape = cfgs[0].shape_order;
    P.waves = tune ? tune->waves : 0;
    if (P.waves != 0 && P.waves != 1 && P.waves != 2 && P.waves != 4 && P.waves != 8)
        return fail(FPIC_EINVAL, "waves must be 1, 2, 4 or 8");
    P.spg = (tune && tune->steps_per_graph) ? tune->steps_per_graph : 8;
    if (P.spg < 1 || P.spg > 256)
        return fail(FPIC_EINVAL, "steps_per_graph must be in 1..256");
    const int policy = tune ? tune->cache_policy : 0;
    if (policy < 0 || policy > 2)
        return fail(FPIC_EINVAL, "cache_policy must be 0, 1 or 2");
    if (policy == 0) {
        // Streaming pays where one box's state nearly fills or just
        // overflows the 256 MB Infinity Cache.  Default against streaming,
        // us per step in the built-in launch shape: 111 MB (2048 x 378) 202
        // against 217, 163 MB (3000 x 378) equal, 218 MB (4000 x 378) 381
        // against 361, 272 MB (5000 x 378) 489 against 467, 381 MB (7000 x
        // 378) 700 against 705; batches, whose boxes are swept one after
        // another, gain nothing (24 boxes, 11.5 M particles: 3094 against
        // 3131).
        const int64_t state0 = (int64_t)cfgs[0].ncell[2] * cfgs[0].ndir * 18 * (int64_t)sizeof(double);
        P.nt = nsim == 1 && state0 >= (int64_t)176 << 20 && state0 <= (int64_t)320 << 20;
    } else {
        P.nt = policy == 2;
    }
    const int fused = tune ? tune->fused : 0;
    if (fused < 0 || fused > 2)
        return fail(FPIC_EINVAL, "fused must be 0, 1 or 2");
    int dpw = (tune && tune->dirs_per_wave) ? tune->dirs_per_wave : 0;
    if (dpw < 0 || dpw > 256)
        return fail(FPIC_EINVAL, "dirs_per_wave must be in 0..256");
    choose_shape(nsim, cfgs, P.waves, dpw);
    // Slopes formed again pay where a stage is bound by its memory traffic.
    // With one direction a wave it is bound by latency, and storing them is
    // faster (us per step: 256 x 378 94.6 against 97.9, 2048 x 64 87 against
    // 91, 32 x 26 66 against 76); the results are the same bits.
    P.rk = fused == 0 && dpw == 1 ? 0 : 2 - fused;
    P.sims.resize(nsim);
    int64_t nwork = 0, np_all = 0;
    int nc_min = INT32_MAX, ng_max = 0;
    for (int i = 0; i < nsim; ++i) {
        const int64_t dpg = (int64_t)P.waves * std::min(dpw, cfgs[i].ndir);
        const int ng = (int)((cfgs[i].ndir + dpg - 1) / dpg);
        nwork += (int64_t)((cfgs[i].ncell[2] + TILE - 1) / TILE) * ng;
        ng_max = std::max(ng_max, ng);
        np_all += (int64_t)cfgs[i].ncell[2] * cfgs[i].ndir;
        nc_min = std::min(nc_min, cfgs[i].ncell[2]);
    }
    // (room for every launch shape and slope form of a small box, so that one
    // tried in the workspace of another fits)
    const bool small = !external_state && np_all <= kMaxStepParticles && nc_min >= kMinStepCells;
    P.steps = small && fused == 0 && dpw == 1 && nwork <= kMaxStepWgs && ng_max <= kMaxStepGroups;
    Carver cv;
    for (int i = 0; i < nsim; ++i) {
        SimPlan &s = P.sims[i];
        s.ncell = cfgs[i].ncell[2];
        s.ndir = cfgs[i].ndir;
        s.np = (int64_t)s.ncell * s.ndir;
        s.ntile = (s.ncell + TILE - 1) / TILE;
        s.dpw = std::min(dpw, s.ndir);
        const int dpg = s.dpw * P.waves;
        s.ngroup = (s.ndir + dpg - 1) / dpg;
        P.max_dpw = std::max(P.max_dpw, s.dpw);
        const size_t st = sizeof(double) * 18 * (size_t)s.np;
        const size_t sk = sizeof(double) * NK * (size_t)s.np;
        s.o_tab = cv.take(sizeof(double) * 7 * s.ndir);
        s.o_Y = cv.take(external_state ? 0 : st);
        s.o_K1 = cv.take(sk);
        s.o_K2 = cv.take(sk);
        s.o_K3 = cv.take(sk);
        s.o_G0 = cv.take(sizeof(double) * NG * s.ncell);
        s.o_G1 = cv.take(sizeof(double) * NG * s.ncell);
        s.o_G2 = cv.take(sizeof(double) * NG * s.ncell);
        s.o_G3 = cv.take(sizeof(double) * NG * s.ncell);
        s.o_part = cv.take(sizeof(double) * (size_t)s.ngroup * NG * s.ntile * TILE);
        s.o_edge = cv.take(sizeof(double) * (size_t)s.ngroup * NG * n_edges(P.shape) * s.ntile);
        s.o_part2 = cv.take(small ? sizeof(double) * (size_t)s.ngroup * NG * s.ntile * TILE : 0);
        s.o_edge2 = cv.take(small ? sizeof(double) * (size_t)s.ngroup * NG * n_edges(P.shape) * s.ntile : 0);
        s.o_step = cv.take(sizeof(int64_t));
        P.nwork += s.ntile * s.ngroup;
        P.nred += s.ntile;
    }
    P.o_desc = cv.take(sizeof(SimDesc) * nsim);
    // global (cost-sorted) table followed by the per-simulation tables
    P.o_work = cv.take(sizeof(WorkItem) * 2 * (size_t)P.nwork);
    P.o_red = cv.take(sizeof(RedItem) * (size_t)P.nred);
    P.o_scratch = cv.take(sizeof(double) * (3 + 18 + 18 * kRedBlocks + 3 * kRedBlocks));
    P.o_bar = cv.take(small ? sizeof(unsigned) * kBarWords : 0);
    P.total = align_up(cv.off);
    return FPIC_OK;
}

}  // namespace

struct fpic_batch {
    Plan plan;
    hipStream_t stream = nullptr;  // caller's
    hipStream_t cap = nullptr;     // private capture stream
    char *ws = nullptr;
    SimDesc *ddesc = nullptr;
    WorkItem *dwork = nullptr;     // [nwork] sorted, then [nwork] per-sim
    RedItem *dred = nullptr;
    double *dscratch = nullptr;
    double *hbuf = nullptr;        // pinned host staging
    std::vector<SimDesc> hdesc;
    std::vector<int> swork_off, sred_off;
    std::vector<bool> state_set;
    hipGraphExec_t g1 = nullptr, gK = nullptr;
    bool steps = false;            // whole steps in one launch (fpic_1d_steps.h)
    unsigned launches = 0, gen = 0;  // such launches, and their grid barriers, so far
    hipEvent_t done = nullptr;     // after the latest such launch
    fpic_batch *steps_next = nullptr;  // (g_steps_head)
    bool launching = false;        // done not yet recorded for it
    int cus = 0, steps_held = 0;
    // how long its workgroups wait to be resident together before those that
    // are do the work, in ticks of 10 ns (kArriveRule: see run_steps)
    unsigned long long arrive_ticks = kArriveRule;
    unsigned bar_ticks = 2000000000u;  // and at a barrier before it gives up (20 s)
    int device = 0;
    double cell_volume = 1.0;      // of simulation 0
    // reverse mode (single 1D box)
    struct Adj {
        bool forward_done = false;
        int64_t n_start = 0, nsteps = 0;
        int L = 0, nseg = 0;
        char *ws = nullptr;
        size_t o_ckpt = 0, o_segY = 0, o_segK = 0, o_segG = 0, o_lam = 0, o_lcur = 0,
               o_dres = 0, o_GA = 0, o_dw = 0, o_descF = 0, o_descR = 0, o_out = 0, total = 0;
        std::vector<std::pair<int, hipGraphExec_t>> recompute, reverse;  // by length
    } adj;
};

struct fpic_ctx {
    fpic_batch *b = nullptr;       // 1D
    fpic3d::Ctx3D *c3 = nullptr;   // 3D
};

namespace {

int capture_steps(fpic_batch *b, int nsteps, hipGraphExec_t *exec)
{
    const Plan &P = b->plan;
    HIPCHECK(hipStreamBeginCapture(b->cap, hipStreamCaptureModeThreadLocal));
    hipError_t err = hipSuccess;
    for (int s = 0; s < nsteps && err == hipSuccess; ++s)
        for (int st = M_S1; st <= M_S4 && err == hipSuccess; ++st) {
            err = launch_stage1d(st, b->dwork, P.nwork, b->ddesc, P.waves, P.max_dpw, P.shape, P.nt, P.rk, b->cap);
            if (err == hipSuccess)
                err = launch_reduce1d(b->dred, P.nred, b->ddesc, st, nullptr,
                                      st == M_S4 ? 1 : 0, b->cap);
        }
    hipGraph_t graph = nullptr;
    hipError_t e2 = hipStreamEndCapture(b->cap, &graph);
    if (err != hipSuccess) {
        if (graph)
            (void)hipGraphDestroy(graph);
        return fail(FPIC_EHIP, std::string("kernel launch during capture: ") + hipGetErrorString(err));
    }
    HIPCHECK(e2);
    hipError_t e3 = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    HIPCHECK(e3);
    return FPIC_OK;
}

// The step graphs; a context that runs whole steps in one launch captures
// them only if it is stepped while its stream is being captured or while
// other contexts' launches leave no room.
int ensure_graphs(fpic_batch *b)
{
    int rc = b->g1 ? FPIC_OK : capture_steps(b, 1, &b->g1);
    if (!rc && b->plan.spg > 1 && !b->gK)
        rc = capture_steps(b, b->plan.spg, &b->gK);
    return rc;
}

// Whether a launch of whole steps gave up a wait (see GridBar).
int steps_ok(const fpic_batch *b)
{
    int failed;
    std::memcpy(&failed, b->hbuf + kFailed, sizeof failed);
    return failed ? fail(FPIC_EHIP, "the workgroups of a step launch did not run together") : FPIC_OK;
}

// Contexts whose latest launch of whole steps may still run, per device.  The
// workgroups of such a launch wait for one another, so launches that may run
// at the same time must fit the chip together.  They do if each workgroup
// could have a CU of its own on every XCD (the dispatcher hands workgroups to
// the XCDs in turn, so that n of them take at most ceil(n / kXcds) CUs on
// each): whatever order they are dispatched in, a place is then left for the
// next one.  A call that finds no room steps with one launch per stage, which
// waits for nothing: no stream ever waits for another one's.
constexpr int kXcds = 8, kMaxStepDevices = 64;
std::mutex g_steps_mu;
fpic_batch *g_steps_head[kMaxStepDevices];

void steps_unlist(fpic_batch *b)
{
    for (fpic_batch **p = &g_steps_head[b->device]; *p; p = &(*p)->steps_next)
        if (*p == b) {
            *p = b->steps_next;
            return;
        }
}

// Whether a launch of b may start beside those that may still run; if so, b
// counts among them.  Launches of one stream never run at the same time, so
// the latest stands for them, with the most that any of them takes
// (hipStreamPerThread names a stream per thread).
bool steps_reserve(fpic_batch *b)
{
    const int mine = (b->plan.nwork + kXcds - 1) / kXcds * kXcds;
    std::lock_guard<std::mutex> lock(g_steps_mu);
    auto same = [&](const fpic_batch *x) {
        return x == b || (x->stream == b->stream && b->stream != hipStreamPerThread && !x->launching);
    };
    auto room = [&]() {
        int sum = 0;
        for (fpic_batch *x = g_steps_head[b->device]; x; x = x->steps_next)
            sum += same(x) ? 0 : x->steps_held;
        return sum == 0 || sum + mine <= b->cus;
    };
    auto drop = [&](auto done) {
        for (fpic_batch *x = g_steps_head[b->device], *next; x; x = next) {
            next = x->steps_next;
            if (done(x))
                steps_unlist(x);
        }
    };
    if (!room()) {
        // without the launches that have finished (relaxed mode: another
        // thread may be capturing)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        drop([](const fpic_batch *x) { return !x->launching && hipEventQuery(x->done) == hipSuccess; });
        (void)hipGetLastError();  // not ready is no error
        (void)hipThreadExchangeStreamCaptureMode(&mode);
        if (!room())
            return false;
    }
    int held = mine;
    drop([&](const fpic_batch *x) {
        if (same(x))
            held = std::max(held, x->steps_held);
        return same(x);
    });
    b->steps_held = held;
    b->steps_next = g_steps_head[b->device];
    g_steps_head[b->device] = b;
    b->launching = true;
    return true;
}

// nsteps steps of the descriptors ds + j stride in one launch, after
// steps_reserve.  Its workgroups wait for one another at most 3 ms and about
// as long as the steps take (100 us each): an idle chip takes 1 to 4 us, one
// with other kernels on it as long as those run (products of 4096 x 4096
// matrices 53 us, sweeps over 2 GB 2.1 ms), and another process' launch of
// whole steps, which may hold a part of the chip while this one holds the rest
// (two processes, 2048 x 64, once in 530 launches), would never make room.
int run_steps(fpic_batch *b, const SimDesc *ds, int stride, int keep, int nsteps)
{
    const Plan &P = b->plan;
    const unsigned long long arrive =
        b->arrive_ticks == kArriveRule ? 300000ull + 10000ull * (unsigned)nsteps : b->arrive_ticks;
    const GridBar bar{reinterpret_cast<unsigned *>(b->ws + P.o_bar), b->launches, b->gen, arrive,
                      reinterpret_cast<int *>(b->hbuf + kFailed), b->bar_ticks};
    hipError_t e = launch_steps1d(b->dwork, P.nwork, ds, stride, keep, P.waves, P.shape, nsteps, bar, b->stream);
    if (e == hipSuccess) {
        b->launches += 1u;
        b->gen += 4u * (unsigned)nsteps;
        e = hipEventRecord(b->done, b->stream);
    }
    std::lock_guard<std::mutex> lock(g_steps_mu);
    b->launching = false;
    return e == hipSuccess ? FPIC_OK : fail(FPIC_EHIP, std::string("step launch: ") + hipGetErrorString(e));
}

}  // namespace

// For tests: how long the workgroups of this context's step launches wait for
// one another (0: the first ones do the work).
int fpic::set_arrive_ticks(void *ctx, unsigned long long ticks)
{
    fpic_ctx *c = static_cast<fpic_ctx *>(ctx);
    if (!c || !c->b || !c->b->steps)
        return fail(FPIC_EINVAL, "not a context that runs whole steps in one launch");
    c->b->arrive_ticks = ticks;
    return FPIC_OK;
}

extern "C" int fpic_test_step_waits(fpic_ctx *ctx, fpic_batch *batch, unsigned long long arrive_ticks,
                                    unsigned bar_ticks)
{
    fpic_batch *b = ctx ? ctx->b : batch;
    if (!b || !b->steps)
        return fail(FPIC_EINVAL, "not a context that runs whole steps in one launch");
    b->arrive_ticks = arrive_ticks;
    b->bar_ticks = bar_ticks;
    return FPIC_OK;
}

extern "C" int fpic_test_step_launches(fpic_ctx *ctx, fpic_batch *batch)
{
    fpic_batch *b = ctx ? ctx->b : batch;
    return b && b->steps ? (int)b->launches : -1;
}

namespace {

// The dispatcher hands workgroup b to XCD b % 8, and each XCD has its own
// L2.  Place item i of the preferred sequence at launch slot b such that
// every XCD receives one contiguous run of the sequence.
void xcd_order(const std::vector<WorkItem> &seq, std::vector<WorkItem> &out)
{
    const size_t n = seq.size();
    out.assign(n, WorkItem{0, 0, 0, 0});
    const size_t per = n / kXcds, extra = n % kXcds;
    // XCD x takes items [start_x, start_x + count_x) of seq
    std::vector<size_t> start(kXcds), count(kXcds);
    size_t at = 0;
    for (int x = 0; x < kXcds; ++x) {
        count[x] = per + ((size_t)x < extra ? 1 : 0);
        start[x] = at;
        at += count[x];
    }
    std::vector<size_t> used(kXcds, 0);
    for (size_t b = 0; b < n; ++b) {
        int x = (int)(b % kXcds);
        // slots beyond an XCD's share go to the next XCD with items left
        for (int tries = 0; tries < kXcds && used[x] >= count[x]; ++tries)
            x = (x + 1) % kXcds;
        out[b] = seq[start[x] + used[x]++];
    }
}

// Host copies of everything a batch uploads into its workspace: the
// per-simulation direction tables, the descriptors, the work tables (the
// cost-sorted global table, then one contiguous table per simulation) and
// the reduction table.  Device pointers in the descriptors point into ws.
struct HostTables {
    std::vector<double> tab;           // every simulation's [7][ndir] table
    std::vector<size_t> tab_off;       // where simulation i's table starts in tab
    std::vector<SimDesc> desc;
    std::vector<WorkItem> work;
    std::vector<RedItem> red;
    std::vector<int> swork_off, sred_off;
};

void build_tables(const Plan &P, const fpic_config *cfgs, char *ws, HostTables &T)
{
    const int nsim = P.nsim;
    T = HostTables();
    T.desc.resize(nsim);
    std::vector<WorkItem> persim;
    std::vector<std::pair<int, WorkItem>> costed;
    for (int i = 0; i < nsim; ++i) {
        const fpic_config &c = cfgs[i];
        const SimPlan &s = P.sims[i];
        const double dV = c.dx[0] * c.dx[1] * c.dx[2];
        const size_t t0 = T.tab.size();
        T.tab_off.push_back(t0);
        T.tab.resize(t0 + 7 * (size_t)s.ndir, 0.0);
        double *tab = T.tab.data() + t0;
        for (int d = 0; d < s.ndir; ++d) {
            tab[0 * s.ndir + d] = c.dirs[3 * d + 0];
            tab[1 * s.ndir + d] = c.dirs[3 * d + 1];
            tab[2 * s.ndir + d] = c.dirs[3 * d + 2];
            tab[3 * s.ndir + d] = c.N[d] / dV;
            tab[4 * s.ndir + d] = c.Nbar[d] / dV;
            tab[5 * s.ndir + d] = c.N[d];
            tab[6 * s.ndir + d] = c.Nbar[d];
        }
        SimDesc &D = T.desc[i];
        std::memset(&D, 0, sizeof D);
        D.ncell = s.ncell;
        D.ndir = s.ndir;
        D.ntile = s.ntile;
        D.ngroup = s.ngroup;
        D.dpw = s.dpw;
        D.dpg = s.dpw * P.waves;
        D.shape = P.shape;
        D.np = s.np;
        D.dt = c.dt;
        D.dz = c.dx[2];
        // packed upper triangle of hvac; the matter potential adds to the
        // diagonal for neutrinos and subtracts for antineutrinos (before
        // the conjugation that forms Hbar)
        const double *h = c.hvac;
        const double hv[9] = {h[0], h[8], h[16], h[2], h[3], h[4], h[5], h[10], h[11]};
        for (int k = 0; k < 9; ++k) {
            D.hvac[k] = hv[k] + (k < 3 ? c.vmat[k] : 0.0);
            D.hvacb[k] = hv[k] - (k < 3 ? c.vmat[k] : 0.0);
        }
        const double *tb = reinterpret_cast<const double *>(ws + s.o_tab);
        D.vx = tb;
        D.vy = tb + s.ndir;
        D.vz = tb + 2 * s.ndir;
        D.wN = tb + 3 * s.ndir;
        D.wNb = tb + 4 * s.ndir;
        D.Nw = tb + 5 * s.ndir;
        D.Nbw = tb + 6 * s.ndir;
        D.Y = reinterpret_cast<double *>(ws + s.o_Y);
        D.Yout = D.Y;
        D.K1 = reinterpret_cast<double *>(ws + s.o_K1);
        D.K2 = reinterpret_cast<double *>(ws + s.o_K2);
        D.K3 = reinterpret_cast<double *>(ws + s.o_K3);
        double *g0 = reinterpret_cast<double *>(ws + s.o_G0);
        double *g1 = reinterpret_cast<double *>(ws + s.o_G1);
        double *g2 = reinterpret_cast<double *>(ws + s.o_G2);
        double *g3 = reinterpret_cast<double *>(ws + s.o_G3);
        // the stage-1 and stage-2 grids g0, g1 stay until stage 4 has read them
        D.G[0] = g0;
        D.G[1] = g1;
        D.G[2] = g2;
        D.G[3] = g3;
        D.G[4] = g0;
        D.part = reinterpret_cast<double *>(ws + s.o_part);
        D.edge = reinterpret_cast<double *>(ws + s.o_edge);
        D.part2 = reinterpret_cast<double *>(ws + s.o_part2);
        D.edge2 = reinterpret_cast<double *>(ws + s.o_edge2);
        // (launches of whole steps store no slope in the context's own
        // buffers; with two tiles or more, 16 ndir ncell > 108 ndir ntile)
        D.xch = D.K1;
        D.red = reinterpret_cast<double *>(ws + P.o_scratch);
        D.step = reinterpret_cast<int64_t *>(ws + s.o_step);

        T.swork_off.push_back((int)persim.size());
        T.sred_off.push_back((int)T.red.size());
        const int dpg = D.dpg;
        for (int t = 0; t < s.ntile; ++t) {
            for (int g = 0; g < s.ngroup; ++g) {
                WorkItem w{i, t, g, 0};
                const int nd = std::min(dpg, s.ndir - g * dpg);
                persim.push_back(w);
                costed.push_back({nd, w});
            }
            T.red.push_back(RedItem{i, t});
        }
    }
    // Longest work first so the tail of the launch holds the short items;
    // among equals, direction group outer and tile inner, so neighbouring
    // tiles of one group (which share cache lines at their edges) are
    // consecutive.
    std::stable_sort(costed.begin(), costed.end(),
                     [](const std::pair<int, WorkItem> &a, const std::pair<int, WorkItem> &b2) {
                         if (a.first != b2.first)
                             return a.first > b2.first;
                         if (a.second.sim != b2.second.sim)
                             return a.second.sim < b2.second.sim;
                         if (a.second.group != b2.second.group)
                             return a.second.group < b2.second.group;
                         return a.second.tile < b2.second.tile;
                     });
    {
        std::vector<WorkItem> seq;
        for (auto &cw : costed)
            seq.push_back(cw.second);
        xcd_order(seq, T.work);
    }
    {
        std::vector<WorkItem> tmp;
        for (int i = 0; i < nsim; ++i) {
            // per-simulation tables get the same treatment, simulation by
            // simulation (each is launched on its own)
            const SimPlan &s = P.sims[i];
            std::vector<WorkItem> one;
            for (int g = 0; g < s.ngroup; ++g)
                for (int t = 0; t < s.ntile; ++t)
                    one.push_back(WorkItem{i, t, g, 0});
            xcd_order(one, tmp);
            T.work.insert(T.work.end(), tmp.begin(), tmp.end());
        }
    }
    for (int i = 0; i < nsim; ++i)
        T.swork_off[i] += P.nwork;
}

int batch_build(int nsim, const fpic_config *cfgs, const fpic_tuning *tune, void *workspace,
                size_t bytes, fpic_stream stream, fpic_batch **out)
{
    if (!out)
        return fail(FPIC_EINVAL, "out is null");
    *out = nullptr;
    Plan P;
    int rc = make_plan(nsim, cfgs, tune, P);
    if (rc)
        return rc;
    if (!workspace || bytes < P.total)
        return fail(FPIC_EINVAL, "workspace missing or smaller than fpic_workspace_bytes");
    if (reinterpret_cast<uintptr_t>(workspace) % 256)
        return fail(FPIC_EINVAL, "workspace must be 256-byte aligned");

    fpic_batch *b = new fpic_batch();
    b->plan = P;
    b->stream = static_cast<hipStream_t>(stream);
    b->ws = static_cast<char *>(workspace);
    b->ddesc = reinterpret_cast<SimDesc *>(b->ws + P.o_desc);
    b->dwork = reinterpret_cast<WorkItem *>(b->ws + P.o_work);
    b->dred = reinterpret_cast<RedItem *>(b->ws + P.o_red);
    b->dscratch = reinterpret_cast<double *>(b->ws + P.o_scratch);
    b->state_set.assign(nsim, false);
    b->cell_volume = cfgs[0].dx[0] * cfgs[0].dx[1] * cfgs[0].dx[2];

    auto cleanup = [&](int code) {
        fpic_batch_destroy(b);
        return code;
    };

    HostTables T;
    build_tables(P, cfgs, b->ws, T);
    b->hdesc = T.desc;
    b->swork_off = T.swork_off;
    b->sred_off = T.sred_off;
    hipError_t e = hipSuccess;
    for (int i = 0; i < nsim && e == hipSuccess; ++i)
        e = hipMemcpy(b->ws + P.sims[i].o_tab, T.tab.data() + T.tab_off[i],
                      sizeof(double) * 7 * (size_t)P.sims[i].ndir, hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(b->ddesc, T.desc.data(), sizeof(SimDesc) * nsim, hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(b->dwork, T.work.data(), sizeof(WorkItem) * T.work.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipMemcpy(b->dred, T.red.data(), sizeof(RedItem) * T.red.size(), hipMemcpyHostToDevice);
    if (e == hipSuccess)
        e = hipHostMalloc(reinterpret_cast<void **>(&b->hbuf), sizeof(double) * 64, hipHostMallocDefault);
    if (e == hipSuccess)
        e = hipStreamCreateWithFlags(&b->cap, hipStreamNonBlocking);
    if (e != hipSuccess)
        return cleanup(fail(FPIC_EHIP, std::string("create: ") + hipGetErrorString(e)));

    b->hbuf[kFailed] = 0.0;
    b->steps = P.steps && hipGetDevice(&b->device) == hipSuccess && b->device < kMaxStepDevices &&
               hipDeviceGetAttribute(&b->cus, hipDeviceAttributeMultiprocessorCount, b->device) == hipSuccess &&
               steps1d_fits(P.nwork, P.waves, P.shape);
    if (b->steps) {
        // (a copy like the tables above, finished when it returns: a memset on
        // the null stream may still run then, and a non-blocking stream does
        // not wait for it)
        const std::vector<unsigned> zero(kBarWords, 0u);
        e = hipMemcpy(b->ws + P.o_bar, zero.data(), sizeof(unsigned) * kBarWords, hipMemcpyHostToDevice);
        if (e == hipSuccess)
            e = hipEventCreateWithFlags(&b->done, hipEventDisableTiming);
        if (e != hipSuccess)
            return cleanup(fail(FPIC_EHIP, std::string("create: ") + hipGetErrorString(e)));
    } else {
        rc = ensure_graphs(b);
        if (rc)
            return cleanup(rc);
    }
    *out = b;
    return FPIC_OK;
}

int sim_work(fpic_batch *b, int sim, int *off, int *n, int *roff, int *rn)
{
    const SimPlan &s = b->plan.sims[sim];
    *off = b->swork_off[sim];
    *n = s.ntile * s.ngroup;
    *roff = b->sred_off[sim];
    *rn = s.ntile;
    return 0;
}

int batch_set_state(fpic_batch *b, int sim, const double *state, int64_t step0)
{
    if (!b || sim < 0 || sim >= b->plan.nsim || !state)
        return fail(FPIC_EINVAL, "set_state: bad batch, simulation index or state pointer");
    if (int rc = steps_ok(b))
        return rc;
    const SimPlan &s = b->plan.sims[sim];
    const SimDesc &D = b->hdesc[sim];
    HIPCHECK(hipMemcpyAsync(D.Y, state, sizeof(double) * 18 * s.np, hipMemcpyDeviceToDevice, b->stream));
    HIPCHECK(launch_set_step(b->ddesc, sim, sim + 1, step0, b->stream));
    int off, n, roff, rn;
    sim_work(b, sim, &off, &n, &roff, &rn);
    HIPCHECK(launch_stage1d(M_DEPOSIT, b->dwork + off, n, b->ddesc, b->plan.waves, b->plan.max_dpw, b->plan.shape,
                            b->plan.nt, 0, b->stream));
    HIPCHECK(launch_reduce1d(b->dred + roff, rn, b->ddesc, 0, nullptr, 0, b->stream));
    b->state_set[sim] = true;
    return FPIC_OK;
}

int batch_step(fpic_batch *b, int64_t nsteps)
{
    if (!b || nsteps < 0)
        return fail(FPIC_EINVAL, "step: bad batch or negative step count");
    for (bool ok : b->state_set)
        if (!ok)
            return fail(FPIC_ESTATE, "step before set_state");
    const int K = b->plan.spg;
    int64_t left = nsteps;
    if (b->steps) {
        int rc = steps_ok(b);
        if (rc)
            return rc;
        hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
        if (left > 0 && hipStreamIsCapturing(b->stream, &cs) == hipSuccess && cs == hipStreamCaptureStatusNone) {
            for (; left > 0 && steps_reserve(b); left -= kStepsPerLaunch) {
                rc = run_steps(b, b->ddesc, 0, 0, (int)std::min<int64_t>(left, kStepsPerLaunch));
                if (rc)
                    return rc;
            }
            if (left <= 0)
                return FPIC_OK;
        }
        (void)hipGetLastError();
        rc = ensure_graphs(b);
        if (rc)
            return rc;
    }
    while (K > 1 && left >= K) {
        HIPCHECK(hipGraphLaunch(b->gK, b->stream));
        left -= K;
    }
    while (left > 0) {
        HIPCHECK(hipGraphLaunch(b->g1, b->stream));
        --left;
    }
    return FPIC_OK;
}

int batch_totals(fpic_batch *b, int sim, double *out18)
{
    const SimPlan &s = b->plan.sims[sim];
    const int nblk = (int)std::max<int64_t>(1, std::min<int64_t>(kRedBlocks, (s.np + 255) / 256));
    HIPCHECK(launch_totals(b->ddesc, sim, nblk, b->dscratch, b->stream));
    HIPCHECK(hipMemcpyAsync(b->hbuf, b->dscratch, sizeof(double) * 18, hipMemcpyDeviceToHost, b->stream));
    HIPCHECK(hipStreamSynchronize(b->stream));
    std::memcpy(out18, b->hbuf, sizeof(double) * 18);
    return steps_ok(b);
}

}  // namespace

// ------------------------------------------------------------------ batch ABI
extern "C" {

const char *fpic_last_error(void) { return g_err.c_str(); }

int fpic_batch_workspace_bytes(int32_t nsim, const fpic_config *cfgs, const fpic_tuning *tune,
                               size_t *bytes)
{
    if (!bytes)
        return fail(FPIC_EINVAL, "bytes is null");
    Plan P;
    int rc = make_plan(nsim, cfgs, tune, P);
    if (rc)
        return rc;
    *bytes = P.total;
    return FPIC_OK;
}

int fpic_batch_create(int32_t nsim, const fpic_config *cfgs, const fpic_tuning *tune, void *workspace,
                      size_t workspace_bytes, fpic_stream stream, fpic_batch **out)
{
    return batch_build(nsim, cfgs, tune, workspace, workspace_bytes, stream, out);
}

int fpic_batch_set_state(fpic_batch *b, int32_t sim, const double *state, int64_t step0)
{
    return batch_set_state(b, sim, state, step0);
}

int fpic_batch_get_state(fpic_batch *b, int32_t sim, double *state)
{
    if (!b || sim < 0 || sim >= b->plan.nsim || !state)
        return fail(FPIC_EINVAL, "get_state: bad batch, simulation index or state pointer");
    if (int rc = steps_ok(b))
        return rc;
    const SimDesc &D = b->hdesc[sim];
    HIPCHECK(hipMemcpyAsync(state, D.Y, sizeof(double) * 18 * D.np, hipMemcpyDeviceToDevice, b->stream));
    return FPIC_OK;
}

int fpic_batch_step(fpic_batch *b, int64_t nsteps) { return batch_step(b, nsteps); }

int fpic_batch_flavor_totals(fpic_batch *b, double *out)
{
    if (!b || !out)
        return fail(FPIC_EINVAL, "flavor_totals: null argument");
    for (int i = 0; i < b->plan.nsim; ++i) {
        int rc = batch_totals(b, i, out + 18 * (size_t)i);
        if (rc)
            return rc;
    }
    return FPIC_OK;
}

int fpic_batch_sync(fpic_batch *b)
{
    if (!b)
        return fail(FPIC_EINVAL, "null batch");
    HIPCHECK(hipStreamSynchronize(b->stream));
    return steps_ok(b);
}

void fpic_batch_destroy(fpic_batch *b)
{
    if (!b)
        return;
    if (b->stream)
        (void)hipStreamSynchronize(b->stream);
    for (auto &g : b->adj.recompute)
        (void)hipGraphExecDestroy(g.second);
    for (auto &g : b->adj.reverse)
        (void)hipGraphExecDestroy(g.second);
    if (b->done) {
        // (counts until its latest launch has ended)
        (void)hipEventSynchronize(b->done);
        std::lock_guard<std::mutex> lock(g_steps_mu);
        steps_unlist(b);
        (void)hipEventDestroy(b->done);
    }
    if (b->g1)
        (void)hipGraphExecDestroy(b->g1);
    if (b->gK)
        (void)hipGraphExecDestroy(b->gK);
    if (b->cap)
        (void)hipStreamDestroy(b->cap);
    if (b->hbuf)
        (void)hipHostFree(b->hbuf);
    delete b;
}

// ------------------------------------------------------------ single-box ABI
int fpic_workspace_bytes(const fpic_config *cfg, const fpic_tuning *tune, size_t *bytes)
{
    if (!cfg || !bytes)
        return fail(FPIC_EINVAL, "null argument");
    if (!is_1d(*cfg))
        return fpic3d::workspace_bytes(*cfg, tune, bytes);
    return fpic_batch_workspace_bytes(1, cfg, tune, bytes);
}

int fpic_create(const fpic_config *cfg, const fpic_tuning *tune, void *workspace, size_t bytes,
                fpic_stream stream, fpic_ctx **out)
{
    if (!cfg || !out)
        return fail(FPIC_EINVAL, "null argument");
    *out = nullptr;
    fpic_ctx *c = new fpic_ctx();
    int rc;
    if (is_1d(*cfg))
        rc = batch_build(1, cfg, tune, workspace, bytes, stream, &c->b);
    else
        rc = fpic3d::create(*cfg, tune, workspace, bytes, stream, &c->c3);
    if (rc) {
        delete c;
        return rc;
    }
    *out = c;
    return FPIC_OK;
}

int fpic_set_state(fpic_ctx *c, const double *state, int64_t step0)
{
    if (!c)
        return fail(FPIC_EINVAL, "null context");
    if (c->c3)
        return fpic3d::set_state(c->c3, state, step0);
    return batch_set_state(c->b, 0, state, step0);
}

int fpic_get_state(fpic_ctx *c, double *state)
{
    if (!c)
        return fail(FPIC_EINVAL, "null context");
    if (c->c3)
        return fpic3d::get_state(c->c3, state);
    return fpic_batch_get_state(c->b, 0, state);
}

int fpic_step(fpic_ctx *c, int64_t nsteps)
{
    if (!c)
        return fail(FPIC_EINVAL, "null context");
    if (c->c3)
        return fpic3d::step(c->c3, nsteps);
    return batch_step(c->b, nsteps);
}

int fpic_moments(fpic_ctx *c, double *out)
{
    if (!c || !out)
        return fail(FPIC_EINVAL, "null argument");
    if (c->c3)
        return fpic3d::moments(c->c3, out);
    fpic_batch *b = c->b;
    if (!b->state_set[0])
        return fail(FPIC_ESTATE, "moments before set_state");
    if (int rc = steps_ok(b))
        return rc;
    int off, n, roff, rn;
    sim_work(b, 0, &off, &n, &roff, &rn);
    const int nc = b->plan.sims[0].ncell;
    HIPCHECK(launch_stage1d(M_MOM_NU, b->dwork + off, n, b->ddesc, b->plan.waves, b->plan.max_dpw, b->plan.shape, b->plan.nt, 0, b->stream));
    HIPCHECK(launch_reduce1d(b->dred + roff, rn, b->ddesc, RED_OUT, out, 0, b->stream));
    HIPCHECK(launch_stage1d(M_MOM_NUBAR, b->dwork + off, n, b->ddesc, b->plan.waves, b->plan.max_dpw, b->plan.shape, b->plan.nt, 0, b->stream));
    HIPCHECK(launch_reduce1d(b->dred + roff, rn, b->ddesc, RED_OUT, out + (size_t)NG * nc, 0, b->stream));
    return FPIC_OK;
}

int fpic_flavor_totals(fpic_ctx *c, double *out)
{
    if (!c || !out)
        return fail(FPIC_EINVAL, "null argument");
    if (c->c3)
        return fpic3d::flavor_totals(c->c3, out);
    if (!c->b->state_set[0])
        return fail(FPIC_ESTATE, "flavor_totals before set_state");
    return batch_totals(c->b, 0, out);
}

int fpic_check(fpic_ctx *c, double tol, double *max_trace_err)
{
    if (!c)
        return fail(FPIC_EINVAL, "null context");
    double r[3];
    if (c->c3) {
        int rc = fpic3d::check(c->c3, r);
        if (rc)
            return rc;
    } else {
        fpic_batch *b = c->b;
        if (!b->state_set[0])
            return fail(FPIC_ESTATE, "check before set_state");
        const SimPlan &s = b->plan.sims[0];
        const int nblk = (int)std::max<int64_t>(1, std::min<int64_t>(kRedBlocks, (s.np + 255) / 256));
        HIPCHECK(launch_check(b->ddesc, 0, nblk, b->dscratch, b->stream));
        HIPCHECK(hipMemcpyAsync(b->hbuf, b->dscratch, sizeof(double) * 3, hipMemcpyDeviceToHost, b->stream));
        HIPCHECK(hipStreamSynchronize(b->stream));
        std::memcpy(r, b->hbuf, sizeof r);
        int rc = steps_ok(b);
        if (rc)
            return rc;
    }
    const double e = std::max(r[0], r[1]);
    if (max_trace_err)
        *max_trace_err = e;
    if (r[2] > 0.0)
        return fail(FPIC_ENUMERIC, "state holds NaN or Inf entries");
    if (!(e <= tol))
        return fail(FPIC_ENUMERIC, "trace drift exceeds the tolerance");
    return FPIC_OK;
}

int fpic_domain_averages(fpic_ctx *c, const double *moments, double *out)
{
    if (!c || !moments || !out)
        return fail(FPIC_EINVAL, "domain_averages: null argument");
    hipStream_t s;
    double *scratch, *hbuf;
    int64_t nc;
    if (c->c3) {
        void *sv;
        fpic3d::diag_buffers(c->c3, &sv, &scratch, &hbuf, &nc);
        s = static_cast<hipStream_t>(sv);
    } else {
        s = c->b->stream;
        scratch = c->b->dscratch;
        hbuf = c->b->hbuf;
        nc = c->b->plan.sims[0].ncell;
    }
    // 24 sums, then nblk x 24 partials, in the context's diagnostic scratch
    const int nblk = (int)std::max<int64_t>(1, std::min<int64_t>(128, (nc + 255) / 256));
    HIPCHECK(launch_domain_sums(moments, nc, nblk, scratch + 24, scratch, s));
    HIPCHECK(hipMemcpyAsync(hbuf, scratch, sizeof(double) * 24, hipMemcpyDeviceToHost, s));
    HIPCHECK(hipStreamSynchronize(s));
    if (c->b)
        if (int rc = steps_ok(c->b))
            return rc;
    for (int q = 0; q < 24; ++q)
        out[q] = hbuf[q] / (double)nc;
    return FPIC_OK;
}

int fpic_get_step(fpic_ctx *c, int64_t *step)
{
    if (!c || !step)
        return fail(FPIC_EINVAL, "null argument");
    if (c->c3)
        return fpic3d::get_step(c->c3, step);
    fpic_batch *b = c->b;
    HIPCHECK(hipMemcpyAsync(b->hbuf, b->hdesc[0].step, sizeof(int64_t), hipMemcpyDeviceToHost, b->stream));
    HIPCHECK(hipStreamSynchronize(b->stream));
    std::memcpy(step, b->hbuf, sizeof(int64_t));
    return steps_ok(b);
}

int fpic_sync(fpic_ctx *c)
{
    if (!c)
        return fail(FPIC_EINVAL, "null context");
    if (c->c3)
        return fpic3d::sync(c->c3);
    return fpic_batch_sync(c->b);
}

void fpic_destroy(fpic_ctx *c)
{
    if (!c)
        return;
    if (c->b)
        fpic_batch_destroy(c->b);
    if (c->c3)
        fpic3d::destroy(c->c3);
    delete c;
}

// ------------------------------------------------------------ measurement
int fpic_profile(fpic_ctx *c, int32_t nsteps, double *ms)
{
    if (!c || !ms || nsteps < 1)
        return fail(FPIC_EINVAL, "profile: bad argument");
    if (c->c3)
        return fpic3d::profile(c->c3, nsteps, ms);
    return fpic_batch_profile(c->b, nsteps, ms);
}

int fpic_batch_profile(fpic_batch *b, int32_t nsteps, double *ms)
{
    if (!b || !ms || nsteps < 1)
        return fail(FPIC_EINVAL, "profile: bad argument");
    for (bool ok : b->state_set)
        if (!ok)
            return fail(FPIC_ESTATE, "profile before set_state");
    if (int rc = steps_ok(b))
        return rc;
    const Plan &P = b->plan;
    hipEvent_t ev[9];
    for (auto &e : ev)
        HIPCHECK(hipEventCreate(&e));
    double acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    int rc = FPIC_OK;
    for (int n = 0; n < nsteps && !rc; ++n) {
        hipError_t err = hipEventRecord(ev[0], b->stream);
        for (int st = M_S1; st <= M_S4 && err == hipSuccess; ++st) {
            err = launch_stage1d(st, b->dwork, P.nwork, b->ddesc, P.waves, P.max_dpw, P.shape, P.nt, P.rk, b->stream);
            if (err == hipSuccess)
                err = hipEventRecord(ev[2 * st - 1], b->stream);
            if (err == hipSuccess)
                err = launch_reduce1d(b->dred, P.nred, b->ddesc, st, nullptr,
                                      st == M_S4 ? 1 : 0, b->stream);
            if (err == hipSuccess)
                err = hipEventRecord(ev[2 * st], b->stream);
        }
        if (err == hipSuccess)
            err = hipEventSynchronize(ev[8]);
        for (int k = 0; k < 8 && err == hipSuccess; ++k) {
            float t = 0.f;
            err = hipEventElapsedTime(&t, ev[k], ev[k + 1]);
            acc[k] += t;
        }
        if (err != hipSuccess)
            rc = fail(FPIC_EHIP, std::string("profile: ") + hipGetErrorString(err));
    }
    for (auto &e : ev)
        (void)hipEventDestroy(e);
    for (int k = 0; k < 8; ++k)
        ms[k] = acc[k] / nsteps;
    return rc ? rc : steps_ok(b);
}


}  // extern "C"

// ------------------------------------------------------------ reverse mode
namespace {

void adj_layout(const fpic_batch *b, int64_t nsteps, int L, fpic_batch::Adj &A)
{
    const SimPlan &s = b->plan.sims[0];
    const size_t st = sizeof(double) * 18 * (size_t)s.np;
    const size_t gr = sizeof(double) * NG * (size_t)s.ncell;
    A.L = L;
    A.nseg = (int)((nsteps + L - 1) / L);
    Carver cv;
    A.o_ckpt = cv.take(st * A.nseg);
    A.o_segY = cv.take(st * (L + 1));
    A.o_segK = cv.take(sizeof(double) * NK * (size_t)s.np * 3 * (size_t)L);
    A.o_segG = cv.take(gr * 4 * (size_t)(L + 1));
    A.o_lam = cv.take(2 * st);
    A.o_lcur = cv.take(st);
    A.o_dres = cv.take(st);
    A.o_GA = cv.take(gr);
    A.o_dw = cv.take(sizeof(double) * 2 * (size_t)s.ndir * s.ntile);
    A.o_descF = cv.take(sizeof(SimDesc) * L);
    A.o_descR = cv.take(sizeof(SimDesc) * L);
    A.o_out = cv.take(sizeof(double) * 2 * (size_t)s.ndir);
    A.total = align_up(cv.off);
}

int adj_check_cfg(fpic_ctx *c, const fpic_adjoint_cfg *a)
{
    if (!c || !a)
        return fail(FPIC_EINVAL, "adjoint: null argument");
    if (c->c3 || !c->b || c->b->plan.nsim != 1)
        return fail(FPIC_EUNSUPPORTED, "the adjoint covers single 1D boxes");
    if (a->nsteps < 1 || a->ckpt_every < 1)
        return fail(FPIC_EINVAL, "adjoint: nsteps and ckpt_every must be >= 1");
    return FPIC_OK;
}

// capture `fn` (which launches on stream s) into an executable graph
template <class F>
int capture(hipStream_t s, F fn, hipGraphExec_t *exec)
{
    HIPCHECK(hipStreamBeginCapture(s, hipStreamCaptureModeThreadLocal));
    hipError_t err = fn();
    hipGraph_t graph = nullptr;
    hipError_t e2 = hipStreamEndCapture(s, &graph);
    if (err != hipSuccess) {
        if (graph)
            (void)hipGraphDestroy(graph);
        return fail(FPIC_EHIP, std::string("launch during capture: ") + hipGetErrorString(err));
    }
    HIPCHECK(e2);
    hipError_t e3 = hipGraphInstantiate(exec, graph, nullptr, nullptr, 0);
    (void)hipGraphDestroy(graph);
    HIPCHECK(e3);
    return FPIC_OK;
}

int adj_graph(fpic_batch *b, bool reverse, int len, hipGraphExec_t *out)
{
    auto &cache = reverse ? b->adj.reverse : b->adj.recompute;
    for (auto &g : cache)
        if (g.first == len) {
            *out = g.second;
            return FPIC_OK;
        }
    const Plan &P = b->plan;
    const SimDesc *F = reinterpret_cast<const SimDesc *>(b->adj.ws + b->adj.o_descF);
    const SimDesc *R = reinterpret_cast<const SimDesc *>(b->adj.ws + b->adj.o_descR);
    hipGraphExec_t g = nullptr;
    int rc;
    if (!reverse) {
        rc = capture(b->cap, [&]() -> hipError_t {
            for (int j = 0; j < len; ++j)
                for (int st = M_S1; st <= M_S4; ++st) {
                    // the reverse sweep reads every stored slope, k1 included
                    hipError_t e = launch_stage1d(st, b->dwork, P.nwork, F + j, P.waves, P.max_dpw, P.shape, P.nt,
                                                  0, b->cap);
                    if (e == hipSuccess)
                        e = launch_reduce1d(b->dred, P.nred, F + j, st, nullptr, st == M_S4 ? 1 : 0, b->cap);
                    if (e != hipSuccess)
                        return e;
                }
            return hipSuccess;
        }, &g);
    } else {
        rc = capture(b->cap, [&]() -> hipError_t {
            for (int j = len - 1; j >= 0; --j) {
                // sources of stage 4, then (gather of stage s+1 with the
                // sources of stage s) for s = 3, 2, 1, then the gather of
                // stage 1; each source deposit is closed by a reduction
                for (int kind = 4; kind >= 0; --kind) {
                    hipError_t e = launch_adj1d(kind, b->dwork, P.nwork, R + j, P.waves, P.max_dpw, P.shape, b->cap);
                    if (e == hipSuccess && kind > 0)
                        e = launch_reduce1d(b->dred, P.nred, R + j, RED_GA, nullptr, 0, b->cap);
                    if (e != hipSuccess)
                        return e;
                }
                hipError_t e = launch_tick(R + j, -1, b->cap);
                if (e != hipSuccess)
                    return e;
            }
            return hipSuccess;
        }, &g);
    }
    if (rc)
        return rc;
    cache.push_back({len, g});
    *out = g;
    return FPIC_OK;
}

int read_step(fpic_batch *b, int64_t *step)
{
    HIPCHECK(hipMemcpyAsync(b->hbuf, b->hdesc[0].step, sizeof(int64_t), hipMemcpyDeviceToHost, b->stream));
    HIPCHECK(hipStreamSynchronize(b->stream));
    std::memcpy(step, b->hbuf, sizeof(int64_t));
    return steps_ok(b);
}

}  // namespace

extern "C" {

int fpic_adjoint_workspace_bytes(fpic_ctx *c, const fpic_adjoint_cfg *a, size_t *bytes)
{
    int rc = adj_check_cfg(c, a);
    if (rc)
        return rc;
    if (!bytes)
        return fail(FPIC_EINVAL, "bytes is null");
    fpic_batch::Adj A;
    adj_layout(c->b, a->nsteps, (int)std::min<int64_t>(a->ckpt_every, a->nsteps), A);
    *bytes = A.total;
    return FPIC_OK;
}

int fpic_adjoint_forward(fpic_ctx *c, const fpic_adjoint_cfg *a, void *ws, size_t bytes)
{
    int rc = adj_check_cfg(c, a);
    if (rc)
        return rc;
    fpic_batch *b = c->b;
    if (!b->state_set[0])
        return fail(FPIC_ESTATE, "adjoint forward before set_state");
    const int L = (int)std::min<int64_t>(a->ckpt_every, a->nsteps);
    fpic_batch::Adj A;
    adj_layout(b, a->nsteps, L, A);
    if (!ws || bytes < A.total || reinterpret_cast<uintptr_t>(ws) % 256)
        return fail(FPIC_EINVAL, "adjoint workspace missing, too small or misaligned");
    // graphs of an earlier layout point at old descriptors: drop them
    for (auto &g : b->adj.recompute)
        (void)hipGraphExecDestroy(g.second);
    for (auto &g : b->adj.reverse)
        (void)hipGraphExecDestroy(g.second);
    A.ws = static_cast<char *>(ws);
    b->adj = A;
    rc = read_step(b, &b->adj.n_start);
    if (rc)
        return rc;
    b->adj.nsteps = a->nsteps;

    // per-step descriptors of a segment
    const SimPlan &sp = b->plan.sims[0];
    const size_t st = 18 * (size_t)sp.np, sk = NK * (size_t)sp.np, gr = NG * (size_t)sp.ncell;
    double *segY = reinterpret_cast<double *>(A.ws + A.o_segY);
    double *segK = reinterpret_cast<double *>(A.ws + A.o_segK);
    double *segG = reinterpret_cast<double *>(A.ws + A.o_segG);
    double *lam = reinterpret_cast<double *>(A.ws + A.o_lam);
    double *dw = reinterpret_cast<double *>(A.ws + A.o_dw);
    std::vector<SimDesc> F(L), R(L);
    for (int j = 0; j < L; ++j) {
        SimDesc D = b->hdesc[0];
        D.Y = segY + st * j;
        D.Yout = segY + st * (j + 1);
        D.K1 = segK + sk * (3 * (size_t)j + 0);
        D.K2 = segK + sk * (3 * (size_t)j + 1);
        D.K3 = segK + sk * (3 * (size_t)j + 2);
        for (int q = 0; q < 4; ++q)
            D.G[q] = segG + gr * (4 * (size_t)j + q);
        D.G[4] = segG + gr * (4 * (size_t)(j + 1));
        D.GA = reinterpret_cast<double *>(A.ws + A.o_GA);
        D.lam[0] = lam;
        D.lam[1] = lam + st;
        D.lcur = reinterpret_cast<double *>(A.ws + A.o_lcur);
        D.dres = reinterpret_cast<double *>(A.ws + A.o_dres);
        D.dwN = dw;
        D.dwNb = dw + (size_t)sp.ndir * sp.ntile;
        F[j] = D;
        R[j] = D;
    }
    HIPCHECK(hipMemcpyAsync(A.ws + A.o_descF, F.data(), sizeof(SimDesc) * L, hipMemcpyHostToDevice, b->stream));
    HIPCHECK(hipMemcpyAsync(A.ws + A.o_descR, R.data(), sizeof(SimDesc) * L, hipMemcpyHostToDevice, b->stream));
    HIPCHECK(hipStreamSynchronize(b->stream));

    // forward with checkpoints
    double *ckpt = reinterpret_cast<double *>(A.ws + A.o_ckpt);
    int64_t left = a->nsteps;
    for (int seg = 0; seg < A.nseg; ++seg) {
        HIPCHECK(hipMemcpyAsync(ckpt + st * seg, b->hdesc[0].Y, sizeof(double) * st,
                                hipMemcpyDeviceToDevice, b->stream));
        const int64_t n = std::min<int64_t>(L, left);
        rc = batch_step(b, n);
        if (rc)
            return rc;
        left -= n;
    }
    b->adj.forward_done = true;
    return FPIC_OK;
}

int fpic_adjoint_backward(fpic_ctx *c, const double *dLdy_end, double *dLdy0, double *dLdN,
                          double *dLdNbar)
{
    if (!c || !c->b || c->c3)
        return fail(FPIC_EINVAL, "adjoint backward: bad context");
    fpic_batch *b = c->b;
    fpic_batch::Adj &A = b->adj;
    if (!A.forward_done)
        return fail(FPIC_ESTATE, "adjoint backward before fpic_adjoint_forward");
    if (!dLdy_end || !dLdy0 || !dLdN || !dLdNbar)
        return fail(FPIC_EINVAL, "adjoint backward: null argument");
    const SimPlan &sp = b->plan.sims[0];
    const Plan &P = b->plan;
    const size_t st = 18 * (size_t)sp.np;
    double *ckpt = reinterpret_cast<double *>(A.ws + A.o_ckpt);
    double *segY = reinterpret_cast<double *>(A.ws + A.o_segY);
    double *lam = reinterpret_cast<double *>(A.ws + A.o_lam);
    double *dw = reinterpret_cast<double *>(A.ws + A.o_dw);
    double *outw = reinterpret_cast<double *>(A.ws + A.o_out);
    const SimDesc *F = reinterpret_cast<const SimDesc *>(A.ws + A.o_descF);
    const int64_t n_end = A.n_start + A.nsteps;
    hipStream_t s = b->stream;

    HIPCHECK(hipMemcpyAsync(lam + st * (size_t)(n_end & 1), dLdy_end, sizeof(double) * st,
                            hipMemcpyDeviceToDevice, s));
    HIPCHECK(launch_fill(dw, 2 * (size_t)sp.ndir * sp.ntile, 0.0, s));
    int off, n, roff, rn;
    sim_work(b, 0, &off, &n, &roff, &rn);
    for (int seg = A.nseg - 1; seg >= 0; --seg) {
        const int64_t n0 = A.n_start + (int64_t)seg * A.L;
        const int len = (int)std::min<int64_t>(A.L, n_end - n0);
        // restore the checkpoint and recompute the segment, keeping its
        // states, slopes and moment grids
        HIPCHECK(hipMemcpyAsync(segY, ckpt + st * seg, sizeof(double) * st, hipMemcpyDeviceToDevice, s));
        HIPCHECK(launch_set_step(F, 0, 1, n0, s));
        HIPCHECK(launch_stage1d(M_DEPOSIT, b->dwork + off, n, F, P.waves, P.max_dpw, P.shape, P.nt, 0, s));
        HIPCHECK(launch_reduce1d(b->dred + roff, rn, F, 0, nullptr, 0, s));
        hipGraphExec_t g = nullptr;
        const bool whole = b->steps && steps_reserve(b);
        int rc = whole ? run_steps(b, F, 1, 1, len) : adj_graph(b, false, len, &g);
        if (rc)
            return rc;
        if (!whole)
            HIPCHECK(hipGraphLaunch(g, s));
        // sweep the segment backwards
        HIPCHECK(launch_set_step(F, 0, 1, n0 + len - 1, s));
        rc = adj_graph(b, true, len, &g);
        if (rc)
            return rc;
        HIPCHECK(hipGraphLaunch(g, s));
    }
    HIPCHECK(hipMemcpyAsync(dLdy0, lam + st * (size_t)(A.n_start & 1), sizeof(double) * st,
                            hipMemcpyDeviceToDevice, s));
    // the kernels accumulate dL/d(N/dV); dL/dN = dL/d(N/dV) / dV
    HIPCHECK(launch_tile_sum(dw, sp.ndir, sp.ntile, 1.0, outw, s));
    HIPCHECK(launch_tile_sum(dw + (size_t)sp.ndir * sp.ntile, sp.ndir, sp.ntile, 1.0, outw + sp.ndir, s));
    std::vector<double> h(2 * (size_t)sp.ndir);
    HIPCHECK(hipMemcpyAsync(h.data(), outw, sizeof(double) * h.size(), hipMemcpyDeviceToHost, s));
    // restore the step counter of the context (its state was never touched)
    HIPCHECK(launch_set_step(b->ddesc, 0, 1, n_end, s));
    HIPCHECK(hipStreamSynchronize(s));
    int rc = steps_ok(b);
    if (rc)
        return rc;
    const double inv_dV = 1.0 / b->cell_volume;
    for (int d = 0; d < sp.ndir; ++d) {
        dLdN[d] = h[d] * inv_dV;
        dLdNbar[d] = h[sp.ndir + d] * inv_dV;
    }
    return FPIC_OK;
}

}  // extern "C"

extern "C" {
// ------------------------------------------------------------- autotuning
// Milliseconds per step of one candidate launch shape (or < 0 when it does
// not fit the workspace or makes too many partial sums).
static int time_candidate(int nsim, const fpic_config *cfgs, const fpic_tuning &t, void *workspace,
                          size_t bytes, fpic_stream stream, double *ms_out, int nrep = 16)
{
    *ms_out = -1.0;
    hipStream_t s = static_cast<hipStream_t>(stream);
    Plan P;
    if (make_plan(nsim, cfgs, &t, P))
        return fail(FPIC_EINVAL, g_err);
    if (P.total > bytes)
        return FPIC_OK;
    // skip shapes whose partial sums would dwarf the grid
    for (auto &sp : P.sims)
        if (sp.ngroup > 96)
            return FPIC_OK;
    fpic_batch *b = nullptr;
    int rc = batch_build(nsim, cfgs, &t, workspace, bytes, stream, &b);
    if (rc)
        return rc;
    // Candidates run from step 1000: by then every direction's shift has long
    // left the alignment of the rows at step 0, as in a run's steady state
    // (timed from step 0, the order of nearly equal shapes can differ).
    constexpr int64_t kTuneStep0 = 1000;
    for (int i = 0; i < nsim; ++i) {
        hipError_t e = launch_fill_state(b->ddesc, i, s);
        if (e == hipSuccess)
            e = launch_set_step(b->ddesc, i, i + 1, kTuneStep0, s);
        if (e != hipSuccess) {
            fpic_batch_destroy(b);
            return fail(FPIC_EHIP, hipGetErrorString(e));
        }
        int off, n, roff, rn;
        sim_work(b, i, &off, &n, &roff, &rn);
        (void)launch_stage1d(M_DEPOSIT, b->dwork + off, n, b->ddesc, P.waves, P.max_dpw, P.shape, P.nt, 0, s);
        (void)launch_reduce1d(b->dred + roff, rn, b->ddesc, 0, nullptr, 0, s);
        b->state_set[i] = true;
    }
    hipEvent_t e0, e1;
    (void)hipEventCreate(&e0);
    (void)hipEventCreate(&e1);
    int rc2 = batch_step(b, 8);
    (void)hipEventRecord(e0, s);
    if (!rc2)
        rc2 = batch_step(b, nrep);
    (void)hipEventRecord(e1, s);
    hipError_t es = hipEventSynchronize(e1);
    float ms = 0.f;
    (void)hipEventElapsedTime(&ms, e0, e1);
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    fpic_batch_destroy(b);
    if (rc2)
        return rc2;
    if (es != hipSuccess)
        return fail(FPIC_EHIP, hipGetErrorString(es));
    *ms_out = ms / nrep;
    return FPIC_OK;
}

int fpic_autotune(int32_t nsim, const fpic_config *cfgs, void *workspace, size_t bytes,
                  fpic_stream stream, fpic_tuning *best, double *ms_per_step)
{
    if (!best)
        return fail(FPIC_EINVAL, "best is null");
    if (nsim == 1 && cfgs && !is_1d(cfgs[0]))
        return fpic3d::autotune(cfgs[0], workspace, bytes, stream, best, ms_per_step);
    // launch shapes with the size-chosen cache policy, timed over 16 steps
    std::vector<std::pair<double, fpic_tuning>> timed;
    for (int waves : {1, 2, 4, 8})
        for (int dpw : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32}) {
            const fpic_tuning t{waves, dpw, 8, 0};
            double per;
            int rc = time_candidate(nsim, cfgs, t, workspace, bytes, stream, &per);
            if (rc)
                return rc;
            if (per >= 0.0)
                timed.push_back({per, t});
        }
    if (timed.empty())
        return fail(FPIC_EINVAL, "workspace too small for every candidate shape");
    std::stable_sort(timed.begin(), timed.end(),
                     [](const std::pair<double, fpic_tuning> &a, const std::pair<double, fpic_tuning> &c) {
                         return a.first < c.first;
                     });
    // the leaders (at most four, within 5% of the fastest) and then the
    // other two cache policies for the best of them, each by the median of
    // three runs of 64 steps: single short runs differ by about 1%, as much
    // as the leading shapes do
    auto precise = [&](const fpic_tuning &t, double *per) -> int {
        double r[3];
        for (int k = 0; k < 3; ++k) {
            int rc = time_candidate(nsim, cfgs, t, workspace, bytes, stream, &r[k], 64);
            if (rc)
                return rc;
        }
        std::sort(r, r + 3);
        *per = r[1];
        return FPIC_OK;
    };
    double best_ms = 1e300;
    fpic_tuning bt = timed[0].second;
    for (size_t i = 0; i < timed.size() && i < 4 && timed[i].first <= 1.05 * timed[0].first; ++i) {
        double per;
        int rc = precise(timed[i].second, &per);
        if (rc)
            return rc;
        if (per >= 0.0 && per < best_ms) {
            best_ms = per;
            bt = timed[i].second;
        }
    }
    for (int policy : {1, 2}) {
        fpic_tuning t = bt;
        t.cache_policy = policy;
        double per;
        int rc = precise(t, &per);
        if (rc)
            return rc;
        if (per >= 0.0 && per < best_ms) {
            best_ms = per;
            bt = t;
        }
    }
    // and fewer slopes formed again (1: k1 only; 2: none, all stored)
    for (int fused : {1, 2}) {
        fpic_tuning t = bt;
        t.fused = fused;
        double per;
        int rc = precise(t, &per);
        if (rc)
            return rc;
        if (per >= 0.0 && per < best_ms) {
            best_ms = per;
            bt = t;
        }
    }
    *best = bt;
    if (ms_per_step)
        *ms_per_step = best_ms;
    return FPIC_OK;
}

}  // extern "C"

// ---------------------------------------------------- allocation-free entry
// Device scratch of fpic_step_noalloc: every buffer a 1D box needs besides
// its state (direction tables, descriptor, work tables, the three stored
// slopes, the two moment grids, the partial sums and the step counter).
// Each device the library runs on holds its own copy until the process
// ends.  In host code `scratch` names a host-side stand-in, not device
// memory: host code reaches the array only through the address that
// hipGetSymbolAddress returns on each device (scratch_base below).
namespace {
constexpr size_t kScratchBytes = FPIC_NOALLOC_SCRATCH_BYTES;
}  // namespace
static __device__ __align__(256) char scratch[kScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_base[kMaxDevices];

// The device address of `scratch` on the calling thread's current device,
// looked up once per device.
int scratch_base(char **out)
{
    int dev = -1;
    HIPCHECK(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices)
        return fail(FPIC_EUNSUPPORTED, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_base[dev]) {
        void *p = nullptr;
        HIPCHECK(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || reinterpret_cast<uintptr_t>(p) % 256)
            return fail(FPIC_EHIP, "hipGetSymbolAddress gave no 256-byte aligned address");
        g_scratch_base[dev] = p;
    }
    *out = static_cast<char *>(g_scratch_base[dev]);
    return FPIC_OK;
}
}  // namespace

extern "C" {

int fpic_step_noalloc(const fpic_config *cfg, const fpic_tuning *tune, double *state,
                      int64_t step0, int64_t nsteps, fpic_stream stream)
{
    if (!cfg || !state)
        return fail(FPIC_EINVAL, "step_noalloc: null cfg or state");
    if (nsteps < 0)
        return fail(FPIC_EINVAL, "step_noalloc: negative step count");
    if (reinterpret_cast<uintptr_t>(state) % sizeof(double))
        return fail(FPIC_EINVAL, "step_noalloc: state must be 8-byte aligned");
    if (!is_1d(*cfg))
        return fail(FPIC_EUNSUPPORTED, "step_noalloc: 1D boxes only (ncell = {1, 1, nz})");
    Plan P;
    int rc = make_plan(1, cfg, tune, P, true);
    if (rc)
        return rc;
    if (P.total > kScratchBytes) {
        char buf[200];
        std::snprintf(buf, sizeof buf,
                      "step_noalloc: this box needs %zu bytes of scratch; the limit is %zu "
                      "(use fpic_create with a workspace instead)",
                      P.total, kScratchBytes);
        return fail(FPIC_EINVAL, buf);
    }
    char *ws = nullptr;
    rc = scratch_base(&ws);
    if (rc)
        return rc;
    HostTables T;
    build_tables(P, cfg, ws, T);
    T.desc[0].Y = state;   // stepped in place
    T.desc[0].Yout = state;
    hipStream_t s = static_cast<hipStream_t>(stream);
    SimDesc *ddesc = reinterpret_cast<SimDesc *>(ws + P.o_desc);
    WorkItem *dwork = reinterpret_cast<WorkItem *>(ws + P.o_work);
    RedItem *dred = reinterpret_cast<RedItem *>(ws + P.o_red);
    // stream-ordered uploads: a call queued behind an earlier call on the
    // same stream sees its own tables
    HIPCHECK(hipMemcpyAsync(ws + P.sims[0].o_tab, T.tab.data(), sizeof(double) * T.tab.size(),
                            hipMemcpyHostToDevice, s));
    HIPCHECK(hipMemcpyAsync(ddesc, T.desc.data(), sizeof(SimDesc), hipMemcpyHostToDevice, s));
    HIPCHECK(hipMemcpyAsync(dwork, T.work.data(), sizeof(WorkItem) * (size_t)P.nwork,
                            hipMemcpyHostToDevice, s));
    HIPCHECK(hipMemcpyAsync(dred, T.red.data(), sizeof(RedItem) * T.red.size(),
                            hipMemcpyHostToDevice, s));
    // as fpic_set_state: step counter, then the first-stage moments
    HIPCHECK(launch_set_step(ddesc, 0, 1, step0, s));
    HIPCHECK(launch_stage1d(M_DEPOSIT, dwork, P.nwork, ddesc, P.waves, P.max_dpw, P.shape, P.nt, 0, s));
    HIPCHECK(launch_reduce1d(dred, P.nred, ddesc, 0, nullptr, 0, s));
    // as fpic_step, one launch per kernel instead of a graph
    for (int64_t n = 0; n < nsteps; ++n)
        for (int st = M_S1; st <= M_S4; ++st) {
            HIPCHECK(launch_stage1d(st, dwork, P.nwork, ddesc, P.waves, P.max_dpw, P.shape, P.nt, P.rk, s));
            HIPCHECK(launch_reduce1d(dred, P.nred, ddesc, st, nullptr, st == M_S4 ? 1 : 0, s));
        }
    // the host tables above must outlive their copies
    HIPCHECK(hipStreamSynchronize(s));
    return FPIC_OK;
}

}  // extern "C"
