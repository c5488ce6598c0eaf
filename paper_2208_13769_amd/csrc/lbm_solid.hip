// lbm_solid.hip -- single-plate host runtime and C ABI (include/lbm_solid.h).
//
// A handle owns no device memory: the caller's workspace is carved into two
// copies of the state (ping-pong), a read-out staging area, reduction
// scratch and a flag word. lbm_step only enqueues kernels on the caller's
// stream.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "host_common.hpp"
#include "split_plan.hpp"

using namespace lbm;

namespace {

struct Layout {
    StateLayout state;
    size_t staging, staging_bytes;
    size_t partials, small, total;
    // walled workspace: a third buffer of j (the extrapolation variant), the material
    // mask [ny][nx] bytes, and the lists of the split plans of one and two
    // steps (split_plan.hpp)
    size_t scratch, mask, list[2], total_walled;
};

// Entries of a split plan's list (fused tiles and windows) there is room for.
size_t list_capacity(int nx, int ny) { return 4096 + (size_t)nx * ny / 128; }

Layout make_layout(int nx, int ny, lbm_precision p)
{
    Layout L{};
    L.state = state_layout(nx, ny, p);
    size_t off = L.state.bytes;
    L.staging = off;
    L.staging_bytes = staging_bytes_for(nx, ny);
    off = align_up(off + L.staging_bytes);
    L.partials = off;
    off = align_up(off + kMaxDiagBlocks * 8 * sizeof(double));
    L.small = off;  // flag word + final diagnostics
    off = align_up(off + 64 * sizeof(double));
    L.total = off;
    L.scratch = off;
    L.mask = align_up(off + 2 * (size_t)nx * ny * elem_sizes(p).j);
    L.list[0] = align_up(L.mask + (size_t)nx * ny);
    L.list[1] = align_up(L.list[0] + sizeof(int4) * list_capacity(nx, ny));
    L.total_walled = align_up(L.list[1] + sizeof(int4) * list_capacity(nx, ny));
    return L;
}

}  // namespace

// Device scratch of lbm_read_diagnostics_noalloc: the per-block partial sums
// of the diagnostics kernel (kMaxDiagBlocks blocks, 8 doubles each) and the
// folded values (8 doubles). Each GPU holds its own copy until the process
// ends; every call on a GPU shares it.
constexpr size_t kNoAllocDiagDoubles = (size_t)kMaxDiagBlocks * 8 + 8;
static __device__ __align__(256) double scratch[kNoAllocDiagDoubles];

struct lbm_solver {
    int nx = 0, ny = 0;
    int device = 0;  // the device current at lbm_create
    int cus = 256;   // its compute units
    double dx = 1.0;
    lbm_precision prec = LBM_FP64;
    lbm_scheme scheme = LBM_SCHEME_PC;
    char *ws = nullptr;
    size_t ws_bytes = 0;
    hipStream_t stream = nullptr;
    Layout L{};
    int cur = 0;  // copy holding the current state
    int jslot = 0, jback = 1;  // buffers of the current j and of the one before it (j extrapolated)
    // From the first captured step on a graph holds the addresses of these
    // buffers: where the state lies then depends only on the steps since
    // set_fields, odd or even, as with one launch per step, and `home` is the
    // copy (jhome, jhome_back the buffers of j) of an even number of them.
    bool fixed = false;
    int home = 0, jhome = 0, jhome_back = 1;
    bool material = false, fields = false;
    double rho0 = 1, lam = 0, mu = 0, tau = 1;
    double body[2] = {0, 0};
    int bc[4] = {LBM_BC_PERIODIC, LBM_BC_PERIODIC, LBM_BC_PERIODIC, LBM_BC_PERIODIC};
    double bcval[4][2] = {};
    // Momentum walls move with velocity j* / rho0: the wall of edge e is at
    // uwb[e] + j*_L n at step n (lattice units). Changing j* at step n moves
    // uwb so that the displacement stays continuous.
    double uwb[4][2] = {};
    double f_scale = 1.0;
    int64_t steps = 0;
    Shape shape{}, created_shape{};  // of the fused kernel now, and as lbm_create planned it
    int spl = 1;  // time steps per launch (1, or 2 with the predictor-corrector)
    int sr = 0;   // stochastic rounding of 16-bit populations
    unsigned long long seed = 0;
    bool force_general = false;  // run the general step even without x walls
    bool fused_set = false;      // the caller chose the fused kernel or its launch shape
    Shape pair_shape{};          // launch shape of the library's own two-step launches (plan_pairs)
    bool pair_for = false;       // it is planned
    bool has_mask = false;       // holes (lbm_set_mask)
    std::vector<unsigned char> mask_host;  // host copy of the mask (1 material, 0 hole)
    // how launches of one and of two steps split the plate between the fused
    // kernel and windows; rebuilt when the mask or the kind of an edge changes
    SplitPlan split[2];
    // The windows of a large split plate run on a second stream beside the
    // fused share (forked from and joined back into the handle's stream each
    // launch); created on first use, default priority.
    hipStream_t aux = nullptr;
    char *pin = nullptr;  // page-locked, kPinBytes; from the second read or the first sample on
    int reads = 0;
    hipEvent_t fork = nullptr, join = nullptr;
    ~lbm_solver()
    {
        if (aux) (void)hipStreamSynchronize(aux);
        if (fork) (void)hipEventDestroy(fork);
        if (join) (void)hipEventDestroy(join);
        if (aux) (void)hipStreamDestroy(aux);
        if (!pin) return;
        // (a handle may go while another stream is being captured, which a free
        // in any but the relaxed mode would end)
        hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
        const bool relaxed = hipThreadExchangeStreamCaptureMode(&mode) == hipSuccess;
        (void)hipHostFree(pin);
        if (relaxed) (void)hipThreadExchangeStreamCaptureMode(&mode);
    }

    // plates that the fused kernel's walled form cannot run whole
    bool general() const
    {
        return force_general || has_mask || bc[LBM_EDGE_XMIN] != LBM_BC_PERIODIC || scheme == LBM_SCHEME_EXTRAP;
    }
    // Whether windows (window_kernel.hpp) run the whole plate: where the caller
    // asked for the general step; with j extrapolated unless a plate with walls
    // is large enough for the periodic form to run most of it; else, unless the
    // caller chose the fused kernel or its shape, up to the size where the
    // fused kernel (with windows at walls and holes) caught up. us per step,
    // windows / that: periodic FP64 700^2 31.9 / 31.8, FP32 1000^2 27.6 / 27.1,
    // FP32_U64 1400^2 53 / 48, FP16 1400^2 65 / 61; y walls FP64 700^2 34 / 39,
    // 1000^2 70 / 49, FP32 1000^2 33.8 / 34.1, FP32_U64 39 / 43, FP16 1400^2 73
    // / 71; four walls, and with a hole, FP64 700^2 43 / 42, 46 / 46, FP32 900^2 32
    // / 30, 35 / 38, 1000^2 42 / 31, 48 / 39, FP32_U64 950^2 43 / 40, 48 / 48, FP16
    // 950^2 51 / 51, 57 / 52. The explicit scheme's windows lose three rings a step
    // where these lose five: four walls 1000^2 FP64 47 / 57, FP32 24 / 32, FP32_U64
    // 27 / 36, FP16 31 / 35; y walls FP64 1000^2 39 / 52, 1700^2 128 / 148. Narrow
    // plates go by their sites too.
    bool windows() const
    {
        if (scheme == LBM_SCHEME_EXTRAP) return !walls() || (double)nx * ny <= 3e5;
        if (force_general && !split_edges()) return true;
        if (fused_set && !split_edges()) return false;
        static const double limits[2][3][4] = {{{5e5, 1.0e6, 1.2e6, 1.2e6},     // periodic: FP64, FP32, FP32_U64, 16-bit
                                                {6e5, 1.0e6, 1.1e6, 1.8e6},     // y walls
                                                {5e5, 8.5e5, 9.0e5, 8.5e5}},    // x walls or holes
                                               {{5e5, 1.0e6, 1.2e6, 1.2e6},     // the explicit scheme
                                                {2.9e6, 1.0e6, 1.1e6, 1.8e6},
                                                {5e5, 1.0e6, 1.0e6, 1.0e6}}};
        const auto &limit = limits[scheme == LBM_SCHEME_EXPLICIT];
        const int kind = split_edges() ? 2 : bc[LBM_EDGE_YMIN] != LBM_BC_PERIODIC ? 1 : 0;
        return (double)nx * ny <= limit[kind][win_class(prec)];
    }
    void drop_plans()
    {
        for (SplitPlan &p : split) p.built = false;
        pair_for = false;
    }
    // any wall or hole
    bool walls() const { return split_edges() || bc[LBM_EDGE_YMIN] != LBM_BC_PERIODIC; }
    // x walls or holes: the fused kernel can run a share of the plate at most
    bool split_edges() const { return has_mask || bc[LBM_EDGE_XMIN] != LBM_BC_PERIODIC; }
    const unsigned char *mask_ptr() const
    {
        return has_mask ? reinterpret_cast<const unsigned char *>(ws + L.mask) : nullptr;
    }
    std::string err;

    void *fptr(int c) const { return ws + L.state.f[c]; }
    void *uptr(int c) const { return ws + L.state.u[c]; }
    // With j extrapolated a step reads j of the two states before it while it
    // writes the next: three buffers take turns.
    void *jbuf(int k) const { return k == 2 ? ws + L.scratch : ws + L.state.j[k]; }
    int jfree() const { return 3 - jslot - jback; }
    void *jptr(int c) const
    {
        return scheme == LBM_SCHEME_EXTRAP ? jbuf(c == cur ? jslot : jback) : ws + L.state.j[c];
    }
    unsigned *flag() const { return reinterpret_cast<unsigned *>(ws + L.small); }
    Units units() const { return Units{dx, rho0, lam, mu}; }

    // lattice velocity of edge e's wall (zero unless a momentum wall)
    double wall_speed(int e, int a) const
    {
        return bc[e] == LBM_BC_DIRICHLET_J && material ? bcval[e][a] / units().momentum() : 0.0;
    }
    double load_bound() const { return load_population_bound(units(), nx, ny, bc, bcval, body); }
    // 16-bit storage: lower the population scale (rescaling the stored
    // populations on the stream) when the loads now set could drive the
    // populations beyond the headroom of the current scale
    hipError_t refit_scale()
    {
        if (!fields || (prec != LBM_FP16_STORE && prec != LBM_BF16_STORE)) return hipSuccess;
        const double need = load_bound();
        if (!(need * f_scale > kScaledHeadroom)) return hipSuccess;
        const double ns = population_scale(need);
        const hipError_t e = plate_rescale(prec, fptr(cur), (size_t)nx * ny, ns / f_scale, stream);
        if (e == hipSuccess) f_scale = ns;
        return e;
    }
    // set edge e's rule and value, keeping its wall displacement continuous
    // at the current step
    void set_edge(int e, int kind, double v0, double v1)
    {
        const double n = (double)steps;
        const double now[2] = {uwb[e][0] + wall_speed(e, 0) * n, uwb[e][1] + wall_speed(e, 1) * n};
        bc[e] = kind;
        bcval[e][0] = v0;
        bcval[e][1] = v1;
        for (int a = 0; a < 2; ++a) uwb[e][a] = now[a] - wall_speed(e, a) * n;
    }

    // the page-locked buffer (its allocation costs two pageable copies); reads
    // go without where there is none
    void want_pin()
    {
        if (!pin && hipHostMalloc(reinterpret_cast<void **>(&pin), kPinBytes, hipHostMallocDefault) != hipSuccess) {
            (void)hipGetLastError();
            pin = nullptr;
        }
    }

    PlateIO io() const
    {
        PlateIO p{};
        p.nx = nx;
        p.ny = ny;
        p.prec = prec;
        p.U = units();
        p.bc_lo = bc[LBM_EDGE_YMIN];
        p.bc_hi = bc[LBM_EDGE_YMAX];
        p.bc_left = bc[LBM_EDGE_XMIN];
        p.bc_right = bc[LBM_EDGE_XMAX];
        for (int a = 0; a < 2; ++a) {
            p.val_lo[a] = bcval[LBM_EDGE_YMIN][a];
            p.val_hi[a] = bcval[LBM_EDGE_YMAX][a];
            p.val_left[a] = bcval[LBM_EDGE_XMIN][a];
            p.val_right[a] = bcval[LBM_EDGE_XMAX][a];
            p.uwb_lo[a] = uwb[LBM_EDGE_YMIN][a];
            p.uwb_hi[a] = uwb[LBM_EDGE_YMAX][a];
            p.uwb_left[a] = uwb[LBM_EDGE_XMIN][a];
            p.uwb_right[a] = uwb[LBM_EDGE_XMAX][a];
        }
        p.f = fptr(cur);
        p.u = uptr(cur);
        p.j = jptr(cur);
        p.f_other = fptr(cur ^ 1);
        p.f_scale = f_scale;
        p.staging = reinterpret_cast<double *>(ws + L.staging);
        p.staging_bytes = L.staging_bytes;
        p.partials = reinterpret_cast<double *>(ws + L.partials);
        p.diag_out = reinterpret_cast<double *>(ws + L.small + 64);
        p.mask = mask_ptr();
        p.stream = stream;
        p.pin = pin;
        p.flag = flag();
        return p;
    }
};

namespace {

thread_local std::string g_create_error;

lbm_status fail(lbm_solver *h, lbm_status s, const std::string &msg)
{
    if (h)
        h->err = msg;
    else
        g_create_error = msg;
    return s;
}

lbm_status hip_fail(lbm_solver *h, hipError_t e, const char *what)
{
    return fail(h, LBM_ERR_HIP, std::string(what) + ": " + hipGetErrorString(e));
}

#define HIP_TRY(h, call)                                     \
    do {                                                     \
        hipError_t e_ = (call);                              \
        if (e_ != hipSuccess) return hip_fail(h, e_, #call); \
    } while (0)

int resident_blocks(const lbm_solver *h, int block, int spl, int walled_form = -1)
{
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    const bool pc = h->scheme == LBM_SCHEME_PC;
    // the kernel form of the handle's y edges, unless one is asked for
    const bool walled = walled_form >= 0 ? walled_form != 0 : h->bc[LBM_EDGE_YMIN] != LBM_BC_PERIODIC;
    int per_cu = 0;
    switch (h->prec) {
    case LBM_FP64: per_cu = Kernels<PrecF64>::resident_per_cu(block, spl, pc, walled); break;
    case LBM_FP32: per_cu = Kernels<PrecF32>::resident_per_cu(block, spl, pc, walled); break;
    case LBM_FP16_STORE: per_cu = Kernels<PrecF16>::resident_per_cu(block, spl, pc, walled); break;
    case LBM_FP32_U64: per_cu = Kernels<PrecF32U64>::resident_per_cu(block, spl, pc, walled); break;
    default: per_cu = Kernels<PrecBF16>::resident_per_cu(block, spl, pc, walled); break;
    }
    return per_cu * cus;
}

// whether two steps per launch fit the LDS with this block size, for the
// handle's precision and y boundaries
bool two_step_fits(const lbm_solver *h, int block)
{
    const bool walled = h->bc[LBM_EDGE_YMIN] != LBM_BC_PERIODIC;
    switch (h->prec) {
    case LBM_FP64: return Kernels<PrecF64>::step2_ok(block, walled);
    case LBM_FP32: return Kernels<PrecF32>::step2_ok(block, walled);
    case LBM_FP16_STORE: return Kernels<PrecF16>::step2_ok(block, walled);
    case LBM_FP32_U64: return Kernels<PrecF32U64>::step2_ok(block, walled);
    default: return Kernels<PrecBF16>::step2_ok(block, walled);
    }
}

// a two-step tiling whose block no longer fits (the y edges stopped being
// periodic) runs with 256 threads
void refit_two_step(lbm_solver *h)
{
    if (h->spl == 2 && !two_step_fits(h, h->shape.block))
        h->shape = make_shape(h->nx, h->ny, h->prec, h->scheme, 256, h->shape.n_segs, 2);
}

void plan_launch(lbm_solver *h)
{
    const int halo = stencil_halo(h->prec, h->scheme, h->spl);
    // narrowest block whose strip covers the width, else 256 threads
    int block = 256;
    if (h->nx <= 64 - 2 * halo)
        block = 64;
    else if (h->nx <= 128 - 2 * halo)
        block = 128;
    const Shape probe = make_shape(h->nx, h->ny, h->prec, h->scheme, block, 1, h->spl);
    const int resident = std::max(resident_blocks(h, block, h->spl), probe.n_strips);
    // A block marches its rows one after another, so on a small plate the
    // step takes as long as the longest march: use the shortest segments (1,
    // 2, 4 or 8 rows) whose recomputed halo rows keep the launch within one
    // wave of resident blocks and about 1.5 M thread-rows (measured on 64^2
    // to 512^2 plates: 1.6-2.5 times faster than 16-row segments).
    for (int rows = 1; rows <= 8; rows *= 2) {
        const long long segs = (h->ny + rows - 1) / rows;
        const long long work = (long long)probe.n_strips * segs * (rows + 2 * halo + 1) * block;
        if (probe.n_strips * segs <= resident && work <= 1500000) {
            h->shape = make_shape(h->nx, h->ny, h->prec, h->scheme, block, (int)segs, h->spl);
            return;
        }
    }
    // otherwise as many segments as fit one wave of resident blocks (the last
    // wave of a longer grid would run part-empty), each of at least 16 rows
    int n_segs = resident / probe.n_strips;
    n_segs = std::max(1, std::min(n_segs, h->ny / 16));
    h->shape = make_shape(h->nx, h->ny, h->prec, h->scheme, block, n_segs, h->spl);
}

// Threads per block of the library's own two-step launches over `sites` sites
// of a periodic plate (or the part of a plate clear of walls): 128 (two or
// more blocks per compute unit, which cover each other's barriers) up to the
// sizes where the narrower strips' halo columns cost more; us per step with
// 128 / 256 threads: FP64 1400^2 74 / 77, 1900^2 115 / 116, 2999 x 2501 221 /
// 208; FP32 1400^2 36.0 / 38.5, 1900^2 62.6 / 60.6, 2999 x 2501 120 / 113;
// FP32_U64 1900^2 83 / 81, 2999 x 2501 146 / 139.
int pair_block(lbm_precision p, double sites) { return sites < (p == LBM_FP64 ? 5e6 : 2.5e6) ? 128 : 256; }

// Launch shape of two steps per launch on a periodic plate that the caller
// chose none for: one wave of resident blocks whatever the rows of a segment
// (one step per launch before: FP64 1400^2 115 us per step, 2999 x 2501 379;
// FP32 49, 213; FP32_U64 1900^2 121, 2999 x 2501 229).
bool plan_pairs(lbm_solver *h)
{
    if (max_steps_per_launch(h->prec, h->scheme) < 2 || h->walls()) return false;
    if (h->pair_for) return true;
    const int block = pair_block(h->prec, (double)h->nx * h->ny);
    const Shape probe = make_shape(h->nx, h->ny, h->prec, h->scheme, block, 1, 2);
    const int segs = std::max(1, std::min(resident_blocks(h, block, 2) / probe.n_strips, h->ny / 4));
    h->pair_shape = make_shape(h->nx, h->ny, h->prec, h->scheme, block, segs, 2);
    h->pair_for = true;
    return true;
}

// Sites from which a split plate's windows run beside the fused share on a
// second stream: below, forking and joining costs more than the overlap gives
// (us per step, one stream / two: with a hole FP64 4096^2 484 / 437, 2000^2
// 152 / 155; FP32_U64 271 / 267, 97 / 102; FP16 364 / 358, 122 / 132).
constexpr double kBesideSites = 1e7;

// Blocks of a plan's fused share: all that the device holds at once, but with the
// explicit scheme in the 32-bit forms two per compute unit of the five (four)
// that fit: longer segments recompute fewer halo rows (us per step, all / two:
// with a hole FP32 2500^2 182 / 167, 4096^2 389 / 366, FP32_U64 193 / 185, 425 /
// 411; four walls 4096^2 424 / 405, 469 / 454). FP64 holds two, the 16-bit forms
// three (1800^2 81, with two 84). In FP64 a plate of 4.4 to 7 million
// sites with holes runs 0.9 per compute unit, beside windows that take a last
// strip of 16 columns too (2100^2 223 / 216, 2400^2 257 / 250, 2500^2 303 / 286,
// 2600^2 318 / 311; outside, 2000^2 181 / 194, 2800^2 346 / 351).
bool lean_share(const lbm_solver *h)
{
    const double sites = (double)h->nx * h->ny;
    return h->scheme == LBM_SCHEME_EXPLICIT && h->prec == LBM_FP64 && h->has_mask && sites >= 4.4e6 && sites < 7e6;
}

int share_blocks(const lbm_solver *h, int block, int steps)
{
    const int all = resident_blocks(h, block, steps, 0);
    if (lean_share(h)) return std::min(all, (int)(0.9 * h->cus));
    const bool two = h->scheme == LBM_SCHEME_EXPLICIT && !deviation_storage(h->prec);
    return two ? std::min(all, 2 * h->cus) : all;
}

// Split of the plate between the fused kernel and windows for launches of
// `steps` steps, not used where the plate leaves the fused kernel no worthwhile
// share (or the lists no room).
hipError_t build_split(lbm_solver *h, int steps)
{
    SplitPlan &p = h->split[steps - 1];
    p = SplitPlan{};
    p.built = true;
    const int nx = h->nx, ny = h->ny;
    const SplitEdges e{nx, ny, h->bc[LBM_EDGE_XMIN] == LBM_BC_PERIODIC, h->bc[LBM_EDGE_YMIN] == LBM_BC_PERIODIC,
                       stencil_halo(h->prec, h->scheme, steps), h->prec == LBM_FP64 ? 16 : 32};
    const int reach = h->scheme == LBM_SCHEME_EXPLICIT ? win_reach<0>() : win_reach<1>();
    const bool extrap = h->scheme == LBM_SCHEME_EXTRAP;
    p.beside = h->split_edges() && ((double)nx * ny >= kBesideSites || lean_share(h));
    int mw = 0, mh = 0;
    auto windows = [&](const std::vector<Rect> &rects, int edges, WinGrid &g, int &shape) {
        const bool dev = deviation_storage(h->prec);
        shape = choose_window(h->cus, win_class(h->prec), edges, rects.data(), (int)rects.size(), reach, dev, steps, steps).shape;
        const int hh = steps * reach + (dev ? 1 : 0);
        mw = win_out(kWinShapes[shape].w, hh);
        mh = win_out(kWinShapes[shape].h, hh);
        g.nsteps = steps;
    };
    const int rest = h->general() ? WIN_GENERAL : WIN_YWALLS;
    if (!h->has_mask) {
        const Rect box = split_box(e);
        if (box.w < kSplitMinCols || box.h < kSplitMinRows) return hipSuccess;
        const int block = steps == 2 ? pair_block(h->prec, (double)box.w * box.h) : 256;
        p.shape = make_shape(nx, ny, h->prec, h->scheme, block, 1, steps);
        p.box = box;
        p.shape.n_strips = (box.w + p.shape.strip_w - 1) / p.shape.strip_w;
        p.shape.n_segs = std::max(1, std::min(share_blocks(h, block, steps) / p.shape.n_strips, box.h / 8));
        auto regions = [&](const std::vector<Rect> &rects, WinGrid &g) {
            for (const Rect &r : rects) {
                g.reg[g.n_regions] = win_region(r, mw, mh, g.nb);
                g.nb += win_blocks(g.reg[g.n_regions++]);
            }
        };
        const std::vector<Rect> rects = split_frame(e, box);
        windows(rects, rest, p.win, p.win_shape);
        regions(rects, p.win);
        if (extrap) {
            windows({box}, WIN_PERIODIC, p.inner, p.inner_shape);
            regions({box}, p.inner);
        }
        p.use = true;
        return hipSuccess;
    }
    p.shape = make_shape(nx, ny, h->prec, h->scheme, 256, 1, steps);
    std::vector<int4> list;
    std::vector<Rect> rects;
    split_mask(e, h->mask_host.data(), extrap ? nx : p.shape.strip_w, lean_share(h) ? 32 : 0,
               extrap ? 1 : share_blocks(h, 256, steps), list, rects);
    if (list.empty()) return hipSuccess;
    if (extrap) {
        std::vector<Rect> clear;
        for (const int4 &t : list) clear.push_back(Rect{t.x, t.z, t.y, t.w - t.z});
        list.clear();
        windows(clear, WIN_PERIODIC, p.inner, p.inner_shape);
        split_windows(nx, h->mask_host.data(), clear, mw, mh, list);
        p.inner.nb = (int)list.size();
    }
    p.n_fused = (int)list.size();
    windows(rects, rest, p.win, p.win_shape);
    split_windows(nx, h->mask_host.data(), rects, mw, mh, list);
    if (list.size() > list_capacity(nx, ny)) return hipSuccess;
    p.win.nb = (int)list.size() - p.n_fused;
    hipError_t err = hipMemcpyAsync(h->ws + h->L.list[steps - 1], list.data(), sizeof(int4) * list.size(),
                                    hipMemcpyHostToDevice, h->stream);
    if (!err) err = hipStreamSynchronize(h->stream);
    if (err) {
        p.built = false;
        return err;
    }
    p.fused_list = reinterpret_cast<const int4 *>(h->ws + h->L.list[steps - 1]);
    p.win.list = p.fused_list + p.n_fused;
    if (extrap) p.inner.list = p.fused_list;
    p.use = true;
    return hipSuccess;
}

hipError_t plan_split(lbm_solver *h, int steps)
{
    if (h->split[steps - 1].built) return hipSuccess;
    try {
        return build_split(h, steps);
    } catch (const std::bad_alloc &) {  // (no exception may leave a C entry)
        h->split[steps - 1] = SplitPlan{};
        return hipErrorOutOfMemory;
    }
}

}  // namespace

extern "C" {

size_t lbm_workspace_bytes(int nx, int ny, lbm_precision p)
{
    if (nx < 5 || ny < 5 || !valid_precision(p)) return 0;
    return make_layout(nx, ny, p).total;
}

size_t lbm_workspace_bytes_walled(int nx, int ny, lbm_precision p)
{
    if (nx < 5 || ny < 5 || !valid_precision(p)) return 0;
    return make_layout(nx, ny, p).total_walled;
}

lbm_status lbm_create(int nx, int ny, double dx, lbm_precision p, lbm_scheme s, void *dev_workspace,
                      size_t ws_bytes, void *hip_stream, lbm_solver **out)
{
    if (!out) return fail(nullptr, LBM_ERR_ARG, "out is NULL");
    *out = nullptr;
    if (nx < 5 || ny < 5) return fail(nullptr, LBM_ERR_ARG, "nx and ny must be >= 5");
    if (!(dx > 0.0) || !std::isfinite(dx)) return fail(nullptr, LBM_ERR_ARG, "dx must be positive");
    if (!valid_precision(p)) return fail(nullptr, LBM_ERR_ARG, "unknown precision");
    if (s != LBM_SCHEME_PC && s != LBM_SCHEME_EXPLICIT && s != LBM_SCHEME_EXTRAP)
        return fail(nullptr, LBM_ERR_ARG, "unknown scheme");
    if (!dev_workspace) return fail(nullptr, LBM_ERR_ARG, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(dev_workspace) % kAlign)
        return fail(nullptr, LBM_ERR_ARG, "workspace not 256-byte aligned");
    if ((long long)nx * ny > (1LL << 29)) return fail(nullptr, LBM_ERR_UNSUPPORTED, "more than 2^29 sites");
    const Layout L = make_layout(nx, ny, p);
    if (ws_bytes < L.total) return fail(nullptr, LBM_ERR_NOMEM, "workspace smaller than lbm_workspace_bytes()");
    if (s == LBM_SCHEME_EXTRAP && ws_bytes < L.total_walled)
        return fail(nullptr, LBM_ERR_NOMEM, "the extrapolation scheme needs lbm_workspace_bytes_walled() bytes");
    lbm_solver *h = new (std::nothrow) lbm_solver();
    if (!h) return fail(nullptr, LBM_ERR_NOMEM, "host allocation failed");
    h->nx = nx;
    h->ny = ny;
    h->dx = dx;
    h->prec = p;
    h->scheme = s;
    h->ws = static_cast<char *>(dev_workspace);
    h->ws_bytes = ws_bytes;
    h->stream = static_cast<hipStream_t>(hip_stream);
    h->L = L;
    if (hipGetDevice(&h->device) != hipSuccess) h->device = 0;
    if (hipDeviceGetAttribute(&h->cus, hipDeviceAttributeMultiprocessorCount, h->device) != hipSuccess || h->cus < 1)
        h->cus = 256;
    plan_launch(h);
    h->created_shape = h->shape;
    *out = h;
    return LBM_OK;
}

lbm_status lbm_set_material(lbm_solver *h, double rho0, double lambda, double mu, double tau_over_dt)
{
    if (!h) return LBM_ERR_ARG;
    if (!(rho0 > 0) || !std::isfinite(rho0)) return fail(h, LBM_ERR_ARG, "rho0 must be positive");
    if (!(mu > 0) || !std::isfinite(mu)) return fail(h, LBM_ERR_ARG, "mu must be positive");
    if (!(lambda + mu > 0) || !std::isfinite(lambda)) return fail(h, LBM_ERR_ARG, "lambda + mu must be positive");
    if (!(tau_over_dt > 0.5) || !std::isfinite(tau_over_dt)) return fail(h, LBM_ERR_ARG, "tau/dt must exceed 1/2");
    if (h->fields) return fail(h, LBM_ERR_STATE, "set the material before the fields");
    h->rho0 = rho0;
    h->lam = lambda;
    h->mu = mu;
    h->tau = tau_over_dt;
    h->material = true;
    return LBM_OK;
}

lbm_status lbm_set_body_force(lbm_solver *h, const double b[2])
{
    if (!h) return LBM_ERR_ARG;
    if (!b) return fail(h, LBM_ERR_ARG, "NULL argument");
    if (!std::isfinite(b[0]) || !std::isfinite(b[1])) return fail(h, LBM_ERR_ARG, "body force not finite");
    h->body[0] = b[0];
    h->body[1] = b[1];
    HIP_TRY(h, h->refit_scale());
    return LBM_OK;
}

lbm_status lbm_set_boundary(lbm_solver *h, lbm_edge e, lbm_bc bc, const double value[2])
{
    if (!h) return LBM_ERR_ARG;
    if (e < LBM_EDGE_XMIN || e > LBM_EDGE_YMAX) return fail(h, LBM_ERR_ARG, "unknown edge");
    if (bc < LBM_BC_PERIODIC || bc > LBM_BC_NEUMANN_T) return fail(h, LBM_ERR_ARG, "unknown boundary rule");
    if ((e == LBM_EDGE_XMIN || e == LBM_EDGE_XMAX) && bc != LBM_BC_PERIODIC && h->ws_bytes < h->L.total_walled)
        return fail(h, LBM_ERR_NOMEM, "walls on the x edges need a workspace of lbm_workspace_bytes_walled() bytes");
    if (bc != LBM_BC_PERIODIC && (!value || !std::isfinite(value[0]) || !std::isfinite(value[1])))
        return fail(h, LBM_ERR_ARG, "boundary value missing or not finite");
    const int other = e == LBM_EDGE_YMIN ? LBM_EDGE_YMAX
                      : e == LBM_EDGE_YMAX ? LBM_EDGE_YMIN
                      : e == LBM_EDGE_XMIN ? LBM_EDGE_XMAX
                                           : LBM_EDGE_XMIN;
    if (h->has_mask && (h->bc[e] == LBM_BC_PERIODIC) != (bc == LBM_BC_PERIODIC))
        return fail(h, LBM_ERR_STATE, "a mask was checked against the edges: make edges periodic or not before it");
    if (bc == LBM_BC_PERIODIC && h->bc[other] != LBM_BC_PERIODIC) {
        // periodic edges come in pairs
        h->set_edge(other, LBM_BC_PERIODIC, 0.0, 0.0);
    }
    if (bc != LBM_BC_PERIODIC && h->bc[other] == LBM_BC_PERIODIC) {
        // the opposite edge stops being periodic: it becomes a wall at rest until set
        h->set_edge(other, LBM_BC_DIRICHLET_J, 0.0, 0.0);
    }
    if ((h->bc[e] == LBM_BC_PERIODIC) != (bc == LBM_BC_PERIODIC)) h->drop_plans();
    h->set_edge(e, bc, bc == LBM_BC_PERIODIC ? 0.0 : value[0], bc == LBM_BC_PERIODIC ? 0.0 : value[1]);
    refit_two_step(h);
    HIP_TRY(h, h->refit_scale());
    return LBM_OK;
}

lbm_status lbm_set_tiling(lbm_solver *h, int block, int n_segs)
{
    if (!h) return LBM_ERR_ARG;
    if (block != 64 && block != 128 && block != 256 && block != 512)
        return fail(h, LBM_ERR_ARG, "block must be 64, 128, 256 or 512");
    if (n_segs < 1 || n_segs > h->ny) return fail(h, LBM_ERR_ARG, "n_segs must be in [1, ny]");
    if ((long long)h->nx * n_segs > (1LL << 30)) return fail(h, LBM_ERR_ARG, "too many blocks");
    if (h->spl == 2 && !two_step_fits(h, block))
        return fail(h, LBM_ERR_UNSUPPORTED, "two steps per launch with this block size exceed the LDS");
    h->shape = make_shape(h->nx, h->ny, h->prec, h->scheme, block, n_segs, h->spl);
    h->fused_set = true;
    return LBM_OK;
}

lbm_status lbm_set_steps_per_launch(lbm_solver *h, int k)
{
    if (!h) return LBM_ERR_ARG;
    if (k != 1 && k != 2) return fail(h, LBM_ERR_ARG, "steps per launch must be 1 or 2");
    if (k == 2 && h->scheme != LBM_SCHEME_PC)
        return fail(h, LBM_ERR_UNSUPPORTED, "two steps per launch need the predictor-corrector scheme");
    if (k == 2 && max_steps_per_launch(h->prec, h->scheme) < 2)
        return fail(h, LBM_ERR_UNSUPPORTED, "16-bit population storage runs one step per launch");
    h->spl = k;
    h->fused_set = true;
    const int block = k == 2 && !two_step_fits(h, h->shape.block) ? 256 : h->shape.block;
    h->shape = make_shape(h->nx, h->ny, h->prec, h->scheme, block, h->shape.n_segs, k);
    return LBM_OK;
}

lbm_status lbm_resident_blocks(const lbm_solver *h, int block, int steps_per_launch, int *blocks)
{
    if (!h || !blocks) return LBM_ERR_ARG;
    *blocks = 0;
    if (block != 64 && block != 128 && block != 256 && block != 512) return LBM_OK;
    if (steps_per_launch != 1 && steps_per_launch != 2) return LBM_OK;
    if (steps_per_launch == 2 && h->scheme != LBM_SCHEME_PC) return LBM_OK;
    *blocks = resident_blocks(h, block, steps_per_launch);
    return LBM_OK;
}

lbm_status lbm_set_mask(lbm_solver *h, const unsigned char *solid)
{
    if (!h) return LBM_ERR_ARG;
    if (h->fields) return fail(h, LBM_ERR_STATE, "set the mask before the fields");
    if (!solid) {
        h->has_mask = false;
        h->mask_host.clear();
        h->drop_plans();
        return LBM_OK;
    }
    if (h->ws_bytes < h->L.total_walled)
        return fail(h, LBM_ERR_NOMEM, "holes need a workspace of lbm_workspace_bytes_walled() bytes");
    const int nx = h->nx, ny = h->ny;
    const bool perx = h->bc[LBM_EDGE_XMIN] == LBM_BC_PERIODIC, pery = h->bc[LBM_EDGE_YMIN] == LBM_BC_PERIODIC;
    auto hole = [&](int x, int y) {
        if (y < 0 || y >= ny) {
            if (!pery) return false;
            y = (y % ny + ny) % ny;
        }
        if (x < 0 || x >= nx) {
            if (!perx) return false;
            x = (x % nx + nx) % nx;
        }
        return solid[(size_t)y * nx + x] == 0;
    };
    bool any_material = false;
    for (int y = 0; y < ny; ++y)
        for (int x = 0; x < nx; ++x) {
            if (hole(x, y)) {
                if (((y == 0 || y == ny - 1) && !pery) || ((x == 0 || x == nx - 1) && !perx))
                    return fail(h, LBM_ERR_ARG, "a hole touches a wall edge");
                continue;
            }
            any_material = true;
            if ((hole(x - 1, y) && hole(x + 1, y)) || (hole(x, y - 1) && hole(x, y + 1)))
                return fail(h, LBM_ERR_ARG, "material one node thick between holes");
        }
    if (!any_material) return fail(h, LBM_ERR_ARG, "no material node");
    std::vector<unsigned char> dev(solid, solid + (size_t)nx * ny);
    for (auto &m : dev) m = m ? 1 : 0;
    HIP_TRY(h, hipMemcpyAsync(h->ws + h->L.mask, dev.data(), (size_t)nx * ny, hipMemcpyHostToDevice, h->stream));
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    h->mask_host.swap(dev);
    h->has_mask = true;
    h->drop_plans();
    return LBM_OK;
}

lbm_status lbm_set_general_path(lbm_solver *h, int on)
{
    if (!h) return LBM_ERR_ARG;
    // (holes, x walls and the extrapolation scheme already hold the walled
    // workspace; the general step of any other plate needs no more)
    h->force_general = on != 0;
    h->fused_set = !on;
    return LBM_OK;
}

lbm_status lbm_set_default_plan(lbm_solver *h)
{
    if (!h) return LBM_ERR_ARG;
    h->force_general = false;
    h->fused_set = false;
    h->spl = 1;
    h->shape = h->created_shape;
    return LBM_OK;
}

lbm_status lbm_get_edges(const lbm_solver *h, int kinds[4], int *has_mask)
{
    if (!h || !kinds || !has_mask) return LBM_ERR_ARG;
    for (int e = 0; e < 4; ++e) kinds[e] = h->bc[e];
    *has_mask = h->has_mask;
    return LBM_OK;
}

lbm_status lbm_set_rounding(lbm_solver *h, lbm_rounding r, uint64_t seed)
{
    if (!h) return LBM_ERR_ARG;
    if (r != LBM_ROUND_NEAREST && r != LBM_ROUND_STOCHASTIC) return fail(h, LBM_ERR_ARG, "unknown rounding");
    if (r == LBM_ROUND_STOCHASTIC && h->prec != LBM_FP16_STORE && h->prec != LBM_BF16_STORE)
        return fail(h, LBM_ERR_UNSUPPORTED, "stochastic rounding needs 16-bit population storage");
    h->sr = r == LBM_ROUND_STOCHASTIC;
    h->seed = seed;
    return LBM_OK;
}

lbm_status lbm_get_steps_per_launch(const lbm_solver *h, int *k)
{
    if (!h || !k) return LBM_ERR_ARG;
    *k = h->spl;
    return LBM_OK;
}

lbm_status lbm_get_tiling(const lbm_solver *h, int *block, int *n_segs)
{
    if (!h || !block || !n_segs) return LBM_ERR_ARG;
    *block = h->shape.block;
    *n_segs = h->shape.n_segs;
    return LBM_OK;
}

lbm_status lbm_get_dt(const lbm_solver *h, double *dt)
{
    if (!h || !dt) return LBM_ERR_ARG;
    if (!h->material) return LBM_ERR_STATE;
    *dt = h->units().dt();
    return LBM_OK;
}

lbm_status lbm_set_fields(lbm_solver *h, const double *u0, const double *v0)
{
    if (!h) return LBM_ERR_ARG;
    if (!u0 || !v0) return fail(h, LBM_ERR_ARG, "u0 or v0 is NULL");
    if (!h->material) return fail(h, LBM_ERR_STATE, "set the material before the fields");
    h->cur = h->home;
    h->jslot = h->jhome;
    h->jback = h->jhome_back;
    for (auto &w : h->uwb) w[0] = w[1] = 0.0;  // every wall starts undisplaced
    double scale = 1.0;
    bool nonfinite = false;
    const hipError_t e = plate_start(h->io(), u0, v0, h->load_bound(), &scale, &nonfinite);
    if (e != hipSuccess) return hip_fail(h, e, "start-up");
    if (nonfinite) return fail(h, LBM_ERR_ARG, "initial fields not finite");
    h->f_scale = scale;
    if (h->scheme == LBM_SCHEME_EXTRAP)  // j one step back: j(0) before the first step
        HIP_TRY(h, hipMemcpyAsync(h->jbuf(h->jback), h->jbuf(h->jslot), 2 * (size_t)h->nx * h->ny * elem_sizes(h->prec).j,
                                  hipMemcpyDeviceToDevice, h->stream));
    HIP_TRY(h, hipMemsetAsync(h->flag(), 0, sizeof(unsigned), h->stream));
    HIP_TRY(h, hipStreamSynchronize(h->stream));
    h->steps = 0;
    h->fields = true;
    return LBM_OK;
}

lbm_status lbm_step(lbm_solver *h, int64_t nsteps)
{
    if (!h) return LBM_ERR_ARG;
    if (nsteps < 0) return fail(h, LBM_ERR_ARG, "nsteps < 0");
    if (!h->fields) return fail(h, LBM_ERR_STATE, "set the fields before stepping");
    StepParams sp{};
    sp.nx = h->nx;
    sp.ny = h->ny;
    sp.plane = (long long)h->nx * h->ny;
    fill_physics(sp, h->units(), h->tau, h->body, h->bc[LBM_EDGE_YMIN], h->bcval[LBM_EDGE_YMIN],
                 h->bc[LBM_EDGE_YMAX], h->bcval[LBM_EDGE_YMAX]);
    for (int a = 0; a < 2; ++a) {
        sp.uwb_lo[a] = h->uwb[LBM_EDGE_YMIN][a];
        sp.uwb_hi[a] = h->uwb[LBM_EDGE_YMAX][a];
    }
    sp.f_scale = h->f_scale;
    sp.f_inv_scale = 1.0 / h->f_scale;
    sp.strip_w = h->shape.strip_w;
    sp.halo_a = h->shape.halo_a;
    sp.n_strips = h->shape.n_strips;
    sp.n_segs = h->shape.n_segs;
    sp.flag = h->flag();
    sp.sr = h->sr;
    sp.seed = h->seed;
    const int nblocks = h->shape.n_strips * h->shape.n_segs;
    const bool pc = h->scheme == LBM_SCHEME_PC;
    // A captured call, and from the first one on every call of the handle,
    // leaves the state in the buffers that one launch per step leaves it in, so
    // that a graph of an even number of steps can be replayed with even eager
    // calls and restarts between: an even number of two-step launches, and two
    // buffers of j with a copy of the older one (the rotation of three comes
    // round after six steps).
    hipStreamCaptureStatus capture = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(h->stream, &capture) != hipSuccess) (void)hipGetLastError();
    const bool captured = capture == hipStreamCaptureStatusActive;
    if (captured && !h->fixed) {
        const bool odd = h->steps & 1;
        h->fixed = true;
        h->home = odd ? h->cur ^ 1 : h->cur;
        h->jhome = odd ? h->jback : h->jslot;
        h->jhome_back = odd ? h->jslot : h->jback;
    }
    const int64_t paired = h->fixed ? nsteps / 4 * 4 : nsteps / 2 * 2;  // steps that two-step launches may take
    auto advance = [&](auto &p) {  // state pointers and index of the next launch
        p.f_in = h->fptr(h->cur);
        p.u_in = h->uptr(h->cur);
        p.j_in = h->jptr(h->cur);
        p.f_out = h->fptr(h->cur ^ 1);
        p.u_out = h->uptr(h->cur ^ 1);
        p.j_out = h->jptr(h->cur ^ 1);
        p.step = h->steps;
    };
    auto done = [&](int n) {
        h->cur ^= 1;
        const int next = h->fixed ? h->jback : h->jfree();
        h->jback = h->jslot;
        h->jslot = next;
        h->steps += n;
    };
    const bool whole_windows = h->windows();
    const bool split = !whole_windows && h->walls() && (h->split_edges() || h->scheme == LBM_SCHEME_EXTRAP || !h->fused_set);
    int64_t k = 0;
    if (whole_windows || split) {
        GenParams gp{};
        gp.nx = h->nx;
        gp.ny = h->ny;
        gp.plane = sp.plane;
        gp.omega = sp.omega;
        gp.lam = sp.lam;
        gp.mu = sp.mu;
        gp.bx = sp.bx;
        gp.by = sp.by;
        const Units U = h->units();
        // windows of a plate that the fused kernel can run keep its arithmetic
        const int edges = h->general() ? (h->walls() ? WIN_GENERAL : WIN_PERIODIC)
                                       : (h->walls() ? WIN_YWALLS : WIN_PERIODIC);
        for (int e = 0; e < 4; ++e) {
            gp.bc[e] = h->bc[e];
            for (int a = 0; a < 2; ++a) {  // j* -> lattice momentum, T* -> lattice stress (each path's own rounding)
                gp.val[e][a] = h->bc[e] == LBM_BC_DIRICHLET_J ? h->bcval[e][a] / U.momentum()
                               : edges == WIN_GENERAL         ? h->bcval[e][a] / U.stress()
                                                              : h->bcval[e][a] * (1.0 / U.stress());
                gp.uwb[e][a] = h->uwb[e][a];
            }
        }
        gp.f_scale = sp.f_scale;
        gp.f_inv_scale = sp.f_inv_scale;
        gp.sr = sp.sr;
        gp.seed = sp.seed;
        gp.pc = h->scheme == LBM_SCHEME_EXTRAP ? 2 : (pc ? 1 : 0);
        gp.flag = sp.flag;
        gp.mask = h->mask_ptr();
        auto windows = [&](const WinGrid &g, int shape, int form, hipStream_t st) {
            return LBM_DISPATCH(h->prec, window_step<PR>(gp, g, form, shape, st));
        };
        auto next = [&]() -> hipError_t {
            advance(gp);
            if (gp.pc != 2) return hipSuccess;
            gp.j_prev = gp.j_out;  // j of the step before, and the third buffer
            void *const third = h->jbuf(h->jfree());
            if (!h->fixed) {
                gp.j_out = third;
                return hipSuccess;
            }
            gp.j_prev = third;
            return hipMemcpyAsync(third, gp.j_out, 2 * (size_t)h->nx * h->ny * elem_sizes(h->prec).j,
                                  hipMemcpyDeviceToDevice, h->stream);
        };
        if (split) {
            // The fused kernel's periodic form over the part of the plate
            // clear of walls and holes, windows over the rest: both read the
            // state of step n and write disjoint sites of the new one.
            for (int n = max_steps_per_launch(h->prec, h->scheme); n >= 1; --n) {
                const int64_t end = n == 2 ? paired : nsteps;
                if (end - k < n) continue;
                // y walls alone, one step: the fused kernel's walled form (below)
                if (n == 1 && !h->split_edges() && gp.pc != 2) continue;
                // the upload of a mask's lists waits for the stream
                if (captured && h->has_mask && !h->split[n - 1].built) continue;
                HIP_TRY(h, plan_split(h, n));
                const SplitPlan &p = h->split[n - 1];
                if (!p.use) continue;
                StepParams fp = sp;
                fp.bc_lo = fp.bc_hi = BC_PERIODIC;
                fp.strip_w = p.shape.strip_w;
                fp.halo_a = p.shape.halo_a;
                fp.n_strips = p.shape.n_strips;
                fp.n_segs = p.shape.n_segs;
                fp.x_lo = p.box.x;
                fp.x_end = p.box.x + p.box.w;
                fp.y_lo = p.box.y;
                fp.y_end = p.box.y + p.box.h;
                const int nb = p.shape.n_strips * p.shape.n_segs;
                const bool beside = p.beside;
                if (beside && !h->aux) {
                    HIP_TRY(h, hipStreamCreateWithFlags(&h->aux, hipStreamNonBlocking));
                    HIP_TRY(h, hipEventCreateWithFlags(&h->fork, hipEventDisableTiming));
                    HIP_TRY(h, hipEventCreateWithFlags(&h->join, hipEventDisableTiming));
                }
                for (; k + n <= end; k += n) {
                    advance(fp);
                    HIP_TRY(h, next());
                    if (beside) {
                        HIP_TRY(h, hipEventRecord(h->fork, h->stream));
                        HIP_TRY(h, hipStreamWaitEvent(h->aux, h->fork, 0));
                    }
                    if (p.inner.nb > 0)
                        HIP_TRY(h, windows(p.inner, p.inner_shape, WIN_PERIODIC, h->stream));
                    else if (p.fused_list)
                        HIP_TRY(h, n == 2 ? LBM_DISPATCH(h->prec, Kernels<PR>::step2_list(fp, p.fused_list, p.n_fused, h->stream))
                                          : LBM_DISPATCH(h->prec, Kernels<PR>::step_list(fp, p.fused_list, p.n_fused, pc, h->stream)));
                    else
                        HIP_TRY(h, n == 2 ? LBM_DISPATCH(h->prec, Kernels<PR>::step2(fp, p.shape.block, nb, h->stream))
                                          : LBM_DISPATCH(h->prec, Kernels<PR>::step(fp, p.shape.block, nb, pc, h->stream)));
                    HIP_TRY(h, windows(p.win, p.win_shape, edges, beside ? h->aux : h->stream));
                    if (beside) {
                        HIP_TRY(h, hipEventRecord(h->join, h->aux));
                        HIP_TRY(h, hipStreamWaitEvent(h->stream, h->join, 0));
                    }
                    done(n);
                }
            }
        }
        if (whole_windows || h->split_edges() || gp.pc == 2) {
            const Rect plate{0, 0, h->nx, h->ny};
            const int reach = gp.pc ? win_reach<1>() : win_reach<0>();
            const bool dev = deviation_storage(h->prec);
            while (k < nsteps) {
                const WinChoice c = choose_window(h->cus, win_class(h->prec), edges, &plate, 1, reach, dev, 1,
                                                  paired - k >= 2 && gp.pc != 2 ? kWinMaxSteps : 1);
                const int hh = c.steps * reach + (dev ? 1 : 0);
                WinGrid g{};
                g.nsteps = c.steps;
                g.n_regions = 1;
                g.reg[0] = win_region(plate, win_out(kWinShapes[c.shape].w, hh), win_out(kWinShapes[c.shape].h, hh), 0);
                g.nb = win_blocks(g.reg[0]);
                const int64_t end = c.steps > 1 ? paired : nsteps;
                for (; k + c.steps <= end; k += c.steps) {
                    HIP_TRY(h, next());
                    HIP_TRY(h, windows(g, c.shape, edges, h->stream));
                    done(c.steps);
                }
            }
            return LBM_OK;
        }
    }
    const bool pairs = !h->fused_set && nsteps >= 2 && plan_pairs(h);
    if (h->spl == 2 || pairs) {
        StepParams sp2 = sp;
        const Shape &shape = pairs ? h->pair_shape : h->shape;
        sp2.strip_w = shape.strip_w;
        sp2.halo_a = shape.halo_a;
        sp2.n_strips = shape.n_strips;
        sp2.n_segs = shape.n_segs;
        const int nb2 = shape.n_strips * shape.n_segs;
        for (; k + 2 <= paired; k += 2) {
            advance(sp2);
            HIP_TRY(h, LBM_DISPATCH(h->prec, Kernels<PR>::step2(sp2, shape.block, nb2, h->stream)));
            done(2);
        }
    }
    for (; k < nsteps; ++k) {
        advance(sp);
        HIP_TRY(h, LBM_DISPATCH(h->prec, Kernels<PR>::step(sp, h->shape.block, nblocks, pc, h->stream)));
        done(1);
    }
    return LBM_OK;
}

lbm_status lbm_read_fields(lbm_solver *h, double *u, double *v, double *P, lbm_diagnostics *d)
{
    if (!h) return LBM_ERR_ARG;
    if (!h->fields) return fail(h, LBM_ERR_STATE, "no fields set");
    double out[7] = {0, 0, 0, 0, 0, 0, 0};
    if (h->reads++ > 0) h->want_pin();
    bool flagged = false;
    const hipError_t e = plate_read(h->io(), (double)h->steps, u, v, P, d ? out : nullptr, &flagged);
    if (e != hipSuccess) return hip_fail(h, e, "read-out");
    unsigned flag = 0;
    if (flagged) {
        flag = *reinterpret_cast<const unsigned *>(h->pin);
    } else {
        HIP_TRY(h, hipMemcpyAsync(&flag, h->flag(), sizeof(unsigned), hipMemcpyDeviceToHost, h->stream));
        HIP_TRY(h, hipStreamSynchronize(h->stream));
    }
    if (d) {
        d->momentum[0] = out[0];
        d->momentum[1] = out[1];
        d->mass_moment = out[2];
        d->energy = out[3];
        d->min_J = out[4];
        d->max_strain = out[5];
        d->unstable = (out[6] != 0.0 || flag != 0) ? 1 : 0;
        d->reserved = 0;
        d->steps = h->steps;
    }
    if (flag != 0) return fail(h, LBM_ERR_UNSTABLE, "J <= 0 or a non-finite value appeared");
    return LBM_OK;
}

namespace {

// Device address of `scratch` on each device, looked up once per device with
// that device current (the array's name is a host-side stand-in, not the
// device address).
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
double *g_scratch_ptr[kMaxDevices] = {};

hipError_t device_scratch(int dev, double **out)
{
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (!g_scratch_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        g_scratch_ptr[dev] = static_cast<double *>(p);
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}

}  // namespace

lbm_status lbm_read_diagnostics_noalloc(lbm_solver *h, lbm_diagnostics *d)
{
    if (!h) return LBM_ERR_ARG;
    if (!d) return fail(h, LBM_ERR_ARG, "d is NULL");
    if (!h->fields) return fail(h, LBM_ERR_STATE, "no fields set");
    // the diagnostics grid is capped at kMaxDiagBlocks blocks
    const size_t n = (size_t)h->nx * h->ny;
    const size_t nblocks = std::min<size_t>(kMaxDiagBlocks, (n + 255) / 256);
    if (nblocks * 8 + 8 > kNoAllocDiagDoubles)
        return fail(h, LBM_ERR_UNSUPPORTED, "diagnostics need more scratch than the static array holds");
    int cur = 0;
    HIP_TRY(h, hipGetDevice(&cur));
    if (cur != h->device) HIP_TRY(h, hipSetDevice(h->device));
    double *sp = nullptr;
    hipError_t e = device_scratch(h->device, &sp);
    double out[7] = {0, 0, 0, 0, 0, 0, 0};
    unsigned flag = 0;
    if (e == hipSuccess) {
        PlateIO io = h->io();
        io.partials = sp;
        io.diag_out = sp + (size_t)kMaxDiagBlocks * 8;
        e = plate_read(io, (double)h->steps, nullptr, nullptr, nullptr, out);
    }
    if (e == hipSuccess) e = hipMemcpyAsync(&flag, h->flag(), sizeof(unsigned), hipMemcpyDeviceToHost, h->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(h->stream);
    if (cur != h->device) {
        const hipError_t e2 = hipSetDevice(cur);
        if (e == hipSuccess) e = e2;
    }
    if (e != hipSuccess) return hip_fail(h, e, "diagnostics");
    d->momentum[0] = out[0];
    d->momentum[1] = out[1];
    d->mass_moment = out[2];
    d->energy = out[3];
    d->min_J = out[4];
    d->max_strain = out[5];
    d->unstable = (out[6] != 0.0 || flag != 0) ? 1 : 0;
    d->reserved = 0;
    d->steps = h->steps;
    if (flag != 0) return fail(h, LBM_ERR_UNSTABLE, "J <= 0 or a non-finite value appeared");
    return LBM_OK;
}

lbm_status lbm_read_derived(lbm_solver *h, double *sigma, double *E, double *W)
{
    if (!h) return LBM_ERR_ARG;
    if (!h->fields) return fail(h, LBM_ERR_STATE, "no fields set");
    const hipError_t e = plate_read_derived(h->io(), (double)h->steps, sigma, E, W);
    if (e != hipSuccess) return hip_fail(h, e, "read-out");
    return LBM_OK;
}

lbm_status lbm_sample(lbm_solver *h, int n, const int *x, const int *y, double *out)
{
    if (!h) return LBM_ERR_ARG;
    if (!h->fields) return fail(h, LBM_ERR_STATE, "no fields set");
    if (n < 0 || (n > 0 && (!x || !y || !out))) return fail(h, LBM_ERR_ARG, "invalid node list");
    if (n > sample_capacity(h->io())) return fail(h, LBM_ERR_ARG, "too many nodes for one call");
    for (int k = 0; k < n; ++k)
        if (x[k] < 0 || x[k] >= h->nx || y[k] < 0 || y[k] >= h->ny) return fail(h, LBM_ERR_ARG, "node outside the plate");
    h->want_pin();
    const hipError_t e = plate_sample(h->io(), (double)h->steps, n, x, y, out);
    if (e != hipSuccess) return hip_fail(h, e, "sample");
    return LBM_OK;
}

lbm_status lbm_sample_series(lbm_solver *h, int n, const int *x, const int *y, int64_t nsteps, int64_t every, double *out)
{
    if (!h) return LBM_ERR_ARG;
    if (every < 1 && nsteps > 0) return fail(h, LBM_ERR_ARG, "every < 1");
    lbm_status st = lbm_sample(h, n, x, y, out);  // (checks the nodes)
    if (st != LBM_OK) return st;
    // samples after the first (every may be as large as an int64_t)
    const int64_t m = nsteps > 0 ? nsteps / every + (nsteps % every != 0) : 0;
    const size_t vb = (size_t)17 * n * sizeof(double), ib = align_up((size_t)n * sizeof(int));
    // samples that the page-locked buffer holds at once (the nodes stand in
    // it since the call above)
    const size_t room = h->pin && n > 0 && kPinHead + ib + vb <= kPinBytes ? (kPinBytes - kPinHead - ib) / vb : 0;
    int64_t got = 0;
    while (got < m) {
        const int64_t batch = room ? std::min<int64_t>(m - got, (int64_t)room) : 1;
        double *vals = room ? reinterpret_cast<double *>(h->pin + kPinHead + ib) : nullptr;
        for (int64_t q = 0; q < batch; ++q) {
            if ((st = lbm_step(h, std::min(every, nsteps - (got + q) * every))) != LBM_OK) {
                (void)hipStreamSynchronize(h->stream);  // samples may be on their way to the buffer
                return st;
            }
            if (room)
                HIP_TRY(h, enqueue_sample(h->io(), (double)h->steps, n, reinterpret_cast<const int *>(h->pin + kPinHead),
                                          vals + q * 17 * (size_t)n));
        }
        double *to = out + (size_t)(got + 1) * 17 * n;
        if (room) {
            HIP_TRY(h, hipStreamSynchronize(h->stream));
            std::copy(vals, vals + batch * 17 * (size_t)n, to);
        } else if ((st = lbm_sample(h, n, x, y, to)) != LBM_OK) {
            return st;
        }
        got += batch;
    }
    return LBM_OK;
}

void lbm_destroy(lbm_solver *h) { delete h; }

const char *lbm_last_error(const lbm_solver *h) { return h ? h->err.c_str() : g_create_error.c_str(); }

}  // extern "C"
