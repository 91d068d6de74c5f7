// Host runtime behind the C ABI in ce.h: parameter validation, device memory
// layout (library-owned or carved from a caller arena), loading with FP64 ->
// storage conversion, the start-up half step, step launches (plain or as
// captured step-block graphs), diagnostics and readback.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <new>

#include "ce_sim.hpp"

using namespace ce;
using namespace ce::host;

namespace {
thread_local char g_err[512] = "";

// Memory kept from destroyed simulations, oldest first (see device_memory).
struct Kept {
    void *mem;
    size_t bytes;
    int device;
};
std::mutex g_kept_mu;
Kept g_kept[kKeptBlocks];
int g_kept_n = 0;
size_t g_kept_bytes = 0;

// Threads inside the library, and the lock of a thread that has to be alone:
// one that enters counts itself first and then waits for the lock, so a
// holder of it that finds itself alone stays so.
std::atomic<int> g_inside{0};
std::mutex g_alone_mu;
thread_local int t_depth = 0;   // calls of this thread, one within the other

// Halt words: allocated together, the free ones in a list.
std::mutex g_halt_mu;
unsigned *g_halt = nullptr;
unsigned *g_halt_free[kHaltWords];
int g_halt_n = 0;

Kept take_kept(int at)   // g_kept_mu held
{
    const Kept k = g_kept[at];
    for (int i = at + 1; i < g_kept_n; i++) g_kept[i - 1] = g_kept[i];
    g_kept_n--;
    g_kept_bytes -= k.bytes;
    return k;
}
}  // namespace

namespace ce {
namespace host {

Use::Use()
{
    if (t_depth++ > 0) return;
    g_inside.fetch_add(1);
    std::lock_guard<std::mutex> wait(g_alone_mu);
}

Use::~Use()
{
    if (--t_depth == 0) g_inside.fetch_sub(1);
}

Alone::Alone() : lock(g_alone_mu), alone(g_inside.load() == 1) {}

ce_status fail(ce_status st, const char *fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return st;
}


void give_back_kept_memory()
{
    std::lock_guard<std::mutex> g(g_kept_mu);
    while (g_kept_n > 0) (void)hipFree(take_kept(0).mem);
}

hipError_t device_memory(size_t bytes, void **out)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    {
        std::lock_guard<std::mutex> g(g_kept_mu);
        for (int i = g_kept_n - 1; i >= 0; i--)
            if (g_kept[i].bytes == bytes && g_kept[i].device == dev) {
                *out = take_kept(i).mem;
                return hipSuccess;
            }
    }
    e = hipMalloc(out, bytes);
    if (e == hipErrorOutOfMemory) {
        (void)hipGetLastError();
        give_back_kept_memory();
        e = hipMalloc(out, bytes);
    }
    return e;
}

void release_device_memory(void *mem, size_t bytes, int device)
{
    if (bytes > kKeptBytes) {
        (void)hipFree(mem);
        return;
    }
    std::lock_guard<std::mutex> g(g_kept_mu);
    while (g_kept_n == kKeptBlocks || g_kept_bytes + bytes > kKeptBytes) (void)hipFree(take_kept(0).mem);
    g_kept[g_kept_n++] = Kept{mem, bytes, device};
    g_kept_bytes += bytes;
}

void ready_halt_words()
{
    std::lock_guard<std::mutex> g(g_halt_mu);
    if (g_halt) return;
    void *mem = nullptr;
    if (hipHostMalloc(&mem, kHaltWords * sizeof(unsigned), hipHostMallocPortable) != hipSuccess) {
        (void)hipGetLastError();
        return;
    }
    g_halt = static_cast<unsigned *>(mem);
    for (g_halt_n = 0; g_halt_n < kHaltWords; g_halt_n++) g_halt_free[g_halt_n] = g_halt + g_halt_n;
}

unsigned *take_halt_word()
{
    std::lock_guard<std::mutex> g(g_halt_mu);
    if (g_halt_n == 0) return nullptr;
    unsigned *w = g_halt_free[--g_halt_n];
    __atomic_store_n(w, 0u, __ATOMIC_RELAXED);
    return w;
}

void give_halt_word(unsigned *w)
{
    if (!w) return;
    std::lock_guard<std::mutex> g(g_halt_mu);
    g_halt_free[g_halt_n++] = w;
}

long long sites_of(const ce_params *p)
{
    long long n = 1;
    for (int d = 0; d < p->dims; d++) n *= p->N;
    return n;
}

Layout layout_of(const ce_params *p)
{
    Layout L;
    const long long ns = sites_of(p);
    const size_t elem = p->precision == CE_FP64 ? 8 : 4;
    // partial-sum rows: one per block, and one per tile for tilings of up
    // to 16 N tiles of a 3-D lattice (the tiled pass sums per tile then)
    L.nblocks = p->dims == 3 ? (int)std::max<long long>(kMaxBlocks, 16LL * p->N) : kMaxBlocks;
    L.field_bytes = align_up((size_t)ns * elem);
    size_t off = 0;
    L.off_fields = off;
    off += 4 * (size_t)p->nfields * L.field_bytes;
    L.off_scalars = off;
    off += align_up(sizeof(Scalars));
    L.off_partials = off;
    off += align_up((size_t)L.nblocks * kMaxSums * sizeof(double));
    L.off_ticket = off;
    static_assert((1 + kTileCounters) * sizeof(unsigned int) <= kAlign, "ticket and tile counters share one line");
    off += kAlign;
    L.off_sync = off;
    off += align_up((size_t)kSyncWords * sizeof(unsigned long long));
    L.off_ring = off;
    off += align_up((size_t)kLogCap * sizeof(ce_energy));
    L.off_maxabs = off;
    off += kAlign;
    L.staging_elems = std::min<long long>(ns, kStagingElems);
    L.off_staging = off;
    off += align_up((size_t)L.staging_elems * sizeof(double));
    L.total = off;
    return L;
}

ce_status validate(const ce_params *p)
{
    if (!p) return fail(CE_EINVAL, "params is NULL");
    if (p->dims < 1 || p->dims > 3) return fail(CE_EINVAL, "dims must be 1, 2 or 3 (got %d)", p->dims);
    if (p->N < 4 || p->N % 4 != 0) return fail(CE_EINVAL, "N must be a multiple of 4 and >= 4 (got %d)", p->N);
    if (p->nfields < 1 || p->nfields > CE_MAX_FIELDS)
        return fail(CE_EINVAL, "nfields must be 1..%d (got %d)", CE_MAX_FIELDS, p->nfields);
    if (p->precision != CE_FP32 && p->precision != CE_FP64)
        return fail(CE_EINVAL, "precision must be CE_FP32 or CE_FP64");
    if (p->model != CE_MODEL_QUARTIC && p->model != CE_MODEL_POLYNOMIAL)
        return fail(CE_EINVAL, "unknown model %d", p->model);
    if (p->model == CE_MODEL_QUARTIC && p->nterms != 0)
        return fail(CE_EINVAL, "the quartic model takes no polynomial terms (nterms = %d)", p->nterms);
    if (p->model == CE_MODEL_POLYNOMIAL) {
        if (p->nterms < 1 || p->nterms > CE_MAX_TERMS)
            return fail(CE_EINVAL, "the polynomial model needs 1..%d terms (got %d)", CE_MAX_TERMS, p->nterms);
        if (p->lambda != 0.0 || p->vacuum != 0.0)
            return fail(CE_EINVAL, "the polynomial model takes lambda and vacuum as terms; set them to 0");
        for (int i = 0; i < CE_MAX_FIELDS; i++)
            if (p->G[i] != 0.0 || p->mu2[i] != 0.0)
                return fail(CE_EINVAL, "the polynomial model takes couplings and masses as terms; set G and mu2 to 0");
        for (int t = 0; t < p->nterms; t++) {
            const ce_term &tm = p->terms[t];
            if (!isfinite(tm.coef)) return fail(CE_EINVAL, "term %d: coefficient must be finite", t);
            int deg = 0;
            for (int i = 0; i < CE_MAX_FIELDS; i++) {
                if (tm.exp[i] < 0 || tm.exp[i] > CE_MAX_EXP)
                    return fail(CE_EINVAL, "term %d: exponent %d of field %d outside 0..%d", t, tm.exp[i], i,
                                CE_MAX_EXP);
                if (i >= p->nfields && tm.exp[i] != 0)
                    return fail(CE_EINVAL, "term %d: field %d does not exist (nfields = %d)", t, i, p->nfields);
                deg += tm.exp[i];
            }
            if (deg > CE_MAX_DEGREE)
                return fail(CE_EINVAL, "term %d: degree %d above %d", t, deg, CE_MAX_DEGREE);
        }
    }
    if (p->expansion != 0 && p->expansion != 1) return fail(CE_EINVAL, "expansion must be 0 or 1");
    if (!(p->L > 0) || !isfinite(p->L)) return fail(CE_EINVAL, "L must be positive and finite");
    if (!(p->dt > 0) || !isfinite(p->dt)) return fail(CE_EINVAL, "dt must be positive and finite");
    if (!(p->lambda >= 0) || !isfinite(p->lambda)) return fail(CE_EINVAL, "lambda must be >= 0");
    for (int i = 0; i < CE_MAX_FIELDS; i++) {
        if (!isfinite(p->G[i]) || p->G[i] < 0) return fail(CE_EINVAL, "G[%d] must be >= 0", i);
        if (!isfinite(p->mu2[i])) return fail(CE_EINVAL, "mu2[%d] must be finite", i);
    }
    if (!isfinite(p->vacuum)) return fail(CE_EINVAL, "vacuum must be finite");
    if (p->expansion && !(p->kappa > 0 && isfinite(p->kappa)))
        return fail(CE_EINVAL, "kappa must be positive with expansion");
    // site indices are 64-bit; 2^40 sites is far beyond any lattice that fits
    // in HBM.  The bound is checked before each multiplication: N^dims itself
    // can exceed 64 bits.
    long long ns = 1;
    for (int d = 0; d < p->dims; d++) {
        if (ns > (1LL << 40) / p->N) return fail(CE_EINVAL, "lattice too large (N^dims > 2^40 sites)");
        ns *= p->N;
    }
    const double dx = p->L / p->N;
    const double w = p->dt * 2.0 * sqrt((double)p->dims) / dx;
    if (!(w < 2.0))
        return fail(CE_EINVAL, "leapfrog unstable: dt*2*sqrt(dims)/dx = %g >= 2", w);
    return CE_OK;
}

void drop_graphs(ce_sim *s)
{
    for (int b = 0; b < 2; b++) {
        if (s->graph[b]) (void)hipGraphExecDestroy(s->graph[b]);
        s->graph[b] = nullptr;
    }
    s->graph_k = 0;
}

ce_status build_graph(ce_sim *s, int parity)
{
    if (!s->cap_stream) CE_HIP(hipStreamCreateWithFlags(&s->cap_stream, hipStreamNonBlocking));
    hipGraph_t g = nullptr;
    CE_HIP(hipStreamBeginCapture(s->cap_stream, hipStreamCaptureModeThreadLocal));
    hipError_t err = hipSuccess;
    for (int k = 0; k < s->step_block && err == hipSuccess; k++)
        err = launch_pass(s->lat, s->p.precision, (parity + k) & 1, s->resident.kernel ? kGuardedStep : kStep,
                          s->cap_stream);
    hipError_t e2 = hipStreamEndCapture(s->cap_stream, &g);
    if (err != hipSuccess || e2 != hipSuccess) {
        if (g) (void)hipGraphDestroy(g);
        return fail(CE_EDEVICE, "step-block capture failed: %s",
                    hipGetErrorString(err != hipSuccess ? err : e2));
    }
    hipGraphExec_t ex = nullptr;
    err = hipGraphInstantiate(&ex, g, nullptr, nullptr, 0);
    (void)hipGraphDestroy(g);
    if (err != hipSuccess) return fail(CE_EDEVICE, "graph instantiate failed: %s", hipGetErrorString(err));
    s->graph[parity] = ex;
    s->graph_k = s->step_block;
    return CE_OK;
}

hipError_t launch_resident(ce_sim *s, int steps)
{
    int src = s->cur;
    Start start{s->wait, s->halt};
    void *args[] = {&s->lat, &src, &steps, &start};
    const dim3 grid(s->resident.blocks), block(s->resident.threads);
    // a single block waits for nobody
    const hipError_t e = s->resident.blocks > 1
                             ? hipLaunchCooperativeKernel(s->resident.kernel, grid, block, args, 0, s->stream)
                             : hipLaunchKernel(s->resident.kernel, grid, block, args, 0, s->stream);
    if (e != hipSuccess) return e;
    s->unsettled = true;
    s->cur ^= steps & 1;
    s->step += steps;
    return hipSuccess;
}

hipError_t clear_arrivals(ce_sim *s)
{
    static const unsigned long long none = 0;
    return hipMemcpyAsync(s->lat.sync + kArrivals, &none, sizeof(none), hipMemcpyHostToDevice, s->stream);
}

ce_status take_missing_steps(ce_sim *s, const long long *left)
{
    Scalars sc;
    CE_HIP(hipMemcpyAsync(&sc, s->lat.sc, sizeof(sc), hipMemcpyDeviceToHost, s->stream));
    CE_HIP(hipStreamSynchronize(s->stream));
    if (sc.halted == kRuns) return CE_OK;
    if (sc.halted != kNotStarted)
        return fail(CE_EDEVICE, "a resident launch lost its blocks' sums by step %lld: the state is lost", sc.step);
    const long long missing = s->step - sc.step;
    if (missing < 0) return fail(CE_EDEVICE, "halted at step %lld, ahead of step %lld", sc.step, s->step);
    CE_HIP(clear_arrivals(s));
    // the state is where it was, in the buffer of its own step
    const int runs = kRuns, from = s->cur ^ (int)(missing & 1);
    CE_HIP(hipMemcpyAsync(&s->lat.sc->halted, &runs, sizeof(runs), hipMemcpyHostToDevice, s->stream));
    for (long long k = 0; k < missing; k++)
        CE_HIP(launch_pass(s->lat, s->p.precision, (from + (int)(k & 1)) & 1, kStep, s->stream));
    if (left) {
        CE_HIP(hipMemcpyAsync(&s->lat.sc->cur, &s->cur, sizeof(int), hipMemcpyHostToDevice, s->stream));
        CE_HIP(hipMemcpyAsync(&s->lat.sc->remaining, left, sizeof(*left), hipMemcpyHostToDevice, s->stream));
    }
    CE_HIP(hipStreamSynchronize(s->stream));
    return CE_OK;
}

ce_status settle(ce_sim *s)
{
    s->unsettled = false;
    if (!halt_seen(s)) return CE_OK;
    // plain launches from now on: other work holds the units
    s->resident = ce_sim::Resident{};
    s->resident_planned = true;
    const ce_status st = take_missing_steps(s, nullptr);
    if (st == CE_OK) __atomic_store_n(s->halt, 0u, __ATOMIC_RELAXED);
    return st;
}

ce_status device_cus(int *cus)
{
    int dev = 0;
    CE_HIP(hipGetDevice(&dev));
    CE_HIP(hipDeviceGetAttribute(cus, hipDeviceAttributeMultiprocessorCount, dev));
    return CE_OK;
}

const void *resident_kernel(const ce_params *p, const ce_launch &c, bool ragged, bool batched)
{
    if (c.kernel == CE_KERNEL_STREAM2D)
        return stream2d_groups(p->N, c.planes) > kSyncRows ? nullptr
               : p->model == kPoly ? resident_stream2d_model<kPoly>(p->precision, p->nfields, c.planes, batched)
                                   : resident_stream2d_model<kQuartic>(p->precision, p->nfields, c.planes, batched);
    if ((!ragged && p->N % c.planes != 0) ||
        tiled_tiles(p->N, c.sites_per_thread, c.lanes_per_row, c.block, c.planes) > kSyncRows)
        return nullptr;
    return p->model == kPoly ? resident_tiled_model<kPoly>(p->precision, p->nfields, c.sites_per_thread,
                                                           c.lanes_per_row, c.block, c.planes, ragged, batched)
                             : resident_tiled_model<kQuartic>(p->precision, p->nfields, c.sites_per_thread,
                                                              c.lanes_per_row, c.block, c.planes, ragged,
                                                              batched);
}

// Built resident passes that are so short of registers that plain launches of
// the same tiling are as fast or faster (us a step, resident and plain): three
// FP64 fields in the direct pass, 32^3 12.0 and 11.4, 48^3 20.5 and 13.5,
// except where a block holds whole planes and there are few (16^3 7.5 and 10.2);
// in units of four rows, 768^2 25.6 and 21.9; three FP32 fields of the
// polynomial model in units of eight, 1280^2 44.7 and 43.8.
bool resident_pays(const Lattice &lat, int precision)
{
    if (lat.nf < 3) return true;
    if (lat.kind == kDirect && lat.dims == 3 && precision == CE_FP64)
        return lat.N <= 16 && kBlock % (lat.N * lat.N / 4) == 0;
    if (lat.kind == kStream2d) return precision == CE_FP64 ? lat.zc < 4 : lat.model != kPoly || lat.zc < 8;
    return true;
}

// The resident pass that takes the same steps as s's launch, if there is one:
// its blocks must all be resident at once, one per published row.
void plan_resident(ce_sim *s)
{
    s->resident = ce_sim::Resident{};
    s->resident_planned = true;
    const Lattice &lat = s->lat;
    if (!resident_pays(lat, s->p.precision)) return;
    ce_sim::Resident r;
    if (lat.kind == kDirect) {
        // one quad per thread, and no block without one; VB blocks of the
        // launch are taken as one, so that at most kSyncRows remain
        if ((lat.nsites / 4 + kBlock - 1) / kBlock != lat.nblocks) return;
        const int vb = (lat.nblocks + kSyncRows - 1) / kSyncRows;
        r.kernel = s->p.model == kPoly ? resident_direct_model<kPoly>(s->p.precision, lat.dims, lat.nf, vb)
                                       : resident_direct_model<kQuartic>(s->p.precision, lat.dims, lat.nf, vb);
        r.blocks = (lat.nblocks + vb - 1) / vb;
        r.threads = kBlock * vb + 64;
    } else if (lat.kind == kTiled3d) {
        const ce_launch c{CE_KERNEL_TILED3D, lat.vec, lat.lpr, lat.bs, lat.zc, 0};
        r.kernel = resident_kernel(&s->p, c, lat.ragged != 0, false);
        r.blocks = (int)tiled_tiles(lat.N, lat.vec, lat.lpr, lat.bs, lat.zc);
        r.threads = lat.bs + 64;
    } else if (lat.kind == kStream2d) {
        // the streaming pass sums per block: one group of units each
        if (stream2d_groups(lat.N, lat.zc) != lat.nblocks) return;
        r.kernel = resident_kernel(&s->p, ce_launch{CE_KERNEL_STREAM2D, 4, 64, kBlock, lat.zc, lat.nblocks}, false, false);
        r.blocks = lat.nblocks;
        r.threads = kBlock + 64;
    }
    if (!r.kernel) return;
    if (!s->halt) s->halt = take_halt_word();
    if (!s->halt) return;
    // the fewest steps worth a launch: a cooperative one costs about 22 us
    // (32^3: 4 steps 36 us plain, 40 resident, 6 steps 54 and 48; 64^3: 2 steps
    // 27 and 32, 3 steps 40 and 37), a single block's 3 (1-D 1024: 2 steps 10.9
    // and 7.4)
    r.min_steps = r.blocks == 1 ? 2 : lat.kind == kDirect ? 5 : 3;
    int cus = 0, per = 0;
    if (device_cus(&cus) != CE_OK) return;
    if (r.blocks > 1 &&
        (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, r.kernel, r.threads, 0) != hipSuccess ||
         (long long)per * cus < r.blocks)) {
        (void)hipGetLastError();
        return;
    }
    s->resident = r;
}

// Validate cfg for the lattice and fill the kernel-facing fields of lat.
ce_status apply_launch(ce_sim *s, const ce_launch &cfg)
{
    // planned by the first call that steps: pool members never do
    s->resident = ce_sim::Resident{};
    s->resident_planned = false;
    Lattice &lat = s->lat;
    if (cfg.grid < 0 || cfg.grid > kMaxBlocks) return fail(CE_EINVAL, "grid must be 0..%d", kMaxBlocks);
    if (cfg.kernel == CE_KERNEL_DIRECT) {
        int g = cfg.grid ? cfg.grid : pass_blocks(s->p.dims, s->p.N);
        s->grid = g;
        RaggedTiling r;
        if (ragged_tiling(s->p.precision, s->p.dims, s->p.N, &r)) {
            // summed per tile, so the result does not depend on the blocks
            lat.kind = kTiled3d;
            lat.ragged = 1;
            lat.vec = 4;
            lat.lpr = r.lpr;
            lat.bs = kBlock;
            lat.zc = r.planes;
            lat.nblocks = std::min(g, r.tiles);
        } else {
            lat.kind = kDirect;
            lat.ragged = 0;
            lat.vec = lat.lpr = lat.bs = lat.zc = 0;
            lat.nblocks = g;
        }
    } else if (cfg.kernel == CE_KERNEL_TILED3D) {
        if (!tiled_shape_built(cfg.sites_per_thread, cfg.lanes_per_row, cfg.block))
            return fail(CE_EINVAL, "tiled shape (sites_per_thread=%d, lanes_per_row=%d, block=%d) is not built",
                        cfg.sites_per_thread, cfg.lanes_per_row, cfg.block);
        if (!tiled_fits(s->p.dims, s->p.N, cfg.sites_per_thread, cfg.lanes_per_row, cfg.block, cfg.planes))
            return fail(CE_EINVAL, "tiled launch (%d x %d tile, planes=%d) does not fit dims=%d N=%d",
                        cfg.sites_per_thread * cfg.lanes_per_row, cfg.block / cfg.lanes_per_row, cfg.planes,
                        s->p.dims, s->p.N);
        const long long tiles =
            tiled_tiles(s->p.N, cfg.sites_per_thread, cfg.lanes_per_row, cfg.block, cfg.planes);
        int g = cfg.grid;
        if (g == 0) {
            int cus = 0;
            ce_status st = device_cus(&cus);
            if (st != CE_OK) return st;
            const int per = tiled_resident_blocks(s->p.model, s->p.precision, s->p.nfields, cfg.sites_per_thread,
                                                  cfg.lanes_per_row, cfg.block);
            if (per < 1) return fail(CE_EDEVICE, "tiled kernel cannot be resident");
            // as many blocks as stay resident, then evened out so every block
            // walks the same number of tiles; a multiple of 8 keeps each
            // XCD on one contiguous slab of tiles
            long long resident = (long long)per * cus;
            if (resident > kMaxBlocks) resident = kMaxBlocks;
            const long long rounds = (tiles + resident - 1) / resident;
            long long want = (tiles + rounds - 1) / rounds;
            if (want >= 8) want = (want + 7) / 8 * 8;
            if (want > kMaxBlocks) want = kMaxBlocks / 8 * 8;
            g = (int)want;
        }
        lat.kind = kTiled3d;
        lat.ragged = 0;
        lat.vec = cfg.sites_per_thread;
        lat.lpr = cfg.lanes_per_row;
        lat.bs = cfg.block;
        lat.zc = cfg.planes;
        lat.nblocks = s->grid = g;
    } else if (cfg.kernel == CE_KERNEL_STREAM2D) {
        if (!stream2d_fits(s->p.dims, s->p.N, cfg.planes))
            return fail(CE_EINVAL, "2-D streaming launch (rows=%d) does not fit dims=%d N=%d", cfg.planes,
                        s->p.dims, s->p.N);
        const long long groups = stream2d_groups(s->p.N, cfg.planes);
        int g = cfg.grid;
        if (g == 0) {
            int cus = 0;
            ce_status st = device_cus(&cus);
            if (st != CE_OK) return st;
            long long resident = (long long)stream2d_resident_blocks() * cus;
            if (resident < 1) return fail(CE_EDEVICE, "2-D streaming kernel cannot be resident");
            if (resident > kMaxBlocks) resident = kMaxBlocks;
            const long long rounds = (groups + resident - 1) / resident;
            long long want = (groups + rounds - 1) / rounds;
            if (want >= 8) want = (want + 7) / 8 * 8;
            if (want > kMaxBlocks) want = kMaxBlocks / 8 * 8;
            g = (int)want;
        }
        lat.kind = kStream2d;
        lat.vec = 4;
        lat.lpr = 64;
        lat.bs = kBlock;
        lat.zc = cfg.planes;
        lat.ragged = 0;
        lat.nblocks = s->grid = g;
        // the shape is fixed: report it whatever the caller passed
        s->launch = ce_launch{CE_KERNEL_STREAM2D, 4, 64, kBlock, cfg.planes, cfg.grid};
        drop_graphs(s);
        return CE_OK;
    } else {
        return fail(CE_EINVAL, "unknown kernel %d", cfg.kernel);
    }
    s->launch = cfg;
    drop_graphs(s);
    return CE_OK;
}

// The library's default launch.  3-D lattices use the tiled kernel with the
// widest tile that divides N (256 x 4 sites, 4 per thread, then 64 x 16,
// then 32 x 32): wide tiles keep the x halo to 2 of every 8 cache lines.
// Large lattices keep every resident block busy with the longest chunks that
// give every block the same whole number of tiles (three chunks of 342, 342
// and 340 planes at 1024^3, four tiles a block); lattices that a resident pass
// can take are cut into up to 256 tiles; medium ones get two tiles or so per
// compute unit, else one (N >= 64) with the tallest chunks that allow it;
// smaller ones take the tallest chunks that leave three tiles per compute
// unit, or the direct kernel when they cannot give one tile per compute unit.
ce_launch default_launch(const ce_params *p, int cus)
{
    ce_launch c{CE_KERNEL_DIRECT, 0, 0, 0, 0, 0};
    if (p->dims == 2) {
        // lattices that a resident pass can take: the shortest units that
        // leave no more groups of four than it has blocks.  (The polynomial
        // model's units of sixteen rows only where they fill the chip: 1536^2 x 2
        // fields, 144 groups, took 52.0 us a step, plain units of eight take 36.6.)
        for (int rows = 1; rows <= 16; rows *= 2) {
            const ce_launch r{CE_KERNEL_STREAM2D, 4, 64, kBlock, rows, 0};
            if (!stream2d_fits(2, p->N, rows) || !resident_kernel(p, r, false, false)) continue;
            if (p->model == kPoly && rows == 16 && stream2d_groups(p->N, rows) < cus) continue;
            return r;
        }
        // rows per unit: the tallest (up to 64) that still gives every
        // compute unit a group of four units
        for (int rows = 64; rows >= 8; rows /= 2)
            if (stream2d_fits(2, p->N, rows) && (stream2d_groups(p->N, rows) >= cus || rows == 8)) {
                c.kernel = CE_KERNEL_STREAM2D;
                c.sites_per_thread = 4;
                c.lanes_per_row = 64;
                c.block = kBlock;
                c.planes = rows;
                return c;
            }
        return c;
    }
    if (p->dims != 3) return c;
    const int shapes[3][3] = {{4, 64, 256}, {4, 16, 256}, {4, 8, 256}};
    for (int a = 0; a < 3; a++) {
        const int v = shapes[a][0], l = shapes[a][1], bs = shapes[a][2];
        if (!tiled_fits(3, p->N, v, l, bs, p->N)) continue;
        // Large lattices: every block that fits stays resident (full
        // occupancy hides the most memory latency).  Each z chunk re-reads
        // two halo planes from memory, so chunks are as long as possible:
        // the fewest chunks per column that give every block the same whole
        // number (>= 2) of tiles.  Else short z chunks, so the last, partial
        // round of tiles is a small part of the pass.
        long long resident = (long long)tiled_resident_blocks(p->model, p->precision, p->nfields, v, l, bs) * cus;
        if (resident > kMaxBlocks) resident = kMaxBlocks;
        if (resident >= 8) resident = resident / 8 * 8;
        const long long cols = tiled_tiles(p->N, v, l, bs, p->N);
        // A lattice whose columns divide the resident blocks (up to three a
        // compute unit) has one tile for each, with no second start and the
        // fewest halo planes (512^3, ms a step with one tile a block and with
        // the rule below: one field 0.378 and 0.447, two 0.799 and 0.834,
        // three 1.21 and 1.22; FP64, two 1.82 and 1.85.  A single chunk, the
        // whole column, gains nothing: FP64, three, 2.78 and 2.75).
        const long long one = std::min<long long>(resident, 3LL * cus);
        if (one > cols && one % cols == 0 && p->N / (one / cols) >= 64) {
            const int nz = (int)(one / cols), planes = (p->N + nz - 1) / nz;
            if ((p->N + planes - 1) / planes == nz) {
                c.kernel = CE_KERNEL_TILED3D;
                c.sites_per_thread = v;
                c.lanes_per_row = l;
                c.block = bs;
                c.planes = planes;
                c.grid = (int)one;
                return c;
            }
        }
        for (int nz = 1; nz <= p->N / 64 && resident > 0; nz++) {
            const long long tiles = cols * nz;
            const int planes = (p->N + nz - 1) / nz;  // nz chunks of near-equal length
            if ((p->N + planes - 1) / planes == nz && tiles >= 2 * resident && tiles % resident == 0) {
                c.kernel = CE_KERNEL_TILED3D;
                c.sites_per_thread = v;
                c.lanes_per_row = l;
                c.block = bs;
                c.planes = planes;
                c.grid = (int)resident;
                return c;
            }
        }
        for (int z = 32; z >= 16 && resident > 0; z /= 2)
            if (p->N % z == 0 && tiled_tiles(p->N, v, l, bs, z) >= (z == 32 ? 8 : 4) * resident) {
                c.kernel = CE_KERNEL_TILED3D;
                c.sites_per_thread = v;
                c.lanes_per_row = l;
                c.block = bs;
                c.planes = z;
                c.grid = (int)resident;
                return c;
            }
    }
    // Lattices that a resident pass can take: the shortest chunks (up to 8
    // planes) that leave no more tiles than it has blocks, so that the step's
    // sites are spread over as many compute units as there are (64^3 x 2
    // fields: 4.8 us a step with 256 tiles of one plane, 5.3 with 128 of two,
    // 8.0 with 64 of four).  The tile shapes are those it is built for.
    for (int a = 0; a < 2; a++) {
        const bool fp64 = p->precision == CE_FP64;
        const int v = fp64 ? 2 : 4, l = (fp64 ? 32 : 16) >> a, bs = fp64 ? 512 : 256;
        // two planes at least where one gains the resident pass nothing and
        // costs single steps (64^3 in FP64, one and two fields: 4.1 and 5.8 us a
        // step, single ones 18.3 and 20.3; one plane 4.3 and 5.8, 22.8 and 25.0)
        const int least = fp64 && p->model == kQuartic && p->nfields <= 2 ? 2 : 1;
        for (int z = least; z <= 8 && p->N >= 64; z *= 2) {
            if (p->N % z || !tiled_fits(3, p->N, v, l, bs, z) || tiled_tiles(p->N, v, l, bs, z) > kSyncRows) continue;
            const ce_launch r{CE_KERNEL_TILED3D, v, l, bs, z, 0};
            if (resident_kernel(p, r, false, false)) return r;
        }
    }
    // Medium lattices: all tiles resident at once, two to a compute unit, two
    // and a half of the 256-site ones where three fit (us a step, and with the
    // rule below: 192^3 x 2 fields 57 and 63, FP64 108 and 117; 224^3 x 2 112
    // and 122; 256^3 x 2 115 and 120, FP64 229 and 283, one field 60 and 69;
    // 288^3 x 2 210 and 215; three tiles a unit were 4% behind two at 192^3,
    // one 41%).  Chunks of at most 64 planes: with 88, 352^3 x 2 took 399 us
    // against 362.
    for (int a = 0; a < 3; a++) {
        const int v = shapes[a][0], l = shapes[a][1], bs = shapes[a][2];
        if (!tiled_fits(3, p->N, v, l, bs, p->N)) continue;
        const int fit = tiled_resident_blocks(p->model, p->precision, p->nfields, v, l, bs);
        if (fit < 2) break;
        const long long cols = tiled_tiles(p->N, v, l, bs, p->N);
        const int nz = (int)((l == 64 && fit >= 3 ? 5LL * cus / 2 : 2LL * cus) / cols);
        if (nz < 4 || p->N / nz < 8 || p->N > 64 * nz) break;
        c.kernel = CE_KERNEL_TILED3D;
        c.sites_per_thread = v;
        c.lanes_per_row = l;
        c.block = bs;
        c.planes = (p->N + nz - 1) / nz;
        c.grid = 0;
        return c;
    }
    if (p->N >= 64) {
        // Medium lattices (64^3 .. 256^3 and the like): one tile per compute
        // unit where the lattice has that many, with the tallest chunks that
        // still give them, else the shortest (2 planes).  Widest tiles first,
        // 512-thread blocks where the tile is 256 sites wide.  On 64^3,
        // 128^3 and 256^3 x 2 fields this is the fastest configuration found
        // by timing every shape and chunk length (128^3: 3.2x the direct pass).
        const int pref[5][3] = {{4, 64, 512}, {4, 64, 256}, {4, 16, 256}, {2, 32, 512}, {4, 8, 256}};
        for (int a = 0; a < 5; a++) {
            const int v = pref[a][0], l = pref[a][1], bs = pref[a][2];
            if (!tiled_fits(3, p->N, v, l, bs, 2) || p->N % 2) continue;
            int planes = 2;
            for (int z = 2; z <= p->N; z *= 2)
                if (p->N % z == 0 && tiled_tiles(p->N, v, l, bs, z) >= cus) planes = z;
            c.kernel = CE_KERNEL_TILED3D;
            c.sites_per_thread = v;
            c.lanes_per_row = l;
            c.block = bs;
            c.planes = planes;
            c.grid = 0;
            return c;
        }
    }
    for (int a = 0; a < 3; a++) {
        const int v = shapes[a][0], l = shapes[a][1], bs = shapes[a][2];
        if (!tiled_fits(3, p->N, v, l, bs, p->N)) continue;
        // smaller lattices: the tallest chunks that still give three tiles
        // per compute unit; the grid is evened over the rounds
        int planes = 0;
        for (int z = p->N; z >= 16; z /= 2) {
            if (p->N % z) continue;
            planes = z;
            if (tiled_tiles(p->N, v, l, bs, z) >= 3LL * cus) break;
        }
        if (planes == 0 || tiled_tiles(p->N, v, l, bs, planes) < cus) continue;
        c.kernel = CE_KERNEL_TILED3D;
        c.sites_per_thread = v;
        c.lanes_per_row = l;
        c.block = bs;
        c.planes = planes;
        return c;
    }
    return ce_launch{CE_KERNEL_DIRECT, 0, 0, 0, 0, 0};
}

}  // namespace host
}  // namespace ce

extern "C" {

const char *ce_last_error(void) { return g_err; }

ce_status ce_get_launch(const ce_sim *s, ce_launch *out)
{
    if (!s || !out) return fail(CE_EINVAL, "NULL argument");
    *out = s->launch;
    out->grid = s->grid;
    return CE_OK;
}

ce_status ce_set_launch(ce_sim *s, const ce_launch *cfg)
{
    const Use use;
    if (!s || !cfg) return fail(CE_EINVAL, "NULL argument");
    if (s->unsettled) {
        // steps left out of a halted state are those of the launch as it is
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        CE_HIP(hipStreamIsCapturing(s->stream, &cap));
        if (cap == hipStreamCaptureStatusNone) {
            CE_HIP(hipStreamSynchronize(s->stream));
            const ce_status st = settle(s);
            if (st != CE_OK) return st;
        }
    }
    const ce_launch old = s->launch;
    const Lattice saved = s->lat;
    const ce_sim::Resident resident = s->resident;
    const int grid = s->grid;
    ce_status st = apply_launch(s, *cfg);
    if (st != CE_OK) {
        s->grid = grid;
        s->launch = old;
        s->lat = saved;
        s->resident = resident;
    }
    return st;
}

ce_status ce_required_bytes(const ce_params *p, size_t *out)
{
    ce_status st = validate(p);
    if (st != CE_OK) return st;
    if (!out) return fail(CE_EINVAL, "out is NULL");
    *out = layout_of(p).total;
    return CE_OK;
}

ce_status ce_create(const ce_params *p, ce_sim **out)
{
    const Use use;
    ce_status st = validate(p);
    if (st != CE_OK) return st;
    if (!out) return fail(CE_EINVAL, "out is NULL");
    *out = nullptr;
    ce_sim *s = new (std::nothrow) ce_sim();
    if (!s) return fail(CE_ENOMEM, "host allocation failed");
    s->p = *p;
    s->lay = layout_of(p);
    const Layout &L = s->lay;
    if (p->arena) {
        if ((uintptr_t)p->arena % kAlign) {
            delete s;
            return fail(CE_EINVAL, "arena must be %zu-byte aligned", kAlign);
        }
        if (p->arena_bytes < L.total) {
            delete s;
            return fail(CE_ENOMEM, "arena holds %zu bytes, %zu needed", p->arena_bytes, L.total);
        }
        s->base = static_cast<char *>(p->arena);
    } else {
        void *mem = nullptr;
        hipError_t e = device_memory(L.total, &mem);
        if (e == hipSuccess) e = hipGetDevice(&s->device);
        s->base = static_cast<char *>(mem);
        if (e != hipSuccess) {
            delete s;
            (void)hipGetLastError();
            return fail(CE_ENOMEM, "hipMalloc(%zu) failed: %s", L.total, hipGetErrorString(e));
        }
        s->own_mem = true;
    }
    if (p->stream) {
        s->stream = static_cast<hipStream_t>(p->stream);
    } else {
        hipError_t e = hipStreamCreateWithFlags(&s->stream, hipStreamNonBlocking);
        if (e != hipSuccess) {
            ce_destroy(s);
            return fail(CE_EDEVICE, "stream creation failed: %s", hipGetErrorString(e));
        }
        s->own_stream = true;
    }
    Lattice &lat = s->lat;
    memset(&lat, 0, sizeof(lat));
    for (int b = 0; b < 2; b++)
        for (int i = 0; i < p->nfields; i++) {
            lat.d[b][i] = s->base + L.off_fields + ((size_t)(b * p->nfields + i)) * L.field_bytes;
            lat.p[b][i] = s->base + L.off_fields + ((size_t)((2 + b) * p->nfields + i)) * L.field_bytes;
        }
    lat.dims = p->dims;
    lat.N = p->N;
    lat.nf = p->nfields;
    lat.expansion = p->expansion;
    lat.nsites = sites_of(p);
    lat.dt = p->dt;
    const double dx = p->L / p->N;
    lat.inv_dx2 = 1.0 / (dx * dx);
    lat.lambda = p->lambda;
    lat.kappa = p->kappa;
    lat.vacuum = p->vacuum;
    for (int i = 0; i < kMaxFields; i++) {
        lat.G[i] = i < p->nfields ? p->G[i] : 0.0;
        lat.mu2[i] = i < p->nfields ? p->mu2[i] : 0.0;
    }
    lat.G[0] = 0.0;
    // polynomial model: the terms of degree >= 1 go to the kernels; constant
    // terms are a vacuum energy (a^4 V0 in the program variables)
    lat.model = p->model;
    lat.nterms = 0;
    if (p->model == CE_MODEL_POLYNOMIAL) {
        for (int t = 0; t < p->nterms; t++) {
            const ce_term &tm = p->terms[t];
            int deg = 0;
            for (int i = 0; i < CE_MAX_FIELDS; i++) deg += tm.exp[i];
            if (deg == 0) {
                lat.vacuum += tm.coef;
                continue;
            }
            const int k = lat.nterms++;
            lat.tcoef[k] = tm.coef;
            lat.tdeg[k] = deg;
            for (int i = 0; i < kMaxFields; i++) lat.texp[k][i] = tm.exp[i];
        }
    }
    lat.dt_f = (float)lat.dt;
    lat.inv_dx2_f = (float)lat.inv_dx2;
    lat.lambda_f = (float)lat.lambda;
    lat.qlam_f = (float)(0.25 * lat.lambda);
    for (int i = 0; i < kMaxFields; i++) {
        lat.G_f[i] = (float)lat.G[i];
        lat.hG_f[i] = (float)(0.5 * lat.G[i]);
    }
    lat.sc = reinterpret_cast<Scalars *>(s->base + L.off_scalars);
    lat.partials = reinterpret_cast<double *>(s->base + L.off_partials);
    lat.ticket = reinterpret_cast<unsigned int *>(s->base + L.off_ticket);
    lat.slots = L.nblocks;
    lat.sync = reinterpret_cast<unsigned long long *>(s->base + L.off_sync);
    lat.ring = reinterpret_cast<ce_energy *>(s->base + L.off_ring);
    lat.columns = s->base + L.off_staging;
    ready_halt_words();
    {
        int cus = 0;
        ce_status st2 = device_cus(&cus);
        if (st2 == CE_OK) st2 = apply_launch(s, default_launch(p, cus));
        if (st2 != CE_OK) {
            const ce_status keep = st2;
            char msg[sizeof(g_err)];
            memcpy(msg, g_err, sizeof(msg));
            ce_destroy(s);
            memcpy(g_err, msg, sizeof(msg));
            return keep;
        }
    }
    s->maxabs = reinterpret_cast<unsigned int *>(s->base + L.off_maxabs);
    s->staging = reinterpret_cast<double *>(s->base + L.off_staging);

    Scalars init{};
    init.a = 1.0;
    init.a_next = 1.0;
    init.first_bad = -1;
    hipError_t e = hipMemcpyAsync(lat.sc, &init, sizeof(init), hipMemcpyHostToDevice, s->stream);
    if (e == hipSuccess) e = hipMemsetAsync(lat.ticket, 0, L.off_ring - L.off_ticket, s->stream);
    if (e == hipSuccess) e = hipMemsetAsync(s->maxabs, 0, kAlign, s->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(s->stream);
    if (e != hipSuccess) {
        ce_destroy(s);
        return fail(CE_EDEVICE, "initialisation failed: %s", hipGetErrorString(e));
    }
    *out = s;
    return CE_OK;
}

ce_status ce_load_fields(ce_sim *s, int32_t first, int32_t count, const double *phi,
                         const double *phidot)
{
    const Use use;
    if (!s) return fail(CE_EINVAL, "sim is NULL");
    if (s->started) return fail(CE_ESTATE, "fields already loaded and evolved");
    // compared without forming first + count, which could overflow
    if (first < 0 || count < 1 || first >= s->p.nfields || count > s->p.nfields - first)
        return fail(CE_EINVAL, "field range of %d fields from %d outside 0..%d", count, first, s->p.nfields);
    if (!phi || !phidot) return fail(CE_EINVAL, "phi and phidot must be non-NULL");
    const long long ns = s->lat.nsites;
    const long long chunk = s->lay.staging_elems;
    const size_t elem = s->p.precision == CE_FP64 ? 8 : 4;
    for (int i = 0; i < count; i++) {
        const int fi = first + i;
        // homogeneous reference: the mean of an evenly strided sample of at
        // most 2^16 sites.  Any value near the volume mean works (the stored
        // deviation is exact relative to it, and the reference then moves
        // with the mean derivative); the sample keeps the deviations at the
        // size of the fluctuations without a host pass over the whole field.
        const double *fsrc = phi + (long long)i * ns;
        const long long stride = std::max<long long>(1, ns >> 16);
        double part[8] = {0, 0, 0, 0, 0, 0, 0, 0};
        long long cnt = 0;
        for (long long k = 0; k < ns; k += stride, cnt++) part[cnt & 7] += fsrc[k];
        const double acc = ((part[0] + part[1]) + (part[2] + part[3])) + ((part[4] + part[5]) + (part[6] + part[7]));
        s->m_host[fi] = acc / (double)cnt;
        if (!isfinite(s->m_host[fi])) return fail(CE_EINVAL, "initial field %d is not finite", fi);
        CE_HIP(hipMemcpyAsync(&s->lat.sc->m[fi], &s->m_host[fi], sizeof(double), hipMemcpyHostToDevice,
                              s->stream));
        for (int which = 0; which < 2; which++) {
            const double *src = (which == 0 ? phi : phidot) + (long long)i * ns;
            void *dst = which == 0 ? s->lat.d[s->cur][fi] : s->lat.p[s->cur][fi];
            const double ref = which == 0 ? s->m_host[fi] : 0.0;
            for (long long off = 0; off < ns; off += chunk) {
                const long long n = std::min(chunk, ns - off);
                CE_HIP(hipMemcpyAsync(s->staging, src + off, (size_t)n * sizeof(double),
                                      hipMemcpyHostToDevice, s->stream));
                CE_HIP(launch_convert(s->staging, ref, static_cast<char *>(dst) + (size_t)off * elem,
                                      s->p.precision, n, which == 0 ? s->maxabs + fi : s->maxabs + 3,
                                      s->stream));
            }
        }
        s->loaded |= 1u << fi;
    }
    CE_HIP(hipStreamSynchronize(s->stream));
    if (s->loaded != (1u << s->p.nfields) - 1) return CE_OK;
    return start_run(s);
}

}  // extern "C"

namespace ce {
namespace host {

ce_status start_run(ce_sim *s)
{
    // all fields present: stability including the potential's curvature,
    // bounded with the largest |f| of every field
    unsigned int bits[4];
    CE_HIP(hipMemcpy(bits, s->maxabs, sizeof(bits), hipMemcpyDeviceToHost));
    // a rejected set of fields must be loaded again; the maxima start over
    auto reject = [s]() -> ce_status {
        s->loaded = 0;
        CE_HIP(hipMemsetAsync(s->maxabs, 0, kAlign, s->stream));
        CE_HIP(hipStreamSynchronize(s->stream));
        return CE_EINVAL;
    };
    double M[CE_MAX_FIELDS] = {0, 0, 0};
    for (int i = 0; i < s->p.nfields; i++) {
        float v;
        memcpy(&v, &bits[i], sizeof(v));
        M[i] = v;
    }
    float vd;
    memcpy(&vd, &bits[3], sizeof(vd));
    if (!isfinite(vd)) {
        ce_status st = reject();
        return st != CE_EINVAL ? st : fail(CE_EINVAL, "initial derivatives are not finite");
    }
    double m2max = 0.0;
    for (int i = 0; i < s->p.nfields; i++) {
        if (!isfinite(M[i])) {
            ce_status st = reject();
            return st != CE_EINVAL ? st : fail(CE_EINVAL, "initial field %d is not finite", i);
        }
    }
    const int nf = s->p.nfields;
    for (int i = 0; i < nf; i++) {
        double m2;
        if (s->p.model == CE_MODEL_POLYNOMIAL) {
            // Gershgorin bound on the Hessian of V at |f_j| <= M_j (a = 1):
            // row i sums |d^2 V / df_i df_j| over j, term by term
            m2 = 0.0;
            const Lattice &L = s->lat;
            for (int t = 0; t < L.nterms; t++) {
                const double c = fabs(L.tcoef[t]);
                for (int j = 0; j < nf; j++) {
                    const int ei = L.texp[t][i], ej = L.texp[t][j];
                    double h = c;
                    for (int k = 0; k < nf; k++) {
                        int e = L.texp[t][k];
                        if (k == i) {
                            h *= (double)e;
                            e -= 1;
                        }
                        if (k == j) {
                            h *= (double)(k == i ? ei - 1 : ej);
                            e -= 1;
                        }
                        if (e < 0) {
                            h = 0.0;
                            break;
                        }
                        for (int q = 0; q < e; q++) h *= M[k];
                    }
                    m2 += h;
                }
            }
        } else if (i == 0) {
            m2 = 3.0 * s->p.lambda * M[0] * M[0] + s->p.mu2[0];
            for (int j = 1; j < nf; j++) m2 += s->p.G[j] * M[j] * M[j];
        } else {
            m2 = s->p.G[i] * M[0] * M[0] + s->p.mu2[i];
        }
        m2max = std::max(m2max, m2);
    }
    const double dx = s->p.L / s->p.N;
    const double w = s->p.dt * sqrt(4.0 * s->p.dims / (dx * dx) + m2max);
    if (!(w < 2.0)) {
        ce_status st = reject();
        return st != CE_EINVAL ? st
                               : fail(CE_EINVAL, "leapfrog unstable for these fields: dt*sqrt(4d/dx^2 + m^2_max) = %g >= 2", w);
    }
    CE_HIP(launch_pass(s->lat, s->p.precision, s->cur, kInit, s->stream));
    s->started = true;
    s->step = 0;
    return CE_OK;
}

}  // namespace host
}  // namespace ce

extern "C" {

ce_status ce_set_step_block(ce_sim *s, int32_t k)
{
    if (!s) return fail(CE_EINVAL, "sim is NULL");
    if (k < 0 || k > 4096) return fail(CE_EINVAL, "step block must be 0..4096");
    if (k != s->step_block) drop_graphs(s);
    s->step_block = k;
    return CE_OK;
}

ce_status ce_set_wait_limit(ce_sim *s, double ms)
{
    if (!s) return fail(CE_EINVAL, "sim is NULL");
    if (!(ms >= 0.0) || ms > 1e6) return fail(CE_EINVAL, "wait limit must be 0..1e6 ms");
    s->wait = (unsigned long long)(ms * (double)kTicksPerMs);
    return CE_OK;
}

ce_status ce_step(ce_sim *s, int64_t nsteps)
{
    const Use use;
    if (!s) return fail(CE_EINVAL, "sim is NULL");
    if (nsteps < 0) return fail(CE_EINVAL, "nsteps must be >= 0");
    if (!s->started) return fail(CE_ESTATE, "load every field before stepping");
    long long left = nsteps;
    // A resident pass takes the steps of a call where they are enough to pay
    // for its launch.  Plain launches (step block 0) and captured streams take
    // the steps one by one; the results are the same.
    if (s->step_block > 0 && left > 1 && (!s->resident_planned || s->resident.kernel)) {
        hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
        CE_HIP(hipStreamIsCapturing(s->stream, &cap));
        const bool free = cap == hipStreamCaptureStatusNone;
        if (free && !s->resident_planned) plan_resident(s);
        while (free && s->resident.kernel && left >= s->resident.min_steps) {
            const Alone alone;
            if (!alone && s->resident.blocks > 1) break;
            int n = (int)std::min<long long>(left, kResidentSteps);
            if (launch_resident(s, n) != hipSuccess) {
                // refused, nothing queued: plain launches until the next plan
                (void)hipGetLastError();
                s->resident = ce_sim::Resident{};
                break;
            }
            left -= n;
        }
    }
    if (s->step_block > 0) {
        while (left >= s->step_block) {
            if (!s->graph[s->cur]) {
                ce_status st = build_graph(s, s->cur);
                if (st != CE_OK) return st;
            }
            CE_HIP(hipGraphLaunch(s->graph[s->cur], s->stream));
            s->cur = (s->cur + s->step_block) & 1;
            s->step += s->step_block;
            left -= s->step_block;
        }
    }
    // behind a resident launch that may have left the state halted
    const Mode mode = s->unsettled ? kGuardedStep : kStep;
    if (left > 0 && mode == kGuardedStep && !guarded_built(s->lat, s->p.precision))
        return fail(CE_ESTATE, "launch set under capture behind steps not waited for: wait for the simulation first");
    for (; left > 0; left--) {
        CE_HIP(launch_pass(s->lat, s->p.precision, s->cur, mode, s->stream));
        s->cur ^= 1;
        s->step += 1;
    }
    return CE_OK;
}

ce_status ce_time_steps(ce_sim *s, int64_t nsteps, float *ms)
{
    const Use use;
    if (!s || !ms) return fail(CE_EINVAL, "NULL argument");
    hipEvent_t e0 = nullptr, e1 = nullptr;
    CE_HIP(hipEventCreate(&e0));
    hipError_t err = hipEventCreate(&e1);
    if (err != hipSuccess) {
        (void)hipEventDestroy(e0);
        return fail(CE_EDEVICE, "hipEventCreate failed: %s", hipGetErrorString(err));
    }
    ce_status st = CE_OK;
    err = hipEventRecord(e0, s->stream);
    if (err == hipSuccess) {
        st = ce_step(s, nsteps);
        if (st == CE_OK) err = hipEventRecord(e1, s->stream);
        if (st == CE_OK && err == hipSuccess) err = hipEventSynchronize(e1);
        if (st == CE_OK && err == hipSuccess) err = hipEventElapsedTime(ms, e0, e1);
        if (st == CE_OK && err == hipSuccess) st = settle(s);
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (st != CE_OK) return st;
    if (err != hipSuccess) return fail(CE_EDEVICE, "event timing failed: %s", hipGetErrorString(err));
    return CE_OK;
}

ce_status ce_sync(ce_sim *s)
{
    const Use use;
    if (!s) return fail(CE_EINVAL, "sim is NULL");
    CE_HIP(hipStreamSynchronize(s->stream));
    return settle(s);
}

ce_status ce_get_step(const ce_sim *s, int64_t *step)
{
    if (!s || !step) return fail(CE_EINVAL, "NULL argument");
    *step = s->step;
    return CE_OK;
}

ce_status ce_energies(ce_sim *s, ce_energy *out)
{
    const Use use;
    if (!s || !out) return fail(CE_EINVAL, "NULL argument");
    if (!s->started) return fail(CE_ESTATE, "no diagnostics before every field is loaded");
    CE_HIP(hipStreamSynchronize(s->stream));
    {
        const ce_status st = settle(s);
        if (st != CE_OK) return st;
    }
    CE_HIP(hipMemcpy(out, s->lat.ring + (s->step % kLogCap), sizeof(ce_energy), hipMemcpyDeviceToHost));
    Scalars sc;
    CE_HIP(hipMemcpy(&sc, s->lat.sc, sizeof(sc), hipMemcpyDeviceToHost));
    if (sc.halted != kRuns)
        return fail(CE_EDEVICE, "a resident launch lost its blocks' sums by step %lld: the state is lost", sc.step);
    if (out->step != s->step)
        return fail(CE_EDEVICE, "diagnostics record for step %lld holds step %lld", (long long)s->step,
                    (long long)out->step);
    if (sc.first_bad >= 0)
        return fail(CE_ENONFINITE, "non-finite volume sum first at step %lld", sc.first_bad);
    return CE_OK;
}

ce_status ce_energy_log(ce_sim *s, int32_t count, ce_energy *out)
{
    const Use use;
    if (!s || !out) return fail(CE_EINVAL, "NULL argument");
    if (!s->started) return fail(CE_ESTATE, "no diagnostics before every field is loaded");
    if (count < 1 || count > kLogCap || count > s->step + 1)
        return fail(CE_EINVAL, "count must be 1..min(%d, step+1)", kLogCap);
    CE_HIP(hipStreamSynchronize(s->stream));
    {
        const ce_status st = settle(s);
        if (st != CE_OK) return st;
    }
    const long long first = s->step - count + 1;
    for (int k = 0; k < count;) {
        const long long idx = (first + k) % kLogCap;
        const int run = (int)std::min<long long>(count - k, kLogCap - idx);
        CE_HIP(hipMemcpy(out + k, s->lat.ring + idx, (size_t)run * sizeof(ce_energy),
                         hipMemcpyDeviceToHost));
        k += run;
    }
    return CE_OK;
}

static ce_status read_fields(ce_sim *s, double *f, double *fdot)
{
    const long long ns = s->lat.nsites;
    const long long chunk = s->lay.staging_elems / 2;  // f and fdot share the staging block
    for (int i = 0; i < s->p.nfields; i++) {
        for (long long off = 0; off < ns; off += chunk) {
            const long long n = std::min(chunk, ns - off);
            double *df = s->staging;
            double *dp = s->staging + chunk;
            CE_HIP(launch_readback(s->lat, s->p.precision, s->cur, i, s->started ? 1 : 0, off, nullptr, n,
                                   f ? df : nullptr, fdot ? dp : nullptr, s->stream));
            if (f)
                CE_HIP(hipMemcpyAsync(f + (long long)i * ns + off, df, (size_t)n * sizeof(double),
                                      hipMemcpyDeviceToHost, s->stream));
            if (fdot)
                CE_HIP(hipMemcpyAsync(fdot + (long long)i * ns + off, dp, (size_t)n * sizeof(double),
                                      hipMemcpyDeviceToHost, s->stream));
            CE_HIP(hipStreamSynchronize(s->stream));
        }
    }
    return CE_OK;
}

ce_status ce_read_fields(ce_sim *s, double *f, double *fdot)
{
    const Use use;
    if (!s) return fail(CE_EINVAL, "sim is NULL");
    if (s->loaded != (1u << s->p.nfields) - 1) return fail(CE_ESTATE, "fields not loaded");
    const ce_status st = read_fields(s, f, fdot);
    if (st != CE_OK || !halt_seen(s)) return st;
    // the steps before it had not all been taken
    const ce_status st2 = settle(s);
    return st2 != CE_OK ? st2 : read_fields(s, f, fdot);
}

ce_status ce_read_sites(ce_sim *s, int32_t field, int64_t count, const int64_t *sites, double *f,
                        double *fdot)
{
    const Use use;
    if (!s) return fail(CE_EINVAL, "sim is NULL");
    if (s->loaded != (1u << s->p.nfields) - 1) return fail(CE_ESTATE, "fields not loaded");
    if (field < 0 || field >= s->p.nfields) return fail(CE_EINVAL, "field %d out of range", field);
    const long long per = s->lay.staging_elems / 3;
    if (count < 0 || count > (1LL << 20) || count > per)
        return fail(CE_EINVAL, "count must be 0..%lld", std::min(per, 1LL << 20));
    if (count == 0) return CE_OK;
    if (!sites) return fail(CE_EINVAL, "sites is NULL");
    const long long ns = s->lat.nsites;
    for (long long i = 0; i < count; i++)
        if (sites[i] < 0 || sites[i] >= ns) return fail(CE_EINVAL, "site %lld out of range", (long long)sites[i]);
    long long *dsites = reinterpret_cast<long long *>(s->staging);
    double *df = s->staging + per;
    double *dp = s->staging + 2 * per;
    CE_HIP(hipMemcpyAsync(dsites, sites, (size_t)count * sizeof(long long), hipMemcpyHostToDevice, s->stream));
    CE_HIP(launch_readback(s->lat, s->p.precision, s->cur, field, s->started ? 1 : 0, 0, dsites, count,
                           f ? df : nullptr, fdot ? dp : nullptr, s->stream));
    if (f) CE_HIP(hipMemcpyAsync(f, df, (size_t)count * sizeof(double), hipMemcpyDeviceToHost, s->stream));
    if (fdot) CE_HIP(hipMemcpyAsync(fdot, dp, (size_t)count * sizeof(double), hipMemcpyDeviceToHost, s->stream));
    CE_HIP(hipStreamSynchronize(s->stream));
    if (!halt_seen(s)) return CE_OK;
    // the steps before it had not all been taken
    const ce_status st = settle(s);
    return st != CE_OK ? st : ce_read_sites(s, field, count, sites, f, fdot);
}

ce_status ce_release_memory(void)
{
    const Use use;
    give_back_kept_memory();
    return CE_OK;
}

void ce_destroy(ce_sim *s)
{
    const Use use;
    if (!s) return;
    // memory is kept only if everything that used it is known to have ended:
    // steps captured on the stream may be running from a graph on another one
    bool idle = s->stream && hipStreamSynchronize(s->stream) == hipSuccess;
    if (s->own_mem && idle) idle = hipDeviceSynchronize() == hipSuccess;
    drop_graphs(s);
    if (s->cap_stream) (void)hipStreamDestroy(s->cap_stream);
    if (s->own_stream && s->stream) (void)hipStreamDestroy(s->stream);
    if (s->own_mem && s->base) {
        if (idle)
            release_device_memory(s->base, s->lay.total, s->device);
        else
            (void)hipFree(s->base);
    }
    if (idle) give_halt_word(s->halt);   // else a launch may still write it
    delete s;
}

}  // extern "C"
