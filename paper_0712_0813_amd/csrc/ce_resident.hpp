// Shared by the resident passes: kernels that keep a lattice's state on the
// chip over many steps of one launch.
//
// A small lattice's step is latency: launching, loading the scalar state and
// the sites, reducing the volume sums and running the tail take longer than
// the sites do.  A resident pass launches once for a run of steps.  Each block
// owns a fixed part of the lattice and keeps its d and p in registers; per
// step the blocks exchange the sites their neighbours need through the
// lattice's own ping-pong buffers, and their FP64 partial sums through `sync`.
// Every block then forms the same totals in the same order and runs the same
// FP64 tail, so the coefficients of the next step need no second exchange.
//
// Exchange.  All shared words move with agent-scope accesses (written through
// to, and read from, the memory side of the XCDs' caches), so no cache is
// flushed.  Within a step a block stores its boundary sites, waits until they
// have arrived, and then publishes its sums: a reader that has seen a block's
// sums of step n may read its boundary of step n.  A sum is published as two
// 64-bit words, each half of the value with the step's tag, so seeing the tag
// is seeing the value: there is no separate flag and no second round trip.
// Two sets of words alternate, as the two buffers do for the boundary: a block
// publishes step n+2 only after it has the totals of n+1, hence after every
// block has published n+1, hence after every block has read what was published
// of step n.
//
// Two hops: block q < NQ adds up sum q of every block and publishes the total,
// once for each eighth of the blocks (kTotalCopies), and every block waits for
// the totals alone.  What costs is many waves polling a few lines, which holds
// up the stores that would end the wait: with every block reading every
// block's sums, and every wave waiting for its neighbours', the exchange took
// 2.6 us at 32 blocks and 11 us at 256.  A launch of fewer blocks than sums
// does read every block's.
//
// Waiting.  Blocks wait for each other, so every block of the launch must be
// resident at once: the launch is cooperative, and the host offers it only
// when the occupancy query says the grid fits.  That query counts an empty GPU:
// a long kernel of another stream or another process's grid may hold units.  So
// the blocks check in before the first step, and only when all have (all run,
// and none is taken off its unit before it ends) does the launch start.  When
// they have not in Start::wait, they agree to leave, with nothing written but
// Scalars::halted, and the host takes the steps by plain launches.
// A wait of a started launch is bounded as well: past kSpinLimit polls (seconds;
// a step takes microseconds) the block takes the sums as NaN, waits no more and
// leaves kLost in Scalars::halted, which the host reports as a device error.
#pragma once

#include "ce_device.hpp"

namespace ce {
namespace dev {

constexpr int kSpinLimit = 1 << 22;

// Cache-policy bits of an agent-scope buffer access on gfx950: sc1.
constexpr int kAgentPolicy = 16;

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ __amdgpu_buffer_rsrc_t agent_buffer(void *base)
{
    // raw buffer: stride 0, num_records in bytes, gfx9 dword3 (32-bit data);
    // resident lattices are far below 2 GiB an array
    return __builtin_amdgcn_make_buffer_rsrc(base, (short)0, 0x7ffffff0, 0x00020000);
}

// Agent-scope access to the quad (4 sites) at byte offset o.
__device__ __forceinline__ Quad<float> agent_load_quad(__amdgpu_buffer_rsrc_t b, unsigned o, float)
{
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(b, (int)o, 0, kAgentPolicy);
    return Quad<float>{{__uint_as_float(v.x), __uint_as_float(v.y), __uint_as_float(v.z), __uint_as_float(v.w)}};
}
__device__ __forceinline__ double from_words(unsigned lo, unsigned hi)
{
    return __longlong_as_double(((long long)hi << 32) | lo);
}
__device__ __forceinline__ Quad<double> agent_load_quad(__amdgpu_buffer_rsrc_t b, unsigned o, double)
{
    const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(b, (int)o, 0, kAgentPolicy);
    const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(b, (int)o + 16, 0, kAgentPolicy);
    return Quad<double>{{from_words(v.x, v.y), from_words(v.z, v.w), from_words(w.x, w.y), from_words(w.z, w.w)}};
}
__device__ __forceinline__ float agent_load(__amdgpu_buffer_rsrc_t b, unsigned o, float)
{
    return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, (int)o, 0, kAgentPolicy));
}
__device__ __forceinline__ double agent_load(__amdgpu_buffer_rsrc_t b, unsigned o, double)
{
    const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(b, (int)o, 0, kAgentPolicy);
    return from_words(v.x, v.y);
}
__device__ __forceinline__ void agent_store(__amdgpu_buffer_rsrc_t b, unsigned o, float v)
{
    __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), b, (int)o, 0, kAgentPolicy);
}
__device__ __forceinline__ void agent_store(__amdgpu_buffer_rsrc_t b, unsigned o, double d)
{
    const long long bits = __double_as_longlong(d);
    const u32x2 v = {(unsigned)(bits & 0xffffffffLL), (unsigned)(bits >> 32)};
    __builtin_amdgcn_raw_buffer_store_b64(v, b, (int)o, 0, kAgentPolicy);
}
__device__ __forceinline__ void agent_store(__amdgpu_buffer_rsrc_t b, unsigned o, const float (&q)[4])
{
    const u32x4 v = {__float_as_uint(q[0]), __float_as_uint(q[1]), __float_as_uint(q[2]), __float_as_uint(q[3])};
    __builtin_amdgcn_raw_buffer_store_b128(v, b, (int)o, 0, kAgentPolicy);
}
__device__ __forceinline__ void agent_store(__amdgpu_buffer_rsrc_t b, unsigned o, const double (&q)[4])
{
    unsigned w[8];
#pragma unroll
    for (int e = 0; e < 4; e++) {
        const long long bits = __double_as_longlong(q[e]);
        w[2 * e] = (unsigned)(bits & 0xffffffffLL);
        w[2 * e + 1] = (unsigned)(bits >> 32);
    }
    const u32x4 v = {w[0], w[1], w[2], w[3]}, u = {w[4], w[5], w[6], w[7]};
    __builtin_amdgcn_raw_buffer_store_b128(v, b, (int)o, 0, kAgentPolicy);
    __builtin_amdgcn_raw_buffer_store_b128(u, b, (int)o + 16, 0, kAgentPolicy);
}

__device__ __forceinline__ void store_lds(float *p, const float (&q)[4])
{
    f32x4 v = {q[0], q[1], q[2], q[3]};
    *reinterpret_cast<f32x4 *>(p) = v;
}
__device__ __forceinline__ void store_lds(double *p, const double (&q)[4])
{
    f64x2 a = {q[0], q[1]}, b = {q[2], q[3]};
    reinterpret_cast<f64x2 *>(p)[0] = a;
    reinterpret_cast<f64x2 *>(p)[1] = b;
}
__device__ __forceinline__ void load_lds(const float *p, float (&q)[4])
{
    const f32x4 v = *reinterpret_cast<const f32x4 *>(p);
    q[0] = v.x, q[1] = v.y, q[2] = v.z, q[3] = v.w;
}
__device__ __forceinline__ void load_lds(const double *p, double (&q)[4])
{
    const f64x2 a = reinterpret_cast<const f64x2 *>(p)[0], b = reinterpret_cast<const f64x2 *>(p)[1];
    q[0] = a.x, q[1] = a.y, q[2] = b.x, q[3] = b.y;
}

// The same for VEC sites.
template <typename T, int VEC>
__device__ __forceinline__ Vec<T, VEC> agent_load_vec(__amdgpu_buffer_rsrc_t b, unsigned o)
{
    Vec<T, VEC> v;
    if constexpr (VEC == 4) {
        const Quad<T> q = agent_load_quad(b, o, T());
#pragma unroll
        for (int e = 0; e < 4; e++) v.v[e] = q.v[e];
    } else {
        static_assert(VEC == 2 && sizeof(T) == 8, "pairs are built for FP64");
        const u32x4 w = __builtin_amdgcn_raw_buffer_load_b128(b, (int)o, 0, kAgentPolicy);
        v.v[0] = from_words(w.x, w.y);
        v.v[1] = from_words(w.z, w.w);
    }
    return v;
}
__device__ __forceinline__ void agent_store(__amdgpu_buffer_rsrc_t b, unsigned o, const double (&q)[2])
{
    const long long x = __double_as_longlong(q[0]), y = __double_as_longlong(q[1]);
    const u32x4 v = {(unsigned)(x & 0xffffffffLL), (unsigned)(x >> 32), (unsigned)(y & 0xffffffffLL), (unsigned)(y >> 32)};
    __builtin_amdgcn_raw_buffer_store_b128(v, b, (int)o, 0, kAgentPolicy);
}
__device__ __forceinline__ void store_lds(double *p, const double (&q)[2])
{
    f64x2 a = {q[0], q[1]};
    *reinterpret_cast<f64x2 *>(p) = a;
}
__device__ __forceinline__ void load_lds(const double *p, double (&q)[2])
{
    const f64x2 a = *reinterpret_cast<const f64x2 *>(p);
    q[0] = a.x, q[1] = a.y;
}

// Wait until every store this wave has issued has arrived.
__device__ __forceinline__ void stores_arrived()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_waitcnt(0);
}

// Word j of row r of the sums published for step `tag`: one column of
// kSyncRows rows per word, so that a wavefront reading 64 rows reads
// contiguous memory.
__device__ __forceinline__ unsigned long long *sync_word(const Lattice &lat, int j, int row, unsigned tag)
{
    return lat.sync + (long long)((tag & 1u) * (2 * kMaxSums) + j) * kSyncRows + row;
}

// Publish the block's totals (lane q: sum q) as row `row` of step `tag`.  The
// boundary stores of every wave have arrived (stores_arrived before the last
// barrier).
template <int NQ>
__device__ __forceinline__ void publish_row(const Lattice &lat, double tot, int row, unsigned tag)
{
    const int lane = __lane_id();
    if (lane < NQ) {
        const long long bits = __double_as_longlong(tot);
        const unsigned long long t = (unsigned long long)tag << 32;
        __hip_atomic_store(sync_word(lat, 2 * lane, row, tag), t | (unsigned)(bits & 0xffffffffLL), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(sync_word(lat, 2 * lane + 1, row, tag), t | (unsigned)(bits >> 32), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    }
}

// Sums of row `row` at step `tag`, waited for.  alive: cleared when a wait
// ran out; the sums are NaN from then on.
template <int NQ>
__device__ __forceinline__ void collect_row(const Lattice &lat, int row, unsigned tag, double (&acc)[NQ], bool &alive)
{
    unsigned long long w[2 * NQ];
    bool seen = false;
    for (int spin = 0; alive && !seen && spin < kSpinLimit; spin++) {
        unsigned miss = 0;
#pragma unroll
        for (int j = 0; j < 2 * NQ; j++)
            w[j] = __hip_atomic_load(sync_word(lat, j, row, tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
        for (int j = 0; j < 2 * NQ; j++) miss |= (unsigned)(w[j] >> 32) ^ tag;
        seen = miss == 0;
    }
    alive = alive && seen;
#pragma unroll
    for (int q = 0; q < NQ; q++) acc[q] = seen ? from_words((unsigned)w[2 * q], (unsigned)w[2 * q + 1]) : __builtin_nan("");
}

// The value lane `lane` holds, in every lane.
__device__ __forceinline__ float lane_copy(float v, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), lane));
}
__device__ __forceinline__ double lane_copy(double v, int lane)
{
    const long long b = __double_as_longlong(v);
    return from_words((unsigned)__builtin_amdgcn_readlane((int)(b & 0xffffffffLL), lane),
                      (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), lane));
}

// Coefficients of the next pass from the scalars the tail left in LDS; the
// model's constants in c stay.
template <typename T, int NF, int MODEL>
__device__ __forceinline__ void next_coef(PassCoef<T, NF> &c, const PassScalars<T> &ps)
{
#pragma unroll
    for (int i = 0; i < NF; i++) {
        c.cf[i].beta = uniform(ps.beta);
        c.cf[i].bm = uniform(ps.bm[i]);
        c.cf[i].r = uniform(ps.r[i]);
        c.cf[i].m1 = uniform(ps.m1[i]);
        c.m2a[i] = uniform(ps.m2a[i]);
        c.hm[i] = uniform(ps.hm[i]);
    }
    if constexpr (MODEL == kPoly) {
#pragma unroll
        for (int t = 0; t < kMaxTerms; t++) c.tc[t] = uniform(ps.tc[t]);
    }
}

// The tag of the last step a resident pass took, after the totals.  Block 0
// writes it when it has every block's last step, so every block has read it.
__device__ __forceinline__ unsigned long long *last_tag(const Lattice &lat)
{
    return lat.sync + kLastTag;
}

// Word j of copy c of the totals of step `tag`, after the rows.
__device__ __forceinline__ unsigned long long *total_word(const Lattice &lat, int c, int j, unsigned tag)
{
    return lat.sync + (long long)2 * (2 * kMaxSums) * kSyncRows + ((tag & 1u) * kTotalCopies + c) * kTotalWords + j;
}

__device__ __forceinline__ int halted(const Lattice &lat)
{
    return __hip_atomic_load(&lat.sc->halted, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// Leave the lattice halted, for the host to see once the launch has ended.
__device__ __forceinline__ void halt(const Lattice &lat, int why, const Start &start)
{
    __hip_atomic_store(&lat.sc->halted, why, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(start.halt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
}

// The blocks of a launch that have checked in, and whether they were told to leave.
__device__ __forceinline__ unsigned long long *arrivals(const Lattice &lat) { return lat.sync + kArrivals; }
constexpr unsigned long long kNoStart = 1ull << 32;   // in the word of arrivals

// What a launch's blocks made of their check-in.
enum { kGo = 0, kLeave = 1, kLeaveAndHalt = 2 };   // the last: one block's, which halts the lattices

// One thread of each of the nblk blocks that work together.  They go when all
// have arrived.  A block that has waited long enough marks the word, but only
// while some are missing: so it says either that all came or that none goes,
// also to blocks that come to run only when the others have left, and to later
// launches, until the host clears it.  After a start the launch clears it.
// (One round trip to memory, while the state loads: 2 us a launch; with
// arrivals and decision in words of their own 4.)
__device__ __forceinline__ int check_in(const Lattice &lat, int nblk, const Start &start)
{
    unsigned long long *word = arrivals(lat);
    const unsigned long long all = (unsigned long long)nblk;
    if (start.wait == 0)   // no block arrives
        return __hip_atomic_fetch_or(word, kNoStart, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < kNoStart ? kLeaveAndHalt
                                                                                                       : kLeave;
    unsigned long long w = __hip_atomic_fetch_add(word, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) + 1;
    const unsigned long long t0 = wall_clock64();
    while (w < all && wall_clock64() - t0 < start.wait) {
        __builtin_amdgcn_s_sleep(1);
        w = __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    // (each failed exchange has seen another arrival or the mark)
    while (w < all)
        if (__hip_atomic_compare_exchange_strong(word, &w, w | kNoStart, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                 __HIP_MEMORY_SCOPE_AGENT))
            return kLeaveAndHalt;
    return w == all ? kGo : kLeave;
}

// Whether the launch starts, the same in every thread of the block and every
// block of the lattice; every thread calls it, once.
__device__ __forceinline__ bool launch_starts(const Lattice &lat, int nblk, const Start &start)
{
    __shared__ int go;
    if (threadIdx.x == blockDim.x - 64) {   // of the service wave, which has nothing else to do yet
        const int r = nblk > 1 ? check_in(lat, nblk, start) : halted(lat) == kRuns ? kGo : kLeave;
        if (r == kLeaveAndHalt) halt(lat, kNotStarted, start);
        go = r == kGo;
    }
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(go) != 0;
}

// One wavefront: sum q over the nblk <= kSyncRows = 256 published rows, in the
// order of finish_pass (lane trees over 64 rows each, those in order).
__device__ __forceinline__ double sum_rows(const Lattice &lat, int q, int nblk, unsigned tag, bool &alive)
{
    static_assert(kSyncRows == 256, "four rows a lane");
    const int lane = __lane_id();
    unsigned long long w[8];
    bool seen = false;
    for (int spin = 0; alive && !seen && spin < kSpinLimit; spin++) {
        unsigned miss = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            const int row = lane + 64 * k;
#pragma unroll
            for (int h = 0; h < 2; h++)
                w[2 * k + h] = row < nblk ? __hip_atomic_load(sync_word(lat, 2 * q + h, row, tag), __ATOMIC_RELAXED,
                                                              __HIP_MEMORY_SCOPE_AGENT)
                                          : (unsigned long long)tag << 32;
        }
#pragma unroll
        for (int j = 0; j < 8; j++) miss |= (unsigned)(w[j] >> 32) ^ tag;
        seen = __ballot(miss != 0) == 0;
    }
    alive = alive && seen;
    double v[4];
#pragma unroll
    for (int k = 0; k < 4; k++) v[k] = seen ? from_words((unsigned)w[2 * k], (unsigned)w[2 * k + 1]) : __builtin_nan("");
    const double s = tree_sum<5, 4>(v);   // lanes 0, 16, 32, 48: the four trees
    return ((lane_copy(s, 0) + lane_copy(s, 16)) + lane_copy(s, 32)) + lane_copy(s, 48);
}

// One wavefront: the totals over every block's row of step `tag`; lane q
// receives sum q.
template <int NQ>
__device__ __forceinline__ double collect_totals(const Lattice &lat, int rank, int nblk, unsigned tag, double *scratch,
                                                 bool &alive)
{
    const int lane = __lane_id();
    const int q = min(lane, NQ - 1);
    if (nblk < NQ) {
        double acc[NQ];
        if (lane < nblk) {
            collect_row<NQ>(lat, lane, tag, acc, alive);
        } else {
#pragma unroll
            for (int k = 0; k < NQ; k++) acc[k] = 0.0;
        }
        const double v = tree_sum<5, NQ>(acc);
        const int k = tree_index<NQ>();
        if (k >= 0) scratch[k] = v;
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const double tot = scratch[q];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        return tot;
    }
    const unsigned long long t = (unsigned long long)tag << 32;
    if (rank < NQ) {
        const long long bits = __double_as_longlong(sum_rows(lat, rank, nblk, tag, alive));
        if (lane < 2 * kTotalCopies)
            __hip_atomic_store(total_word(lat, lane >> 1, 2 * rank + (lane & 1), tag),
                               t | ((lane & 1) ? (unsigned)(bits >> 32) : (unsigned)(bits & 0xffffffffLL)),
                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    unsigned long long lo = t, hi = t;
    bool seen = false;
    const int copy = rank % kTotalCopies;
    for (int spin = 0; alive && !seen && spin < kSpinLimit; spin++) {
        lo = __hip_atomic_load(total_word(lat, copy, 2 * q, tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        hi = __hip_atomic_load(total_word(lat, copy, 2 * q + 1, tag), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        seen = __ballot((((unsigned)(lo >> 32) ^ tag) | ((unsigned)(hi >> 32) ^ tag)) != 0) == 0;
    }
    alive = alive && seen;
    return seen ? from_words((unsigned)lo, (unsigned)hi) : __builtin_nan("");
}

// The wave after those that work the sites: it publishes the block's sums and
// runs the tail, so neither holds up a wave's sites nor needs registers beside
// them.  The block's row is made of GROUPS rows of the plain pass, each of
// WAVES wavefronts' sums in order (red), those in order.  Barriers per step,
// matched by the other waves: (1) the step's drifted sites are in LDS, (2) the
// waves' sums are in red and their boundary stores have arrived, (3; several
// blocks) every block has published the step, so its boundary may be read, (4)
// the next pass's coefficients are in `next`.
// The block is the `rank`-th of the nblk that work the lattice.
template <typename T, int NF, int GROUPS, int WAVES>
__device__ __forceinline__ void service_wave(const Lattice &lat, int steps, int rank, int nblk, int row,
                                             const double (*red)[kMaxSums], PassScalars<T> &next, const Start &start)
{
    constexpr int NQ = kSumsPerField * NF + 1;
    __shared__ double scratch[2 * kMaxSums];
    const int lane = threadIdx.x & 63;
    const int q = min(lane, NQ - 1);
    bool alive = true;
    LaneTail<T, NF> tail;
    tail.load(lat);
    const unsigned epoch = (unsigned)*last_tag(lat);
    for (int step = 0; step < steps; step++) {
        const unsigned tag = epoch + (unsigned)step + 1u;
        tail.prepare(lat);
        __syncthreads();   // (1)
        __syncthreads();   // (2)
        double tot = 0.0;
#pragma unroll
        for (int v = 0; v < GROUPS; v++) {
            double r = red[WAVES * v][q];
#pragma unroll
            for (int w = 1; w < WAVES; w++) r += red[WAVES * v + w][q];
            tot = GROUPS == 1 ? r : tot + r;
        }
        if (nblk > 1) {
            publish_row<NQ>(lat, tot, row, tag);
            tot = collect_totals<NQ>(lat, rank, nblk, tag, scratch, alive);
            __syncthreads();   // (3)
        }
        tail.solve(lat, tot, scratch);
        tail.next_pass(lat, next);
        __syncthreads();   // (4)
        if (rank == 0) tail.record(lat);
        tail.advance();
    }
    if (__ballot(!alive) != 0 && lane == 0) halt(lat, kLost, start);
    if (rank == 0) {
        // every block has published its last step, hence gone past its check-in
        if (lane == 0) __hip_atomic_store(arrivals(lat), 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        tail.store(lat);
        if (lane == 0) {
            lat.sc->cur ^= steps & 1;
            if (lat.sc->remaining > 0) lat.sc->remaining -= min((long long)steps, lat.sc->remaining);
            *last_tag(lat) = epoch + (unsigned)steps;
        }
    }
}

// A pool's resident launch: up to k steps of each of n lattices that nblk
// blocks work.  The grid's blocks form groups of nblk; group g takes lattices
// g, g + groups, ... one after the other, each for all its steps.  A group checks
// in at the first of them that has steps to take; one that does not start leaves
// all those halted, with no steps to take.
template <typename Body>
__device__ __forceinline__ void run_members(const Lattice *lats, int n, int nblk, int k, const Start &start, Body body)
{
    const int rank = blockIdx.x % nblk, groups = gridDim.x / nblk;
    auto member = [&](int l) -> const Lattice & {
        return *(const Lattice *)((const __attribute__((address_space(4))) Lattice *)lats + l);
    };
    int l = blockIdx.x / nblk;
    if (nblk > 1) {
        __shared__ int go;
        while (l < n && member(l).sc->remaining <= 0) l += groups;
        if (l >= n) return;
        if (threadIdx.x == blockDim.x - 64) {
            const int r = check_in(member(l), nblk, start);
            if (r == kLeaveAndHalt)
                for (int m = l; m < n; m += groups)
                    if (member(m).sc->remaining > 0) {
                        halt(member(m), kNotStarted, start);
                        member(m).sc->remaining = 0;
                    }
            go = r == kGo;
        }
        __syncthreads();
        if (!__builtin_amdgcn_readfirstlane(go)) return;
    }
    for (; l < n; l += groups) {
        const Lattice &lat = member(l);
        // the steps left and the buffer change only when every block of the
        // group has published the last step, so all read the same
        const int steps = (int)min((long long)k, lat.sc->remaining);
        if (steps <= 0) continue;
        body(lat, lat.sc->cur, steps, rank, nblk);
        __syncthreads();   // the next lattice takes over the block's LDS
    }
}

}  // namespace dev
}  // namespace ce
