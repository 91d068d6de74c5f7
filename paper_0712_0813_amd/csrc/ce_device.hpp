// Device helpers shared by the lattice kernels: vector loads, the one
// definition of the drift, FP64 block sums, and the FP64 tails that turn the
// volume sums of a pass into the scale-factor update and the diagnostics.
#pragma once

#include <math.h>

#include "ce_internal.hpp"

namespace ce {
namespace dev {

// Pointers into device memory, typed as global so loads and stores compile to
// global_* instructions (generic pointers taken from a struct would become
// flat_* accesses, which share the LDS wait counter).
template <typename T>
using gptr = __attribute__((address_space(1))) T *;
template <typename T>
using gcptr = const __attribute__((address_space(1))) T *;

template <typename T>
__device__ __forceinline__ gptr<T> as_global(void *p)
{
    return (gptr<T>)p;
}

template <typename T>
struct Quad {
    T v[4];
};

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef double f64x2 __attribute__((ext_vector_type(2)));

// VEC consecutive x sites of one array.
template <typename T, int VEC>
struct Vec {
    T v[VEC];
};

__device__ __forceinline__ Vec<float, 2> load_vec2(gcptr<float> base, long long s)
{
    const f32x2 q = *(gcptr<f32x2>)(base + s);
    return Vec<float, 2>{{q.x, q.y}};
}
__device__ __forceinline__ Vec<double, 2> load_vec2(gcptr<double> base, long long s)
{
    const f64x2 q = *(gcptr<f64x2>)(base + s);
    return Vec<double, 2>{{q.x, q.y}};
}
// Stores of a pass's outputs: streaming (nontemporal), since nothing reads
// them again within the pass; this keeps L2 for the halo lines.
__device__ __forceinline__ void store_vec2(gptr<float> base, long long s, const Vec<float, 2> &q)
{
    f32x2 v;
    v.x = q.v[0];
    v.y = q.v[1];
    __builtin_nontemporal_store(v, (gptr<f32x2>)(base + s));
}
__device__ __forceinline__ void store_vec2(gptr<double> base, long long s, const Vec<double, 2> &q)
{
    f64x2 v;
    v.x = q.v[0];
    v.y = q.v[1];
    __builtin_nontemporal_store(v, (gptr<f64x2>)(base + s));
}

// Cache-policy bits of a buffer store on gfx950: sc0 (1) | nt (2) | sc1 (16).
constexpr int kStreamPolicy = 1 | 2 | 16;

__device__ __forceinline__ Quad<float> load_quad(gcptr<float> base, long long s)
{
    const f32x4 q = *(gcptr<f32x4>)(base + s);
    return Quad<float>{{q.x, q.y, q.z, q.w}};
}
__device__ __forceinline__ Quad<double> load_quad(gcptr<double> base, long long s)
{
    const f64x2 a = *(gcptr<f64x2>)(base + s);
    const f64x2 b = *(gcptr<f64x2>)(base + s + 2);
    return Quad<double>{{a.x, a.y, b.x, b.y}};
}
__device__ __forceinline__ void store_quad(gptr<float> base, long long s, const Quad<float> &q)
{
    f32x4 v;
    v.x = q.v[0];
    v.y = q.v[1];
    v.z = q.v[2];
    v.w = q.v[3];
    __builtin_nontemporal_store(v, (gptr<f32x4>)(base + s));
}
// Streaming store of 4 FP32 values at element s of a plane whose base is the
// same in every lane (s < 2^29): a buffer store with system scope and the
// nontemporal hint (sc0 sc1 nt), the policy for data written once and not
// read again by the same kernel; measured, it leaves more of L2 to the halo
// rows other tiles still have to read.  Results are those of store_quad;
// only the cache policy differs.
__device__ __forceinline__ void store_quad_stream(gptr<float> plane, unsigned s, const Quad<float> &q)
{
    typedef float f4_t __attribute__((ext_vector_type(4)));
    f4_t v;
    v.x = q.v[0];
    v.y = q.v[1];
    v.z = q.v[2];
    v.w = q.v[3];
    // raw buffer: stride 0, num_records in bytes, gfx9 dword3 (32-bit data)
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc((void *)plane, (short)0, 0x7ffffff0, 0x00020000);
    __builtin_amdgcn_raw_buffer_store_b128(v, rs, (int)(s * 4u), 0, kStreamPolicy);
}
__device__ __forceinline__ void store_quad(gptr<double> base, long long s, const Quad<double> &q)
{
    f64x2 a, b;
    a.x = q.v[0];
    a.y = q.v[1];
    b.x = q.v[2];
    b.y = q.v[3];
    __builtin_nontemporal_store(a, (gptr<f64x2>)(base + s));
    __builtin_nontemporal_store(b, (gptr<f64x2>)(base + s + 2));
}

__device__ __forceinline__ float fma_t(float a, float b, float c) { return __builtin_fmaf(a, b, c); }
__device__ __forceinline__ double fma_t(double a, double b, double c) { return __builtin_fma(a, b, c); }

// Per-field coefficients of one pass, in the storage type.
template <typename T>
struct FieldCoef {
    T beta;  // deferred c-term coefficient
    T bm;    // beta * m, rounded once
    T r;     // reference derivative
    T m1;    // reference field at n+1, rounded once (potential only)
};

// Derivative at n+1/2 and drifted deviation at n+1.  The one definition used
// for a site's own value and for every neighbour value, so both are bitwise
// identical.
template <typename T>
__device__ __forceinline__ T fdot_of(T d, T p, const FieldCoef<T> &c)
{
    return fma_t(c.beta, d, p) + c.bm;
}
template <typename T>
__device__ __forceinline__ T drift(T d, T p, const FieldCoef<T> &c, T dt)
{
    return fma_t(dt, fdot_of(d, p, c) - c.r, d);
}

// Value of `v` held by the lane below / above (whole-wave DPP shift by one;
// lane 0 / lane 63 receive 0).
__device__ __forceinline__ float lane_from_left(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x138, 0xF, 0xF, false));
}
__device__ __forceinline__ float lane_from_right(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x130, 0xF, 0xF, false));
}
__device__ __forceinline__ double lane_from_left(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), 0x138, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x138, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ double lane_from_right(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)(b & 0xffffffffLL), 0x130, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), 0x130, 0xF, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Work item of the j-th round of block b in a persistent grid of `grid`
// blocks over `nitems` items, -1 when done.  The hardware places block b on
// XCD b mod 8; when the grid and the item count are multiples of 8, each XCD
// takes one contiguous eighth of the items (neighbouring items share that
// XCD's L2), else items go round robin.
__device__ __forceinline__ long long xcd_item(int b, int j, int grid, long long nitems)
{
    if ((grid & 7) == 0 && (nitems & 7) == 0) {
        const long long per = nitems >> 3;
        const long long idx = (long long)(b >> 3) + (long long)j * (grid >> 3);
        return idx < per ? (long long)(b & 7) * per + idx : -1;
    }
    const long long t = (long long)b + (long long)j * grid;
    return t < nitems ? t : -1;
}

// ---- FP64 sums over a wavefront --------------------------------------------
// NQ sums are reduced together: at each of the six levels of the lane tree
// (lane pairs 32, 16, 8, 4, 2, 1 apart) the lanes of a pair exchange one half
// of the sums each, so a level halves the number of sums a lane holds.  13
// sums take 16 additions and 19 exchanges instead of the 78 of each a full
// butterfly per sum takes; the additions that form any one sum, and their
// order, are those of the butterfly.

// Value of the lane 2^BIT away.
template <int BIT>
__device__ __forceinline__ double lane_pair(double v)
{
    const long long b = __double_as_longlong(v);
    int lo = (int)(b & 0xffffffffLL), hi = (int)(b >> 32);
    if constexpr (BIT == 3) {          // rotate by 8 within 16 lanes
        lo = __builtin_amdgcn_update_dpp(0, lo, 0x128, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0x128, 0xF, 0xF, false);
    } else if constexpr (BIT == 2) {   // mirror 8 lanes, then mirror 4
        lo = __builtin_amdgcn_update_dpp(0, lo, 0x141, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0x141, 0xF, 0xF, false);
        lo = __builtin_amdgcn_update_dpp(0, lo, 0x1B, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0x1B, 0xF, 0xF, false);
    } else if constexpr (BIT == 1) {
        lo = __builtin_amdgcn_update_dpp(0, lo, 0x4E, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0x4E, 0xF, 0xF, false);
    } else {
        static_assert(BIT == 0, "wider pairs use the lane swaps");
        lo = __builtin_amdgcn_update_dpp(0, lo, 0xB1, 0xF, 0xF, false);
        hi = __builtin_amdgcn_update_dpp(0, hi, 0xB1, 0xF, 0xF, false);
    }
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Lanes with bit BIT clear: a plus the pair lane's a; lanes with it set: the
// same of b.
template <int BIT>
__device__ __forceinline__ double pair_add(double a, double b)
{
    if constexpr (BIT >= 4) {
        const long long ab = __double_as_longlong(a), bb = __double_as_longlong(b);
        const unsigned alo = (unsigned)(ab & 0xffffffffLL), ahi = (unsigned)(ab >> 32);
        const unsigned blo = (unsigned)(bb & 0xffffffffLL), bhi = (unsigned)(bb >> 32);
        unsigned l0, l1, h0, h1;
        if constexpr (BIT == 5) {
            const auto l = __builtin_amdgcn_permlane32_swap(alo, blo, false, false);
            const auto h = __builtin_amdgcn_permlane32_swap(ahi, bhi, false, false);
            l0 = l[0], l1 = l[1], h0 = h[0], h1 = h[1];
        } else {
            const auto l = __builtin_amdgcn_permlane16_swap(alo, blo, false, false);
            const auto h = __builtin_amdgcn_permlane16_swap(ahi, bhi, false, false);
            l0 = l[0], l1 = l[1], h0 = h[0], h1 = h[1];
        }
        return __longlong_as_double(((long long)h0 << 32) | l0) + __longlong_as_double(((long long)h1 << 32) | l1);
    } else {
        const bool up = (__lane_id() >> BIT) & 1;
        const double keep = up ? b : a, send = up ? a : b;
        return keep + lane_pair<BIT>(send);
    }
}

template <int BIT, int N, int K>
__device__ __forceinline__ double tree_sum(double (&v)[K])
{
    if constexpr (BIT < 0) {
        static_assert(N == 1, "six levels take up to 64 sums");
        return v[0];
    } else if constexpr (N == 1) {
        v[0] = BIT >= 4 ? pair_add<(BIT >= 4 ? BIT : 4)>(v[0], v[0]) : v[0] + lane_pair<(BIT < 4 ? BIT : 0)>(v[0]);
        return tree_sum<BIT - 1, 1>(v);
    } else {
        constexpr int H = (N + 1) / 2;
#pragma unroll
        for (int j = 0; j < H; j++) v[j] = pair_add<BIT>(v[j], j + H < N ? v[j + H] : v[j]);
        return tree_sum<BIT - 1, H>(v);
    }
}

// Which sum a lane holds after tree_sum<5, NQ> (-1: a copy of no use).
template <int NQ>
__device__ __forceinline__ int tree_index()
{
    int n[6], h[6];
    int m = NQ;
#pragma unroll
    for (int l = 0; l < 6; l++) {
        n[l] = m;
        h[l] = m == 1 ? 0 : (m + 1) / 2;
        m = (m + 1) / 2;
    }
    const int lane = __lane_id();
    int q = 0;
    bool ok = true;
#pragma unroll
    for (int l = 5; l >= 0; l--) {
        const int bit = (lane >> (5 - l)) & 1;
        if (n[l] == 1)
            ok &= bit == 0;   // one writer per sum
        else
            q += bit * h[l];
        ok &= q < n[l];
    }
    return ok ? q : -1;
}

// Sum acc[0..NQ) over the block (blockDim.x a multiple of 64, red holding
// one row per wave); the totals land in red[0][q].  Fixed order: the lane
// tree within a wave, then the waves in order.
template <int NQ>
__device__ __forceinline__ void block_sum(double (&acc)[NQ], double (*red)[kMaxSums])
{
    const int wave = threadIdx.x >> 6;
    const int nwaves = blockDim.x >> 6;
    const double v = tree_sum<5, NQ>(acc);
    const int q = tree_index<NQ>();
    if (q >= 0) red[wave][q] = v;
    __syncthreads();
    if (threadIdx.x < NQ) {
        double s = red[0][threadIdx.x];
        for (int w = 1; w < nwaves; w++) s += red[w][threadIdx.x];
        red[0][threadIdx.x] = s;
    }
    __syncthreads();
}

template <typename T>
__device__ __forceinline__ double round_to_storage(double v)
{
    return (double)(T)v;
}

// a^k, k = -4..3, formed by repeated multiplication or division: what a
// polynomial term of degree 4 - k is scaled with.
struct Powers {
    double p[4], m[5];   // a^0..a^3, a^0..a^-4
};
__device__ __forceinline__ Powers powers_of(double a)
{
    Powers w;
    w.p[0] = w.m[0] = 1.0;
#pragma unroll
    for (int j = 1; j < 4; j++) w.p[j] = w.p[j - 1] * a;
#pragma unroll
    for (int j = 1; j < 5; j++) w.m[j] = w.m[j - 1] / a;
    return w;
}
__device__ __forceinline__ double power(const Powers &w, int k)
{
    switch (k) {   // uniform: k comes from the model
    case 3: return w.p[3];
    case 2: return w.p[2];
    case 1: return w.p[1];
    case -1: return w.m[1];
    case -2: return w.m[2];
    case -3: return w.m[3];
    case -4: return w.m[4];
    default: return 1.0;
    }
}
static_assert(CE_MAX_DEGREE == 8, "powers_of covers degrees 1..8");

// The scalar state a tail reads and writes, held in registers: one lattice's
// a(t) and homogeneous references at step n, with the coefficients of the
// next pass derived from them.
template <int NF>
struct RunState {
    double a, a_next, adot_half, beta, tau;
    long long step, first_bad;
    double m[NF], fdot_mean[NF], r[NF];
};

// Scalar loads, all independent: the state is the same for every lane, and
// no kernel that calls this changes it before its tail.
template <int NF>
__device__ __forceinline__ RunState<NF> load_state(const Lattice &lat)
{
    const auto *sc = (const __attribute__((address_space(4))) Scalars *)lat.sc;
    RunState<NF> s;
    s.a = sc->a;
    s.a_next = sc->a_next;
    s.adot_half = sc->adot_half;
    s.beta = sc->beta;
    s.tau = sc->tau;
    s.step = sc->step;
    s.first_bad = sc->first_bad;
#pragma unroll
    for (int i = 0; i < NF; i++) {
        s.m[i] = sc->m[i];
        s.fdot_mean[i] = sc->fdot_mean[i];
        s.r[i] = sc->r[i];
    }
    return s;
}

// Coefficients of the pass that follows state s, in the storage type.
template <typename T, int NF>
__device__ __forceinline__ void fill_pass_scalars(PassScalars<T> &ps, const RunState<NF> &s, const Lattice &lat,
                                                  const Powers &w)
{
    const double a2 = s.a_next * s.a_next;
    ps.beta = (T)s.beta;
#pragma unroll
    for (int i = 0; i < kMaxFields; i++) {
        if (i < NF) {
            const int k = i < NF ? i : 0;
            ps.bm[i] = (T)(s.beta * s.m[k]);
            ps.r[i] = (T)s.r[k];
            ps.m1[i] = (T)(s.m[k] + lat.dt * s.r[k]);
            ps.m2a[i] = (T)(a2 * lat.mu2[i]);
            ps.hm[i] = (T)(0.5 * a2 * lat.mu2[i]);
        } else {
            ps.bm[i] = ps.r[i] = ps.m1[i] = ps.m2a[i] = ps.hm[i] = (T)0;
        }
    }
    // a term of degree D of the physical potential is coef a^(4 - D) in the
    // program variables
#pragma unroll
    for (int t = 0; t < kMaxTerms; t++)
        ps.tc[t] = t < lat.nterms ? (T)(lat.tcoef[t] * power(w, 4 - lat.tdeg[t])) : (T)0;
}

// Store state s and the next pass's coefficients (one thread).
template <int NF>
__device__ __forceinline__ void store_state(const Lattice &lat, const RunState<NF> &s)
{
#pragma clang fp contract(off)
    Scalars *sc = lat.sc;
    sc->a = s.a;
    sc->a_next = s.a_next;
    sc->adot_half = s.adot_half;
    sc->beta = s.beta;
    sc->tau = s.tau;
    sc->step = s.step;
    sc->first_bad = s.first_bad;
    const double a2 = s.a_next * s.a_next;
#pragma unroll
    for (int i = 0; i < kMaxFields; i++) {
        const int k = i < NF ? i : 0;
        if (i < NF) {
            sc->m[i] = s.m[k];
            sc->fdot_mean[i] = s.fdot_mean[k];
            sc->r[i] = s.r[k];
        }
        sc->nx_m1[i] = i < NF ? s.m[k] + lat.dt * s.r[k] : 0.0;
        sc->nx_hm[i] = i < NF ? 0.5 * a2 * lat.mu2[i] : 0.0;
    }
    Powers w;
    if (lat.nterms > 0) w = powers_of(s.a_next);
    fill_pass_scalars<float, NF>(sc->nxf, s, lat, w);
    fill_pass_scalars<double, NF>(sc->nxd, s, lat, w);
}

// FP64 tail after a step pass n -> n+1, worked by one wavefront.  Sums of
// field i at 6i: sum d, sum d^2, sum d Lap d, sum ubar^2, sum ubar, sum ubar d,
// all at n+1, with ubar = (fdot^{n+1/2} + p^{n+3/2})/2; last: sum V.
//
// Bound by latency: it is one chain of dependent FP64 divisions (each about
// 100 cycles) that everything else waits for.  So lane q divides sum q, lane i
// works field i, what does not depend on the sums is prepared before they
// arrive, and the diagnostics come after the next pass's coefficients.  (One
// thread working all of it on arrays in scratch memory took most of the 12 us
// of a step of a 1024-site line.)
template <typename T, int NF>
struct LaneTail {
    static constexpr int NQ = kSumsPerField * NF + 1;
    // step n (uniform), and the lane's field i = min(lane, NF - 1)
    double a, a1, y, beta, tau;
    long long step, first_bad;
    int i;
    double m, fdot_mean, r;
    // the lane's polynomial term and mass
    double tcoef, mu2;
    int tpow;
    // prepared
    double m1, ns_m1sq, A4, B, C0, vac;
    // of the solved step
    double x, abar, c, V, gsum, sum_uf, u0, t3, sumf2, grad;
    bool bad;

    __device__ __forceinline__ void load(const Lattice &lat)
    {
        const Scalars *sc = lat.sc;
        const int lane = __lane_id();
        i = min(lane, NF - 1);
        a = sc->a;
        a1 = sc->a_next;
        y = sc->adot_half;
        beta = sc->beta;
        tau = sc->tau;
        step = sc->step;
        first_bad = sc->first_bad;
        m = sc->m[i];
        fdot_mean = sc->fdot_mean[i];
        r = sc->r[i];
        tcoef = 0.0;
        tpow = 0;
        mu2 = lat.mu2[0];
#pragma unroll
        for (int f = 1; f < NF; f++) mu2 = i == f ? lat.mu2[f] : mu2;
#pragma unroll
        for (int t = 0; t < kMaxTerms; t++)
            if (lane == t && t < lat.nterms) {
                tcoef = lat.tcoef[t];
                tpow = 4 - lat.tdeg[t];
            }
    }

    // What the sums are not needed for.
    __device__ __forceinline__ void prepare(const Lattice &lat)
    {
#pragma clang fp contract(off)
        const double dt = lat.dt, Ns = (double)lat.nsites;
        m1 = m + dt * r;
        ns_m1sq = Ns * m1 * m1;
        const double A = dt / (4.0 * a1);
        A4 = 4.0 * A;
        B = 1.0 + dt * y / (2.0 * a1);
        C0 = dt * y * y / (4.0 * a1) - y;
        const double a1sq = a1 * a1;
        vac = a1sq * a1sq * lat.vacuum;
    }

    // From the sums (lane q: sum q) to the state at n+1.  scratch: 2 kMaxSums
    // doubles of LDS of this wavefront's own.
    __device__ __forceinline__ void solve(const Lattice &lat, double tot, double *scratch)
    {
#pragma clang fp contract(off)
        const double dt = lat.dt, Ns = (double)lat.nsites;
        const int lane = __lane_id();
        if (lane < NQ) {
            scratch[lane] = tot;
            scratch[kMaxSums + lane] = tot / Ns;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        const double *t = scratch + kSumsPerField * i, *u = t + kMaxSums;
        gsum = 0.0;
#pragma unroll
        for (int f = 0; f < NF; f++) gsum += -0.5 * scratch[kMaxSums + kSumsPerField * f + 2];
        // mean comoving potential at n+1, with the vacuum term a^4 V0
        V = scratch[kMaxSums + NQ - 1] + vac;
        x = abar = c = 0.0;
        if (lat.expansion) {
            // a'^{n+3/2} from the time-centred kick of a' (quadratic in x; the
            // root continuous with a'^{n+1/2}, written without cancellation)
            const double S = lat.kappa * (2.0 / 3.0 * gsum + V) / a1;
            const double C = C0 - dt * S;
            x = -2.0 * C / (B + sqrt(B * B - A4 * C));
            abar = 0.5 * (x + y);
            c = (S - abar * abar / a1) / a1;
        }
        beta = dt * c;
        u0 = u[0];
        grad = -0.5 * u[2];
        t3 = t[3];
        sumf2 = ns_m1sq + 2.0 * m1 * t[0] + t[1];
        sum_uf = m1 * t[4] + t[5];
        // mean of fdot^{n+3/2} = mean p^{n+3/2} + beta_{n+1} mean f^{n+1},
        // mean p^{n+3/2} = 2 mean ubar - mean fdot^{n+1/2}
        fdot_mean = 2.0 * u[4] - fdot_mean + beta * (m1 + u0);
        m = m1;
        r = round_to_storage<T>(fdot_mean);
        bad = __ballot(lane < NQ && !isfinite(tot)) != 0 || !isfinite(x) || !isfinite(c);
        a = a1;
        a1 = lat.expansion ? a + dt * x : 1.0;
        step += 1;
        tau += dt;
        if (bad && first_bad < 0) first_bad = step;
    }

    // Coefficients of the next pass (lane i: field i; lane t: term t).
    template <typename U>
    __device__ __forceinline__ void next_pass(const Lattice &lat, PassScalars<U> &ps) const
    {
#pragma clang fp contract(off)
        const int lane = __lane_id();
        const double a2 = a1 * a1;
        if (lane == 0) ps.beta = (U)beta;
        if (lane < kMaxFields) {
            const bool on = lane < NF;
            ps.bm[lane] = on ? (U)(beta * m) : (U)0;
            ps.r[lane] = on ? (U)r : (U)0;
            ps.m1[lane] = on ? (U)(m + lat.dt * r) : (U)0;
            ps.m2a[lane] = on ? (U)(a2 * mu2) : (U)0;
            ps.hm[lane] = on ? (U)(0.5 * a2 * mu2) : (U)0;
        }
        if (lat.nterms > 0) {
            // a term of degree D of the physical potential is coef a^(4 - D)
            // in the program variables
            double w = 1.0;
#pragma unroll
            for (int j = 0; j < 3; j++) w = j < tpow ? w * a1 : w;
#pragma unroll
            for (int j = 0; j < 4; j++) w = j < -tpow ? w / a1 : w;
            if (lane < kMaxTerms) ps.tc[lane] = (U)(tcoef * w);
        } else if (lane < kMaxTerms) {
            ps.tc[lane] = (U)0;
        }
    }
    static_assert(CE_MAX_DEGREE == 8, "powers of a from -4 to 3");

    // Diagnostics of the solved step; y is a'^{n+1/2} until advance().
    __device__ __forceinline__ void record(const Lattice &lat) const
    {
#pragma clang fp contract(off)
        const double Ns = (double)lat.nsites;
        const int lane = __lane_id();
        // kinetic energy of u = (fdot^{n+1/2} + fdot^{n+3/2})/2 - (abar/a) f
        //                     = ubar + eta f,  eta = dt c/2 - abar/a
        const double eta = 0.5 * lat.dt * c - abar / a;
        const double kin = 0.5 * (t3 + 2.0 * eta * sum_uf + eta * eta * sumf2) / Ns;
        double rho = V;
        const double own = kin + grad;
#pragma unroll
        for (int f = 0; f < NF; f++) rho += __shfl(own, f, 64);
        ce_energy *e = lat.ring + step % kLogCap;
        if (lane < kMaxFields) {
            const bool on = lane < NF;
            e->kin[lane] = on ? kin : 0.0;
            e->grad[lane] = on ? grad : 0.0;
            e->mean[lane] = on ? m1 + u0 : 0.0;
            e->mean_sq[lane] = on ? sumf2 / Ns : 0.0;
        }
        if (lane == 0) {
            e->step = step;
            e->tau = tau;
            e->a = a;
            e->adot = abar;
            e->hubble = abar / (a * a);
            e->pot = V;
            e->rho = rho;
            e->friedmann_residual =
                (lat.expansion && abar != 0.0) ? (abar * abar - lat.kappa * rho / 3.0) / (abar * abar) : 0.0;
            e->nonfinite = bad;
            e->pad_ = 0;
        }
    }

    __device__ __forceinline__ void advance() { y = x; }

    // The state in memory, with the next pass's coefficients (after advance).
    __device__ __forceinline__ void store(const Lattice &lat) const
    {
#pragma clang fp contract(off)
        Scalars *sc = lat.sc;
        const int lane = __lane_id();
        if (lane == 0) {
            sc->a = a;
            sc->a_next = a1;
            sc->adot_half = y;
            sc->beta = beta;
            sc->tau = tau;
            sc->step = step;
            sc->first_bad = first_bad;
        }
        if (lane < NF) {
            sc->m[lane] = m;
            sc->fdot_mean[lane] = fdot_mean;
            sc->r[lane] = r;
        }
        if (lane < kMaxFields) {
            sc->nx_m1[lane] = lane < NF ? m + lat.dt * r : 0.0;
            sc->nx_hm[lane] = lane < NF ? 0.5 * (a1 * a1) * mu2 : 0.0;
        }
        next_pass(lat, sc->nxf);
        next_pass(lat, sc->nxd);
    }
};

// FP64 tail of the start-up pass.  Sums of field i at 6i: sum d, sum d^2,
// sum d Lap d, sum fdot(0)^2, sum p^{1/2}, (unused); last: sum V at a = 1.
template <typename T, int NF>
__device__ __forceinline__ void init_tail(const Lattice &lat, RunState<NF> &s, const double *tot, ce_energy &e)
{
#pragma clang fp contract(off)
    const double Ns = (double)lat.nsites;
    const double dt = lat.dt;
    double gsum = 0.0, rho = 0.0;
#pragma unroll
    for (int i = 0; i < kMaxFields; i++) e.kin[i] = e.grad[i] = e.mean[i] = e.mean_sq[i] = 0.0;
#pragma unroll
    for (int i = 0; i < NF; i++) {
        const double *t = tot + kSumsPerField * i;
        const double m = s.m[i];
        e.kin[i] = 0.5 * t[3] / Ns;
        e.grad[i] = -0.5 * t[2] / Ns;
        e.mean[i] = m + t[0] / Ns;
        e.mean_sq[i] = (Ns * m * m + 2.0 * m * t[0] + t[1]) / Ns;
        gsum += e.grad[i];
        rho += e.kin[i] + e.grad[i];
    }
    const double V = tot[kSumsPerField * NF] / Ns + lat.vacuum;  // a = 1
    rho += V;
    double ap0 = 0.0, app0 = 0.0;
    if (lat.expansion) {
        ap0 = sqrt(lat.kappa * rho / 3.0);
        app0 = -ap0 * ap0 + lat.kappa * (2.0 / 3.0 * gsum + V);
    }
    const double aph = ap0 + 0.5 * dt * app0;
    // fdot^{1/2} = fdot(0) + a'(0) f + dt/2 (Lap f - V' + a''(0) f): the stored
    // half kick omits the two f terms, beta_0 = a'(0) + dt/2 a''(0).
    const double beta0 = aph;
    int bad = 0;
#pragma unroll
    for (int i = 0; i < NF; i++) {
        const double fm = tot[kSumsPerField * i + 4] / Ns + beta0 * e.mean[i];
        s.fdot_mean[i] = fm;
        s.r[i] = round_to_storage<T>(fm);
    }
#pragma unroll
    for (int q = 0; q <= kSumsPerField * NF; q++) bad |= !isfinite(tot[q]);
    bad |= !isfinite(ap0);   // a negative energy density cannot start an expanding run
    e.step = 0;
    e.tau = 0.0;
    e.a = 1.0;
    e.adot = ap0;
    e.hubble = ap0;
    e.pot = V;
    e.rho = rho;
    e.friedmann_residual =
        (lat.expansion && ap0 != 0.0) ? (ap0 * ap0 - lat.kappa * rho / 3.0) / (ap0 * ap0) : 0.0;
    e.nonfinite = bad;
    e.pad_ = 0;
    s.a = 1.0;
    s.adot_half = aph;
    s.a_next = lat.expansion ? 1.0 + dt * aph : 1.0;
    s.beta = beta0;
    s.tau = 0.0;
    s.step = 0;
    s.first_bad = bad ? 0 : -1;
}

// Partial sum q of block or tile `row`: one column per sum, so that the
// last block's reads of a column by consecutive threads are contiguous.
__device__ __forceinline__ double *partial_at(const Lattice &lat, int q, long long row)
{
    return lat.partials + (long long)q * lat.slots + row;
}

// Store the block's totals (red[0], after block_sum) as row `row` of the
// partial sums: agent-scope stores, written through this XCD's L2, by threads
// of wave 0, whose finish_pass waits for them.
template <int NQ>
__device__ __forceinline__ void put_partials(const Lattice &lat, const double (*red)[kMaxSums], long long row)
{
    if (threadIdx.x < NQ)
        __hip_atomic_store(partial_at(lat, threadIdx.x, row), red[0][threadIdx.x], __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
}

// Last-block reduction of the partial sums in a fixed order, then the FP64
// tail.  Every block calls this after writing its partials with put_partials.
// The `grid` blocks (this lattice's share of the launch) wrote `rows` rows of
// partials between them (one per block, or one per tile); the block that takes
// the last ticket reduces them in row order and clears the tile counters for
// the next launch (every other block has finished taking tiles by then).
//
// Ordering: wave 0 wrote the block's rows through to memory and waits until
// they have arrived before it takes the ticket, and the last block reads them
// past its caches, so no block writes back or invalidates an L2: a full fence
// per block evicted the halos that the other blocks on its XCD were about to
// re-read, and a release alone still wrote the L2 back.
//
// Each thread sums rows threadIdx.x, + blockDim.x, ... in that order; with
// R > 1 it loads R of them before adding them, so R rows' loads are in
// flight at once (the sums, and so the result, are the same for every R).
// RUNS (the direct pass, 256 threads): up to kRunRows rows a thread are
// consecutive ones instead, as a resident block adds the rows of the blocks it stands for.
template <typename T, int NF, int MODE, int R = 1, bool RUNS = false>
__device__ __forceinline__ void finish_pass(const Lattice &lat, int grid, int rows, double (*red)[kMaxSums])
{
    constexpr int NQ = kSumsPerField * NF + 1;
    __shared__ int s_last;
    LaneTail<T, NF> tail;
    if (MODE == kStep && threadIdx.x < 64) {
        // the state is this launch's input until the last block's tail
        tail.load(lat);
        tail.prepare(lat);
    }
    if (grid > 1 || rows > 1) {
        __syncthreads();
        if (threadIdx.x < 64) {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            __builtin_amdgcn_s_waitcnt(0);   // wave 0's rows have arrived
            if (threadIdx.x == 0)
                s_last = __hip_atomic_fetch_add(lat.ticket, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
                         (unsigned int)(grid - 1);
        }
        __syncthreads();
        if (!s_last) return;
        double acc[NQ];
#pragma unroll
        for (int q = 0; q < NQ; q++) acc[q] = 0.0;
        int stride = (int)blockDim.x;
        int b = threadIdx.x;
        if constexpr (RUNS) {
            if (rows <= kRunRows * stride) {
                const int run = (rows + stride - 1) / stride;
                b *= run;
                rows = min(rows, b + run);
                stride = 1;
            }
        }
        if constexpr (R > 1) {
            for (; b + (R - 1) * stride < rows; b += R * stride) {
                double v[R][NQ];
#pragma unroll
                for (int r = 0; r < R; r++) {
#pragma unroll
                    for (int q = 0; q < NQ; q++)
                        v[r][q] = __hip_atomic_load(partial_at(lat, q, b + r * stride), __ATOMIC_RELAXED,
                                                    __HIP_MEMORY_SCOPE_AGENT);
                }
#pragma unroll
                for (int r = 0; r < R; r++)
#pragma unroll
                    for (int q = 0; q < NQ; q++) acc[q] += v[r][q];
            }
        }
        for (; b < rows; b += stride) {
            double v[NQ];
#pragma unroll
            for (int q = 0; q < NQ; q++)
                v[q] = __hip_atomic_load(partial_at(lat, q, b), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#pragma unroll
            for (int q = 0; q < NQ; q++) acc[q] += v[q];
        }
        block_sum<NQ>(acc, red);
    }   // one block, one row: its totals are the lattice's
    if (threadIdx.x < 64) {
        if (MODE == kStep) {
            const double tot = threadIdx.x < NQ ? red[0][threadIdx.x] : 0.0;
            __shared__ double scratch[2 * kMaxSums];
            tail.solve(lat, tot, scratch);
            tail.record(lat);
            tail.advance();
            tail.store(lat);
        }
        if (threadIdx.x == 0) {
            if (MODE == kStep) {
                lat.sc->cur ^= 1;
                if (lat.sc->remaining > 0) lat.sc->remaining -= 1;
            } else {
                RunState<NF> st = load_state<NF>(lat);
                ce_energy e;
                init_tail<T, NF>(lat, st, red[0], e);
                store_state<NF>(lat, st);
                lat.ring[e.step % kLogCap] = e;
            }
            if (grid > 1 || rows > 1)
                for (int i = 0; i <= kTileCounters; i++)
                    __hip_atomic_store(lat.ticket + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
}


// All coefficients of one pass, computed once per thread from the lattice
// description and the FP64 scalar state.
template <typename T, int NF>
struct PassCoef {
    T dt, inv_dx2, lam, kick;
    T G[NF], m2a[NF];
    FieldCoef<T> cf[NF];
    T qlam;              // lambda / 4
    T hG[NF];            // G_j / 2
    T hm[NF];            // a^2 mu2_i / 2 at the kick
    bool has_mass;
    // polynomial model: terms of degree >= 1, scaled coefficients and exponents
    int nterms;
    T tc[kMaxTerms];
    int texp[kMaxTerms][NF];
};

__device__ __forceinline__ float uniform(float v)
{
    return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(v)));
}
__device__ __forceinline__ double uniform(double v)
{
    const long long b = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readfirstlane((int)(b & 0xffffffffLL));
    const int hi = __builtin_amdgcn_readfirstlane((int)(b >> 32));
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// Every coefficient is the same in all lanes; keep them in scalar registers.
template <typename T, int NF>
__device__ __forceinline__ void make_uniform(PassCoef<T, NF> &c)
{
    c.dt = uniform(c.dt);
    c.inv_dx2 = uniform(c.inv_dx2);
    c.lam = uniform(c.lam);
    c.kick = uniform(c.kick);
    c.qlam = uniform(c.qlam);
#pragma unroll
    for (int i = 0; i < NF; i++) {
        c.G[i] = uniform(c.G[i]);
        c.m2a[i] = uniform(c.m2a[i]);
        c.cf[i].beta = uniform(c.cf[i].beta);
        c.cf[i].bm = uniform(c.cf[i].bm);
        c.cf[i].r = uniform(c.cf[i].r);
        c.cf[i].m1 = uniform(c.cf[i].m1);
        c.hG[i] = uniform(c.hG[i]);
        c.hm[i] = uniform(c.hm[i]);
    }
    c.has_mass = __builtin_amdgcn_readfirstlane((int)c.has_mass) != 0;
}

template <typename T>
__device__ __forceinline__ T static_coef(double d, float f)
{
    if constexpr (sizeof(T) == 4)
        return f;
    else
        return d;
}

template <typename T>
using cscalars = const __attribute__((address_space(4))) Scalars *;

template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) PassScalars<T> &pass_scalars(cscalars<T> s)
{
    if constexpr (sizeof(T) == 4)
        return s->nxf;
    else
        return s->nxd;
}

// Coefficients of a pass.  A step pass reads the ones the previous tail
// published (scalar loads: the values are the same for every lane and this
// kernel writes them only after every block has read them); the start-up pass
// derives its own (beta = 0, a = 1, m unchanged).
template <typename T, int NF, int MODEL, int MODE>
__device__ __forceinline__ PassCoef<T, NF> make_coef(const Lattice &lat)
{
    PassCoef<T, NF> c;
    if constexpr (MODEL == kPoly) {
        c.nterms = __builtin_amdgcn_readfirstlane(lat.nterms);
        for (int t = 0; t < kMaxTerms; t++)
#pragma unroll
            for (int i = 0; i < NF; i++) c.texp[t][i] = __builtin_amdgcn_readfirstlane(lat.texp[t][i]);
        if (MODE == kStep) {
            const auto &ps = pass_scalars<T>((cscalars<T>)lat.sc);
            for (int t = 0; t < kMaxTerms; t++) c.tc[t] = ps.tc[t];
        } else {
            for (int t = 0; t < kMaxTerms; t++) c.tc[t] = uniform((T)lat.tcoef[t]);  // a = 1
        }
    }
    c.dt = static_coef<T>(lat.dt, lat.dt_f);
    c.inv_dx2 = static_coef<T>(lat.inv_dx2, lat.inv_dx2_f);
    c.lam = static_coef<T>(lat.lambda, lat.lambda_f);
    c.qlam = static_coef<T>(0.25 * lat.lambda, lat.qlam_f);
    c.has_mass = false;
#pragma unroll
    for (int i = 0; i < NF; i++) {
        c.G[i] = static_coef<T>(lat.G[i], lat.G_f[i]);
        c.hG[i] = static_coef<T>(0.5 * lat.G[i], lat.hG_f[i]);
        c.has_mass |= lat.mu2[i] != 0.0;
    }
    if (MODE == kStep) {
        const cscalars<T> cs = (cscalars<T>)lat.sc;
        const auto &ps = pass_scalars<T>(cs);
        c.kick = c.dt;
#pragma unroll
        for (int i = 0; i < NF; i++) {
            c.m2a[i] = ps.m2a[i];
            c.cf[i].beta = ps.beta;
            c.cf[i].bm = ps.bm[i];
            c.cf[i].r = ps.r[i];
            c.cf[i].m1 = ps.m1[i];
            c.hm[i] = ps.hm[i];
        }
    } else {
        const Scalars *sc = lat.sc;
        c.kick = (T)(0.5 * lat.dt);
#pragma unroll
        for (int i = 0; i < NF; i++) {
            c.m2a[i] = (T)lat.mu2[i];
            c.hm[i] = (T)(0.5 * lat.mu2[i]);
            const double m = sc->m[i];
            c.cf[i].beta = (T)0;
            c.cf[i].bm = (T)0;
            c.cf[i].r = (T)0;
            c.cf[i].m1 = (T)m;
        }
        make_uniform(c);
    }
    return c;
}

// Own-site derivative at n+1/2 and deviation at n+1 (kInit: unchanged).
template <typename T, int NF, int MODE>
__device__ __forceinline__ void own_drift(const PassCoef<T, NF> &c, int i, T d, T p, T &fdot, T &d1)
{
    if (MODE == kStep) {
        fdot = fdot_of(d, p, c.cf[i]);
        d1 = fma_t(c.dt, fdot - c.cf[i].r, d);
    } else {
        fdot = p;
        d1 = d;
    }
}

// Neighbour deviation at n+1 (same arithmetic as own_drift).
template <typename T, int NF, int MODE>
__device__ __forceinline__ T nbr_drift(const PassCoef<T, NF> &c, int i, T d, T p)
{
    return (MODE == kStep) ? drift(d, p, c.cf[i], c.dt) : d;
}

// One site: potential derivative and kick, plus the site's terms of the
// volume sums added into `part` (storage type).
//   d1[i]   deviation of field i at n+1,  fdot[i] derivative at n+1/2,
//   lap[i]  Laplacian of d1 at the site;  pn[i] receives the new stored
//   derivative.  Every kernel calls this, so all kernels round alike.
// With FP32 storage the per-site terms are formed in FP32 and a thread adds
// its few sites in FP32 before folding them into its FP64 accumulators
// (flush_sums); with FP64 storage everything is FP64.
// Polynomial model at one site: V = sum_t tc_t prod_i v_i^e_ti and
// dV/dv_i = sum_t tc_t (d v_i^e_ti / dv_i) prod_{j != i} v_j^e_tj.  Powers
// come from repeated multiplication, the derivative of v^e alongside by the
// product rule ((v^k)' v + v^k = (v^(k+1))'), so no exponent is ever a
// floating-point factor.  Exponents and coefficients are uniform.
template <typename T, int NF>
__device__ __forceinline__ void poly_potential(const PassCoef<T, NF> &c, const T (&v)[NF], T &V, T (&dV)[NF])
{
    V = (T)0;
#pragma unroll
    for (int i = 0; i < NF; i++) dV[i] = (T)0;
    // unrolled over the term slots, so every table index is a constant and
    // the tables stay in scalar registers
#pragma unroll
    for (int t = 0; t < kMaxTerms; t++) {
        if (t >= c.nterms) break;
        T pw[NF], dpw[NF];
#pragma unroll
        for (int i = 0; i < NF; i++) {
            T x = (T)1, dx = (T)0;
            for (int k = 0; k < c.texp[t][i]; k++) {
                dx = fma_t(dx, v[i], x);
                x = x * v[i];
            }
            pw[i] = x;
            dpw[i] = dx;
        }
        T mono = pw[0];
#pragma unroll
        for (int i = 1; i < NF; i++) mono = mono * pw[i];
        V = fma_t(c.tc[t], mono, V);
#pragma unroll
        for (int i = 0; i < NF; i++) {
            T prod = dpw[i];
#pragma unroll
            for (int j = 0; j < NF; j++)
                if (j != i) prod = prod * pw[j];
            dV[i] = fma_t(c.tc[t], prod, dV[i]);
        }
    }
}

template <typename T, int NF, int MODEL, int MODE, int NQ>
__device__ __forceinline__ void site_update(const PassCoef<T, NF> &c, const T (&d1)[NF], const T (&fdot)[NF],
                                            const T (&lap)[NF], T (&pn)[NF], T (&part)[NQ])
{
    if constexpr (MODEL == kPoly) {
        T v[NF], dV[NF], Vs;
#pragma unroll
        for (int i = 0; i < NF; i++) v[i] = c.cf[i].m1 + d1[i];
        poly_potential<T, NF>(c, v, Vs, dV);
#pragma unroll
        for (int i = 0; i < NF; i++) {
            pn[i] = fma_t(c.kick, lap[i] - dV[i], fdot[i]);
            const T dd = d1[i];
            T *a = part + kSumsPerField * i;
            a[0] += dd;
            a[1] = fma_t(dd, dd, a[1]);
            a[2] = fma_t(dd, lap[i], a[2]);
            if (MODE == kStep) {
                const T ub = (T)0.5 * (fdot[i] + pn[i]);
                a[3] = fma_t(ub, ub, a[3]);
                a[4] += ub;
                a[5] = fma_t(ub, dd, a[5]);
            } else {
                a[3] = fma_t(fdot[i], fdot[i], a[3]);
                a[4] += pn[i];
            }
        }
        part[kSumsPerField * NF] += Vs;
        return;
    }
    T v[NF];
#pragma unroll
    for (int i = 0; i < NF; i++) v[i] = c.cf[i].m1 + d1[i];
    T chi2 = (T)0;
#pragma unroll
    for (int j = 1; j < NF; j++) chi2 = fma_t(c.G[j] * v[j], v[j], chi2);
    const T v0sq = v[0] * v[0];
    T Vs = (c.qlam * v0sq) * v0sq;
#pragma unroll
    for (int i = 0; i < NF; i++) {
        T dV = (i == 0) ? fma_t(c.lam * v0sq, v[0], v[0] * chi2) : (c.G[i] * v0sq) * v[i];
        dV = fma_t(c.m2a[i], v[i], dV);
        pn[i] = fma_t(c.kick, lap[i] - dV, fdot[i]);
        const T dd = d1[i];
        T *a = part + kSumsPerField * i;
        a[0] += dd;
        a[1] = fma_t(dd, dd, a[1]);
        a[2] = fma_t(dd, lap[i], a[2]);
        if (MODE == kStep) {
            const T ub = (T)0.5 * (fdot[i] + pn[i]);
            a[3] = fma_t(ub, ub, a[3]);
            a[4] += ub;
            a[5] = fma_t(ub, dd, a[5]);
        } else {
            a[3] = fma_t(fdot[i], fdot[i], a[3]);
            a[4] += pn[i];
        }
        const T vsq = v[i] * v[i];
        if (i > 0) Vs = fma_t(c.hG[i] * v0sq, vsq, Vs);
        if (c.has_mass) Vs = fma_t(c.hm[i], vsq, Vs);
    }
    part[kSumsPerField * NF] += Vs;
}

template <typename T, int NQ>
__device__ __forceinline__ void clear_part(T (&part)[NQ])
{
#pragma unroll
    for (int q = 0; q < NQ; q++) part[q] = (T)0;
}

template <typename T, int NQ>
__device__ __forceinline__ void flush_sums(const T (&part)[NQ], double (&acc)[NQ])
{
#pragma unroll
    for (int q = 0; q < NQ; q++) acc[q] += (double)part[q];
}

}  // namespace dev
}  // namespace ce
