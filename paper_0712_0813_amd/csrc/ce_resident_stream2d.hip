// Resident form of the 2-D streaming pass: many steps in one launch of a
// lattice whose groups of four units (256 x-sites by R rows, one unit per
// wavefront) are at most kSyncRows.  See ce_resident.hpp for the exchange
// between blocks.
//
// A wavefront owns one unit; a lane owns 4 x-sites of every row of it, d in
// LDS and p in registers.  The y neighbours are the lane's own rows, and at
// the unit's ends the quads of the units above and below, which only this lane
// needs; x neighbours come from the adjacent lane, and at the unit's edges
// from the neighbouring units' edge columns, packed in the staging chunk (or
// from the far end of the wavefront where a unit is a whole row).  Nothing is
// shared between the wavefronts of a block but their sums.  The arithmetic of
// a site and the sums' order (rows in turn, lane tree, waves in order, blocks
// in order) are those of the streaming pass, so a step taken here is bitwise a
// step taken there.
//
// Two FP32 fields, us a step, here and with one launch a step: 256^2 4.2 and
// 9.2, 512^2 4.7 and 11.9, 1024^2 7.7 and 17.0, 2048^2 17.7 and 36.1.
// The small ones are the exchange (2.1 us) and the tail (0.7); 2048^2 is the sites
// at one wavefront a SIMD, which issues vector instructions in 45% of the cycles.
#include "ce_resident.hpp"

#ifndef CE_UNIT_MODEL
#error "compile this file once per model, with -DCE_UNIT_MODEL=0 and -DCE_UNIT_MODEL=1"
#endif

namespace ce {
namespace {

using namespace dev;

constexpr int kSeg = 256;   // x sites per unit

// The block is the `rank`-th of the nblk that work the lattice.
// CHECK: the block checks in here (a pool's has done so).
template <typename T, int NF, int MODEL, int R, bool CHECK>
__device__ __forceinline__ void resident_stream2d_body(const Lattice &lat, int src, int steps, int rank, int nblk,
                                                       const Start &start)
{
    constexpr int NQ = kSumsPerField * NF + 1;
    constexpr int WAVES = kBlock / 64;
    static_assert(2 * R <= 64, "one lane per edge site of a unit");
    // packed columns: [buffer][unit][left, right][field][d, p][row]
    constexpr unsigned CSTRIDE = NF * 2 * R;
    __shared__ __align__(16) T lds[WAVES][R][NF][kSeg];
    __shared__ T edges[WAVES][2][NF][R];
    __shared__ double red[WAVES][kMaxSums];
    __shared__ PassScalars<T> next;

    if (threadIdx.x >= kBlock) {
        if (!CHECK || launch_starts(lat, nblk, start))
            service_wave<T, NF, 1, WAVES>(lat, steps, rank, nblk, rank, red, next, start);
        return;
    }
    const int N = lat.N;
    const int nseg = N / kSeg, nrow = N / R;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int unit = (int)xcd_item(rank, 0, nblk, nblk) * WAVES + wave;
    const bool active = unit < nseg * nrow;
    const int seg = unit % nseg, ur = unit / nseg;
    const int y0 = ur * R;
    const bool wrap = nseg == 1;

    // element offsets: own quad of row 0, the quads above and below the unit
    const unsigned own_x = (unsigned)(seg * kSeg + 4 * lane);
    const unsigned own = (unsigned)y0 * N + own_x;
    const unsigned yoff[2] = {(unsigned)((y0 + N - 1) % N) * N + own_x, (unsigned)((y0 + R) % N) * N + own_x};
    // edge site (side, row) loaded by this lane, in the array and packed: the
    // left neighbour's right column is this unit's left one
    const int eside = lane / R, erow = lane % R;
    const bool edge_lane = active && !wrap && lane < 2 * R;
    const unsigned ex = (unsigned)(y0 + erow) * N +
                        (unsigned)((eside ? (seg + 1) * kSeg : seg * kSeg + N - 1) % N);
    const int from = ur * nseg + (eside ? (seg == nseg - 1 ? 0 : seg + 1) : (seg == 0 ? nseg - 1 : seg - 1));
    const unsigned cread = (unsigned)(from * 2 + 1 - eside) * CSTRIDE + (unsigned)erow;
    const bool column = active && !wrap && (lane == 0 || lane == 63);
    const unsigned cwrite = (unsigned)(unit * 2 + (lane != 0)) * CSTRIDE;
    const __amdgpu_buffer_rsrc_t cols = agent_buffer(lat.columns);
    const unsigned csize = (unsigned)(nseg * nrow) * 2 * CSTRIDE;   // of one buffer's columns

    PassCoef<T, NF> c = make_coef<T, NF, MODEL, kStep>(lat);

    T p[R][NF][4];
#pragma unroll
    for (int k = 0; k < R; k++)
#pragma unroll
        for (int i = 0; i < NF; i++) {
            Quad<T> dq{}, pq{};
            if (active) {
                const unsigned o = (own + k * N) * (unsigned)sizeof(T);
                dq = agent_load_quad(agent_buffer(lat.d[src][i]), o, T());
                pq = agent_load_quad(agent_buffer(lat.p[src][i]), o, T());
            }
            store_lds(&lds[wave][k][i][4 * lane], dq.v);
#pragma unroll
            for (int e = 0; e < 4; e++) p[k][i][e] = pq.v[e];
        }

    // stored values of the halo at the current step
    Quad<T> yd[2][NF], yp[2][NF];
    T xd[NF], xp[NF];
    auto load_halo = [&](int buf, bool packed) {
#pragma unroll
        for (int i = 0; i < NF; i++) {
            const __amdgpu_buffer_rsrc_t bd = agent_buffer(lat.d[buf][i]), bp = agent_buffer(lat.p[buf][i]);
            if (active) {
#pragma unroll
                for (int s = 0; s < 2; s++) {
                    yd[s][i] = agent_load_quad(bd, yoff[s] * (unsigned)sizeof(T), T());
                    yp[s][i] = agent_load_quad(bp, yoff[s] * (unsigned)sizeof(T), T());
                }
            }
            if (edge_lane) {
                const unsigned o = buf * csize + cread + i * 2 * R;
                xd[i] = packed ? agent_load(cols, o * (unsigned)sizeof(T), T())
                               : agent_load(bd, ex * (unsigned)sizeof(T), T());
                xp[i] = packed ? agent_load(cols, (o + R) * (unsigned)sizeof(T), T())
                               : agent_load(bp, ex * (unsigned)sizeof(T), T());
            }
        }
    };
#pragma unroll
    for (int i = 0; i < NF; i++) {
        yd[0][i] = yd[1][i] = yp[0][i] = yp[1][i] = Quad<T>{};
        xd[i] = xp[i] = (T)0;
    }
    load_halo(src, false);   // no step has packed the columns yet
    if (CHECK && !launch_starts(lat, nblk, start)) return;

    for (int step = 0; step < steps; step++) {
        const int out = src ^ 1 ^ (step & 1);
        const bool last = step + 1 == steps;
        // the lane's place in a row of LDS, as an offset the compiler cannot
        // see through: it would otherwise keep d in registers as well
        int at = 4 * lane;
        asm volatile("" : "+v"(at));
        // drift in place: d becomes the new deviation, p the derivative at n+1/2
        T yn[2][NF][4];
#pragma unroll
        for (int i = 0; i < NF; i++) {
#pragma unroll
            for (int k = 0; k < R; k++) {
                T d[4];
                load_lds(&lds[wave][k][i][at], d);
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    T fdot, d1;
                    own_drift<T, NF, kStep>(c, i, d[e], p[k][i][e], fdot, d1);
                    d[e] = d1;
                    p[k][i][e] = fdot;
                }
                store_lds(&lds[wave][k][i][at], d);
            }
#pragma unroll
            for (int s = 0; s < 2; s++)
#pragma unroll
                for (int e = 0; e < 4; e++) yn[s][i][e] = nbr_drift<T, NF, kStep>(c, i, yd[s][i].v[e], yp[s][i].v[e]);
            if (edge_lane) edges[wave][eside][i][erow] = nbr_drift<T, NF, kStep>(c, i, xd[i], xp[i]);
        }
        __syncthreads();   // (1)
        asm volatile("" : "+v"(at));
        double acc[NQ];
#pragma unroll
        for (int j = 0; j < NQ; j++) acc[j] = 0.0;
        T below[NF][4], cur[NF][4], above[NF][4];   // rows k-1, k, k+1
#pragma unroll
        for (int i = 0; i < NF; i++) {
#pragma unroll
            for (int e = 0; e < 4; e++) below[i][e] = yn[0][i][e];
            load_lds(&lds[wave][0][i][at], cur[i]);
        }
#pragma unroll
        for (int k = 0; k < R; k++) {
            __builtin_amdgcn_sched_barrier(0);   // one row at a time: registers
            T lap[4][NF];
#pragma unroll
            for (int i = 0; i < NF; i++) {
                T xl = lane_from_left(cur[i][3]);
                T xr = lane_from_right(cur[i][0]);
                if (wrap) {
                    const T first = lane_copy(cur[i][0], 0), end = lane_copy(cur[i][3], 63);
                    if (lane == 0) xl = end;
                    if (lane == 63) xr = first;
                } else {
                    if (lane == 0) xl = edges[wave][0][i][k];
                    if (lane == 63) xr = edges[wave][1][i][k];
                }
                if (k + 1 < R) {
                    load_lds(&lds[wave][k + 1 < R ? k + 1 : k][i][at], above[i]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; e++) above[i][e] = yn[1][i][e];
                }
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    const T l = e == 0 ? xl : cur[i][e == 0 ? 0 : e - 1];
                    const T r = e == 3 ? xr : cur[i][e == 3 ? 3 : e + 1];
                    const T pr = (l + r) + (above[i][e] + below[i][e]);
                    lap[e][i] = fma_t((T)-4, cur[i][e], pr) * c.inv_dx2;
                }
            }
            T part[NQ];
            clear_part(part);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                T d1s[NF], fds[NF], pn[NF];
#pragma unroll
                for (int i = 0; i < NF; i++) {
                    d1s[i] = cur[i][e];
                    fds[i] = p[k][i][e];
                }
                site_update<T, NF, MODEL, kStep, NQ>(c, d1s, fds, lap[e], pn, part);
#pragma unroll
                for (int i = 0; i < NF; i++) p[k][i][e] = pn[i];
            }
            flush_sums(part, acc);
            // add them now: left to itself the compiler sinks every row's
            // additions to the last one and holds the parts until then
#pragma unroll
            for (int j = 0; j < NQ; j++) asm volatile("" : "+v"(acc[j]));
            if (active && (last || k == 0 || k == R - 1)) {
                const unsigned o = (own + k * N) * (unsigned)sizeof(T);
#pragma unroll
                for (int i = 0; i < NF; i++) {
                    agent_store(agent_buffer(lat.d[out][i]), o, cur[i]);
                    agent_store(agent_buffer(lat.p[out][i]), o, p[k][i]);
                }
            }
            if (column) {
#pragma unroll
                for (int i = 0; i < NF; i++) {
                    const unsigned o = out * csize + cwrite + i * 2 * R + k;
                    // values, not a choice between two array elements, which
                    // would put the arrays in scratch memory
                    const T dl = cur[i][0], dr = cur[i][3], pl = p[k][i][0], pr = p[k][i][3];
                    agent_store(cols, o * (unsigned)sizeof(T), lane == 0 ? dl : dr);
                    agent_store(cols, (o + R) * (unsigned)sizeof(T), lane == 0 ? pl : pr);
                }
            }
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int e = 0; e < 4; e++) {
                    below[i][e] = cur[i][e];
                    cur[i][e] = above[i][e];
                }
        }
        if (!active) {
#pragma unroll
            for (int j = 0; j < NQ; j++) acc[j] = 0.0;
        }
        {
            const double v = tree_sum<5, NQ>(acc);
            const int j = tree_index<NQ>();
            if (j >= 0) red[wave][j] = v;
        }
        stores_arrived();
        __syncthreads();   // (2)
        if (nblk > 1) __syncthreads();   // (3)
        if (!last) load_halo(out, true);      // while the service wave runs the tail
        __syncthreads();   // (4)
        next_coef<T, NF, MODEL>(c, next);
    }
}

template <typename T, int NF, int MODEL, int R>
__global__ __launch_bounds__(kBlock + 64) void resident_stream2d_kernel(Lattice lat, int src, int steps, Start start)
{
    resident_stream2d_body<T, NF, MODEL, R, true>(lat, src, steps, blockIdx.x, gridDim.x, start);
}

// Up to k steps of each of n lattices; see run_members.
template <typename T, int NF, int MODEL, int R>
__global__ __launch_bounds__(kBlock + 64) void resident_stream2d_batched(const Lattice *lats, int n, int nblk, int k,
                                                                         Start start)
{
    run_members(lats, n, nblk, k, start, [&](const Lattice &lat, int src, int steps, int rank, int blocks) {
        resident_stream2d_body<T, NF, MODEL, R, false>(lat, src, steps, rank, blocks, start);
    });
}

// Built where p and the halo come near the registers of a thread (a block of five
// waves has 256) and the units in LDS.  Some spill and still beat plain launches
// of the same units (us a step, resident and plain): two FP32 fields in sixteen
// rows, 31 spilled, 2048^2 17.8 and 36.3; one FP64 field, 158, 17.6 and 36.6; two
// in eight rows, 205, 1280^2 20.9 and 31.9.  Where they do not, they are not taken
// (resident_pays).
template <typename T, int NF, int R>
constexpr bool built()
{
    return 4 * R * NF * (int)sizeof(T) / 4 <= 128 && R * NF * kSeg * 4 * (int)sizeof(T) <= 150 * 1024;
}

template <typename T, int NF, int MODEL, int R>
const void *kernel_if_built(bool batched)
{
    if constexpr (built<T, NF, R>()) {
        if (!batched) return (const void *)resident_stream2d_kernel<T, NF, MODEL, R>;
        // pools: FP32 units of eight or sixteen rows (see member_launch)
        if constexpr (sizeof(T) == 4 && R >= 8) return (const void *)resident_stream2d_batched<T, NF, MODEL, R>;
    }
    return nullptr;
}

template <typename T, int NF, int MODEL>
const void *kernel_rows(int rows, bool batched)
{
    switch (rows) {
    case 1: return kernel_if_built<T, NF, MODEL, 1>(batched);
    case 2: return kernel_if_built<T, NF, MODEL, 2>(batched);
    case 4: return kernel_if_built<T, NF, MODEL, 4>(batched);
    case 8: return kernel_if_built<T, NF, MODEL, 8>(batched);
    case 16: return kernel_if_built<T, NF, MODEL, 16>(batched);
    default: return nullptr;
    }
}

template <typename T, int MODEL>
const void *kernel_nf(int nf, int rows, bool batched)
{
    switch (nf) {
    case 1: return kernel_rows<T, 1, MODEL>(rows, batched);
    case 2: return kernel_rows<T, 2, MODEL>(rows, batched);
    case 3: return kernel_rows<T, 3, MODEL>(rows, batched);
    default: return nullptr;
    }
}

}  // namespace

// This unit's model (the source is compiled once per model).
constexpr int kUnit = CE_UNIT_MODEL;

template <>
const void *resident_stream2d_model<kUnit>(int precision, int nf, int rows, bool batched)
{
    return precision == CE_FP64 ? kernel_nf<double, kUnit>(nf, rows, batched)
                                : kernel_nf<float, kUnit>(nf, rows, batched);
}

}  // namespace ce
