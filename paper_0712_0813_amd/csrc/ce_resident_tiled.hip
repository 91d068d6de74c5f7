// Resident form of the tiled 3-D pass: many steps in one launch of a lattice
// whose tiles (VEC LPR x BS/LPR sites by ZP planes) are at most kSyncRows.  See
// ce_resident.hpp for the exchange between blocks.
//
// A block owns one tile; a thread owns the VEC sites of its (x, y) place in every
// plane of it.  d stays in LDS, where neighbours read it, p in registers (both
// in registers spilled 180 of them with two FP32 fields and eight planes).
// Per step the tile is drifted in place and the halo rows and columns of every
// plane are put around it (y neighbours, and x neighbours at the tile's
// edges); z neighbours are the thread's own planes, and at the tile's ends the
// sites of the tile above or below, which only this thread needs.  Rows and
// planes are exchanged through the ping-pong buffers; edge columns, whose
// sites there lie a line apart, are packed in the staging chunk (128^3 x 2
// fields: 13.1 us a step before, 5 us of it loading the halo).  The arithmetic of a site and the sums' order (the planes in
// turn, lane tree, waves in order, tile rows in order) are those of the tiled
// pass, so a step taken here is bitwise a step taken there.
//
// Two FP32 fields, us a step, here and with one launch a step: 64^3 4.9 and
// 13.4, 96^3 8.1 and 19.4, 128^3 10.5 and 29.3.  Of 10.5, the sites take 6.9, exchange
// and tail the rest.  With one wavefront of sites a SIMD, vector instructions are
// issued in 42% of the cycles (128^3; 47% in a pool of 64^3): bound by the latency
// of dependent instructions, LDS and the exchange, not by their number.
#include "ce_resident.hpp"

#ifndef CE_UNIT_MODEL
#error "compile this file once per model, with -DCE_UNIT_MODEL=0 and -DCE_UNIT_MODEL=1"
#endif

namespace ce {
namespace {

using namespace dev;

// The block is the `rank`-th of the nblk that work the lattice.  RAGGED: a tile
// at the end of a row or column holds vx x vy sites, and every tile zlen <= ZP
// planes (see the tiled pass).
// CHECK: the block checks in here (a pool's has done so).
template <typename T, int NF, int MODEL, int VEC, int LPR, int BS, int ZP, bool RAGGED, bool CHECK>
__device__ __forceinline__ void resident_tiled_body(const Lattice &lat, int src, int steps, int rank, int nblk,
                                                    const Start &start)
{
    constexpr int NQ = kSumsPerField * NF + 1;
    constexpr int TX = VEC * LPR, TY = BS / LPR;
    constexpr int PLANE = (TY + 2) * TX;          // rows -1 .. TY of the tile
    constexpr int FSTRIDE = PLANE + 2 * TY;       // then the columns left and right of it
    constexpr int NY = 2 * ZP * LPR, HY = (NY + BS - 1) / BS;   // halo groups of rows, per thread
    constexpr int NX = 2 * ZP * TY, HX = (NX + BS - 1) / BS;    // halo sites of columns, per thread
    // packed columns: [buffer][tile][left, right][field][d, p][plane][row]
    constexpr unsigned CSTRIDE = NF * 2 * ZP * TY;
    __shared__ __align__(16) T lds[ZP][NF][FSTRIDE];
    __shared__ double red[BS / 64][kMaxSums];
    __shared__ PassScalars<T> next;

    const int N = lat.N;
    const int ntx = RAGGED ? (N + TX - 1) / TX : N / TX, nty = RAGGED ? (N + TY - 1) / TY : N / TY;
    const int nz = RAGGED ? (N + lat.zc - 1) / lat.zc : N / ZP;
    // neighbouring tiles on one XCD, as in the tiled pass
    const int tile = (int)xcd_item(rank, 0, nblk, nblk);
    const int t = threadIdx.x;
    if (t >= BS) {
        if (!CHECK || launch_starts(lat, nblk, start))
            service_wave<T, NF, 1, BS / 64>(lat, steps, rank, nblk, tile, red, next, start);
        return;
    }
    const int wave = t >> 6;
    const int tx = tile % ntx, ty = tile / ntx % nty, tz = tile / (ntx * nty);
    const int x0 = tx * TX, y0 = ty * TY, z0 = RAGGED ? tz * N / nz : tz * ZP;
    const int vx = RAGGED ? min(TX, N - x0) : TX, vy = RAGGED ? min(TY, N - y0) : TY;
    const int zlen = RAGGED ? (tz + 1) * N / nz - z0 : ZP;
    const int q = t % LPR, y = t / LPR;
    const unsigned NN = (unsigned)N * N;
    const bool wrap = ntx == 1;   // a tile row is a lattice row: its ends are neighbours

    // element offsets in an array, and in a plane of LDS
    const bool ok = !RAGGED || (VEC * q < vx && y < vy);   // the thread has sites
    const unsigned own_xy = ok ? (unsigned)((y0 + y) * N + x0 + VEC * q) : (unsigned)(y0 * N + x0);
    const unsigned own = (unsigned)z0 * NN + own_xy;
    const unsigned zoff[2] = {(unsigned)((z0 + N - 1) % N) * NN + own_xy, (unsigned)((z0 + zlen) % N) * NN + own_xy};
    unsigned yoff[HY], xoff[HX], cread[HX];
    int yslot[HY], xslot[HX];
    bool ydo[HY], xdo[HX];
#pragma unroll
    for (int m = 0; m < HY; m++) {
        const int h = t + m * BS;
        const int side = h / (ZP * LPR), k = h / LPR % ZP, g = h % LPR;
        ydo[m] = h < NY && (!RAGGED || (k < zlen && VEC * g < vx));
        yoff[m] = (unsigned)(z0 + k) * NN + (unsigned)(((side ? y0 + vy : y0 + N - 1) % N) * N + x0 + VEC * g);
        yslot[m] = k * (NF * FSTRIDE) + (side ? (vy + 1) * TX : 0) + VEC * g;
    }
#pragma unroll
    for (int m = 0; m < HX; m++) {
        const int h = t + m * BS;
        const int side = h / (ZP * TY), k = h / TY % ZP, r = h % TY;
        xdo[m] = h < NX && !wrap && (!RAGGED || (k < zlen && r < vy));
        xoff[m] = (unsigned)(z0 + k) * NN + (unsigned)((y0 + r) * N + (side ? x0 + vx : x0 + N - 1) % N);
        xslot[m] = k * (NF * FSTRIDE) + PLANE + side * TY + r;
        // the left neighbour's right column is this tile's left one
        const int from = side ? tile + (tx == ntx - 1 ? 1 - ntx : 1) : tile + (tx == 0 ? ntx - 1 : -1);
        cread[m] = (unsigned)(from * 2 + 1 - side) * CSTRIDE + (unsigned)(k * TY + r);
    }
    T *const all = &lds[0][0][0];
    const int left = wrap ? (y + 1) * TX + vx - 1 : PLANE + y;        // the site left of the row
    const int right = wrap ? (y + 1) * TX : PLANE + TY + y;           // and right of it
    const bool row_end = RAGGED ? VEC * (q + 1) == vx : q == LPR - 1;
    const bool edge = y == 0 || y == vy - 1;
    // (a ragged tile may be one thread wide: its sites are both columns)
    const bool column[2] = {ok && !wrap && q == 0, ok && !wrap && row_end};
    const unsigned cwrite = (unsigned)tile * 2 * CSTRIDE + (unsigned)y;

    PassCoef<T, NF> c = make_coef<T, NF, MODEL, kStep>(lat);

    T p[ZP][NF][VEC];
#pragma unroll
    for (int k = 0; k < ZP; k++)
#pragma unroll
        for (int i = 0; i < NF; i++) {
            const unsigned o = (own + (RAGGED ? min(k, zlen - 1) : k) * NN) * (unsigned)sizeof(T);
            const Vec<T, VEC> dq = agent_load_vec<T, VEC>(agent_buffer(lat.d[src][i]), o);
            const Vec<T, VEC> pq = agent_load_vec<T, VEC>(agent_buffer(lat.p[src][i]), o);
            if (ok) store_lds(&lds[k][i][(y + 1) * TX + VEC * q], dq.v);
#pragma unroll
            for (int e = 0; e < VEC; e++) p[k][i][e] = pq.v[e];
        }

    // stored values of the halo at the current step
    Vec<T, VEC> zd[2][NF], zp[2][NF], yd[HY][NF], yp[HY][NF];
    T xd[HX][NF], xp[HX][NF];
    const __amdgpu_buffer_rsrc_t cols = agent_buffer(lat.columns);
    const unsigned csize = nblk * 2 * CSTRIDE;   // of one buffer's columns
    auto load_halo = [&](int buf, bool packed) {
#pragma unroll
        for (int i = 0; i < NF; i++) {
            const __amdgpu_buffer_rsrc_t bd = agent_buffer(lat.d[buf][i]), bp = agent_buffer(lat.p[buf][i]);
#pragma unroll
            for (int s = 0; s < 2; s++) {
                zd[s][i] = agent_load_vec<T, VEC>(bd, zoff[s] * (unsigned)sizeof(T));
                zp[s][i] = agent_load_vec<T, VEC>(bp, zoff[s] * (unsigned)sizeof(T));
            }
#pragma unroll
            for (int m = 0; m < HY; m++)
                if (ydo[m]) {
                    yd[m][i] = agent_load_vec<T, VEC>(bd, yoff[m] * (unsigned)sizeof(T));
                    yp[m][i] = agent_load_vec<T, VEC>(bp, yoff[m] * (unsigned)sizeof(T));
                }
#pragma unroll
            for (int m = 0; m < HX; m++)
                if (xdo[m]) {
                    const unsigned o = buf * csize + cread[m] + i * 2 * ZP * TY;
                    xd[m][i] = packed ? agent_load(cols, o * (unsigned)sizeof(T), T())
                                      : agent_load(bd, xoff[m] * (unsigned)sizeof(T), T());
                    xp[m][i] = packed ? agent_load(cols, (o + ZP * TY) * (unsigned)sizeof(T), T())
                                      : agent_load(bp, xoff[m] * (unsigned)sizeof(T), T());
                }
        }
    };
    load_halo(src, false);   // no step has packed the columns yet
    if (CHECK && !launch_starts(lat, nblk, start)) return;

    for (int step = 0; step < steps; step++) {
        const int out = src ^ 1 ^ (step & 1);
        const bool last = step + 1 == steps;
        // the thread's place in a plane of LDS, as an offset the compiler
        // cannot see through: it would otherwise keep d in registers as well
        int at = (y + 1) * TX + VEC * q;
        asm volatile("" : "+v"(at));
        // drift in place: d becomes the new deviation, p the derivative at n+1/2
        T zn[2][NF][VEC];
#pragma unroll
        for (int i = 0; i < NF; i++) {
#pragma unroll
            for (int k = 0; k < ZP; k++) {
                T d[VEC];
                load_lds(&lds[k][i][at], d);
#pragma unroll
                for (int e = 0; e < VEC; e++) {
                    T fdot, d1;
                    own_drift<T, NF, kStep>(c, i, d[e], p[k][i][e], fdot, d1);
                    d[e] = d1;
                    p[k][i][e] = fdot;
                }
                if (ok) store_lds(&lds[k][i][at], d);
            }
#pragma unroll
            for (int s = 0; s < 2; s++)
#pragma unroll
                for (int e = 0; e < VEC; e++) zn[s][i][e] = nbr_drift<T, NF, kStep>(c, i, zd[s][i].v[e], zp[s][i].v[e]);
#pragma unroll
            for (int m = 0; m < HY; m++)
                if (ydo[m]) {
                    T h[VEC];
#pragma unroll
                    for (int e = 0; e < VEC; e++) h[e] = nbr_drift<T, NF, kStep>(c, i, yd[m][i].v[e], yp[m][i].v[e]);
                    store_lds(all + i * FSTRIDE + yslot[m], h);
                }
#pragma unroll
            for (int m = 0; m < HX; m++)
                if (xdo[m]) all[i * FSTRIDE + xslot[m]] = nbr_drift<T, NF, kStep>(c, i, xd[m][i], xp[m][i]);
        }
        __syncthreads();   // (1)
        double acc[NQ];
#pragma unroll
        for (int j = 0; j < NQ; j++) acc[j] = 0.0;
        asm volatile("" : "+v"(at));
        T below[NF][VEC], cur[NF][VEC], above[NF][VEC];   // planes k-1, k, k+1
#pragma unroll
        for (int i = 0; i < NF; i++) {
#pragma unroll
            for (int e = 0; e < VEC; e++) below[i][e] = zn[0][i][e];
            load_lds(&lds[0][i][at], cur[i]);
        }
#pragma unroll
        for (int k = 0; k < ZP; k++) {
            __builtin_amdgcn_sched_barrier(0);
            if (RAGGED && k >= zlen) break;
            const bool top_plane = RAGGED ? k + 1 == zlen : k + 1 == ZP;
            T lap[VEC][NF];
#pragma unroll
            for (int i = 0; i < NF; i++) {
                const T *P = lds[k][i];
                T xl = lane_from_left(cur[i][VEC - 1]);
                T xr = lane_from_right(cur[i][0]);
                if (q == 0) xl = P[left];
                if (row_end) xr = P[right];
                T up[VEC], dn[VEC];
                load_lds(&P[at - TX], up);
                load_lds(&P[at + TX], dn);
                if (!top_plane) {
                    load_lds(&lds[k + 1 < ZP ? k + 1 : k][i][at], above[i]);
                } else {
#pragma unroll
                    for (int e = 0; e < VEC; e++) above[i][e] = zn[1][i][e];
                }
#pragma unroll
                for (int e = 0; e < VEC; e++) {
                    const T l = e == 0 ? xl : cur[i][e == 0 ? 0 : e - 1];
                    const T r = e == VEC - 1 ? xr : cur[i][e == VEC - 1 ? e : e + 1];
                    const T pr = ((l + r) + (dn[e] + up[e])) + (above[i][e] + below[i][e]);
                    lap[e][i] = fma_t((T)-6, cur[i][e], pr) * c.inv_dx2;
                }
            }
            T part[NQ];
            clear_part(part);
#pragma unroll
            for (int e = 0; e < VEC; e++) {
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
            if (ok) flush_sums(part, acc);
            // add them now: left to itself the compiler sinks every plane's
            // additions to the last one and holds the parts until then (30
            // registers a plane with two FP32 fields)
#pragma unroll
            for (int j = 0; j < NQ; j++) asm volatile("" : "+v"(acc[j]));
            if (ok && (last || edge || k == 0 || top_plane)) {
                const unsigned o = (own + k * NN) * (unsigned)sizeof(T);
#pragma unroll
                for (int i = 0; i < NF; i++) {
                    agent_store(agent_buffer(lat.d[out][i]), o, cur[i]);
                    agent_store(agent_buffer(lat.p[out][i]), o, p[k][i]);
                }
            }
#pragma unroll
            for (int side = 0; side < 2; side++)
                if (column[side]) {
#pragma unroll
                    for (int i = 0; i < NF; i++) {
                        const unsigned o = out * csize + cwrite + side * CSTRIDE + (i * 2 * ZP + k) * TY;
                        agent_store(cols, o * (unsigned)sizeof(T), cur[i][side ? VEC - 1 : 0]);
                        agent_store(cols, (o + ZP * TY) * (unsigned)sizeof(T), p[k][i][side ? VEC - 1 : 0]);
                    }
                }
#pragma unroll
            for (int i = 0; i < NF; i++)
#pragma unroll
                for (int e = 0; e < VEC; e++) {
                    below[i][e] = cur[i][e];
                    cur[i][e] = above[i][e];
                }
        }
        {
            const double v = tree_sum<5, NQ>(acc);
            const int j = tree_index<NQ>();
            if (j >= 0) red[wave][j] = v;
        }
        stores_arrived();
        __syncthreads();   // (2)
        if (nblk > 1) __syncthreads();   // (3)
        if (!last) load_halo(out, true); // while the service wave runs the tail
        __syncthreads();   // (4)
        next_coef<T, NF, MODEL>(c, next);
    }
}

// Waves per SIMD aimed at: three leave 168 registers and room for two blocks on a
// compute unit, where the state of a thread is small enough (two FP32 fields in
// eight planes take 243 registers and get one).
template <typename T, int NF, int BS, int ZP>
constexpr int waves_wanted()
{
    return BS == 256 && sizeof(T) == 4 && NF <= 2 && NF * ZP <= 8 ? 3 : 1;
}

template <typename T, int NF, int MODEL, int VEC, int LPR, int BS, int ZP, bool RAGGED>
__global__ __launch_bounds__(BS + 64, (waves_wanted<T, NF, BS, ZP>())) void
resident_tiled_kernel(Lattice lat, int src, int steps, Start start)
{
    resident_tiled_body<T, NF, MODEL, VEC, LPR, BS, ZP, RAGGED, true>(lat, src, steps, blockIdx.x, gridDim.x, start);
}

// Up to k steps of each of n lattices; see run_members.
template <typename T, int NF, int MODEL, int VEC, int LPR, int BS, int ZP>
__global__ __launch_bounds__(BS + 64, (waves_wanted<T, NF, BS, ZP>())) void
resident_tiled_batched(const Lattice *lats, int n, int nblk, int k, Start start)
{
    run_members(lats, n, nblk, k, start, [&](const Lattice &lat, int src, int steps, int rank, int blocks) {
        resident_tiled_body<T, NF, MODEL, VEC, LPR, BS, ZP, false, false>(lat, src, steps, rank, blocks, start);
    });
}

// Built where p and the halo come near the registers of a thread (a block of five
// waves has 256, one of nine 168: the service wave is the one too many) and the
// tile in LDS.  Some spill and still beat plain launches of the same tiling (us a
// step, resident and plain): three FP64 fields in one plane, 90 spilled, 64^3 8.4
// and 27.5, in two planes, 200, 14.2 and 23.7; three FP32 fields in eight planes,
// 102, 128^3 22.4 and 35.7.
template <typename T, int NF, int VEC, int LPR, int BS, int ZP>
constexpr bool built()
{
    constexpr int tile = (BS / LPR + 2) * VEC * LPR + 2 * (BS / LPR);
    return VEC * ZP * NF * (int)sizeof(T) / 4 <= (BS == 256 ? 96 : 36) &&
           ZP * NF * tile * (int)sizeof(T) <= 150 * 1024;
}

template <typename T, int NF, int MODEL, int VEC, int LPR, int BS, int ZP>
const void *kernel_if_built(bool ragged, bool batched)
{
    if constexpr (built<T, NF, VEC, LPR, BS, ZP>()) {
        // ragged tiles: FP32, eight planes (see ragged_tiling)
        if (ragged) {
            if constexpr (sizeof(T) == 4 && ZP == 8)
                return batched ? nullptr
                               : (const void *)resident_tiled_kernel<T, NF, MODEL, VEC, LPR, BS, ZP, true>;
            return nullptr;
        }
        if (!batched) return (const void *)resident_tiled_kernel<T, NF, MODEL, VEC, LPR, BS, ZP, false>;
        // pools: FP32 tiles of four or eight planes (see member_launch)
        if constexpr (sizeof(T) == 4 && ZP >= 4)
            return (const void *)resident_tiled_batched<T, NF, MODEL, VEC, LPR, BS, ZP>;
    }
    return nullptr;
}

template <typename T, int NF, int MODEL, int VEC, int LPR, int BS>
const void *kernel_planes(int planes, bool ragged, bool batched)
{
    if (ragged) planes = planes <= 8 ? 8 : 0;   // at most that many
    switch (planes) {
    case 1: return kernel_if_built<T, NF, MODEL, VEC, LPR, BS, 1>(ragged, batched);
    case 2: return kernel_if_built<T, NF, MODEL, VEC, LPR, BS, 2>(ragged, batched);
    case 4: return kernel_if_built<T, NF, MODEL, VEC, LPR, BS, 4>(ragged, batched);
    case 8: return kernel_if_built<T, NF, MODEL, VEC, LPR, BS, 8>(ragged, batched);
    default: return nullptr;
    }
}

// FP32: four sites per thread, tiles of 64 x 16 and 32 x 32 sites.  FP64: two
// sites per thread on twice the threads, the same tiles; four spilled.
template <typename T, int NF, int MODEL>
const void *kernel_shape(int vec, int lpr, int bs, int planes, bool ragged, bool batched)
{
    if constexpr (sizeof(T) == 4) {
        if (vec == 4 && lpr == 16 && bs == 256) return kernel_planes<T, NF, MODEL, 4, 16, 256>(planes, ragged, batched);
        if (vec == 4 && lpr == 8 && bs == 256) return kernel_planes<T, NF, MODEL, 4, 8, 256>(planes, ragged, batched);
    } else {
        if (vec == 2 && lpr == 32 && bs == 512) return kernel_planes<T, NF, MODEL, 2, 32, 512>(planes, ragged, batched);
        if (vec == 2 && lpr == 16 && bs == 512) return kernel_planes<T, NF, MODEL, 2, 16, 512>(planes, ragged, batched);
    }
    return nullptr;
}

template <typename T, int MODEL>
const void *kernel_nf(int nf, int vec, int lpr, int bs, int planes, bool ragged, bool batched)
{
    switch (nf) {
    case 1: return kernel_shape<T, 1, MODEL>(vec, lpr, bs, planes, ragged, batched);
    case 2: return kernel_shape<T, 2, MODEL>(vec, lpr, bs, planes, ragged, batched);
    case 3: return kernel_shape<T, 3, MODEL>(vec, lpr, bs, planes, ragged, batched);
    default: return nullptr;
    }
}

}  // namespace

// This unit's model (the source is compiled once per model).
constexpr int kUnit = CE_UNIT_MODEL;

template <>
const void *resident_tiled_model<kUnit>(int precision, int nf, int vec, int lpr, int bs, int planes, bool ragged, bool batched)
{
    return precision == CE_FP64 ? kernel_nf<double, kUnit>(nf, vec, lpr, bs, planes, ragged, batched)
                                : kernel_nf<float, kUnit>(nf, vec, lpr, bs, planes, ragged, batched);
}

}  // namespace ce
