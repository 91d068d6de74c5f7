// Resident form of the direct pass (any dimension): many steps of a lattice
// that one quad (4 x-sites) per thread covers, in one launch.  See
// ce_resident.hpp for the exchange between blocks.
//
// Block b owns the quads [b Q, (b+1) Q), Q = 256 VB threads, which are VB
// consecutive blocks of the direct pass's launch: thread t's quad, the
// arithmetic of a site, and the sums' order (lane tree, waves in order, the VB
// rows of the block in order, then the rows as finish_pass adds them) are
// those of the direct pass, so a step taken here is bitwise a step taken
// there.  A neighbour quad inside the block comes from LDS, any other from
// the neighbour's published sites; whether a quad has to be published is the
// same question asked by the other side (the stencil is symmetric).
//
// Bound by latency: the sites, their sums, the exchange of the sums and the
// tail follow one another (a 1024-site FP64 line: 1.9 us a step against 5.2
// plain; 32^3 x 2 fields, 32 blocks: 4.4 against 8.8).
#include "ce_resident.hpp"

#ifndef CE_UNIT_MODEL
#error "compile this file once per model, with -DCE_UNIT_MODEL=0 and -DCE_UNIT_MODEL=1"
#endif

namespace ce {
namespace {

using namespace dev;

template <typename T, int D, int NF, int MODEL, int VB>
__global__ __launch_bounds__(kBlock *VB + 64) void resident_direct_kernel(Lattice lat, int src, int steps, Start start)
{
    constexpr int NQ = kSumsPerField * NF + 1;
    constexpr int Q = kBlock * VB;
    constexpr int ND = 2 * (D - 1);   // y+, y-, z+, z-
    __shared__ __align__(16) T lds[NF][4 * Q];
    __shared__ double red[4 * VB][kMaxSums];
    __shared__ PassScalars<T> next;

    const int t = threadIdx.x, wave = t >> 6;
    if (t >= Q) {
        if (launch_starts(lat, gridDim.x, start))
            service_wave<T, NF, VB, 4>(lat, steps, blockIdx.x, gridDim.x, blockIdx.x, red, next, start);
        return;
    }
    const int N = lat.N;
    const int nquads = (int)(lat.nsites / 4);
    const int rowq = N / 4;
    const int q0 = blockIdx.x * Q;
    const int nblk = gridDim.x;
    const int me = q0 + t;
    const bool own = me < nquads;
    const int nown = min(Q, nquads - q0);

    // neighbour quads: x-, x+, then y+, y-, z+, z-
    int nbr[2 + ND];
    {
        const int k = own ? me : q0;
        const int row = k / rowq, xq = k - row * rowq;
        nbr[0] = xq == 0 ? k + rowq - 1 : k - 1;
        nbr[1] = xq == rowq - 1 ? k - (rowq - 1) : k + 1;
        if constexpr (D >= 2) {
            const int y = row % N;
            nbr[2] = y == N - 1 ? k - (N - 1) * rowq : k + rowq;
            nbr[3] = y == 0 ? k + (N - 1) * rowq : k - rowq;
        }
        if constexpr (D == 3) {
            const int plane = rowq * N;
            const int z = row / N;
            nbr[4] = z == N - 1 ? k - (N - 1) * plane : k + plane;
            nbr[5] = z == 0 ? k + (N - 1) * plane : k - plane;
        }
    }
    // far: the neighbour is another block's
    bool far[2 + ND], shared_quad = false;
#pragma unroll
    for (int n = 0; n < 2 + ND; n++) {
        far[n] = own && (unsigned)(nbr[n] - q0) >= (unsigned)nown;
        shared_quad |= far[n];
    }

    PassCoef<T, NF> c = make_coef<T, NF, MODEL, kStep>(lat);

    T d[NF][4], p[NF][4];
#pragma unroll
    for (int i = 0; i < NF; i++) {
        Quad<T> dq{}, pq{};
        if (own) {
            // agent scope like every access to the arrays here: no line of
            // them may stay in an L2
            dq = agent_load_quad(agent_buffer(lat.d[src][i]), (unsigned)me * (4u * sizeof(T)), T());
            pq = agent_load_quad(agent_buffer(lat.p[src][i]), (unsigned)me * (4u * sizeof(T)), T());
        }
#pragma unroll
        for (int e = 0; e < 4; e++) {
            d[i][e] = dq.v[e];
            p[i][e] = pq.v[e];
        }
    }

    // stored values of the far neighbours at the current step
    Quad<T> fd[ND > 0 ? ND : 1][NF], fp[ND > 0 ? ND : 1][NF];
    T xd[2][NF], xp[2][NF];
#pragma unroll
    for (int i = 0; i < NF; i++) {
#pragma unroll
        for (int n = 0; n < ND; n++) fd[n][i] = fp[n][i] = Quad<T>{};
        xd[0][i] = xd[1][i] = xp[0][i] = xp[1][i] = (T)0;
    }
    auto load_far = [&](int buf) {
#pragma unroll
        for (int i = 0; i < NF; i++) {
            const __amdgpu_buffer_rsrc_t bd = agent_buffer(lat.d[buf][i]), bp = agent_buffer(lat.p[buf][i]);
#pragma unroll
            for (int n = 0; n < ND; n++)
                if (far[2 + n]) {
                    const unsigned o = (unsigned)nbr[2 + n] * (4u * sizeof(T));
                    fd[n][i] = agent_load_quad(bd, o, T());
                    fp[n][i] = agent_load_quad(bp, o, T());
                }
#pragma unroll
            for (int n = 0; n < 2; n++)
                if (far[n]) {
                    const unsigned o = ((unsigned)nbr[n] * 4u + (n == 0 ? 3u : 0u)) * sizeof(T);
                    xd[n][i] = agent_load(bd, o, T());
                    xp[n][i] = agent_load(bp, o, T());
                }
        }
    };
    if (nblk > 1) load_far(src);
    if (!launch_starts(lat, nblk, start)) return;

    for (int step = 0; step < steps; step++) {
        const int out = src ^ 1 ^ (step & 1);
        const bool last = step + 1 == steps;
        // drift; the drifted quad goes to LDS for its neighbours in the block
        T fdot[NF][4];
#pragma unroll
        for (int i = 0; i < NF; i++) {
            T d1[4];
#pragma unroll
            for (int e = 0; e < 4; e++) {
                own_drift<T, NF, kStep>(c, i, d[i][e], p[i][e], fdot[i][e], d1[e]);
                d[i][e] = d1[e];
            }
            store_lds(&lds[i][4 * t], d1);
        }
        __syncthreads();   // (1)
        double acc[NQ];
#pragma unroll
        for (int q = 0; q < NQ; q++) acc[q] = 0.0;
        if (own) {
            T lap[4][NF];
#pragma unroll
            for (int i = 0; i < NF; i++) {
                const T dl = far[0] ? nbr_drift<T, NF, kStep>(c, i, xd[0][i], xp[0][i]) : lds[i][4 * (nbr[0] - q0) + 3];
                const T dr = far[1] ? nbr_drift<T, NF, kStep>(c, i, xd[1][i], xp[1][i]) : lds[i][4 * (nbr[1] - q0)];
                T pair[4];
                pair[0] = dl + d[i][1];
                pair[1] = d[i][0] + d[i][2];
                pair[2] = d[i][1] + d[i][3];
                pair[3] = d[i][2] + dr;
                T nb[ND > 0 ? ND : 1][4];
#pragma unroll
                for (int n = 0; n < ND; n++) {
                    if (far[2 + n]) {
#pragma unroll
                        for (int e = 0; e < 4; e++)
                            nb[n][e] = nbr_drift<T, NF, kStep>(c, i, fd[n][i].v[e], fp[n][i].v[e]);
                    } else {
                        load_lds(&lds[i][4 * (nbr[2 + n] - q0)], nb[n]);
                    }
                }
#pragma unroll
                for (int n = 0; n < ND; n += 2) {
#pragma unroll
                    for (int e = 0; e < 4; e++) pair[e] += nb[n][e] + nb[n + 1][e];
                }
#pragma unroll
                for (int e = 0; e < 4; e++) lap[e][i] = fma_t((T)(-2 * D), d[i][e], pair[e]) * c.inv_dx2;
            }
            T part[NQ];
            clear_part(part);
#pragma unroll
            for (int e = 0; e < 4; e++) {
                T d1s[NF], fds[NF], pn[NF];
#pragma unroll
                for (int i = 0; i < NF; i++) {
                    d1s[i] = d[i][e];
                    fds[i] = fdot[i][e];
                }
                site_update<T, NF, MODEL, kStep, NQ>(c, d1s, fds, lap[e], pn, part);
#pragma unroll
                for (int i = 0; i < NF; i++) p[i][e] = pn[i];
            }
            if (last || shared_quad) {
                const unsigned o = (unsigned)me * (4u * sizeof(T));
#pragma unroll
                for (int i = 0; i < NF; i++) {
                    agent_store(agent_buffer(lat.d[out][i]), o, d[i]);
                    agent_store(agent_buffer(lat.p[out][i]), o, p[i]);
                }
            }
            flush_sums(part, acc);
        }
        {
            const double v = tree_sum<5, NQ>(acc);
            const int q = tree_index<NQ>();
            if (q >= 0) red[wave][q] = v;
        }
        if (nblk > 1) stores_arrived();
        __syncthreads();   // (2)
        if (nblk > 1) {
            __syncthreads();   // (3)
            if (!last) load_far(out);   // while the service wave runs the tail
        }
        __syncthreads();   // (4)
        next_coef<T, NF, MODEL>(c, next);
    }
}

// Largest VB built: the quads of the four y and z neighbours stay in registers
// beside the state, and a larger block has fewer (68^3 x 3 fields on two blocks
// as one: 17.1 us a step spilled, 14.8 plain).
template <typename T, int D, int NF>
constexpr int max_vb()
{
    constexpr int words = NF * (int)sizeof(T) / 4;
    return D == 3 ? (words == 1 ? 3 : words == 2 ? 2 : 1) : words <= 2 ? 3 : words <= 4 ? 2 : 1;
}

template <typename T, int D, int NF, int MODEL>
const void *kernel_vb(int vb)
{
    if (vb == 1) return (const void *)resident_direct_kernel<T, D, NF, MODEL, 1>;
    if constexpr (max_vb<T, D, NF>() >= 2)
        if (vb == 2) return (const void *)resident_direct_kernel<T, D, NF, MODEL, 2>;
    if constexpr (max_vb<T, D, NF>() >= 3)
        if (vb == 3) return (const void *)resident_direct_kernel<T, D, NF, MODEL, 3>;
    return nullptr;
}

template <typename T, int D, int MODEL>
const void *kernel_nf(int nf, int vb)
{
    switch (nf) {
    case 1: return kernel_vb<T, D, 1, MODEL>(vb);
    case 2: return kernel_vb<T, D, 2, MODEL>(vb);
    case 3: return kernel_vb<T, D, 3, MODEL>(vb);
    default: return nullptr;
    }
}

template <typename T, int MODEL>
const void *kernel_dims(int dims, int nf, int vb)
{
    switch (dims) {
    case 1: return kernel_nf<T, 1, MODEL>(nf, vb);
    case 2: return kernel_nf<T, 2, MODEL>(nf, vb);
    case 3: return kernel_nf<T, 3, MODEL>(nf, vb);
    default: return nullptr;
    }
}

}  // namespace

// This unit's model (the source is compiled once per model).
constexpr int kUnit = CE_UNIT_MODEL;

template <>
const void *resident_direct_model<kUnit>(int precision, int dims, int nf, int vb)
{
    return precision == CE_FP64 ? kernel_dims<double, kUnit>(dims, nf, vb) : kernel_dims<float, kUnit>(dims, nf, vb);
}

}  // namespace ce
