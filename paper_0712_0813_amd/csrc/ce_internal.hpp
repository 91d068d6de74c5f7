// Internal declarations shared by the host runtime and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ce.h"

namespace ce {

constexpr int kMaxFields = CE_MAX_FIELDS;
constexpr int kMaxTerms = CE_MAX_TERMS;
// Model of the potential, a compile-time parameter of every pass kernel.
enum ModelKind { kQuartic = CE_MODEL_QUARTIC, kPoly = CE_MODEL_POLYNOMIAL };
constexpr int kLogCap = CE_ENERGY_LOG;
// FP64 volume sums per field (see the kernels for their meaning), plus sum V
constexpr int kSumsPerField = 6;
constexpr int kMaxSums = kSumsPerField * kMaxFields + 1;
constexpr int kBlock = 256;

// Per-field coefficients of one step pass in the storage type T.
template <typename T>
struct PassScalars {
    T beta;                 // deferred c-term coefficient
    T bm[kMaxFields];       // beta * m, rounded once
    T r[kMaxFields];        // reference derivative
    T m1[kMaxFields];       // reference field at n+1, rounded once
    T m2a[kMaxFields];      // a_{n+1}^2 mu2_i
    T hm[kMaxFields];       // a_{n+1}^2 mu2_i / 2
    T tc[kMaxTerms];        // polynomial model: coef_t a_{n+1}^(4 - D_t)
};

// FP64 scalar state of one lattice at integer step n, resident on the device.
//
// Storage split: field i at step n is f_i(x) = m[i] + d_i(x), with the
// homogeneous reference m[i] in FP64 and the deviation d_i in the storage
// type; the derivative at n+1/2 is fdot_i(x) = p_i(x) + beta (m[i] + d_i(x)).
struct Scalars {
    double a;          // a^n
    double a_next;     // a^{n+1} = a^n + dt a'^{n+1/2}
    double adot_half;  // a'^{n+1/2}
    double beta;       // deferred c-term coefficient (see above)
    double tau;
    long long step;
    long long first_bad;            // first step with a non-finite sum, -1 if none
    long long remaining;            // pool members: steps still to take (0: the lattice is idle)
    int cur;                        // pool members: buffer holding the current state
    int halted;                     // Halt: why the lattice stands still, 0 if it does not
    double m[kMaxFields];           // homogeneous reference of f_i at step n
    double fdot_mean[kMaxFields];   // volume mean of fdot_i^{n+1/2}
    double r[kMaxFields];           // fdot_mean rounded to the storage type
    // Coefficients of the next step pass, derived from the values above by
    // whoever wrote them last (start-up or step tail), in both storage types.
    // Kernels read them with scalar loads.
    PassScalars<float> nxf;
    PassScalars<double> nxd;
    double nx_m1[kMaxFields];       // m + dt r: FP64 reference at n+1
    double nx_hm[kMaxFields];       // a_{n+1}^2 mu2_i / 2
};

// One lattice as the kernels see it.  d[b][i], p[b][i]: buffer b (ping-pong)
// of field i, element type per precision.
struct Lattice {
    void *d[2][kMaxFields];
    void *p[2][kMaxFields];
    int dims, N, nf, expansion;
    long long nsites;
    double dt, inv_dx2, lambda, kappa, vacuum;
    double G[kMaxFields], mu2[kMaxFields];
    float dt_f, inv_dx2_f, lambda_f, G_f[kMaxFields];  // the same, rounded to FP32
    float qlam_f, hG_f[kMaxFields];                     // lambda/4, G/2 in FP32
    // polynomial model: the terms of degree >= 1 (constant terms are summed
    // into `vacuum`): coefficient, exponent per field, total degree
    int model, nterms;
    double tcoef[kMaxTerms];
    int texp[kMaxTerms][kMaxFields];
    int tdeg[kMaxTerms];
    Scalars *sc;
    double *partials;      // [kMaxSums][slots]: per sum, one entry per block or per tile (tiled pass)
    unsigned int *ticket;  // last-block counter, then the tiled pass's tile counters; 0 between launches
    int slots;             // entries per sum in `partials` (at least kMaxBlocks)
    ce_energy *ring;       // [kLogCap]
    unsigned long long *sync;  // resident passes: published sums [2][2 kMaxSums][kSyncRows], then totals [2][8][kTotalWords], the last step's tag, the blocks checked in
    void *columns;         // resident passes: edge columns of the tiles or units (the staging chunk, idle during steps)
    int nblocks;           // blocks of the step launch (fixed per lattice)
    int kind;              // kDirect or kTiled3d
    int vec;               // tiled: consecutive x sites per thread (2 or 4)
    int lpr;               // tiled: threads per tile row (tile is vec*lpr x bs/lpr sites)
    int bs;                // tiled: threads per block
    int ragged;            // tiled: tiles at the ends of rows and columns are cut short
    int zc;                // tiled: planes streamed per tile; 2-D streaming: rows per unit
    int per_group;         // 2-D streaming, batched: sums per group of units, as when each has its block
    int first_block;       // batched launches: this lattice's first block
};

enum Kind { kDirect = 0, kTiled3d = 1, kStream2d = 2 };
constexpr int kMaxBlocks = 4096;  // blocks per launch; partial-sum rows per lattice at least this
constexpr int kRunRows = 3;      // blocks of the direct pass that one resident block takes at most
constexpr int kSyncRows = 256;    // blocks of a resident pass at most
constexpr int kTotalWords = 48;  // words kept for one copy of the totals (2 kMaxSums, whole lines)
constexpr int kTotalCopies = 8;  // of the totals
constexpr int kLastTag = 2 * (2 * kMaxSums * kSyncRows + kTotalCopies * kTotalWords);  // Lattice::sync: the last step's tag
constexpr int kArrivals = kLastTag + 1;   // and the blocks checked in
constexpr int kSyncWords = kLastTag + 2;
constexpr int kTileCounters = 8;  // the tiled pass's tile counters, one per XCD, after the ticket

enum Mode { kStep = 0, kInit = 1, kGuardedStep = 2 };   // the last: kStep that leaves a halted lattice alone

// Scalars::halted.  Blocks of a resident launch wait for each other, so none
// of them works before all of them run.  Where that does not come about in time
// (other work holds the compute units), the launch ends with the state as it
// was and kNotStarted; every later step leaves such a lattice alone until the
// host, which sees the launch's halt word, has taken the missing steps by plain
// launches (a pool's member has no steps left to take until then).  kLost: a block that had started stopped; the sums are lost.
enum Halt { kRuns = 0, kNotStarted = 1, kLost = 2 };

// What a resident launch's blocks agree with on whether it starts.
struct Start {
    unsigned long long wait;   // ticks (100 MHz) to wait for the other blocks; 0: do not start
    unsigned *halt;            // page-locked host memory: set to 1 when a lattice halts
};

// Launch one pass over `lat` reading buffer `src` and writing buffer 1-src
// (kStep, kGuardedStep) or updating the derivative of buffer `src` in place
// (kInit).
hipError_t launch_pass(const Lattice &lat, int precision, int src, Mode mode, hipStream_t st);

// Each kernel family is compiled once per model (the source built with
// CE_UNIT_MODEL = kQuartic and = kPoly); these are the per-model entry points
// the dispatchers above pick from by lat.model.
template <int MODEL>
hipError_t launch_direct_model(const Lattice &lat, int precision, int src, Mode mode, hipStream_t st);
template <int MODEL>
hipError_t launch_batched_direct_model(const Lattice *lats, const int *blk_lat, int total_blocks, int grid,
                                       const Lattice &proto, int precision, hipStream_t st);
template <int MODEL>
int direct_batched_resident_model(const Lattice &proto, int precision);
template <int MODEL>
hipError_t launch_tiled_model(const Lattice &lat, int precision, int src, Mode mode, hipStream_t st);
template <int MODEL>
hipError_t launch_batched_tiled_model(const Lattice *lats, const int *blk_lat, int total_blocks, int grid,
                                      const Lattice &proto, int precision, hipStream_t st);
template <int MODEL>
int tiled_batched_resident_model(const Lattice &proto, int precision);
template <int MODEL>
int tiled_resident_blocks_model(int precision, int nf, int vec, int lpr, int bs);
template <int MODEL>
hipError_t launch_stream2d_model(const Lattice &lat, int precision, int src, Mode mode, hipStream_t st);
template <int MODEL>
hipError_t launch_batched_stream2d_model(const Lattice *lats, const int *blk_lat, int total_blocks, int grid,
                                         const Lattice &proto, int precision, hipStream_t st);
template <int MODEL>
int stream2d_batched_resident_model(const Lattice &proto, int precision);
// Kernel of the resident direct pass (vb consecutive blocks of the direct
// launch per block), nullptr where that is not built.  Arguments: Lattice,
// int src, int steps, Start; 256 vb + 64 threads.
template <int MODEL>
const void *resident_direct_model(int precision, int dims, int nf, int vb);
// The same of the tiled 3-D pass (tiles of `planes` whole planes, one per
// block; bs + 64 threads), and of its batched form: arguments const Lattice
// *lats, int lattices, int tiles of each, int steps, Start.
template <int MODEL>
const void *resident_tiled_model(int precision, int nf, int vec, int lpr, int bs, int planes, bool ragged,
                                 bool batched);
// The same of the 2-D streaming pass (units of `rows` rows, a group of four per
// block; 320 threads) and its batched form.
template <int MODEL>
const void *resident_stream2d_model(int precision, int nf, int rows, bool batched);
#define CE_DECLARE_MODEL_ENTRIES(M)                                                                             \
    template <> hipError_t launch_direct_model<M>(const Lattice &, int, int, Mode, hipStream_t);                \
    template <> hipError_t launch_batched_direct_model<M>(const Lattice *, const int *, int, int, const Lattice &, \
                                                          int, hipStream_t);                                     \
    template <> int direct_batched_resident_model<M>(const Lattice &, int);                                     \
    template <> const void *resident_direct_model<M>(int, int, int, int);                                       \
    template <> const void *resident_tiled_model<M>(int, int, int, int, int, int, bool, bool);                  \
    template <> const void *resident_stream2d_model<M>(int, int, int, bool);                                    \
    template <> hipError_t launch_tiled_model<M>(const Lattice &, int, int, Mode, hipStream_t);                 \
    template <> hipError_t launch_batched_tiled_model<M>(const Lattice *, const int *, int, int, const Lattice &, \
                                                         int, hipStream_t);                                      \
    template <> int tiled_batched_resident_model<M>(const Lattice &, int);                                      \
    template <> int tiled_resident_blocks_model<M>(int, int, int, int, int);                                    \
    template <> hipError_t launch_stream2d_model<M>(const Lattice &, int, int, Mode, hipStream_t);              \
    template <> hipError_t launch_batched_stream2d_model<M>(const Lattice *, const int *, int, int,             \
                                                            const Lattice &, int, hipStream_t);                  \
    template <> int stream2d_batched_resident_model<M>(const Lattice &, int);
CE_DECLARE_MODEL_ENTRIES(kQuartic)
CE_DECLARE_MODEL_ENTRIES(kPoly)
#undef CE_DECLARE_MODEL_ENTRIES

// Blocks a direct pass over this lattice uses (fixes the reduction order).
int pass_blocks(int dims, int N);
// Tiled 3-D pass: whether (N, lpr, zc) fits, its tile count, and the largest
// grid that keeps every block resident.
// Whether launch_pass has kGuardedStep for this launch (every direct and 2-D
// streaming one, tiled ones of the shapes a resident pass takes).
bool guarded_built(const Lattice &lat, int precision);
bool tiled_shape_built(int vec, int lpr, int bs);
bool tiled_fits(int dims, int N, int vec, int lpr, int bs, int zc);
long long tiled_tiles(int N, int vec, int lpr, int bs, int zc);
// The tiling a direct launch of a lattice that no tile divides runs on, if any
// (4 sites per thread, 256 threads).
struct RaggedTiling {
    int lpr, planes;
    int tiles;
};
bool ragged_tiling(int precision, int dims, int N, RaggedTiling *out);
int tiled_resident_blocks(int model, int precision, int nf, int vec, int lpr, int bs);
hipError_t launch_tiled(const Lattice &lat, int precision, int src, Mode mode, hipStream_t st);

// One step pass over many lattices of one class (same precision, dims,
// field count and kernel shape).  lats: device array of descriptors;
// blk_lat: lattice index of every per-lattice block (total_blocks entries).
// `grid` hardware blocks (1..total_blocks) walk the per-lattice blocks
// b, b + grid, ...; each per-lattice block computes exactly what block
// (b - first_block) of a lone launch of its lattice computes.  Each lattice
// reads its buffer parity from its scalar state and is skipped once its
// remaining-step count is 0.
hipError_t launch_batched(const Lattice *lats, const int *blk_lat, int total_blocks, int grid, const Lattice &proto,
                          int precision, hipStream_t st);
// Blocks of the class's batched kernel that fit on one compute unit.
int batched_resident_blocks(const Lattice &proto, int precision);
hipError_t launch_batched_tiled(const Lattice *lats, const int *blk_lat, int total_blocks, int grid,
                                const Lattice &proto, int precision, hipStream_t st);
int tiled_batched_resident(const Lattice &proto, int precision);

// 2-D streaming pass: units of 256 x sites by `rows` rows, four per block.
bool stream2d_fits(int dims, int N, int rows);
long long stream2d_groups(int N, int rows);
int stream2d_resident_blocks();
hipError_t launch_stream2d(const Lattice &lat, int precision, int src, Mode mode, hipStream_t st);
hipError_t launch_batched_stream2d(const Lattice *lats, const int *blk_lat, int total_blocks, int grid,
                                   const Lattice &proto, int precision, hipStream_t st);
int stream2d_batched_resident(const Lattice &proto, int precision);

// dst = (storage)(src - ref) for one chunk, plus running max |src| (as float bits).
hipError_t launch_convert(const double *src, double ref, void *dst, int precision, long long n,
                          unsigned int *maxabs_bits, hipStream_t st);
// storage -> FP64 readback of field `field`: f = m + d and the derivative as a
// step rebuilds it.  sites == NULL: the n consecutive sites from `first`;
// otherwise the n listed sites.
hipError_t launch_readback(const Lattice &lat, int precision, int buf, int field, int started,
                           long long first, const long long *sites, long long n, double *out_f,
                           double *out_fdot, hipStream_t st);

}  // namespace ce
