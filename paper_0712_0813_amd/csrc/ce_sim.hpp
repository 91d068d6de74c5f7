// Host-side state of one simulation and the runtime helpers shared by the
// single-lattice API and the batched pool.
#pragma once

#include <mutex>

#include "ce_internal.hpp"

namespace ce {
namespace host {

constexpr size_t kAlign = 256;
constexpr long long kStagingElems = 1LL << 24;  // 128 MiB of FP64 per staging chunk (a 256^3 field in one)

inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

struct Layout {
    size_t field_bytes;   // one array of one field
    size_t off_fields;    // 4 * nf arrays
    size_t off_scalars, off_partials, off_ticket, off_sync, off_ring, off_maxabs, off_staging;
    size_t total;
    long long staging_elems;
    int nblocks;
};


// Every call that uses the GPU holds a Use while it runs.  Cooperative launches
// are taken only by a thread that is alone in the library, and other threads'
// calls wait (some 20 us) while one is: a server whose admission threads worked
// beside such launches ended in a host fault, and what the runtime does with
// them on several threads at once is not known.  Where other threads are in the
// library, the steps are plain or batched launches, with the same results.
class Use {
public:
    Use();
    ~Use();
    Use(const Use &) = delete;
};
class Alone {
public:
    Alone();   // by a thread with a Use
    explicit operator bool() const { return alone; }

private:
    std::lock_guard<std::mutex> lock;
    bool alone;
};

// Record a failure for ce_last_error() and return `st`.
ce_status fail(ce_status st, const char *fmt, ...);

#define CE_HIP(call)                                                                                    \
    do {                                                                                                \
        hipError_t e_ = (call);                                                                         \
        if (e_ != hipSuccess) return ::ce::host::fail(CE_EDEVICE, "%s failed: %s", #call, hipGetErrorString(e_)); \
    } while (0)
long long sites_of(const ce_params *p);
Layout layout_of(const ce_params *p);
ce_status validate(const ce_params *p);
ce_status device_cus(int *cus);

// Device memory of simulations, on the current device.  A destroyed
// simulation's memory is kept for the next one of its size (allocating 1.3 GB
// and giving it back took 15 ms of starting a 256^3 run over and over, the run's
// own work 1.5 ms): at most kKeptBytes in kKeptBlocks blocks, the oldest given
// back first, all of it as soon as an allocation fails.  Any thread may call
// these; nothing queued uses memory that is handed to release_device_memory.
constexpr size_t kKeptBytes = (size_t)4 << 30;
constexpr int kKeptBlocks = 8;
hipError_t device_memory(size_t bytes, void **out);
void release_device_memory(void *mem, size_t bytes, int device);
void give_back_kept_memory();

// A word of page-locked memory, zero, that a resident launch writes if its
// lattice halts (see Halt), so that the host learns of it with no copy; nullptr
// if none is left (of kHaltWords, allocated by the process's first simulation
// and held until it ends), and no resident pass is planned then.
constexpr int kHaltWords = 1024;
void ready_halt_words();
unsigned *take_halt_word();
void give_halt_word(unsigned *w);

// Steps of one resident launch at most: a millisecond or two, for which other
// work on the GPU may have to wait.
constexpr int kResidentSteps = 256;

// Ticks of the GPU's clock (100 MHz) a resident launch waits for its blocks.
// A launch queued behind another's blocks gets its units within that one's
// time (at most some milliseconds of a resident launch, 7 ms of a 1024^3 pass,
// of which a few may come first).
constexpr unsigned long long kTicksPerMs = 100000;
constexpr unsigned long long kStartWait = 200 * kTicksPerMs;

}  // namespace host
}  // namespace ce

struct ce_sim {
    ce_params p;
    ce::host::Layout lay;
    ce::Lattice lat;
    hipStream_t stream = nullptr;
    bool own_stream = false;
    hipStream_t cap_stream = nullptr;
    char *base = nullptr;
    bool own_mem = false;
    int device = 0;         // where base is
    double *staging = nullptr;
    unsigned int *maxabs = nullptr;
    int cur = 0;            // buffer holding the current state
    long long step = 0;
    unsigned loaded = 0;    // bit per field
    bool started = false;
    int step_block = 32;
    double m_host[CE_MAX_FIELDS] = {0, 0, 0};  // homogeneous references at load time
    ce_launch launch{CE_KERNEL_DIRECT, 0, 0, 0, 0, 0};
    int grid = 0;           // blocks of the launch as reported (a ragged tiling may use fewer)
    hipGraphExec_t graph[2] = {nullptr, nullptr};  // step block starting from buffer 0 / 1
    int graph_k = 0;
    // resident pass for the current launch (kernel nullptr: none)
    struct Resident {
        const void *kernel = nullptr;
        int blocks = 0, threads = 0, min_steps = 0;
    } resident;
    bool resident_planned = false;   // for the launch as it is now
    unsigned *halt = nullptr;        // set by a resident launch that left the lattice halted
    bool unsettled = false;          // a resident launch has been queued since settle()
    unsigned long long wait = ce::host::kStartWait;
};

namespace ce {
namespace host {

// Validate a launch configuration for the simulation and apply it.
ce_status apply_launch(ce_sim *s, const ce_launch &cfg);
// Every field is present (loaded or generated): check leapfrog stability with
// the recorded field maxima and queue the start-up half step.
ce_status start_run(ce_sim *s);
void drop_graphs(ce_sim *s);
// After a launch that did not start: blocks check in from none again.
hipError_t clear_arrivals(ce_sim *s);
// The steps that queued launches left out of a halted lattice, by plain launches
// on its stream, which has nothing else queued; it has run when this returns.
// left: of a pool's member, the steps it still has to be given (its scalar
// state then says so, and in which buffer it is).
ce_status take_missing_steps(ce_sim *s, const long long *left);
// The same for a simulation whose stream has been waited for: nothing to do
// unless a launch set its halt word.
ce_status settle(ce_sim *s);
inline bool halt_seen(const ce_sim *s) { return s->halt && __atomic_load_n(s->halt, __ATOMIC_ACQUIRE) != 0; }
// Kernel of the resident pass of a tiled (ragged: on ragged tiles) or 2-D
// streaming launch with one tile or group of units per block (batched: of its
// pool form), nullptr if none.
const void *resident_kernel(const ce_params *p, const ce_launch &c, bool ragged, bool batched);

}  // namespace host
}  // namespace ce
