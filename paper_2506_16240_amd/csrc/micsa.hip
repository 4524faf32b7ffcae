// libmicsa: host side of the C ABI declared in include/micsa.h.
//
// The context owns the device state of S*R lattices in the byte layout
// (geometry.hpp), the installed schedule, the sweep counter k and an energy
// tally per lattice.  Every entry point validates its arguments, enqueues
// kernels on the context's stream and reports failures as status codes.
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>

#include <atomic>
#include <chrono>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <algorithm>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "bitplane_kernels.hpp"
#include "bitplane_sweep.hpp"
#include "cells.hpp"
#include "fused_kernels.hpp"
#include "fused2_kernels.hpp"
#include "msc_kernels.hpp"
#include "msc2_kernels.hpp"
#include "observables.hpp"
#include "pins.hpp"
#include "micsa.h"

using namespace micsa;

namespace micsa {

static std::mutex g_pin_lock;
static struct {
    int device;
    uint8_t* p;
} g_pins[kIdlePins];
static size_t g_pin_count = 0;

uint8_t* take_pin(int device)
{
    {
        std::lock_guard<std::mutex> hold(g_pin_lock);
        for (size_t i = 0; i < g_pin_count; ++i)
            if (g_pins[i].device == device) {
                uint8_t* p = g_pins[i].p;
                g_pins[i] = g_pins[--g_pin_count];
                return p;
            }
    }
    void* p = nullptr;
    if (hipHostMalloc(&p, kPinHead + kPinBytes, hipHostMallocDefault) == hipSuccess) return static_cast<uint8_t*>(p);
    (void)hipGetLastError();
    return nullptr;
}

void give_pin(int device, uint8_t* pin)
{
    {
        std::lock_guard<std::mutex> hold(g_pin_lock);
        if (g_pin_count < kIdlePins) {
            g_pins[g_pin_count++] = {device, pin};
            return;
        }
    }
    (void)hipHostFree(pin);
}

}  // namespace micsa

namespace {

constexpr int kBlock = 256;
constexpr int kTimingKinds = 5;
enum TimingKind { kTimeSweep = 0, kTimeRefresh = 1, kTimeHeatBath = 2, kTimeReduce = 3, kTimeMetropolis = 4 };
constexpr int kAlgos = 4;  // MICSA, HEATBATH, WALKERS, METROPOLIS

struct Schedule {
    bool set = false;
    int32_t kind = MICSA_SCHED_CONST;
    int32_t period = 1;
    double T0 = 1.0, T1 = 1.0;
    int64_t n_sweeps = 0;
    int64_t n_steps = 0;  // timesteps that start in [0, n_sweeps): ceil(n_sweeps / gamma)
    std::vector<double> table;
};

// Where the state of a captured context lies between calls (see rest_state):
// in the planes or in the layout's own arrays, in which copies, and the
// wanderings that the levels there owe.
struct Rest {
    bool planes = false;
    uint8_t *spin = nullptr, *dem = nullptr;
    uint64_t *bspin = nullptr, *bdm0 = nullptr, *bdm1 = nullptr;
    uint64_t *ms = nullptr, *md0 = nullptr, *md1 = nullptr;
    uint8_t fcur[6] = {};
    int32_t fowed[6] = {};
    int32_t pend = -1;
};

// How the cell sweep runs a context's lattices.
struct CellPlan {
    bool ok = false;
    CellTile f{};
    int nr = 1, xm = 0;
    unsigned block = 64;
    int sweeps = 0;   // sweeps per launch of a tiled lattice; 0: the tile is the lattice, any number
    double cost = 0;  // estimated cycles per sweep of every lattice
    double load = 0;  // of a launch's operands
    double brief = 0;  // of a short call (CellPlans): of the whole call
};

// The plan of long calls and, where that has tiles, of what a call's last n <=
// kBriefSweeps sweeps run on: rings for six sweeps cost a launch of one sweep
// several times the lattice (8 x 400 x 400 x 8 28.7 us, 19.0 per byte half).
constexpr int kBriefSweeps = 8;
struct CellPlans {
    CellPlan main, brief[kBriefSweeps + 1];
    CellPlan walk;  // of long calls of one walker per site, whose kernels hold more in registers
};

// Device blocks and streams that a serving pool hands from one job to the next.
// Allocating and freeing them per job cost a pool of 16 jobs 33 of its 76 ms:
// a free waits for everything the device has in flight, of other jobs too, and
// the device then idles until the host has fed it again.  A block is given
// back once its job's streams have finished, so the next job may write it at
// once, if it is at most a quarter larger than the job needs and within what
// the job may hold.  What lies idle is bounded by limit (the budget less what the
// admitted jobs are charged) and freed when the pool holds no job.  Contexts of
// one pool may be used from several threads: every access holds the lock.
struct JobStore {
    struct Block {
        int device;
        size_t bytes;
        void* p;
        bool kept = false;  // a captured graph may hold its address
    };
    std::mutex lock;
    std::vector<Block> idle;  // oldest first
    std::vector<std::pair<int, hipStream_t>> streams;
    size_t held = 0, limit = 0;  // bytes of idle, and their bound

    static constexpr size_t kStreams = 32;  // idle streams kept at most

    void trim(size_t to)
    {
        size_t n = 0;
        while (n < idle.size() && held > to) {
            held -= idle[n].bytes;
            (void)hipFree(idle[n++].p);
        }
        idle.erase(idle.begin(), idle.begin() + (long)n);
    }
    ~JobStore()
    {
        trim(0);
        for (auto& s : streams) (void)hipStreamDestroy(s.second);
    }
};

}  // namespace

struct micsa_ctx {
    micsa_params p{};
    hipStream_t stream = nullptr;
    // a pool's small jobs sweep on this stream, the pool's; `stream` is another
    // one while such a job is set up and after it has finished (see micsa_pool)
    hipStream_t sweep_stream = nullptr;
    // device memory: blocks of this context, from the pool's store if it has
    // one; what is known at creation lies in the first, filled from its start
    JobStore* store = nullptr;
    std::vector<JobStore::Block> owned;
    uint8_t* arena = nullptr;
    size_t arena_left = 0;
    int device = 0;  // the device current at creation, which holds the state
    int cus = 0;     // its compute units
    Geom g{};
    int L = 0;  // lattices = S * R
    int gamma = 1;  // daemons (walkers) per site; a timestep is gamma sweeps
    // device state (byte layout), double-buffered: the fused sweep reads the
    // current buffers and writes the alternate ones, then the two swap
    uint8_t* spin = nullptr;  // [L][2][Nh] current
    uint8_t* dem = nullptr;   // [L][2][Nh] current
    uint8_t* spin_alt = nullptr;
    uint8_t* dem_alt = nullptr;
    // bit-plane layout (MICSA_LAYOUT_BITPLANE): 64 samples per word
    bool bit = false;
    int32_t G = 0;              // lane groups
    uint64_t* bspin = nullptr;  // [G][R][2][Nh]
    uint64_t* bdm0 = nullptr;   // [G][R][2][Nh]
    uint64_t* bdm1 = nullptr;   // [G][R][2][Nh]
    uint64_t* bJ = nullptr;     // [G][6][Nh]
    // one-launch bit-plane sweep (bitplane_sweep.hpp): it writes these, then
    // they swap with the current arrays (allocated on first use)
    uint64_t *bspin_alt = nullptr, *bdm0_alt = nullptr, *bdm1_alt = nullptr;
    uint64_t *bdr0 = nullptr, *bdr1 = nullptr;  // levels of the next refresh, drawn ahead
    // the bit-plane tally is kept by the one-launch sweep only; a per-half
    // sweep leaves it stale until the spins are written again
    bool tally_ok = true;
    // multispin working planes (msc_kernels.hpp), allocated on first use
    uint64_t* ms = nullptr;   // [L][2][rows][Lx/128] spins
    uint64_t* md0 = nullptr;  // daemon level bit 0, same shape
    uint64_t* md1 = nullptr;  // daemon level bit 1
    uint64_t* mb = nullptr;   // [L][6][rows][Lx/128] couplings of the even sites
    uint64_t *ms_alt = nullptr, *md0_alt = nullptr, *md1_alt = nullptr;  // written by the one-launch sweep
    int32_t msc_fused = 1;  // multispin: 1 = one launch per sweep (z march), 0 = one per half sweep
    // one-launch multispin sweep: levels of the next refresh drawn ahead on a
    // side stream (default priority) while the sweeps before it run
    int32_t draw_ahead = 1;
    uint64_t *mdr0 = nullptr, *mdr1 = nullptr;  // drawn levels, shape of md0 / md1
    hipStream_t draw_stream = nullptr;
    hipEvent_t draw_free = nullptr, draw_done = nullptr;
    // sweep kernel selection (MICSA_OPT_*)
    int32_t kernel_opt = MICSA_KERNEL_AUTO;
    int32_t tile_y = 0, tile_z = 0;
    int32_t xcd_map = 2;  // XCD-aware tile order for the fused sweeps (2: z bands on the multispin sweep)
    int32_t prefetch = 1;  // steps of loads in flight in the fused MicSA sweep (1 or 2)
    int32_t temporal = 2;  // MicSA sweeps per pass of the fused kernel (1 or 2)
    int32_t msc_pass = 2;  // MicSA sweeps per pass of the one-launch multispin sweep (1 or 2)
    int32_t use_graphs = 0;
    // walkers on the fused sweep: parity of a forward-X wandering the stored
    // daemons still owe (applied by the next fused sweep on load), or -1
    int32_t pend_wander = -1;
    // where the state is: in the layout's own arrays (home), in the bit planes
    // (ms, md0, md1: multispin and cell sweeps leave it there), or in both.
    // Whatever reads the home arrays unpacks the planes first, whatever
    // writes them makes the planes stale.
    bool home_ok = true, planes_ok = false;
    // cell sweeps (cells.hpp): launch plan, and the levels of cdr_n refreshes
    // from index cdr_rho0 on, drawn ahead (room for cdr_cap of them)
    CellPlan plan;
    CellPlan brief[kBriefSweeps + 1];
    CellPlan walk;
    // what the sweep call under way runs on against the rule for long calls, and
    // the us that short calls have lost where they are (see choose_arrays)
    bool off_cells = false, on_cells = false;
    double lag = 0;
    bool no_room = false;  // there was none for the planes: the paths on the layout's own arrays, until a new schedule
    MscTile tile2{};  // tile of the two-sweep multispin pass (follows the tile options)
    uint32_t *cdr0 = nullptr, *cdr1 = nullptr;
    int64_t cdr_rho0 = 0, cdr_n = 0, cdr_cap = 0;
    uint32_t* cdc = nullptr;  // the baselines' drawn comparisons, where the levels' buffer holds too few sweeps
    size_t cdc_bytes = 0;
    bool captured = false;   // a sweep call was captured into a graph (see begin_sweeps)
    bool capturing = false;  // the sweep call under way is being captured
    int depth = 0;           // begin_sweeps not yet ended
    Rest rest;
    size_t draw_room = 0;  // bytes for them (0: chosen by size)
    // several daemon (walker) families: level planes of each in two copies,
    // the copy that is current, and the parity of the wandering the planes of
    // a family owe (-1: none; the home arrays never owe one then)
    uint32_t* fl[2][6] = {};
    uint8_t fcur[6] = {};
    int32_t fowed[6] = {-1, -1, -1, -1, -1, -1};
    // refresh sweep whose levels the multispin draw planes hold, drawn during
    // an earlier call (-1: none)
    int64_t msc_drawn = -1;
    // replayable graphs of kGraphSweeps sweeps for the per-half paths, per algo
    int64_t* d_k = nullptr;  // device copy of the sweep counter
    hipStream_t cap_stream = nullptr;
    hipGraphExec_t gexec[kAlgos] = {};
    const void* gkey[kAlgos] = {};  // state buffer the graph was captured with
    unsigned long long* tally = nullptr;  // [L][kSlots]
    unsigned long long* red = nullptr;    // [max(L, S)][kSlots] reduction scratch
    // pinned host memory that kernels write the results of small reads to
    // (allocated by the first read), and the last ticket given (fetch)
    uint8_t* pin = nullptr;
    bool pin_failed = false;
    uint32_t ticket = 0;
    // device-pointer logging: one row of slots [2][L][kSlots] (energy, then
    // level sums), and the cell sweep's (U, sum m) pairs, grown on demand
    unsigned long long* logslots = nullptr;
    long long* rlog = nullptr;
    size_t rlog_cap = 0;  // entries of rlog
    // workspace of one call on the context's stream (host logs, C4, large
    // states), kept up to 16 MiB: a free waits for the device, 50 us and more
    void* work = nullptr;
    size_t work_cap = 0;
    uint32_t* lograw = nullptr;  // lanes' words of a logged launch of cell sweeps, and its room in rows
    int64_t lograw_rows = 0;
    Schedule sched;
    // device tables of the installed schedule, one entry per refresh index
    DaemonThresholds* d_dth = nullptr;
    HeatBathThresholds* d_hth = nullptr;
    MetropolisThresholds* d_mth = nullptr;
    std::vector<uint8_t> h_tables;  // what they were copied from (the copy may be under way)
    int64_t k = 0;
    std::string err;
    // timing
    bool timing = false;
    std::vector<std::pair<hipEvent_t, hipEvent_t>> events[kTimingKinds];
    double time_ms[kTimingKinds] = {};
    int64_t launches[kTimingKinds] = {};
};

namespace {

int fail(micsa_ctx* c, int status, const std::string& msg)
{
    if (c) c->err = msg;
    return status;
}

int need_home(micsa_ctx* c);
int own_home(micsa_ctx* c);
int rest_state(micsa_ctx* c);

#define HIP_TRY(ctx, call)                                                                       \
    do {                                                                                         \
        hipError_t e_ = (call);                                                                  \
        if (e_ != hipSuccess)                                                                    \
            return fail((ctx), MICSA_EHIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
    } while (0)

// ---------------------------------------------------------- device memory
void* dev_alloc(size_t bytes)
{
    // also while the thread's stream is being captured: an allocation is no
    // part of the graph
    hipStreamCaptureMode mode = hipStreamCaptureModeRelaxed;
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    void* p = nullptr;
    const hipError_t e = hipMalloc(&p, bytes);
    (void)hipThreadExchangeStreamCaptureMode(&mode);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return nullptr;
    }
    return p;
}

constexpr size_t arena_size(size_t bytes) { return (bytes + 255) / 256 * 256; }

// A block of the context's own, of at most `most` bytes (0: of its size).  From a
// store: the smallest idle one that fits, else a new one (of four sizes per factor
// of two, so that it fits other jobs too), for which idle ones make room.
void* own_block(micsa_ctx* c, size_t bytes, size_t most = 0)
{
    JobStore::Block b{c->device, arena_size(std::max<size_t>(bytes, 1)), nullptr, false};
    if (JobStore* s = c->store) {
        const size_t need = b.bytes;
        most = std::min(std::max(most, need), need + need / 4);
        size_t step = 256;
        while (7 * step < need) step *= 2;
        b.bytes = std::min((need + step - 1) / step * step, most);
        std::lock_guard<std::mutex> hold(s->lock);
        size_t at = s->idle.size();
        for (size_t i = 0; i < s->idle.size(); ++i) {
            const JobStore::Block& q = s->idle[i];
            if (q.device == b.device && q.bytes >= need && q.bytes <= most &&
                (at == s->idle.size() || q.bytes < s->idle[at].bytes))
                at = i;
        }
        if (at < s->idle.size()) {
            b = s->idle[at];
            s->held -= b.bytes;
            s->idle.erase(s->idle.begin() + (long)at);
        } else {
            s->trim(s->limit);
            b.p = dev_alloc(b.bytes);
            if (!b.p && s->held) {
                s->trim(0);
                b.p = dev_alloc(b.bytes);
            }
        }
    } else {
        b.p = dev_alloc(b.bytes);
    }
    if (b.p) c->owned.push_back(b);
    return b.p;
}

void* ctx_alloc(micsa_ctx* c, size_t bytes)
{
    const size_t n = arena_size(bytes);
    if (n <= c->arena_left) {
        uint8_t* p = c->arena;
        c->arena += n;
        c->arena_left -= n;
        return p;
    }
    return own_block(c, bytes);
}

template <class T>
bool ctx_alloc(micsa_ctx* c, T*& p, size_t bytes)
{
    return (p = static_cast<T*>(ctx_alloc(c, bytes))) != nullptr;
}

void drop_block(micsa_ctx* c, JobStore::Block b)
{
    b.kept = false;
    if (JobStore* s = c->store) {
        std::lock_guard<std::mutex> hold(s->lock);
        s->idle.push_back(b);
        s->held += b.bytes;
        s->trim(s->limit);
    } else {
        (void)hipFree(b.p);
    }
}

// Free a block before its context (work on it may be queued; a part of the
// arena, and a block that a captured graph may hold, stay until the context
// goes).
void ctx_free(micsa_ctx* c, void* p)
{
    for (size_t i = 0; p && i < c->owned.size(); ++i)
        if (c->owned[i].p == p) {
            if (c->owned[i].kept || c->capturing) return;
            if (c->store) {  // the next owner does not wait for this one's streams
                (void)hipStreamSynchronize(c->stream);
                if (c->draw_stream) (void)hipStreamSynchronize(c->draw_stream);
            }
            drop_block(c, c->owned[i]);
            c->owned.erase(c->owned.begin() + (long)i);
            return;
        }
}

// The same for a buffer of the sweeps that a larger one replaces: what is
// queued on it ends first (nothing is waited for in a captured call, whose
// blocks all stay).
void ctx_retire(micsa_ctx* c, void* p)
{
    if (!p || c->capturing) return;
    (void)hipStreamSynchronize(c->stream);
    ctx_free(c, p);
}

// The workspace, or a block of its own where that would be too large to keep;
// given back before the call ends, its work finished.
void* work_take(micsa_ctx* c, size_t bytes)
{
    if (bytes > (size_t)16 << 20) return ctx_alloc(c, bytes);
    if (c->work_cap < bytes) {
        ctx_retire(c, c->work);
        const size_t n = std::max<size_t>(bytes, (size_t)64 << 10);
        c->work = ctx_alloc(c, n);
        c->work_cap = c->work ? n : 0;
    }
    return c->work;
}

void work_give(micsa_ctx* c, void* p)
{
    if (p == c->work && !c->store) return;
    if (p == c->work) {  // (a pool's job keeps what it is charged for)
        c->work = nullptr;
        c->work_cap = 0;
    }
    ctx_free(c, p);
}

// A stream of default priority, and its end (its work has finished).
hipError_t take_stream(JobStore* s, int device, hipStream_t* out)
{
    if (s) {
        std::lock_guard<std::mutex> hold(s->lock);
        for (size_t i = 0; i < s->streams.size(); ++i)
            if (s->streams[i].first == device) {
                *out = s->streams[i].second;
                s->streams.erase(s->streams.begin() + (long)i);
                return hipSuccess;
            }
    }
    return hipStreamCreateWithFlags(out, hipStreamNonBlocking);
}

void drop_stream(JobStore* s, int device, hipStream_t q)
{
    if (s) {
        std::lock_guard<std::mutex> hold(s->lock);
        if (s->streams.size() < JobStore::kStreams) {
            s->streams.emplace_back(device, q);
            return;
        }
    }
    (void)hipStreamDestroy(q);
}

// ----------------------------------------------------------- schedule maths
// Refresh points and temperatures (Sec. 2.7-2.8).  Host double arithmetic,
// compiled without FMA contraction so the thresholds are reproducible.
bool is_refresh(int64_t k, int32_t P) { return P >= 1 ? (k % P == 0) : (((k + 1) & k) == 0); }

int64_t refresh_index(int64_t k, int32_t P)
{
    if (P >= 1) return k / P;
    int64_t rho = -1;
    for (int64_t t = k + 1; t > 0; t >>= 1) ++rho;
    return rho;
}

// Refreshes over the timesteps of the schedule (Sec. 2.8: with gamma
// daemons per site a timestep is gamma sweeps; refresh points count timesteps).
int64_t refresh_count(const Schedule& s)
{
    return s.n_steps <= 0 ? 0 : refresh_index(s.n_steps - 1, s.period) + 1;
}

double temperature(const Schedule& s, int64_t rho)
{
    switch (s.kind) {
    case MICSA_SCHED_CONST: return s.T0;
    case MICSA_SCHED_LINEAR: {
        const int64_t n = refresh_count(s);
        if (n <= 1) return s.T0;
        const double f = (double)rho / (double)(n - 1);
        return s.T0 * (1.0 - f) + s.T1 * f;
    }
    default: return (rho >= 0 && rho < (int64_t)s.table.size()) ? s.table[(size_t)rho] : NAN;
    }
}

// t_k = floor(2^32 * P(m <= k)), P(m <= k) = (1 - e^{-4 beta (k+1)}) / (1 - e^{-16 beta}).
DaemonThresholds daemon_thresholds(double T)
{
    const double beta = 1.0 / T;
    uint64_t t[3];
    for (int k = 0; k < 3; ++k)
        t[k] = (uint64_t)std::floor(std::expm1(-4.0 * beta * (double)(k + 1)) / std::expm1(-16.0 * beta) *
                                    4294967296.0);
    return {t[0], t[1], t[2]};
}

// tau_v = floor(2^32 / (1 + e^{-2 beta h})), h = 6 - 2v.
HeatBathThresholds heatbath_thresholds(double T)
{
    const double beta = 1.0 / T;
    HeatBathThresholds th;
    for (int v = 0; v < 7; ++v)
        th.tau[v] = (uint64_t)std::floor(4294967296.0 / (1.0 + std::exp(-2.0 * beta * (double)(6 - 2 * v))));
    return th;
}

// theta_q = floor(2^32 e^{-beta dH}) for dH = 4q - 12 > 0, 2^32 for dH <= 0.
MetropolisThresholds metropolis_thresholds(double T)
{
    const double beta = 1.0 / T;
    MetropolisThresholds th;
    for (int q = 0; q < 7; ++q) {
        const int dH = 4 * q - 12;
        th.tau[q] = dH <= 0 ? 4294967296ull : (uint64_t)std::floor(std::exp(-beta * (double)dH) * 4294967296.0);
    }
    return th;
}

// The per-refresh table of a canonical baseline, and its timing kind.
const HeatBathThresholds* canonical_table(const micsa_ctx* c, int32_t algo)
{
    return algo == MICSA_ALGO_METROPOLIS ? c->d_mth : c->d_hth;
}

int canonical_timing(int32_t algo) { return algo == MICSA_ALGO_METROPOLIS ? kTimeMetropolis : kTimeHeatBath; }

// --------------------------------------------------------------- launching
dim3 grid_for(int64_t threads, int y)
{
    return dim3((unsigned)((threads + kBlock - 1) / kBlock), (unsigned)y, 1);
}

struct TimedLaunch {
    micsa_ctx* c;
    int kind;
    hipEvent_t a = nullptr, b = nullptr;
    TimedLaunch(micsa_ctx* ctx, int kd) : c(ctx), kind(kd)
    {
        if (c->timing) {
            if (hipEventCreate(&a) != hipSuccess || hipEventCreate(&b) != hipSuccess) {
                a = b = nullptr;
                return;
            }
            (void)hipEventRecord(a, c->stream);
        }
    }
    ~TimedLaunch()
    {
        if (a && b) {
            (void)hipEventRecord(b, c->stream);
            c->events[kind].push_back({a, b});
        }
    }
};

int check_launch(micsa_ctx* c, const char* what)
{
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fail(c, MICSA_EHIP, std::string(what) + ": " + hipGetErrorString(e));
    return MICSA_OK;
}

// Zero the accumulator slots of n entities.
int zero_slots(micsa_ctx* c, unsigned long long* p, int64_t n)
{
    k_fill_i64<<<grid_for(n * kSlots, 1), kBlock, 0, c->stream>>>(p, n * kSlots, 0ull);
    return check_launch(c, "k_fill_i64");
}

// A small read: its last kernel writes the result to pinned host memory, and a
// single work-group also the ticket that the host waits for (at most 1 ms, then
// it waits for the stream, which also reports errors).  A copy to pageable
// memory and a stream synchronisation took 23 us for 512 bytes, a kernel that
// writes pinned memory and a synchronisation 11.7, the ticket 6.4; at 256 KiB
// 33 and 22, above that the copy is faster.
constexpr size_t kTicketBytes = (size_t)16 << 10;

bool have_pin(micsa_ctx* c)
{
    if (c->pin) return true;
    if (c->pin_failed) return false;
    c->pin = take_pin(c->device);
    if (!c->pin) {
        c->pin_failed = true;
        return false;
    }
    *reinterpret_cast<volatile uint32_t*>(c->pin) = c->ticket = 0;
    return true;
}

// run(dst, ticket, value) launches it, as one work-group that ends with
// give_ticket(ticket, value) where `one`.
template <class Run>
int fetch(micsa_ctx* c, size_t bytes, void* host, bool one, Run run)
{
    uint8_t* const dst = c->pin + kPinHead;
    volatile uint32_t* const flag = reinterpret_cast<volatile uint32_t*>(c->pin);
    const uint32_t value = ++c->ticket;
    run(dst, one ? reinterpret_cast<uint32_t*>(c->pin) : nullptr, value);
    if (int st = check_launch(c, "read")) return st;
    bool done = false;
    if (one) {
        const auto limit = std::chrono::steady_clock::now() + std::chrono::milliseconds(1);
        for (int i = 0; !done; ++i) {
            done = *flag == value;
            if ((i & 255) == 255 && std::chrono::steady_clock::now() > limit) break;
        }
        std::atomic_thread_fence(std::memory_order_acquire);
    }
    if (!done) HIP_TRY(c, hipStreamSynchronize(c->stream));
    std::memcpy(host, dst, bytes);
    return MICSA_OK;
}

// Device memory (a multiple of 8 bytes, as is its address) to the host.
int read_device(micsa_ctx* c, const void* dev, void* host, size_t bytes)
{
    if (bytes <= kPinBytes && have_pin(c)) {
        const bool one = bytes <= kTicketBytes;
        return fetch(c, bytes, host, one, [&](void* dst, uint32_t* ticket, uint32_t value) {
            k_to_host<<<one ? 1u : (unsigned)((bytes + 8191) / 8192), 1024, 0, c->stream>>>(
                static_cast<const uint64_t*>(dev), (int64_t)(bytes / 8), static_cast<uint64_t*>(dst), ticket, value);
        });
    }
    HIP_TRY(c, hipMemcpyAsync(host, dev, bytes, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return MICSA_OK;
}

// The slots of n entities, summed per entity.
int read_slots(micsa_ctx* c, const unsigned long long* dev, int64_t n, std::vector<int64_t>& out)
{
    out.assign((size_t)n, 0);
    if ((size_t)n * 8 <= kPinBytes && have_pin(c))
        // (a wave per entity: up to eight rounds of one work-group)
        return fetch(c, (size_t)n * 8, out.data(), n <= 128, [&](void* dst, uint32_t* ticket, uint32_t value) {
            k_sum_slots<<<ticket ? 1u : (unsigned)((n + 15) / 16), 1024, 0, c->stream>>>(
                dev, n, static_cast<long long*>(dst), ticket, value);
        });
    std::vector<int64_t> raw((size_t)(n * kSlots));
    HIP_TRY(c, hipMemcpyAsync(raw.data(), dev, raw.size() * 8, hipMemcpyDeviceToHost, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    for (int64_t e = 0; e < n; ++e)
        for (int k = 0; k < kSlots; ++k) out[(size_t)e] += raw[(size_t)(e * kSlots + k)];
    return MICSA_OK;
}

// tally <- E (slot 0 = E, other slots 0).
int set_tally(micsa_ctx* c, const std::vector<int64_t>& E)
{
    std::vector<int64_t> raw((size_t)c->L * kSlots, 0);
    for (int l = 0; l < c->L; ++l) raw[(size_t)l * kSlots] = E[(size_t)l];
    HIP_TRY(c, hipMemcpyAsync(c->tally, raw.data(), raw.size() * 8, hipMemcpyHostToDevice, c->stream));
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return MICSA_OK;
}

GeomB geomb(const micsa_ctx* c) { return GeomB{c->g, c->G, c->p.lane_mode}; }

int word_lattices(const micsa_ctx* c) { return bp_word_lattices(geomb(c)); }

// Launch shape of the one-launch bit-plane sweep: TZ planes per work-group
// (1, or 2 with TILE_Z = 2), one thread per word of a plane, LDS for TZ + 4
// odd and TZ + 2 even planes.
struct BpLaunch {
    BpTile f;
    unsigned block;
    size_t lds;
};

BpLaunch bp_launch(const micsa_ctx* c)
{
    BpLaunch b{};
    const int Kx = c->p.Lx / 2;
    const int P = c->p.Ly * Kx;
    if (P > 1024) {
        // kb_sweep_rows: tiles of TY rows plus two ring rows on each side, a
        // word position per thread; TY keeps the rows computed per plane
        // (nty (TY + 4)) smallest, the larger TY on ties
        const int tymax = std::min(1024 / Kx - 4, c->p.Ly);
        int best = 0;
        int64_t cost = 0;
        for (int ty = 1; ty <= tymax; ++ty) {
            const int64_t n = (c->p.Ly + ty - 1) / ty, w = n * (ty + 4);
            if (!best || w <= cost) {
                best = ty;
                cost = w;
            }
        }
        if (c->tile_y > 0) best = std::min(c->tile_y, tymax);
        const int TY = std::max(best, 1);
        b.f = BpTile{1, c->p.Lz, P, TY, (c->p.Ly + TY - 1) / TY};
        const int PT = (TY + 4) * Kx;
        b.block = (unsigned)((PT + 63) / 64 * 64);
        b.lds = std::max((size_t)8 * PT * 8, (size_t)(b.block / 64) * 64 * 8);
        return b;
    }
    const int TZ = c->tile_z == 2 && c->p.Lz % 2 == 0 && P <= 512 ? 2 : 1;
    b.f = BpTile{TZ, c->p.Lz / TZ, P, c->p.Ly, 1};
    b.block = (unsigned)((P + 63) / 64 * 64);
    const size_t planes = (size_t)(2 * TZ + 6) * P * 8, part = (size_t)(b.block / 64) * 64 * 8;
    b.lds = std::max(planes, part);
    return b;
}

bool bp_rows(const BpLaunch& b) { return b.f.nty > 1 || b.f.P > 1024; }

// The one-launch sweep fits: a word position per thread (at most 1024 per
// work-group: a whole plane, or TY + 4 >= 5 rows of one) and LDS within a
// work-group's 160 KB.
bool bp_fits(const micsa_ctx* c, const BpLaunch& b)
{
    if (bp_rows(b)) return 1024 / (c->p.Lx / 2) - 4 >= 1 && b.lds <= 160 * 1024;
    return b.f.P <= (b.f.TZ == 1 ? 1024 : 512) && b.lds <= 160 * 1024;
}

// AUTO takes the one-launch sweep where a plane fits a work-group; on larger
// planes its row tiles (kb_sweep_rows) run only on request (KERNEL_FUSED):
// there the per-half kernels are faster (8.6 against 11.9 us per sweep at
// L = 64 on one MI355X), but keep no per-lane tally.
bool bp_one_launch(const micsa_ctx* c)
{
    if (!c->bit || c->kernel_opt == MICSA_KERNEL_SIMPLE) return false;
    const BpLaunch b = bp_launch(c);
    return bp_fits(c, b) && (!bp_rows(b) || c->kernel_opt == MICSA_KERNEL_FUSED);
}

// One-launch bit-plane sweep; with drawn the levels are read from the drawn
// planes (a refresh drawn ahead).
int launch_bp_sweep(micsa_ctx* c, bool drawn)
{
    const BpLaunch b = bp_launch(c);
    if (!c->bspin_alt) {
        const size_t words = (size_t)word_lattices(c) * 2 * (size_t)c->g.Nh;
        bool ok = true;
        for (uint64_t** q : {&c->bspin_alt, &c->bdm0_alt, &c->bdm1_alt})
            ok = ok && ctx_alloc(c, *q, words * 8);
        if (!ok) {
            for (uint64_t** q : {&c->bspin_alt, &c->bdm0_alt, &c->bdm1_alt}) {
                ctx_free(c, *q);
                *q = nullptr;
            }
            return fail(c, MICSA_ENOMEM, "bit-plane sweep buffers");
        }
    }
    const auto kern = bp_rows(b) ? kb_sweep_rows<true> : b.f.TZ == 2 ? kb_sweep<true, 2> : kb_sweep<true, 1>;
    if (b.lds > 64 * 1024 &&
        hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)b.lds) != hipSuccess)
        return fail(c, MICSA_EHIP, "kb_sweep LDS attribute");
    const dim3 grid((unsigned)(b.f.ntz * b.f.nty * word_lattices(c)));
    {
        TimedLaunch t(c, kTimeSweep);
        kern<<<grid, b.block, b.lds, c->stream>>>(geomb(c), b.f, c->bspin, drawn ? c->bdr0 : c->bdm0,
                                                  drawn ? c->bdr1 : c->bdm1, c->bJ, c->bspin_alt, c->bdm0_alt,
                                                  c->bdm1_alt, c->tally);
    }
    const int st = check_launch(c, "kb_sweep");
    if (st) return st;
    std::swap(c->bspin, c->bspin_alt);
    std::swap(c->bdm0, c->bdm0_alt);
    std::swap(c->bdm1, c->bdm1_alt);
    return MICSA_OK;
}

int64_t next_refresh(const micsa_ctx* c, int64_t from, int64_t end);

// Draw the levels of bit-plane refresh sweep kr into the drawn planes on the
// side stream, after everything the library stream holds so far (the sweep
// that last read them); the refresh sweep waits for draw_done.
int draw_bp_levels(micsa_ctx* c, int64_t kr)
{
    const int64_t rho = refresh_index(kr, c->sched.period);
    const double T = temperature(c->sched, rho);
    if (!(T > 0.0) || !std::isfinite(T)) return fail(c, MICSA_ERANGE, "no temperature for this refresh");
    if (!c->bdr0) {
        const size_t words = (size_t)word_lattices(c) * 2 * (size_t)c->g.Nh;
        if (!ctx_alloc(c, c->bdr0, words * 8) || !ctx_alloc(c, c->bdr1, words * 8)) {
            ctx_free(c, c->bdr0);
            c->bdr0 = c->bdr1 = nullptr;
            return fail(c, MICSA_ENOMEM, "bit-plane drawn levels");
        }
    }
    if (!c->draw_stream) {
        HIP_TRY(c, take_stream(c->store, c->device, &c->draw_stream));
        HIP_TRY(c, hipEventCreateWithFlags(&c->draw_free, hipEventDisableTiming));
        HIP_TRY(c, hipEventCreateWithFlags(&c->draw_done, hipEventDisableTiming));
    }
    HIP_TRY(c, hipEventRecord(c->draw_free, c->stream));
    HIP_TRY(c, hipStreamWaitEvent(c->draw_stream, c->draw_free, 0));
    kb_refresh<<<dim3(bp_refresh_blocks(c->g), (unsigned)word_lattices(c)), 256, 0, c->draw_stream>>>(
        geomb(c), c->bdr0, c->bdr1, (uint32_t)rho, daemon_thresholds(T));
    const int st = check_launch(c, "kb_refresh (drawn ahead)");
    if (st) return st;
    HIP_TRY(c, hipEventRecord(c->draw_done, c->draw_stream));
    return MICSA_OK;
}

// MicSA sweeps k .. k + n - 1 of the bit-plane layout on the one-launch
// sweep; the levels of each refresh are drawn ahead on the side stream
// (OPT_DRAW_AHEAD, default) while the sweeps before it run, or in place just
// before it.
int sweep_bitplane(micsa_ctx* c, int64_t n)
{
    const int64_t k_end = c->k + n;
    int64_t drawn = -1;
    int st;
    if (c->draw_ahead && (drawn = next_refresh(c, c->k, k_end)) >= 0 && (st = draw_bp_levels(c, drawn))) return st;
    for (int64_t i = 0; i < n; ++i) {
        const int64_t k = c->k;
        const bool refresh = is_refresh(k, c->sched.period);
        const int64_t rho = refresh_index(k, c->sched.period);
        const double T = temperature(c->sched, rho);
        if (!(T > 0.0) || !std::isfinite(T)) return fail(c, MICSA_ERANGE, "no temperature for this refresh");
        const bool use_drawn = refresh && drawn == k;
        if (use_drawn) {
            HIP_TRY(c, hipStreamWaitEvent(c->stream, c->draw_done, 0));
        } else if (refresh) {
            TimedLaunch t(c, kTimeRefresh);
            kb_refresh<<<dim3(bp_refresh_blocks(c->g), (unsigned)word_lattices(c)), 256, 0, c->stream>>>(
                geomb(c), c->bdm0, c->bdm1, (uint32_t)rho, daemon_thresholds(T));
            if ((st = check_launch(c, "kb_refresh"))) return st;
        }
        if ((st = launch_bp_sweep(c, use_drawn))) return st;
        if (use_drawn && (drawn = next_refresh(c, k + 1, k_end)) >= 0 && (st = draw_bp_levels(c, drawn))) return st;
        c->k = k + 1;
    }
    return MICSA_OK;
}

int launch_bitplane_sweep(micsa_ctx* c, bool refresh, int64_t rho, double T)
{
    const int WL = word_lattices(c);
    if (refresh) {
        TimedLaunch t(c, kTimeRefresh);
        kb_refresh<<<dim3(bp_refresh_blocks(c->g), (unsigned)WL), 256, 0, c->stream>>>(
            geomb(c), c->bdm0, c->bdm1, (uint32_t)rho, daemon_thresholds(T));
    }
    int st = check_launch(c, "kb_refresh");
    if (st) return st;
    c->tally_ok = false;
    const dim3 grid = grid_for(c->g.Nh, WL);
    {
        TimedLaunch t(c, kTimeSweep);
        kb_micsa_half<0><<<grid, kBlock, 0, c->stream>>>(geomb(c), c->bspin, c->bdm0, c->bdm1, c->bJ);
    }
    if ((st = check_launch(c, "kb_micsa_half<0>"))) return st;
    {
        TimedLaunch t(c, kTimeSweep);
        kb_micsa_half<1><<<grid, kBlock, 0, c->stream>>>(geomb(c), c->bspin, c->bdm0, c->bdm1, c->bJ);
    }
    return check_launch(c, "kb_micsa_half<1>");
}

// Per-lane counts of the bit-plane layout into dst slots (see kb_lane_count).
template <int KIND>
int enqueue_lane_count(micsa_ctx* c, unsigned long long* dst, int ra, int rb)
{
    const int64_t ent = KIND == 2 ? c->p.n_samples : c->L;
    int st = zero_slots(c, dst, ent);
    if (st) return st;
    const int64_t per_block = 128;
    const unsigned ny = (unsigned)(KIND == 2 ? (c->p.lane_mode ? c->p.n_samples : c->G) : word_lattices(c));
    {
        TimedLaunch t(c, kTimeReduce);
        kb_lane_count<KIND><<<dim3((unsigned)((c->g.Nh + per_block - 1) / per_block), ny), 64, 0, c->stream>>>(
            geomb(c), c->bspin, c->bdm0, c->bdm1, c->bJ, ra, rb, per_block, dst);
    }
    return check_launch(c, "kb_lane_count");
}

int launch_refresh(micsa_ctx* c, int64_t rho, double T)
{
    TimedLaunch t(c, kTimeRefresh);
    k_refresh<<<grid_for(c->g.Nh / 4, c->L * c->gamma), kBlock, 0, c->stream>>>(c->g, c->dem, (uint32_t)rho,
                                                                                 daemon_thresholds(T));
    return check_launch(c, "k_refresh");
}

// The resident variant (a small lattice in one or a few work-groups for many
// sweeps per launch: the cell sweep) is asked for, and taken by default before
// every other path, up to this size.
constexpr size_t kResidentLdsMax = 150 * 1024;
constexpr int64_t kResidentChunk = 2048;  // sweeps per launch of a whole lattice

bool resident_eligible(const micsa_ctx* c)
{
    return !c->bit && c->gamma == 1 && (size_t)c->g.Nh * 3 <= kResidentLdsMax;
}

bool use_resident(const micsa_ctx* c)
{
    if (c->kernel_opt == MICSA_KERNEL_RESIDENT) return true;
    return c->kernel_opt == MICSA_KERNEL_AUTO && resident_eligible(c);
}

bool fused_eligible(const micsa_ctx* c)
{
    return !c->bit && c->gamma == 1 && c->p.Lx % 32 == 0 && 5 * (c->p.Lx / 32) <= 1024;
}

// (the one-launch sweep addresses a plane with 32-bit byte offsets: fewer than 2^29 words)
bool msc_eligible(const micsa_ctx* c)
{
    return !c->bit && c->gamma == 1 && c->p.Lx % 128 == 0 && (int64_t)c->g.rows * (c->p.Lx / 128) < (int64_t(1) << 29);
}

// AUTO takes the multispin planes for MicSA calls of at least kMscMinSweeps
// sweeps on lattices the resident kernel does not hold (a call packs and
// unpacks the state once, about the traffic of two sweeps).
constexpr int64_t kMscMinSweeps = 8;

bool msc_one_launch(const micsa_ctx* c);

bool use_msc(const micsa_ctx* c, int64_t n = kMscMinSweeps, int32_t algo = MICSA_ALGO_MICSA)
{
    if (!msc_eligible(c)) return false;
    if (algo == MICSA_ALGO_WALKERS && !msc_one_launch(c)) return false;  // walkers need the one-launch sweep
    if (c->kernel_opt == MICSA_KERNEL_MULTISPIN) return true;
    return c->kernel_opt == MICSA_KERNEL_AUTO && !use_resident(c) && n >= kMscMinSweeps;
}

// The slab form (a lattice too large for one work-group and too narrow for
// the fused sweep; the cell sweep runs it) may be asked for where a plane has at
// most this many 4-site words.
constexpr int kSlabLanes = 1024;
bool slab_eligible(const micsa_ctx* c)
{
    return !c->bit && c->gamma == 1 && (int64_t)c->p.Ly * (c->p.Lx / 8) <= kSlabLanes;
}

bool use_fused(const micsa_ctx* c);

// AUTO takes it for lattices the resident kernel does not hold that are too
// narrow for the fused sweep (Lx < 128).
bool use_slab(const micsa_ctx* c)
{
    if (!slab_eligible(c)) return false;
    if (c->kernel_opt == MICSA_KERNEL_SLAB) return true;
    return c->kernel_opt == MICSA_KERNEL_AUTO && !use_resident(c) && !use_fused(c);
}

// The slab variant's name (micsa_kernel_name): "2" while the lattices have
// fewer planes than the device has compute units.  Both run the cell sweep.
bool slab_pairs(const micsa_ctx* c)
{
    return c->temporal == 2 && (int64_t)c->L * c->p.Lz < (c->cus > 0 ? c->cus : 256);
}

bool use_fused(const micsa_ctx* c)
{
    if (c->bit || c->kernel_opt == MICSA_KERNEL_SIMPLE || c->kernel_opt == MICSA_KERNEL_RESIDENT ||
        c->kernel_opt == MICSA_KERNEL_SLAB)
        return false;
    if (c->kernel_opt == MICSA_KERNEL_FUSED) return true;
    return fused_eligible(c) && c->p.Lx >= 128;
}

// Largest divisor of n not above cap (n >= 1, cap >= 1).
int divisor_at_most(int n, int cap)
{
    for (int d = std::min(n, cap); d > 1; --d)
        if (n % d == 0) return d;
    return 1;
}

// Tile of the fused sweep: TY rows (so that (TY+4) * NC lanes fit a
// work-group of at most 1024), TZ planes chosen to give the device at least
// two work-groups per compute unit when the lattice allows it.
FusedTile choose_tile(const micsa_ctx* c)
{
    FusedTile f;
    f.NC = c->p.Lx / 32;
    const int ty_cap = std::max(1, std::min(32, 1024 / f.NC - 4));
    f.TY = c->tile_y > 0 && c->p.Ly % c->tile_y == 0 ? c->tile_y : divisor_at_most(c->p.Ly, ty_cap);
    f.nty = c->p.Ly / f.TY;
    f.xcd = c->xcd_map;
    if (c->tile_z > 0) {
        f.TZ = c->tile_z;
    } else {
        f.TZ = divisor_at_most(c->p.Lz, 32);
        while (f.TZ > 4 && (int64_t)f.nty * (c->p.Lz / f.TZ) * c->L < 512) {
            const int next = divisor_at_most(c->p.Lz, f.TZ - 1);
            if (next < 4) break;
            f.TZ = next;
        }
    }
    f.ntz = c->p.Lz / f.TZ;
    if ((f.nty * f.ntz) % 8 != 0) f.xcd = 0;
    return f;
}

CellGeom cell_geom(const micsa_ctx* c);
uint32_t* w32(uint64_t* p);

// The alternate byte arrays (allocated with the context where a path that
// needs them is the default, else by the first call that takes one).
int need_alt(micsa_ctx* c)
{
    const size_t state = (size_t)c->L * 2 * (size_t)c->g.Nh;
    if (!c->spin_alt) ctx_alloc(c, c->spin_alt, state);
    if (!c->dem_alt) ctx_alloc(c, c->dem_alt, state * (size_t)c->gamma);
    return c->spin_alt && c->dem_alt ? MICSA_OK : fail(c, MICSA_ENOMEM, "alternate state buffers");
}

int launch_fused_sweep(micsa_ctx* c, bool refresh, int64_t rho, double T, int wander = -1)
{
    if (int st = need_alt(c)) return st;
    const FusedTile f = choose_tile(c);
    const int lanes = (f.TY + 4) * f.NC;
    const int block = (lanes + 63) / 64 * 64;
    const size_t lds = (size_t)64 * (f.TY + 4) * f.NC;
    const dim3 grid((unsigned)(f.nty * (c->p.Lz / f.TZ)), (unsigned)c->L, 1);
    const DaemonThresholds th = refresh ? daemon_thresholds(T) : DaemonThresholds{0, 0, 0};
    {
        TimedLaunch t(c, kTimeSweep);
        const bool pf2 = c->prefetch == 2 && block <= kPf2Lanes;  // larger tiles run the one-step variant
        const auto kern = refresh ? (pf2 ? k_micsa_sweep_fused<true, 2> : k_micsa_sweep_fused<true, 1>)
                                  : (pf2 ? k_micsa_sweep_fused<false, 2> : k_micsa_sweep_fused<false, 1>);
        kern<<<grid, block, lds, c->stream>>>(c->g, f, c->spin, c->dem, c->spin_alt, c->dem_alt, c->tally,
                                              (uint32_t)rho, th, refresh ? -1 : wander);
    }
    const int st = check_launch(c, "k_micsa_sweep_fused");
    if (st) return st;
    std::swap(c->spin, c->spin_alt);
    std::swap(c->dem, c->dem_alt);
    return MICSA_OK;
}

// Tile of the two-sweep kernel: TY + 8 ring rows of NC lanes within
// kSweep2Lanes; the tile options apply where they fit.
FusedTile choose_tile2(const micsa_ctx* c)
{
    FusedTile f = choose_tile(c);
    const int ty_cap = kSweep2Lanes / f.NC - 8;
    if (f.TY > ty_cap) {
        f.TY = divisor_at_most(c->p.Ly, ty_cap);
        f.nty = c->p.Ly / f.TY;
        f.xcd = c->xcd_map && (f.nty * f.ntz) % 8 == 0;
    }
    return f;
}

bool sweep2_eligible(const micsa_ctx* c) { return kSweep2Lanes / (c->p.Lx / 32) - 8 >= 1; }

// Sweeps k and k + 1 in one pass (fused2_kernels.hpp); refreshA / refreshB
// say whether k / k + 1 are refresh points.  Walkers (walk): wanderA is a
// wandering owed from before (-1: none), wanderAB the parity of the
// wandering between the two sweeps.
int launch_fused_sweep2(micsa_ctx* c, bool refreshA, int64_t rhoA, double TA, bool refreshB, int64_t rhoB, double TB,
                        bool walk = false, int wanderA = -1, int wanderAB = -1)
{
    if (int st = need_alt(c)) return st;
    const FusedTile f = choose_tile2(c);
    const int lanes = (f.TY + 8) * f.NC;
    const int block = (lanes + 63) / 64 * 64;
    const size_t lds = (size_t)128 * (f.TY + 8) * f.NC;  // 4 planes x 2 buffers x 16 B per lane slot
    using Kern = void (*)(Geom, FusedTile, const uint8_t*, const uint8_t*, uint8_t*, uint8_t*, unsigned long long*,
                          uint32_t, DaemonThresholds, uint32_t, DaemonThresholds, int, int);
    static const Kern kernels[8] = {
        k_micsa_sweep2_fused<false, false, false>, k_micsa_sweep2_fused<true, false, false>,
        k_micsa_sweep2_fused<false, true, false>,  k_micsa_sweep2_fused<true, true, false>,
        k_micsa_sweep2_fused<false, false, true>,  k_micsa_sweep2_fused<true, false, true>,
        k_micsa_sweep2_fused<false, true, true>,   k_micsa_sweep2_fused<true, true, true>};
    static bool attr_set[8] = {};
    const int which = (refreshA ? 1 : 0) + (refreshB ? 2 : 0) + (walk ? 4 : 0);
    if (!attr_set[which]) {
        const hipError_t e = hipFuncSetAttribute((const void*)kernels[which],
                                                 hipFuncAttributeMaxDynamicSharedMemorySize, (int)kResidentLdsMax);
        if (e != hipSuccess) return fail(c, MICSA_EHIP, std::string("hipFuncSetAttribute: ") + hipGetErrorString(e));
        attr_set[which] = true;
    }
    const dim3 grid((unsigned)(f.nty * f.ntz), (unsigned)c->L, 1);
    const DaemonThresholds thA = refreshA ? daemon_thresholds(TA) : DaemonThresholds{0, 0, 0};
    const DaemonThresholds thB = refreshB ? daemon_thresholds(TB) : DaemonThresholds{0, 0, 0};
    {
        TimedLaunch t(c, kTimeSweep);
        kernels[which]<<<grid, block, lds, c->stream>>>(c->g, f, c->spin, c->dem, c->spin_alt, c->dem_alt, c->tally,
                                                        (uint32_t)rhoA, thA, (uint32_t)rhoB, thB,
                                                        refreshA ? -1 : wanderA, wanderAB);
    }
    const int st = check_launch(c, "k_micsa_sweep2_fused");
    if (st) return st;
    std::swap(c->spin, c->spin_alt);
    std::swap(c->dem, c->dem_alt);
    return MICSA_OK;
}

// Walkers in the two-sweep kernel need a row's chunks in one wave.
bool sweep2_walk_eligible(const micsa_ctx* c)
{
    const int nc = c->p.Lx / 32;
    return c->gamma == 1 && sweep2_eligible(c) && 64 % nc == 0;
}

int launch_micsa_sweep(micsa_ctx* c, int fam)
{
    const int64_t words = (int64_t)c->g.rows * c->g.Wr;
    {
        TimedLaunch t(c, kTimeSweep);
        k_micsa_half<0><<<grid_for(words, c->L), kBlock, 0, c->stream>>>(c->g, c->spin, c->dem, c->tally,
                                                                          fam);
    }
    int st = check_launch(c, "k_micsa_half<0>");
    if (st) return st;
    {
        TimedLaunch t(c, kTimeSweep);
        k_micsa_half<1><<<grid_for(words, c->L), kBlock, 0, c->stream>>>(c->g, c->spin, c->dem, c->tally,
                                                                          fam);
    }
    return check_launch(c, "k_micsa_half<1>");
}

int launch_fused_canonical(micsa_ctx* c, int32_t algo, int64_t k, double T)
{
    if (int st = need_alt(c)) return st;
    const FusedTile f = choose_tile(c);
    const int lanes = (f.TY + 4) * f.NC;
    const int block = (lanes + 63) / 64 * 64;
    const size_t lds = (size_t)64 * (f.TY + 4) * f.NC;
    const dim3 grid((unsigned)(f.nty * (c->p.Lz / f.TZ)), (unsigned)c->L, 1);
    {
        TimedLaunch t(c, canonical_timing(algo));
        if (algo == MICSA_ALGO_METROPOLIS)
            k_heatbath_sweep_fused<1><<<grid, block, lds, c->stream>>>(c->g, f, c->spin, c->spin_alt, c->tally,
                                                                       (uint32_t)(2 * k), metropolis_thresholds(T));
        else
            k_heatbath_sweep_fused<0><<<grid, block, lds, c->stream>>>(c->g, f, c->spin, c->spin_alt, c->tally,
                                                                       (uint32_t)(2 * k), heatbath_thresholds(T));
    }
    const int st = check_launch(c, "k_heatbath_sweep_fused");
    if (st) return st;
    std::swap(c->spin, c->spin_alt);
    return MICSA_OK;
}

// One half sweep of a canonical baseline; with dk the sweep index and the
// table come from device memory (graph form), otherwise from k and th.
template <int P>
void enqueue_canonical_half(micsa_ctx* c, int32_t algo, hipStream_t st, int64_t k, const HeatBathThresholds& th,
                            const int64_t* dk)
{
    const int64_t words = (int64_t)c->g.rows * c->g.Wr;
    const dim3 grid = grid_for(words, c->L);
    const uint32_t time = (uint32_t)(2 * k + P);
    const int32_t period = c->sched.period;
    if (algo == MICSA_ALGO_METROPOLIS)
        k_heatbath_half<P, 1><<<grid, kBlock, 0, st>>>(c->g, c->spin, time, th, c->tally, dk, period, c->d_mth);
    else
        k_heatbath_half<P, 0><<<grid, kBlock, 0, st>>>(c->g, c->spin, time, th, c->tally, dk, period, c->d_hth);
}

int launch_canonical_sweep(micsa_ctx* c, int32_t algo, int64_t k, double T)
{
    if (use_fused(c)) return launch_fused_canonical(c, algo, k, T);
    const HeatBathThresholds th = algo == MICSA_ALGO_METROPOLIS ? metropolis_thresholds(T) : heatbath_thresholds(T);
    {
        TimedLaunch t(c, canonical_timing(algo));
        enqueue_canonical_half<0>(c, algo, c->stream, k, th, nullptr);
    }
    int st = check_launch(c, "k_heatbath_half<0>");
    if (st) return st;
    {
        TimedLaunch t(c, canonical_timing(algo));
        enqueue_canonical_half<1>(c, algo, c->stream, k, th, nullptr);
    }
    return check_launch(c, "k_heatbath_half<1>");
}

// Bond bits of every lattice into its even spin bytes (spins kept).
int enqueue_bonds(micsa_ctx* c)
{
    k_init_couplings<<<grid_for(c->g.Nh / 4, c->L), kBlock, 0, c->stream>>>(c->g, c->spin);
    return check_launch(c, "k_init_couplings");
}

// Count over the planes (k_cells_count) into the slots of n entities.
CellLevels cell_levels(const micsa_ctx* c);
template <int KIND>
int enqueue_cells_count(micsa_ctx* c, int n, int a, int b, unsigned long long* dst)
{
    const CellGeom cg = cell_geom(c);
    // a few words per thread, enough work-groups to fill the device
    const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((cg.plane + 255) / 256, 4096 / std::max(1, n) + 1));
    if (blocks > kSlots)  // fewer store their slots themselves
        if (int st = zero_slots(c, dst, n)) return st;
    {
        TimedLaunch t(c, kTimeReduce);
        k_cells_count<KIND><<<dim3((unsigned)blocks, (unsigned)n), 256, 0, c->stream>>>(
            cg, reinterpret_cast<const uint32_t*>(c->ms), cell_levels(c), reinterpret_cast<const uint32_t*>(c->mb), a,
            b, dst);
    }
    return check_launch(c, "k_cells_count");
}

// Enqueue: dst[l] = unsatisfied bonds of lattice l, from scratch.
int enqueue_energy(micsa_ctx* c, unsigned long long* dst)
{
    if (c->bit && !c->planes_ok) return enqueue_lane_count<0>(c, dst, 0, 0);
    if (c->planes_ok) return enqueue_cells_count<0>(c, c->L, 0, 0, dst);
    int st = zero_slots(c, dst, c->L);
    if (st) return st;
    TimedLaunch t(c, kTimeReduce);
    k_unsat_bonds<<<grid_for((int64_t)c->g.rows * c->g.Wr, c->L), kBlock, 0, c->stream>>>(c->g, c->spin,
                                                                                           dst);
    return check_launch(c, "k_unsat_bonds");
}

int enqueue_level_sum(micsa_ctx* c, unsigned long long* dst)
{
    if (c->bit && !c->planes_ok) return enqueue_lane_count<1>(c, dst, 0, 0);
    if (c->planes_ok) return enqueue_cells_count<1>(c, c->L, 0, 0, dst);
    int st = zero_slots(c, dst, c->L);
    if (st) return st;
    TimedLaunch t(c, kTimeReduce);
    const int64_t wpl = (int64_t)c->gamma * 2 * c->g.Nh / 4;  // every family of the lattice
    k_level_sum<<<grid_for(wpl, c->L), kBlock, 0, c->stream>>>(wpl, reinterpret_cast<const uint32_t*>(c->dem),
                                                               dst);
    return check_launch(c, "k_level_sum");
}

int64_t n_sites(const micsa_ctx* c) { return (int64_t)c->p.Lx * c->p.Ly * c->p.Lz; }

// Natural index i -> (parity, h) of the byte layout.
inline void split_index(const micsa_ctx* c, int64_t i, int& par, int64_t& h)
{
    const int x = (int)(i % c->p.Lx);
    const int64_t row = i / c->p.Lx;
    const int y = (int)(row % c->p.Ly), z = (int)(row / c->p.Ly);
    par = (x + y + z) & 1;
    h = i >> 1;
}

// ------------------------------------------------------- replayable graphs
// The per-half paths (byte layout without the resident/fused kernels, and
// the bit-plane layout) launch 3 kernels per sweep, so small and mid-size
// lattices are bound by launch overhead.  Their sweeps are captured once per
// context as a graph of kGraphSweeps sweeps whose kernels take the sweep
// index from a device counter (refresh kernels that skip non-refresh
// sweeps, thresholds from the schedule tables) and replayed.
constexpr int kGraphSweeps = 16;

bool use_graph(const micsa_ctx* c)
{
    return c->use_graphs && !c->timing && c->gamma == 1 && (c->bit || (!use_resident(c) && !use_fused(c)));
}

// One sweep in device-counter form on stream st.
int enqueue_dev_sweep(micsa_ctx* c, int32_t algo, hipStream_t st)
{
    const int32_t P = c->sched.period;
    if (c->bit) {
        const int WL = word_lattices(c);
        kb_refresh_dev<<<dim3(bp_refresh_blocks(c->g), (unsigned)WL), 256, 0, st>>>(
            geomb(c), c->bdm0, c->bdm1, c->d_k, P, c->d_dth);
        const dim3 grid = grid_for(c->g.Nh, WL);
        kb_micsa_half<0><<<grid, kBlock, 0, st>>>(geomb(c), c->bspin, c->bdm0, c->bdm1, c->bJ);
        kb_micsa_half<1><<<grid, kBlock, 0, st>>>(geomb(c), c->bspin, c->bdm0, c->bdm1, c->bJ);
        c->tally_ok = false;
    } else {
        const int64_t words = (int64_t)c->g.rows * c->g.Wr;
        if (algo == MICSA_ALGO_MICSA) {
            k_refresh_dev<<<grid_for(c->g.Nh / 4, c->L), kBlock, 0, st>>>(c->g, c->dem, c->d_k, P, c->d_dth);
            k_micsa_half<0><<<grid_for(words, c->L), kBlock, 0, st>>>(c->g, c->spin, c->dem, c->tally, 0);
            k_micsa_half<1><<<grid_for(words, c->L), kBlock, 0, st>>>(c->g, c->spin, c->dem, c->tally, 0);
        } else {
            const HeatBathThresholds none{};
            enqueue_canonical_half<0>(c, algo, st, 0, none, c->d_k);
            enqueue_canonical_half<1>(c, algo, st, 0, none, c->d_k);
        }
    }
    k_count_sweep<<<1, 1, 0, st>>>(c->d_k);
    return check_launch(c, "device-counter sweep");
}

int sweep_graph(micsa_ctx* c, int32_t algo, int64_t n)
{
    const void* key = c->bit ? (const void*)c->bspin : (const void*)c->spin;
    hipGraphExec_t& ex = c->gexec[algo];
    if (ex && c->gkey[algo] != key) {  // state buffers moved since the capture
        (void)hipGraphExecDestroy(ex);
        ex = nullptr;
    }
    if (!c->d_k && !ctx_alloc(c, c->d_k, 8)) return fail(c, MICSA_EHIP, "sweep counter");
    if (!ex && n >= kGraphSweeps) {
        if (!c->cap_stream) HIP_TRY(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
        HIP_TRY(c, hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal));
        int st = MICSA_OK;
        for (int i = 0; i < kGraphSweeps && !st; ++i) st = enqueue_dev_sweep(c, algo, c->cap_stream);
        hipGraph_t graph = nullptr;
        const hipError_t e = hipStreamEndCapture(c->cap_stream, &graph);
        if (st) return st;
        if (e != hipSuccess) return fail(c, MICSA_EHIP, std::string("hipStreamEndCapture: ") + hipGetErrorString(e));
        const hipError_t e2 = hipGraphInstantiate(&ex, graph, nullptr, nullptr, 0);
        (void)hipGraphDestroy(graph);
        if (e2 != hipSuccess) {
            ex = nullptr;
            return fail(c, MICSA_EHIP, std::string("hipGraphInstantiate: ") + hipGetErrorString(e2));
        }
        c->gkey[algo] = key;
    }
    k_set_counter<<<1, 1, 0, c->stream>>>(c->d_k, c->k);
    int64_t done = 0;
    if (ex)
        for (; done + kGraphSweeps <= n; done += kGraphSweeps) HIP_TRY(c, hipGraphLaunch(ex, c->stream));
    for (; done < n; ++done) {
        const int st = enqueue_dev_sweep(c, algo, c->stream);
        if (st) return st;
    }
    c->k += n;
    return MICSA_OK;
}

// Checks shared by every sweep entry point.
int check_sweep(micsa_ctx* c, int32_t algo, int64_t n)
{
    if (algo != MICSA_ALGO_MICSA && algo != MICSA_ALGO_HEATBATH && algo != MICSA_ALGO_WALKERS &&
        algo != MICSA_ALGO_METROPOLIS)
        return fail(c, MICSA_EINVAL, "unknown algo");
    if (c->bit && algo == MICSA_ALGO_WALKERS) return fail(c, MICSA_EINVAL, "walkers run in the byte layout");
    if (c->bit && algo != MICSA_ALGO_MICSA)
        return fail(c, MICSA_EINVAL, "the heat-bath and Metropolis baselines run in the byte layout");
    if (n < 0) return fail(c, MICSA_EINVAL, "negative sweep count");
    if (!c->sched.set) return fail(c, MICSA_ESTATE, "no schedule installed");
    if (c->k + n > c->sched.n_sweeps) return fail(c, MICSA_ERANGE, "sweeps beyond the schedule length");
    return MICSA_OK;
}

// Wandering step of every walker family at the end of timestep t (each
// family along its own direction, the half of the cycle given by t's parity).
int launch_wander_families(micsa_ctx* c, const WanderParity& wp)
{
    const int64_t words = (int64_t)c->g.rows * c->g.Wr;
    {
        TimedLaunch tl(c, kTimeSweep);
        k_wander<<<grid_for(words, c->L * c->gamma), kBlock, 0, c->stream>>>(c->g, c->dem, wp);
    }
    return check_launch(c, "k_wander");
}

int launch_wander(micsa_ctx* c, int64_t t)
{
    const int32_t p = (int32_t)(t & 1);
    return launch_wander_families(c, WanderParity{{p, p, p, p, p, p}});
}

// Tile of the one-launch multispin sweep: TY rows x TZ planes per work-group
// ((TY + 4) Lx / 128 lanes; the last tile along y holds the rows left over).
// Automatic TY: the most rows whose lanes, ring of 4 rows included, fill
// whole waves, up to three (Lx = 512: 44 rows, 192 lanes), so that no wave
// runs mostly empty; TZ divides Lz.
MscTile msc_tile(const micsa_ctx* c)
{
    const int W = c->p.Lx / 128;
    MscTile f{};
    if (c->tile_y) {
        f.TY = c->tile_y;
    } else {
        int rows = 0;
        for (int r = 5; r * W <= 192; ++r)
            if ((r * W) % 64 == 0) rows = r;
        f.TY = rows ? std::min(rows - 4, c->p.Ly) : divisor_at_most(c->p.Ly, std::max(1, 256 / W - 4));
    }
    f.TZ = c->tile_z ? c->tile_z : divisor_at_most(c->p.Lz, 8);
    f.nty = (c->p.Ly + f.TY - 1) / f.TY;
    f.ntz = c->p.Lz / f.TZ;
    f.xcd = c->xcd_map == 2 && f.ntz % 8 == 0 ? 2 : (c->xcd_map && (f.nty * f.ntz) % 8 == 0 ? 1 : 0);
    return f;
}

// Tile of the two-sweep multispin pass (msc2_kernels.hpp): lanes of 32 sites,
// (TY + 8) rows of Lx / 64 words, or every row of the lattice without a ring
// where they fit, by TZ planes; neither need divide its side.  The automatic
// tile is the one with the least estimated time: TZ + 6 steps of a chain's
// latency and the issue and LDS time of the waves a unit holds (2.4 GHz
// cycles).  Measured, us per pass of 512^3 by rows x planes, with the waves per
// unit: 32 x 16 30.3 (10), 24 x 16 32.0 (12), 32 x 32 34.2 (5), 56 x 32 38 (8),
// 24 x 8 37 (two rounds of 12); of 32 lattices of 128^3: 128 x 8 18.8 (8), 128 x
// 16 21.1 (4); of 256^3: 24 x 4 11.0 (6), 24 x 16 17.0 (4).
constexpr int kMscPassSweeps = 2;
constexpr double kMsc2Chain = 1500, kMsc2Wave = 150, kMsc2Launch = 3600;

int msc2_block(const MscTile& f, int W) { return ((f.TY + (f.nty > 1 ? 4 * kMscPassSweeps : 0)) * W + 63) / 64 * 64; }

size_t msc2_lds(const MscTile& f, int W) { return (size_t)4 * kMsc2Words * (size_t)(msc2_block(f, W) + W); }

// Estimated cycles per launch (two sweeps of every lattice).
double msc2_cost(const micsa_ctx* c, const MscTile& f)
{
    const int W = c->p.Lx / 64, waves = msc2_block(f, W) / 64, cus = c->cus > 0 ? c->cus : 256;
    const int fit = (int)std::max<size_t>(1, std::min<size_t>((size_t)160 * 1024 / msc2_lds(f, W), (size_t)(16 / waves)));
    const double per_cu = std::ceil((double)f.nty * f.ntz * c->L / cus);
    const double m = std::min<double>(per_cu, fit), rounds = std::ceil(per_cu / fit);
    return rounds * (f.TZ + 6) * (kMsc2Chain + kMsc2Wave * m * waves) + kMsc2Launch;
}

MscTile msc2_plan(const micsa_ctx* c)
{
    if (!msc_eligible(c)) return MscTile{};
    const int W = c->p.Lx / 64, ring = 4 * kMscPassSweeps, Ly = c->p.Ly, Lz = c->p.Lz;
    MscTile best{};
    double cost = 0;
    auto consider = [&](int TY, int TZ) {
        MscTile f{};
        f.TY = TY;
        f.TZ = TZ;
        f.nty = (Ly + TY - 1) / TY;
        f.ntz = (Lz + TZ - 1) / TZ;
        f.xcd = c->xcd_map && f.nty * f.ntz >= 8;
        if (msc2_block(f, W) > kMsc2Lanes && !c->tile_y) return;
        const double t = msc2_cost(c, f);
        if (!best.TY || t < cost) {
            best = f;
            cost = t;
        }
    };
    for (int ny = 1; ny <= Ly && (ny == 1 || Ly / ny >= 6); ++ny) {
        const int TY = c->tile_y ? c->tile_y : (Ly + ny - 1) / ny;
        if (c->tile_y || ny == 1 || (TY + ring) * W <= kMsc2Lanes)
            for (int nz = 1; nz <= Lz; nz = nz < 16 ? nz + 1 : nz + nz / 8) {
                consider(TY, c->tile_z ? c->tile_z : (Lz + nz - 1) / nz);
                if (c->tile_z) break;
            }
        if (c->tile_y || ((TY + ring) * W <= 64 && best.TY)) break;  // narrower than a wave: no use
    }
    return best;
}

// The pass fits a work-group: lanes and LDS (at most 96 KiB).
bool msc2_fits(const micsa_ctx* c)
{
    const MscTile& f = c->tile2;
    const int W = c->p.Lx / 64;
    return c->msc_pass == 2 && f.TY > 0 && msc2_block(f, W) <= kMsc2Lanes && msc2_lds(f, W) <= 96 * 1024;
}

bool msc_one_launch(const micsa_ctx* c)
{
    return c->msc_fused && ((msc_tile(c).TY + 4) * (c->p.Lx / 128) + 63) / 64 * 64 <= kMscSweepLanes;
}

// Draw-ahead grid, beside the sweeps: up to four waves per SIMD, which fill the
// slots that the sweep's waves (of a higher issue priority) leave.  512^3 with a
// refresh every 20 sweeps takes 18.3 us per sweep with 1024 blocks, 17.7 with
// 4096, 19.0 with a thread per word (15.5 without refreshes); 32 lattices of
// 128^3 with one every 10: 13.3, 11.2, 12.3 (9.5).
constexpr int64_t kDrawBlocks = 4096;


// Launch the draw of refresh sweep kr's levels on the side stream, after
// everything the library stream holds so far (the previous refresh sweep
// reads the same planes); the refresh sweep waits for draw_done.
// alone: nothing of the call runs beside the draw (a refresh at the call's
// first sweep), so it takes a full grid, a thread per word
int draw_levels(micsa_ctx* c, int64_t kr, bool alone = false)
{
    const int64_t rho = refresh_index(kr, c->sched.period);
    const double T = temperature(c->sched, rho);
    if (!(T > 0.0) || !std::isfinite(T)) return fail(c, MICSA_ERANGE, "no temperature for this refresh");
    CellDraw D{};
    D.cg = cell_geom(c);
    D.dr0 = w32(c->mdr0);
    D.dr1 = w32(c->mdr1);
    D.dth = c->d_dth;
    D.rho0 = rho;
    D.n = 1;
    D.L = c->L;
    D.families = 1;
    const int64_t full = (D.cg.plane + 63) / 64;
    const int64_t blocks = alone ? std::min<int64_t>(full, 65535)
                                 : std::max<int64_t>(1, std::min<int64_t>(full, kDrawBlocks / c->L));
    HIP_TRY(c, hipEventRecord(c->draw_free, c->stream));
    HIP_TRY(c, hipStreamWaitEvent(c->draw_stream, c->draw_free, 0));
    k_cells_draw<<<dim3((unsigned)blocks, (unsigned)c->L), 64, 0, c->draw_stream>>>(D);
    const int st = check_launch(c, "k_cells_draw");
    if (st) return st;
    HIP_TRY(c, hipEventRecord(c->draw_done, c->draw_stream));
    return MICSA_OK;
}

// Sweep of refresh rho (gamma = 1).
int64_t refresh_sweep(int64_t rho, int32_t P) { return P >= 1 ? rho * P : ((int64_t)1 << rho) - 1; }

// First refresh sweep in [from, end), or -1.
int64_t next_refresh(const micsa_ctx* c, int64_t from, int64_t end)
{
    const int32_t P = c->sched.period;
    const int64_t k = is_refresh(from, P) ? from : refresh_sweep(refresh_index(from, P) + 1, P);
    return k < end ? k : -1;
}

// MicSA sweeps k .. k + n - 1 on multispin planes: pack the byte state
// unless the planes are live, sweep (two sweeps per launch where the pass
// applies, else one launch per sweep marching along z, or one per half
// sweep; refresh levels drawn ahead on the side stream, or in the sweep),
// and leave the planes live.  Walkers (one-launch only): each sweep applies
// the previous timestep's wandering as it loads the levels; the last one is
// left owed to the byte layout (pend_wander).
MscGeom msc_geom(const micsa_ctx* c)
{
    MscGeom m;
    m.W = c->p.Lx / 128;
    m.R = c->g.rows;
    m.plane = (int64_t)m.R * m.W;
    return m;
}

CellGeom cell_geom(const micsa_ctx* c)
{
    CellGeom cg;
    cg.g = c->g;
    cg.W = (c->g.Kx + 31) / 32;
    cg.bdiv = msc_eligible(c) ? 1 : c->g.R;  // the multispin kernels read a set of couplings per lattice
    cg.plane = (int64_t)c->g.rows * cg.W;
    return cg;
}

uint32_t* w32(uint64_t* p) { return reinterpret_cast<uint32_t*>(p); }

// Current level planes of every family.
CellLevels cell_levels(const micsa_ctx* c)
{
    CellLevels lv{};
    lv.families = c->gamma;
    if (c->gamma == 1) {
        lv.d0[0] = w32(c->md0);
        lv.d1[0] = w32(c->md1);
        return lv;
    }
    const int64_t words = (int64_t)c->L * 2 * cell_geom(c).plane;
    for (int a = 0; a < c->gamma; ++a) {
        lv.d0[a] = c->fl[c->fcur[a]][a];
        lv.d1[a] = lv.d0[a] + words;
    }
    return lv;
}

// Unpack the planes into the layout's own arrays if those are stale (before
// anything reads them).
int need_home(micsa_ctx* c)
{
    // (between calls of a captured context a replay may have moved on the planes)
    const bool replayed = c->captured && c->rest.planes && c->planes_ok && c->depth == 0;
    if (c->home_ok && !replayed) return MICSA_OK;
    const CellGeom cg = cell_geom(c);
    {
        TimedLaunch t(c, kTimeReduce);
        if (c->bit)
            k_cells_unpack_bits<<<dim3((unsigned)((2 * cg.plane + 3) / 4), (unsigned)word_lattices(c)), 256, 0,
                                  c->stream>>>(geomb(c), cg, w32(c->ms), w32(c->md0), w32(c->md1), c->bspin, c->bdm0,
                                               c->bdm1);
        else
            k_cells_unpack<<<dim3((unsigned)((cg.plane + 255) / 256), (unsigned)c->L), 256, 0, c->stream>>>(
                cg, w32(c->ms), cell_levels(c), w32(c->mb), c->spin, c->dem);
    }
    int st = check_launch(c, "k_cells_unpack");
    bool owes = false;
    for (int a = 0; a < c->gamma && c->gamma > 1; ++a) owes = owes || c->fowed[a] >= 0;
    if (!st && owes) {
        WanderParity wp{{-1, -1, -1, -1, -1, -1}};
        for (int a = 0; a < c->gamma; ++a) wp.p[a] = c->fowed[a];
        st = launch_wander_families(c, wp);
    }
    if (!st) c->home_ok = true;
    return st;
}

// The same before something writes them.
int own_home(micsa_ctx* c)
{
    const int st = need_home(c);
    if (!st) c->planes_ok = false;
    return st;
}

// Pack the planes if they are stale (before a sweep on them, which then owns
// the state).
int need_planes(micsa_ctx* c)
{
    if (c->planes_ok) return MICSA_OK;
    const CellGeom cg = cell_geom(c);
    {
        TimedLaunch t(c, kTimeReduce);
        if (c->bit)
            k_cells_pack_bits<<<dim3((unsigned)((2 * cg.plane + 3) / 4), (unsigned)word_lattices(c)), 256, 0,
                                c->stream>>>(geomb(c), cg, c->bspin, c->bdm0, c->bdm1, c->bJ, w32(c->ms), w32(c->md0),
                                             w32(c->md1), w32(c->mb));
        else
            k_cells_pack<<<dim3((unsigned)((cg.plane + 255) / 256), (unsigned)c->L), 256, 0, c->stream>>>(
                cg, c->spin, c->dem, w32(c->ms), cell_levels(c), w32(c->mb));
    }
    const int st = check_launch(c, "k_cells_pack");
    for (int32_t& o : c->fowed) o = -1;
    if (!st) c->planes_ok = true;
    return st;
}

// The multispin planes a sweep call needs (the alternates for the one-launch
// sweep, the drawn levels for the draw ahead) and the draw stream.  A failed
// allocation frees only what this call allocated (the planes may hold the
// live state).
int msc_alloc(micsa_ctx* c, bool one, bool ahead)
{
    const MscGeom m = msc_geom(c);
    const size_t words = (size_t)c->L * 2 * (size_t)m.plane;
    std::vector<uint64_t**> fresh;
    auto get = [&](uint64_t** q, size_t n) {
        if (*q) return true;
        if (!ctx_alloc(c, *q, n * 8)) return false;
        fresh.push_back(q);
        return true;
    };
    bool ok = get(&c->ms, words) && get(&c->md0, words) && get(&c->md1, words) && get(&c->mb, words * 3);
    if (ok && one) ok = get(&c->ms_alt, words) && get(&c->md0_alt, words) && get(&c->md1_alt, words);
    if (ok && ahead) ok = get(&c->mdr0, words) && get(&c->mdr1, words);
    if (!ok) {
        for (uint64_t** q : fresh) {
            ctx_free(c, *q);
            *q = nullptr;
        }
        return fail(c, MICSA_ENOMEM, "multispin planes");
    }
    if (ahead && !c->draw_stream) {
        HIP_TRY(c, take_stream(c->store, c->device, &c->draw_stream));
        HIP_TRY(c, hipEventCreateWithFlags(&c->draw_free, hipEventDisableTiming));
        HIP_TRY(c, hipEventCreateWithFlags(&c->draw_done, hipEventDisableTiming));
    }
    return MICSA_OK;
}

// How far past the end of a call the next refresh's levels are drawn ahead
// (they are ready for the next call if it starts there).
constexpr int64_t kMscDrawWindow = 1024;

int sweep_msc(micsa_ctx* c, int64_t n, bool walkers = false)
{
    const MscGeom m = msc_geom(c);
    const MscTile f = msc_tile(c);
    const int lanes = (f.TY + 4) * m.W;
    const bool one = msc_one_launch(c);
    const bool ahead = one && c->draw_ahead;
    const bool fits2 = msc2_fits(c);
    const MscTile f2 = c->tile2;
    if (int st = msc_alloc(c, one, ahead)) return st;
    int st = MICSA_OK;
    const int64_t k_end = c->k + n;
    int64_t drawn = -1;  // refresh sweep whose levels the draw planes hold (or are being drawn)
    // The first refresh of the call may have been drawn during the previous
    // one.  A refresh at the call's first sweep has no sweep of the call to
    // hide a draw behind: its levels (which depend on the schedule only) are
    // drawn by a full grid, enqueued before the pack so that the two run side
    // by side, and the call's first sweeps read them like any other.
    if (ahead && (drawn = next_refresh(c, c->k, k_end)) >= 0 && drawn != c->msc_drawn &&
        (st = draw_levels(c, drawn, drawn == c->k)))
        return st;
    c->msc_drawn = -1;
    if ((st = need_planes(c))) return st;
    c->home_ok = false;
    const dim3 grid((unsigned)((m.plane + 255) / 256), (unsigned)c->L);
    const dim3 sgrid((unsigned)(f.nty * f.ntz), (unsigned)c->L);
    const unsigned sblock = (unsigned)((lanes + 63) / 64 * 64);
    const size_t slds = (size_t)96 * lanes;  // 6 planes x 2 step buffers x 8 B per lane
    for (int64_t i = 0; i < n; ++i) {
        const int64_t k = c->k;
        const bool refresh = is_refresh(k, c->sched.period);
        const int64_t rho = refresh_index(k, c->sched.period);
        const double T = temperature(c->sched, rho);
        if (!(T > 0.0) || !std::isfinite(T)) return fail(c, MICSA_ERANGE, "no temperature for this refresh");
        const DaemonThresholds th = refresh ? daemon_thresholds(T) : DaemonThresholds{0, 0, 0};
        // walkers pass their levels' carry words between the lanes of a row,
        // which share a wave when Lx / 128 divides 64
        if (one && (walkers ? 64 % (2 * m.W) == 0 : c->pend_wander < 0) && i + 1 < n && fits2) {
            // sweeps k and k + 1 in one pass; a refresh among them reads its
            // drawn levels (at most one refresh per pass, drawn ahead)
            const bool refresh2 = is_refresh(k + 1, c->sched.period);
            const bool ok2 = (!refresh || (ahead && drawn == k)) && (!refresh2 || (ahead && drawn == k + 1)) &&
                             !(refresh && refresh2);
            if (ok2) {
                if (refresh || refresh2) HIP_TRY(c, hipStreamWaitEvent(c->stream, c->draw_done, 0));
                const int n2 = f2.nty * f2.ntz;
                const dim3 grid2((unsigned)(f2.xcd ? (n2 + 7) / 8 * 8 : n2), (unsigned)c->L);
                const unsigned block2 = (unsigned)msc2_block(f2, 2 * m.W);
                const size_t lds2 = msc2_lds(f2, 2 * m.W);
                const auto kern = walkers ? (refresh2 ? k_msc_sweep_multi<kMscPassSweeps, 1, true>
                                                      : k_msc_sweep_multi<kMscPassSweeps, -1, true>)
                                          : (refresh2 ? k_msc_sweep_multi<kMscPassSweeps, 1, false>
                                                      : k_msc_sweep_multi<kMscPassSweeps, -1, false>);
                if (lds2 > 64 * 1024 &&
                    hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds2) !=
                        hipSuccess)
                    return fail(c, MICSA_EHIP, "k_msc_sweep_multi LDS attribute");
                CellGeom a_g = cell_geom(c);
                MscTile a_f = f2;
                const uint32_t *a_s = w32(c->ms), *a_d0 = w32(refresh ? c->mdr0 : c->md0),
                               *a_d1 = w32(refresh ? c->mdr1 : c->md1), *a_b = w32(c->mb), *a_r0 = w32(c->mdr0),
                               *a_r1 = w32(c->mdr1);
                uint32_t *o_s = w32(c->ms_alt), *o_d0 = w32(c->md0_alt), *o_d1 = w32(c->md1_alt);
                unsigned long long* a_t = c->tally;
                // walkers: the wandering owed to sweep k's levels (none after a
                // refresh), and sweep k's own, applied before sweep k + 1 (none
                // when that one refreshes)
                int a_w = walkers && !refresh ? c->pend_wander : -1;
                int a_wA = walkers && !refresh2 ? (int)(k & 1) : -1;
                void* args[] = {&a_g, &a_f, &a_s, &a_d0, &a_d1, &a_b, &a_r0, &a_r1, &o_s, &o_d0, &o_d1,
                                &a_t, &a_w, &a_wA};
                hipEvent_t e0 = nullptr, e1 = nullptr;
                if (c->timing && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)) {
                    if (e0) (void)hipEventDestroy(e0);
                    e0 = e1 = nullptr;
                }
                const hipError_t le =
                    hipExtLaunchKernel((const void*)kern, grid2, block2, args, lds2, c->stream, e0, e1, 0);
                if (e0 && e1) {
                    if (le == hipSuccess) {
                        c->events[kTimeSweep].push_back({e0, e1});
                    } else {
                        (void)hipEventDestroy(e0);
                        (void)hipEventDestroy(e1);
                    }
                }
                if (le != hipSuccess)
                    return fail(c, MICSA_EHIP, std::string("k_msc_sweep_multi: ") + hipGetErrorString(le));
                if ((st = check_launch(c, "k_msc_sweep_multi"))) return st;
                // the next refresh, in this call or (within the window) a later one
                if ((refresh || refresh2) && ahead &&
                    (drawn = next_refresh(c, k + 2, std::min(c->sched.n_sweeps, k_end + kMscDrawWindow))) >= 0 &&
                    (st = draw_levels(c, drawn)))
                    return st;
                std::swap(c->ms, c->ms_alt);
                std::swap(c->md0, c->md0_alt);
                std::swap(c->md1, c->md1_alt);
                // gamma = 1: sweep k + 1 is timestep k + 1; walkers owe its wandering
                c->pend_wander = walkers ? (int32_t)((k + 1) & 1) : -1;
                c->k = k + 2;
                ++i;
                continue;
            }
        }
        if (one) {
            // a refresh sweep with levels drawn ahead is a plain sweep reading them
            const bool use_drawn = refresh && ahead && drawn == k;
            if (use_drawn) HIP_TRY(c, hipStreamWaitEvent(c->stream, c->draw_done, 0));
            {
                const bool fresh = refresh && !use_drawn, walk = !refresh && c->pend_wander >= 0;
                const auto kern = fresh  ? k_msc_sweep<true, 0>
                                  : walk ? (64 % m.W == 0 ? k_msc_sweep<false, 1> : k_msc_sweep<false, 2>)
                                         : k_msc_sweep<false, 0>;
                // arguments typed as the kernel declares them
                Geom a_g = c->g;
                MscGeom a_m = m;
                MscTile a_f = f;
                const uint64_t *a_s = c->ms, *a_d0 = use_drawn ? c->mdr0 : c->md0,
                               *a_d1 = use_drawn ? c->mdr1 : c->md1, *a_b = c->mb;
                uint64_t *o_s = c->ms_alt, *o_d0 = c->md0_alt, *o_d1 = c->md1_alt;
                unsigned long long* a_t = c->tally;
                uint32_t a_rho = (uint32_t)rho;
                DaemonThresholds a_th = th;
                int a_w = refresh ? -1 : c->pend_wander;
                void* args[] = {&a_g,  &a_m, &a_f, &a_s, &a_d0,  &a_d1, &a_b,
                                &o_s,  &o_d0, &o_d1, &a_t, &a_rho, &a_th, &a_w};
                // with timing on, the events belong to the dispatch itself and
                // time the kernel alone (separate event packets around it add
                // a few microseconds per launch)
                hipEvent_t e0 = nullptr, e1 = nullptr;
                if (c->timing && (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess)) {
                    if (e0) (void)hipEventDestroy(e0);
                    e0 = e1 = nullptr;
                }
                const hipError_t le =
                    hipExtLaunchKernel((const void*)kern, sgrid, sblock, args, slds, c->stream, e0, e1, 0);
                if (e0 && e1) {
                    if (le == hipSuccess) {
                        c->events[kTimeSweep].push_back({e0, e1});
                    } else {
                        (void)hipEventDestroy(e0);
                        (void)hipEventDestroy(e1);
                    }
                }
                if (le != hipSuccess) return fail(c, MICSA_EHIP, std::string("k_msc_sweep: ") + hipGetErrorString(le));
            }
            if ((st = check_launch(c, "k_msc_sweep"))) return st;
            // after a refresh: the next one, in this call or (within the
            // window) a later one
            if (refresh && ahead &&
                (drawn = next_refresh(c, k + 1, std::min(c->sched.n_sweeps, k_end + kMscDrawWindow))) >= 0 &&
                (st = draw_levels(c, drawn)))
                return st;
            std::swap(c->ms, c->ms_alt);
            std::swap(c->md0, c->md0_alt);
            std::swap(c->md1, c->md1_alt);
            // gamma = 1: sweep k is timestep k; walkers owe its wandering to the next load
            c->pend_wander = walkers ? (int32_t)(k & 1) : -1;
            c->k = k + 1;
            continue;
        }
        {
            TimedLaunch t(c, kTimeSweep);
            if (refresh)
                k_msc_half<0, true><<<grid, 256, 0, c->stream>>>(c->g, m, c->ms, c->md0, c->md1, c->mb, c->tally,
                                                                (uint32_t)rho, th);
            else
                k_msc_half<0, false><<<grid, 256, 0, c->stream>>>(c->g, m, c->ms, c->md0, c->md1, c->mb, c->tally,
                                                                 (uint32_t)rho, th);
        }
        if ((st = check_launch(c, "k_msc_half<0>"))) return st;
        {
            TimedLaunch t(c, kTimeSweep);
            if (refresh)
                k_msc_half<1, true><<<grid, 256, 0, c->stream>>>(c->g, m, c->ms, c->md0, c->md1, c->mb, c->tally,
                                                                (uint32_t)rho, th);
            else
                k_msc_half<1, false><<<grid, 256, 0, c->stream>>>(c->g, m, c->ms, c->md0, c->md1, c->mb, c->tally,
                                                                 (uint32_t)rho, th);
        }
        if ((st = check_launch(c, "k_msc_half<1>"))) return st;
        c->k = k + 1;
    }
    // the planes keep the state (unpacked when the byte arrays are next
    // needed); a draw for a refresh after this call is joined into the library
    // stream here and kept for the call that starts there
    if (ahead && drawn >= k_end) {
        HIP_TRY(c, hipStreamWaitEvent(c->stream, c->draw_done, 0));
        c->msc_drawn = drawn;
    }
    return MICSA_OK;
}

// Apply a wandering the daemons still owe (walkers on the fused sweep).
int settle_wander(micsa_ctx* c)
{
    if (c->pend_wander < 0) return MICSA_OK;
    if (int st = own_home(c)) return st;  // the wandering kernel moves the byte arrays' levels
    const int st = launch_wander(c, c->pend_wander);
    if (!st) c->pend_wander = -1;
    return st;
}

// ------------------------------------------------------------- cell sweeps
// The launch plan (cells.hpp) of a lattice: the tile and the sweeps per
// launch with the least estimated time per sweep.  The estimate, in cycles
// of 2.4 GHz: a half sweep of a work-group costs its waves' issue slots (four
// SIMDs; 4 cycles per VALU instruction, about 36 per cell and half) or the
// latency of one wave's chain, whichever is longer, and work-groups of one
// unit share its SIMDs; a launch costs kCellLaunch beside that, and its
// operands (72 B per cell computed on) at kCellBytes per cycle.  A whole
// lattice in one work-group pays those once per call.  Measured against it
// on one MI355X, us per sweep: 64^3 x 2, tiles of 8 x 8 rows and 6 sweeps
// per launch 1.32 (estimate 1.41), 16 x 16 and 4 1.68 (1.45), one work-group
// per lattice 1.73 (2.0); 128^3, 16 x 16 and 4 2.92 (2.7); 256^3, 16 x 16 and
// 2 9.4 (6.2).
constexpr double kCellIssue = 4.0 * 36, kCellChain = 340, kCellLaunch = 9000, kCellBytes = 2900;
constexpr int kCellCap = kCellMaxNR * kCellLanes;

bool cells_shape_ok(const micsa_ctx* c)
{
    const CellGeom cg = cell_geom(c);
    return cg.plane < ((int64_t)1 << 30) && cg.W <= kCellCap / 25 && c->p.Ly < (1 << 22) && c->p.Lz < (1 << 22);
}

// Work-groups of a plan on one unit: held at once (by the waves per SIMD that the
// registers allow) and in rounds, and the cycles of a half sweep of those.
struct CellLoad {
    double m, rounds, half;
    int waves;
};

CellLoad cell_load(const micsa_ctx* c, int nr, int xm, unsigned block, int64_t wgs)
{
    CellLoad d;
    d.waves = (int)block / 64;
    const double issue = kCellIssue * (xm == 0 ? 1.0 : (xm == 1 ? 1.15 : 1.2)) * nr;  // of one wave and half
    const int fit = std::max(1, (nr == 1 ? 32 : (nr == 2 ? 20 : 16)) / d.waves), cus = c->cus > 0 ? c->cus : 256;
    const int64_t per_cu = (wgs + cus - 1) / cus, m = std::min<int64_t>(per_cu, fit);
    d.m = (double)m;
    d.rounds = (double)per_cu / d.m;
    d.half = std::max(kCellChain + issue, (double)((m * d.waves + 3) / 4) * issue + 100.0);
    return d;
}

CellPlans cell_plans(const micsa_ctx* c)
{
    CellPlans plans;
    CellPlan& best = plans.main;
    if (!cells_shape_ok(c)) return plans;
    const int W = (c->g.Kx + 31) / 32, Ly = c->p.Ly, Lz = c->p.Lz;
    const int xm = W == 1 ? 0 : (c->g.Kx % 32 == 0 ? 1 : 2);
    // (a context of a tiled lattice weighs over a thousand tiles when it is made, in
    // a few us: few divisions, and a plan put together only where it is the best)
    double brief[kBriefSweeps];  // us of a call of n + 1 sweeps, and the launches of it
    double launches[kBriefSweeps];
    std::fill_n(brief, kBriefSweeps, 1e300);
    auto consider = [&](int TY, int TZ, int nty, int ntz, int T) {
        const int G = 2 * T, GY = TY < Ly ? G : 0, GZ = TZ < Lz ? G : 0, EY = TY + 2 * GY, EZ = TZ + 2 * GZ;
        const int cells = EY * EZ * W;  // (at most kCellCap)
        const int nr = (cells + kCellLanes - 1) / kCellLanes;
        // (four cells of rows with a short last word, or of several families, do
        // not fit the registers; nor do three of several families with more than
        // a word per row: 4 x 160^3 with two daemons 20.8 us per sweep, on two 13.3)
        if (nr > (c->gamma > 1 ? (xm == 0 ? 3 : 2) : (xm == 2 ? 3 : kCellMaxNR)) || ntz > 65535) return;
        const bool whole = nty == 1 && ntz == 1;
        const int block = ((cells + nr - 1) / nr + 63) / 64 * 64;
        const int64_t wgs = (int64_t)nty * ntz * c->L;
        const CellLoad d = cell_load(c, nr, xm, (unsigned)block, wgs);
        const double load = kCellLaunch * d.rounds + (double)cells * (double)wgs * 72.0 / kCellBytes;
        // (several families: at most one sweep of each per launch)
        const double sweep = d.rounds * d.half * 2.0;
        const double t = sweep + (whole ? (c->gamma > 1 ? load / c->gamma : 0.0) : load / T);
        auto put = [&](CellPlan& p, double call) {
            p.ok = true;
            p.f = CellTile{TY, TZ, GY, GZ, EY, EZ, nty, ntz, 1.0f / (float)(EY * W), 1.0f / (float)W, 1.0f / (float)Ly,
                           1.0f / (float)Lz};
            p.nr = nr;
            p.xm = xm;
            p.block = (unsigned)block;
            p.sweeps = whole ? 0 : T;
            p.cost = t;
            p.load = load;
            p.brief = call;
        };
        if (!best.ok || t < best.cost) put(best, 0);
        // (with four cells of rows of several words their kernel spills 56 registers)
        if (nr <= (xm == 1 ? 3 : kCellMaxNR) && (!plans.walk.ok || t < plans.walk.cost)) put(plans.walk, 0);
        bool better = false;
        for (int i = 0; i < kBriefSweeps; ++i) better |= launches[i] * load + (i + 1) * sweep < brief[i];
        for (int i = 0; better && i < kBriefSweeps; ++i)
            if (launches[i] * load + (i + 1) * sweep < brief[i]) {
                brief[i] = launches[i] * load + (i + 1) * sweep;
                put(plans.brief[i + 1], brief[i]);
            }
    };
    std::fill_n(launches, kBriefSweeps, 1.0);
    if ((int64_t)Ly * Lz * W <= kCellCap) consider(Ly, Lz, 1, 1, 1);
    if (best.ok && best.nr <= 2) {  // no tile makes up for its launches here
        plans.walk = best;
        return plans;
    }
    // tiles that divide a side about evenly, a few per factor of two
    auto sides = [](int L) {
        std::vector<int> v;
        int last = 0;
        for (double n = 1; n <= L; n = std::max(n + 1, n * 1.2)) {
            const int t = (int)((L + (int)n - 1) / (int)n);
            if (t != last) v.push_back(t);
            last = t;
        }
        if (last != 1) v.push_back(1);
        return v;
    };
    const std::vector<int> ys = sides(Ly), zs = sides(Lz);
    for (int T : {1, 2, 3, 4, 6, 8}) {
        if (c->gamma > 1 && T > c->gamma) break;
        for (int i = 0; i < kBriefSweeps; ++i) launches[i] = (i + T) / T;
        for (int ty : ys) {
            const int nty = (Ly + ty - 1) / ty;
            for (int tz : zs) {
                if (ty == Ly && tz == Lz) continue;
                if ((int64_t)(ty + (ty < Ly ? 4 * T : 0)) * (tz + (tz < Lz ? 4 * T : 0)) * W <= kCellCap)
                    consider(ty, tz, nty, (Lz + tz - 1) / tz, T);
            }
        }
    }
    return plans;
}

// The plan of the next launch of a call with `left` sweeps to go.  (A whole
// lattice has no second copy of its planes, so that its walkers take its plan.)
const CellPlan& plan_for(const micsa_ctx* c, int64_t left, bool walkers = false)
{
    if (c->plan.sweeps > 0 && left <= kBriefSweeps) return c->brief[left];
    return walkers && c->plan.sweeps > 0 && c->walk.ok ? c->walk : c->plan;
}

// Estimated cycles per sweep of the two-sweep multispin pass.
double msc_cost(const micsa_ctx* c) { return c->tile2.TY > 0 ? msc2_cost(c, c->tile2) / kMscPassSweeps : 1e30; }

// MicSA takes the cell sweep: on request for the resident and slab forms,
// and by default unless the multispin pass is estimated faster (us per sweep,
// cells against the pass: 128^3 2.7 and 12.8, 256^3 9.4 and 5.4, 128^3 x 32
// 20.2 and 9.0, 512^3 73.5 and 15.7).
// The bit-plane layout takes it for calls of at least kMscMinSweeps sweeps
// (a call packs the planes if they are stale) unless a launch shape of its
// own sweep is asked for: 256 x 2 lattices of 32^3 take 0.8 us per sweep, the
// word-wise sweep 8.7.
bool use_cells(const micsa_ctx* c, int64_t n = kMscMinSweeps)
{
    if (!c->plan.ok || c->no_room || c->off_cells) return false;
    if (c->bit)
        return c->kernel_opt == MICSA_KERNEL_AUTO && !c->tile_y && !c->tile_z && !c->use_graphs && !c->draw_ahead &&
               (n >= kMscMinSweeps || c->planes_ok || c->on_cells);
    if (c->kernel_opt == MICSA_KERNEL_RESIDENT || c->kernel_opt == MICSA_KERNEL_SLAB) return true;
    if (c->kernel_opt != MICSA_KERNEL_AUTO || use_graph(c)) return false;
    return !msc_eligible(c) || resident_eligible(c) || c->plan.cost < msc_cost(c);
}

// Planes (with their alternates where tiles read what others write) and room
// for drawn levels.  Drawn levels: as many refreshes as fit 8 MiB or the
// lattices' spins in bytes, whichever is more (1.25 MiB where that holds 256: a
// context below 2 MiB is made and freed in 50 us less; a pool's job: see
// plan_job), at least two (a sweep of a baseline draws the words of one
// and a half).
int64_t cells_draw_cap(const micsa_ctx* c)
{
    const size_t one = (size_t)c->L * 2 * (size_t)cell_geom(c).plane * 4 * 2;
    const size_t few = (size_t)5 << 18;
    const size_t room = c->draw_room ? c->draw_room
                        : few / one >= 256
                            ? few
                            : std::max<size_t>((size_t)8 << 20, (size_t)c->L * 2 * (size_t)c->g.Nh);
    return std::max<int64_t>(2, std::min<int64_t>((int64_t)(room / one), 1024));
}

// Words of the planes (own planes: not those of the multispin sweep).
size_t cells_plane_words(const micsa_ctx* c)
{
    const CellGeom cg = cell_geom(c);
    const size_t words = (size_t)c->L * 2 * (size_t)cg.plane;
    const bool alt = c->plan.sweeps > 0;
    const size_t levels = c->gamma > 1 ? (size_t)4 * c->gamma  // two bits, two copies each
                                       : (alt ? 4 : 2);
    return words * ((alt ? 2 : 1) + levels) + (size_t)(c->L / c->g.R) * 6 * (size_t)cg.plane;
}

// Give back planes that hold no state.
void planes_free(micsa_ctx* c)
{
    if (msc_eligible(c))
        for (uint64_t* q : {c->ms, c->md0, c->md1, c->mb, c->ms_alt, c->md0_alt, c->md1_alt}) ctx_free(c, q);
    else
        ctx_free(c, c->ms);  // one block
    c->ms = c->md0 = c->md1 = c->mb = c->ms_alt = c->md0_alt = c->md1_alt = nullptr;
    for (auto& copy : c->fl) std::fill(copy, copy + 6, nullptr);
}

int cells_alloc(micsa_ctx* c)
{
    const CellGeom cg = cell_geom(c);
    const size_t words = (size_t)c->L * 2 * (size_t)cg.plane;
    const bool fresh = !c->ms;
    if (!c->ms || (c->plan.sweeps > 0 && !c->ms_alt)) {
        if (msc_eligible(c)) {
            if (int st = msc_alloc(c, true, false)) return st;
        } else {
            const bool alt = c->plan.sweeps > 0;
            uint32_t* a = nullptr;
            if (!ctx_alloc(c, a, cells_plane_words(c) * 4)) return fail(c, MICSA_ENOMEM, "cell planes");
            auto take = [&](uint64_t*& q) {
                q = reinterpret_cast<uint64_t*>(a);
                a += words;
            };
            take(c->ms);
            if (alt) take(c->ms_alt);
            if (c->gamma > 1) {
                for (int copy = 0; copy < 2; ++copy)
                    for (int f = 0; f < c->gamma; ++f, a += 2 * words) c->fl[copy][f] = a;
            } else {
                take(c->md0);
                take(c->md1);
                if (alt) take(c->md0_alt);
                if (alt) take(c->md1_alt);
            }
            c->mb = reinterpret_cast<uint64_t*>(a);
        }
    }
    if (!c->cdr0) {
        int64_t cap = cells_draw_cap(c);
        uint32_t* a = nullptr;
        while (!ctx_alloc(c, a, words * 8 * (size_t)cap)) {  // fewer refreshes where memory is short
            if (cap <= 2) {
                if (fresh) planes_free(c);
                return fail(c, MICSA_ENOMEM, "drawn levels");
            }
            cap = std::max<int64_t>(2, cap / 4);
        }
        c->cdr0 = a;
        c->cdr1 = a + words * (size_t)cap;
        c->cdr_cap = cap;
        c->cdr_n = 0;
    }
    return MICSA_OK;
}

// Draw the levels of the refreshes from sweep kr on that a call ending before
// k_end needs, as many as there is room for; of a small lattice also later
// ones, until the launch fills a good part of the device (they are kept for
// the calls that follow, until the schedule changes).
CellDraw cells_draw_slice(micsa_ctx* c, int64_t kr, int64_t k_end)
{
    const CellGeom cg = cell_geom(c);
    const int32_t P = c->sched.period;
    const int64_t rho = refresh_index(kr, P);
    const int64_t in_call = refresh_index(k_end - 1, P) - rho + 1;
    const int64_t fill = c->capturing ? 0 : 32768 / std::max<int64_t>(1, cg.plane * c->L);
    const int64_t n = std::max<int64_t>(
        1, std::min<int64_t>({std::max(in_call, fill), c->cdr_cap, refresh_count(c->sched) - rho}));
    CellDraw D{};
    D.cg = cg;
    D.dr0 = c->cdr0;
    D.dr1 = c->cdr1;
    D.dth = c->d_dth;
    D.rho0 = rho;
    D.stride = (int64_t)c->L * 2 * cg.plane;
    D.n = (int32_t)n;
    D.L = c->L;
    D.families = 1;
    c->cdr_rho0 = rho;
    c->cdr_n = n;
    return D;
}

int64_t cells_draw_blocks(const CellDraw& D) { return std::min<int64_t>((D.n * D.cg.plane + 63) / 64, 16384); }

using CellKernel = void (*)(CellSweep);
template <int ALG, bool RING>
CellKernel cell_kernel(int nr, int xm)
{
    static const CellKernel k[kCellMaxNR][3] = {
        {k_cells_sweep<1, 0, ALG, RING>, k_cells_sweep<1, 1, ALG, RING>, k_cells_sweep<1, 2, ALG, RING>},
        {k_cells_sweep<2, 0, ALG, RING>, k_cells_sweep<2, 1, ALG, RING>, k_cells_sweep<2, 2, ALG, RING>},
        {k_cells_sweep<3, 0, ALG, RING>, k_cells_sweep<3, 1, ALG, RING>, k_cells_sweep<3, 2, ALG, RING>},
        {k_cells_sweep<4, 0, ALG, RING>, k_cells_sweep<4, 1, ALG, RING>, nullptr}};
    return k[nr - 1][xm];
}

template <int ALG>
CellKernel cell_kernel(const CellPlan& p)
{
    return p.sweeps > 0 ? cell_kernel<ALG, true>(p.nr, p.xm) : cell_kernel<ALG, false>(p.nr, p.xm);
}

// The launch's planes and shape (J holds its sweeps, draws and logging).
void fill_cells(const micsa_ctx* c, CellSweep& J, const CellPlan& pl)
{
    J.cg = cell_geom(c);
    J.f = pl.f;
    J.s_in = w32(c->ms);
    J.d0_in = w32(c->md0);
    J.d1_in = w32(c->md1);
    J.bond = w32(c->mb);
    const bool whole = pl.sweeps == 0;
    J.s_out = w32(whole ? c->ms : c->ms_alt);
    J.d0_out = w32(whole ? c->md0 : c->md0_alt);
    J.d1_out = w32(whole ? c->md1 : c->md1_alt);
    J.tally = c->tally;
    J.period = c->sched.period;
    J.lattices = c->L;
    J.inv_bdiv = 1.0f / (float)J.cg.bdiv;
}

// One launch of the cell kernel on the planes; tiles go from one copy to the
// other.
int launch_cells(micsa_ctx* c, int alg, CellSweep& J, const CellPlan& pl, const CellFamilies* F = nullptr)
{
    fill_cells(c, J, pl);
    {
        TimedLaunch t(c, alg == 1 ? kTimeHeatBath : (alg == 2 ? kTimeMetropolis : kTimeSweep));
        const dim3 grid((unsigned)pl.f.nty, (unsigned)pl.f.ntz, (unsigned)c->L);
        if (alg == 4) {
            using Kern = void (*)(CellSweep, CellFamilies);
            static const Kern k[3][3] = {
                {k_cells_sweep_families<1, 0>, k_cells_sweep_families<1, 1>, k_cells_sweep_families<1, 2>},
                {k_cells_sweep_families<2, 0>, k_cells_sweep_families<2, 1>, k_cells_sweep_families<2, 2>},
                {k_cells_sweep_families<3, 0>, k_cells_sweep_families<3, 1>, k_cells_sweep_families<3, 2>}};
            k[pl.nr - 1][pl.xm]<<<grid, pl.block, 0, c->stream>>>(J, *F);
        } else {
            static const CellKernel drawing[2][kCellMaxNR] = {
                {k_cells_sweep_drawing<1, 1>, k_cells_sweep_drawing<2, 1>, k_cells_sweep_drawing<3, 1>,
                 k_cells_sweep_drawing<4, 1>},
                {k_cells_sweep_drawing<1, 2>, k_cells_sweep_drawing<2, 2>, k_cells_sweep_drawing<3, 2>,
                 k_cells_sweep_drawing<4, 2>}};
            const CellKernel k = J.tab      ? drawing[alg - 1][pl.nr - 1]
                                 : alg == 0 ? cell_kernel<0>(pl)
                                 : alg == 1 ? cell_kernel<1>(pl)
                                 : alg == 2 ? cell_kernel<2>(pl)
                                            : cell_kernel<3>(pl);
            k<<<grid, pl.block, 0, c->stream>>>(J);
        }
    }
    if (int st = check_launch(c, "k_cells_sweep")) return st;
    if (pl.sweeps > 0) {
        std::swap(c->ms, c->ms_alt);
        if (alg == 0 || alg == 3) {  // the baselines leave the levels where they are
            std::swap(c->md0, c->md0_alt);
            std::swap(c->md1, c->md1_alt);
        }
    }
    return MICSA_OK;
}

// Logging fields of a launch of the sweeps from done on, in a call that logs
// every stride sweeps to dlog.
void cell_log(micsa_ctx* c, CellSweep& J, bool logged, int64_t done, int64_t stride)
{
    J.log = logged ? c->lograw : nullptr;
    if (!logged) return;
    J.log_stride = (int32_t)std::min<int64_t>(stride, INT32_MAX);
    J.log_first = (int32_t)std::min<int64_t>(stride - done % stride, INT32_MAX);
}

// Room for the lanes' words of `rows` logged rows, or for as many as fit 8 MiB
// (launches are cut accordingly).
bool log_room(micsa_ctx* c, int64_t rows)
{
    const int64_t row = (int64_t)c->L * c->plan.block;
    const int64_t want = std::max<int64_t>(1, std::min<int64_t>(rows, ((int64_t)2 << 20) / row));
    if (c->lograw_rows >= want) return true;
    ctx_retire(c, c->lograw);
    c->lograw_rows = 0;
    if (!ctx_alloc(c, c->lograw, (size_t)(want * row) * 4)) return false;
    c->lograw_rows = want;
    return true;
}

// Sweeps of a logged launch at most.
int64_t log_most(const micsa_ctx* c, int64_t most, int64_t stride)
{
    return stride >= most ? most : std::min(most, c->lograw_rows * stride);
}

// The rows that sweeps [done, done + n) of the call ended.
int write_log(micsa_ctx* c, int64_t done, int64_t n, int64_t stride, const unsigned long long* levels, long long* dlog)
{
    const int64_t r0 = done / stride, e = ((done + n) / stride - r0) * c->L;
    if (e == 0) return MICSA_OK;
    k_cells_log_rows<<<(unsigned)((e + 3) / 4), 256, 0, c->stream>>>(c->lograw, e, (int)c->plan.block, levels, c->L,
                                                                   dlog + r0 * c->L * 2);
    return check_launch(c, "k_cells_log_rows");
}

// The next launch of MicSA sweeps from sweep k on, in a run to k_end: its
// sweeps (at most `most`; up to the first refresh beyond the drawn ones) and
// its refreshes.  *draw is set, with the slice in *D, if their levels have to
// be drawn first.
CellSweep cells_next(micsa_ctx* c, int64_t k, int64_t k_end, int64_t most, bool* draw, CellDraw* D)
{
    const int32_t P = c->sched.period;
    const int64_t stride_w = (int64_t)c->L * 2 * cell_geom(c).plane;
    int64_t len = std::min(k_end - k, most), slot = 0;
    const int64_t kr = next_refresh(c, k, k + len);
    *draw = false;
    if (kr >= 0) {
        const int64_t rho = refresh_index(kr, P);
        if (rho < c->cdr_rho0 || rho >= c->cdr_rho0 + c->cdr_n) {
            *D = cells_draw_slice(c, kr, k_end);
            *draw = true;
        }
        slot = rho - c->cdr_rho0;
        const int64_t beyond = c->cdr_rho0 + c->cdr_n;  // first refresh not drawn
        if (refresh_index(k + len - 1, P) >= beyond) len = refresh_sweep(beyond, P) - k;
    }
    CellSweep J{};
    J.dr0 = c->cdr0 + slot * stride_w;
    J.dr1 = c->cdr1 + slot * stride_w;
    J.dr_stride = stride_w;
    J.k0 = k;
    J.n = (int32_t)len;
    J.ref0 = kr >= 0 && kr < k + len ? (int32_t)(kr - k) : (int32_t)len;
    return J;
}

// MicSA (or one walker per site) sweeps k .. k + n - 1 on the cell kernel.
// dlog (whole-lattice plans only): every `stride` sweeps (U, sum m) of each
// lattice to dlog[row][lattice][2].
int sweep_cells(micsa_ctx* c, int64_t n, long long* dlog, int64_t stride, bool walkers = false)
{
    int st;
    if ((st = cells_alloc(c)) || (st = need_planes(c))) return st;
    const int64_t k_first = c->k, k_end = c->k + n;
    c->home_ok = false;
    while (c->k < k_end) {
        const int64_t k = c->k;
        bool draw;
        CellDraw D;
        const CellPlan& pl = plan_for(c, k_end - k, walkers);
        const int64_t most = pl.sweeps > 0 ? pl.sweeps : kResidentChunk;
        CellSweep J = cells_next(c, k, k_end, dlog ? log_most(c, most, stride) : most, &draw, &D);
        if (draw) {
            {
                TimedLaunch t(c, kTimeRefresh);
                k_cells_draw<<<dim3((unsigned)cells_draw_blocks(D), (unsigned)c->L), 64, 0, c->stream>>>(D);
            }
            if ((st = check_launch(c, "k_cells_draw"))) return st;
        }
        cell_log(c, J, dlog, k - k_first, stride);
        J.wander0 = walkers && J.ref0 > 0 ? c->pend_wander : -1;
        if ((st = launch_cells(c, walkers ? 3 : 0, J, pl))) return st;
        if (dlog && (st = write_log(c, k - k_first, J.n, stride, nullptr, dlog))) return st;
        c->k = k + J.n;
        c->pend_wander = walkers ? (int32_t)((c->k - 1) & 1) : -1;
    }
    return MICSA_OK;
}

// Several daemons or walkers per site: at most one sweep of each family per
// launch, each with its own level planes; a refresh (before a timestep's
// first sweep) redraws all of them in place.
int sweep_cells_families(micsa_ctx* c, int64_t n, bool walkers)
{
    int st;
    if ((st = cells_alloc(c)) || (st = need_planes(c))) return st;
    const CellGeom cg = cell_geom(c);
    const int gamma = c->gamma;
    const int64_t words = (int64_t)c->L * 2 * cg.plane, k_end = c->k + n;
    const int32_t P = c->sched.period;
    while (c->k < k_end) {
        if ((st = need_planes(c))) return st;
        c->home_ok = false;
        if (c->k % gamma == 0 && is_refresh(c->k / gamma, P)) {
            CellDraw D{};
            const CellLevels lv = cell_levels(c);
            D.cg = cg;
            for (int a = 0; a < gamma; ++a) {
                D.fam0[a] = lv.d0[a];
                D.fam1[a] = lv.d1[a];
                c->fowed[a] = -1;
            }
            D.dth = c->d_dth;
            D.rho0 = refresh_index(c->k / gamma, P);
            D.n = 1;
            D.L = c->L;
            D.families = gamma;
            {
                TimedLaunch t(c, kTimeRefresh);
                k_cells_draw<<<dim3((unsigned)std::min<int64_t>((cg.plane + 63) / 64, 16384), (unsigned)(c->L * gamma)),
                               64, 0, c->stream>>>(D);
            }
            if ((st = check_launch(c, "k_cells_draw"))) return st;
        }
        CellSweep J{};
        CellFamilies F{};
        const CellPlan& pl = plan_for(c, k_end - c->k);
        const int64_t most = std::min<int64_t>(k_end - c->k, pl.sweeps > 0 ? std::min(pl.sweeps, gamma) : gamma);
        J.k0 = c->k;
        int64_t len = 0;
        bool settle = false;  // a family would owe a second wandering
        while (len < most && !settle) {
            const int64_t k = c->k + len, t = k / gamma;
            const int a = (int)(k - t * gamma);
            if (len > 0 && a == 0 && is_refresh(t, P)) break;
            const int in = c->fcur[a];
            F.in0[len] = c->fl[in][a];
            F.in1[len] = c->fl[in][a] + words;
            F.out0[len] = c->fl[1 - in][a];
            F.out1[len] = c->fl[1 - in][a] + words;
            F.dir[len] = a < 3 ? 2 * a : 2 * (a - 3) + 1;  // +x, +y, +z, -x, -y, -z
            F.owed[len] = c->fowed[a];
            c->fowed[a] = -1;
            c->fcur[a] = (uint8_t)(1 - in);
            ++len;
            if (walkers && a == gamma - 1) {
                for (int f = 0; f < gamma; ++f) settle = settle || c->fowed[f] >= 0;
                if (!settle)
                    for (int f = 0; f < gamma; ++f) c->fowed[f] = (int32_t)(t & 1);
            }
        }
        J.n = (int32_t)len;
        J.ref0 = J.n;
        if ((st = launch_cells(c, 4, J, pl, &F))) return st;
        c->k += len;
        if (settle) {  // (other algorithms ran the sweeps that would have used the family's levels)
            if ((st = own_home(c)) || (st = need_planes(c))) return st;
            c->home_ok = false;
            for (int f = 0; f < gamma; ++f) c->fowed[f] = (int32_t)((c->k / gamma - 1) & 1);
        }
    }
    return MICSA_OK;
}

// Walkers on the cell kernel: against the per-half kernels and their wandering
// pass always; against the multispin pass (one walker per site) by the two
// estimates; against the fused byte sweeps where the plan's estimate (a fifth
// more for the wandering) stays below theirs, 8 us for the launches or 1400
// updates/ns, twice what they reach.  us per sweep, cells against fused: 160^3
// 5.5 and 12.4, 160^3 x 16 29 and 73, 192^3 x 4 10.8 and 35, 224 x 64 x 64 3.5
// and 11.9, 320^3 21 and 44, 352^3 32 and 49.
bool use_cells_walkers(const micsa_ctx* c, int64_t n)
{
    if (!c->plan.ok || c->no_room || c->off_cells || c->bit) return false;
    if (c->kernel_opt != MICSA_KERNEL_AUTO && c->kernel_opt != MICSA_KERNEL_RESIDENT &&
        c->kernel_opt != MICSA_KERNEL_SLAB)
        return false;
    if (c->gamma > 1 || c->kernel_opt != MICSA_KERNEL_AUTO) return true;
    const CellPlan& pl = plan_for(c, n, true);
    if (use_msc(c, n, MICSA_ALGO_WALKERS)) return pl.cost < msc_cost(c);
    const double sites = (double)c->L * 2.0 * (double)c->g.Nh;
    return !use_fused(c) || pl.cost * 1.2 / 2.4e3 < std::max(8.0, sites / 1.4e6);
}

// The heat bath and Metropolis on the cell kernel: their comparisons drawn
// for as many sweeps as there is room for by one launch on the whole device,
// then the sweeps.  Against the byte-wise kernels, which pay one Philox call
// per four updates and about as much again for the comparisons, in the sweep
// itself: at most 700 updates/ns on a full device, where the draws alone run
// at about 1550 and the sweep adds its plan's estimate.  Lattices too narrow
// for the fused kernel pay two launches per sweep there.  us per sweep of the
// heat bath (Metropolis), cells against fused: 128^3 5.6 (4.7) and 20 (21), 128^3 x
// 32 60 (57) and 138 (154), 256^3 21 (19) and 34 (37), 512^3 136 (120) and 190 (210).
bool use_cells_canonical(const micsa_ctx* c)
{
    if (!c->plan.ok || c->no_room || c->off_cells || c->bit) return false;
    if (c->kernel_opt == MICSA_KERNEL_RESIDENT) return true;
    if (c->kernel_opt != MICSA_KERNEL_AUTO || use_graph(c)) return false;
    if (!use_fused(c)) return true;
    const double sites = (double)c->L * 2.0 * (double)c->g.Nh;
    return c->plan.cost / 2.4e3 + sites / 1.5e6 < sites / 0.68e6;
}

// The baselines on a whole lattice of one word per row, n sweeps: drawn in the
// sweep itself (one launch, no words through memory, but a lattice's draws on its
// own unit) or ahead on the whole device.  Cycles of either: a Philox call with
// its comparisons takes a wave 510 where a SIMD has several and 800 alone; ahead,
// a wave draws a word of 4 n4 sites in 650 + 305 n4, and the words go out and in
// at 4 TB/s; a launch costs 8000.  Heat bath, us per sweep in the sweep / ahead,
// calls of 60 sweeps: 256 of 8 x 64 x 64 9.5 / 21.5, 1024 of them 38 / 113, 16 of
// them 9.5 / 5.1, 4096 of 8^3 3.0 / 4.8, 512 of 32^3 14.8 / 14.4, 64^3 x 64 49 /
// 14; calls of one sweep: 8^3 4.2 / 7.9, 512 of 16^3 6.4 / 10.0, 32^3 10.7 / 7.5.
bool cells_draw_in_place(const micsa_ctx* c, int alg, int64_t n)
{
    const CellPlan& pl = c->plan;
    if (pl.sweeps > 0 || pl.xm != 0) return false;
    const CellLoad d = cell_load(c, pl.nr, pl.xm, pl.block, c->L);
    const double cells = (double)c->L * (double)cell_geom(c).plane, n4 = c->g.Kx / 4;
    const double simds = 4.0 * (c->cus > 0 ? c->cus : 256);
    const double call = std::max(800.0, 510.0 * std::ceil(d.m * d.waves / 4.0)) * pl.nr * n4;
    const double here = 8000.0 + (double)n * 2.0 * d.rounds * (d.half + 500.0 + call);
    const double draw = cells * 2.0 / 64.0 * std::max(1100.0, 650.0 + 305.0 * n4) / simds;
    const double words = cells * 2.0 * (alg == 1 ? 3.0 : 2.0) * 4.0 / 1750.0;
    const double ahead = 16000.0 * std::ceil((double)n / 20.0) + (double)n * (pl.cost + draw + words);
    return here * 1.1 < ahead;
}

int sweep_cells_canonical(micsa_ctx* c, int32_t algo, int64_t n, long long* dlog, int64_t stride)
{
    int st;
    if ((st = cells_alloc(c)) || (st = need_planes(c))) return st;
    const CellGeom cg = cell_geom(c);
    const int alg = algo == MICSA_ALGO_METROPOLIS ? 2 : 1, K = alg == 1 ? 3 : 2;
    const int64_t k_first = c->k, k_end = c->k + n, plane = (int64_t)c->L * cg.plane;
    c->home_ok = false;
    if (dlog && (st = enqueue_level_sum(c, c->red))) return st;  // the levels of every logged row
    if (cells_draw_in_place(c, alg, n)) {
        while (c->k < k_end) {
            const int64_t m = std::min(k_end - c->k, dlog ? log_most(c, kResidentChunk, stride) : kResidentChunk);
            CellSweep J{};
            J.tab = canonical_table(c, algo);
            J.gamma = c->gamma;
            // sweeps to the table's next entry
            const int64_t step = (int64_t)c->sched.period * c->gamma;
            J.ref0 = (int32_t)std::min<int64_t>(step > 0 ? (step - c->k % step) % step : 0, INT32_MAX);
            cell_log(c, J, dlog, c->k - k_first, stride);
            J.k0 = c->k;
            J.n = (int32_t)m;
            if ((st = launch_cells(c, alg, J, c->plan))) return st;
            if (dlog && (st = write_log(c, c->k - k_first, m, stride, c->red, dlog))) return st;
            c->k += m;
        }
        return MICSA_OK;
    }
    c->cdr_n = 0;  // the buffer holds the baselines' draws from here on
    // Sweeps drawn at once: those that fit the levels' buffer, or one of its own
    // of up to 128 MiB where that gives more and a launch could use them (512
    // lattices of 32^3: one sweep per draw and launch 26 us per sweep, ten 15).
    const size_t per = (size_t)2 * K * (size_t)plane * 4;
    int64_t room = std::min<int64_t>((int64_t)((size_t)4 * plane * c->cdr_cap * 4 / per), 4096);
    const int64_t useful = std::min<int64_t>({n, c->plan.sweeps > 0 ? c->plan.sweeps : 20, (int64_t)(((size_t)128 << 20) / per)});
    uint32_t* draws = c->cdr0;
    if (useful > room) {
        if (c->cdc_bytes < per * (size_t)useful) {
            ctx_retire(c, c->cdc);
            c->cdc_bytes = ctx_alloc(c, c->cdc, per * (size_t)useful) ? per * (size_t)useful : 0;
        }
        if (c->cdc_bytes) {
            draws = c->cdc;
            room = useful;
        }
    }
    while (c->k < k_end) {
        const int64_t len = std::min<int64_t>(k_end - c->k, room), k_draw = c->k;
        CellCanon D{};
        D.cg = cg;
        D.dr = draws;
        D.tab = canonical_table(c, algo);
        D.k0 = k_draw;
        D.n = (int32_t)len;
        D.period = c->sched.period;
        D.L = c->L;
        D.gamma = c->gamma;
        const dim3 grid((unsigned)std::min<int64_t>((cg.plane + 63) / 64, 16384), (unsigned)c->L, (unsigned)(2 * len));
        {
            TimedLaunch t(c, canonical_timing(algo));
            if (alg == 1)
                k_cells_draw_canonical<1><<<grid, 64, 0, c->stream>>>(D);
            else
                k_cells_draw_canonical<2><<<grid, 64, 0, c->stream>>>(D);
        }
        if ((st = check_launch(c, "k_cells_draw_canonical"))) return st;
        while (c->k < k_draw + len) {
            const CellPlan& pl = plan_for(c, k_end - c->k);
            const int64_t most = pl.sweeps > 0 ? pl.sweeps : len;
            const int64_t m = std::min(k_draw + len - c->k, dlog ? log_most(c, most, stride) : most);
            CellSweep J{};
            J.dr0 = draws + (c->k - k_draw) * 2 * K * plane;
            cell_log(c, J, dlog, c->k - k_first, stride);
            J.k0 = c->k;
            J.n = (int32_t)m;
            if ((st = launch_cells(c, alg, J, pl))) return st;
            if (dlog && (st = write_log(c, c->k - k_first, m, stride, c->red, dlog))) return st;
            c->k += m;
        }
    }
    return MICSA_OK;
}

// A finished job of a pool that sweeps again does so on the pool's stream.
void run_stream(micsa_ctx* c)
{
    if (!c || !c->sweep_stream || c->stream == c->sweep_stream) return;
    (void)hipStreamSynchronize(c->stream);
    c->stream = c->sweep_stream;
}

bool stream_captured(hipStream_t s)
{
    hipStreamCaptureStatus on = hipStreamCaptureStatusNone;
    if (s && hipStreamIsCapturing(s, &on) != hipSuccess) (void)hipGetLastError();
    return on != hipStreamCaptureStatusNone;
}

// Calls that wait for the stream: refused before they change anything.
int refuse_capture(micsa_ctx* c)
{
    return stream_captured(c->stream) ? fail(c, MICSA_ESTATE, "this call waits for its stream, which is being captured")
                                      : MICSA_OK;
}

// Every block that the context has now stays until the context goes.
void keep_blocks(micsa_ctx* c)
{
    for (JobStore::Block& b : c->owned) b.kept = true;
}

// A sweep call that is captured into a graph runs whenever the graph is
// replayed: it must find the state where every call and every replay leaves
// it, may not rely on levels that an earlier call drew into buffers a replay
// overwrites, and the buffers it holds the addresses of must live as long as
// the context.  So the place where the state lies when the first call is
// captured (the planes if they are current, else the layout's own arrays: no
// settling of earlier work becomes part of the graph), with the copies it lies
// in and the wanderings it owes, is where every later call that changes the
// state puts it back (rest_state), every sweep call draws what it needs, and
// no buffer is freed before the context.
int begin_sweeps(micsa_ctx* c)
{
    if (c->depth++) return MICSA_OK;
    run_stream(c);
    c->capturing = stream_captured(c->stream);
    if (c->capturing) {
        keep_blocks(c);
        if (!c->captured) {
            Rest& x = c->rest;
            x.planes = c->planes_ok;
            x.spin = c->spin, x.dem = c->dem;
            x.bspin = c->bspin, x.bdm0 = c->bdm0, x.bdm1 = c->bdm1;
            x.ms = c->ms, x.md0 = c->md0, x.md1 = c->md1;
            std::copy_n(c->fcur, 6, x.fcur);
            std::copy_n(c->fowed, 6, x.fowed);
            x.pend = c->pend_wander;
            (x.planes ? c->home_ok : c->planes_ok) = false;
            c->captured = true;
        }
    }
    if (!c->captured) return MICSA_OK;
    c->cdr_n = 0;
    c->msc_drawn = -1;
    if (c->rest.planes) c->home_ok = false;  // (read before a replay)
    return MICSA_OK;
}

int end_sweeps(micsa_ctx* c, int st)
{
    c->off_cells = c->on_cells = false;
    if (--c->depth) return st;
    if (!st) st = rest_state(c);
    if (c->capturing) keep_blocks(c);
    c->capturing = false;
    return st;
}

// The state of a captured context back to where it rests: copied where it
// ended in the other copy of its arrays; by way of the layout's own arrays
// where its levels owe other wanderings (which are exchanges: applied once
// more, they are owed again) or where it has to change its layout.
template <class T>
int rest_copy(micsa_ctx* c, T*& now, T*& other, T* place, size_t bytes)
{
    if (now == place) return MICSA_OK;
    k_copy_u64<<<(unsigned)std::min<size_t>((bytes / 8 + 255) / 256, 4096), 256, 0, c->stream>>>(
        reinterpret_cast<const uint64_t*>(now), (int64_t)(bytes / 8), reinterpret_cast<uint64_t*>(place));
    other = now;
    now = place;
    return check_launch(c, "k_copy_u64");
}

// The end of a synchronous call that has changed the state.
int rest_and_wait(micsa_ctx* c)
{
    if (int st = rest_state(c)) return st;
    HIP_TRY(c, hipStreamSynchronize(c->stream));
    return MICSA_OK;
}

int rest_state(micsa_ctx* c)
{
    if (!c->captured) return MICSA_OK;
    const Rest& x = c->rest;
    const size_t plane_bytes = (size_t)c->L * 2 * (size_t)cell_geom(c).plane * 4;
    int st;
    if (x.planes && c->planes_ok && c->pend_wander == x.pend &&
        (c->gamma == 1 || (std::equal(x.fcur, x.fcur + 6, c->fcur) && std::equal(x.fowed, x.fowed + 6, c->fowed)))) {
        c->home_ok = false;
        if ((st = rest_copy(c, c->ms, c->ms_alt, x.ms, plane_bytes))) return st;
        if ((st = rest_copy(c, c->md0, c->md0_alt, x.md0, plane_bytes))) return st;
        return rest_copy(c, c->md1, c->md1_alt, x.md1, plane_bytes);
    }
    if ((st = own_home(c))) return st;
    if (c->pend_wander != x.pend) {
        if (c->pend_wander >= 0 && (st = launch_wander(c, c->pend_wander))) return st;
        c->pend_wander = -1;
        if (x.pend >= 0 && (st = launch_wander(c, x.pend))) return st;
        c->pend_wander = x.pend;
    }
    if (x.planes) {
        WanderParity wp{{-1, -1, -1, -1, -1, -1}};
        bool owes = false;
        for (int a = 0; a < c->gamma && c->gamma > 1; ++a) owes = (wp.p[a] = x.fowed[a]) >= 0 || owes;
        if (owes && (st = launch_wander_families(c, wp))) return st;
        if (c->ms != x.ms) std::swap(c->ms, c->ms_alt);
        if (c->md0 != x.md0) std::swap(c->md0, c->md0_alt);
        if (c->md1 != x.md1) std::swap(c->md1, c->md1_alt);
        std::copy_n(x.fcur, 6, c->fcur);
        if ((st = need_planes(c))) return st;
        std::copy_n(x.fowed, 6, c->fowed);
        c->home_ok = false;
        return MICSA_OK;
    }
    if (c->bit) {
        const size_t bytes = (size_t)word_lattices(c) * 2 * (size_t)c->g.Nh * 8;
        if ((st = rest_copy(c, c->bspin, c->bspin_alt, x.bspin, bytes))) return st;
        if ((st = rest_copy(c, c->bdm0, c->bdm0_alt, x.bdm0, bytes))) return st;
        return rest_copy(c, c->bdm1, c->bdm1_alt, x.bdm1, bytes);
    }
    const size_t bytes = (size_t)c->L * 2 * (size_t)c->g.Nh;
    if ((st = rest_copy(c, c->spin, c->spin_alt, x.spin, bytes))) return st;
    return rest_copy(c, c->dem, c->dem_alt, x.dem, bytes * (size_t)c->gamma);
}

bool takes_cells(const micsa_ctx* c, int32_t algo, int64_t n)
{
    return algo == MICSA_ALGO_MICSA     ? use_cells(c, n)
           : algo == MICSA_ALGO_WALKERS ? use_cells_walkers(c, n)
                                        : use_cells_canonical(c);
}

// Calls that the cell sweep takes but that the word-wise or per-half kernels do
// faster: of one or two sweeps on large lattices in bit planes (every launch
// loads and stores the planes of each lattice apart), and on rows of few sites
// (planes of mostly empty words).  Estimates in us, fitted to 50 shapes: a call on
// cells costs its plan and 3 us; the kernels on the words (per site of 64 lanes)
// and bytes as below.  One sweep, on cells / on its own arrays: bit planes 64 x
// 128^3 58 / 47, 64 x 104^3 31 / 27, 64 x 8 x 64 x 64 11.8 / 7.2; bytes, 8 of 8 x
// 400 x 400, MicSA 26 / 23, heat bath 45 / 30 (60 sweeps: 30.3 / 28.6).
// The state moves from the planes to those arrays, and back for the next long
// call: a short call stays where its state is until such calls have lost what the
// move costs, and on the planes as long as there is a tally to lose.
void choose_arrays(micsa_ctx* c, int32_t algo, int64_t n)
{
    if (!c->bit && (c->g.Kx > 12 || c->plan.sweeps == 0 || c->kernel_opt != MICSA_KERNEL_AUTO)) return;
    if (c->captured || c->no_room || !c->plan.ok || algo == MICSA_ALGO_WALKERS || !takes_cells(c, algo, kMscMinSweeps)) return;
    if (c->bit && !bp_one_launch(c) && c->tally_ok) return;  // (the per-half kernels keep no tally)
    const double sites = (double)c->L * 2.0 * (double)c->g.Nh;
    const CellPlan& pl = plan_for(c, n);
    // (the cost of a tiled plan has its launches in it)
    double cells = (pl.cost * (double)n + (pl.sweeps > 0 ? 0.0 : pl.load)) / 2.4e3 + 3.0, home, move;
    if (c->bit) {
        const double lanes = 64.0 * (double)word_lattices(c) * 2.0 * (double)c->g.Nh;
        home = (bp_one_launch(c) ? std::max(8.0, 4.0 + lanes / 2.4e6) : std::max(18.0, lanes / 3.6e6)) * (double)n;
        move = 20.0 + lanes / 2e6;
    } else if (algo == MICSA_ALGO_MICSA) {
        home = std::max(10.0, 3.0 + sites / 0.62e6) * (double)n;
        move = 20.0 + sites / 1e6;
    } else {
        const double words = (double)c->L * (double)cell_geom(c).plane, heat = algo == MICSA_ALGO_HEATBATH ? 1.0 : 0.85;
        const double simds = 4.0 * (c->cus > 0 ? c->cus : 256);
        const double draw = words * 2.0 / 64.0 * std::max(1100.0, 650.0 + 305.0 * c->g.Kx / 4) / simds;
        cells += (double)n * heat * (draw + words * 48.0 / 1750.0) / 2.4e3 + 3.0;
        home = std::max(12.0, 4.0 + sites / 0.40e6) * (double)n;
        move = 20.0 + sites / 1e6;
    }
    const bool on = c->planes_ok && !c->home_ok, off = c->home_ok && !c->planes_ok;
    if (home * 1.25 < cells) {
        c->off_cells = !on || (c->lag += cells - home) >= move;
        if (c->off_cells) c->lag = 0;
    } else if (off && c->bit && n < kMscMinSweeps && cells * 1.1 < home) {
        c->on_cells = (c->lag += home - cells) >= move;
        if (c->on_cells) c->lag = 0;
    } else {
        c->lag = 0;
    }
}

// Room for the planes of a call that takes the cell sweep.  Without it the call
// runs on the layout's own arrays, and so do those that follow until a schedule
// is installed (each would wait for an allocation to fail).
void find_room(micsa_ctx* c, int32_t algo, int64_t n)
{
    if (c->ms && c->cdr0 && (c->plan.sweeps == 0 || c->ms_alt)) return;  // there
    if (n <= 0 || !takes_cells(c, algo, n) || cells_alloc(c) == MICSA_OK) return;
    c->no_room = true;
    c->err.clear();
}

// A sweep call of this algorithm logs inside its launches (one work-group
// per lattice).
bool logs_in_kernel(micsa_ctx* c, int32_t algo, int64_t n)
{
    find_room(c, algo, n);
    if (c->plan.sweeps > 0) return false;
    if (algo == MICSA_ALGO_WALKERS) return c->gamma == 1 && use_cells_walkers(c, n);
    if (algo == MICSA_ALGO_MICSA) return c->gamma == 1 && use_cells(c, n);
    return c->gamma == 1 && use_cells_canonical(c);
}

int sweep_logging(micsa_ctx* c, int32_t algo, int64_t n, long long* dlog, int64_t stride)
{
    if (n <= 0) return MICSA_OK;
    if (int st = begin_sweeps(c)) return end_sweeps(c, st);
    return end_sweeps(c, algo == MICSA_ALGO_MICSA || algo == MICSA_ALGO_WALKERS
                             ? sweep_cells(c, n, dlog, stride, algo == MICSA_ALGO_WALKERS)
                             : sweep_cells_canonical(c, algo, n, dlog, stride));
}

int sweep_run(micsa_ctx* c, int32_t algo, int64_t n);

int sweep_impl(micsa_ctx* c, int32_t algo, int64_t n)
{
    if (!c) return MICSA_EINVAL;
    if (int st = check_sweep(c, algo, n)) return st;
    if (int st = begin_sweeps(c)) return end_sweeps(c, st);
    return end_sweeps(c, sweep_run(c, algo, n));
}

int sweep_run(micsa_ctx* c, int32_t algo, int64_t n)
{
    int st0 = check_sweep(c, algo, n);
    if (st0) return st0;
    if (n > 0) choose_arrays(c, algo, n);
    find_room(c, algo, n);
    // walkers (gamma = 1) on the fused sweep carry their wandering into the
    // next sweep's loads; every other path needs the daemons in place
    const bool walk_cells = algo == MICSA_ALGO_WALKERS && use_cells_walkers(c, n);
    const bool walk_msc = algo == MICSA_ALGO_WALKERS && !walk_cells && use_msc(c, n, algo);
    const bool walk_fused = algo == MICSA_ALGO_WALKERS && !walk_cells && !c->bit && c->gamma == 1 && use_fused(c);
    // the one-launch multispin sweep takes an owed wandering on its loads
    // (and leaves one), as the fused byte sweep does
    if (!walk_cells && !walk_fused && !walk_msc && !(algo == MICSA_ALGO_MICSA && !use_cells(c, n) && use_msc(c, n) && msc_one_launch(c)) &&
        (st0 = settle_wander(c)))
        return st0;
    if (walk_cells || (algo == MICSA_ALGO_MICSA && use_cells(c, n))) {
        if (n <= 0) return MICSA_OK;
        return c->gamma > 1 ? sweep_cells_families(c, n, walk_cells) : sweep_cells(c, n, nullptr, 0, walk_cells);
    }
    if (walk_msc) return n > 0 ? sweep_msc(c, n, true) : MICSA_OK;
    if (algo == MICSA_ALGO_MICSA && use_msc(c, n)) return n > 0 ? sweep_msc(c, n) : MICSA_OK;
    if ((algo == MICSA_ALGO_HEATBATH || algo == MICSA_ALGO_METROPOLIS) && use_cells_canonical(c))
        return n > 0 ? sweep_cells_canonical(c, algo, n, nullptr, 0) : MICSA_OK;
    // every other path sweeps the layout's own arrays
    if ((st0 = own_home(c))) return st0;
    if (algo != MICSA_ALGO_WALKERS) {
        if (use_graph(c) && n >= kGraphSweeps) return sweep_graph(c, algo, n);
    }
    if (algo == MICSA_ALGO_MICSA && bp_one_launch(c)) return sweep_bitplane(c, n);
    for (int64_t i = 0; i < n; ++i) {
        // sweep k is sweep fam of timestep t (Sec. 2.8)
        const int64_t k = c->k;
        const int64_t t = k / c->gamma;
        const int fam = (int)(k - t * c->gamma);
        const int64_t rho = refresh_index(t, c->sched.period);
        const double T = temperature(c->sched, rho);
        if (!(T > 0.0) || !std::isfinite(T)) return fail(c, MICSA_ERANGE, "no temperature for this refresh");
        int st;
        if (walk_fused && c->temporal == 2 && i + 1 < n && sweep2_walk_eligible(c)) {
            // timesteps t and t + 1 (gamma = 1) in one pass, wandering between them in registers
            const bool refreshB = is_refresh(t + 1, c->sched.period);
            const int64_t rhoB = refresh_index(t + 1, c->sched.period);
            const double TB = temperature(c->sched, rhoB);
            if (!(TB > 0.0) || !std::isfinite(TB)) return fail(c, MICSA_ERANGE, "no temperature for this refresh");
            if ((st = launch_fused_sweep2(c, is_refresh(t, c->sched.period), rho, T, refreshB, rhoB, TB, true,
                                          c->pend_wander, (int)(t & 1))))
                return st;
            c->pend_wander = (int32_t)((t + 1) & 1);
            c->k = k + 2;
            ++i;
            continue;
        }
        if (algo == MICSA_ALGO_MICSA && c->temporal == 2 && i + 1 < n && use_fused(c) && sweep2_eligible(c)) {
            // sweeps k and k + 1 in one pass (gamma = 1 on the fused path)
            const bool refreshB = is_refresh(k + 1, c->sched.period);
            const int64_t rhoB = refresh_index(k + 1, c->sched.period);
            const double TB = temperature(c->sched, rhoB);
            if (!(TB > 0.0) || !std::isfinite(TB)) return fail(c, MICSA_ERANGE, "no temperature for this refresh");
            if ((st = launch_fused_sweep2(c, is_refresh(k, c->sched.period), rho, T, refreshB, rhoB, TB))) return st;
            c->k = k + 2;
            ++i;
            continue;
        }
        if (algo == MICSA_ALGO_MICSA || algo == MICSA_ALGO_WALKERS) {
            const bool refresh = fam == 0 && is_refresh(t, c->sched.period);
            if (c->bit) {
                if ((st = launch_bitplane_sweep(c, refresh, rho, T))) return st;
            } else if (walk_fused) {
                // a refresh redraws every daemon, so an owed wandering lapses
                if ((st = launch_fused_sweep(c, refresh, rho, T, c->pend_wander))) return st;
                c->pend_wander = (int32_t)(t & 1);  // this timestep's wandering, owed to the next sweep
            } else if (use_fused(c)) {
                if ((st = launch_fused_sweep(c, refresh, rho, T))) return st;
            } else {
                if (refresh && (st = launch_refresh(c, rho, T))) return st;
                if ((st = launch_micsa_sweep(c, fam))) return st;
            }
            if (algo == MICSA_ALGO_WALKERS && !walk_fused && fam == c->gamma - 1 && (st = launch_wander(c, t)))
                return st;
        } else {
            if ((st = launch_canonical_sweep(c, algo, k, T))) return st;
        }
        c->k = k + 1;
    }
    return MICSA_OK;
}

void free_all(micsa_ctx* c)
{
    if (!c) return;
    if (c->draw_stream) (void)hipStreamSynchronize(c->draw_stream);
    if (c->draw_free) (void)hipEventDestroy(c->draw_free);
    if (c->draw_done) (void)hipEventDestroy(c->draw_done);
    if (c->draw_stream) drop_stream(c->store, c->device, c->draw_stream);
    for (auto& e : c->gexec)
        if (e) (void)hipGraphExecDestroy(e);
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    for (auto& v : c->events)
        for (auto& e : v) {
            (void)hipEventDestroy(e.first);
            (void)hipEventDestroy(e.second);
        }
    for (const JobStore::Block& b : c->owned) drop_block(c, b);
    if (c->pin) give_pin(c->device, c->pin);
}

// tally <- energies recomputed from the state, on the device.
int tally_from_state(micsa_ctx* c)
{
    if (int st = enqueue_energy(c, c->red)) return st;
    k_tally_from_bonds<<<(unsigned)c->L, kSlots, 0, c->stream>>>(c->red, n_sites(c), c->tally);
    return check_launch(c, "k_tally_from_bonds");
}

// Parameters a context accepts (include/micsa.h, micsa_create).
bool params_ok(const micsa_params* p)
{
    if (p->Lx < 8 || p->Lx % 8 || p->Ly < 2 || p->Ly % 2 || p->Lz < 2 || p->Lz % 2) return false;
    if (p->n_samples < 1 || p->n_samples >= (1 << 24) || p->n_replicas < 1) return false;
    if (p->layout != MICSA_LAYOUT_BYTE && p->layout != MICSA_LAYOUT_BITPLANE) return false;
    const int64_t N = (int64_t)p->Lx * p->Ly * p->Lz;
    if (N >= ((int64_t)1 << 32) || (int64_t)p->n_samples * p->n_replicas >= (1 << 16)) return false;
    const int gamma = p->gamma == 0 ? 1 : p->gamma;
    if (gamma < 1 || gamma > 6 || (gamma > 1 && p->layout != MICSA_LAYOUT_BYTE)) return false;
    if (p->lane_mode != MICSA_LANES_SAMPLES && p->lane_mode != MICSA_LANES_REPLICAS) return false;
    if (p->lane_mode == MICSA_LANES_REPLICAS && p->layout != MICSA_LAYOUT_BITPLANE) return false;
    return (int64_t)gamma * N / 4 < ((int64_t)1 << 32);  // daemon counters (a*N + i) >> 2 fit 32 bits
}

}  // namespace

// =================================================================== C ABI
extern "C" {

const char* micsa_status_string(int status)
{
    switch (status) {
    case MICSA_OK: return "ok";
    case MICSA_EINVAL: return "invalid argument";
    case MICSA_ENOMEM: return "out of device memory";
    case MICSA_EHIP: return "HIP runtime error";
    case MICSA_ESTATE: return "invalid state";
    case MICSA_ERANGE: return "out of range";
    default: return "unknown status";
    }
}

const char* micsa_last_error(const micsa_ctx* ctx) { return ctx ? ctx->err.c_str() : "null context"; }

// Parameters, geometry and launch plans (no device memory); the plans are those
// of `like` if that is a context of the same parameters and device.
static int setup_ctx(micsa_ctx* c, const micsa_params* p, hipStream_t stream, const micsa_ctx* like = nullptr)
{
    const int64_t N = (int64_t)p->Lx * p->Ly * p->Lz;
    const int gamma = p->gamma == 0 ? 1 : p->gamma;
    int st = MICSA_OK;
    if (hipGetDevice(&c->device) != hipSuccess) {
        (void)hipGetLastError();
        c->device = 0;
        st = MICSA_EHIP;
    }
    if (st || hipDeviceGetAttribute(&c->cus, hipDeviceAttributeMultiprocessorCount, c->device) != hipSuccess) {
        (void)hipGetLastError();
        c->cus = 0;
    }
    c->p = *p;
    c->p.gamma = gamma;
    c->gamma = gamma;
    c->stream = stream;
    c->L = p->n_samples * p->n_replicas;
    c->bit = p->layout == MICSA_LAYOUT_BITPLANE;
    // the bit-plane sweep is latency-bound: a draw beside it slows it more
    // than the draw costs in place (measured on MI355X), so it draws in place
    if (c->bit) c->draw_ahead = 0;
    c->G = p->lane_mode == MICSA_LANES_REPLICAS ? (p->n_replicas + 63) / 64 : (p->n_samples + 63) / 64;
    Geom& g = c->g;
    g.Lx = p->Lx;
    g.Ly = p->Ly;
    g.Lz = p->Lz;
    g.Kx = p->Lx / 2;
    g.Wr = g.Kx / 4;
    g.rows = p->Ly * p->Lz;
    g.Nh = N / 2;
    g.S = p->n_samples;
    g.R = p->n_replicas;
    g.key0 = (uint32_t)p->seed;
    g.key1 = (uint32_t)(p->seed >> 32);
    g.gamma = gamma;

    const bool same = like && like->device == c->device && like->cus == c->cus;
    if (same) {
        c->plan = like->plan;
        c->walk = like->walk;
        std::copy(std::begin(like->brief), std::end(like->brief), c->brief);
    } else {
        const CellPlans plans = cell_plans(c);
        c->plan = plans.main;
        c->walk = plans.walk;
        std::copy(std::begin(plans.brief), std::end(plans.brief), c->brief);
    }
    c->tile2 = same ? like->tile2 : msc2_plan(c);
    return st;
}

// Device memory that a context takes when it is created: the state's own arrays
// with the reductions' slots, and the working buffers of the sweep path that the
// lattice takes by default.
struct CtxBytes {
    bool alt, cells, msc;  // the fused sweeps' second copies; which planes
    size_t state, dstate, words, bonds, nred;
    size_t home, work;
};

static CtxBytes ctx_bytes(const micsa_ctx* c)
{
    CtxBytes b{};
    const Geom& g = c->g;
    b.nred = (size_t)std::max(c->L, c->p.n_samples);
    b.state = (size_t)c->L * 2 * (size_t)g.Nh;
    b.dstate = b.state * (size_t)c->gamma;  // every daemon family
    b.words = (size_t)word_lattices(c) * 2 * (size_t)g.Nh;
    b.bonds = c->bit ? (size_t)bp_coupling_sets(geomb(c)) * 6 * (size_t)g.Nh * 8 : 0;
    // the fused sweeps go from one copy to the other
    b.alt = !c->bit && fused_eligible(c) && c->p.Lx >= 128;
    b.cells = use_cells(c);
    b.msc = !b.cells && !c->bit && c->gamma == 1 && msc_eligible(c);
    b.home = arena_size((size_t)c->L * kSlots * 8) + arena_size(b.nred * kSlots * 8) +
             (c->bit ? 3 * arena_size(b.words * 8) + arena_size(b.bonds)
                     : (b.alt ? 2 : 1) * (arena_size(b.state) + arena_size(b.dstate)));
    if (b.msc || (b.cells && msc_eligible(c))) {
        const size_t mw = (size_t)c->L * 2 * (size_t)msc_geom(c).plane * 8;
        b.work = (b.msc ? 8 : 6) * arena_size(mw) + arena_size(3 * mw);
    } else if (b.cells) {
        b.work = arena_size(cells_plane_words(c) * 4);
    }
    if (b.cells)
        b.work += arena_size((size_t)c->L * 2 * (size_t)cell_geom(c).plane * 8 * (size_t)cells_draw_cap(c));
    return b;
}

// most: size of its block at most (0: what it needs); spare: whether it may do
// without the working buffers for now.
static int create_ctx(const micsa_params* p, hipStream_t stream, const micsa_ctx* like, size_t most, bool spare,
                      JobStore* store, micsa_ctx** out)
{
    if (!out) return MICSA_EINVAL;
    *out = nullptr;
    if (!p) return MICSA_EINVAL;
    if (!params_ok(p)) return MICSA_EINVAL;
    const int gamma = p->gamma == 0 ? 1 : p->gamma;

    micsa_ctx* c = new (std::nothrow) micsa_ctx();
    if (!c) return MICSA_ENOMEM;
    if (const int st = setup_ctx(c, p, stream, like)) {
        delete c;
        return st;
    }
    c->draw_room = like ? like->draw_room : 0;
    c->store = store;
    if (stream_captured(stream)) {  // the initial state is no part of a graph
        delete c;
        return MICSA_EHIP;
    }
    const Geom& g = c->g;

    const CtxBytes B = ctx_bytes(c);
    const auto [alt, cells, msc, state, dstate, words, bonds, nred, home, work] = B;
    // One allocation for all of it: nine took 90 us of the 230 us that a 16^3
    // context took to set up.  Working buffers that do not fit now are tried
    // again by the first sweep call.
    c->arena = static_cast<uint8_t*>(own_block(c, home + work, most));
    c->arena_left = home + work;
    if (!c->arena && spare) {
        c->arena = static_cast<uint8_t*>(own_block(c, home));
        c->arena_left = home;
    }
    bool ok = c->arena && ctx_alloc(c, c->tally, (size_t)c->L * kSlots * 8) &&
              ctx_alloc(c, c->red, nred * kSlots * 8);
    if (ok && !c->bit) {
        ok = ctx_alloc(c, c->spin, state) && ctx_alloc(c, c->dem, dstate);
        if (ok && alt) ok = need_alt(c) == MICSA_OK;
    } else if (ok) {
        ok = ctx_alloc(c, c->bspin, words * 8) && ctx_alloc(c, c->bdm0, words * 8) &&
             ctx_alloc(c, c->bdm1, words * 8) && ctx_alloc(c, c->bJ, bonds);
    }
    if (!ok) {
        (void)hipGetLastError();
        free_all(c);
        delete c;
        return MICSA_ENOMEM;
    }
    int st = MICSA_OK;
    if (!c->bit) {
        // spins first, then the bond bits into the even spin bytes
        k_init_spins<<<grid_for(g.Nh / 4, c->L), kBlock, 0, c->stream>>>(g, c->spin);
        st = check_launch(c, "k_init_spins");
        if (!st) st = enqueue_bonds(c);
        if (!st && hipMemsetAsync(c->dem, 0, dstate, c->stream) != hipSuccess) st = MICSA_EHIP;
    } else {
        const int WL = word_lattices(c);
        kb_init_couplings<<<dim3((unsigned)((g.Nh + 3) / 4), (unsigned)bp_coupling_sets(geomb(c))), 256, 0,
                            c->stream>>>(geomb(c), c->bJ);
        st = check_launch(c, "kb_init_couplings");
        if (!st) {
            kb_init_spins<<<dim3((unsigned)((g.Nh / 2 + 3) / 4), (unsigned)WL), 256, 0, c->stream>>>(geomb(c),
                                                                                               c->bspin);
            st = check_launch(c, "kb_init_spins");
        }
        if (!st && (hipMemsetAsync(c->bdm0, 0, words * 8, c->stream) != hipSuccess ||
                    hipMemsetAsync(c->bdm1, 0, words * 8, c->stream) != hipSuccess))
            st = MICSA_EHIP;
    }
    if (!st) st = tally_from_state(c);
    if (st) {
        free_all(c);
        delete c;
        return st;
    }
    if (cells) {
        if (cells_alloc(c) != MICSA_OK) c->err.clear();
    } else if (msc) {
        if (msc_alloc(c, true, true) != MICSA_OK) c->err.clear();
    }
    *out = c;
    return MICSA_OK;
}

int micsa_create(const micsa_params* p, void* hip_stream, micsa_ctx** out) 
{
    return create_ctx(p, (hipStream_t)hip_stream, nullptr, 0, true, nullptr, out);
}


int micsa_destroy(micsa_ctx* ctx)
{
    if (!ctx) return MICSA_OK;
    (void)hipStreamSynchronize(ctx->stream);
    free_all(ctx);
    delete ctx;
    return MICSA_OK;
}

int micsa_set_schedule(micsa_ctx* ctx, const micsa_schedule* s)
{
    if (!ctx) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (!s) return fail(ctx, MICSA_EINVAL, "null schedule");
    if (s->refresh_period < 0) return fail(ctx, MICSA_EINVAL, "refresh_period < 0");
    if (s->n_sweeps < 0) return fail(ctx, MICSA_EINVAL, "n_sweeps < 0");
    Schedule n;
    n.set = true;
    n.kind = s->kind;
    n.period = s->refresh_period;
    n.T0 = s->T0;
    n.T1 = s->T1;
    n.n_sweeps = s->n_sweeps;
    n.n_steps = (s->n_sweeps + ctx->gamma - 1) / ctx->gamma;
    auto okT = [](double T) { return T > 0.0 && std::isfinite(T); };
    if (s->kind == MICSA_SCHED_CONST) {
        if (!okT(s->T0)) return fail(ctx, MICSA_EINVAL, "T0 must be positive and finite");
    } else if (s->kind == MICSA_SCHED_LINEAR) {
        if (!okT(s->T0) || !okT(s->T1)) return fail(ctx, MICSA_EINVAL, "T0, T1 must be positive and finite");
    } else if (s->kind == MICSA_SCHED_TABLE) {
        if (!s->T_table || s->T_len < refresh_count(n))
            return fail(ctx, MICSA_EINVAL, "T_table must cover every refresh of the schedule");
        n.table.assign(s->T_table, s->T_table + s->T_len);
        for (double T : n.table)
            if (!okT(T)) return fail(ctx, MICSA_EINVAL, "table temperatures must be positive and finite");
    } else {
        return fail(ctx, MICSA_EINVAL, "unknown schedule kind");
    }
    // threshold tables for every refresh of the schedule (read by the draws)
    const int64_t nrho = std::max<int64_t>(refresh_count(n), 1);
    const size_t o_h = (size_t)nrho * sizeof(DaemonThresholds), o_m = o_h + (size_t)nrho * sizeof(HeatBathThresholds);
    std::vector<uint8_t> tab(o_m + (size_t)nrho * sizeof(MetropolisThresholds));
    static_assert(sizeof(DaemonThresholds) % 8 == 0 && sizeof(HeatBathThresholds) % 8 == 0, "tables of 64-bit words");
    auto* dth = reinterpret_cast<DaemonThresholds*>(tab.data());
    auto* hth = reinterpret_cast<HeatBathThresholds*>(tab.data() + o_h);
    auto* mth = reinterpret_cast<MetropolisThresholds*>(tab.data() + o_m);
    for (int64_t rho = 0; rho < nrho; ++rho) {
        const double T = temperature(n, rho);
        dth[rho] = daemon_thresholds(T);
        hth[rho] = heatbath_thresholds(T);
        mth[rho] = metropolis_thresholds(T);
    }
    uint8_t* d = nullptr;
    if (!ctx_alloc(ctx, d, tab.size())) return fail(ctx, MICSA_ENOMEM, "schedule tables");
    if (ctx->d_dth) HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));  // the tables in use go
    if (hipMemcpyAsync(d, tab.data(), tab.size(), hipMemcpyHostToDevice, ctx->stream) != hipSuccess) {
        ctx_free(ctx, d);
        return fail(ctx, MICSA_EHIP, "schedule tables");
    }
    if (ctx->d_dth) ctx_free(ctx, ctx->d_dth);
    ctx->h_tables = std::move(tab);
    for (auto& e : ctx->gexec)  // captured graphs point at the old tables
        if (e) {
            (void)hipGraphExecDestroy(e);
            e = nullptr;
        }
    ctx->d_dth = reinterpret_cast<DaemonThresholds*>(d);
    ctx->d_hth = reinterpret_cast<HeatBathThresholds*>(d + o_h);
    ctx->d_mth = reinterpret_cast<MetropolisThresholds*>(d + o_m);
    ctx->sched = std::move(n);
    ctx->no_room = false;
    ctx->cdr_n = 0;  // levels drawn ahead under the old temperatures
    ctx->msc_drawn = -1;
    return MICSA_OK;
}

int micsa_sweep(micsa_ctx* ctx, int32_t algo, int64_t n) { return sweep_impl(ctx, algo, n); }

static int sweep_logged_d(micsa_ctx* ctx, int32_t algo, int64_t n, int64_t stride, int64_t* E_log, int64_t* D_log)
{
    const int64_t rows = n / stride;
    const int L = ctx->L;
    const int64_t N = n_sites(ctx);
    int st;
    if (logs_in_kernel(ctx, algo, n) && log_room(ctx, rows)) {
        const size_t need = (size_t)rows * L * 2;
        if (need > ctx->rlog_cap) {
            // (by a factor of two where the old one stays)
            const size_t cap = ctx->captured ? std::max(need, 2 * ctx->rlog_cap) : need;
            ctx_retire(ctx, ctx->rlog);  // enqueued work may still use it
            ctx->rlog_cap = 0;
            if (!ctx_alloc(ctx, ctx->rlog, cap * 8)) return fail(ctx, MICSA_ENOMEM, "log buffer");
            ctx->rlog_cap = cap;
        }
        if ((algo != MICSA_ALGO_WALKERS && (st = settle_wander(ctx))) ||
            (st = sweep_logging(ctx, algo, n, ctx->rlog, stride)))
            return st;
        const int64_t e = rows * L;
        k_log_from_pairs<<<(unsigned)((e + 255) / 256), 256, 0, ctx->stream>>>(
            ctx->rlog, e, N, reinterpret_cast<long long*>(E_log), reinterpret_cast<long long*>(D_log));
        return check_launch(ctx, "k_log_from_pairs");
    }
    if (!ctx->logslots && !ctx_alloc(ctx, ctx->logslots, (size_t)2 * L * kSlots * 8))
        return fail(ctx, MICSA_ENOMEM, "log slots");
    unsigned long long* U = ctx->logslots;
    unsigned long long* Ms = ctx->logslots + (size_t)L * kSlots;
    for (int64_t r = 0; r < rows; ++r) {
        if ((st = sweep_impl(ctx, algo, stride))) return st;
        if (E_log && (st = enqueue_energy(ctx, U))) return st;
        if (D_log && (st = enqueue_level_sum(ctx, Ms))) return st;
        k_log_from_slots<<<(unsigned)((L + 255) / 256), 256, 0, ctx->stream>>>(
            U, Ms, L, N, E_log ? reinterpret_cast<long long*>(E_log + r * L) : nullptr,
            D_log ? reinterpret_cast<long long*>(D_log + r * L) : nullptr);
        if ((st = check_launch(ctx, "k_log_from_slots"))) return st;
    }
    return n > rows * stride ? sweep_impl(ctx, algo, n - rows * stride) : MICSA_OK;
}

int micsa_sweep_logged_d(micsa_ctx* ctx, int32_t algo, int64_t n, int64_t stride, int64_t* E_log,
                         int64_t* D_log)
{
    if (!ctx) return MICSA_EINVAL;
    if (stride < 1) return fail(ctx, MICSA_EINVAL, "stride must be >= 1");
    if (!ctx->sched.set) return fail(ctx, MICSA_ESTATE, "no schedule installed");
    if (n < 0 || ctx->k + n > ctx->sched.n_sweeps) return fail(ctx, MICSA_ERANGE, "sweeps beyond the schedule");
    if (int st = check_sweep(ctx, algo, n)) return st;
    if (n / stride == 0 || (!E_log && !D_log)) return sweep_impl(ctx, algo, n);
    // (the buffers of the logs belong to the call: see begin_sweeps)
    const int st = begin_sweeps(ctx);
    return end_sweeps(ctx, st ? st : sweep_logged_d(ctx, algo, n, stride, E_log, D_log));
}

int micsa_sweep_logged(micsa_ctx* ctx, int32_t algo, int64_t n, int64_t stride, int64_t* E_log, int64_t* D_log)
{
    if (!ctx) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (stride < 1) return fail(ctx, MICSA_EINVAL, "stride must be >= 1");
    if (!ctx->sched.set) return fail(ctx, MICSA_ESTATE, "no schedule installed");
    if (n < 0 || ctx->k + n > ctx->sched.n_sweeps) return fail(ctx, MICSA_ERANGE, "sweeps beyond the schedule");
    run_stream(ctx);
    const int64_t rows = n / stride;
    const int L = ctx->L;
    int st0 = check_sweep(ctx, algo, n);
    if (st0) return st0;
    if (logs_in_kernel(ctx, algo, n) && log_room(ctx, rows)) {
        if (algo != MICSA_ALGO_WALKERS && (st0 = settle_wander(ctx))) return st0;
        long long* rlog = nullptr;
        if (rows > 0 && !(rlog = static_cast<long long*>(work_take(ctx, (size_t)rows * L * 2 * 8))))
            return fail(ctx, MICSA_ENOMEM, "log buffer");
        int st = sweep_logging(ctx, algo, n, rows > 0 ? rlog : nullptr, stride);
        std::vector<int64_t> h((size_t)rows * L * 2);
        if (!st && rows > 0) st = read_device(ctx, rlog, h.data(), h.size() * 8);
        work_give(ctx, rlog);
        if (st) return st;
        const int64_t N = n_sites(ctx);
        for (int64_t r = 0; r < rows; ++r)
            for (int l = 0; l < L; ++l) {
                if (E_log) E_log[r * L + l] = 2 * h[(size_t)((r * L + l) * 2)] - 3 * N;
                if (D_log) D_log[r * L + l] = 4 * h[(size_t)((r * L + l) * 2 + 1)];
            }
        return MICSA_OK;
    }
    unsigned long long* dlog = nullptr;
    const size_t row_len = (size_t)L * 2 * kSlots;
    if (rows > 0 && !(dlog = static_cast<unsigned long long*>(work_take(ctx, (size_t)rows * row_len * 8))))
        return fail(ctx, MICSA_ENOMEM, "log buffer");
    int st = MICSA_OK;
    int64_t done = 0;
    for (int64_t r = 0; r < rows && !st; ++r) {
        st = sweep_impl(ctx, algo, stride);
        done += stride;
        if (!st) st = enqueue_energy(ctx, dlog + (size_t)r * row_len);
        if (!st) st = enqueue_level_sum(ctx, dlog + (size_t)r * row_len + (size_t)L * kSlots);
    }
    if (!st && n > done) st = sweep_impl(ctx, algo, n - done);
    std::vector<int64_t> h;
    if (!st && rows > 0) st = read_slots(ctx, dlog, rows * L * 2, h);
    if (!st && hipStreamSynchronize(ctx->stream) != hipSuccess) st = fail(ctx, MICSA_EHIP, "sync");
    work_give(ctx, dlog);
    if (st) return st;
    const int64_t N = n_sites(ctx);
    for (int64_t r = 0; r < rows; ++r)
        for (int l = 0; l < L; ++l) {
            if (E_log) E_log[r * L + l] = 2 * h[(size_t)(r * L * 2 + l)] - 3 * N;
            if (D_log) D_log[r * L + l] = 4 * h[(size_t)(r * L * 2 + L + l)];
        }
    return MICSA_OK;
}

int micsa_sync(micsa_ctx* ctx)
{
    if (!ctx) return MICSA_EINVAL;
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    return MICSA_OK;
}

static int read_red(micsa_ctx* c, int64_t n, std::vector<int64_t>& out) { return read_slots(c, c->red, n, out); }

int micsa_read_energy(micsa_ctx* ctx, int64_t* E)
{
    if (!ctx || !E) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    int st = enqueue_energy(ctx, ctx->red);
    std::vector<int64_t> U;
    if (st || (st = read_red(ctx, ctx->L, U))) return st;
    const int64_t N = n_sites(ctx);
    for (int l = 0; l < ctx->L; ++l) E[l] = 2 * U[(size_t)l] - 3 * N;
    return MICSA_OK;
}

int micsa_read_energy_tally(micsa_ctx* ctx, int64_t* E)
{
    if (!ctx || !E) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (ctx->bit && !ctx->tally_ok)
        return fail(ctx, MICSA_ESTATE, "the bit-plane tally is kept by the one-launch sweep only (a per-half "
                                       "sweep ran since the spins were last set)");
    std::vector<int64_t> v;
    int st = read_slots(ctx, ctx->tally, ctx->L, v);
    if (st) return st;
    for (int l = 0; l < ctx->L; ++l) E[l] = v[(size_t)l];
    return MICSA_OK;
}

int micsa_read_demon_energy(micsa_ctx* ctx, int64_t* D)
{
    if (!ctx || !D) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    int st = enqueue_level_sum(ctx, ctx->red);
    std::vector<int64_t> v;
    if (st || (st = read_red(ctx, ctx->L, v))) return st;
    for (int l = 0; l < ctx->L; ++l) D[l] = 4 * v[(size_t)l];
    return MICSA_OK;
}

// D[s][mu][r] = #{(pair, x) : w_x != w_{x + r e_mu}} summed over the replica
// pairs of sample s (observables.hpp), for r = 0 .. rmax.
static int c4_counts(micsa_ctx* c, const C4Geom& cg, std::vector<int64_t>& D)
{
    const int64_t ent = (int64_t)c->p.n_samples * 3 * (cg.rmax + 1);
    const int64_t per_pair = (int64_t)2 * c->g.rows * cg.E;
    const int64_t total = (int64_t)c->p.n_samples * cg.npair;
    const int64_t budget_words = ((int64_t)256 << 20) / 4;  // at most 256 MiB of packed pairs at a time
    const int64_t chunk = std::max<int64_t>(1, std::min<int64_t>({total, budget_words / per_pair, 65535}));
    uint8_t* const buf = static_cast<uint8_t*>(work_take(c, (size_t)ent * kSlots * 8 + (size_t)(chunk * per_pair) * 4));
    if (!buf) return fail(c, MICSA_ENOMEM, "correlation buffers");
    unsigned long long* dD = reinterpret_cast<unsigned long long*>(buf);
    uint32_t* Q = reinterpret_cast<uint32_t*>(buf + (size_t)ent * kSlots * 8);
    int st = zero_slots(c, dD, ent);
    const int64_t valid = (int64_t)2 * c->g.rows * cg.Wv;
    for (int64_t sp0 = 0; sp0 < total && !st; sp0 += chunk) {
        const unsigned n = (unsigned)std::min(chunk, total - sp0);
        {
            TimedLaunch t(c, kTimeReduce);
            if (c->bit)
                k_pack_overlap<true><<<dim3((unsigned)((per_pair + 255) / 256), n), 256, 0, c->stream>>>(
                    geomb(c), cg, (int)sp0, nullptr, c->bspin, Q);
            else
                k_pack_overlap<false><<<dim3((unsigned)((per_pair + 255) / 256), n), 256, 0, c->stream>>>(
                    geomb(c), cg, (int)sp0, c->spin, nullptr, Q);
        }
        if ((st = check_launch(c, "k_pack_overlap"))) break;
        {
            TimedLaunch t(c, kTimeReduce);
            k_c4_count<<<dim3((unsigned)((valid + 255) / 256), (unsigned)(3 * (cg.rmax + 1)), n), 256, 0,
                         c->stream>>>(c->g, cg, (int)sp0, Q, dD);
        }
        st = check_launch(c, "k_c4_count");
    }
    if (!st) st = read_slots(c, dD, ent, D);
    work_give(c, buf);
    return st;
}

static C4Geom c4_geom(const micsa_ctx* c)
{
    C4Geom cg;
    cg.E = (c->g.Kx + 63) / 32;
    cg.Wv = (c->g.Kx + 31) / 32;
    cg.rmax = std::max({c->p.Lx, c->p.Ly, c->p.Lz}) / 2;
    cg.npair = c->p.n_replicas * (c->p.n_replicas - 1) / 2;
    return cg;
}

int micsa_read_c4(micsa_ctx* ctx, int64_t* G)
{
    if (!ctx || !G) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = need_home(ctx)) return st_;
    if (ctx->p.n_replicas < 2) return fail(ctx, MICSA_EINVAL, "C4 needs at least two replicas");
    const C4Geom cg = c4_geom(ctx);
    std::vector<int64_t> D;
    const int st = c4_counts(ctx, cg, D);
    if (st) return st;
    const int64_t N = n_sites(ctx);
    const int side[3] = {ctx->p.Lx, ctx->p.Ly, ctx->p.Lz};
    for (int s = 0; s < ctx->p.n_samples; ++s)
        for (int mu = 0; mu < 3; ++mu)
            for (int r = 0; r <= cg.rmax; ++r) {
                const int64_t e = ((int64_t)s * 3 + mu) * (cg.rmax + 1) + r;
                G[e] = 2 * r <= side[mu] ? N * cg.npair - 2 * D[(size_t)e] : 0;
            }
    return MICSA_OK;
}

// ------------------------------------------- C4 into a static scratch array
// The overlap rows and the count slots of micsa_read_c4 live in `scratch`, a
// file-scope device array (one copy per device, held until the process
// ends), so this call allocates nothing.  Host code never passes the
// array's name to a kernel or a copy: it uses the device address that
// hipGetSymbolAddress returns for the device the context lives on.
constexpr size_t kC4ScratchBytes = (size_t)32 << 20;
static __device__ __align__(256) uint8_t scratch[kC4ScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
uint8_t* g_scratch_addr[kMaxDevices] = {};

// Device address of `scratch` on the context's device (looked up once per
// device, with that device current).
int scratch_address(micsa_ctx* c, uint8_t** out)
{
    if (c->device < 0 || c->device >= kMaxDevices) return fail(c, MICSA_EINVAL, "device index beyond the scratch table");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_addr[c->device]) {
        int prev = 0;
        HIP_TRY(c, hipGetDevice(&prev));
        if (prev != c->device) HIP_TRY(c, hipSetDevice(c->device));
        void* ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (prev != c->device) (void)hipSetDevice(prev);
        if (e != hipSuccess || !ptr)
            return fail(c, MICSA_EHIP, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_addr[c->device] = static_cast<uint8_t*>(ptr);
    }
    *out = g_scratch_addr[c->device];
    return MICSA_OK;
}

size_t align256(size_t n) { return (n + 255) & ~(size_t)255; }
}  // namespace

int micsa_read_c4_static(micsa_ctx* ctx, int64_t* G)
{
    if (!ctx || !G) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = need_home(ctx)) return st_;
    if (ctx->p.n_replicas < 2) return fail(ctx, MICSA_EINVAL, "C4 needs at least two replicas");
    const C4Geom cg = c4_geom(ctx);
    const int64_t ent = (int64_t)ctx->p.n_samples * 3 * (cg.rmax + 1);
    const int64_t per_pair = (int64_t)2 * ctx->g.rows * cg.E;  // 32-bit words of one pair's rows
    const int64_t total = (int64_t)ctx->p.n_samples * cg.npair;
    const size_t slots_bytes = align256((size_t)ent * kSlots * 8), sums_bytes = align256((size_t)ent * 8);
    const size_t head = slots_bytes + sums_bytes;
    if (head + (size_t)per_pair * 4 > kC4ScratchBytes)
        return fail(ctx, MICSA_ERANGE, "lattice too large for the 32 MiB static scratch (use micsa_read_c4)");
    uint8_t* base = nullptr;
    int st = scratch_address(ctx, &base);
    if (st) return st;
    auto* dD = reinterpret_cast<unsigned long long*>(base);
    auto* sums = reinterpret_cast<long long*>(base + slots_bytes);
    auto* Q = reinterpret_cast<uint32_t*>(base + head);
    const int64_t chunk =
        std::max<int64_t>(1, std::min<int64_t>({total, (int64_t)((kC4ScratchBytes - head) / 4) / per_pair, 65535}));
    // the array keeps the previous call's contents: clear the count slots
    k_fill_i64<<<grid_for(ent * kSlots, 1), kBlock, 0, ctx->stream>>>(dD, ent * kSlots, 0ull);
    if ((st = check_launch(ctx, "k_fill_i64"))) return st;
    const int64_t valid = (int64_t)2 * ctx->g.rows * cg.Wv;
    for (int64_t sp0 = 0; sp0 < total; sp0 += chunk) {
        const unsigned n = (unsigned)std::min(chunk, total - sp0);
        if (ctx->bit)
            k_pack_overlap<true><<<dim3((unsigned)((per_pair + 255) / 256), n), 256, 0, ctx->stream>>>(
                geomb(ctx), cg, (int)sp0, nullptr, ctx->bspin, Q);
        else
            k_pack_overlap<false><<<dim3((unsigned)((per_pair + 255) / 256), n), 256, 0, ctx->stream>>>(
                geomb(ctx), cg, (int)sp0, ctx->spin, nullptr, Q);
        if ((st = check_launch(ctx, "k_pack_overlap"))) return st;
        k_c4_count<<<dim3((unsigned)((valid + 255) / 256), (unsigned)(3 * (cg.rmax + 1)), n), 256, 0,
                     ctx->stream>>>(ctx->g, cg, (int)sp0, Q, dD);
        if ((st = check_launch(ctx, "k_c4_count"))) return st;
    }
    k_sum_slots<<<(unsigned)((ent + 15) / 16), 1024, 0, ctx->stream>>>(dD, ent, sums, nullptr, 0u);
    if ((st = check_launch(ctx, "k_sum_slots"))) return st;
    HIP_TRY(ctx, hipMemcpyAsync(G, sums, (size_t)ent * 8, hipMemcpyDeviceToHost, ctx->stream));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    const int64_t N = n_sites(ctx);
    const int side[3] = {ctx->p.Lx, ctx->p.Ly, ctx->p.Lz};
    for (int s = 0; s < ctx->p.n_samples; ++s)
        for (int mu = 0; mu < 3; ++mu)
            for (int r = 0; r <= cg.rmax; ++r) {
                const int64_t e = ((int64_t)s * 3 + mu) * (cg.rmax + 1) + r;
                G[e] = 2 * r <= side[mu] ? N * cg.npair - 2 * G[e] : 0;
            }
    return MICSA_OK;
}

int micsa_read_xi(micsa_ctx* ctx, double* xi12, double* xi23)
{
    if (!ctx || !xi12 || !xi23) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = need_home(ctx)) return st_;
    if (ctx->p.n_replicas < 2) return fail(ctx, MICSA_EINVAL, "xi needs at least two replicas");
    const C4Geom cg = c4_geom(ctx);
    std::vector<int64_t> G((size_t)ctx->p.n_samples * 3 * (cg.rmax + 1));
    int st = micsa_read_c4(ctx, G.data());
    if (st) return st;
    const int64_t N = n_sites(ctx);
    const int rmin = std::min({ctx->p.Lx, ctx->p.Ly, ctx->p.Lz}) / 2;
    for (int s = 0; s < ctx->p.n_samples; ++s) {
        // C4(r): mean over the three axes, normalised so that C4(0) = 1;
        // I_n = sum_{r = 0}^{rmin} r^n C4(r); xi12 = I2/I1, xi23 = I3/I2
        double I[4] = {0, 0, 0, 0};
        for (int r = 0; r <= rmin; ++r) {
            int64_t sum = 0;
            for (int mu = 0; mu < 3; ++mu) sum += G[(size_t)(((int64_t)s * 3 + mu) * (cg.rmax + 1) + r)];
            const double c4 = (double)sum / (3.0 * (double)N * (double)cg.npair);
            double pw = 1.0;
            for (int n = 0; n < 4; ++n) {
                I[n] += pw * c4;
                pw *= (double)r;
            }
        }
        if (!(I[1] > 0.0) || !(I[2] > 0.0)) {
            xi12[s] = xi23[s] = NAN;
        } else {
            xi12[s] = I[2] / I[1];
            xi23[s] = I[3] / I[2];
        }
    }
    return MICSA_OK;
}

int micsa_read_overlap(micsa_ctx* ctx, int32_t a, int32_t b, int64_t* Q)
{
    if (!ctx || !Q) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (a < 0 || b < 0 || a >= ctx->p.n_replicas || b >= ctx->p.n_replicas || a == b)
        return fail(ctx, MICSA_EINVAL, "replica indices out of range or equal");
    const int S = ctx->p.n_samples;
    int st;
    if (ctx->planes_ok) {
        if ((st = enqueue_cells_count<2>(ctx, S, a, b, ctx->red))) return st;
    } else if (ctx->bit) {
        if ((st = enqueue_lane_count<2>(ctx, ctx->red, a, b))) return st;
    } else {
        if ((st = zero_slots(ctx, ctx->red, S))) return st;
        const int64_t wpl = 2 * ctx->g.Nh / 4;
        {
            TimedLaunch t(ctx, kTimeReduce);
            k_differ_count<<<grid_for(wpl, S), kBlock, 0, ctx->stream>>>(
                wpl, ctx->p.n_replicas, a, b, reinterpret_cast<const uint32_t*>(ctx->spin), ctx->red);
        }
        if ((st = check_launch(ctx, "k_differ_count"))) return st;
    }
    std::vector<int64_t> v;
    if ((st = read_red(ctx, S, v))) return st;
    const int64_t N = n_sites(ctx);
    for (int s = 0; s < S; ++s) Q[s] = N - 2 * v[(size_t)s];
    return MICSA_OK;
}

// Byte-layout arrays of `count` parity-split lattices ([count][2][Nh]: the
// spins, or the daemons with count = L * gamma) -> host [count][N].
static int read_state(micsa_ctx* ctx, const uint8_t* dev, uint8_t* host, int64_t count, uint8_t mask = 0xFF)
{
    // in natural order by the device: small states to pinned memory, larger
    // ones by way of a buffer of at most 32 MiB
    const int64_t words = count * n_sites(ctx) / 8;
    const auto launch = [&](int64_t w0, int64_t n, void* dst, unsigned blocks, uint32_t* ticket, uint32_t value) {
        k_natural<<<blocks, 1024, 0, ctx->stream>>>(ctx->g, dev, w0, n, 0x01010101u * mask, static_cast<uint2*>(dst),
                                                   ticket, value);
    };
    if ((size_t)words * 8 <= kPinBytes && have_pin(ctx)) {
        const bool one = (size_t)words * 8 <= kTicketBytes;
        return fetch(ctx, (size_t)words * 8, host, one, [&](void* dst, uint32_t* ticket, uint32_t value) {
            launch(0, words, dst, one ? 1u : (unsigned)((words + 1023) / 1024), ticket, value);
        });
    }
    const int64_t chunk = std::min<int64_t>(words, (int64_t)4 << 20);
    uint2* const buf = static_cast<uint2*>(work_take(ctx, (size_t)chunk * 8));
    if (!buf) {  // no room: as it lies, put in order here
        const int64_t N = n_sites(ctx);
        std::vector<uint8_t> raw((size_t)count * 2 * (size_t)ctx->g.Nh);
        HIP_TRY(ctx, hipMemcpyAsync(raw.data(), dev, raw.size(), hipMemcpyDeviceToHost, ctx->stream));
        HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
        for (int64_t l = 0; l < count; ++l)
            for (int64_t i = 0; i < N; ++i) {
                int par;
                int64_t h;
                split_index(ctx, i, par, h);
                host[(int64_t)l * N + i] = raw[((size_t)l * 2 + par) * ctx->g.Nh + h] & mask;
            }
        return MICSA_OK;
    }
    int st = MICSA_OK;
    for (int64_t w0 = 0; w0 < words && !st; w0 += chunk) {
        const int64_t n = std::min(chunk, words - w0);
        launch(w0, n, buf, (unsigned)((n + 1023) / 1024), nullptr, 0u);
        st = check_launch(ctx, "k_natural");
        if (!st && (hipMemcpyAsync(host + w0 * 8, buf, (size_t)n * 8, hipMemcpyDeviceToHost, ctx->stream) != hipSuccess ||
                    hipStreamSynchronize(ctx->stream) != hipSuccess))
            st = fail(ctx, MICSA_EHIP, "state copy");
    }
    work_give(ctx, buf);
    return st;
}

// Bit-plane words [WL][2][Nh] -> host values [S][R][N]; with two planes
// (daemons) the value is bit0 + 2 bit1.
static int read_words(micsa_ctx* ctx, const uint64_t* w0, const uint64_t* w1, uint8_t* host)
{
    const int64_t N = n_sites(ctx);
    const int R = ctx->p.n_replicas;
    const GeomB gb = geomb(ctx);
    const size_t n = (size_t)word_lattices(ctx) * 2 * (size_t)ctx->g.Nh;
    std::vector<uint64_t> a(n), b(w1 ? n : 0);
    HIP_TRY(ctx, hipMemcpyAsync(a.data(), w0, n * 8, hipMemcpyDeviceToHost, ctx->stream));
    if (w1) HIP_TRY(ctx, hipMemcpyAsync(b.data(), w1, n * 8, hipMemcpyDeviceToHost, ctx->stream));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    for (int s = 0; s < ctx->p.n_samples; ++s)
        for (int r = 0; r < R; ++r)
            for (int64_t i = 0; i < N; ++i) {
                int par;
                int64_t h;
                split_index(ctx, i, par, h);
                int lane;
                const size_t idx = ((size_t)bp_word_of(gb, s, r, lane) * 2 + par) * ctx->g.Nh + h;
                uint8_t v = (uint8_t)((a[idx] >> lane) & 1u);
                if (w1) v = (uint8_t)(v | (((b[idx] >> lane) & 1u) << 1));
                host[((int64_t)s * R + r) * N + i] = v;
            }
    return MICSA_OK;
}

int micsa_read_spins(micsa_ctx* ctx, uint8_t* sigma)
{
    if (!ctx || !sigma) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = need_home(ctx)) return st_;
    if (ctx->bit) return read_words(ctx, ctx->bspin, nullptr, sigma);
    return read_state(ctx, ctx->spin, sigma, ctx->L, 1);  // bit 0: even bytes also hold their bonds
}

int micsa_read_demons(micsa_ctx* ctx, uint8_t* m)
{
    if (!ctx || !m) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = need_home(ctx)) return st_;
    if (ctx->bit) return read_words(ctx, ctx->bdm0, ctx->bdm1, m);
    int st = settle_wander(ctx);
    if (!st) st = read_state(ctx, ctx->dem, m, (int64_t)ctx->L * ctx->gamma);
    return st || !ctx->captured ? st : rest_and_wait(ctx);
}

int micsa_read_couplings(micsa_ctx* ctx, uint8_t* j)
{
    if (!ctx || !j) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = need_home(ctx)) return st_;
    const Geom& g = ctx->g;
    const int S = ctx->p.n_samples;
    std::vector<uint8_t> jbytes;
    std::vector<uint64_t> wplanes;
    if (ctx->bit) {
        wplanes.resize((size_t)bp_coupling_sets(geomb(ctx)) * 6 * g.Nh);
        HIP_TRY(ctx, hipMemcpyAsync(wplanes.data(), ctx->bJ, wplanes.size() * 8, hipMemcpyDeviceToHost, ctx->stream));
    } else {
        // bits 1..6 of the even spin bytes of replica 0 of each sample
        jbytes.resize((size_t)S * g.Nh);
        for (int s = 0; s < S; ++s)
            HIP_TRY(ctx, hipMemcpyAsync(jbytes.data() + (size_t)s * g.Nh,
                                        ctx->spin + (size_t)s * ctx->p.n_replicas * 2 * g.Nh, (size_t)g.Nh,
                                        hipMemcpyDeviceToHost, ctx->stream));
        for (auto& b : jbytes) b = (uint8_t)(b >> 1);
    }
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    const int64_t N = n_sites(ctx);
    auto bit = [&](int s, int d, int64_t h) -> uint32_t {
        if (ctx->bit && ctx->p.lane_mode == MICSA_LANES_REPLICAS)  // broadcast words: every bit the same
            return (uint32_t)(wplanes[((size_t)s * 6 + d) * g.Nh + (size_t)h] & 1u);
        if (ctx->bit)
            return (uint32_t)((wplanes[((size_t)(s / 64) * 6 + d) * g.Nh + (size_t)h] >> (s % 64)) & 1u);
        return (uint32_t)(jbytes[(size_t)s * g.Nh + (size_t)h] >> d) & 1u;
    };
    for (int s = 0; s < S; ++s)
        for (int64_t i = 0; i < N; ++i) {
            const int x = (int)(i % g.Lx), y = (int)((i / g.Lx) % g.Ly), z = (int)(i / ((int64_t)g.Lx * g.Ly));
            uint8_t v = 0;
            if (((x + y + z) & 1) == 0) {
                const int64_t h = i >> 1;
                v = (uint8_t)(bit(s, kPx, h) | (bit(s, kPy, h) << 1) | (bit(s, kPz, h) << 2));
            } else {
                // forward bonds of an odd site are the backward bonds of its even neighbours
                auto idx = [&](int xx, int yy, int zz) {
                    return ((xx % g.Lx) + (int64_t)g.Lx * ((yy % g.Ly) + (int64_t)g.Ly * (zz % g.Lz))) >> 1;
                };
                v = (uint8_t)(bit(s, kMx, idx(x + 1, y, z)) | (bit(s, kMy, idx(x, y + 1, z)) << 1) |
                              (bit(s, kMz, idx(x, y, z + 1)) << 2));
            }
            j[(int64_t)s * N + i] = v;
        }
    return MICSA_OK;
}

static int write_state(micsa_ctx* ctx, uint8_t* dev, const uint8_t* host, uint8_t maxv, int64_t count)
{
    const int64_t N = n_sites(ctx);
    std::vector<uint8_t> buf((size_t)count * 2 * (size_t)ctx->g.Nh);
    for (int64_t l = 0; l < count; ++l)
        for (int64_t i = 0; i < N; ++i) {
            const uint8_t v = host[(int64_t)l * N + i];
            if (v > maxv) return fail(ctx, MICSA_EINVAL, "value out of range");
            int par;
            int64_t h;
            split_index(ctx, i, par, h);
            buf[((size_t)l * 2 + par) * ctx->g.Nh + h] = v;
        }
    HIP_TRY(ctx, hipMemcpyAsync(dev, buf.data(), buf.size(), hipMemcpyHostToDevice, ctx->stream));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    return MICSA_OK;
}

// Host values [S][R][N] -> bit-plane words (bit0 into w0, bit1 into w1).
static int write_words(micsa_ctx* ctx, uint64_t* w0, uint64_t* w1, const uint8_t* host, uint8_t maxv)
{
    const int64_t N = n_sites(ctx);
    const int R = ctx->p.n_replicas;
    const GeomB gb = geomb(ctx);
    const size_t n = (size_t)word_lattices(ctx) * 2 * (size_t)ctx->g.Nh;
    std::vector<uint64_t> a(n, 0), b(w1 ? n : 0, 0);
    for (int s = 0; s < ctx->p.n_samples; ++s)
        for (int r = 0; r < R; ++r)
            for (int64_t i = 0; i < N; ++i) {
                const uint8_t v = host[((int64_t)s * R + r) * N + i];
                if (v > maxv) return fail(ctx, MICSA_EINVAL, "value out of range");
                int par;
                int64_t h;
                split_index(ctx, i, par, h);
                int lane;
                const size_t idx = ((size_t)bp_word_of(gb, s, r, lane) * 2 + par) * ctx->g.Nh + h;
                a[idx] |= (uint64_t)(v & 1u) << lane;
                if (w1) b[idx] |= (uint64_t)(v >> 1) << lane;
            }
    HIP_TRY(ctx, hipMemcpyAsync(w0, a.data(), n * 8, hipMemcpyHostToDevice, ctx->stream));
    if (w1) HIP_TRY(ctx, hipMemcpyAsync(w1, b.data(), n * 8, hipMemcpyHostToDevice, ctx->stream));
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    return MICSA_OK;
}

int micsa_write_spins(micsa_ctx* ctx, const uint8_t* sigma)
{
    if (!ctx || !sigma) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = own_home(ctx)) return st_;
    int st = ctx->bit ? write_words(ctx, ctx->bspin, nullptr, sigma, 1) : write_state(ctx, ctx->spin, sigma, 1, ctx->L);
    if (!st && !ctx->bit) st = enqueue_bonds(ctx);  // the written bytes hold spins only: restore the bond bits
    if (st) {
        (void)rest_and_wait(ctx);
        return st;
    }
    if ((st = tally_from_state(ctx))) return st;
    ctx->tally_ok = true;
    return rest_and_wait(ctx);
}

int micsa_write_demons(micsa_ctx* ctx, const uint8_t* m)
{
    if (!ctx || !m) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = own_home(ctx)) return st_;
    const int st = ctx->bit ? write_words(ctx, ctx->bdm0, ctx->bdm1, m, 3)
                            : write_state(ctx, ctx->dem, m, 3, (int64_t)ctx->L * ctx->gamma);
    if (!st) ctx->pend_wander = -1;  // the written daemons are where they are
    const int back = rest_and_wait(ctx);
    return st ? st : back;
}

// ------------------------------------------------------------- checkpoint
// Image: CkHeader, the schedule table (T_len doubles), the tally per lattice
// (int64), spins [L][N], daemons [L][gamma][N], couplings [S][N] (bytes),
// then the FNV-1a hash of everything before it.
namespace {
constexpr char kCkMagic[8] = {'M', 'I', 'C', 'S', 'A', '-', 'C', 'K'};
constexpr uint32_t kCkVersion = 1;

struct CkHeader {
    char magic[8];
    uint32_t version;
    uint32_t header_bytes;
    micsa_params p;
    int64_t k;
    int32_t sched_set, sched_kind, sched_period, reserved;
    double T0, T1;
    int64_t n_sweeps, T_len;
    uint64_t total_bytes;
};

uint64_t fnv1a(const uint8_t* d, size_t n)
{
    uint64_t h = 1469598103934665603ull;
    for (size_t i = 0; i < n; ++i) {
        h ^= d[i];
        h *= 1099511628211ull;
    }
    return h;
}

size_t ck_bytes(const micsa_ctx* c, int64_t T_len)
{
    const size_t N = (size_t)n_sites(c), L = (size_t)c->L;
    return sizeof(CkHeader) + (size_t)T_len * 8 + L * 8 + L * N + L * (size_t)c->gamma * N +
           (size_t)c->p.n_samples * N + 8;
}

bool same_params(const micsa_params& a, const micsa_params& b)
{
    return a.Lx == b.Lx && a.Ly == b.Ly && a.Lz == b.Lz && a.n_samples == b.n_samples &&
           a.n_replicas == b.n_replicas && a.layout == b.layout && a.gamma == b.gamma &&
           a.lane_mode == b.lane_mode && a.seed == b.seed;
}
}  // namespace

int micsa_save(micsa_ctx* ctx, void* buf, size_t* len)
{
    if (!ctx || !len) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = need_home(ctx)) return st_;
    const int64_t T_len = ctx->sched.set ? (int64_t)ctx->sched.table.size() : 0;
    const size_t total = ck_bytes(ctx, T_len);
    if (!buf) {
        *len = total;
        return MICSA_OK;
    }
    if (*len < total) {
        *len = total;
        return fail(ctx, MICSA_ERANGE, "checkpoint buffer smaller than micsa_save's size");
    }
    const size_t N = (size_t)n_sites(ctx), L = (size_t)ctx->L;
    uint8_t* out = static_cast<uint8_t*>(buf);
    CkHeader h;
    std::memset(&h, 0, sizeof h);
    std::memcpy(h.magic, kCkMagic, 8);
    h.version = kCkVersion;
    h.header_bytes = (uint32_t)sizeof(CkHeader);
    h.p = ctx->p;
    h.k = ctx->k;
    h.sched_set = ctx->sched.set ? 1 : 0;
    h.sched_kind = ctx->sched.kind;
    h.sched_period = ctx->sched.period;
    h.T0 = ctx->sched.T0;
    h.T1 = ctx->sched.T1;
    h.n_sweeps = ctx->sched.n_sweeps;
    h.T_len = T_len;
    h.total_bytes = total;
    size_t o = sizeof(CkHeader);
    if (T_len) std::memcpy(out + o, ctx->sched.table.data(), (size_t)T_len * 8);
    o += (size_t)T_len * 8;
    int st;
    // reading the daemons first applies an owed walker wandering
    uint8_t* tally = out + o;
    uint8_t* spins = tally + L * 8;
    uint8_t* dems = spins + L * N;
    uint8_t* coup = dems + L * (size_t)ctx->gamma * N;
    if ((st = micsa_read_demons(ctx, dems))) return st;
    if ((st = micsa_read_spins(ctx, spins))) return st;
    if ((st = micsa_read_couplings(ctx, coup))) return st;
    std::vector<int64_t> E(L);
    st = ctx->bit && !ctx->tally_ok ? micsa_read_energy(ctx, E.data()) : micsa_read_energy_tally(ctx, E.data());
    if (st) return st;
    std::memcpy(tally, E.data(), L * 8);
    h.k = ctx->k;
    std::memcpy(out, &h, sizeof h);
    const uint64_t hash = fnv1a(out, total - 8);
    std::memcpy(out + total - 8, &hash, 8);
    *len = total;
    return MICSA_OK;
}

int micsa_load(micsa_ctx* ctx, const void* buf, size_t len)
{
    if (!ctx) return MICSA_EINVAL;
    if (int st_ = refuse_capture(ctx)) return st_;
    if (int st_ = need_home(ctx)) return st_;
    if (!buf) return fail(ctx, MICSA_EINVAL, "null checkpoint");
    const uint8_t* in = static_cast<const uint8_t*>(buf);
    CkHeader h;
    if (len < sizeof h) return fail(ctx, MICSA_EINVAL, "checkpoint too short");
    std::memcpy(&h, in, sizeof h);
    if (std::memcmp(h.magic, kCkMagic, 8) != 0 || h.version != kCkVersion || h.header_bytes != sizeof(CkHeader))
        return fail(ctx, MICSA_EINVAL, "not a checkpoint of this library version");
    if (!same_params(h.p, ctx->p))
        return fail(ctx, MICSA_EINVAL, "checkpoint of a context with other parameters");
    if (h.T_len < 0 || h.T_len > (int64_t)(len / 8) || h.k < 0) return fail(ctx, MICSA_EINVAL, "corrupt checkpoint");
    const size_t total = ck_bytes(ctx, h.T_len);
    if (h.total_bytes != total || len < total) return fail(ctx, MICSA_EINVAL, "checkpoint size mismatch");
    uint64_t hash;
    std::memcpy(&hash, in + total - 8, 8);
    if (hash != fnv1a(in, total - 8)) return fail(ctx, MICSA_EINVAL, "checkpoint checksum mismatch");
    const size_t N = (size_t)n_sites(ctx), L = (size_t)ctx->L;
    const uint8_t* table = in + sizeof(CkHeader);
    const uint8_t* tally = table + (size_t)h.T_len * 8;
    const uint8_t* spins = tally + L * 8;
    const uint8_t* dems = spins + L * N;
    const uint8_t* coup = dems + L * (size_t)ctx->gamma * N;
    // the couplings follow from the seed: they must be this context's
    std::vector<uint8_t> mine((size_t)ctx->p.n_samples * N);
    int st = micsa_read_couplings(ctx, mine.data());
    if (st) return st;
    if (std::memcmp(mine.data(), coup, mine.size()) != 0)
        return fail(ctx, MICSA_EINVAL, "checkpoint couplings differ from the context's");
    for (size_t i = 0; i < L * N; ++i)
        if (spins[i] > 1) return fail(ctx, MICSA_EINVAL, "checkpoint spin out of range");
    for (size_t i = 0; i < L * (size_t)ctx->gamma * N; ++i)
        if (dems[i] > 3) return fail(ctx, MICSA_EINVAL, "checkpoint daemon level out of range");
    if (h.sched_set) {
        micsa_schedule s{};
        s.kind = h.sched_kind;
        s.refresh_period = h.sched_period;
        s.T0 = h.T0;
        s.T1 = h.T1;
        s.n_sweeps = h.n_sweeps;
        std::vector<double> tb((size_t)h.T_len);
        if (h.T_len) std::memcpy(tb.data(), table, (size_t)h.T_len * 8);
        s.T_table = tb.empty() ? nullptr : tb.data();
        s.T_len = h.T_len;
        if ((st = micsa_set_schedule(ctx, &s))) return st;
    } else {
        ctx->sched = Schedule{};
        ctx->cdr_n = 0;
        ctx->msc_drawn = -1;
    }
    if ((st = micsa_write_spins(ctx, spins))) return st;
    if ((st = micsa_write_demons(ctx, dems))) return st;
    {
        std::vector<int64_t> E(L);
        std::memcpy(E.data(), tally, L * 8);
        if ((st = set_tally(ctx, E))) return st;
    }
    ctx->k = h.k;
    return MICSA_OK;
}

int micsa_get_counters(micsa_ctx* ctx, int64_t* k, int64_t* rho)
{
    if (!ctx) return MICSA_EINVAL;
    if (k) *k = ctx->k;
    if (rho) *rho = refresh_index(ctx->k / ctx->gamma, ctx->sched.set ? ctx->sched.period : 1);
    return MICSA_OK;
}

int micsa_get_thresholds(micsa_ctx* ctx, int64_t rho, uint64_t t[3])
{
    if (!ctx || !t) return MICSA_EINVAL;
    if (!ctx->sched.set) return fail(ctx, MICSA_ESTATE, "no schedule installed");
    if (rho < 0 || rho >= std::max<int64_t>(refresh_count(ctx->sched), 1))
        return fail(ctx, MICSA_ERANGE, "refresh index outside the schedule");
    const DaemonThresholds th = daemon_thresholds(temperature(ctx->sched, rho));
    t[0] = th.t0;
    t[1] = th.t1;
    t[2] = th.t2;
    return MICSA_OK;
}

int micsa_get_heatbath_thresholds(micsa_ctx* ctx, int64_t rho, uint64_t tau[7])
{
    if (!ctx || !tau) return MICSA_EINVAL;
    if (!ctx->sched.set) return fail(ctx, MICSA_ESTATE, "no schedule installed");
    if (rho < 0 || rho >= std::max<int64_t>(refresh_count(ctx->sched), 1))
        return fail(ctx, MICSA_ERANGE, "refresh index outside the schedule");
    const HeatBathThresholds th = heatbath_thresholds(temperature(ctx->sched, rho));
    for (int v = 0; v < 7; ++v) tau[v] = th.tau[v];
    return MICSA_OK;
}

int micsa_get_metropolis_thresholds(micsa_ctx* ctx, int64_t rho, uint64_t theta[7])
{
    if (!ctx || !theta) return MICSA_EINVAL;
    if (!ctx->sched.set) return fail(ctx, MICSA_ESTATE, "no schedule installed");
    if (rho < 0 || rho >= std::max<int64_t>(refresh_count(ctx->sched), 1))
        return fail(ctx, MICSA_ERANGE, "refresh index outside the schedule");
    const MetropolisThresholds th = metropolis_thresholds(temperature(ctx->sched, rho));
    for (int q = 0; q < 7; ++q) theta[q] = th.tau[q];
    return MICSA_OK;
}

int micsa_set_timing(micsa_ctx* ctx, int32_t enable)
{
    if (!ctx) return MICSA_EINVAL;
    ctx->timing = enable != 0;
    return MICSA_OK;
}

int micsa_get_timing(micsa_ctx* ctx, int32_t kind, double* total_ms, int64_t* launches)
{
    if (!ctx || kind < 0 || kind >= kTimingKinds) return MICSA_EINVAL;
    HIP_TRY(ctx, hipStreamSynchronize(ctx->stream));
    for (int kd = 0; kd < kTimingKinds; ++kd) {
        for (auto& e : ctx->events[kd]) {
            float ms = 0.f;
            if (hipEventElapsedTime(&ms, e.first, e.second) == hipSuccess) {
                ctx->time_ms[kd] += ms;
                ctx->launches[kd] += 1;
            }
            (void)hipEventDestroy(e.first);
            (void)hipEventDestroy(e.second);
        }
        ctx->events[kd].clear();
    }
    if (total_ms) *total_ms = ctx->time_ms[kind];
    if (launches) *launches = ctx->launches[kind];
    return MICSA_OK;
}

const char* micsa_kernel_name(const micsa_ctx* ctx, int32_t algo)
{
    if (ctx && ctx->bit)
        return algo == MICSA_ALGO_MICSA
                   ? (bp_one_launch(ctx) && !use_graph(ctx) ? (bp_rows(bp_launch(ctx)) ? "kb_sweep_rows" : "kb_sweep")
                                                            : "kb_micsa_half")
                   : "";
    if (ctx && algo == MICSA_ALGO_MICSA && !use_resident(ctx) && !use_slab(ctx) && use_cells(ctx))
        return "k_cells_sweep";
    if (ctx && algo == MICSA_ALGO_MICSA && use_msc(ctx))  // a long call runs its sweeps in pairs where it can
        return msc_one_launch(ctx) ? (msc2_fits(ctx) ? "k_msc_sweep_multi" : "k_msc_sweep") : "k_msc_half";
    // (the names of the forms that callers ask for by option stay: lattices of
    // the resident and slab forms run the cell sweep too)
    if (ctx && algo == MICSA_ALGO_WALKERS && use_cells_walkers(ctx, kMscMinSweeps)) return "k_cells_sweep";
    // walkers on the fused sweeps wander on the next sweep's loads
    if (ctx && algo == MICSA_ALGO_WALKERS && use_msc(ctx, kMscMinSweeps, algo))
        return msc_one_launch(ctx) && msc2_fits(ctx) && 64 % (ctx->p.Lx / 64) == 0 ? "k_msc_sweep_multi"
                                                                                    : "k_msc_sweep";
    if (algo == MICSA_ALGO_WALKERS)
        return ctx && use_fused(ctx) && ctx->gamma == 1
                   ? (ctx->temporal == 2 && sweep2_walk_eligible(ctx) ? "k_micsa_sweep2_fused" : "k_micsa_sweep_fused")
                   : "k_micsa_half+k_wander";
    if (ctx && use_resident(ctx))
        return algo == MICSA_ALGO_HEATBATH ? "k_resident<1>" : (algo == MICSA_ALGO_METROPOLIS ? "k_resident<2>" : "k_resident<0>");
    if (ctx && (algo == MICSA_ALGO_HEATBATH || algo == MICSA_ALGO_METROPOLIS) && use_cells_canonical(ctx))
        return "k_cells_sweep";
    if (algo == MICSA_ALGO_HEATBATH)
        return ctx && use_fused(ctx) ? "k_heatbath_sweep_fused<0>" : "k_heatbath_half<0>";
    if (algo == MICSA_ALGO_METROPOLIS)
        return ctx && use_fused(ctx) ? "k_heatbath_sweep_fused<1>" : "k_heatbath_half<1>";
    if (ctx && use_fused(ctx))
        return ctx->temporal == 2 && sweep2_eligible(ctx) ? "k_micsa_sweep2_fused" : "k_micsa_sweep_fused";
    if (ctx && use_slab(ctx)) return slab_pairs(ctx) ? "k_micsa_slab2" : "k_micsa_slab";
    return "k_micsa_half";
}

int micsa_set_option(micsa_ctx* ctx, int32_t option, int64_t value)
{
    if (!ctx) return MICSA_EINVAL;
    switch (option) {
    case MICSA_OPT_SWEEP_KERNEL:
        if (value != MICSA_KERNEL_AUTO && value != MICSA_KERNEL_SIMPLE && value != MICSA_KERNEL_FUSED &&
            value != MICSA_KERNEL_RESIDENT && value != MICSA_KERNEL_MULTISPIN && value != MICSA_KERNEL_SLAB)
            return fail(ctx, MICSA_EINVAL, "unknown sweep kernel");
        if (value == MICSA_KERNEL_SLAB && !slab_eligible(ctx))
            return fail(ctx, MICSA_EINVAL, "the slab sweep needs the byte layout, gamma = 1 and Ly * Lx / 8 <= 1024");
        if (value == MICSA_KERNEL_MULTISPIN && !msc_eligible(ctx))
            return fail(ctx, MICSA_EINVAL, "the multispin sweep needs the byte layout, gamma = 1 and Lx % 128 == 0");
        if (value == MICSA_KERNEL_RESIDENT && !resident_eligible(ctx))
            return fail(ctx, MICSA_EINVAL, "the resident sweep needs a byte-layout lattice of at most 102400 sites");
        if (value == MICSA_KERNEL_FUSED && ctx->bit && !bp_fits(ctx, bp_launch(ctx)))
            return fail(ctx, MICSA_EINVAL, "the one-launch bit-plane sweep needs five rows of a plane in a work-group");
        if (value == MICSA_KERNEL_FUSED && !ctx->bit && !fused_eligible(ctx))
            return fail(ctx, MICSA_EINVAL, "the fused sweep needs Lx % 32 == 0");
        ctx->kernel_opt = (int32_t)value;
        return MICSA_OK;
    case MICSA_OPT_TILE_Y:
        if (value < 0 || value > ctx->p.Ly || (value > 0 && (value + 4) * (ctx->p.Lx / 32) > 1024))
            return fail(ctx, MICSA_EINVAL, "tile_y must be at most Ly and fit a work-group");
        ctx->tile_y = (int32_t)value;
        ctx->tile2 = msc2_plan(ctx);
        return MICSA_OK;
    case MICSA_OPT_GRAPHS:
        if (value != 0 && value != 1) return fail(ctx, MICSA_EINVAL, "graphs is 0 or 1");
        ctx->use_graphs = (int32_t)value;
        return MICSA_OK;
    case MICSA_OPT_DRAW_AHEAD:
        if (value != 0 && value != 1) return fail(ctx, MICSA_EINVAL, "draw_ahead is 0 or 1");
        ctx->draw_ahead = (int32_t)value;
        return MICSA_OK;
    case MICSA_OPT_MSC_FUSED:
        if (value != 0 && value != 1) return fail(ctx, MICSA_EINVAL, "msc_fused is 0 or 1");
        ctx->msc_fused = (int32_t)value;
        return MICSA_OK;
    case MICSA_OPT_TEMPORAL:
        if (value != 1 && value != 2) return fail(ctx, MICSA_EINVAL, "temporal is 1 or 2");
        ctx->temporal = (int32_t)value;
        return MICSA_OK;
    case MICSA_OPT_MSC_PASS:
        if (value != 1 && value != 2) return fail(ctx, MICSA_EINVAL, "msc_pass is 1 or 2");
        ctx->msc_pass = (int32_t)value;
        return MICSA_OK;
    case MICSA_OPT_PREFETCH:
        if (value != 1 && value != 2) return fail(ctx, MICSA_EINVAL, "prefetch is 1 or 2");
        ctx->prefetch = (int32_t)value;
        return MICSA_OK;
    case MICSA_OPT_XCD_MAP:
        if (value < 0 || value > 2) return fail(ctx, MICSA_EINVAL, "xcd_map is 0, 1 or 2");
        ctx->xcd_map = (int32_t)value;
        ctx->tile2 = msc2_plan(ctx);
        return MICSA_OK;
    case MICSA_OPT_TILE_Z:
        if (value < 0 || (value > 0 && ctx->p.Lz % value != 0))
            return fail(ctx, MICSA_EINVAL, "tile_z must divide Lz");
        ctx->tile_z = (int32_t)value;
        ctx->tile2 = msc2_plan(ctx);
        return MICSA_OK;
    default: return fail(ctx, MICSA_EINVAL, "unknown option");
    }
}

}  // extern "C"

// =========================================================== serving pool
namespace {

struct PoolJob {
    int64_t id = 0;
    micsa_params p{};
    Schedule sched;  // copied schedule (table owned here)
    int32_t state = MICSA_JOB_QUEUED;
    size_t bytes = 0;
    micsa_ctx* ctx = nullptr;
    // Small lattices (batches()) run in the pool's batched launches on the pool
    // stream; every other job gets a stream of its own (default
    // priority), so large jobs overlap with each other and with the batch.
    bool batched = false;
    hipStream_t stream = nullptr;
    hipEvent_t ev[2] = {nullptr, nullptr};  // end of the last two chunks of sweeps
    int64_t chunks = 0;                     // chunks enqueued so far
    int64_t last_batch = -1;                // batched jobs: the batch that holds their latest chunk
    // from submission on: launch plans; and what the job may hold, the most
    // first: planes and levels drawn for up to 16 refreshes, planes and two
    // refreshes, the state's own arrays alone
    CellPlans plans;
    MscTile tile2{};
    int device = 0, cus = 0;
    size_t draw_room[2] = {0, 0};
    size_t need[3] = {0, 0, 0};
    size_t charged = 0;  // while admitted
};

size_t footprint(const micsa_params* p)
{
    const size_t N = (size_t)p->Lx * p->Ly * p->Lz;
    const size_t L = (size_t)p->n_samples * p->n_replicas;
    const size_t slots = (L + (size_t)p->n_samples) * kSlots * 8;
    if (p->layout == MICSA_LAYOUT_BITPLANE) {
        const bool reps = p->lane_mode == MICSA_LANES_REPLICAS;
        const size_t WL = reps ? (size_t)p->n_samples * (((size_t)p->n_replicas + 63) / 64)
                               : (((size_t)p->n_samples + 63) / 64) * p->n_replicas;
        const size_t NJ = reps ? (size_t)p->n_samples : ((size_t)p->n_samples + 63) / 64;
        return 2 * WL * N * 8 * 3 + NJ * 6 * (N / 2) * 8 + slots;  // state and its alternate
    }
    const size_t gamma = p->gamma == 0 ? 1 : (size_t)p->gamma;
    // spin and daemon bytes, and as much again: second copies, or planes and drawn levels
    size_t bytes = 2 * L * N * (1 + gamma) + slots;
    // the multispin planes beside both copies: spins and two level planes, their
    // alternates, the drawn levels (2) and the six coupling planes of the even
    // sites (3 words per word of sites), each 1 bit per site: 11/8 B per site
    // per lattice
    if (gamma == 1 && p->Lx % 128 == 0) bytes += 11 * L * N / 8;
    // lattices in tiles have second copies of the planes too, and longer calls to
    // draw levels for
    else if (gamma == 1 && (size_t)p->Ly * (p->Lx / 8) <= (size_t)kSlabLanes && N / 2 * 3 > kResidentLdsMax &&
             p->Lx < 128)
        bytes += 2 * L * N;
    return bytes;
}

// What a job of this shape (setup_ctx, draw_room set) holds.  A bit-plane
// job, whose chunks may be too short for the planes, has second copies of its
// words then.
size_t job_need(const micsa_ctx* shape)
{
    const CtxBytes b = ctx_bytes(shape);
    return b.home + b.work + (bp_one_launch(shape) ? 3 * arena_size(b.words * 8) : 0);
}

// Plans and needs of a job (without a device: as for 256 compute units).  Drawn
// levels at most: 16 refreshes (a chunk of sweeps seldom has more) within 1 MiB or
// 2.5 bytes per site and lattice, whichever is more.
void plan_job(PoolJob& j)
{
    micsa_ctx shape;
    (void)setup_ctx(&shape, &j.p, nullptr);
    j.plans.main = shape.plan;
    j.plans.walk = shape.walk;
    std::copy(std::begin(shape.brief), std::end(shape.brief), j.plans.brief);
    j.tile2 = shape.tile2;
    j.device = shape.device;
    j.cus = shape.cus;
    const size_t one = (size_t)shape.L * 2 * (size_t)cell_geom(&shape).plane * 8;
    const size_t sites = (size_t)shape.L * 2 * (size_t)shape.g.Nh;
    j.draw_room[0] = std::min(16 * one, std::max((size_t)1 << 20, sites * 5 / 2));
    j.draw_room[1] = 1;  // (at least two)
    for (int v = 0; v < 3; ++v) {
        shape.draw_room = v < 2 ? j.draw_room[v] : 1;
        shape.plan.ok = shape.plan.ok && v < 2;
        j.need[v] = job_need(&shape);
    }
}

}  // namespace

struct micsa_pool {
    size_t budget = 0, used = 0;
    int32_t max_running = 1;
    hipStream_t stream = nullptr;
    int64_t next_id = 1;
    std::vector<PoolJob> jobs;  // every job not yet released, in arrival order
    // batches: two in flight at most, each with its tables (the host may refill
    // one while the other is read)
    uint8_t* d_tab[2] = {nullptr, nullptr};
    uint8_t* h_tab[2] = {nullptr, nullptr};  // pinned host copy of each, kept until its launches have finished
    size_t tab_cap[2] = {0, 0};
    hipEvent_t bev[2] = {nullptr, nullptr};
    int64_t batches = 0;
    // Small jobs are set up on a stream of their own and move to the pool's for
    // their batches; finished ones are read on it, so that neither waits for
    // the batches in flight.
    hipStream_t side = nullptr;
    int side_device = 0;
    JobStore store;
};

namespace {

// The chunk slot `n` of a job (or of the batch) may be refilled once the
// chunk two before it has finished.
bool slot_free(hipEvent_t e)
{
    if (!e) return true;
    const hipError_t q = hipEventQuery(e);
    if (q == hipErrorNotReady) return false;
    (void)hipGetLastError();
    return true;
}

// (the stream's work has finished)
void free_job_stream(micsa_pool* pool, PoolJob& j, int device)
{
    for (auto& e : j.ev)
        if (e) {
            (void)hipEventDestroy(e);
            e = nullptr;
        }
    if (j.stream) {
        drop_stream(&pool->store, device, j.stream);
        j.stream = nullptr;
    }
}

}  // namespace

extern "C" {

int micsa_pool_footprint(const micsa_params* p, size_t* bytes)
{
    if (!p || !bytes) return MICSA_EINVAL;
    *bytes = footprint(p);
    return MICSA_OK;
}

int micsa_pool_create(size_t hbm_budget, int32_t max_running, void* hip_stream, micsa_pool** out)
{
    if (!out) return MICSA_EINVAL;
    *out = nullptr;
    if (hbm_budget == 0 || max_running < 1) return MICSA_EINVAL;
    micsa_pool* pool = new (std::nothrow) micsa_pool();
    if (!pool) return MICSA_ENOMEM;
    pool->budget = hbm_budget;
    pool->max_running = max_running;
    pool->stream = (hipStream_t)hip_stream;
    *out = pool;
    return MICSA_OK;
}

int micsa_pool_destroy(micsa_pool* pool)
{
    if (!pool) return MICSA_OK;
    (void)hipStreamSynchronize(pool->stream);
    for (auto& j : pool->jobs) {
        const int device = j.ctx ? j.ctx->device : 0;
        if (j.ctx) micsa_destroy(j.ctx);  // synchronises the job's stream
        free_job_stream(pool, j, device);
    }
    if (pool->side) drop_stream(&pool->store, pool->side_device, pool->side);
    for (int b = 0; b < 2; ++b) {
        if (pool->d_tab[b]) (void)hipFree(pool->d_tab[b]);
        if (pool->h_tab[b]) (void)hipHostFree(pool->h_tab[b]);
        if (pool->bev[b]) (void)hipEventDestroy(pool->bev[b]);
    }
    delete pool;
    return MICSA_OK;
}

int micsa_pool_sync(micsa_pool* pool)
{
    if (!pool) return MICSA_EINVAL;
    if (hipStreamSynchronize(pool->stream) != hipSuccess) return MICSA_EHIP;
    if (pool->side && hipStreamSynchronize(pool->side) != hipSuccess) return MICSA_EHIP;
    for (auto& j : pool->jobs)
        if (j.stream && hipStreamSynchronize(j.stream) != hipSuccess) return MICSA_EHIP;
    return MICSA_OK;
}

int micsa_pool_submit(micsa_pool* pool, const micsa_params* p, const micsa_schedule* s, int64_t* job)
{
    if (!pool || !p || !s || !job) return MICSA_EINVAL;
    // validate parameters and schedule the same way a context would
    if (!params_ok(p)) return MICSA_EINVAL;
    if (s->refresh_period < 0 || s->n_sweeps < 1) return MICSA_EINVAL;
    auto okT = [](double T) { return T > 0.0 && std::isfinite(T); };
    if (s->kind == MICSA_SCHED_CONST ? !okT(s->T0)
        : s->kind == MICSA_SCHED_LINEAR ? !(okT(s->T0) && okT(s->T1))
        : s->kind != MICSA_SCHED_TABLE)
        return MICSA_EINVAL;
    PoolJob j;
    j.p = *p;
    j.sched.set = true;
    j.sched.kind = s->kind;
    j.sched.period = s->refresh_period;
    j.sched.T0 = s->T0;
    j.sched.T1 = s->T1;
    j.sched.n_sweeps = s->n_sweeps;
    j.sched.n_steps = (s->n_sweeps + std::max(p->gamma, 1) - 1) / std::max(p->gamma, 1);
    if (s->kind == MICSA_SCHED_TABLE) {
        if (!s->T_table || s->T_len < refresh_count(j.sched)) return MICSA_EINVAL;
        j.sched.table.assign(s->T_table, s->T_table + s->T_len);
    }
    j.bytes = footprint(p);
    if (j.bytes > pool->budget) return MICSA_EINVAL;
    plan_job(j);
    j.id = pool->next_id++;
    *job = j.id;
    pool->jobs.push_back(std::move(j));
    return MICSA_OK;
}

static PoolJob* find_job(micsa_pool* pool, int64_t id)
{
    for (auto& j : pool->jobs)
        if (j.id == id) return &j;
    return nullptr;
}

// Jobs that share batched launches: lattices of at most two cells per lane of
// one work-group, in the byte layout.
static bool batches(const micsa_ctx* c)
{
    return use_cells(c) && !c->bit && c->gamma == 1 && c->plan.sweeps == 0 && c->plan.nr <= 2;
}

// Enqueue the next chunk of the batched jobs, if one of the two batches is free:
// in rounds of one draw launch (the refresh levels that run out) and one sweep
// launch per kernel form, each over the lattices of every job.
static int enqueue_batch(micsa_pool* pool, int64_t sweeps)
{
    const int slot = (int)(pool->batches & 1);
    if (!slot_free(pool->bev[slot])) return MICSA_OK;
    struct Part {
        PoolJob* j;
        int64_t k, end;  // next sweep, end of the chunk
    };
    std::vector<Part> parts;
    for (auto& j : pool->jobs) {
        if (j.state != MICSA_JOB_RUNNING || !j.batched) continue;
        micsa_ctx* c = j.ctx;
        const int64_t n = std::min<int64_t>(sweeps, c->sched.n_sweeps - c->k);
        if (n <= 0) continue;
        if (const int st = need_planes(c)) return st;  // (a batched job has had its planes since it was admitted)
        c->home_ok = false;
        parts.push_back(Part{&j, c->k, c->k + n});
    }
    if (parts.empty()) return MICSA_OK;
    struct Launch {
        int nr, xm;  // nr = 0: a draw
        unsigned block, items, blocks;
        size_t first;  // of its items
    };
    std::vector<CellSweep> jobs;
    std::vector<CellDraw> draws;
    std::vector<CellItem> items;
    std::vector<Launch> seq;
    for (bool more = true; more;) {
        more = false;
        const size_t d0 = items.size();
        int64_t dblocks = 1;
        std::vector<std::pair<micsa_ctx*, size_t>> round;  // jobs of the round and their entries
        for (auto& p : parts) {
            if (p.k >= p.end) continue;
            micsa_ctx* c = p.j->ctx;
            bool draw;
            CellDraw D;
            CellSweep J = cells_next(c, p.k, p.end, kResidentChunk, &draw, &D);
            fill_cells(c, J, c->plan);
            if (draw) {
                for (int l = 0; l < c->L; ++l) items.push_back(CellItem{(int32_t)draws.size(), l});
                draws.push_back(D);
                dblocks = std::max(dblocks, cells_draw_blocks(D));
            }
            round.emplace_back(c, jobs.size());
            jobs.push_back(J);
            p.k += J.n;
            more = more || p.k < p.end;
        }
        if (items.size() > d0)
            seq.push_back(Launch{0, 0, 64, (unsigned)(items.size() - d0), (unsigned)std::min<int64_t>(dblocks, 1024), d0});
        for (int nr = 1; nr <= 2; ++nr)
            for (int xm = 0; xm < 3; ++xm) {
                const size_t s0 = items.size();
                unsigned block = 0;
                for (auto& r : round) {
                    if (r.first->plan.nr != nr || r.first->plan.xm != xm) continue;
                    for (int l = 0; l < r.first->L; ++l) items.push_back(CellItem{(int32_t)r.second, l});
                    block = std::max(block, r.first->plan.block);
                }
                if (block) seq.push_back(Launch{nr, xm, block, (unsigned)(items.size() - s0), 1, s0});
            }
    }
    // one table: jobs, draws, items
    const size_t o_d = (jobs.size() * sizeof(CellSweep) + 63) / 64 * 64;
    const size_t o_i = o_d + (draws.size() * sizeof(CellDraw) + 63) / 64 * 64;
    const size_t bytes = o_i + items.size() * sizeof(CellItem);
    if (bytes > pool->tab_cap[slot]) {
        if (pool->d_tab[slot]) (void)hipFree(pool->d_tab[slot]);
        if (pool->h_tab[slot]) (void)hipHostFree(pool->h_tab[slot]);
        pool->d_tab[slot] = pool->h_tab[slot] = nullptr;
        pool->tab_cap[slot] = 0;
        const size_t cap = std::max<size_t>(2 * bytes, (size_t)1 << 20);
        if (hipMalloc(&pool->d_tab[slot], cap) != hipSuccess || hipHostMalloc(&pool->h_tab[slot], cap) != hipSuccess) {
            (void)hipGetLastError();
            return MICSA_ENOMEM;
        }
        pool->tab_cap[slot] = cap;
    }
    uint8_t* const h = pool->h_tab[slot];
    std::memcpy(h, jobs.data(), jobs.size() * sizeof(CellSweep));
    if (!draws.empty()) std::memcpy(h + o_d, draws.data(), draws.size() * sizeof(CellDraw));
    std::memcpy(h + o_i, items.data(), items.size() * sizeof(CellItem));
    if (!pool->bev[slot] && hipEventCreateWithFlags(&pool->bev[slot], hipEventDisableTiming) != hipSuccess)
        return MICSA_EHIP;
    if (hipMemcpyAsync(pool->d_tab[slot], h, bytes, hipMemcpyHostToDevice, pool->stream) != hipSuccess)
        return MICSA_EHIP;
    const auto* dj = reinterpret_cast<const CellSweep*>(pool->d_tab[slot]);
    const auto* dd = reinterpret_cast<const CellDraw*>(pool->d_tab[slot] + o_d);
    const auto* di = reinterpret_cast<const CellItem*>(pool->d_tab[slot] + o_i);
    using Kern = void (*)(const CellSweep*, const CellItem*);
    static const Kern kern[2][3] = {{k_cells_sweep_batch<1, 0>, k_cells_sweep_batch<1, 1>, k_cells_sweep_batch<1, 2>},
                                    {k_cells_sweep_batch<2, 0>, k_cells_sweep_batch<2, 1>, k_cells_sweep_batch<2, 2>}};
    for (const Launch& q : seq) {
        if (q.nr == 0)
            for (unsigned y = 0; y < q.items; y += 65535)
                k_cells_draw_batch<<<dim3(q.blocks, std::min(65535u, q.items - y)), q.block, 0, pool->stream>>>(
                    dd, di + q.first + y);
        else
            kern[q.nr - 1][q.xm]<<<q.items, q.block, 0, pool->stream>>>(dj, di + q.first);
        if (hipGetLastError() != hipSuccess) return MICSA_EHIP;
    }
    if (hipEventRecord(pool->bev[slot], pool->stream) != hipSuccess) return MICSA_EHIP;
    for (auto& p : parts) {
        p.j->ctx->k = p.end;
        p.j->last_batch = pool->batches;
    }
    ++pool->batches;
    return MICSA_OK;
}

// What lies idle, and the footprints of the jobs that hold memory, fit the budget.
static void limit_store(micsa_pool* pool, size_t used)
{
    std::lock_guard<std::mutex> hold(pool->store.lock);
    pool->store.limit = pool->budget > used ? pool->budget - used : 0;
    pool->store.trim(pool->store.limit);
}

static int pool_batch(micsa_pool* pool, int64_t sweeps)
{
    const int st = enqueue_batch(pool, sweeps);
    if (st)  // slices of drawn levels may have been planned and not launched
        for (auto& j : pool->jobs)
            if (j.batched && j.ctx) j.ctx->cdr_n = 0;
    return st;
}

int micsa_pool_step(micsa_pool* pool, int64_t sweeps, int32_t* running, int32_t* queued)
{
    if (!pool || sweeps < 0) return MICSA_EINVAL;
    // 1. retire jobs whose last chunk has finished on the device (a batch's
    // event is recorded again only after that batch has finished)
    for (auto& j : pool->jobs) {
        if (j.state != MICSA_JOB_RUNNING || j.ctx->k < j.ctx->sched.n_sweeps) continue;
        const bool fin = j.batched ? (j.last_batch < 0 || pool->batches > j.last_batch + 2 ||
                                      slot_free(pool->bev[j.last_batch & 1]))
                                   : (j.chunks == 0 || slot_free(j.ev[(j.chunks - 1) & 1]));
        if (!fin) continue;
        j.state = MICSA_JOB_DONE;
        if (j.batched) j.ctx->stream = pool->side;  // until it sweeps again (run_stream)
    }
    // 2. admit queued jobs in arrival order while they fit
    int32_t nrun = 0;
    for (auto& j : pool->jobs) nrun += j.state == MICSA_JOB_RUNNING;
    // what the queued jobs that fit now leave of the budget: from it a job may hold
    // more than its footprint
    size_t spare = pool->budget - std::min(pool->budget, pool->used);
    int64_t places = (int64_t)pool->max_running - nrun;
    for (const auto& j : pool->jobs) {
        if (j.state != MICSA_JOB_QUEUED) continue;
        if (places-- <= 0 || j.bytes > spare) break;
        spare -= j.bytes;
    }
    for (auto& j : pool->jobs) {
        if (j.state != MICSA_JOB_QUEUED) continue;
        if (nrun >= pool->max_running || pool->used + j.bytes > pool->budget) break;
        micsa_params pr = j.p;
        micsa_ctx* probe = nullptr;
        micsa_ctx like, shape;
        like.device = j.device;
        like.cus = j.cus;
        like.plan = j.plans.main;
        like.walk = j.plans.walk;
        std::copy(std::begin(j.plans.brief), std::end(j.plans.brief), like.brief);
        like.tile2 = j.tile2;
        if (const int st = setup_ctx(&shape, &pr, nullptr, &like)) return st;
        // as much as fits; the state's own arrays always do.  (The footprint has
        // reduction slots for one replica of each sample and no padding.)
        const size_t most = j.bytes + spare + (size_t)(shape.L - shape.p.n_samples) * kSlots * 8 + 4096;
        int fit = 0;
        while (fit < 2 && j.need[fit] > most) ++fit;
        shape.draw_room = j.draw_room[std::min(fit, 1)];
        shape.plan.ok = shape.plan.ok && fit < 2;
        const size_t charge = std::max(j.bytes, j.need[fit]);
        bool batched = batches(&shape);
        const int device = shape.device;
        if (batched && pool->side && pool->side_device != device) {
            if (hipStreamSynchronize(pool->side) != hipSuccess) return MICSA_EHIP;
            for (auto& o : pool->jobs)  // their reads go on where they swept
                if (o.ctx && o.ctx->stream == pool->side) o.ctx->stream = pool->stream;
            drop_stream(&pool->store, pool->side_device, pool->side);
            pool->side = nullptr;
        }
        if (batched && !pool->side) {
            if (take_stream(&pool->store, device, &pool->side) != hipSuccess) {
                (void)hipGetLastError();
                pool->side = nullptr;
                return MICSA_EHIP;
            }
            pool->side_device = device;
        }
        const auto own_stream = [&] {
            if (take_stream(&pool->store, device, &j.stream) == hipSuccess &&
                hipEventCreateWithFlags(&j.ev[0], hipEventDisableTiming) == hipSuccess &&
                hipEventCreateWithFlags(&j.ev[1], hipEventDisableTiming) == hipSuccess)
                return (int)MICSA_OK;
            (void)hipGetLastError();
            return (int)MICSA_EHIP;
        };
        if (!batched && own_stream() != MICSA_OK) {
            free_job_stream(pool, j, device);
            return MICSA_EHIP;
        }
        limit_store(pool, pool->used + charge);
        // A device that is fuller than the budget says: the job waits for those
        // that run, and alone does without what it lacks.
        const auto drop = [&] {
            if (j.ctx) micsa_destroy(j.ctx);
            j.ctx = nullptr;
            free_job_stream(pool, j, device);
            limit_store(pool, pool->used);
        };
        int st = create_ctx(&pr, batched ? pool->side : j.stream, &shape, most - std::min(most, j.need[fit] - ctx_bytes(&shape).home - ctx_bytes(&shape).work),
                            nrun == 0, &pool->store, &probe);
        if (st) {
            drop();
            if (st == MICSA_ENOMEM) break;  // retry next step
            return st;
        }
        j.ctx = probe;
        micsa_schedule cs{j.sched.kind, j.sched.period, j.sched.T0, j.sched.T1, j.sched.n_sweeps,
                          j.sched.table.empty() ? nullptr : j.sched.table.data(), (int64_t)j.sched.table.size()};
        if ((st = micsa_set_schedule(j.ctx, &cs))) {
            drop();
            if (st == MICSA_ENOMEM) break;
            return st;
        }
        if (batched) {
            if (hipStreamSynchronize(pool->side) != hipSuccess) return MICSA_EHIP;
            find_room(j.ctx, MICSA_ALGO_MICSA, kMscMinSweeps);
            batched = !j.ctx->no_room;
            if (batched) {
                j.ctx->stream = j.ctx->sweep_stream = pool->stream;
            } else {
                if (own_stream() != MICSA_OK) {
                    drop();
                    return MICSA_EHIP;
                }
                j.ctx->stream = j.stream;
            }
        }
        j.batched = batched;
        j.state = MICSA_JOB_RUNNING;
        size_t holds = j.need[fit] - ctx_bytes(&shape).home - ctx_bytes(&shape).work;
        for (const JobStore::Block& b : j.ctx->owned)
            if (b.p != j.ctx->d_dth) holds += b.bytes;
        j.charged = std::max(j.bytes, holds);
        spare -= std::min(spare, j.charged - j.bytes);
        pool->used += j.charged;
        limit_store(pool, pool->used);
        ++nrun;
    }
    // 3. enqueue the next chunk of sweeps of every running job with a free
    // chunk slot (at most two chunks in flight per job, and per batch).
    // Nothing waits for the device: the call returns once the work is queued.
    if (const int st = pool_batch(pool, sweeps)) return st;
    for (auto& j : pool->jobs) {
        if (j.state != MICSA_JOB_RUNNING || j.batched) continue;
        micsa_ctx* c = j.ctx;
        const int64_t n = std::min<int64_t>(sweeps, c->sched.n_sweeps - c->k);
        const int slot = (int)(j.chunks & 1);
        if (n <= 0 || !slot_free(j.ev[slot])) continue;
        const int st = micsa_sweep(c, MICSA_ALGO_MICSA, n);
        if (st) return st;
        if (hipEventRecord(j.ev[slot], j.stream) != hipSuccess) return MICSA_EHIP;
        ++j.chunks;
    }
    int32_t r = 0, q = 0;
    for (auto& j : pool->jobs) {
        r += j.state == MICSA_JOB_RUNNING;
        q += j.state == MICSA_JOB_QUEUED;
    }
    if (running) *running = r;
    if (queued) *queued = q;
    return MICSA_OK;
}

int micsa_pool_job_state(micsa_pool* pool, int64_t job, int32_t* state, int64_t* k)
{
    if (!pool) return MICSA_EINVAL;
    PoolJob* j = find_job(pool, job);
    if (!j) {
        if (job >= 1 && job < pool->next_id) {  // released
            if (state) *state = MICSA_JOB_RELEASED;
            if (k) *k = -1;
            return MICSA_OK;
        }
        return MICSA_EINVAL;
    }
    if (state) *state = j->state;
    if (k) *k = j->ctx ? j->ctx->k : 0;
    return MICSA_OK;
}

int micsa_pool_job_context(micsa_pool* pool, int64_t job, micsa_ctx** ctx)
{
    if (!pool || !ctx) return MICSA_EINVAL;
    PoolJob* j = find_job(pool, job);
    if (!j || !j->ctx) return MICSA_EINVAL;
    *ctx = j->ctx;
    return MICSA_OK;
}

int micsa_pool_release(micsa_pool* pool, int64_t job)
{
    if (!pool) return MICSA_EINVAL;
    for (size_t i = 0; i < pool->jobs.size(); ++i) {
        PoolJob& j = pool->jobs[i];
        if (j.id != job) continue;
        if (j.state != MICSA_JOB_DONE) return MICSA_EINVAL;
        const int device = j.ctx->device;
        limit_store(pool, pool->used - j.charged);
        micsa_destroy(j.ctx);  // synchronises the job's stream
        free_job_stream(pool, j, device);
        pool->used -= j.charged;
        pool->jobs.erase(pool->jobs.begin() + (long)i);
        if (pool->jobs.empty()) limit_store(pool, pool->budget);
        return MICSA_OK;
    }
    return MICSA_EINVAL;
}

}  // extern "C"
