// spx_host.hpp -- host-side plan object and error plumbing of libspx.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <cstring>
#include <string>
#include <type_traits>
#include <vector>

#include "../../include/spx.h"
#include "spx_device.hpp"

namespace spx {

void set_error(const std::string& msg);

#define SPX_HIP(call)                                                                                   \
    do {                                                                                                \
        hipError_t e_ = (call);                                                                         \
        if (e_ != hipSuccess) {                                                                         \
            ::spx::set_error(std::string("HIP error: ") + hipGetErrorString(e_) + " at " + __FILE__ + ":" + \
                             std::to_string(__LINE__));                                                 \
            return SPX_EDEVICE;                                                                         \
        }                                                                                               \
    } while (0)

#define SPX_TRY(call)                          \
    do {                                       \
        int r_ = (call);                       \
        if (r_ != SPX_OK) return r_;           \
    } while (0)

// FP64 constants of one (config, cathode) segment, in the chamber frame.
struct SegHost {
    int cfg, cath;
    double cat_c[3], cat_n[3], cat_u[3], cat_v[3], cat_R;
    double sub_c[3], sub_n[3], sub_u[3], sub_v[3], half_u, half_v, du, dv;
    int shape, nu, nv;
    double ch_R, zlo, zhi, z_mid;
    double rt_mu, rt_sig, PhiA, QB, dPhi;
    double Us, Emax, smax, Lambda;
    double Ms, Mg, mu_red, a_mm, eps_per_eV;
    double n_mm3, kT, vth, vg, E_th, lam_th;
    int gas_motion;
    double pressure;
    std::vector<double> rt_r, rt_d;   // measured racetrack nodes (empty: truncated normal)
    std::vector<spx_object> objs;     // absorbing objects of the run (chamber frame)
    double cosc[6];                   // emission law coefficients
    uint64_t N, bin_off, first_rec;
    double cost;          // relative expected work per particle (ticket ordering)
};

// A thermalised atom handed from the ballistic to the diffusive phase (FP32 48 B, FP64 80 B).
template <typename R> struct alignas(16) ThermRec {
    R x[3], xc[3];              // compensated position (chamber frame)
    R E;                        // energy at thermalisation (reported in the record)
    R lam;                      // the segment's lam_th ln 2 and Philox counter word: the two
    uint32_t cfgcat;            // numbers of the segment a diffusive step needs
    uint32_t pid;               // particle index within its segment (~0: empty slot)
    uint32_t seg;               // segment
    uint32_t e;                 // events taken so far
};
static_assert(sizeof(ThermRec<float>) == 48, "ThermRec layout");
static_assert(sizeof(ThermRec<double>) == 80, "ThermRec layout");

// Launch arguments of the transport kernels of a precision (one round = one chunk of the
// ticket space: the ballistic phase of every ticket, then the diffusive phase of the atoms
// it thermalised).
template <typename R> struct TransportArgs {
    const SegDev<R>* segs;
    TabDev<R> tab;
    const uint64_t* tfirst;     // [n_seg + 1] first ticket of each position in ticket order
    const uint32_t* torder;     // [n_seg] segment at each position
    ThermRec<R>* queue;         // thermalised atoms of the round (capacity >= tickets of a round)
    uint64_t* qstate;           // [QS_TICKETS] ballistic ticket counter, [QS_QUEUE] queue length,
                                // [QS_DIFFUSIVE] diffusive ticket counter
    uint64_t* times;            // whole kernel: ticks that sampled waves spent in either phase, start, end (nullable)
    unsigned long long* counts;
    unsigned long long* counters;
    spx_record* records;
    unsigned long long* arr_E;  // arrival energy histograms [n_seg][SPX_ARRIVAL_E_BINS] (nullable)
    unsigned long long* arr_A;  // arrival angle histograms [n_seg][SPX_ARRIVAL_A_BINS] (nullable with arr_E)
    unsigned long long* esum;   // per tally bin: arrival energies in units of 2^-24 eV (nullable with arr_E)
    const R* e_edges;           // [SPX_ARRIVAL_E_BINS + 1] energy edges, eV
    const R* c_edges;           // [SPX_ARRIVAL_A_BINS + 1] cos(k deg)
    uint64_t tbase;             // first ticket of the round
    uint64_t total;             // tickets of the round
    uint32_t k0, k1;            // Philox key (seed words)
    uint32_t cap;
    int32_t n_seg;
    int32_t n_simd;             // SIMDs of the device
    int32_t refill_min;         // diffusive phase: refill a wave's dead lanes once at least this many
    int32_t refill_ballistic;   // ballistic phase: the same threshold
    int32_t defer_min;          // diffusive phase: held steps a wave's surface tests wait for at least
    int32_t walk_idle;          // diffusive phase: ... and the idle rounds of the lanes that hold them
    uint32_t chunk_ballistic;   // ballistic phase: tickets a wave claims per atomic (whole kernel: tickets of a wave)
    uint32_t wave_slots;        // whole kernel: queue slots of a wave
    uint32_t n_bins;            // tally bins of the plan
    int32_t lds_counters;       // per-segment counters privatised in LDS
    int32_t lds_tally;          // whole tally privatised in LDS (u32 per bin)
    int32_t lds_arrivals;       // arrival histograms privatised in LDS (u32)
};

// Output buffers of one run (device pointers; all but counts and counters nullable).
struct Outputs {
    uint64_t* counts = nullptr;
    uint64_t* counters = nullptr;
    double* profiles = nullptr;
    spx_record* records = nullptr;
    uint64_t* arr_E = nullptr;
    uint64_t* arr_A = nullptr;
    uint64_t* esum = nullptr;
};

// Blocks of 256 threads that a launch may have: the threads of a grid have to fit 32 bits (a larger grid is
// not refused but cut off, and the rest of the work not done).
constexpr int64_t GRID_MAX = ((1ll << 32) - 1) / 256;
constexpr uint64_t ROUND_MAX = 1ull << 28;   // tickets per round: a 12.9 GB queue of thermalised atoms
// FP64 rounds: 1.3 GB of queue; where that much is not free, half the round, down to the smallest
constexpr uint64_t ROUND_MAX64 = 1ull << 24, ROUND_MIN64 = 1ull << 16;
constexpr uint64_t QUEUE_CHUNK = 64;         // queue slots a wave reserves per atomic
// exactly one lane per slot: a hand-over of up to 64 atoms continues into at most one fresh
// run, and a wave marks its unused reserved slots one per lane
static_assert(QUEUE_CHUNK == 64, "queue runs hold one slot per lane of a wave");
// The round's three counters (ballistic tickets, queue length, diffusive tickets) sit 256 bytes
// apart: every wave's claims and queue reservations are atomics on them, and on one cache line
// the two kinds of atomics of the ballistic phase would queue behind each other.  QS_TIMES: the times of
// the plan's last run in one kernel.
constexpr uint64_t QS_TICKETS = 0, QS_QUEUE = 32, QS_DIFFUSIVE = 64, QS_TIMES = 96, QSTATE_WORDS = 128;
constexpr uint64_t QUEUE_SLACK_WAVES = 8192;  // waves that may leave slots unused (32 per CU, 256 CUs)
constexpr size_t LDS_COUNTERS_MAX = 16384;   // bytes: up to 256 segments
constexpr int RT_MAX_NODES = 256;             // nodes of a measured racetrack profile
constexpr int OBJ_MAX_SEG = 32;               // absorbing objects of one (config, cathode) run
constexpr uint64_t TICKET_CHUNK = 128;       // queued atoms a diffusive wave claims per global atomic, at most
constexpr uint64_t TICKET_CHUNK_MIN = 8;     // tickets of either phase a wave claims per global atomic, at least
// launch tickets a ballistic wave claims per global atomic, at most: ballistic histories are
// short, so their waves come back for tickets often and small chunks queue them on the one
// counter; the chunk of a round is also kept small enough for every wave to take several
constexpr uint64_t TICKET_CHUNK_BALLISTIC_MAX = 512;
constexpr int DEFER_MIN = 8;                  // default: held diffusive steps that trigger a wave's surface tests
// Dead lanes a wave refills at, of a plan that is not tuned: four cathodes 6.13 ms (6.35 at 8 and 8, 6.12
// at 8 and 24), single target 35.8 (36.7, 36.9), half the 64-chamber sweep 93.5 (95.9, 95.2), 2.3e6
// atoms from four cathodes 1.29 (1.32, 1.28).
constexpr int REFILL = 4, REFILL_BALLISTIC = 16;
// Idle rounds of held lanes (summed over the lanes) that one pass of the surface tests is worth
// without absorbing objects.  Diffusive kernel, single target / four cathodes / half the 64-chamber
// sweep: 34.5 / 3.46 / 85.7 ms at 64, 33.9 / 3.37 / 84.0 at 128, 34.1 / 3.46 / 84.4 at 192, 35.9 /
// 3.82 / 88.4 at 400.
constexpr int WALK_IDLE = 128;
// The same for the FP64 walk, whose rounds cost as much as a test pass: 9e6 atoms at 0.5 / 0 / 2 Pa took
// 62.2 ms at 96 idle rounds, 60.4 at 64.
constexpr int WALK_IDLE64 = 64;
// Refill thresholds of the FP64 phases (four cathodes, 2.3e6 atoms: 4.95 ms with the ballistic phase
// refilled at 16 dead lanes, 4.66 at 24, 6.1 at 8; the diffusive phase differs by 1 % between 2 and 8).
constexpr int REFILL64 = 2, REFILL_BALLISTIC64 = 24;
constexpr size_t LDS_TALLY_MAX = 49152;      // bytes: up to 12288 bins
constexpr size_t LDS_ARRIVALS_MAX = 4096;     // bytes: arrival histograms of up to 6 segments

// One kernel launch of a run with its arguments stored by value.  A run of the batched path
// is a list of these: enqueued on a stream as they are made, or made into the kernel nodes of
// a graph whose arguments can later be replaced in the instantiated graph (a new seed or new
// output buffers then need no new graph).
struct KLaunch {
    const void* func = nullptr;
    dim3 grid{1, 1, 1}, block{1, 1, 1};
    uint32_t smem = 0;
    int phase = 0;              // 1: the ballistic kernel of a round, 2: its diffusive kernel, 3: both in one, else 0
    int n_args = 0;
    uint16_t off[8] = {};
    uint16_t last_size = 0;
    alignas(16) unsigned char buf[384] = {};

    template <typename T> void arg(const T& v)
    {
        static_assert(std::is_trivially_copyable<T>::value, "kernel arguments are copied bytewise");
        size_t o = n_args ? (size_t)off[n_args - 1] + last_size : 0;
        o = (o + alignof(T) - 1) / alignof(T) * alignof(T);
        if (n_args >= 8 || o + sizeof(T) > sizeof(buf)) {
            n_args = -1;              // reported by the sinks: never launched
            return;
        }
        std::memcpy(buf + o, &v, sizeof(T));
        off[n_args++] = (uint16_t)o;
        last_size = (uint16_t)sizeof(T);
    }
    // pointers to the stored arguments, as hipLaunchKernel and graph kernel nodes take them
    void pointers(void** p) const
    {
        for (int i = 0; i < n_args; ++i) p[i] = const_cast<unsigned char*>(buf) + off[i];
    }
    // same kernel and launch geometry (the arguments may differ)
    bool same_shape(const KLaunch& o) const
    {
        return func == o.func && grid.x == o.grid.x && block.x == o.block.x && smem == o.smem && phase == o.phase &&
               n_args == o.n_args;
    }
    bool same_args(const KLaunch& o) const { return std::memcmp(buf, o.buf, sizeof(buf)) == 0; }
};

// Receiver of the launches of a run, in order.
struct LaunchSink {
    virtual int put(const KLaunch& k) = 0;
    virtual ~LaunchSink() = default;
};

// Launch geometry of the two persistent transport kernels, thresholds of all.
struct Shape {
    int blocks = 0, blocks_diff = 0, threads = 256, refill_min = REFILL, refill_ballistic = REFILL_BALLISTIC,
        defer_min = DEFER_MIN;
    bool whole = true;          // rounds of up to whole_limit() take both phases in one kernel
};

// Queue of thermalised atoms and ticket counters a run works in: the plan's own allocation, or
// caller-independent static scratch.  Rounds hold at most round_max tickets.
struct QueueMem {
    void* queue = nullptr;       // ThermRec<R> of the plan's precision
    uint64_t cap = 0;            // slots
    uint64_t* qstate = nullptr;  // QSTATE_WORDS words: the round's counters
    uint64_t* times = nullptr;   // qstate + QS_TIMES in runs that spx_phase_times answers for
    uint64_t round_max = ROUND_MAX;
};

}  // namespace spx

struct spx_plan {
    int device = 0;
    spx_params params{};
    std::vector<spx::SegHost> seg;
    int n_seg = 0;
    bool has_objects = false;               // a segment has absorbing objects
    uint64_t n_objects = 0;                 // objects over all segments
    double p_lo = 0.0, p_hi = 0.0;          // least and greatest pressure of a segment
    uint64_t n_bins_total = 0, n_particles_total = 0;
    std::vector<uint64_t> h_bin_off, h_first;
    std::vector<double> h_betamax;          // FP64 beta_max table copy (host)
    std::vector<double> seg_norm;           // 1 / (N * bin area) per segment

    hipStream_t work_stream = nullptr;
    double* d_theta64 = nullptr;
    double* d_betamax64 = nullptr;
    float* d_theta32 = nullptr;
    float* d_betamax32 = nullptr;
    spx::SegDev<float>* d_seg32 = nullptr;
    spx::SegDev<double>* d_seg64 = nullptr;
    float* d_edges32 = nullptr;               // arrival bin edges: energy [61] then cos [91]
    double* d_edges64 = nullptr;
    spx::ObjDev<float>* d_obj32 = nullptr;    // absorbing objects of all segments
    spx::ObjDev<double>* d_obj64 = nullptr;
    spx::RtNode<float>* d_rt32 = nullptr;     // measured racetracks of all segments
    spx::RtNode<double>* d_rt64 = nullptr;
    uint64_t* d_tfirst = nullptr;
    uint32_t* d_torder = nullptr;
    unsigned char* d_queue = nullptr;       // thermalised atoms of a round (ThermRec of the precision)
    uint64_t queue_cap = 0;                 // slots
    uint64_t round_max = spx::ROUND_MAX;    // tickets per round, at most
    spx::Shape shape64;                     // launch of the FP64 kernels
    uint64_t* d_qstate = nullptr;           // ticket counters and queue length
    std::vector<hipEvent_t> phase_events;   // recorded in the graph: round start, ballistic end, diffusive end
    uint64_t* d_bin_off = nullptr;          // [n_seg + 1]
    double* d_seg_norm = nullptr;           // [n_seg]
    uint64_t n_tickets = 0;

    int blocks = 0, threads = 256, refill_min = spx::REFILL, refill_ballistic = spx::REFILL_BALLISTIC,
        defer_min = spx::DEFER_MIN;
    int blocks_diff = 0;                    // grid of the diffusive kernel: blocks, capped at its resident limit
    int max_blocks_per_cu = 0, n_cu = 0;

    hipGraph_t graph = nullptr;
    hipGraphExec_t graph_exec = nullptr;
    std::vector<spx::KLaunch> graph_launches;   // the kernel nodes' launches, in graph order
    std::vector<hipGraphNode_t> graph_nodes;     // ... and their nodes
    uint64_t graph_instantiations = 0;           // graphs built and instantiated
    uint64_t graph_updates = 0;                  // kernel nodes whose arguments were replaced
    // stream order between runs on different streams: recorded after each run, waited for by
    // the next run or autotune (all of them share the plan's queue and ticket counters)
    hipEvent_t done_event = nullptr;
    bool done_recorded = false;
};

namespace spx {
using Plan = spx_plan;
int build_tables(Plan* P);
// events (nullable, not while capturing): 3 per round, recorded at the round's start, after
// its ballistic phase and after its diffusive phase.
// The launches of one run over tickets [0, total) of `tfirst` in rounds of at most
// q.round_max tickets: zero the outputs, per round reset / ballistic / diffusive, normalise.
// R: the plan's precision.
template <typename R>
int build_transport(Plan* P, uint64_t seed, const Outputs& o, const uint64_t* tfirst, uint64_t total,
                    const Shape& sh, const QueueMem& q, LaunchSink& sink);
// A sink that launches on `st`; with `events` (3 per round, not while capturing) it records one
// before each ballistic kernel, one after it and one after the diffusive kernel (a kernel for both
// phases: one before it and both others after it).
struct StreamSink : LaunchSink {
    hipStream_t st;
    const hipEvent_t* events;
    size_t round = 0;
    StreamSink(hipStream_t s, const hipEvent_t* e) : st(s), events(e) {}
    int put(const KLaunch& k) override;
};
uint64_t rounds_of(uint64_t total, uint64_t round_max = ROUND_MAX);
// Tickets of a round that takes both phases in one kernel, at most; 0: rounds take a kernel per phase.
uint64_t whole_limit(const Plan* P, const Shape& sh);
// The plan's current launch geometry and thresholds.
Shape plan_shape(const Plan* P);
// Launch geometry of the FP64 kernels of a plan.
int shape_transport64(Plan* P);
// Arrival bin edges in double (as the FP64 path uses them); the FP32 path rounds them to float.
void arrival_edges(double* e_edges, double* c_edges);
// resident blocks per CU of the ballistic and of the diffusive kernel at this block size
int occupancy_transport32(const Plan* P, int threads, int* bpc_ballistic, int* bpc_diffusive);
}  // namespace spx
