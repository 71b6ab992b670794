// transport.hip -- the transport kernels of both precisions and their tallies.
//
// Every (configuration, cathode) segment of a plan runs in rounds of at most ROUND_MAX (FP64:
// ROUND_MAX64) tickets, a long round as two persistent launches, another as one (whole_kernel).  (FP64
// runs in a caller's graph: k_plain64.)
// The ballistic phase takes every ticket of the round from its launch through its flights and
// collisions; an atom that ends on a surface (or escapes) is finished there, an atom that
// thermalises is handed over to a queue in HBM (48 B, in FP64 80 B, with the two numbers of its
// segment a step needs).  The diffusive phase then runs the walks of the queued atoms.  Each lane
// holds one atom in registers; when lanes die, the wave claims a run of tickets with a single
// atomic (ballot + mbcnt prefix gives each dead lane its ticket).  Splitting the history at thermalisation keeps every lane of a wave in the same
// kind of event: new atoms (ballistic) and walkers (diffusive) never share a wave.  The
// random numbers are keyed by (seed, segment, particle, event), so the result does not
// depend on which lane, wave or launch ran an atom, nor on the queue order.  Deposits go
// to a per-block LDS tally (or 64-bit global atomics when it does not fit); per-segment
// counters are accumulated in registers while a lane stays in one segment.
//
// The kernels are written once for R = float and R = double.  FP32 walks add their steps to an offset
// from the centre of a clearance ball, FP64 walks to the compensated position itself, and in both a
// step is tested against the surfaces only where it leaves the ball, so that FP64 outcomes are those of
// testing every step, bit for bit.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "spx_host.hpp"

namespace spx {

__device__ __forceinline__ void add_counters(unsigned long long* C, const uint32_t* acc)
{
#pragma unroll
    for (int i = 0; i < N_COUNTERS; ++i)
        if (acc[i]) atomicAdd(&C[i], (unsigned long long)acc[i]);
}

template <typename R>
__device__ __forceinline__ void write_record(spx_record* rec, const SegDev<R>& s, uint32_t pid, const Particle<R>& p,
                                             const Term& t)
{
    spx_record r;
    r.x = (double)p.x[0] - (double)p.xc[0];
    r.y = (double)p.x[1] - (double)p.xc[1];
    r.z = ((double)p.x[2] - (double)p.xc[2]) + (double)s.z_mid;
    r.E = (double)p.E;
    r.state = (uint32_t)t.state;
    r.bin = t.state == HIT_DEPOSITED ? (uint32_t)t.bin : 0xFFFFFFFFu;
    r.events = p.e;
    r.diffusive = p.ndiff;
    r.cos_in = (double)t.cos_in;
    rec[s.first_rec + pid] = r;
}

// Per-lane bookkeeping of the batched kernel: counters of the lane's current segment,
// flushed to the block's LDS counters (or HBM) when the lane moves to another segment.
// WALKS: of the diffusive phase, where every history that ends had thermalised, so that this counter
// is the sum of the endings and needs no register.
template <bool WALKS> struct LaneAcc {
    int seg = -1;
    uint32_t c[N_COUNTERS] = {};
};

struct BlockTally {
    unsigned long long* lcnt;   // LDS per-segment counters (valid if a.lds_counters)
    uint32_t* ltally;           // LDS tally (valid if a.lds_tally)
    uint32_t* larr;             // LDS arrival histograms [n_seg][E bins + A bins] (valid if a.lds_arrivals)
};

constexpr int ARR_BINS = SPX_ARRIVAL_E_BINS + SPX_ARRIVAL_A_BINS;

// Arrival tallies of one deposit: energy and angle histograms of its segment, energy sum of
// its tally bin.
template <typename R>
__device__ __forceinline__ void tally_arrival(const TransportArgs<R>& a, const BlockTally& bt, int seg, uint64_t bin,
                                              double E, double cos_in)
{
    const int be = energy_bin(a.e_edges, (R)E);
    const int ba = angle_bin(a.c_edges, (R)cos_in);
    if (a.lds_arrivals) {
        atomicAdd(&bt.larr[seg * ARR_BINS + be], 1u);
        atomicAdd(&bt.larr[seg * ARR_BINS + SPX_ARRIVAL_E_BINS + ba], 1u);
    } else {
        atomicAdd(&a.arr_E[(size_t)seg * SPX_ARRIVAL_E_BINS + be], 1ull);
        atomicAdd(&a.arr_A[(size_t)seg * SPX_ARRIVAL_A_BINS + ba], 1ull);
    }
    atomicAdd(&a.esum[bin], energy_units(E));
}

template <typename R, bool WALKS>
__device__ __forceinline__ void flush_acc(const TransportArgs<R>& a, const BlockTally& bt, LaneAcc<WALKS>& acc)
{
    if (acc.seg < 0) return;
    if (WALKS) acc.c[C_THERMALIZED] = acc.c[C_DEPOSITED] + acc.c[C_WALL] + acc.c[C_ESCAPED];
    if (a.lds_counters) {
#pragma unroll
        for (int i = 0; i < N_COUNTERS; ++i)
            if (acc.c[i]) atomicAdd(&bt.lcnt[acc.seg * N_COUNTERS + i], (unsigned long long)acc.c[i]);
    } else {
        add_counters(a.counters + (size_t)acc.seg * N_COUNTERS, acc.c);
    }
#pragma unroll
    for (int i = 0; i < N_COUNTERS; ++i) acc.c[i] = 0;
}

// End of a history: counters, tally, optional record; the lane becomes free.
template <bool ARR, typename R, bool WALKS>
__device__ __forceinline__ void terminate(const TransportArgs<R>& a, const BlockTally& bt, const SegDev<R>& s,
                                          uint32_t pid, Particle<R>& p, const Term& t, LaneAcc<WALKS>& acc)
{
    // static indices only: the counters stay in registers
    acc.c[C_DEPOSITED] += (t.state == HIT_DEPOSITED) ? 1u : 0u;
    acc.c[C_WALL] += (t.state == HIT_WALL) ? 1u : 0u;
    acc.c[C_ESCAPED] += (t.state == HIT_ESCAPED) ? 1u : 0u;
    if (WALKS) acc.c[C_DIFFUSIVE] += p.ndiff;
    else acc.c[C_COLLISIONS] += p.ncoll;
    // the FP64 path counts every diffusive step: those that ended in the gas and the last one
    // (unless the history stopped at the event cap); the FP32 path counts at the test
    if (WALKS && std::is_same<R, double>::value) acc.c[C_TESTED] += p.ndiff + (t.state != HIT_ESCAPED ? 1u : 0u);
    if (t.state == HIT_DEPOSITED) {
        const uint64_t b = s.bin_off + (uint64_t)t.bin;
        if (a.lds_tally) atomicAdd(&bt.ltally[b], 1u);
        else atomicAdd(&a.counts[b], 1ull);
        if (ARR) tally_arrival(a, bt, acc.seg, b, (double)p.E, (double)t.cos_in);
    }
    if (a.records) write_record(a.records, s, pid, p, t);
    p.st = ST_DEAD;
}

// Tickets a wave claims at once out of `total`: at most `most`, in a small run the share of one SIMD.
// There the phase lasts as long as its longest histories, which step fastest alone on a SIMD: with
// 128 tickets a claim, 1e4 atoms (one target, 0.5 Pa) ran on 80 waves of 1024 SIMDs' (0.147 +
// 0.392 ms ballistic + diffusive; a SIMD's share: 0.126 + 0.265), 1e5 in 0.156 + 0.453 (0.153 +
// 0.411).  Sharing among two or four times as many waves: 0.130 + 0.298 and 0.130 + 0.319; 0.159 +
// 0.430 and 0.202 + 0.481.
__host__ __device__ __forceinline__ uint64_t chunk_of(uint64_t total, int n_simd, uint64_t most)
{
    const uint64_t share = (total + (uint64_t)n_simd - 1) / (uint64_t)n_simd;
    return share < TICKET_CHUNK_MIN ? TICKET_CHUNK_MIN : share < most ? share : most;
}

// Number of set bits of the wave-wide mask m in the lanes below this one (mbcnt).
__device__ __forceinline__ uint64_t lanes_below(uint64_t m)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Lane 0's value, in scalar registers (the whole wave is here).
__device__ __forceinline__ uint64_t first_lane(uint64_t v)
{
    return ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(v >> 32)) << 32) |
           (uint32_t)__builtin_amdgcn_readfirstlane((int)v);
}

// Wave-private run of tickets [tk, tk_end), claimed CHUNK at a time from a global counter with
// one atomic, so that refills rarely touch the counter.  A round's tickets and queue slots fit 32 bits
// (at most 2^28 of them).
struct Tickets {
    uint32_t tk = 0, tk_end = 0;
    bool drained = false;     // wave-uniform: the ticket space is exhausted
};
constexpr uint32_t NO_TICKET = ~0u;
static_assert(ROUND_MAX + QUEUE_SLACK_WAVES * QUEUE_CHUNK < NO_TICKET, "tickets of a round fit 32 bits");

// Tickets for the dead lanes `dead` of the wave: consecutive tickets of the wave's run in lane
// order.  Returns this lane's ticket, or NO_TICKET when it gets none.  OWN: the wave has the run it
// started with and claims no other.
template <bool OWN, bool SCALAR>
__device__ __forceinline__ uint32_t claim(Tickets& T, uint64_t* counter, uint32_t chunk, uint32_t total, uint64_t dead,
                                          int lane)
{
    if (!OWN && T.tk == T.tk_end) {
        unsigned long long base = 0;
        if (lane == 0) base = atomicAdd((unsigned long long*)counter, (unsigned long long)chunk);
        base = SCALAR ? first_lane(base) : __shfl(base, 0);
        if (base >= total) {
            T.drained = true;
            return NO_TICKET;
        }
        T.tk = (uint32_t)base;
        T.tk_end = total - T.tk > chunk ? T.tk + chunk : total;
    }
    const uint32_t n_dead = (uint32_t)__popcll(dead);
    const uint32_t avail = T.tk_end - T.tk;
    const uint32_t take = avail < n_dead ? avail : n_dead;
    const uint32_t base = T.tk;
    T.tk += take;
    if (OWN) T.drained = T.tk == T.tk_end;
    const uint32_t rank = (uint32_t)lanes_below(dead);
    return (((dead >> lane) & 1ull) && rank < take) ? base + rank : NO_TICKET;
}

// The queued atoms of the waves of a block (both phases in one kernel), walked by whichever of its waves is
// free: slots [next, end) of each wave, end 0 until its ballistic phase is over.
struct BlockQueue {
    uint32_t* next;
    uint32_t* end;
    uint32_t wave, waves;
};

// Slots for the dead lanes of the wave, as claim: from the list it took from last, its own at first, or the
// next one that holds any.  Lists that are not there yet are left to their waves: nobody waits.
__device__ __forceinline__ uint32_t claim_shared(Tickets& T, BlockQueue& B, uint64_t dead, int lane)
{
    const uint32_t n_dead = (uint32_t)__popcll(dead);
    for (uint32_t tried = 0; tried < B.waves; ++tried) {
        const uint32_t end = (uint32_t)__builtin_amdgcn_readfirstlane(
            (int)__hip_atomic_load(&B.end[B.wave], __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP));
        // (an end of 0 has to fail here: next means nothing yet)
        if ((uint32_t)__builtin_amdgcn_readfirstlane((int)__hip_atomic_load(&B.next[B.wave], __ATOMIC_RELAXED,
                                                                            __HIP_MEMORY_SCOPE_WORKGROUP)) < end) {
            uint32_t base = 0;
            if (lane == 0)
                base = __hip_atomic_fetch_add(&B.next[B.wave], n_dead, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            base = (uint32_t)__builtin_amdgcn_readfirstlane((int)base);
            if (base < end) {
                const uint32_t rank = (uint32_t)lanes_below(dead);
                return ((dead >> lane) & 1ull) && rank < end - base ? base + rank : NO_TICKET;
            }
        }
        B.wave = B.wave + 1 < B.waves ? B.wave + 1 : 0;
    }
    T.drained = true;
    return NO_TICKET;
}

// Dynamic LDS: per-segment counters (u64, when lds_counters), the tally (u32, when lds_tally), the
// arrival histograms (u32, when lds_arrivals).
template <typename R>
__device__ __forceinline__ void lds_setup(const TransportArgs<R>& a, BlockTally& bt, unsigned long long* lds)
{
    bt.lcnt = lds;
    bt.ltally = (uint32_t*)(lds + (a.lds_counters ? (size_t)a.n_seg * N_COUNTERS : 0));
    bt.larr = bt.ltally + (a.lds_tally ? a.n_bins : 0u);
    const uint32_t words = (uint32_t)(bt.larr - (uint32_t*)lds) + (a.lds_arrivals ? (uint32_t)(a.n_seg * ARR_BINS) : 0u);
    for (uint32_t i = threadIdx.x; i < words / 4; i += blockDim.x) ((uint4*)lds)[i] = make_uint4(0u, 0u, 0u, 0u);
    if (threadIdx.x < (words & 3u)) ((uint32_t*)lds)[(words & ~3u) + threadIdx.x] = 0;
    __syncthreads();
}

template <typename R>
__device__ __forceinline__ void lds_flush(const TransportArgs<R>& a, const BlockTally& bt)
{
    __syncthreads();
    if (a.lds_counters)
        for (int i = threadIdx.x; i < a.n_seg * N_COUNTERS; i += blockDim.x)
            if (bt.lcnt[i]) atomicAdd(&a.counters[i], bt.lcnt[i]);
    if (a.lds_tally) {
        constexpr uint32_t U = 8;       // LDS reads in flight
        for (uint32_t i0 = threadIdx.x; i0 < a.n_bins; i0 += U * blockDim.x) {
            uint32_t v[U];
#pragma unroll
            for (uint32_t k = 0; k < U; ++k) {
                const uint32_t i = i0 + k * blockDim.x;
                v[k] = i < a.n_bins ? bt.ltally[i] : 0u;
            }
#pragma unroll
            for (uint32_t k = 0; k < U; ++k)
                if (v[k]) atomicAdd(&a.counts[i0 + k * blockDim.x], (unsigned long long)v[k]);
        }
    }
    if (a.lds_arrivals)
        for (int i = threadIdx.x; i < a.n_seg * ARR_BINS; i += blockDim.x)
            if (bt.larr[i]) {
                const int k = i / ARR_BINS, j = i % ARR_BINS;
                unsigned long long* dst = j < SPX_ARRIVAL_E_BINS
                                              ? &a.arr_E[(size_t)k * SPX_ARRIVAL_E_BINS + j]
                                              : &a.arr_A[(size_t)k * SPX_ARRIVAL_A_BINS + (j - SPX_ARRIVAL_E_BINS)];
                atomicAdd(dst, (unsigned long long)bt.larr[i]);
            }
}

// Wave-private run of queue slots [q, q_end), reserved QUEUE_CHUNK at a time with one
// atomic on the queue length.  Slots a wave leaves unused are marked empty when it exits.
struct QRun {
    uint64_t q = 0, q_end = 0;
};

// Lanes whose atom thermalised in the last flight hand it to the diffusive queue and become
// free.  Slots come from the wave's run (a hand-over may continue into a fresh run).  Their
// collisions are counted here; thermalisation itself is counted when the walk ends.
template <typename R>
__device__ __forceinline__ void hand_over(const TransportArgs<R>& a, const SegDev<R>& S, uint32_t pid, int seg,
                                          Particle<R>& p, LaneAcc<false>& acc, QRun& Q, int lane)
{
    const uint64_t T = __ballot(p.st == ST_DIFFUSIVE);
    if (T == 0) return;
    const uint64_t n = (uint64_t)__popcll(T);
    const uint64_t rem = Q.q_end - Q.q;
    uint64_t fresh = 0;
    if (rem < n) {
        unsigned long long b = 0;
        if (lane == 0) b = atomicAdd((unsigned long long*)&a.qstate[QS_QUEUE], (unsigned long long)QUEUE_CHUNK);
        fresh = first_lane(b);
    }
    if (p.st == ST_DIFFUSIVE) {
        const uint64_t rank = lanes_below(T);
        const uint64_t slot = rank < rem ? Q.q + rank : fresh + (rank - rem);   // < queue capacity
        ThermRec<R> r;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            r.x[i] = p.x[i];
            r.xc[i] = p.xc[i];
        }
        r.E = p.E;
        r.pid = pid;
        r.seg = (uint32_t)seg;
        r.e = p.e;
        r.lam = S.lam_l2;
        r.cfgcat = S.cfgcat;
        a.queue[slot] = r;
        acc.c[C_COLLISIONS] += p.ncoll;
        p.st = ST_DEAD;
    }
    if (rem < n) {
        Q.q = fresh + (n - rem);
        Q.q_end = fresh + QUEUE_CHUNK;
    } else {
        Q.q += n;
    }
}

// Mark the wave's unused reserved slots as empty (pid ~0).
template <typename R>
__device__ __forceinline__ void close_run(const TransportArgs<R>& a, const QRun& Q, int lane)
{
    if (Q.q + (uint64_t)lane < Q.q_end) a.queue[Q.q + lane].pid = 0xFFFFFFFFu;
}

// A history that ended in the ballistic phase waits for the wave's next refill point, where the
// ended histories and the thermalised atoms of the wave are settled together (a lane would idle
// until then anyway): its outcome is packed into the clearance-radius register, unused in this
// phase, as state | bin << 2.
constexpr int ST_ENDED = 3;

__device__ __forceinline__ float pack_end(float, uint32_t bits) { return __uint_as_float(bits); }
__device__ __forceinline__ double pack_end(double, uint32_t bits) { return __hiloint2double(0, (int)bits); }
__device__ __forceinline__ uint32_t end_bits(float r2) { return __float_as_uint(r2); }
__device__ __forceinline__ uint32_t end_bits(double r2) { return (uint32_t)__double2loint(r2); }
template <typename R> __device__ __forceinline__ void mark_ended(Particle<R>& p, const Term& t)
{
    p.st = ST_ENDED;
    p.r2 = pack_end((R)0, (uint32_t)t.state | ((uint32_t)(t.bin < 0 ? 0 : t.bin) << 2));
}

// Settle the wave's ended histories (counters, tally, record) and queue its thermalised atoms.
// The incidence cosine of a deposit is recomputed from its direction, with the operations of
// hit_term.
template <bool ARR, typename R>
__device__ __forceinline__ void settle_ballistic(const TransportArgs<R>& a, const BlockTally& bt,
                                                 const SegDev<R>* __restrict__ segs, uint32_t pid, int seg,
                                                 Particle<R>& p, LaneAcc<false>& acc, QRun& Q, int lane)
{
    if (__ballot(p.st == ST_ENDED) != 0 && p.st == ST_ENDED) {
        const SegDev<R>& s = segs[seg];
        const uint32_t bits = end_bits(p.r2);
        Term t;
        t.state = (int)(bits & 3u);
        t.bin = t.state == HIT_DEPOSITED ? (int)(bits >> 2) : -1;
        t.cos_in = t.state == HIT_DEPOSITED ? (float)(-dot3(p.d, s.sub_n)) : 0.f;
        terminate<ARR>(a, bt, s, pid, p, t, acc);
    }
    if (__ballot(p.st == ST_DIFFUSIVE) != 0) hand_over(a, segs[seg], pid, seg, p, acc, Q, lane);
}

// Ballistic flights of the lanes in `mine`, all of segment S (uniform: its constants stay in scalar
// registers) until the wave should refill (lanes that ended, thermalised or are free count) or
// none of them flies.
template <typename O, typename R>
__device__ __forceinline__ void ballistic_loop(const TransportArgs<R>& a, const SegDev<R>* S, uint32_t pid,
                                               Particle<R>& p, bool mine, bool drained)
{
    for (;;) {
        // the FP64 constants do not fit the scalar registers: read again for every flight (an empty
        // asm hides that the pointer is the same), not kept across flights in spilled vector registers
        if (std::is_same<R, double>::value) asm volatile("" : "+s"(S));
        if (mine && p.st == ST_BALLISTIC) {
            const Term t = step_mode<O>(*S, a.tab, a.k0, a.k1, pid, a.cap, p);
            if (t.state != HIT_NONE) mark_ended(p, t);
        }
        if (__ballot(mine && p.st == ST_BALLISTIC) == 0) break;
        if (!drained && __popcll(__ballot(p.st != ST_BALLISTIC)) >= a.refill_ballistic) break;
    }
}

// Histories of lanes at the event cap (rare) escape, ended one segment at a time.
template <bool ARR, typename R>
__device__ __forceinline__ void escape_capped(const TransportArgs<R>& a, const BlockTally& bt,
                                              const SegDev<R>* __restrict__ segs, int seg, uint32_t pid,
                                              Particle<R>& p, LaneAcc<true>& acc, bool capped)
{
    for (uint64_t C = __ballot(capped); C != 0;) {
        const int sL = __builtin_amdgcn_readlane(seg, __ffsll((unsigned long long)C) - 1);
        const bool mine = capped && seg == sL;
        C &= ~__ballot(mine);
        if (mine) {
            capped = false;
            p.ndiff = p.e - p.ndiff;
            terminate<ARR>(a, bt, segs[sL], pid, p, Term{HIT_ESCAPED, -1, 0.f}, acc);
        }
    }
}

// The held steps of the wave, tested together, each lane with its own segment's geometry.  (A second copy of the
// test, for lanes of one segment with the geometry in scalar registers, was slower: half the 64-chamber
// sweep 93.5 ms with it, 92.2 without.)
template <bool ARR, bool OBJ, typename R>
__device__ __forceinline__ void resolve_held(const TransportArgs<R>& a, const BlockTally& bt,
                                             const SegDev<R>* __restrict__ segs, int seg, uint32_t pid,
                                             Particle<R>& p, Walk<R>& wk, LaneAcc<true>& acc, bool held)
{
    if (std::is_same<R, float>::value) acc.c[C_TESTED] += held ? 1u : 0u;
    if (held) {
        const SegDev<R>& S = segs[seg];
        GeoOf<OBJ, R> geo(S);
        const Term t = diffusive_resolve(S, geo, p, wk, std::conditional_t<OBJ, OwnObjects, NoObjects>());
        if (t.state != HIT_NONE) {
            p.ndiff = p.e - p.ndiff - 1u;
            terminate<ARR>(a, bt, S, pid, p, t, acc);
        }
    }
}

// Diffusive steps of the wave's walkers with deferred surface tests: groups of steps (walk_group),
// the steps that left their balls tested together after each.  Walkers within a group's length of
// the event cap are rare: while the wave has one, it takes single steps.  Returns when the wave
// should refill, has no walker left, or walks its last ones cooperatively; no step is held then.
template <bool ARR, bool OBJ, typename R>
__device__ __forceinline__ void diffusive_loop(const TransportArgs<R>& a, const BlockTally& bt,
                                               const SegDev<R>* __restrict__ segs, int seg, R lam_l2,
                                               uint32_t cfgcat, uint32_t pid, Particle<R>& p, Walk<R>& wk,
                                               LaneAcc<true>& acc, bool drained)
{
    constexpr uint32_t REACH = 2 * WALK_ADVANCES + 1;     // events a group takes at most
    const uint32_t far = a.cap > REACH ? a.cap - REACH : 0u;
    uint64_t M = __ballot(p.st == ST_DIFFUSIVE);
    for (;;) {
        bool held = false;
        if (__ballot(p.st == ST_DIFFUSIVE && p.e >= far) == 0) {
            if (p.st == ST_DIFFUSIVE) {
                const int A = __popcll(M);
                held = walk_group(lam_l2, cfgcat, a.k0, a.k1, pid, A, a.defer_min < A ? a.defer_min : A, a.walk_idle,
                                  p, wk);
            }
        } else {
            const bool walks = p.st == ST_DIFFUSIVE;
            escape_capped<ARR>(a, bt, segs, seg, pid, p, acc, walks && p.e >= a.cap);
            if (p.st == ST_DIFFUSIVE) held = diffusive_single(lam_l2, cfgcat, a.k0, a.k1, pid, p, wk);
        }
        if (__ballot(held) != 0) resolve_held<ARR, OBJ>(a, bt, segs, seg, pid, p, wk, acc, held);
        M = __ballot(p.st == ST_DIFFUSIVE);
        if (M == 0 || (!drained && __popcll(__ballot(p.st == ST_DEAD)) >= a.refill_min) ||
            (drained && __popcll(M) <= Walk<R>::COOP))
            break;
    }
}

// Ballistic phase: every ticket of the round (WHOLE: of the run T that the wave starts with, its queue slots
// from Q.q on), from launch until the atom ends on a surface, escapes, or thermalises (then it is queued for the
// diffusive phase).  LIMITED: the slots may not hold them all; it ends while the lanes' atoms still fit.
// Returns the wave's next free slot and its next ticket.
template <bool ARR, bool OBJ, bool WHOLE, bool LIMITED, typename R>
__device__ __forceinline__ QRun ballistic_phase(TransportArgs<R>& a, const BlockTally& bt,
                                                const SegDev<R>* __restrict__ segs, Tickets T, QRun Q, int lane)
{
    using O = std::conditional_t<OBJ, OwnObjects, NoObjects>;
    Particle<R> p;
    p.st = ST_DEAD;
    p.e = p.ndiff = p.ncoll = 0;
    uint32_t pid = 0;
    int seg = 0;
    LaneAcc<false> acc;
    int cur_pos = 0, last_pos = 0;        // wave-uniform current position in ticket order ...
    uint64_t cur_lo = 0, cur_hi = 0;      // ... and its ticket range (empty until the first refill)
    int cur_seg = 0;                      // ... and its segment
    for (;;) {
        settle_ballistic<ARR>(a, bt, segs, pid, seg, p, acc, Q, lane);
        const uint64_t dead = __ballot(p.st == ST_DEAD);
        const int n_dead = __popcll(dead);
        const bool drained = T.drained || (LIMITED && Q.q_end - Q.q < 64);
        if (!drained && n_dead > 0 && (n_dead >= a.refill_ballistic || n_dead == 64)) {
            const uint32_t my = claim<WHOLE, true>(T, &a.qstate[QS_TICKETS], a.chunk_ballistic, (uint32_t)a.total,
                                                   dead, lane);
            if (my != NO_TICKET) {
                const uint64_t g = a.tbase + my;
                // the ticket's position in ticket order: the wave's current one (tickets of a
                // run are consecutive, segments long), else a binary search of the prefix table
                int lo = cur_pos;
                if (!(g >= cur_lo && g < cur_hi)) {
                    lo = 0;
                    int hi = a.n_seg;
                    while (hi - lo > 1) {
                        const int mid = (lo + hi) >> 1;
                        if (a.tfirst[mid] <= g) lo = mid; else hi = mid;
                    }
                }
                last_pos = lo;
                const int sg = (int)a.torder[lo];
                pid = (uint32_t)(g - a.tfirst[lo]);
                if (sg != acc.seg) {
                    flush_acc(a, bt, acc);
                    acc.seg = sg;
                }
                seg = sg;
                start(segs[seg], a.k0, a.k1, pid, p);
                acc.c[C_LAUNCHED] += 1;
            }
            // the position of the wave's last new ticket becomes the current one
            const uint64_t got = __ballot(my != NO_TICKET);
            if (got != 0) {
                cur_pos = __builtin_amdgcn_readlane(last_pos, 63 - __clzll((long long)got));
                cur_seg = __builtin_amdgcn_readlane(seg, 63 - __clzll((long long)got));
                cur_lo = a.tfirst[cur_pos];
                cur_hi = a.tfirst[cur_pos + 1];
            }
        }
        const uint64_t B = __ballot(p.st == ST_BALLISTIC);
        if (B == 0) {
            if (drained) break;
            continue;
        }
        int s0 = __builtin_amdgcn_readlane(seg, __ffsll((unsigned long long)B) - 1);
        if constexpr (std::is_same<R, double>::value) {
            // lanes of other segments wait their turn: a second copy of the flight with per-lane
            // constants would only spill.  Those of segments that get no new lanes go first, or they
            // would wait for as long as the present one has tickets (4.9e6 atoms of four cathodes in one
            // kernel, a wave at a boundary: 9.3 ms, 6.3 this way)
            const uint64_t old = B & __ballot(seg != cur_seg);
            if (old != 0) s0 = __builtin_amdgcn_readlane(seg, __ffsll((unsigned long long)old) - 1);
            ballistic_loop<O>(a, segs + s0, pid, p, seg == s0, T.drained || drained);
        } else if (__ballot(p.st == ST_BALLISTIC && seg != s0) == 0) {
            ballistic_loop<O>(a, segs + s0, pid, p, true, T.drained || drained);
        } else if (p.st == ST_BALLISTIC) {
            // lanes of several segments: one flight with per-lane constants
            const SegDev<R>& s = segs[seg];
            const Term t = step_mode<O>(s, a.tab, a.k0, a.k1, pid, a.cap, p);
            if (t.state != HIT_NONE) mark_ended(p, t);
        }
    }
    if (!WHOLE) close_run(a, Q, lane);
    flush_acc(a, bt, acc);
    return QRun{Q.q, T.tk};
}

template <bool ARR, bool OBJ, typename R>
__device__ __forceinline__ void ballistic_kernel(TransportArgs<R>& a, const SegDev<R>* segs)
{
    extern __shared__ unsigned long long lds[];
    BlockTally bt;
    lds_setup(a, bt, lds);
    ballistic_phase<ARR, OBJ, false, false>(a, bt, segs, Tickets(), QRun(), (int)(threadIdx.x & 63));
    lds_flush(a, bt);
}

// At most 96 VGPRs: five waves per SIMD or more hide the latency of the transcendental and
// integer-multiply chains.  73 are used without absorbing objects (85 with tickets and queue slots in
// vector registers): six waves per SIMD, four cathodes 3.04 -> 2.95 ms, the 64-chamber sweep's half 14.1
// -> 13.5; asked for seven (72 VGPRs), 2.97 and 13.7.
template <bool ARR, bool OBJ>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(5)))
k_ballistic32(TransportArgs<float> a, const SegDev<float>* __restrict__ segs)
{
    ballistic_kernel<ARR, OBJ>(a, segs);
}
// Three waves per SIMD (at most 168 VGPRs) in both FP64 kernels, without spills: four waves spilled
// 64 registers in the walk (9e5 atoms at 0.5 / 0 / 2 Pa: 13.8 ms at three, 15.8 at four).
template <bool ARR, bool OBJ>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
k_ballistic64(TransportArgs<double> a, const SegDev<double>* __restrict__ segs)
{
    ballistic_kernel<ARR, OBJ>(a, segs);
}

// The last walks of a drained wave (its lanes in D, at most Walk<R>::COOP, none with a held step), walked
// to their ends by the whole wave: each walker gets a span of 64, 32, 16, 8, 4 or (FP64) 2 lanes, all of which
// hold its state, and lane j of the span draws step e + 1 + j.  A pass takes every walker's steps up to the
// first that leaves its ball (or to the event cap), then tests those.  Spans are laid out anew as
// walkers end.  Bound by the latency of one pass, the longest walks being all that is left: the state
// stays replicated in the span, so a pass starts without shuffles, and the surfaces are read once per
// layout (GeoOf).
template <bool ARR, bool OBJ, bool WHOLE, typename R>
__device__ __forceinline__ void tail_walk(const TransportArgs<R>& a, const BlockTally& bt,
                                          const SegDev<R>* __restrict__ segs, uint64_t D, int seg, R lam_l2,
                                          uint32_t cfgcat, uint32_t pid, Particle<R>& p, Walk<R>& wk, LaneAcc<true>& acc,
                                          int lane)
{
    flush_acc(a, bt, acc);
    acc.seg = -1;
    while (D != 0) {
        // layout: walker q (in lane order) moves to span q
        const int n = __popcll(D);
        const int sh = n == 1 ? 6 : n == 2 ? 5 : n <= 4 ? 4 : n <= 8 ? 3 : n <= 16 ? 2 : 1;
        const int span = 1 << sh, slot = lane >> sh, j = lane & (span - 1), base = lane & ~(span - 1);
        int home = 0;
        if ((D >> lane) & 1ull) home = (int)lanes_below(D);
        home = __builtin_amdgcn_ds_permute((((D >> lane) & 1ull) ? home : 63) << 2, lane);
        const int src = __shfl(home, slot);
        pid = (uint32_t)__shfl((int)pid, src);
        seg = __shfl(seg, src);
        cfgcat = (uint32_t)__shfl((int)cfgcat, src);
        lam_l2 = __shfl(lam_l2, src);
        p.e = (uint32_t)__shfl((int)p.e, src);
        p.ndiff = (uint32_t)__shfl((int)p.ndiff, src);
        p.E = __shfl(p.E, src);
        p.r2 = __shfl(p.r2, src);
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            p.x[i] = __shfl(p.x[i], src);
            p.xc[i] = __shfl(p.xc[i], src);
        }
        wk = lane_walk(wk, src);
        bool alive = slot < n;
        p.st = alive ? ST_DIFFUSIVE : ST_DEAD;
        const bool lead = alive && j == 0;
        if (lead && acc.seg != seg) {
            flush_acc(a, bt, acc);
            acc.seg = seg;
        }
        const SegDev<R>& S = segs[seg];
        GeoOf<OBJ && !WHOLE, R> geo(S);
        const uint64_t span_mask = sh == 6 ? ~0ull : (1ull << span) - 1;
        for (;;) {
            const uint32_t ej = p.e + 1u + (uint32_t)j;
            R dir[3];
            const R ell = any_draw(lam_l2, diffusive_block(pid, ej, cfgcat, a.k0, a.k1), (ej & 1u) != 0, dir);
            const bool allowed = ej <= a.cap && ej > (uint32_t)j;
            const auto at = spot_of(p);
            const auto t = chain_steps(at, ell, dir, sh, j, allowed, alive, wk, p.r2);
            const uint64_t stay = (__ballot(allowed && spot_holds(t, wk, p.r2)) >> base) & span_mask;
            const int f = stay == span_mask ? span : __ffsll((unsigned long long)~stay) - 1;   // steps taken
            const auto to = lane_spot(t, base + (f > 0 ? f - 1 : 0));
            if (f > 0) stand_at(p, to);
            p.e += (uint32_t)f;
            const bool stop = alive && f < span, held = stop && p.e < a.cap;
            const int hl = base + (f < span ? f : 0);
            const R hell = __shfl(ell, hl);
            R hd[3];
#pragma unroll
            for (int i = 0; i < 3; ++i) hd[i] = __shfl(dir[i], hl);
            Term end{HIT_NONE, -1, 0.f};
            if (held) {
                ++p.e;
                p.r2 = hell;
#pragma unroll
                for (int i = 0; i < 3; ++i) p.d[i] = hd[i];
                end = diffusive_resolve(S, geo, p, wk, std::conditional_t<OBJ, SpanObjects, NoObjects>(sh, j));
                if (std::is_same<R, float>::value && lead) acc.c[C_TESTED] += 1u;
            } else if (stop) {
                end.state = HIT_ESCAPED;
            }
            if (end.state != HIT_NONE) {
                if (lead) {
                    p.ndiff = p.e - p.ndiff - (held ? 1u : 0u);
                    terminate<ARR>(a, bt, segs[seg], pid, p, end, acc);
                }
                alive = false;
            }
            D = __ballot(alive && j == 0);
            const int live = __popcll(D);
            if (live == 0 || (sh < 6 && 2 * live <= (64 >> sh))) break;
        }
    }
    p.st = ST_DEAD;
}

// Diffusive phase: the walks of the `total` atoms queued by the ballistic phase of the round (WHOLE: of
// the wave's own slots T).  Lanes of any segments walk together (the step needs only two per-lane
// numbers of the segment), so a wave never falls back to one step at a time.
template <bool ARR, bool OBJ, bool WHOLE, typename R>
__device__ __forceinline__ void diffusive_phase(TransportArgs<R>& a, const BlockTally& bt,
                                                const SegDev<R>* __restrict__ segs, BlockQueue B, uint32_t total,
                                                uint32_t chunk, int lane)
{
    Particle<R> p;
    Walk<R> wk;
    p.st = ST_DEAD;
    p.e = p.ndiff = p.ncoll = 0;
    uint32_t pid = 0;
    int seg = 0;
    R lam_l2 = (R)0;           // the lane's segment: thermal mean free path (times ln 2), Philox word
    uint32_t cfgcat = 0;
    LaneAcc<true> acc;
    Tickets T;
    for (;;) {
        const uint64_t dead = __ballot(p.st == ST_DEAD);
        const int n_dead = __popcll(dead);
        if (!T.drained && n_dead > 0 && (n_dead >= a.refill_min || n_dead == 64)) {
            const uint32_t my = WHOLE ? claim_shared(T, B, dead, lane)
                                      : claim<false, false>(T, &a.qstate[QS_DIFFUSIVE], chunk, total, dead, lane);
            const uint32_t qpid = my != NO_TICKET ? a.queue[my].pid : 0xFFFFFFFFu;
            if (qpid != 0xFFFFFFFFu) {                 // empty slots (left unused by a wave) are skipped
                const ThermRec<R> r = a.queue[my];
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    p.x[i] = r.x[i];
                    p.xc[i] = r.xc[i];
                }
                p.E = r.E;
                p.e = r.e;
                p.ndiff = r.e;         // events before the walk
                p.ncoll = 0;
                p.r2 = (R)-1;          // no clearance ball yet: the first step is tested
                p.st = ST_DIFFUSIVE;
                pid = r.pid;
                const int sg = (int)r.seg;
                if (sg != acc.seg) {
                    flush_acc(a, bt, acc);
                    acc.seg = sg;
                }
                seg = sg;
                lam_l2 = r.lam;
                cfgcat = r.cfgcat;
            }
        }
        const uint64_t D = __ballot(p.st == ST_DIFFUSIVE);
        if (D == 0) {
            if (T.drained) break;
            continue;
        }
        if (T.drained && __popcll(D) <= Walk<R>::COOP) {
            tail_walk<ARR, OBJ, WHOLE>(a, bt, segs, D, seg, lam_l2, cfgcat, pid, p, wk, acc, lane);
            break;
        }
        diffusive_loop<ARR, OBJ>(a, bt, segs, seg, lam_l2, cfgcat, pid, p, wk, acc, T.drained);
    }
    flush_acc(a, bt, acc);
}

template <bool ARR, bool OBJ, typename R>
__device__ __forceinline__ void diffusive_kernel(TransportArgs<R>& a, const SegDev<R>* segs)
{
    extern __shared__ unsigned long long lds[];
    const uint32_t total = (uint32_t)a.qstate[QS_QUEUE];   // written by the ballistic phase of this round
    if (total == 0) return;        // (clearing and flushing the LDS of a full grid takes 60 us)
    BlockTally bt;
    lds_setup(a, bt, lds);
    const uint32_t chunk = (uint32_t)chunk_of(total, a.n_simd, TICKET_CHUNK);
    diffusive_phase<ARR, OBJ, false>(a, bt, segs, BlockQueue(), total, chunk, (int)(threadIdx.x & 63));
    lds_flush(a, bt);
}

// At most 96 VGPRs: five waves per SIMD.  The few spills (8 to 25 registers) lie outside the steps of the
// walk; four waves without them were slower in large runs.
template <bool ARR, bool OBJ>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(5)))
k_diffusive32(TransportArgs<float> a, const SegDev<float>* __restrict__ segs)
{
    diffusive_kernel<ARR, OBJ>(a, segs);
}

// Bound by VALU issue as the FP32 walk is (an FP64 instruction takes four clocks too): 430
// instructions a round of two steps, most of them the library's log2 and sincospi.  One thread per
// atom through its whole history, every step tested, took 77 ms for 9e5 atoms at 0.5 / 0 / 2 Pa and
// 34.2 ms for 2.3e6 from four cathodes; the two phases take 12.9 and 4.7 ms.
template <bool ARR, bool OBJ>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
k_diffusive64(TransportArgs<double> a, const SegDev<double>* __restrict__ segs)
{
    diffusive_kernel<ARR, OBJ>(a, segs);
}

// Both phases of a run in one kernel (whole_waves says which): a wave takes a fixed run of chunk_ballistic
// tickets through the ballistic phase, its thermalised atoms into the run's own queue slots, and then
// walks those and what is left of its block's; where the queue holds fewer slots than that, in several
// passes, its own walks only.  Such a run is bound by the latency of its longest
// histories; here no walk waits for the slowest flight of another wave nor for a launch, and no
// counter is shared between blocks: atomics on one line go at 11 ns each.  1e5 atoms of one cathode 0.372
// -> 0.288 ms, 1e6 from four 0.84 -> 0.62, 4.6e6 1.80 -> 1.60; without gas 5e6 0.59 -> 0.13.  LIMITED: 4.6e6 from the
// scratch array in one launch 1.77 ms (four rounds 2.50, five of a kernel per phase 3.70); as a run-time
// switch it cost the instance with objects and arrivals 8 % in spills.
template <bool ARR, bool OBJ, bool LIMITED, typename R>
__device__ __forceinline__ void whole_kernel(TransportArgs<R>& a, const SegDev<R>* segs)
{
    extern __shared__ unsigned long long lds[];
    constexpr int WAVES = 16;          // of a block, at most
    __shared__ uint32_t next[WAVES], end[WAVES];
    BlockTally bt;
    if (threadIdx.x < WAVES) end[threadIdx.x] = 0;
    lds_setup(a, bt, lds);
    const int lane = threadIdx.x & 63;
    // the waves of a block take tickets from all over the run
    const uint32_t own = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const uint32_t wave = own * gridDim.x + blockIdx.x, slot = wave * a.wave_slots;
    const uint32_t total = (uint32_t)a.total;
    Tickets T;
    T.tk = wave * a.chunk_ballistic < total ? wave * a.chunk_ballistic : total;
    T.tk_end = total - T.tk > a.chunk_ballistic ? T.tk + a.chunk_ballistic : total;
    constexpr bool TIMED = std::is_same<R, float>::value;   // (there are no phase times of FP64 runs)
    uint64_t times[2] = {0, 0};
    if (TIMED && a.times && threadIdx.x == 0 && blockIdx.x == 0) a.times[2] = wall_clock64();
    for (;;) {
        T.drained = T.tk == T.tk_end;
        const uint64_t t0 = TIMED ? wall_clock64() : 0;
        const QRun e = ballistic_phase<ARR, OBJ, true, LIMITED>(a, bt, segs, T, QRun{slot, slot + a.wave_slots}, lane);
        const uint64_t t1 = TIMED ? wall_clock64() : 0;
        // publish the wave's records to the block: all lanes' stores, then next, then end
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_wave_barrier();
        if (lane == 0) {
            __hip_atomic_store(&next[own], slot, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
            __hip_atomic_store(&end[own], (uint32_t)e.q, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        }
        __builtin_amdgcn_wave_barrier();
        // (slots that are written again are walked by their wave alone)
        diffusive_phase<ARR, OBJ, true>(a, bt, segs, BlockQueue{next, end, own, LIMITED ? 1u : blockDim.x / 64}, 0u, 0u,
                                        lane);
        times[0] += t1 - t0;
        times[1] += (TIMED ? wall_clock64() : 0) - t1;
        if (!LIMITED) break;
        T.tk = (uint32_t)e.q_end;
        if (T.tk == T.tk_end) break;
    }
    if (TIMED && a.times && threadIdx.x == 0 && blockIdx.x % 8 == 0) {
        atomicAdd((unsigned long long*)&a.times[0], (unsigned long long)times[0]);
        atomicAdd((unsigned long long*)&a.times[1], (unsigned long long)times[1]);
    }
    lds_flush(a, bt);
    if (TIMED && a.times && threadIdx.x == 0) atomicMax((unsigned long long*)&a.times[3], (unsigned long long)wall_clock64());
}

// Four waves per SIMD (FP64: three) fit without spills in the steps.
template <bool ARR, bool OBJ, bool LIMITED>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4)))
k_whole32(TransportArgs<float> a, const SegDev<float>* __restrict__ segs)
{
    whole_kernel<ARR, OBJ, LIMITED>(a, segs);
}
template <bool ARR, bool OBJ>
__global__ void __launch_bounds__(768) __attribute__((amdgpu_waves_per_eu(3)))
k_whole64(TransportArgs<double> a, const SegDev<double>* __restrict__ segs)
{
    whole_kernel<ARR, OBJ, false>(a, segs);
}

// FP64 runs that share nothing with other runs of their plan: a thread takes a ticket through its whole history,
// every diffusive step tested (a ball of no radius), with no queue and no counters in memory.  For runs
// recorded into a caller's graph, whose replays may overlap with any other work of the plan, and for plans
// whose queue does not fit the memory.  The operations of a history, and so the outputs, are those of the two
// phases, bit for bit.  9e5 atoms at 0.5 / 0 / 2 Pa take 70 ms (the two phases 10.4), 2.3e6 of four cathodes 23.4
// (3.9), 1e5 of one 2.8 (0.77).
template <bool ARR, bool OBJ>
__global__ void __launch_bounds__(256) k_plain64(TransportArgs<double> a, const SegDev<double>* __restrict__ segs)
{
    extern __shared__ unsigned long long lds[];
    using O = std::conditional_t<OBJ, OwnObjects, NoObjects>;
    BlockTally bt;
    lds_setup(a, bt, lds);
    LaneAcc<false> acc;
    for (uint64_t g = (uint64_t)blockIdx.x * 256 + threadIdx.x; g < a.total; g += (uint64_t)gridDim.x * 256) {
        int lo = 0, hi = a.n_seg;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (a.tfirst[mid] <= g) lo = mid; else hi = mid;
        }
        const int seg = (int)a.torder[lo];
        const uint32_t pid = (uint32_t)(g - a.tfirst[lo]);
        const SegDev<double>& s = segs[seg];
        if (seg != acc.seg) {
            flush_acc(a, bt, acc);
            acc.seg = seg;
        }
        Particle<double> p;
        Walk<double> wk;
        Term t{HIT_NONE, -1, 0.f};
        start(s, a.k0, a.k1, pid, p);
        while (t.state == HIT_NONE && p.st == ST_BALLISTIC) t = step_mode<O>(s, a.tab, a.k0, a.k1, pid, a.cap, p);
        const bool walks = t.state == HIT_NONE;
        while (t.state == HIT_NONE) {
            if (p.e >= a.cap) {
                t.state = HIT_ESCAPED;
                break;
            }
            p.r2 = -1.0;
            diffusive_single(s.lam_l2, s.cfgcat, a.k0, a.k1, pid, p, wk);
            t = diffusive_resolve(s, s, p, wk, O());
            p.ndiff += t.state == HIT_NONE ? 1u : 0u;
        }
        acc.c[C_LAUNCHED] += 1u;
        acc.c[C_THERMALIZED] += walks ? 1u : 0u;
        acc.c[C_DIFFUSIVE] += p.ndiff;
        acc.c[C_TESTED] += p.ndiff + (walks && t.state != HIT_ESCAPED ? 1u : 0u);
        terminate<ARR>(a, bt, s, pid, p, t, acc);
    }
    flush_acc(a, bt, acc);
    lds_flush(a, bt);
}

// Ranges of words to clear: a run's outputs and a round's counters.
struct Ranges {
    uint64_t* p[6] = {};
    uint64_t n[6] = {};
    void add(uint64_t* q, uint64_t m)
    {
        int i = 0;
        while (n[i] != 0) ++i;
        p[i] = q;
        n[i] = q ? m : 0;
    }
};

// (A kernel, so that it can sit in a graph; one for all ranges, a launch costs more than clearing them.)
__global__ void k_clear(Ranges c)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
#pragma unroll
    for (int k = 0; k < 6; ++k)
        for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < c.n[k]; i += stride) c.p[k][i] = 0;
}

// profiles = counts / (N_seg * bin area); FP64.
__global__ void k_normalize(const unsigned long long* __restrict__ counts, const uint64_t* __restrict__ bin_off,
                            const double* __restrict__ seg_norm, int n_seg, uint64_t n_bins,
                            double* __restrict__ profiles)
{
    const uint64_t stride = (uint64_t)gridDim.x * blockDim.x;
    for (uint64_t b = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; b < n_bins; b += stride) {
        int lo = 0, hi = n_seg;
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (bin_off[mid] <= b) lo = mid; else hi = mid;
        }
        profiles[b] = (double)counts[b] * seg_norm[lo];
    }
}

static int put_clear(const Ranges& c, LaunchSink& sink)
{
    uint64_t n = 0;
    for (uint64_t m : c.n) n = std::max(n, m);
    KLaunch k;
    k.func = (const void*)k_clear;
    k.grid = dim3((unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 + 1 : 4096));
    k.block = dim3(256);
    k.arg(c);
    return sink.put(k);
}

static int put_normalize(Plan* P, const uint64_t* d_counts, double* d_profiles, LaunchSink& sink)
{
    const uint64_t n = P->n_bins_total;
    KLaunch k;
    k.func = (const void*)k_normalize;
    k.grid = dim3((unsigned)((n + 255) / 256 < 4096 ? (n + 255) / 256 + 1 : 4096));
    k.block = dim3(256);
    k.arg((const unsigned long long*)d_counts);
    k.arg((const uint64_t*)P->d_bin_off);
    k.arg((const double*)P->d_seg_norm);
    k.arg((int)P->n_seg);
    k.arg(n);
    k.arg(d_profiles);
    return sink.put(k);
}

int StreamSink::put(const KLaunch& k)
{
    if (k.n_args < 0 || !k.func) {
        set_error("internal: malformed kernel launch");
        return SPX_ESTATE;
    }
    if (events && (k.phase & 1)) SPX_HIP(hipEventRecord(events[3 * round], st));
    void* args[8];
    k.pointers(args);
    SPX_HIP(hipLaunchKernel(k.func, k.grid, k.block, args, k.smem, st));
    if (events && (k.phase & 1)) SPX_HIP(hipEventRecord(events[3 * round + 1], st));
    if (events && (k.phase & 2)) SPX_HIP(hipEventRecord(events[3 * round++ + 2], st));
    return SPX_OK;
}

// Dynamic LDS of the FP32 transport for a plan: counters if they fit, tally if it fits, arrival
// histograms (when requested) if they fit.
size_t transport_lds(const Plan* P, bool arrivals, bool* lds_counters, bool* lds_tally, bool* lds_arrivals)
{
    const size_t cbytes = (size_t)P->n_seg * N_COUNTERS * sizeof(unsigned long long);
    const size_t tbytes = (size_t)P->n_bins_total * sizeof(uint32_t);
    const size_t abytes = (size_t)P->n_seg * ARR_BINS * sizeof(uint32_t);
    *lds_counters = cbytes <= LDS_COUNTERS_MAX;
    *lds_tally = tbytes <= LDS_TALLY_MAX;
    *lds_arrivals = arrivals && abytes <= LDS_ARRIVALS_MAX;
    return (*lds_counters ? cbytes : 0) + (*lds_tally ? tbytes : 0) + (*lds_arrivals ? abytes : 0);
}

namespace {
// The instance of a kernel template <arrival tallies, absorbing objects, ...>.
#define SPX_INSTANCE(kernel, arr, obj, ...)                                                     \
    ((arr) ? ((obj) ? (const void*)kernel<true, true __VA_OPT__(, ) __VA_ARGS__>                \
                    : (const void*)kernel<true, false __VA_OPT__(, ) __VA_ARGS__>)              \
           : ((obj) ? (const void*)kernel<false, true __VA_OPT__(, ) __VA_ARGS__>               \
                    : (const void*)kernel<false, false __VA_OPT__(, ) __VA_ARGS__>))

// The plan's constants and the kernels of a precision.
template <typename R> struct Path;
template <> struct Path<float> {
    static const SegDev<float>* segs(const Plan* P) { return P->d_seg32; }
    static const float* theta(const Plan* P) { return P->d_theta32; }
    static const float* betamax(const Plan* P) { return P->d_betamax32; }
    static const float* edges(const Plan* P) { return P->d_edges32; }
    static const void* ballistic(const Plan* P, bool arr) { return SPX_INSTANCE(k_ballistic32, arr, P->has_objects); }
    static const void* diffusive(const Plan* P, bool arr) { return SPX_INSTANCE(k_diffusive32, arr, P->has_objects); }
    static const void* whole(const Plan* P, bool arr, bool limited)
    {
        return limited ? SPX_INSTANCE(k_whole32, arr, P->has_objects, true)
                       : SPX_INSTANCE(k_whole32, arr, P->has_objects, false);
    }
    static constexpr int IDLE = WALK_IDLE;
    static constexpr bool LIMITED = true;
};
template <> struct Path<double> {
    static const SegDev<double>* segs(const Plan* P) { return P->d_seg64; }
    static const double* theta(const Plan* P) { return P->d_theta64; }
    static const double* betamax(const Plan* P) { return P->d_betamax64; }
    static const double* edges(const Plan* P) { return P->d_edges64; }
    static const void* ballistic(const Plan* P, bool arr) { return SPX_INSTANCE(k_ballistic64, arr, P->has_objects); }
    static const void* diffusive(const Plan* P, bool arr) { return SPX_INSTANCE(k_diffusive64, arr, P->has_objects); }
    // (the queue of an FP64 plan holds its rounds)
    static const void* whole(const Plan* P, bool arr, bool) { return SPX_INSTANCE(k_whole64, arr, P->has_objects); }
    static const void* plain(const Plan* P, bool arr) { return SPX_INSTANCE(k_plain64, arr, P->has_objects); }
    static constexpr int IDLE = WALK_IDLE64;
    static constexpr bool LIMITED = false;
};
}  // namespace

int occupancy_transport32(const Plan* P, int threads, int* bpc_ballistic, int* bpc_diffusive)
{
    bool lc, lt, la;
    const size_t smem = transport_lds(P, false, &lc, &lt, &la);
    int b1 = 0, b2 = 0;
    SPX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&b1, Path<float>::ballistic(P, false), threads, smem));
    SPX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&b2, Path<float>::diffusive(P, false), threads, smem));
    *bpc_ballistic = b1;
    *bpc_diffusive = b2;
    return SPX_OK;
}

// Rounds of a ticket space of `total` tickets: as few as round_max allows, of equal size.
uint64_t rounds_of(uint64_t total, uint64_t round_max)
{
    return total == 0 ? 0 : (total + round_max - 1) / round_max;
}

// Blocks of a round of `total` tickets with a kernel per phase, out of `blocks`: a wave of a small run costs more to start and end
// (its block clears and flushes the LDS tally) than its share of the work, and histories step faster
// with fewer waves on their SIMD.  Waves per SIMD by tickets per lane of one wave per SIMD; ballistic
// + diffusive kernel at 1, 2, 3, 4, 5 of them: 1e4 atoms 0.26, 0.28, 0.31, 0.34, 0.36 ms; 1e5 (1.5 tickets)
// 0.42, 0.45, 0.49, 0.51, 0.53; 2e5, four cathodes (3.1) 0.56, 0.51, 0.55, 0.57, 0.60; 1e6 (15) 1.23,
// 0.95, 0.89, 0.91, 0.92; 2.3e6 (35) 2.34, 1.50, 1.34, 1.31, 1.36.
static int blocks_of(uint64_t total, int blocks, int threads, int n_simd)
{
    const uint64_t per_lane = total / ((uint64_t)n_simd * 64);
    if (per_lane >= 64) return blocks;
    const int w = 1 + (per_lane >= 2) + (per_lane >= 8) + (per_lane >= 24);
    return std::min(blocks, (w * n_simd * 64 + threads - 1) / threads);
}

// Waves per SIMD of a run that takes both phases in one kernel, one block of all of them per CU; 0: two
// kernels.  A kernel per phase waits twice for its longest histories, but shares the work over the whole
// device and has more waves resident, which wins in long runs, and earlier where the chambers differ (the
// waves of a block share walks, blocks do not).  Two kernels / one at 2, 3, 4 waves [ms]: single target
// at 0.5 Pa, 1e5 atoms (1.5 tickets per lane of one wave per SIMD) 0.372 / 0.288, 0.300, 0.324; 1e6 (15)
// 0.80 / 0.68, 0.62, 0.64; 5e6 (76) 1.96 / 2.40, 1.92, 1.74; 1e7 3.29 / 4.55, 3.56, 3.15; four cathodes, 7e6
// 2.38 / 2.97, 2.35, 2.31, 2.3e7 5.95 / 9.2, 7.1, 6.6.  Chambers of 0.1 to 2 Pa: 3e5 atoms 2.96 / 2.32, 2.23,
// 2.24; 1e6 3.59 / 4.03, 3.73, 3.47; 2e6 4.80 / 6.32, 5.40, 5.08.  One chamber at 2 Pa, two / one as the rule has its
// waves: 1e6 5.63 / 5.32, 3e6 12.1 / 11.7, 5e6 17.83 / 17.86.  The pressures count by their extremes alone, and
// the line at a ratio of two is on the safe side for those between: eight chambers from 0.5 Pa up, 2e6 and 5e6
// atoms, to 1.5 times 1.61 / 1.21 and 2.95 / 2.46, to 2.2 times 2.24 / 2.04 and 4.15 / 3.96, to 3 times 3.15 /
// 3.00 and 5.74 / 5.73, to 5 times 6.23 / 6.13 and 10.6 / 11.2; 64 chambers of 0.1 to 2 Pa 4.42 / 4.53 and 6.37 /
// 7.66; ten atoms at 0.1 Pa beside 3e6 at 0.5 1.42 / 1.15.  FP64 (three waves at most): four
// cathodes, 2e5 1.21 / 0.96, 0.88; 5e5 1.78 / 1.36, 1.46; 3e6 4.52 / -, 4.32; single target, 1e6 2.28 / 1.93,
// 2.09; 2e6 3.49 / -, 3.42; 3e6 4.40 / -, 4.81.
uint64_t whole_limit(const Plan* P, const Shape& sh)
{
    const uint64_t lanes = 4 * (uint64_t)P->n_cu * 64;
    if (!sh.whole || (uint64_t)std::min(sh.blocks, sh.blocks_diff) * (uint64_t)sh.threads < lanes)
        return 0;                  // (a grid that the caller made smaller than that stays as it is)
    return (P->p_hi > 2.0 * P->p_lo ? 16 : P->params.precision == 64 ? 32 : 80) * lanes - 1;
}

static int whole_waves(const Plan* P, uint64_t total, const Shape& sh, bool fp64)
{
    if (total == 0 || total > whole_limit(P, sh)) return 0;
    const uint64_t per_lane = total / (4 * (uint64_t)P->n_cu * 64);
    if (fp64) return per_lane < 8 ? 2 : 3;
    return per_lane < 4 ? 2 : per_lane < 20 ? 3 : 4;
}

// The outputs of a run that its kernels add to.
static Ranges output_ranges(const Plan* P, const Outputs& o)
{
    Ranges c;
    c.add(o.counts, P->n_bins_total);
    c.add(o.counters, (uint64_t)P->n_seg * N_COUNTERS);
    if (o.arr_E) {
        c.add(o.arr_E, (uint64_t)P->n_seg * SPX_ARRIVAL_E_BINS);
        c.add(o.arr_A, (uint64_t)P->n_seg * SPX_ARRIVAL_A_BINS);
        c.add(o.esum, P->n_bins_total);
    }
    return c;
}

// The launches of an FP64 run without a queue: 16 blocks a CU at most, whose threads take one ticket after another
// (a block clears and flushes the LDS tally once).
static int put_plain64(Plan* P, TransportArgs<double>& a, const SegDev<double>* segs, uint64_t total, size_t smem,
                       const Outputs& o, LaunchSink& sink)
{
    SPX_TRY(put_clear(output_ranges(P, o), sink));
    if (total > 0) {
        a.total = total;
        KLaunch k;
        k.func = Path<double>::plain(P, a.arr_E != nullptr);
        k.grid = dim3((unsigned)std::min<uint64_t>((total + 255) / 256, 16 * (uint64_t)P->n_cu));
        k.block = dim3(256);
        k.smem = (uint32_t)smem;
        k.arg(a);
        k.arg(segs);
        SPX_TRY(sink.put(k));
    }
    return o.profiles ? put_normalize(P, o.counts, o.profiles, sink) : SPX_OK;
}

template <typename R>
int build_transport(Plan* P, uint64_t seed, const Outputs& o, const uint64_t* tfirst, uint64_t total,
                    const Shape& sh, const QueueMem& q, LaunchSink& sink)
{
    using K = Path<R>;
    TransportArgs<R> a;
    std::memset(&a, 0, sizeof(a));     // padding too: launches are compared bytewise
    a.segs = K::segs(P);
    a.tab.theta = K::theta(P);
    a.tab.betamax = K::betamax(P);
    a.tab.ne = P->params.table_ne;
    a.tab.ns = P->params.table_ns;
    a.tab.xs = (R)((P->params.table_ne - 1) / ((P->params.log_eps_hi - P->params.log_eps_lo) * 3.321928094887362));
    a.tfirst = tfirst;
    a.torder = P->d_torder;
    a.queue = (ThermRec<R>*)q.queue;
    a.qstate = q.qstate;
    a.times = q.times;
    a.counts = (unsigned long long*)o.counts;
    a.counters = (unsigned long long*)o.counters;
    a.records = o.records;
    a.arr_E = (unsigned long long*)o.arr_E;
    a.arr_A = (unsigned long long*)o.arr_A;
    a.esum = (unsigned long long*)o.esum;
    a.e_edges = K::edges(P);
    a.c_edges = K::edges(P) + SPX_ARRIVAL_E_BINS + 1;
    a.k0 = (uint32_t)seed;
    a.k1 = (uint32_t)(seed >> 32);
    a.cap = P->params.event_cap;
    a.n_seg = P->n_seg;
    a.n_simd = 4 * P->n_cu;
    a.refill_min = sh.refill_min;
    a.refill_ballistic = sh.refill_ballistic;
    a.defer_min = sh.defer_min;
    // a pass of the surface tests takes about 180 instructions, and 70 more per absorbing object of
    // the segment (its test and its clearance): the idle rounds it is worth grow with it (four cathodes
    // in chimneys, seven objects a run: diffusive kernel 2.87 ms at 128 idle rounds, 2.66 at 400)
    a.walk_idle = K::IDLE + (int32_t)(K::IDLE * 70 * P->n_objects / (180 * (uint64_t)P->n_seg));
    a.n_bins = (uint32_t)P->n_bins_total;
    bool lc, lt, la;
    const size_t smem = transport_lds(P, o.arr_E != nullptr, &lc, &lt, &la);
    int blocks_diff_arr = sh.blocks_diff;
    if (o.arr_E) {
        int bpc_arr = 0;
        SPX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&bpc_arr, K::diffusive(P, true), sh.threads, smem));
        if (bpc_arr > 0) blocks_diff_arr = std::min(sh.blocks_diff, bpc_arr * P->n_cu);
    }
    a.lds_counters = lc ? 1 : 0;
    a.lds_tally = lt ? 1 : 0;
    a.lds_arrivals = la ? 1 : 0;
    const SegDev<R>* segs = K::segs(P);
    if constexpr (std::is_same<R, double>::value) {
        if (!q.queue) return put_plain64(P, a, segs, total, smem, o, sink);
    }
    const uint64_t n_rounds = rounds_of(total, q.round_max);
    const uint64_t per_round = n_rounds ? (total + n_rounds - 1) / n_rounds : 0;
    const int blocks = blocks_of(per_round, sh.blocks, sh.threads, a.n_simd);
    const int blocks_diff = blocks_of(per_round, a.arr_E ? blocks_diff_arr : sh.blocks_diff, sh.threads, a.n_simd);
    // every queue slot a round can reserve: its atoms plus at most one unused run per wave; in one kernel, its
    // waves have fixed slots, at least a refill's
    const uint64_t waves = (uint64_t)blocks * (uint64_t)((sh.threads + 63) / 64);
    const int ww = whole_waves(P, per_round, sh, std::is_same<R, double>::value);
    const uint64_t whole_grid = std::min<uint64_t>((uint64_t)P->n_cu, std::max<uint64_t>(1, per_round));
    const uint64_t n_whole = whole_grid * 4 * (uint64_t)ww;
    const uint64_t share = ww > 0 ? (per_round + n_whole - 1) / n_whole : 0;
    const uint64_t wave_slots = ww > 0 ? std::min(share, q.cap / n_whole) : 0;
    const bool limited = wave_slots < share;
    if (n_rounds && (ww > 0 ? limited && (wave_slots < 64 || !K::LIMITED)
                            : per_round + waves * QUEUE_CHUNK > q.cap)) {
        set_error("internal: round larger than the thermalisation queue");
        return SPX_ESTATE;
    }
    Ranges clear = output_ranges(P, o);
    // the first round's counters
    clear.add(q.qstate, ww > 0 && q.times ? QSTATE_WORDS : QS_TIMES);
    SPX_TRY(put_clear(clear, sink));
    for (uint64_t r = 0; r < n_rounds; ++r) {
        a.tbase = r * per_round;
        a.total = (a.tbase + per_round < total) ? per_round : total - a.tbase;
        if (ww > 0) {
            a.chunk_ballistic = (uint32_t)share;
            a.wave_slots = (uint32_t)wave_slots;
            KLaunch k;
            k.func = K::whole(P, a.arr_E != nullptr, limited);
            k.grid = dim3((unsigned)whole_grid);
            k.block = dim3((unsigned)(256 * ww));
            k.smem = (uint32_t)smem;
            k.phase = 3;
            k.arg(a);
            k.arg(segs);
            SPX_TRY(sink.put(k));
            continue;
        }
        // the largest power-of-two chunk in [TICKET_CHUNK, TICKET_CHUNK_BALLISTIC_MAX] that
        // still gives every wave about four chunks of the round
        uint64_t cb = TICKET_CHUNK;
        while (2 * cb <= TICKET_CHUNK_BALLISTIC_MAX && 2 * cb * 4 * waves <= a.total) cb *= 2;
        cb = chunk_of(a.total, a.n_simd, cb);
        a.chunk_ballistic = (uint32_t)cb;
        if (r > 0) {
            Ranges c;
            c.add(q.qstate, QS_TIMES);
            SPX_TRY(put_clear(c, sink));
        }
        KLaunch bal;
        bal.func = K::ballistic(P, a.arr_E != nullptr);
        bal.grid = dim3((unsigned)blocks);
        bal.block = dim3((unsigned)sh.threads);
        bal.smem = (uint32_t)smem;
        bal.phase = 1;
        bal.arg(a);
        bal.arg(segs);
        SPX_TRY(sink.put(bal));
        // the instance with the arrival tallies has its own resident limit (fewer waves per SIMD)
        KLaunch dif;
        dif.func = K::diffusive(P, a.arr_E != nullptr);
        dif.grid = dim3((unsigned)blocks_diff);
        dif.block = dim3((unsigned)sh.threads);
        dif.smem = (uint32_t)smem;
        dif.phase = 2;
        dif.arg(a);
        dif.arg(segs);
        SPX_TRY(sink.put(dif));
    }
    if (o.profiles) SPX_TRY(put_normalize(P, o.counts, o.profiles, sink));
    return SPX_OK;
}

template int build_transport<float>(Plan*, uint64_t, const Outputs&, const uint64_t*, uint64_t, const Shape&,
                                    const QueueMem&, LaunchSink&);
template int build_transport<double>(Plan*, uint64_t, const Outputs&, const uint64_t*, uint64_t, const Shape&,
                                     const QueueMem&, LaunchSink&);

// The FP64 kernels run at their resident limits.
int shape_transport64(Plan* P)
{
    bool lc, lt, la;
    const size_t smem = transport_lds(P, false, &lc, &lt, &la);
    Shape& sh = P->shape64;
    sh.threads = 256;
    int b = 0, d = 0;
    SPX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, Path<double>::ballistic(P, false), sh.threads, smem));
    SPX_HIP(hipOccupancyMaxActiveBlocksPerMultiprocessor(&d, Path<double>::diffusive(P, false), sh.threads, smem));
    if (b < 1 || d < 1) {
        set_error("the FP64 transport kernels do not fit on this device");
        return SPX_EDEVICE;
    }
    sh.blocks = b * P->n_cu;
    sh.blocks_diff = d * P->n_cu;
    sh.refill_min = REFILL64;
    sh.refill_ballistic = REFILL_BALLISTIC64;
    sh.defer_min = DEFER_MIN;
    return SPX_OK;
}

void arrival_edges(double* e_edges, double* c_edges)
{
    for (int k = 0; k <= SPX_ARRIVAL_E_BINS; ++k) e_edges[k] = std::pow(10.0, -3.0 + k / 10.0);
    for (int k = 0; k <= SPX_ARRIVAL_A_BINS; ++k) c_edges[k] = std::cos(k * 3.14159265358979323846 / 180.0);
}

}  // namespace spx
