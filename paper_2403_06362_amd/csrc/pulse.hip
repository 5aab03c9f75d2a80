// Pulse in an infinite multiplying medium with secondary particles, for
// gfx950 (the paper's test problem, Sec. "Implementation and Results").
//
// One particle's life (pulse_particle): direction from its first draw,
// flight tau = -ln(u) / sigma_t, census if t + s reaches the last time edge,
// else move, collision-estimator score (an integer count per batch and time
// bin) when x_lo <= x <= x_hi, absorption draw, and on a scattering the
// multiplicity draw n = floor(nu) + (u < nu - floor(nu)).  The n emerging
// particles start at the collision site:
//   hash seeding   the k-th starts its own stream at hash(k, X_p) mod 2^m
//                  (eq. 5; X_p the parent's state after its draws), so any
//                  particle can run anywhere, in any order;
//   stride seeding they continue the source's one stream, depth first.
//
// Schedules:
//   k_pulse_pool (hash: the bank schedule)  a wave is one depth-first walker
//       with 64 lanes: siblings wait in the wave's LDS pool, and one launch
//       runs nearly everything (at the kernel: what bounds it, and where
//       particles go when the pool is full).
//   k_pulse_stride (stride: families)  one source family per lane, depth
//       first on its one stream, every lane flying in every iteration.
//   k_pulse_bank (hash: the event-based schedule)  every launch advances each
//       live particle by one flight and banks all n emerging particles:
//       a wave takes a chunk of input particles through one atomic and stages
//       its appends in LDS, copied to the output bank with one atomic per
//       flush.  Appends are at most n_max per input particle.
//   k_pulse_family (hash)  one source family per lane (sources taken 64 per
//       wave and atomic), walked depth first with a per-lane stack in HBM; an
//       entry holds the siblings still to start of one scattering (X_p and the
//       next key), so the depth is at most the number of scatterings on the
//       current line of descent.  With bank items the same kernel finishes the
//       event schedule's tail: up to a budget of particles per item, the rest
//       banked for the next launch.
// Counts are integers: each is added once per scored collision, in LDS (rows
// per wave, a copy per block) or with 64-bit HBM atomics, so every schedule,
// launch shape and order gives the same counts.
//
// Population control (hash seeding, bank and event schedules; Sec. "Hierarchical Seed
// Splitting": one-off hashed values where no full stream is needed): the
// run is cut into epochs at census times T[(c+1) K].  A particle whose
// flight reaches the census stops at x + mu (C - t) with its direction and
// state (staged per wave in LDS like the appends).  Per batch, N particles
// arrive and M = target leave: arrival X leaves q + [u < r/N] copies
// (q = floor(M/N), r = M mod N) with the one-off value
// u = U(hash(X, hash(c+1, hash(B+1, pc_seed)))) compared exactly in
// integers, and copy k starts the stream hash(k, X) (eq. 5).  All
// particles of a batch share the epoch's weight, so counts stay integers
// and the flux applies the weights.
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "pulse.hpp"

namespace mcrng {

struct PulseLane {
    uint64_t sources = 0, collisions = 0, tallied = 0, scatters = 0, absorbed = 0, census = 0;
    uint64_t secondaries = 0, draws = 0, max_draws = 0;
};

struct PParticle {
    double x, t;
    uint64_t Z;        // stream state, top-aligned (X << (64 - m))
    int32_t tb;        // time bin of t (-1 before the first time edge)
    uint32_t batch;
    double mu;         // direction: a census copy's, or the last flight's
    bool has_mu;       // a census copy keeps its direction; others draw it first
};

enum : uint32_t { PULSE_CENSUS = 0, PULSE_ABSORBED = 1, PULSE_SCATTERED = 2 };

// Runs the particle from its start to its end.  Returns PULSE_CENSUS,
// PULSE_ABSORBED or PULSE_SCATTERED, with *n the number of particles
// emerging (0 unless it scattered); p then holds the collision site and the
// state after the particle's draws (at a census: its start, its state and,
// with DIR, its direction in p.mu).  *draws counts the numbers drawn; a
// scored collision sets *tally to its counter index (the caller adds it
// with wave_tally).  DIR: the particle may carry a direction (census copies).
template <bool DIR>
__device__ __forceinline__ uint32_t pulse_flight(const PulseParams& P, PParticle& p, PulseLane& c,
                                                 uint32_t* draws, uint32_t* n, int64_t* tally) {
    const LcgDev& L = P.lcg;
    *n = 0;
    double mu;
    if (DIR && p.has_mu) {
        mu = p.mu;
    } else {
        p.Z = lcg_next_z(L, p.Z);
        mu = __builtin_fma(uniform_z(p.Z), 2.0, -1.0);   // exact
        *draws += 1;
    }
    p.Z = lcg_next_z(L, p.Z);
    const double tau = fixed_neg_log(uniform_z(p.Z));
    *draws += 1;
    const double s = quot(tau, P.sigma_t, recip_refined(P.sigma_t));   // the reciprocal is loop-invariant
    const double tn = p.t + s;
    if (!(tn < P.t_end)) {
        if (DIR) p.mu = mu;
        return PULSE_CENSUS;
    }
    const double step = mu * s;
    p.x = p.x + step;
    p.t = tn;
    while (p.tb + 1 < static_cast<int32_t>(P.n_time_bins) && P.t_edges[p.tb + 1] <= p.t) p.tb++;
    c.collisions++;
    if (p.tb >= 0 && P.x_lo <= p.x && p.x <= P.x_hi) {
        *tally = static_cast<int64_t>(p.batch) * P.n_time_bins + p.tb;
        c.tallied++;
    }
    p.Z = lcg_next_z(L, p.Z);
    *draws += 1;
    if (!(p.Z < P.scatter_below)) return PULSE_ABSORBED;
    p.Z = lcg_next_z(L, p.Z);
    *draws += 1;
    *n = P.n_floor + (p.Z < P.frac_below ? 1u : 0u);
    return PULSE_SCATTERED;
}

// pulse_flight plus the end counters (kept out of the branches above so that
// the compiler does not fold them into an indexed array in scratch memory).
// *census is set when the particle reached the census.
template <bool DIR = false>
__device__ __forceinline__ uint32_t pulse_particle(const PulseParams& P, PParticle& p, PulseLane& c,
                                                   uint32_t* draws, int64_t* tally, bool* census = nullptr) {
    uint32_t n = 0;
    const uint32_t r = pulse_flight<DIR>(P, p, c, draws, &n, tally);
    if (census) *census = r == PULSE_CENSUS;
    c.census += static_cast<uint64_t>(r == PULSE_CENSUS);
    c.absorbed += static_cast<uint64_t>(r == PULSE_ABSORBED);
    c.scatters += static_cast<uint64_t>(r == PULSE_SCATTERED);
    c.secondaries += n;
    return n;
}

// Start state (top-aligned) of source i of the run (0-based over all batches).
__device__ __forceinline__ uint64_t pulse_source_state(const PulseParams& P, uint64_t j, uint32_t* batch) {
    const uint64_t b = j / P.per_batch;
    const uint64_t i = j - b * P.per_batch;
    *batch = static_cast<uint32_t>(b);
    if (P.hash) {
        const uint64_t parent = murmur_hash(P.first_batch + b + 1ull, P.seed.base);
        return murmur_hash(i + 1ull, parent) << P.lcg.up;
    }
    return stream_start_z(P.lcg, P.seed, j);
}

__device__ __forceinline__ void note_stream(PulseLane& c, uint64_t draws) {
    c.draws += draws;
    if (draws > c.max_draws) c.max_draws = draws;
}

template <int BLOCK>
__device__ __forceinline__ void tally_lds_begin(const PulseParams& P, unsigned long long* lds_counts) {
    if (P.lds_tally)
        for (uint32_t i = threadIdx.x; i < P.n_counters; i += BLOCK) lds_counts[i] = 0;
    __syncthreads();
}

template <int BLOCK>
__device__ __forceinline__ void tally_lds_end(const PulseParams& P, const unsigned long long* lds_counts) {
    if (!P.lds_tally) return;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < P.n_counters; i += BLOCK)
        if (lds_counts[i] != 0) atomicAdd(reinterpret_cast<unsigned long long*>(P.counts) + i, lds_counts[i]);
}

// Block-level sum of the lane counters into P.diag (one atomic per word
// per block).
template <int BLOCK>
__device__ __forceinline__ void flush_lane_counters(const PulseParams& P, const PulseLane& c) {
    __shared__ unsigned long long acc[kNDiag];
    if (threadIdx.x < kNDiag) acc[threadIdx.x] = 0;
    __syncthreads();
    atomicAdd(&acc[PD_SOURCES], c.sources);
    atomicAdd(&acc[PD_COLLISIONS], c.collisions);
    atomicAdd(&acc[PD_TALLIED], c.tallied);
    atomicAdd(&acc[PD_SCATTERS], c.scatters);
    atomicAdd(&acc[PD_ABSORBED], c.absorbed);
    atomicAdd(&acc[PD_CENSUS], c.census);
    atomicAdd(&acc[PD_SECONDARIES], c.secondaries);
    atomicAdd(&acc[PD_DRAWS], c.draws);
    atomicMax(&acc[PD_MAX_DRAWS], c.max_draws);
    __syncthreads();
    if (threadIdx.x < kNDiag) {
        unsigned long long* d = reinterpret_cast<unsigned long long*>(P.diag) + threadIdx.x;
        if (threadIdx.x == PD_MAX_DRAWS)
            atomicMax(d, acc[threadIdx.x]);
        else
            atomicAdd(d, acc[threadIdx.x]);
    }
}

__device__ __forceinline__ uint32_t lane_prefix(uint64_t mask) {
    return __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(mask >> 32),
                                     __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(mask), 0u));
}

// Lane l's value of v as a wave-uniform (scalar) value: the compiler then
// treats what depends on it (loop exits included) as uniform, where a lane
// shuffle's result would count as divergent.
__device__ __forceinline__ uint64_t lane_value(uint64_t v, int l) {
    const uint32_t lo = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v)), l));
    const uint32_t hi = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(static_cast<uint32_t>(v >> 32)), l));
    return (static_cast<uint64_t>(hi) << 32) | lo;
}

// Adds the wave's scored collisions (tally = counter index, or -1).  When
// all counters fit in LDS (P.lds_tally) each block counts into its own copy
// and adds it to HBM once at its end (tally_lds_begin / tally_lds_end);
// otherwise one 64-bit HBM atomic per distinct counter of the wave.  Either
// way same-address atomics from every wave of the GPU, which serialise, are
// avoided.  Called by the whole wave.
__device__ __forceinline__ void wave_tally(const PulseParams& P, int64_t tally, uint32_t lane,
                                           unsigned long long* lds_counts) {
    if (P.lds_tally) {
        // the block's own copy of every counter (added to HBM at the end)
        if (tally >= 0) atomicAdd(lds_counts + tally, 1ull);
        return;
    }
    uint64_t pending = __ballot(tally >= 0);
    while (pending != 0) {
        const int leader = __ffsll(static_cast<long long>(pending)) - 1;
        const int64_t key = static_cast<int64_t>(lane_value(static_cast<uint64_t>(tally), leader));
        const uint64_t same = __ballot(tally == key);
        if (lane == static_cast<uint32_t>(leader))
            atomicAdd(reinterpret_cast<unsigned long long*>(P.counts) + key,
                      static_cast<unsigned long long>(__popcll(same)));
        pending &= ~same;
    }
}

// ------------------------------------------------------------ bank schedule

// Wave prefix sum of per-lane values v < 16 (one ballot per bit).
__device__ __forceinline__ uint32_t wave_prefix16(uint32_t v, uint32_t* total) {
    uint32_t off = 0, tot = 0;
#pragma unroll
    for (int bit = 0; bit < 4; ++bit) {
        const uint64_t m = __ballot((v >> bit) & 1u);
        off += lane_prefix(m) << bit;
        tot += static_cast<uint32_t>(__popcll(m)) << bit;
    }
    *total = tot;
    return off;
}

// Per-wave staging of appends in LDS: a wave collects the particles it
// banks here and copies them to the output bank with one atomic per
// flush, so the output counter sees one atomic per few iterations of a
// wave instead of one per iteration.
// Entries of a wave's bank stage: 16 KiB per wave (8 KiB at 512 threads,
// 4 KiB at 1024, so that a block fits in LDS).  Larger stages mean fewer
// flushes, each an atomic on the one output counter: 512 entries took the
// event-based passes of the 1000 x 1000 problem from 7.6 to 6.3 ms against
// 256.
constexpr uint32_t bank_stage_entries(int block) { return block >= 1024 ? 128u : (block >= 512 ? 256u : 512u); }

uint32_t pulse_bank_stage(int block) { return bank_stage_entries(block); }

template <uint32_t CAP>
struct BankStage {
    static constexpr uint32_t kCap = CAP;   // 32 B per entry
    double x[kCap];
    double t[kCap];
    uint64_t X[kCap];
    uint32_t batch[kCap];
    int32_t tb[kCap];
};

__device__ __forceinline__ void bank_store(const PulseParams& P, uint64_t o, double x, double t, uint64_t X,
                                           uint32_t batch, int32_t tb) {
    if (o < P.out_cap) {
        P.out.x[o] = x;
        P.out.t[o] = t;
        P.out.X[o] = X;
        P.out.batch[o] = batch;
        P.out.tb[o] = tb;
    } else {
        atomicOr(P.overflow, 1u);
    }
}

// Copies the wave's staged entries to the output bank (one atomic).
template <class Stage>
__device__ __forceinline__ void bank_flush(const PulseParams& P, Stage& S, uint32_t count,
                                               uint32_t lane) {
    __builtin_amdgcn_wave_barrier();
    uint64_t base = 0;
    if (lane == 0) base = atomicAdd(reinterpret_cast<unsigned long long*>(P.out_count), count);
    base = lane_value(base, 0);
    for (uint32_t i = lane; i < count; i += 64) bank_store(P, base + i, S.x[i], S.t[i], S.X[i], S.batch[i], S.tb[i]);
    __builtin_amdgcn_wave_barrier();
}

// Per-wave staging of census arrivals (population control), flushed to
// P.cen with one atomic per flush.
template <uint32_t CAP>
struct CensusStageOf {
    static constexpr uint32_t kCap = CAP;   // 28 B per entry
    double x[kCap];
    double mu[kCap];
    uint64_t X[kCap];
    uint32_t batch[kCap];
};

using CensusStage = CensusStageOf<128>;   // 3.5 KiB per wave

// Returns the arrival count of the block's part just after the flushed entries.
template <class Stage>
__device__ __forceinline__ uint64_t census_flush(const PulseParams& P, Stage& S, uint32_t count, uint32_t lane) {
    __builtin_amdgcn_wave_barrier();
    const uint32_t part = blockIdx.x & (P.cen_parts - 1u);
    PulseCensusEntry* const cen = P.cen + part * P.cen_cap;
    uint64_t base = 0;
    if (lane == 0)
        base = atomicAdd(reinterpret_cast<unsigned long long*>(P.cen_count + part * kPulseCounterStride), count);
    base = lane_value(base, 0);
    for (uint32_t i = lane; i < count; i += 64) {
        const uint64_t o = base + i;
        if (o < P.cen_cap) {
            PulseCensusEntry e;
            e.x = S.x[i];
            e.mu = S.mu[i];
            e.X = S.X[i];
            e.batch = S.batch[i];
            e.pad = 0;
            cen[o] = e;
        } else {
            atomicOr(P.overflow, 1u);
        }
    }
    __builtin_amdgcn_wave_barrier();
    return base + count;
}

// Stages the wave's census arrivals (lanes with at_census) in CS: the point
// x + mu (C - t), the direction and the state.  Called by the whole wave.
__device__ __forceinline__ void census_stage(const PulseParams& P, CensusStage& CS, uint32_t& cstaged,
                                             bool at_census, const PParticle& p, uint32_t lane) {
    const uint64_t cm = __ballot(at_census);
    if (cm == 0) return;
    const uint32_t cnt = static_cast<uint32_t>(__popcll(cm));
    if (cstaged + cnt > CensusStage::kCap) {
        census_flush(P, CS, cstaged, lane);
        cstaged = 0;
    }
    if (at_census) {
        const uint32_t e = cstaged + lane_prefix(cm);
        const double rest = P.t_end - p.t;
        const double step = p.mu * rest;
        CS.x[e] = p.x + step;
        CS.mu[e] = p.mu;
        CS.X[e] = p.Z >> P.lcg.up;
        CS.batch[e] = p.batch;
    }
    cstaged += cnt;
}

// Loads input item j of a bank or copies launch into p.
template <int ITEMS>
__device__ __forceinline__ void load_item(const PulseParams& P, uint64_t j, PParticle& p) {
    if (ITEMS == PULSE_ITEMS_COPIES) {
        const PulseCensusEntry e = P.copies[j];
        p.x = e.x;
        p.mu = e.mu;
        p.has_mu = true;
        p.Z = e.X;
        p.batch = e.batch;
        p.t = P.t_start;
        p.tb = P.tb_start;
    } else {
        p.x = P.in.x[j];
        p.t = P.in.t[j];
        p.Z = P.in.X[j];
        p.batch = P.in.batch[j];
        p.tb = P.in.tb[j];
        p.has_mu = false;
    }
}

// ITEMS: what a launch takes as input (sources, a generation bank, or the
// census copies starting an epoch).  PC: the launch's census (P.t_end) is a
// census of population control, whose arrivals go to P.cen.
template <int ITEMS, bool PC, int BLOCK>
__global__ void __launch_bounds__(BLOCK) k_pulse_bank(PulseParams P) {
    constexpr bool SOURCES = ITEMS == PULSE_ITEMS_SOURCES;
    constexpr bool COPIES = ITEMS == PULSE_ITEMS_COPIES;
    constexpr bool DIR = PC || COPIES;   // particles may carry a direction
    const uint32_t chunk = P.chunk;   // items a wave takes per atomic
    using Stage = BankStage<bank_stage_entries(BLOCK)>;
    __shared__ Stage stage[BLOCK / 64];
    __shared__ CensusStage cstage[PC ? BLOCK / 64 : 1];
    extern __shared__ unsigned long long lds_counts[];
    tally_lds_begin<BLOCK>(P, lds_counts);
    PulseLane c;
    const uint64_t n_items = SOURCES ? P.src_end - P.src_begin : P.n_in;
    const uint32_t lane = threadIdx.x & 63u;
    Stage& S = stage[__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)];
    CensusStage& CS = cstage[PC ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0];
    uint32_t cstaged = 0;              // wave-uniform: entries in CS
    uint64_t wnext = 0, wend = 0;      // wave-uniform: the wave's unassigned items [wnext, wend)
    bool exhausted = false;            // wave-uniform
    uint32_t staged = 0;               // wave-uniform: entries in S
    PParticle p;
    p.x = p.t = 0.0;
    p.Z = 0;
    p.tb = -1;
    p.batch = 0;
    p.mu = 0.0;
    p.has_mu = false;
    bool active = false;
    for (;;) {
        const uint64_t need = __ballot(!active);
        if (need != 0 && wnext == wend && !exhausted) {
            uint64_t b = 0;
            if (lane == 0) b = atomicAdd(reinterpret_cast<unsigned long long*>(P.item_counter), chunk);
            b = lane_value(b, 0);
            if (b + chunk >= n_items) exhausted = true;
            wnext = b < n_items ? b : n_items;
            wend = b + chunk < n_items ? b + chunk : n_items;
        }
        const uint64_t avail = wend - wnext;
        const uint32_t nneed = static_cast<uint32_t>(__popcll(need));
        const uint32_t take = avail < nneed ? static_cast<uint32_t>(avail) : nneed;
        const uint32_t rank = lane_prefix(need);
        const uint64_t mine = wnext + rank;
        wnext += take;
        if (!active && rank < take) {
            const uint64_t j = mine;
            if (SOURCES) {
                p.Z = pulse_source_state(P, P.src_begin + j, &p.batch);
                p.x = 0.0;
                p.t = 0.0;
                p.tb = P.tb0;
                c.sources++;
            } else {
                load_item<ITEMS>(P, j, p);
            }
            active = true;
        }
        if (__ballot(active) == 0 && wnext == wend && exhausted) break;
        uint32_t n = 0;
        int64_t tally = -1;
        bool at_census = false;
        if (active) {
            uint32_t draws = 0;
            n = pulse_particle<DIR>(P, p, c, &draws, &tally, &at_census);
            note_stream(c, draws);   // every particle has its own stream
        }
        wave_tally(P, tally, lane, lds_counts);
        if (PC) census_stage(P, CS, cstaged, at_census, p, lane);
        uint32_t total = 0;
        const uint32_t off = wave_prefix16(n, &total);
        if (total != 0) {
            if (staged + total > Stage::kCap) {
                bank_flush(P, S, staged, lane);
                staged = 0;
            }
            if (total <= Stage::kCap) {
                for (uint32_t k = 1; k <= n; ++k) {
                    const uint32_t e = staged + off + (k - 1);
                    S.x[e] = p.x;
                    S.t[e] = p.t;
                    S.X[e] = murmur_hash(k, p.Z >> P.lcg.up) << P.lcg.up;
                    S.batch[e] = p.batch;
                    S.tb[e] = p.tb;
                }
                staged += total;
            } else {
                // more than the stage holds (large multiplicities): straight to the bank
                uint64_t base = 0;
                if (lane == 0) base = atomicAdd(reinterpret_cast<unsigned long long*>(P.out_count), total);
                base = lane_value(base, 0);
                for (uint32_t k = 1; k <= n; ++k)
                    bank_store(P, base + off + (k - 1), p.x, p.t, murmur_hash(k, p.Z >> P.lcg.up) << P.lcg.up, p.batch, p.tb);
            }
        }
        active = false;
    }
    if (staged != 0) bank_flush(P, S, staged, lane);
    if (PC && cstaged != 0) census_flush(P, CS, cstaged, lane);
    tally_lds_end<BLOCK>(P, lds_counts);
    flush_lane_counters<BLOCK>(P, c);
}

// A source of a wave's chunk, seeded when the chunk is taken.
struct __align__(16) FamilySource {
    uint64_t X;
    uint32_t batch;
    uint32_t pad;
};

// ------------------------------------------------------------ pool kernel (bank schedule)

// Hash seeding lets any lane run any particle, so a wave works as one
// depth-first walker with 64 hands: a lane runs a line of descent (the first
// particle emerging from each scattering) in registers, the siblings go to the
// wave's pool in LDS, and a lane whose line ended takes the newest particle
// of the pool; new items only when the pool is empty.  All lanes fly in every
// iteration, and no particle touches HBM while the pool fits (one iteration
// adds about 7 entries net on the paper's problem, a particle lives about
// `census time` iterations, so about 140 wait at a time).
//   The kernel is bound by vector issue where sources are many (about 190
// instructions per flight at full lanes), by the chains of the longest
// families where they are few.  Generations in HBM (the schedule's former
// kernel: one launch and one read-back per generation, 32 B each way per
// banked particle, waves waiting on the append counter) took 5.9 ms for the
// paper's 1000 x 1000 sources, now 0.86; 5.6 ms for 4096 sources to t = 60, now
// 0.68; 3e7 sources took 101 ms (41.5 as families), now 14.7.
//   Where particles go when the LDS pool is full: its older half to the wave's
// private HBM stack (priv_cap entries, read back when the pool is empty); when
// that is full too, to the launch's output bank; and once the wave has seen
// more than out_budget entries there (or cen_budget census arrivals), it hands
// over everything it holds and ends, so that appends stay within
// out_budget + slack per wave.  A wave also hands over what is left tail_iters
// (32) iterations after the launch's items are taken: families are heavy-tailed,
// and the next launch spreads the rest over all waves.
// LDS entries of a wave's pool.  256 entries leave four 256-thread blocks per
// CU, 128 six: 1000 x 1000 sources 827 against 881 us (more goes through the
// private stack), 4096 sources to t = 60 821 against 659 (more waves in
// flight where each one waits on its own chain).
constexpr uint32_t kPoolEntries = 128;
// Two planes of 16 bytes per entry: consecutive lanes touch consecutive banks
// (entries of 32 bytes side by side conflict two ways).
template <uint32_t CAP>
struct PoolPlanes {
    struct __align__(16) Half {
        uint64_t a, b;
    };
    Half xt[CAP], kb[CAP];
    __device__ __forceinline__ PulsePoolEntry get(uint32_t i) const {
        const Half p = xt[i & (CAP - 1)], q = kb[i & (CAP - 1)];
        PulsePoolEntry e;
        e.x = __longlong_as_double(static_cast<long long>(p.a));
        e.t = __longlong_as_double(static_cast<long long>(p.b));
        e.key = q.a;
        e.batch = static_cast<uint32_t>(q.b);
        e.meta = static_cast<uint32_t>(q.b >> 32);
        return e;
    }
    __device__ __forceinline__ void put(uint32_t i, const PulsePoolEntry& e) {
        Half p, q;
        p.a = static_cast<uint64_t>(__double_as_longlong(e.x));
        p.b = static_cast<uint64_t>(__double_as_longlong(e.t));
        q.a = e.key;
        q.b = (static_cast<uint64_t>(e.meta) << 32) | e.batch;
        xt[i & (CAP - 1)] = p;
        kb[i & (CAP - 1)] = q;
    }
};
constexpr uint32_t kPoolCensusStage = 64;
constexpr uint32_t kRowFlushMask = (1u << 25) - 1u;   // iterations between forced row flushes (32-bit counters)

// (k M ^ (k M >> 47)) M: the part of hash(k, s) that depends on k only.
__device__ __forceinline__ uint64_t child_part(uint64_t k) {
    const uint64_t y = k * kMurmurM;
    return (y ^ (y >> 47)) * kMurmurM;
}
// Start state (top-aligned) of child k of a parent that ended in state X (eq. 5).
__device__ __forceinline__ uint64_t child_state(const LcgDev& L, uint64_t X, uint64_t part) {
    return murmur_sub(murmur_seed_part(X) ^ part) << L.up;
}

// The launch's parameters, read again where they are used: for code that runs
// rarely (a chunk taken, a pool spilled), so that its pointers and sizes do not
// sit in (or spill from) the scalar registers of the flight loop.
__device__ __forceinline__ const PulseParams& rare_params() {
    using Arg = const __attribute__((address_space(4))) PulseParams*;
    uint64_t p = reinterpret_cast<uint64_t>(__builtin_amdgcn_kernarg_segment_ptr());
    asm volatile("" : "+s"(p));
    return *(const PulseParams*)(Arg)p;
}

// Tallies of a wave of the pool and stride kernels.  All counters in the
// block's LDS copy when they fit; else rows of n_time_bins counters in LDS, one
// per batch the wave works on (row b mod P.rows, tagged); collisions of a batch
// without a row count in HBM.  Atomics on one address pass one after another,
// about 10 ns each: where few batches share the counters (P.merge_far) the lanes
// of one counter go as one atomic.  With an atomic per lane 1e6 sources whose
// collisions fall into one of 600 bins took 689 ms (now in LDS: 19), 4 x 200000
// sources 200 ms (now 20); the former schedules, in LDS or merged, 41.
struct WaveTally {
    unsigned long long* counters;   // the block's copy (P.lds_tally)
    uint32_t* rows;
    uint32_t* tags;
    uint32_t nt, lane;
    uint32_t hot, cold;   // MERGE: wave-uniform, iterations to go on merging, iterations without
    __device__ __forceinline__ void begin(const PulseParams& P) {
        hot = 16u;
        cold = 0u;
        if (P.rows != 0) {
            for (uint32_t i = lane; i < P.rows * nt; i += 64u) rows[i] = 0u;
            if (lane < 8u) tags[lane] = 0xffffffffu;
        }
    }
    __device__ __forceinline__ void flush_row(uint32_t r) {
        const PulseParams& R = rare_params();
        const uint32_t tag = __builtin_amdgcn_readfirstlane(tags[r]);
        if (tag == 0xffffffffu) return;
        unsigned long long* c = reinterpret_cast<unsigned long long*>(R.counts) + static_cast<uint64_t>(tag) * nt;
        for (uint32_t i = lane; i < nt; i += 64u) {
            const uint32_t v = rows[r * nt + i];
            if (v != 0u) {
                atomicAdd(c + i, static_cast<unsigned long long>(v));
                rows[r * nt + i] = 0u;
            }
        }
    }
    __device__ __forceinline__ void flush(const PulseParams& P) {
        for (uint32_t r = 0; r < P.rows; ++r) flush_row(r);
    }
    // gives the batches of the lanes in m a row each (another batch's row with
    // the same index goes to HBM first)
    __device__ __forceinline__ void claim(const PulseParams& P, uint64_t m, uint32_t batch) {
        while (m != 0) {
            const uint32_t b = __builtin_amdgcn_readlane(batch, __builtin_ctzll(m));
            const uint32_t r = b & (P.rows - 1u);
            if (__builtin_amdgcn_readfirstlane(tags[r]) != b) {
                flush_row(r);
                if (lane == 0) tags[r] = b;
                __builtin_amdgcn_wave_barrier();
            }
            m &= ~wave_mask(batch == b);
        }
    }
    // MERGE: P.merge_far != 0 (forms of their own: the code costs the study 2%
    // where it never runs)
    template <bool MERGE>
    __device__ __forceinline__ void add(const PulseParams& P, uint64_t scored, uint32_t batch, int32_t bin) {
        if (P.lds_tally) {
            if (in_mask(scored)) atomicAdd(counters + (batch * nt + static_cast<uint32_t>(bin)), 1ull);
            return;
        }
        uint64_t far = scored;
        if (P.rows != 0) {
            const uint32_t r = batch & (P.rows - 1u);
            const uint64_t near = scored & wave_mask(tags[r] == batch);
            if (in_mask(near)) atomicAdd(rows + (__umul24(r, nt) + static_cast<uint32_t>(bin)), 1u);
            far &= ~near;
        }
        // the first lane's counter, and on while at least four lanes share one:
        // up to merge_far that fewer share.  A wave that met no counter of three
        // lanes in its last 16 looks in every eighth of its iterations only: 20 x
        // 5000 sources spread over 600 bins take 433 us (453 looking in each, 370
        // never), 4 x 200000 in one bin 19 ms either way (197 never).
        if (MERGE && far != 0 && (hot != 0u || (++cold & 7u) == 0u)) {
            const PulseParams& R = rare_params();
            unsigned long long* const counts = reinterpret_cast<unsigned long long*>(R.counts);
            hot -= hot != 0u ? 1u : 0u;
            for (uint32_t few = R.merge_far; far != 0 && few != 0u;) {
                const int l = __builtin_ctzll(far);
                const uint32_t b = __builtin_amdgcn_readlane(batch, l), i = __builtin_amdgcn_readlane(bin, l);
                const uint64_t same = far & wave_mask(batch == b) & wave_mask(static_cast<uint32_t>(bin) == i);
                const uint32_t n = mask_count(same);
                if (lane == static_cast<uint32_t>(l))
                    atomicAdd(counts + (static_cast<uint64_t>(b) * nt + i), static_cast<unsigned long long>(n));
                far &= ~same;
                few -= n < 4u ? 1u : 0u;
                hot = n > 2u ? 16u : hot;
            }
        }
        if (far != 0 && in_mask(far))
            atomicAdd(reinterpret_cast<unsigned long long*>(P.counts) +
                          (static_cast<uint64_t>(batch) * nt + static_cast<uint32_t>(bin)), 1ull);
    }
};

// Time bin (-1 before the first edge) of the end times tn of the lanes in m
// (tn below the last edge), whose flights started in bin tb.
__device__ __forceinline__ int32_t flight_bin(const PulseParams& P, const double* l_edges, uint64_t m, double tn, int32_t tb) {
    const uint32_t nt = P.n_time_bins;
    auto edge_at = [&](int32_t i) -> double { return P.edges_lds ? l_edges[i] : P.t_edges[i]; };
    int32_t bin = tb;
    if (P.grid_uniform) {
        int32_t g;   // (the instruction saturates, whatever idle lanes hold)
        asm("v_cvt_i32_f64 %0, %1" : "=v"(g) : "v"((tn - P.t0) * P.inv_dt));
        g = g < 0 ? 0 : g;
        g = g < static_cast<int32_t>(nt) ? g : static_cast<int32_t>(nt) - 1;
        const uint64_t before = wave_mask(tn < edge_at(g)), after = wave_mask(edge_at(g + 1) <= tn);
        bin = g - static_cast<int32_t>(sel_const<1, 0>(before)) + static_cast<int32_t>(sel_const<1, 0>(after));
    } else if (in_mask(m)) {
        while (bin + 1 < static_cast<int32_t>(nt) && edge_at(bin + 1) <= tn) bin++;
    }
    return bin;
}

// Dynamic LDS of both kernels: time edges, the block's counters, the waves' rows.
template <int BLOCK>
__device__ __forceinline__ double* stage_edges(const PulseParams& P, unsigned long long* dyn) {
    double* const l_edges = reinterpret_cast<double*>(dyn);
    if (P.edges_lds)
        for (uint32_t i = threadIdx.x; i <= P.n_time_bins; i += BLOCK) l_edges[i] = P.t_edges[i];
    return l_edges;
}

template <int ITEMS, bool PC, int BLOCK, bool MERGE>
__global__ void __launch_bounds__(BLOCK) k_pulse_pool(PulseParams P) {
    constexpr bool SOURCES = ITEMS == PULSE_ITEMS_SOURCES;
    constexpr bool COPIES = ITEMS == PULSE_ITEMS_COPIES;
    constexpr uint32_t CAP = kPoolEntries;
    constexpr uint32_t kWaves = BLOCK / 64;
    __shared__ PoolPlanes<CAP> s_pool[kWaves];
    __shared__ FamilySource s_src[SOURCES ? kWaves : 1][SOURCES ? 64 : 1];
    __shared__ uint32_t s_tag[kWaves][8];
    __shared__ CensusStageOf<kPoolCensusStage> s_cen[PC ? kWaves : 1];
    __shared__ uint64_t s_part[16];
    __shared__ unsigned long long s_acc[kNDiag];
    extern __shared__ unsigned long long dyn[];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double* const l_edges = stage_edges<BLOCK>(P, dyn);
    WaveTally tally;
    tally.nt = P.n_time_bins;
    tally.lane = lane;
    tally.counters = dyn + (P.edges_lds ? P.n_time_bins + 1 : 0u);
    tally.rows = reinterpret_cast<uint32_t*>(tally.counters) + wid * P.rows * P.n_time_bins;
    tally.tags = s_tag[wid];
    tally.begin(P);
    if (threadIdx.x < 16) s_part[threadIdx.x] = child_part(threadIdx.x);
    if (threadIdx.x < kNDiag) s_acc[threadIdx.x] = 0;
    tally_lds_begin<BLOCK>(P, tally.counters);   // and the barrier for the above

    PoolPlanes<CAP>& pool = s_pool[wid];
    FamilySource* const src = s_src[SOURCES ? wid : 0];
    auto& cen = s_cen[PC ? wid : 0];
    const uint64_t wave = static_cast<uint64_t>(blockIdx.x) * kWaves + wid;
    const uint64_t part1 = child_part(1);
    const double sigma = P.sigma_t;
    const double rsigma = uniform_value(recip_refined(sigma));

    // wave-uniform state
    uint64_t A = 0;                     // lanes holding a particle at the start of its flight
    uint64_t child = 0;                 // of those, lanes whose Z is its parent's final state (start state: eq. 5 with part)
    uint64_t dir = 0;                   // COPIES: lanes whose particle keeps its direction
    uint32_t bot = 0, top = 0;          // the pool holds entries [bot, top) (mod CAP)
    uint32_t npriv = 0;
    // the wave's untaken items [wnext, gend); of sources [wnext, wend) are seeded in src
    uint64_t wnext = P.item_begin + wave * P.first_chunk;
    if (wnext > P.item_part[0]) wnext = P.item_part[0];
    uint64_t gend = wnext + P.first_chunk < P.item_part[0] ? wnext + P.first_chunk : P.item_part[0];
    uint64_t wend = SOURCES ? wnext : gend;
    uint32_t src_off = 0;               // item wnext's place in src
    bool exhausted = P.item_part[0] == P.item_end && wnext == gend, hand_over = false;   // no items left to take
    uint64_t seen = 0;                  // output count after this wave's last append
    uint32_t cstaged = 0, tail = 0, iter = 0;
    uint64_t n_src = 0, n_fly = 0, n_dir = 0, n_coll = 0, n_tal = 0, n_scat = 0, n_extra = 0;
    uint64_t any3 = 0, any4 = 0;        // COPIES: lanes that drew 3 and 4 numbers in a flight with a direction draw
    // the lane's particle
    double x = 0.0, t = 0.0, mu0 = 0.0;
    uint64_t Z = 0, part = part1;
    uint32_t batch = 0;
    int32_t tb = -1;

    // reserves n entries of the output bank (n uniform)
    auto reserve = [&](const PulseParams& R, uint32_t n) -> uint64_t {
        uint64_t base = 0;
        if (lane == 0) base = atomicAdd(reinterpret_cast<unsigned long long*>(R.out_count), static_cast<unsigned long long>(n));
        base = lane_value(base, 0);
        seen = base + n;
        return base;
    };
    auto store_entry = [&](const PulseParams& R, uint64_t o, const PulsePoolEntry& e) {
        bank_store(R, o, e.x, e.t, child_state(R.lcg, e.key, s_part[(e.meta >> 16) & 15u]), e.batch,
                   static_cast<int32_t>(e.meta & 0xffffu) - 1);
    };

    for (;;) {
        uint64_t need = ~A;
        if (need != 0) {
            if (top == bot && npriv != 0) {
                // the newest entries of the private stack
                const PulseParams& R = rare_params();
                const PulsePoolEntry* const priv = R.priv + wave * R.priv_cap;
                const uint32_t cnt = npriv < CAP / 2 ? npriv : CAP / 2;
                npriv -= cnt;
                for (uint32_t i = lane; i < cnt; i += 64u) pool.put(top + i, priv[npriv + i]);
                top += cnt;
                __builtin_amdgcn_wave_barrier();
            }
            uint32_t k = mask_count(need);
            if (top != bot) {
                const uint32_t take = top - bot < k ? top - bot : k;
                const uint32_t rank = mask_rank(need);
                const uint64_t m = need & wave_mask(rank < take);
                if (in_mask(m)) {
                    const PulsePoolEntry e = pool.get(top - 1u - rank);
                    x = e.x;
                    t = e.t;
                    batch = e.batch;
                    tb = static_cast<int32_t>(e.meta & 0xffffu) - 1;
                    Z = e.key;
                    part = s_part[e.meta >> 16];
                }
                top -= take;
                k -= take;
                A |= m;
                child |= m;
                need &= ~m;
                __builtin_amdgcn_wave_barrier();
            }
            if (k != 0 && wnext == wend && !exhausted) {
                const PulseParams& R = rare_params();
                if (wnext == gend) {
                    // (no taking from other blocks' parts: the parts are alike,
                    // and every look at a counter costs as much as a take)
                    const uint32_t s = blockIdx.x & (R.item_parts - 1u);
                    const uint64_t e = R.item_part[s + 1u];
                    uint64_t b = 0;
                    if (lane == 0)
                        b = atomicAdd(reinterpret_cast<unsigned long long*>(R.item_counter + s * kPulseCounterStride),
                                      static_cast<unsigned long long>(R.chunk));
                    b = R.item_part[s] + lane_value(b, 0);
                    wnext = b < e ? b : e;
                    gend = b + R.chunk < e ? b + R.chunk : e;
                    exhausted = wnext == gend;
                    if (ITEMS != PULSE_ITEMS_BANK && R.ranges != nullptr && !exhausted) {
                        gend = uniform_value(R.ranges[2 * b + 1]);
                        wnext = uniform_value(R.ranges[2 * b]);
                    }
                    wend = SOURCES ? wnext : gend;
                }
                if (SOURCES && wnext != gend) {
                    wend = gend - wnext < 64u ? gend : wnext + 64u;
                    const uint64_t j = wnext + lane;
                    if (j < wend) {
                        FamilySource e;
                        e.X = pulse_source_state(R, j, &e.batch);
                        e.pad = 0;
                        src[lane] = e;
                    }
                    src_off = 0;
                    __builtin_amdgcn_wave_barrier();
                }
            }
            if (k != 0 && wnext != wend) {
                const uint64_t avail = wend - wnext;
                const uint32_t take = avail < k ? static_cast<uint32_t>(avail) : k;
                const uint32_t rank = mask_rank(need);
                const uint64_t m = need & wave_mask(rank < take);
                if (in_mask(m)) {
                    const PulseParams& R = rare_params();
                    if (SOURCES) {
                        const FamilySource e = src[src_off + rank];
                        Z = e.X;
                        batch = e.batch;
                        x = 0.0;
                        t = 0.0;
                        tb = R.tb0;
                    } else {
                        PParticle q;
                        load_item<ITEMS>(R, wnext + rank, q);
                        x = q.x;
                        t = q.t;
                        Z = q.Z;
                        batch = q.batch;
                        tb = q.tb;
                        if (COPIES) mu0 = q.mu;
                    }
                }
                if (SOURCES) n_src += take;
                if (COPIES) dir |= m;
                wnext += take;
                src_off += take;
                A |= m;
                if (P.rows != 0) tally.claim(P, m, batch);
            }
        }
        if (A == 0) break;   // no pool, no items
        if (exhausted && ++tail > P.tail_iters) {
            hand_over = true;
            break;
        }
        if ((++iter & kRowFlushMask) == 0) tally.flush(P);

        // one flight of every lane in A (the others compute on what their registers hold)
        if (in_mask(child)) Z = child_state(P.lcg, Z, part);
        child = 0;
        const uint64_t z1 = lcg_next_z(P.lcg, Z);
        double mu = __builtin_fma(uniform_z(z1), 2.0, -1.0);   // exact
        uint64_t z = z1;
        if (COPIES && (dir & A) != 0) {
            mu = sel(dir, mu0, mu);
            z = sel(dir, Z, z1);
        }
        const uint64_t drew = COPIES ? A & ~dir : A;
        z = lcg_next_z(P.lcg, z);
        const double s = quot(fixed_neg_log(uniform_z(z)), sigma, rsigma);
        const double tn = t + s;
        const uint64_t coll = A & wave_mask(tn < P.t_end);
        const uint64_t census = A & ~coll;
        if (PC && census != 0) {
            const uint32_t cnt = mask_count(census);
            if (cstaged + cnt > kPoolCensusStage) {
                const PulseParams& R = rare_params();
                if (census_flush(R, cen, cstaged, lane) > R.cen_budget) hand_over = true;
                cstaged = 0;
            }
            if (in_mask(census)) {
                const uint32_t e = cstaged + mask_rank(census);
                const double rest = P.t_end - t;
                const double step = mu * rest;
                cen.x[e] = x + step;
                cen.mu[e] = mu;
                cen.X[e] = z >> P.lcg.up;
                cen.batch[e] = batch;
            }
            cstaged += cnt;
        }
        const double step = mu * s;
        const double xn = x + step;
        const int32_t bin = flight_bin(P, l_edges, coll, tn, tb);
        const uint64_t scored = coll & wave_mask(bin >= 0) & wave_mask(P.x_lo <= xn) & wave_mask(xn <= P.x_hi);
        tally.add<MERGE>(P, scored, batch, bin);
        const uint64_t z3 = lcg_next_z(P.lcg, z);
        const uint64_t go = coll & wave_mask(z3 < P.scatter_below);
        const uint64_t z4 = lcg_next_z(P.lcg, z3);
        const uint64_t extra = go & wave_mask(z4 < P.frac_below);
        const uint64_t key = z4 >> P.lcg.up;

        n_fly += mask_count(A);
        n_coll += mask_count(coll);
        n_tal += mask_count(scored);
        n_scat += mask_count(go);
        n_extra += mask_count(extra);
        if (COPIES) {
            n_dir += mask_count(drew);
            any4 |= drew & go;
            any3 |= (drew & coll) | (go & dir);
            dir &= ~A;
        }

        // the first emerging particle runs on here, the others go to the pool:
        // n_floor - 1 for every scattering, one more for `extra` (n_floor = 0: none)
        if (in_mask(go)) {
            x = xn;
            t = tn;
            tb = bin;
            Z = key;
            part = part1;
        }
        const uint32_t n_more = P.n_floor != 0 ? (P.n_floor - 1u) * mask_count(go) + mask_count(extra) : 0u;
        if (n_more != 0) {
            const uint32_t off = (P.n_floor - 1u) * mask_rank(go) + mask_rank(extra);
            const uint32_t n = P.n_floor + sel_const<1, 0>(extra);
            bool direct = n_more > CAP;   // large multiplicities
            if (!direct && top - bot + n_more > CAP) {
                const PulseParams& R = rare_params();
                while (!direct && top - bot + n_more > CAP) {
                    const uint32_t cnt = top - bot < CAP / 2 ? top - bot : CAP / 2;
                    if (npriv + cnt <= R.priv_cap) {
                        PulsePoolEntry* const priv = R.priv + wave * R.priv_cap;
                        for (uint32_t i = lane; i < cnt; i += 64u) priv[npriv + i] = pool.get(bot + i);
                        npriv += cnt;
                    } else if (seen <= R.out_budget) {
                        const uint64_t base = reserve(R, cnt);
                        for (uint32_t i = lane; i < cnt; i += 64u) store_entry(R, base + i, pool.get(bot + i));
                    } else {
                        direct = hand_over = true;
                        break;
                    }
                    bot += cnt;
                    __builtin_amdgcn_wave_barrier();
                }
            }
            if (direct) {
                const PulseParams& R = rare_params();
                const uint64_t base = reserve(R, n_more);
                if (seen > R.out_budget) hand_over = true;
                if (in_mask(go))
                    for (uint32_t c = 2; c <= n; ++c)
                        bank_store(R, base + off + (c - 2u), x, t, child_state(R.lcg, key, s_part[c]), batch, tb);
            } else {
                if (in_mask(go))
                    for (uint32_t c = 2; c <= n; ++c) {
                        PulsePoolEntry e;
                        e.x = x;
                        e.t = t;
                        e.key = key;
                        e.batch = batch;
                        e.meta = (c << 16) | static_cast<uint32_t>(tb + 1);
                        pool.put(top + off + (c - 2u), e);
                    }
                top += n_more;
                __builtin_amdgcn_wave_barrier();
            }
        }
        A = P.n_floor != 0 ? go : extra;
        child = A;
        if (hand_over) break;
    }

    const PulseParams& R = rare_params();
    if (hand_over) {
        // everything the wave holds goes to the output bank (every lane in A
        // is past its first flight here, so no direction is lost); items
        // taken but not started go there too, or back to the host as a range
        const PulsePoolEntry* const priv = R.priv + wave * R.priv_cap;
        const uint32_t nl = mask_count(A), np = top - bot;
        uint32_t ni = 0;
        if (ITEMS == PULSE_ITEMS_BANK) ni = static_cast<uint32_t>(gend - wnext);
        if (ITEMS != PULSE_ITEMS_BANK && gend != wnext && lane == 0) {
            const uint64_t o = atomicAdd(reinterpret_cast<unsigned long long*>(R.n_left), 1ull);
            R.left[2 * o] = wnext;
            R.left[2 * o + 1] = gend;
        }
        const uint64_t base = reserve(R, nl + np + npriv + ni);
        if (in_mask(child)) Z = child_state(R.lcg, Z, part);
        if (in_mask(A)) bank_store(R, base + mask_rank(A), x, t, Z, batch, tb);
        for (uint32_t i = lane; i < np; i += 64u) store_entry(R, base + nl + i, pool.get(bot + i));
        for (uint32_t i = lane; i < npriv; i += 64u) store_entry(R, base + nl + np + i, priv[i]);
        if (ITEMS == PULSE_ITEMS_BANK)
            for (uint32_t i = lane; i < ni; i += 64u) {
                const uint64_t j = wnext + i;
                bank_store(R, base + nl + np + npriv + i, R.in.x[j], R.in.t[j], R.in.X[j], R.in.batch[j], R.in.tb[j]);
            }
    }
    if (PC && cstaged != 0) census_flush(R, cen, cstaged, lane);
    tally.flush(P);
    if (lane == 0) {
        auto add = [&](int w, uint64_t v) { atomicAdd(&s_acc[w], static_cast<unsigned long long>(v)); };
        add(PD_SOURCES, n_src);
        add(PD_COLLISIONS, n_coll);
        add(PD_TALLIED, n_tal);
        add(PD_SCATTERS, n_scat);
        add(PD_ABSORBED, n_coll - n_scat);
        add(PD_CENSUS, n_fly - n_coll);
        add(PD_SECONDARIES, n_scat * P.n_floor + n_extra);
        add(PD_DRAWS, (COPIES ? n_dir : n_fly) + n_fly + n_coll + n_scat);
        // numbers of the longest stream: direction, flight, absorption test, multiplicity
        uint32_t d = n_scat != 0 ? 4u : (n_coll != 0 ? 3u : (n_fly != 0 ? 2u : 0u));
        if (COPIES) d = any4 != 0 ? 4u : (any3 != 0 ? 3u : ((n_dir | n_coll) != 0 ? 2u : (n_fly != 0 ? 1u : 0u)));
        atomicMax(&s_acc[PD_MAX_DRAWS], static_cast<unsigned long long>(d));
    }
    tally_lds_end<BLOCK>(P, tally.counters);
    __syncthreads();
    if (threadIdx.x < kNDiag && s_acc[threadIdx.x] != 0) {
        unsigned long long* d = reinterpret_cast<unsigned long long*>(R.diag) + threadIdx.x;
        if (threadIdx.x == PD_MAX_DRAWS)
            atomicMax(d, s_acc[threadIdx.x]);
        else
            atomicAdd(d, s_acc[threadIdx.x]);
    }
}

// ------------------------------------------------------------ stride kernel

// Families of stride seeding: one source family per lane, depth first on the
// source's one stream.  Every lane flies in every iteration: a line that ends
// goes on with the stack's newest sibling, a family that ends with the wave's
// next source.  A lane's stack entry holds the siblings of one scattering
// still to start (x, t, their number and the time bin); its newest
// kStrideDepth entries lie in LDS, one plane per depth (entry d of every lane
// side by side), the older ones in HBM planes (entry d of lane l of the launch
// at d * lanes + l): when the LDS part is full its oldest entry moves out, and
// back when the lane runs out of newer ones (read one flight ahead: some lane
// of a wave needs one in nearly every iteration).
//   The kernel is bound by vector issue and the chains of one wave's flight
// (about 230 instructions; vector units 77% busy).  Against the walk it
// replaces (every entry below the top in HBM, the phases of a family as
// branches: 358 instructions per flight, 108 GB of stack traffic) the
// 3e7-source study went from 38 ms to 19 (18.1 to 19.6 from run to run).
// LDS entries per lane: a power of two, so that an entry's place is its depth
// masked (with 6 entries, a running place and stack addresses computed where
// they are used the study took 5% longer at 237 instructions per flight, now
// 227; that form took 23.9 ms at 3 entries, 19.7 at 6 and 22 at 7, three blocks
// per CU).
constexpr uint32_t kStrideDepth = 4;   // a power of two
constexpr uint32_t kStrideRefill = 3;  // idle lanes at which a wave takes sources (a family ends in 60% of its iterations)

template <int BLOCK, bool MERGE>
__global__ void __launch_bounds__(BLOCK) k_pulse_stride(PulseParams P) {
    constexpr uint32_t kWaves = BLOCK / 64;
    __shared__ double s_xt[kWaves][2][kStrideDepth][64];   // x and t planes
    __shared__ uint32_t s_m[kWaves][kStrideDepth][64];   // siblings left << 16 | time bin + 1
    __shared__ FamilySource s_src[kWaves][64];
    __shared__ uint32_t s_tag[kWaves][8];
    __shared__ unsigned long long s_acc[kNDiag];
    extern __shared__ unsigned long long dyn[];
    const uint32_t lane = threadIdx.x & 63u;
    const uint32_t wid = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    double* const l_edges = stage_edges<BLOCK>(P, dyn);
    WaveTally tally;
    tally.nt = P.n_time_bins;
    tally.lane = lane;
    tally.counters = dyn + (P.edges_lds ? P.n_time_bins + 1 : 0u);
    tally.rows = reinterpret_cast<uint32_t*>(tally.counters) + wid * P.rows * P.n_time_bins;
    tally.tags = s_tag[wid];
    tally.begin(P);
    if (threadIdx.x < kNDiag) s_acc[threadIdx.x] = 0;
    tally_lds_begin<BLOCK>(P, tally.counters);   // and the barrier for the above

    constexpr uint32_t kT = kStrideDepth * 64u;
    double* const sx = &s_xt[wid][0][0][lane];   // entry d at [d mod kStrideDepth x 64], its t at + kT
    uint32_t* const sm = &s_m[wid][0][lane];
    FamilySource* const src = s_src[wid];
    const uint64_t lanes = static_cast<uint64_t>(gridDim.x) * BLOCK;
    const uint64_t gl = static_cast<uint64_t>(blockIdx.x) * BLOCK + threadIdx.x;
    const uint64_t wave = static_cast<uint64_t>(blockIdx.x) * kWaves + wid;
    const double sigma = P.sigma_t;
    const double rsigma = uniform_value(recip_refined(sigma));

    uint64_t A = 0;                     // lanes with a family
    uint64_t wnext = P.item_begin + wave * P.first_chunk;   // the wave's untaken sources [wnext, gend), seeded up to wend
    if (wnext > P.item_part[0]) wnext = P.item_part[0];
    uint64_t gend = wnext + P.first_chunk < P.item_part[0] ? wnext + P.first_chunk : P.item_part[0];
    uint64_t wend = wnext;
    uint32_t src_off = 0;
    bool exhausted = P.item_part[0] == P.item_end && wnext == gend;
    uint32_t iter = 0;
    uint64_t n_src = 0, n_fly = 0, n_coll = 0, n_tal = 0, n_scat = 0, n_extra = 0;
    uint64_t max_draws = 0, over = 0;   // per lane
    double x = 0.0, t = 0.0;
    uint64_t Z = 0, draws = 0;
    uint32_t batch = 0, depth = 0, low = 0;   // entries of the lane's stack, and those of them in HBM
    PulseStackEntry ahead{};            // entry ahead_of - 1, read ahead from HBM
    uint32_t ahead_of = 0;
    // the next entry's place in HBM (entry `low`), and the first one's
    PulseStackEntry* const hbm0 = P.stack + gl;
    PulseStackEntry* hbm = hbm0;
    uint32_t max_depth;                 // in a vector register: the loop's scalar ones are full
    asm("v_mov_b32 %0, %1" : "=v"(max_depth) : "s"(P.stack_depth));
    auto place = [](uint32_t d) { return (d & (kStrideDepth - 1u)) * 64u; };
    int32_t tb = -1;

    for (;;) {
        const uint64_t need = ~A;
        if ((mask_count(need) >= kStrideRefill || A == 0) && !exhausted) {
            if (wnext == wend) {
                const PulseParams& R = rare_params();
                if (wnext == gend) {
                    const uint32_t s = blockIdx.x & (R.item_parts - 1u);
                    const uint64_t e = R.item_part[s + 1u];
                    uint64_t b = 0;
                    if (lane == 0)
                        b = atomicAdd(reinterpret_cast<unsigned long long*>(R.item_counter + s * kPulseCounterStride),
                                      static_cast<unsigned long long>(R.chunk));
                    b = R.item_part[s] + lane_value(b, 0);
                    wnext = b < e ? b : e;
                    gend = b + R.chunk < e ? b + R.chunk : e;
                    exhausted = wnext == gend;
                }
                wend = gend - wnext < 64u ? gend : wnext + 64u;
                const uint64_t j = wnext + lane;
                if (j < wend) {
                    FamilySource e;
                    e.X = pulse_source_state(R, j, &e.batch);
                    e.pad = 0;
                    src[lane] = e;
                }
                src_off = 0;
                __builtin_amdgcn_wave_barrier();
            }
            const uint64_t avail = wend - wnext;
            const uint32_t k = mask_count(need);
            const uint32_t take = avail < k ? static_cast<uint32_t>(avail) : k;
            const uint32_t rank = mask_rank(need);
            const uint64_t m = need & wave_mask(rank < take);
            if (in_mask(m)) {
                const FamilySource e = src[src_off + rank];
                Z = e.X;
                batch = e.batch;
                x = 0.0;
                t = 0.0;
                tb = P.tb0;
                draws = 0;
            }
            n_src += take;
            wnext += take;
            src_off += take;
            A |= m;
            if (P.rows != 0 && m != 0) tally.claim(P, m, batch);
        }
        if (A == 0) {
            if (exhausted) break;
            continue;
        }
        if ((++iter & kRowFlushMask) == 0) tally.flush(P);

        // one flight of every lane in A (the others compute on what their registers hold)
        const uint64_t z1 = lcg_next_z(P.lcg, Z);
        const double mu = __builtin_fma(uniform_z(z1), 2.0, -1.0);   // exact
        const uint64_t z2 = lcg_next_z(P.lcg, z1);
        const double s = quot(fixed_neg_log(uniform_z(z2)), sigma, rsigma);
        const double tn = t + s;
        const uint64_t coll = A & wave_mask(tn < P.t_end);
        const double step = mu * s;
        const double xn = x + step;
        const int32_t bin = flight_bin(P, l_edges, coll, tn, tb);
        const uint64_t scored = coll & wave_mask(bin >= 0) & wave_mask(P.x_lo <= xn) & wave_mask(xn <= P.x_hi);
        tally.add<MERGE>(P, scored, batch, bin);
        const uint64_t z3 = lcg_next_z(P.lcg, z2);
        const uint64_t go = coll & wave_mask(z3 < P.scatter_below);
        const uint64_t z4 = lcg_next_z(P.lcg, z3);
        const uint64_t extra = go & wave_mask(z4 < P.frac_below);
        // the stream goes on from the last number drawn: two of a flight that
        // reached the end, three of an absorption, four of a scattering
        Z = sel(go, z4, sel(coll, z3, z2));
        draws += 2u + sel_const<1, 0>(coll) + sel_const<1, 0>(go);
        n_fly += mask_count(A);
        n_coll += mask_count(coll);
        n_tal += mask_count(scored);
        n_scat += mask_count(go);
        n_extra += mask_count(extra);

        // the first emerging particle runs on; its siblings wait on the stack
        const uint64_t on = P.n_floor != 0 ? go : extra;
        const uint64_t push = P.n_floor >= 2u ? go : (P.n_floor == 1u ? extra : 0ull);
        if (in_mask(go)) {
            x = xn;
            t = tn;
            tb = bin;
        }
        uint64_t lost = 0;   // lanes whose stack would grow past stack_depth: the family is abandoned
        if (push != 0) {
            lost = push & wave_mask(depth == max_depth);
            const uint64_t full = push & ~lost & wave_mask(depth - low == kStrideDepth);
            const uint32_t o = place(depth);   // of the oldest entry in LDS too when they fill it
            if (full != 0 && in_mask(full)) {
                PulseStackEntry e;
                e.x = sx[o];
                e.t = sx[o + kT];
                e.key = sm[o];
                *hbm = e;
                hbm += lanes;
                low++;
            }
            if (in_mask(push & ~lost)) {
                sx[o] = x;
                sx[o + kT] = t;
                sm[o] = ((P.n_floor - 1u + sel_const<1, 0>(extra)) << 16) | static_cast<uint32_t>(tb + 1);
                depth++;
            }
        }
        // lines that ended: the newest sibling, or the end of the family
        const uint64_t ended = A & ~on;
        const uint64_t back = ended & wave_mask(depth != 0);
        const uint64_t dry = back & wave_mask(depth == low);
        const uint32_t o = place(depth - 1u);
        if (dry != 0 && in_mask(dry)) {
            low--;
            hbm -= lanes;
            sx[o] = ahead.x;
            sx[o + kT] = ahead.t;
            sm[o] = static_cast<uint32_t>(ahead.key);
            ahead_of = 0;
        }
        if (in_mask(back)) {
            const uint32_t m = sm[o];
            x = sx[o];
            t = sx[o + kT];
            tb = static_cast<int32_t>(m & 0xffffu) - 1;
            const uint64_t last = wave_mask(m < (2u << 16));
            sm[o] = m - (1u << 16);
            depth -= sel_const<1, 0>(last);
        }
        // a lane whose next sibling is in HBM reads it now: it flies at least
        // once before it needs it
        const uint64_t fetch = A & wave_mask(depth == low) & wave_mask(low != 0) & wave_mask(ahead_of != low);
        if (fetch != 0 && in_mask(fetch)) {
            ahead = *(hbm - lanes);
            ahead_of = low;
        }
        const uint64_t end = (ended & ~back) | lost;
        if (end != 0) {
            if (in_mask(end)) {
                max_draws = draws > max_draws ? draws : max_draws;
                if (draws > P.stride_q) over++;
                depth = 0;
                low = 0;
                hbm = hbm0;
                ahead_of = 0;
            }
            A &= ~end;
            if (lost != 0) {
                const PulseParams& R = rare_params();
                if (lane == 0) atomicOr(R.overflow, 1u);
            }
        }
    }

    const PulseParams& R = rare_params();
    tally.flush(P);
    atomicMax(&s_acc[PD_MAX_DRAWS], static_cast<unsigned long long>(max_draws));
    atomicAdd(&s_acc[PD_OVER_STRIDE], static_cast<unsigned long long>(over));
    if (lane == 0) {
        auto add = [&](int w, uint64_t v) { atomicAdd(&s_acc[w], static_cast<unsigned long long>(v)); };
        add(PD_SOURCES, n_src);
        add(PD_COLLISIONS, n_coll);
        add(PD_TALLIED, n_tal);
        add(PD_SCATTERS, n_scat);
        add(PD_ABSORBED, n_coll - n_scat);
        add(PD_CENSUS, n_fly - n_coll);
        add(PD_SECONDARIES, n_scat * P.n_floor + n_extra);
        add(PD_DRAWS, 2 * n_fly + n_coll + n_scat);
    }
    tally_lds_end<BLOCK>(P, tally.counters);
    __syncthreads();
    if (threadIdx.x < kNDiag && s_acc[threadIdx.x] != 0) {
        unsigned long long* d = reinterpret_cast<unsigned long long*>(R.diag) + threadIdx.x;
        if (threadIdx.x == PD_MAX_DRAWS)
            atomicMax(d, s_acc[threadIdx.x]);
        else
            atomicAdd(d, s_acc[threadIdx.x]);
    }
}

// ------------------------------------------------------------ family schedule

// Banks the particles of keys k0..k1 emerging from a scattering of state
// key at (x, t, tb): a finish launch leaves them to the next generation.
__device__ __forceinline__ void spill(const PulseParams& P, double x, double t, int32_t tb, uint32_t batch,
                                      uint64_t key, uint32_t k0, uint32_t k1) {
    if (k1 < k0) return;
    const uint64_t base = atomicAdd(reinterpret_cast<unsigned long long*>(P.out_count),
                                    static_cast<unsigned long long>(k1 - k0 + 1));
    for (uint32_t k = k0; k <= k1; ++k)
        bank_store(P, base + (k - k0), x, t, murmur_hash(k, key) << P.lcg.up, batch, tb);
}

// ITEMS = sources: the family schedule.  ITEMS = a generation bank (hash
// seeding): a finish launch, which runs each input particle's descendants
// depth first as well, up to P.lane_budget particles per input particle;
// what is left then (the first emerging particle and the stack), and
// siblings that find the stack full, go to the output bank.  So a finish
// launch appends at most (budget + stack_depth + 1) n_max particles and
// banks at most `budget` census arrivals per input particle.
constexpr uint32_t kFamilyChunk = 64;   // items a wave of the family kernel takes per atomic

// A family of a chunk with a tally slot has ended: the lane whose end leaves
// the chunk with no family marks the slot for its wave's flush.
__device__ __forceinline__ void family_ended(uint32_t* slot_alive, int32_t& lsl) {
    if (lsl < 0) return;
    const int32_t s = lsl >> 16;
    lsl = atomicSub(slot_alive + s, 1u) == 1u ? -2 - s : -1;
}

// Banks a lane's whole stack, bottom entry first: the sp entries in HBM,
// then the top entry.
__device__ __forceinline__ void spill_stack(const PulseParams& P, const PulseStackEntry* stack, uint64_t sstride,
                                            uint32_t sp, const PulseStackEntry& top, bool has_top, uint32_t batch) {
    for (uint32_t i = 0; i < sp; ++i) {
        const PulseStackEntry& e = stack[static_cast<uint64_t>(i) * sstride];
        spill(P, e.x, e.t, e.tb, batch, e.key, e.next, e.n);
    }
    if (has_top) spill(P, top.x, top.t, top.tb, batch, top.key, top.next, top.n);
}

template <int ITEMS, bool PC, int BLOCK, bool DEEP, bool SLOTS>
__global__ void __launch_bounds__(BLOCK) k_pulse_family(PulseParams P) {
    constexpr bool SOURCES = ITEMS == PULSE_ITEMS_SOURCES;
    constexpr bool SPILL = !SOURCES;
    constexpr bool DIR = PC;   // census arrivals keep their direction
    __shared__ CensusStage cstage[PC ? BLOCK / 64 : 1];
    extern __shared__ unsigned long long lds_counts[];
    tally_lds_begin<BLOCK>(P, lds_counts);
    PulseLane c;
    const uint32_t lane = threadIdx.x & 63u;
    const uint64_t gl = static_cast<uint64_t>(blockIdx.x) * BLOCK + threadIdx.x;
    // The lane's stack.  DEEP (many families per lane): its top entry in
    // registers (top, valid if has_top), the entries below it in HBM, entry d
    // of every lane of the launch in one plane (stack[d * sstride]), so that
    // a wave's lanes at one depth share lines and the planes in use are a few
    // dense regions.  Otherwise every entry in HBM, the lane's own entries
    // contiguous (stack[d]), the top updated in place: a lane that runs alone
    // on its SIMD waits for each entry anyway, and the registers the top
    // would take cost occupancy.
    PulseStackEntry* const stack = DEEP ? P.stack + gl : P.stack + gl * P.stack_depth;
    const uint64_t sstride = DEEP ? static_cast<uint64_t>(gridDim.x) * BLOCK : 1ull;
    // sources: the wave's current chunk, seeded at once (one per lane) when
    // the chunk is taken, so that a lane taking a source reads it from LDS
    __shared__ FamilySource s_src[SOURCES ? BLOCK / 64 : 1][SOURCES ? kFamilyChunk : 1];
    FamilySource* const ring = s_src[SOURCES ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0];
    uint64_t cbase = 0;        // wave-uniform: the item of ring[0]
    // Tally slots (SLOTS: sources, counters that do not fit one LDS copy per
    // block): each chunk of sources the wave takes gets a slot of
    // 2 x n_time_bins counters in LDS (its sources span at most two batches);
    // its families count there, and the slot goes to HBM once the chunk's
    // last family has ended.  With no slot free the chunk counts straight
    // into HBM.
    constexpr bool SL = SOURCES && SLOTS;
    const uint32_t nslots = SL ? P.tally_slots : 0u;
    const uint32_t nt = P.n_time_bins;
    __shared__ uint32_t s_slot[SL ? BLOCK / 64 : 1][SL ? 2 * kPulseTallySlots : 1];
    uint32_t* const slot_alive = s_slot[SL ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0];
    uint32_t* const slot_b0 = slot_alive + (SL ? kPulseTallySlots : 0);   // first batch of the slot's chunk
    unsigned long long* const wslots =
        lds_counts + static_cast<size_t>(__builtin_amdgcn_readfirstlane(threadIdx.x >> 6)) * nslots * 2u * nt;
    if (SL)
        for (uint32_t i = lane; i < nslots * 2u * nt; i += 64u) wslots[i] = 0ull;
    uint32_t free_mask = nslots >= 32 ? 0xffffffffu : (1u << nslots) - 1u;   // wave-uniform
    int32_t cur_slot = -1;     // wave-uniform: the current chunk's slot
    uint32_t cur_b0 = 0;       // wave-uniform: the current chunk's first batch
    // the lane's family: slot s and the counter of its batch's time bin 0
    // in wslots as (s << 16) | base; -1: counts go to HBM; -2 - s: the lane
    // ended the last family of slot s's chunk (flushed at the next top)
    int32_t lsl = -1;
    CensusStage& CS = cstage[PC ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0];
    uint32_t cstaged = 0;      // wave-uniform: entries in CS
    uint32_t sp = 0;           // entries in HBM (DEEP: below the top)
    PulseStackEntry top{};
    bool has_top = false;
    const uint64_t n_items = SOURCES ? P.src_end - P.src_begin : P.n_in;

    PParticle p;
    p.x = p.t = 0.0;
    p.Z = 0;
    p.tb = -1;
    p.batch = 0;
    p.mu = 0.0;
    p.has_mu = false;
    bool active = false;       // the lane holds a particle of a family
    bool exhausted = false;    // wave-uniform: the item counter has passed the end
    uint64_t wnext = 0, wend = 0;   // wave-uniform: the wave's untaken items [wnext, wend)
    uint32_t pdraws = 0;       // draws of the current particle
    uint32_t budget = 0;       // finish: particles the current item may still start

    for (;;) {
        if (SL) {
            // slots whose chunk has no family left: add them to HBM, clear, free
            uint64_t fm = __ballot(lsl <= -2);
            while (fm != 0) {
                const int leader = __ffsll(static_cast<long long>(fm)) - 1;
                const uint32_t s = static_cast<uint32_t>(-2 - __builtin_amdgcn_readlane(lsl, leader));
                const uint64_t c0 = static_cast<uint64_t>(slot_b0[s]) * nt;
                unsigned long long* const sc = wslots + static_cast<size_t>(s) * 2u * nt;
                for (uint32_t i = lane; i < 2u * nt; i += 64u) {
                    const unsigned long long v = sc[i];
                    if (v != 0ull) {
                        if (c0 + i < P.n_counters) atomicAdd(reinterpret_cast<unsigned long long*>(P.counts) + c0 + i, v);
                        sc[i] = 0ull;
                    }
                }
                free_mask |= 1u << s;
                fm &= fm - 1ull;
            }
            if (lsl <= -2) lsl = -1;
        }
        // lanes without a family take the next items from the wave's chunk
        // (one atomic per kFamilyChunk items: the counter is one address
        // for the whole GPU)
        const uint64_t need = __ballot(!active);
        if (need != 0 && wnext == wend && !exhausted) {
            uint64_t b = 0;
            if (lane == 0) b = atomicAdd(reinterpret_cast<unsigned long long*>(P.family_counter), kFamilyChunk);
            b = lane_value(b, 0);
            if (b + kFamilyChunk >= n_items) exhausted = true;
            wnext = b < n_items ? b : n_items;
            wend = b + kFamilyChunk < n_items ? b + kFamilyChunk : n_items;
            if (SOURCES) {
                const uint64_t j = wnext + lane;
                if (j < wend) {
                    FamilySource e;
                    e.X = pulse_source_state(P, P.src_begin + j, &e.batch);
                    e.pad = 0;
                    ring[lane] = e;
                }
                cbase = wnext;
                __builtin_amdgcn_wave_barrier();
                cur_slot = -1;
                if (SL && nslots != 0 && free_mask != 0 && wend > wnext) {
                    cur_slot = __builtin_ctz(free_mask);
                    free_mask &= free_mask - 1u;
                    cur_b0 = ring[0].batch;
                    if (lane == 0) {
                        slot_alive[cur_slot] = static_cast<uint32_t>(wend - wnext);
                        slot_b0[cur_slot] = cur_b0;
                    }
                    __builtin_amdgcn_wave_barrier();
                }
            }
        }
        if (need != 0 && wnext != wend) {
            const uint64_t avail = wend - wnext;
            const uint32_t nneed = static_cast<uint32_t>(__popcll(need));
            const uint32_t take = avail < nneed ? static_cast<uint32_t>(avail) : nneed;
            const uint32_t rank = lane_prefix(need);
            const uint64_t wbase = wnext;
            wnext += take;
            if (!active && rank < take) {
                const uint64_t j = wbase + rank;
                if (SOURCES) {
                    const FamilySource e = ring[j - cbase];
                    p.Z = e.X;
                    p.batch = e.batch;
                    if (SL)
                        lsl = cur_slot >= 0 ? (cur_slot << 16) | static_cast<int32_t>(static_cast<uint32_t>(cur_slot) * 2u * nt +
                                                                                    (e.batch - cur_b0) * nt)
                                            : -1;
                    p.x = 0.0;
                    p.t = 0.0;
                    p.tb = P.tb0;
                    c.sources++;
                } else {
                    load_item<ITEMS>(P, j, p);
                }
                pdraws = 0;
                sp = 0;
                has_top = false;
                budget = P.lane_budget;
                active = true;
            }
        }
        if (__ballot(active) == 0 && wnext == wend && exhausted) break;
        uint32_t n = 0;
        int64_t tally = -1;
        bool at_census = false;
        if (active) n = pulse_particle<DIR>(P, p, c, &pdraws, &tally, &at_census);
        if (SL) {
            if (tally >= 0 && lsl >= 0)
                atomicAdd(wslots + (lsl & 0xffff) + static_cast<uint32_t>(tally - static_cast<int64_t>(p.batch) * nt), 1ull);
            wave_tally(P, lsl >= 0 ? -1 : tally, lane, lds_counts);   // chunks without a slot
        } else {
            wave_tally(P, tally, lane, lds_counts);
        }
        if (PC) census_stage(P, CS, cstaged, at_census, p, lane);
        if (!active) continue;
        note_stream(c, pdraws);   // the particle's own stream ends here
        pdraws = 0;
        if (SPILL) budget--;
        if (n > 0) {
            if (n > 1) {
                if (sp + (has_top ? 1u : 0u) == P.stack_depth) {   // has_top is false unless DEEP
                    if (SPILL) {
                        spill(P, p.x, p.t, p.tb, p.batch, p.Z >> P.lcg.up, 2, n);
                    } else {
                        atomicOr(P.overflow, 1u);
                        active = false;   // the family is abandoned; the run reports an error
                        if (SL) family_ended(slot_alive, lsl);
                        continue;
                    }
                } else {
                    PulseStackEntry e;
                    e.x = p.x;
                    e.t = p.t;
                    e.key = p.Z >> P.lcg.up;
                    e.tb = p.tb;
                    e.next = 2;
                    e.n = static_cast<uint16_t>(n);
                    if (DEEP) {
                        if (has_top) stack[static_cast<uint64_t>(sp++) * sstride] = top;
                        top = e;
                        has_top = true;
                    } else {
                        stack[sp++] = e;
                    }
                }
            }
            if (SPILL && budget == 0) {
                // out of budget: the first emerging particle and the stack go to the bank
                spill(P, p.x, p.t, p.tb, p.batch, p.Z >> P.lcg.up, 1, 1);
                spill_stack(P, stack, sstride, sp, top, has_top, p.batch);
                sp = 0;
                has_top = false;
                active = false;
                continue;
            }
            p.Z = murmur_hash(1ull, p.Z >> P.lcg.up) << P.lcg.up;
            p.has_mu = false;
            continue;   // the first emerging particle starts at once
        }
        if (DEEP ? !has_top : sp == 0) {
            active = false;
            if (SL) family_ended(slot_alive, lsl);
            continue;
        }
        if (SPILL && budget == 0) {
            spill_stack(P, stack, sstride, sp, top, has_top, p.batch);
            sp = 0;
            has_top = false;
            active = false;
            continue;
        }
        PulseStackEntry& e = DEEP ? top : stack[sp - 1];
        p.x = e.x;
        p.t = e.t;
        p.tb = e.tb;
        p.has_mu = false;
        p.Z = murmur_hash(e.next, e.key) << P.lcg.up;
        if (e.next != e.n) {
            e.next++;
        } else if (!DEEP) {
            --sp;
        } else if (sp > 0) {
            // the entry's last sibling: the entry below becomes the top (its
            // load is in flight while this sibling's line runs)
            top = stack[static_cast<uint64_t>(--sp) * sstride];
        } else {
            has_top = false;
        }
    }
    if (PC && cstaged != 0) census_flush(P, CS, cstaged, lane);
    tally_lds_end<BLOCK>(P, lds_counts);
    flush_lane_counters<BLOCK>(P, c);
}

// ------------------------------------------------------------ population control

// Where arrival i of all parts, in part order, lies in P.cen.
struct CensusIndex {
    uint64_t first[kPulseCensusParts + 1];   // arrivals before part s
    __device__ __forceinline__ void load(const PulseParams& P) {   // one thread; the caller synchronises
        uint64_t n = 0;
        for (uint32_t s = 0; s < P.cen_parts; ++s) {
            first[s] = n;
            n += P.cen_count[s * kPulseCounterStride];
        }
        for (uint32_t s = P.cen_parts; s <= kPulseCensusParts; ++s) first[s] = n;
    }
    __device__ __forceinline__ const PulseCensusEntry& at(const PulseParams& P, uint64_t i) const {
        uint32_t s = 0;   // the last part with first[s] <= i among the first cen_parts
#pragma unroll
        for (uint32_t step = kPulseCensusParts / 2; step != 0; step /= 2)
            if (first[s + step] <= i) s += step;
        return P.cen[s * P.cen_cap + (i - first[s])];
    }
};

// Arrivals per batch at census P.census: a block-local histogram over the
// chunk's batches, added to P.pop once per block.
__global__ void __launch_bounds__(256) k_pulse_census_count(PulseParams P, uint64_t n) {
    __shared__ uint32_t hist[kPulsePcChunkBatches];
    __shared__ CensusIndex idx;
    if (threadIdx.x == 0) idx.load(P);
    for (uint32_t i = threadIdx.x; i < P.n_chunk_batches; i += 256) hist[i] = 0;
    __syncthreads();
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x; i < n;
         i += static_cast<uint64_t>(gridDim.x) * 256) {
        const uint32_t k = idx.at(P, i).batch - P.batch_lo;
        if (k < P.n_chunk_batches)
            atomicAdd(&hist[k], 1u);
        else
            atomicOr(P.overflow, 2u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < P.n_chunk_batches; i += 256)
        if (hist[i] != 0)
            atomicAdd(reinterpret_cast<unsigned long long*>(P.pop) +
                          (static_cast<uint64_t>(P.batch_lo + i) * P.n_census + P.census) * 2,
                      static_cast<unsigned long long>(hist[i]));
}

// Copies left by arrival a: q + [u < r/N] with u the one-off value of the
// arrival's state under the phase seed of (batch, census); the comparison
// ((S >> (m-53)) + 1) N < r 2^53 is exact in 128 bits.
__device__ __forceinline__ uint64_t split_copies(const PulseParams& P, const PulseCensusEntry& a) {
    const LcgDev& L = P.lcg;
    const uint64_t N = P.pop[(static_cast<uint64_t>(a.batch) * P.n_census + P.census) * 2];
    const uint64_t M = P.pc_target;
    const uint64_t q = M / N, r = M - q * N;
    const uint64_t phase = murmur_hash(P.census + 1ull, murmur_hash(P.first_batch + a.batch + 1ull, P.pc_seed));
    const uint64_t S = murmur_hash(a.X, phase) & L.mask;
    const uint64_t j1 = (S >> L.shift53) + 1ull;
    const uint64_t lo = j1 * N, hi = __umul64hi(j1, N);
    const uint64_t rlo = r << 53, rhi = r >> 11;
    const bool extra = hi < rhi || (hi == rhi && lo < rlo);
    return q + (extra ? 1ull : 0ull);
}

// Block exclusive scan of one value per thread (BLOCK = 256).
__device__ __forceinline__ uint64_t block_scan256(uint64_t v, uint64_t* total, uint64_t* s_wave) {
    const uint32_t lane = threadIdx.x & 63u, w = threadIdx.x >> 6;
    uint64_t incl = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const uint64_t o = __shfl_up(incl, off);
        if (lane >= static_cast<uint32_t>(off)) incl += o;
    }
    if (lane == 63) s_wave[w] = incl;
    __syncthreads();
    uint64_t before = 0, all = 0;
#pragma unroll
    for (uint32_t i = 0; i < 4; ++i) {
        if (i < w) before += s_wave[i];
        all += s_wave[i];
    }
    __syncthreads();
    *total = all;
    return before + incl - v;
}

// The copies of every arrival of census P.census.  A block takes a tile of
// 256 x 16 arrivals, counts their copies, reserves room for all of them with
// one atomic, and writes copy k of arrival X as (x, mu, hash(k, X), batch).
__global__ void __launch_bounds__(256) k_pulse_split(PulseParams P, uint64_t n) {
    constexpr uint32_t kPer = 16;
    __shared__ unsigned long long hist[kPulsePcChunkBatches];
    __shared__ uint64_t s_wave[4];
    __shared__ uint64_t s_base;
    __shared__ CensusIndex idx;
    if (threadIdx.x == 0) idx.load(P);
    for (uint32_t i = threadIdx.x; i < P.n_chunk_batches; i += 256) hist[i] = 0;
    __syncthreads();
    const uint64_t tile = 256ull * kPer;
    for (uint64_t t0 = static_cast<uint64_t>(blockIdx.x) * tile; t0 < n; t0 += static_cast<uint64_t>(gridDim.x) * tile) {
        uint64_t mine = 0;
        for (uint32_t t = 0; t < kPer; ++t) {
            const uint64_t i = t0 + t * 256ull + threadIdx.x;
            if (i < n) mine += split_copies(P, idx.at(P, i));
        }
        uint64_t total = 0;
        uint64_t o = block_scan256(mine, &total, s_wave);
        if (threadIdx.x == 0) s_base = atomicAdd(reinterpret_cast<unsigned long long*>(P.copy_count), total);
        __syncthreads();
        o += s_base;
        for (uint32_t t = 0; t < kPer; ++t) {
            const uint64_t i = t0 + t * 256ull + threadIdx.x;
            if (i >= n) continue;
            const PulseCensusEntry a = idx.at(P, i);
            const uint64_t nk = split_copies(P, a);
            for (uint64_t k = 1; k <= nk; ++k, ++o) {
                if (o < P.copy_cap) {
                    PulseCensusEntry e;
                    e.x = a.x;
                    e.mu = a.mu;
                    e.X = murmur_hash(k, a.X) << P.lcg.up;
                    e.batch = a.batch;
                    e.pad = 0;
                    P.copies_out[o] = e;
                } else {
                    atomicOr(P.overflow, 1u);
                }
            }
            const uint32_t kb = a.batch - P.batch_lo;
            if (kb < P.n_chunk_batches)
                atomicAdd(&hist[kb], static_cast<unsigned long long>(nk));
            else
                atomicOr(P.overflow, 2u);
        }
        __syncthreads();   // s_base and s_wave are reused by the next tile
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < P.n_chunk_batches; i += 256)
        if (hist[i] != 0)
            atomicAdd(reinterpret_cast<unsigned long long*>(P.pop) +
                          (static_cast<uint64_t>(P.batch_lo + i) * P.n_census + P.census) * 2 + 1,
                      hist[i]);
}

// ------------------------------------------------------------ flux

// count / (((sigma_t N_b) dx) dt); with population control the count is
// first multiplied by its epoch's weight w_e (w_0 = 1,
// w_{c+1} = (w_c N_c) / M, N_c the batch's arrivals at census c).
__global__ void __launch_bounds__(256) k_pulse_flux(PulseParams P, double* flux) {
    const uint64_t n = static_cast<uint64_t>(P.n_batches) * P.n_time_bins;
    const double dx = P.x_hi - P.x_lo;
    const double nb = static_cast<double>(P.per_batch);
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * 256 + threadIdx.x; i < n;
         i += static_cast<uint64_t>(gridDim.x) * 256) {
        const uint32_t k = static_cast<uint32_t>(i % P.n_time_bins);
        const double dt = P.t_edges[k + 1] - P.t_edges[k];
        const double den = ((P.sigma_t * nb) * dx) * dt;
        if (P.n_census == 0) {
            flux[i] = static_cast<double>(P.counts[i]) / den;
        } else {
            const uint64_t b = i / P.n_time_bins;
            double w = 1.0;
            for (uint32_t e = 0; e < P.n_census && k >= (e + 1) * P.census_every; ++e)
                w = (w * static_cast<double>(P.pop[(b * P.n_census + e) * 2])) / static_cast<double>(P.pc_target);
            flux[i] = (static_cast<double>(P.counts[i]) * w) / den;
        }
    }
}

// ------------------------------------------------------------ launchers

static int device_cus() {
    int dev = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 256;
    return cus > 0 ? cus : 256;
}

template <int BLOCK>
static const void* bank_kernel_b(int items, bool pc) {
    switch (items) {
        case PULSE_ITEMS_SOURCES:
            return pc ? reinterpret_cast<const void*>(k_pulse_bank<PULSE_ITEMS_SOURCES, true, BLOCK>)
                      : reinterpret_cast<const void*>(k_pulse_bank<PULSE_ITEMS_SOURCES, false, BLOCK>);
        case PULSE_ITEMS_COPIES:
            return pc ? reinterpret_cast<const void*>(k_pulse_bank<PULSE_ITEMS_COPIES, true, BLOCK>)
                      : reinterpret_cast<const void*>(k_pulse_bank<PULSE_ITEMS_COPIES, false, BLOCK>);
        default:
            return pc ? reinterpret_cast<const void*>(k_pulse_bank<PULSE_ITEMS_BANK, true, BLOCK>)
                      : reinterpret_cast<const void*>(k_pulse_bank<PULSE_ITEMS_BANK, false, BLOCK>);
    }
}

static const void* bank_kernel(int block, int items, bool pc) {
    switch (block) {
        case 64: return bank_kernel_b<64>(items, pc);
        case 128: return bank_kernel_b<128>(items, pc);
        case 512: return bank_kernel_b<512>(items, pc);
        case 1024: return bank_kernel_b<1024>(items, pc);
        default: return bank_kernel_b<256>(items, pc);
    }
}

static int bank_block(int block) {
    return (block == 64 || block == 128 || block == 512 || block == 1024) ? block : 256;
}

size_t pulse_tally_lds_bytes(const PulseParams& p) { return p.lds_tally ? 8ull * p.n_counters : 0; }

static uint64_t bank_items(const PulseParams& p, int items_kind) {
    return items_kind == PULSE_ITEMS_SOURCES ? p.src_end - p.src_begin : p.n_in;
}

uint32_t pulse_bank_grid(const PulseParams& p, int items_kind, bool pc, int block, uint64_t items) {
    // resident blocks only: waves keep taking chunks of items, so a launch
    // ends with one tail instead of one per wave
    block = bank_block(block);
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, bank_kernel(block, items_kind, pc), block,
                                                     pulse_tally_lds_bytes(p)) != hipSuccess ||
        per_cu < 1)
        per_cu = 1;
    const uint64_t per_block = static_cast<uint64_t>(p.chunk) * static_cast<uint64_t>(block / 64);
    uint64_t blocks = (items + per_block - 1) / per_block;   // a chunk per wave at least
    const uint64_t cap = static_cast<uint64_t>(device_cus()) * static_cast<uint64_t>(per_cu);
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return static_cast<uint32_t>(blocks);
}

hipError_t launch_pulse_bank(const PulseParams& p, int items_kind, bool pc, int block, uint32_t grid,
                             hipStream_t st) {
    if (bank_items(p, items_kind) == 0) return hipSuccess;
    block = bank_block(block);
    PulseParams arg = p;
    void* args[] = {&arg};
    return hipLaunchKernel(bank_kernel(block, items_kind, pc), dim3(grid), dim3(block), args,
                           pulse_tally_lds_bytes(p), st);
}

template <int BLOCK, bool MERGE>
static const void* pool_kernel_b(int items, bool pc) {
    switch (items) {
        case PULSE_ITEMS_SOURCES:
            return pc ? reinterpret_cast<const void*>(k_pulse_pool<PULSE_ITEMS_SOURCES, true, BLOCK, MERGE>)
                      : reinterpret_cast<const void*>(k_pulse_pool<PULSE_ITEMS_SOURCES, false, BLOCK, MERGE>);
        case PULSE_ITEMS_COPIES:
            return pc ? reinterpret_cast<const void*>(k_pulse_pool<PULSE_ITEMS_COPIES, true, BLOCK, MERGE>)
                      : reinterpret_cast<const void*>(k_pulse_pool<PULSE_ITEMS_COPIES, false, BLOCK, MERGE>);
        default:
            return pc ? reinterpret_cast<const void*>(k_pulse_pool<PULSE_ITEMS_BANK, true, BLOCK, MERGE>)
                      : reinterpret_cast<const void*>(k_pulse_pool<PULSE_ITEMS_BANK, false, BLOCK, MERGE>);
    }
}

static const void* pool_kernel(const PulseParams& p, int block, int items, bool pc) {
    auto form = [&](auto b) {
        return p.merge_far != 0 ? pool_kernel_b<b.value, true>(items, pc) : pool_kernel_b<b.value, false>(items, pc);
    };
    switch (block) {
        case 64: return form(std::integral_constant<int, 64>());
        case 128: return form(std::integral_constant<int, 128>());
        case 512: return form(std::integral_constant<int, 512>());
        case 1024: return form(std::integral_constant<int, 1024>());
        default: return form(std::integral_constant<int, 256>());
    }
}

static size_t pool_lds_bytes(const PulseParams& p, int block) {
    size_t b = p.edges_lds ? 8ull * (p.n_time_bins + 1) : 0;
    b += pulse_tally_lds_bytes(p);
    return b + static_cast<size_t>(block / 64) * p.rows * p.n_time_bins * 4u;
}

// Blocks of a pool or stride kernel that fit on one CU; above 64 KiB of dynamic
// LDS the kernel is told so first, here and before its launch.
static hipError_t tally_blocks_per_cu(const void* kern, const PulseParams& p, int block, int* per_cu) {
    const size_t lds = pool_lds_bytes(p, block);
    if (lds > 64 * 1024) {
        const hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    const hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(per_cu, kern, block, lds);
    if (e != hipSuccess) return e;
    return *per_cu < 1 ? hipErrorInvalidConfiguration : hipSuccess;
}

// At most an item per wave and the blocks that fit.  A block ends with atomics
// on the run's counters and diagnostics, about 15 ns each on one address whoever
// adds, so blocks of 64 and 128 threads are no more than six per CU (about as
// many as fit of 256) unless each lane has 8 flights: 247334 sources of 1.3 flights
// took 177 us on 6144 blocks of 64 threads, 88 on 1536 (626051 sources with more
// flights and 700 uneven bins 1061 us on all that fit, 1313 on 1536).
hipError_t pulse_pool_grid(const PulseParams& p, int items_kind, bool pc, int block, uint64_t items, double flights,
                           uint32_t* grid) {
    block = bank_block(block);
    int per_cu = 0;
    const hipError_t e = tally_blocks_per_cu(pool_kernel(p, block, items_kind, pc), p, block, &per_cu);
    if (e != hipSuccess) return e;
    const uint64_t waves = static_cast<uint64_t>(block / 64);
    uint64_t blocks = (items + waves - 1) / waves;   // an item per wave at least
    const uint64_t cus = static_cast<uint64_t>(device_cus());
    uint64_t cap = cus * static_cast<uint64_t>(per_cu);
    const double busy = static_cast<double>(items) * flights / (8.0 * block);
    if (block < 256 && busy < static_cast<double>(cap)) cap = std::min(cap, std::max(6 * cus, static_cast<uint64_t>(busy)));
    if (blocks > cap) blocks = cap;
    *grid = static_cast<uint32_t>(blocks < 1 ? 1 : blocks);
    return hipSuccess;
}

// A wave that last saw at most out_budget entries appends at most one spill more
// (half a pool) before it sees the budget passed, then one iteration's siblings
// (64 (n_max - 1)) and what it holds: its lanes, pool and private stack.  (A
// bank's items that it has taken but not started have room of their own.)
uint64_t pulse_pool_slack(const PulseParams& p, uint32_t n_max) {
    return kPoolEntries / 2 + 64ull * std::max(n_max, 1u) + kPoolEntries + p.priv_cap;
}

hipError_t launch_pulse_pool(const PulseParams& p, int items_kind, bool pc, int block, uint32_t grid, hipStream_t st) {
    if (p.item_end == p.item_begin) return hipSuccess;
    block = bank_block(block);
    PulseParams arg = p;
    void* args[] = {&arg};
    return hipLaunchKernel(pool_kernel(p, block, items_kind, pc), dim3(grid), dim3(block), args,
                           pool_lds_bytes(p, block), st);
}

static uint32_t stream_grid(uint64_t work, uint64_t per_block) {
    uint64_t blocks = (work + per_block - 1) / per_block;
    const uint64_t cap = static_cast<uint64_t>(device_cus()) * 8;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return static_cast<uint32_t>(blocks);
}

hipError_t launch_pulse_census_count(const PulseParams& p, uint64_t n_arrivals, hipStream_t st) {
    if (n_arrivals == 0) return hipSuccess;
    hipLaunchKernelGGL(k_pulse_census_count, dim3(stream_grid(n_arrivals, 256ull * 16)), dim3(256), 0, st, p,
                       n_arrivals);
    return hipGetLastError();
}

hipError_t launch_pulse_split(const PulseParams& p, uint64_t n_arrivals, hipStream_t st) {
    if (n_arrivals == 0) return hipSuccess;
    hipLaunchKernelGGL(k_pulse_split, dim3(stream_grid(n_arrivals, 256ull * 16)), dim3(256), 0, st, p, n_arrivals);
    return hipGetLastError();
}

// Tally slots per wave of the family kernel over sources: when the counters
// do not fit one LDS copy per block, a chunk of 64 sources spans at most two
// batches (at least 64 sources per batch) and the slots of a block fit in
// 32 KiB.  MCRNG_PULSE_SLOTS sets the number (0: per-wave HBM atomics).
template <int BLOCK>
static uint32_t family_tally_slots(const PulseParams& p) {
    if (p.lds_tally || p.per_batch < kFamilyChunk || p.n_time_bins > 64) return 0;
    uint32_t k = kPulseTallySlots;
    if (const char* env = getenv("MCRNG_PULSE_SLOTS")) k = static_cast<uint32_t>(atoi(env));
    if (k > kPulseTallySlots) k = kPulseTallySlots;
    while (k > 0 && static_cast<size_t>(BLOCK / 64) * k * 2u * p.n_time_bins * 8u > 32768u) k /= 2;
    return k;
}

template <int BLOCK>
static hipError_t launch_family_b(const PulseParams& p_in, uint32_t grid, hipStream_t st) {
    PulseParams p = p_in;
    p.tally_slots = family_tally_slots<BLOCK>(p);
    const size_t lds = static_cast<size_t>(BLOCK / 64) * p.tally_slots * 2u * p.n_time_bins * 8u;
    // the register-top stack once every lane has many families to run
    // (MCRNG_PULSE_DEEP = 0 or 1 forces one form: both give the same counts)
    bool deep = p.src_end - p.src_begin >= 16ull * grid * BLOCK;
    if (const char* env = getenv("MCRNG_PULSE_DEEP")) deep = atoi(env) != 0;
    // the slot form only for the default block (other blocks count into HBM)
    constexpr bool kSlots = BLOCK == 256;
    if (!kSlots) p.tally_slots = 0;
    if (p.tally_slots != 0) {
        if (deep)
            hipLaunchKernelGGL((k_pulse_family<PULSE_ITEMS_SOURCES, false, BLOCK, true, kSlots>), dim3(grid),
                               dim3(BLOCK), lds, st, p);
        else
            hipLaunchKernelGGL((k_pulse_family<PULSE_ITEMS_SOURCES, false, BLOCK, false, kSlots>), dim3(grid),
                               dim3(BLOCK), lds, st, p);
    } else {
        if (deep)
            hipLaunchKernelGGL((k_pulse_family<PULSE_ITEMS_SOURCES, false, BLOCK, true, false>), dim3(grid),
                               dim3(BLOCK), pulse_tally_lds_bytes(p), st, p);
        else
            hipLaunchKernelGGL((k_pulse_family<PULSE_ITEMS_SOURCES, false, BLOCK, false, false>), dim3(grid),
                               dim3(BLOCK), pulse_tally_lds_bytes(p), st, p);
    }
    return hipGetLastError();
}

uint32_t pulse_finish_grid(uint64_t items) {
    uint64_t blocks = (items + 255) / 256;
    const uint64_t cap = static_cast<uint64_t>(device_cus()) * 8;
    if (blocks > cap) blocks = cap;
    if (blocks < 1) blocks = 1;
    return static_cast<uint32_t>(blocks);
}

hipError_t launch_pulse_finish(const PulseParams& p, bool pc, uint32_t grid, hipStream_t st) {
    if (p.n_in == 0) return hipSuccess;
    if (pc)
        hipLaunchKernelGGL((k_pulse_family<PULSE_ITEMS_BANK, true, 256, false, false>), dim3(grid), dim3(256),
                           pulse_tally_lds_bytes(p), st, p);
    else
        hipLaunchKernelGGL((k_pulse_family<PULSE_ITEMS_BANK, false, 256, false, false>), dim3(grid), dim3(256),
                           pulse_tally_lds_bytes(p), st, p);
    return hipGetLastError();
}

static const void* stride_kernel(const PulseParams& p, int block) {
    auto form = [&](auto b) {
        return p.merge_far != 0 ? reinterpret_cast<const void*>(k_pulse_stride<b.value, true>)
                                : reinterpret_cast<const void*>(k_pulse_stride<b.value, false>);
    };
    switch (block) {
        case 64: return form(std::integral_constant<int, 64>());
        case 128: return form(std::integral_constant<int, 128>());
        case 512: return form(std::integral_constant<int, 512>());
        case 1024: return form(std::integral_constant<int, 1024>());
        default: return form(std::integral_constant<int, 256>());
    }
}

hipError_t pulse_stride_grid(const PulseParams& p, int block, uint64_t sources, uint32_t* grid) {
    block = bank_block(block);
    int per_cu = 0;
    const hipError_t e = tally_blocks_per_cu(stride_kernel(p, block), p, block, &per_cu);
    if (e != hipSuccess) return e;
    // a family per wave at least: few families spread over the whole chip
    uint64_t blocks = (sources + block / 64 - 1) / (block / 64);
    const uint64_t cap = static_cast<uint64_t>(device_cus()) * static_cast<uint64_t>(per_cu);
    if (blocks > cap) blocks = cap;
    *grid = static_cast<uint32_t>(blocks < 1 ? 1 : blocks);
    return hipSuccess;
}

// Tally rows per wave of the run's pool or stride launches when the counters
// are not in LDS: 2 to 8 within 1 KiB, two up to 512 bins (4 KiB); fewer where
// the block's rows would not fit beside the kernel's static LDS.  (1024 threads
// with 512 bins: 64 KiB of rows beside 97 KiB in the stride kernel and 109 KiB
// in the pool kernel with population control, of 160 KiB.)  The pool kernel
// over sources has the most static LDS of those of a run.
hipError_t pulse_fit_rows(PulseParams* p, bool pc, int block) {
    p->rows = p->merge_far = 0;
    if (p->lds_tally) return hipSuccess;
    // Merging pays where few batches' counters may be hit by all waves, and
    // costs up to 18% where the lanes' counters differ (20 batches of 600 bins: 433
    // against 370 us spread, 4.5 against 9.4 ms in one bin; 128 batches: 1045
    // against 970 us, 14.7 against 18.6 ms).  Without
    // rows every lane's count comes here: more tries.
    const uint32_t merge = p->n_batches <= kPulseMergeBatches ? 1u : 0u;
    p->merge_far = 3u * merge;
    if (p->n_time_bins > kPulseEdgeBins) return hipSuccess;
    block = bank_block(block);
    int dev = 0, lds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return e;
    hipFuncAttributes a;
    e = hipFuncGetAttributes(&a, p->hash ? pool_kernel(*p, block, PULSE_ITEMS_SOURCES, pc) : stride_kernel(*p, block));
    if (e != hipSuccess) return e;
    p->rows = 8;
    while (p->rows > 2 && p->rows * p->n_time_bins > 256) p->rows /= 2;
    while (p->rows > 0 && a.sharedSizeBytes + pool_lds_bytes(*p, block) > static_cast<size_t>(lds)) p->rows /= 2;
    if (p->rows != 0) p->merge_far = merge;
    return hipSuccess;
}

hipError_t launch_pulse_stride(const PulseParams& p, int block, uint32_t grid, hipStream_t st) {
    if (p.item_end == p.item_begin) return hipSuccess;
    block = bank_block(block);
    PulseParams arg = p;
    void* args[] = {&arg};
    return hipLaunchKernel(stride_kernel(p, block), dim3(grid), dim3(block), args, pool_lds_bytes(p, block), st);
}

uint32_t pulse_family_grid(int block) {
    // persistent lanes: 2048 per CU (the stack buffer is sized from this);
    // a run of few sources has its waves spread over the whole chip
    return static_cast<uint32_t>(device_cus()) * static_cast<uint32_t>(2048 / block);
}

hipError_t launch_pulse_family(const PulseParams& p, int block, uint32_t grid, hipStream_t st) {
    if (p.src_end == p.src_begin) return hipSuccess;
    switch (block) {
        case 64: return launch_family_b<64>(p, grid, st);
        case 128: return launch_family_b<128>(p, grid, st);
        case 512: return launch_family_b<512>(p, grid, st);
        case 1024: return launch_family_b<1024>(p, grid, st);
        default: return launch_family_b<256>(p, grid, st);
    }
}

hipError_t launch_pulse_flux(const PulseParams& p, double* flux, hipStream_t st) {
    const uint64_t n = static_cast<uint64_t>(p.n_batches) * p.n_time_bins;
    if (n == 0) return hipSuccess;
    uint64_t blocks = (n + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(k_pulse_flux, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, st, p, flux);
    return hipGetLastError();
}

}  // namespace mcrng
