// Internal types of the pulse-problem kernels (pulse.hip) shared with the
// host-side API.  Not part of the public C ABI (include/mcrng.h).
#pragma once

#include "internal.hpp"

namespace mcrng {

// Diagnostics of the pulse problem, same order as the MCRNG_PD_* words.
enum PulseDiagWord {
    PD_SOURCES = 0, PD_COLLISIONS, PD_TALLIED, PD_SCATTERS, PD_ABSORBED, PD_CENSUS,
    PD_SECONDARIES, PD_DRAWS, PD_MAX_DRAWS, PD_OVER_STRIDE
};

// Particle bank (structure of arrays): particles waiting to start.
struct PulseBankView {
    double* x;
    double* t;
    uint64_t* X;         // start state of the particle's stream, top-aligned (X << (64 - m))
    uint32_t* batch;
    int32_t* tb;
};

// Per-lane stack entry of the family schedule: the siblings of one
// scattering that have not started yet (keys next .. n).
struct PulseStackEntry {
    double x, t;
    uint64_t key;        // hash seeding: the parent's state X_p; stride: siblings left << 16 | time bin + 1
    int32_t tb;          // (hash seeding)
    uint16_t next, n;
};

// A census arrival, or a census copy, of a population-controlled run (32 B).
struct PulseCensusEntry {
    double x, mu;        // census point and direction
    uint64_t X;          // arrival: stream state after its draws; copy: its start state, top-aligned
    uint32_t batch;      // batch of the run (0-based)
    uint32_t pad;
};

// A particle waiting in a wave's pool (k_pulse_pool): child k of a scattering
// at (x, t) whose parent ended in state key.
struct __align__(16) PulsePoolEntry {
    double x, t;
    uint64_t key;        // X_p, the parent's state
    uint32_t batch;
    uint32_t meta;       // k << 16 | time bin + 1
};

// One counter takes about 15 ns per atomic, whoever adds (26000 appends of 64
// census arrivals made a 0.3 ms epoch of the paper's problem 0.68 ms, 20000
// takes of items 0.36): a pool launch's census arrivals and the items its
// waves take dynamically go by 16 counters each, 128 bytes apart.
constexpr uint32_t kPulseCensusParts = 16, kPulseItemParts = 16, kPulseCounterStride = 16;

struct PulseParams {
    LcgDev lcg;
    SeedDev seed;            // hash: base = the global seed s; stride: skip table etc.
    uint64_t first_batch;
    uint64_t per_batch;
    uint32_t n_batches;
    uint32_t n_time_bins;
    uint32_t hash;           // 1: hash seeding (secondaries seeded by eq. 5)
    uint32_t n_floor;        // floor(nu)
    uint64_t frac_below;     // uniform_below(nu - floor(nu)): one more particle below it
    uint64_t scatter_below;  // uniform_below(scatter)
    double sigma_t, x_lo, x_hi, t_end;
    int32_t tb0;             // time bin of t = 0
    uint32_t stack_depth;    // family schedule: entries per lane
    const double* t_edges;   // device, n_time_bins + 1
    uint64_t* counts;        // n_batches x n_time_bins
    uint32_t n_counters;     // n_batches x n_time_bins
    uint32_t lds_tally;      // 1: each block counts into an LDS copy of all counters
    uint32_t tally_slots;    // family schedule over sources, counters not in LDS: per-wave LDS
                             // slots, one per chunk of sources in flight (0: HBM atomics)
    uint64_t* diag;          // kNDiag words (PD_*)
    uint64_t stride_q;       // stride: Q (over-stride count)
    uint64_t src_begin, src_end;   // sources of this launch (0-based over the run)
    PulseBankView in, out;   // bank schedule
    uint64_t n_in;
    uint64_t* out_count;
    uint64_t out_cap;
    uint64_t* item_counter;  // bank schedule: next input particle (taken `chunk` per wave)
    uint32_t chunk;          // bank schedule: input particles a wave takes per atomic
    uint64_t out_budget;     // pool: a wave that sees more entries in the output bank hands over its particles
    uint64_t cen_budget;     // pool: the same for census arrivals
    uint64_t item_begin, item_end;   // pool: the launch's items (sources of the run, copies or bank entries):
    uint32_t first_chunk;            // wave w starts with [item_begin + w first_chunk, ...) up to item_part[0];
    uint64_t item_part[kPulseItemParts + 1];        // part s of the rest, [item_part[s], item_part[s + 1]), is taken `chunk` at a time
    uint32_t item_parts;             // by the blocks b with b mod item_parts = s (a power of two)
    uint64_t* left;          // pool: ranges of taken but unused items (pairs), n_left of them
    uint64_t* n_left;
    const uint64_t* ranges;  // pool: the items are ranges of sources or copies (pairs, none empty), taken one at a time (null: no)
    PulsePoolEntry* priv;    // pool: priv_cap entries per wave behind the LDS pool
    uint32_t priv_cap;
    uint32_t tail_iters;     // pool: iterations of a wave after the launch's items are taken
    uint32_t rows;           // pool: LDS tally rows per wave (a power of two; 0: HBM atomics)
    uint32_t merge_far;      // pool: counts in HBM: counters with few lanes of a wave before the rest go one by one
                             // (0: all one by one)
    uint32_t edges_lds;      // pool: time edges staged in LDS
    uint32_t grid_uniform;   // pool: time edge i is within a quarter of a bin of t0 + i / inv_dt
    double t0, inv_dt;
    uint32_t* overflow;      // set if an append or a stack push found no room
    uint64_t* family_counter;
    PulseStackEntry* stack;  // families: stack_depth entries per lane of the launch.  Stride kernel and
                             // the register-top form of the hash kernel: depth-major (entry d of lane l
                             // at d * lanes + l); the other hash form: a lane's entries together
    // population control (t_end is then the census time of the epoch)
    PulseCensusEntry* cen;   // census arrivals of the epoch
    uint64_t* cen_count;     // arrivals of part s at cen_count[s kPulseCounterStride]
    uint64_t cen_cap;        // capacity of a part: part s starts at cen[s cen_cap]
    uint32_t cen_parts;      // 1, or kPulseCensusParts (block b appends to part b mod cen_parts)
    const PulseCensusEntry* copies;   // copies starting the epoch (taken as items)
    double t_start;          // the census time the copies start at
    int32_t tb_start;        // its time bin
    uint32_t census;         // split: census index c
    uint32_t n_census;       // census points of the run
    uint32_t census_every;   // time bins per epoch (census c at edge (c+1) census_every)
    uint32_t batch_lo;       // split / count: first batch of the chunk (LDS histogram base)
    uint32_t n_chunk_batches;
    uint64_t pc_target, pc_seed;
    uint64_t* pop;           // n_batches x n_census x 2: arrivals, copies
    uint64_t* copy_count;
    uint64_t copy_cap;
    PulseCensusEntry* copies_out;
    uint32_t lane_budget;    // finish launches: particles per input particle before the rest is banked
};

enum PulseItems : int { PULSE_ITEMS_SOURCES = 0, PULSE_ITEMS_BANK = 1, PULSE_ITEMS_COPIES = 2 };
constexpr uint32_t kPulsePcChunkBatches = 4096;   // batches per chunk of a population-controlled run

// Event launches: the grid (resident blocks, at most one chunk of items per
// wave) is chosen first, so that the caller can size the output for it.
// `items` is a PulseItems value; `pc`: the launch's census is a census of
// population control (arrivals are banked in p.cen).
uint32_t pulse_bank_grid(const PulseParams& p, int items_kind, bool pc, int block, uint64_t items);
// Block-local tally copies up to this many counters (16 KiB).  In the pool and
// stride kernels they leave four 256-thread blocks per CU, where tally rows
// leave six, but no row changes hands and no count goes to HBM: 513 to 2048
// counters are up to 3.4 times faster so (3 x 100000 sources in 200 bins 428
// against 1440 us; 60 x 1000 in 20 bins 245 against 255; 100 x 300000 in 20
// bins 15.2 against 14.9 ms).
constexpr uint32_t kPulseLdsCounters = 2048;
constexpr uint32_t kPulseTallySlots = 16;      // most tally slots per wave of the family kernel
// Entries of a wave's LDS stage of appends in k_pulse_bank (output slack).
uint32_t pulse_bank_stage(int block);
hipError_t launch_pulse_bank(const PulseParams& p, int items_kind, bool pc, int block, uint32_t grid,
                             hipStream_t st);
constexpr uint32_t kPulseMergeBatches = 128;   // most batches whose HBM counts are merged (WaveTally)
constexpr uint32_t kPulseEdgeBins = 512;   // most time bins with edges (and tally rows) in LDS
// Sets p->rows (hash: of the pool kernels, else of the stride kernel) for the
// block size; p->edges_lds and p->lds_tally are set before.
hipError_t pulse_fit_rows(PulseParams* p, bool pc, int block);
// Pool launches (bank schedule).  The grid is chosen first (buffers are sized
// for its waves); pulse_pool_slack: entries a wave may append to the output
// bank after it has seen out_budget passed, and census arrivals likewise.
// `flights`: expected flights of an item and all it gives rise to.
hipError_t pulse_pool_grid(const PulseParams& p, int items_kind, bool pc, int block, uint64_t items, double flights,
                           uint32_t* grid);
uint64_t pulse_pool_slack(const PulseParams& p, uint32_t n_max);
constexpr uint64_t kPulsePoolCensusSlack = 256;
hipError_t launch_pulse_pool(const PulseParams& p, int items_kind, bool pc, int block, uint32_t grid, hipStream_t st);
// Population control at census p.census: arrival counts per batch into
// p.pop, then the copies of every arrival into p.copies_out.
hipError_t launch_pulse_census_count(const PulseParams& p, uint64_t n_arrivals, hipStream_t st);
hipError_t launch_pulse_split(const PulseParams& p, uint64_t n_arrivals, hipStream_t st);
uint32_t pulse_family_grid(int block);
// Families of stride seeding: the grid (p.stack holds stack_depth entries per
// lane of it), then the launch over items [item_begin, item_end) taken as by
// the pool.
hipError_t pulse_stride_grid(const PulseParams& p, int block, uint64_t sources, uint32_t* grid);
hipError_t launch_pulse_stride(const PulseParams& p, int block, uint32_t grid, hipStream_t st);
// Finish launch (hash seeding): the generation bank p.in (p.n_in particles)
// run depth first per lane with p.stack (p.stack_depth entries per lane),
// at most p.lane_budget particles per input particle, the rest banked in
// p.out (p.out_count); one 256-thread block per 256 inputs, at most 8 per CU.
uint32_t pulse_finish_grid(uint64_t items);
hipError_t launch_pulse_finish(const PulseParams& p, bool pc, uint32_t grid, hipStream_t st);
hipError_t launch_pulse_family(const PulseParams& p, int block, uint32_t grid, hipStream_t st);
hipError_t launch_pulse_flux(const PulseParams& p, double* flux, hipStream_t st);

}  // namespace mcrng
