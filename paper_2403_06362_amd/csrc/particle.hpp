// One particle event: the per-history arithmetic shared by the history-based
// and the event-sorted schedules, so that both run the identical operation
// sequence for every particle.
//
// An event is split in three parts that a schedule may run at different
// times for one particle (never reordered, never skipped):
//   sample_tau    X = lcg(X); tau = -ln(uniform(X))                 (the flight)
//   geom_pass     distances to collision / edge / time, choice, score, move
//   collide_pass  X = lcg(X), absorbed unless uniform < c; X = lcg(X),
//                 mu = R(2 u - 1); the next part is sample_tau
// The passes work on a whole wave: the lanes to advance come as a wave mask in
// scalar registers and the outcomes go out as wave masks, so that a lane's
// phase costs no vector instruction and both halves of a choice are
// straight-line selects.  (The slab kernels are bound by vector issue: with
// the phases in vector registers and a branch per outcome the long-chain slab
// took 173 vector instructions per event.)
// Every floating-point result is the IEEE operation's, rounded to nearest,
// with no fused multiply-add where the operation is a separate multiply and
// add (the library is built with -ffp-contract=off).  Divisions by a
// cell's sigma_t and by the flight's mu go through the divisor's refined
// reciprocal (quot, device_rng.hpp), which gives the correctly rounded
// quotient; minima and maxima are the compare-and-replace clamps of the
// operation sequence (their operands are never NaN, and a zero's sign never
// reaches a tally, a decision or a stored state).
#pragma once

#include <type_traits>

#include "internal.hpp"

namespace mcrng {

template <bool F32>
struct Particle {
    using R = typename std::conditional<F32, float, double>::type;
    R x, mu, t;         // FP64: global x, t; FP32: x from the cell's left edge, t from the time bin start
    double tau;         // remaining optical depth of the flight (double in both modes)
    R rmu;              // refined reciprocal of mu; NaN when mu == 0 (no edge distance compares below a flight's)
    uint64_t Z;         // top-aligned LCG state
    uint32_t off;       // cell index times sizeof(R)
    int32_t step;       // sizeof(R) with the sign of mu
    int32_t tb;
};

// A cell offset as a signed distance.  A lane that left through the left face
// keeps the offset of the cell before the first, 0 - sizeof(R) in 32 bits, and
// geom_pass forms addresses from it (the arrays have neighbours there): as an
// unsigned distance that address is right only where the compiler has proved
// the pointer to be one into LDS, 32 bits wide, and else 4 GiB off.
constexpr __host__ __device__ int32_t cell_distance(uint32_t off) { return static_cast<int32_t>(off); }
static_assert(cell_distance(0u - 8u) == -8 && cell_distance(2u * (0u - 4u)) == -8 && (cell_distance(0u - 8u) >> 1) == -4,
              "the offset before the first cell is a distance of one cell");

// Cell data of the current problem.  FP64: edge c is the position of edge c
// (n_cells + 1), tedge[t] the time edges.  FP32: entry c + 1 of the edge
// array is the width of cell c (entry 0 is unused), tedge[t] the duration of
// time bin t.  Offsets are cell indices times sizeof(R).
// ONE: one region, so cells are the space bins and sigma_t and c are the
// same in all of them (kept in registers).
template <bool F32, bool ONE>
struct LdsCells {
    using R = typename std::conditional<F32, float, double>::type;
    const char* edge_base;
    const char* sig_base;
    const char* rsig_base;
    const char* below_base;
    const char* bin_base;
    const R* tedge;
    R sig1, rsig1;
    uint64_t below1;
    uint32_t n_off;        // n_cells * sizeof(R)
    int32_t n_time_bins;
    int32_t n_space_bins;
    __device__ __forceinline__ const R* edge(uint32_t off) const { return reinterpret_cast<const R*>(edge_base + cell_distance(off)); }
    __device__ __forceinline__ R sig(uint32_t off) const {
        if constexpr (ONE) return sig1;
        return *reinterpret_cast<const R*>(sig_base + cell_distance(off));
    }
    __device__ __forceinline__ R rsig(uint32_t off, R) const {
        if constexpr (ONE) return rsig1;
        return *reinterpret_cast<const R*>(rsig_base + cell_distance(off));
    }
    // the state bound of the absorption test (uniform_below of the cell's c)
    __device__ __forceinline__ uint64_t below(uint32_t off) const {
        if constexpr (ONE) return below1;
        return *reinterpret_cast<const uint64_t*>(below_base + cell_distance(F32 ? 2u * off : off));
    }
    // 8 x the cell's space bin
    __device__ __forceinline__ uint32_t bin8(uint32_t off) const {
        if constexpr (ONE) return F32 ? 2u * off : off;
        return *reinterpret_cast<const uint32_t*>(bin_base + (F32 ? cell_distance(off) : cell_distance(off) >> 1));
    }
};

// The same from the problem's tables in HBM (edges as LdsCells; FP32 widths
// start at entry 0, so the entry before cell 0's must not be read).
template <bool F32>
struct GlobalCells {
    using R = typename std::conditional<F32, float, double>::type;
    const R* edges;
    const R* sigs;
    const double* scat;
    const int32_t* bins;
    const R* tedge;
    uint32_t n_off;
    int32_t n_time_bins;
    int32_t n_space_bins;
    __device__ __forceinline__ const R* edge(uint32_t off) const { return edges + off / sizeof(R) - (F32 ? 1 : 0); }
    __device__ __forceinline__ R sig(uint32_t off) const { return sigs[off / sizeof(R)]; }
    __device__ __forceinline__ R rsig(uint32_t, R sig) const { return recip_refined(sig); }
    __device__ __forceinline__ uint64_t below(uint32_t off) const { return uniform_below(scat[off / sizeof(R)]); }
    __device__ __forceinline__ uint32_t bin8(uint32_t off) const { return 8u * static_cast<uint32_t>(bins[off / sizeof(R)]); }
};

enum : int { END_NONE = 0, END_LEAK_LEFT, END_LEAK_RIGHT, END_ABSORBED, END_CENSUS };

// Adds q to a tally word pair: the low and the high 32-bit halves of q are
// summed into separate 64-bit words (LDS or global memory); the pair holds
// low + 2^32 high.
__device__ __forceinline__ void pair_score(uint64_t* slot, uint64_t q) {
    atomicAdd(reinterpret_cast<unsigned long long*>(slot), static_cast<unsigned long long>(q & 0xffffffffull));
    atomicAdd(reinterpret_cast<unsigned long long*>(slot + 1), static_cast<unsigned long long>(q >> 32));
}

// Adds lo + 2^32 hi to a global word pair that may collect more than 2^32
// additions: when the low word wraps (it lost 2^64 = 2^32 x 2^32), 2^32 more
// goes to the high word, so the pair's value stays exact below 2^96.
__device__ __forceinline__ void carry_add(uint64_t* slot, uint64_t lo, uint64_t hi) {
    const unsigned long long old = atomicAdd(reinterpret_cast<unsigned long long*>(slot), static_cast<unsigned long long>(lo));
    if (old + lo < old) hi += 1ull << 32;
    if (hi != 0) atomicAdd(reinterpret_cast<unsigned long long*>(slot + 1), static_cast<unsigned long long>(hi));
}

// Tally of an event schedule's particle: word pairs, added plainly or (CARRY)
// with carry_add.
template <bool CARRY>
struct PairTally {
    uint64_t* tally;
    __device__ __forceinline__ void add(uint32_t bin8, double s) const {
        const uint64_t q = quantise(s);
        if constexpr (CARRY)
            carry_add(tally + bin8 / 4, q & 0xffffffffull, q >> 32);
        else
            pair_score(tally + bin8 / 4, q);
    }
};

// A unit's tally slice in LDS: the low limbs of all bins, then (hi_off bytes
// on) the high limbs.  Words of one limb lie next to each other, so lanes in
// neighbouring bins use all banks (as pairs, half of them per add).
struct LimbTally {
    char* lo;
    uint32_t hi_off;
    __device__ __forceinline__ void add(uint32_t bin8, double s) const {
        const Limbs q = quantise_limbs(s);
        char* const w = lo + bin8;
        atomicAdd(reinterpret_cast<unsigned long long*>(w), static_cast<unsigned long long>(q.lo));
        atomicAdd(reinterpret_cast<unsigned long long*>(w + hi_off), static_cast<unsigned long long>(q.hi));
    }
};

template <bool F32>
__device__ __forceinline__ void sample_tau(Particle<F32>& p, const LcgDev& L) {
    p.Z = lcg_next_z(L, p.Z);
    p.tau = fixed_neg_log(uniform_z(p.Z));
}

// Outcomes of a geometry pass, subsets of the lanes it advanced: at a
// collision site; out of the slab (through the face they were heading for);
// past the last time edge.  The others go on with their flight.
struct GeomOut {
    uint64_t coll, leak, census;
};

// One geometry step of the lanes in G; up: the lanes with mu > 0 (kept from
// the collision that drew mu).  FP64, global coordinates:
//   s = tau / sig[c]                                          -> collision
//   se = (E[c+1] - x) / mu if mu > 0, (E[c] - x) / mu if mu < 0, +inf if
//   mu == 0;  if se < s: s = se                               -> edge
//   timed: st = T[tb+1] - t;  if st < s: s = st               -> time
//   score q(s) into (tb, bin[c]);  timed: t = t + s, clamped to T[tb+1]
//   tau = tau - sig * s, clamped at 0
//   edge:  mu > 0: c + 1 (leak right past the last), x = E[c+1]
//          mu < 0: x = E[c], c - 1 (leak left past the first)
//   other: x = x + mu * s, clamped to [E[c], E[c+1]]
//   time:  tb + 1, t = T[tb+1]; census past the last time edge
// FP32, position measured from the cell's left edge and time from the time
// bin's start (W = cell width, DT = bin duration); the remaining optical
// depth tau stays double (a float tau would lose absolute precision over a
// flight's many subtractions, and the flight's last segment, their small
// remainder, would carry it):
//   s = R(tau) / sig[c];  se = (W[c] - x)/mu (mu > 0), (0 - x)/mu (mu < 0),
//   +inf (mu == 0);  timed: st = DT[tb] - t;  strict-less order as in FP64
//   score q(double(s));  timed: t = t + s, clamped to DT[tb]
//   tau = tau - double(sig) double(s) (exact product), clamped at 0
//   edge: mu > 0: c + 1, x = 0;  mu < 0: c - 1, x = W[c - 1]
//   other: x = x + mu s clamped to [0, W[c]];  time: tb + 1, t = 0
// Every lane computes, lanes outside G on whatever their registers hold (an
// ended history's offset may be one cell outside the problem, where the LDS
// arrays have neighbours; with cells in HBM the caller sets it back); only the
// lanes in G score and change state.
template <bool F32, bool TIMED, class Cells, class Tally>
__device__ __forceinline__ GeomOut geom_pass(Particle<F32>& p, const Cells& C, uint64_t G, uint64_t up,
                                             const Tally& tally) {
    using R = typename Particle<F32>::R;
    const uint32_t off = p.off;
    const R* const ed = C.edge(off);
    // FP64: the cell's edges; FP32: the widths of the cell before and of the cell
    R e0, e1 = ed[1];
    if constexpr (std::is_same<Cells, GlobalCells<true>>::value)
        e0 = off != 0 ? ed[0] : R(0);
    else
        e0 = ed[0];
    const R e_lo = F32 ? R(0) : e0, e_hi = e1;
    const R sig = C.sig(off);
    const R depth = static_cast<R>(p.tau);
    const R e_to = in_mask(up) ? e_hi : e_lo;
    const R num = e_to - p.x;
    const R sc = quot(depth, sig, C.rsig(off, sig));
    const R se = quot(num, p.mu, p.rmu);
    uint64_t edge = wave_mask(se < sc);
    R s = min_num(se, sc);   // sc when se is NaN
    if ((wave_mask(below_quot_min(s)) & G) != 0) {
        // a distance below the refined quotients' range: plain divisions
        const R pc = depth / sig;
        const R pe = p.mu == R(0) ? static_cast<R>(__builtin_huge_val()) : num / p.mu;
        edge = wave_mask(pe < pc);
        s = min_num(pe, pc);
    }
    // a set may mix steady and timed problems, an event schedule's wave too
    const uint64_t timed = TIMED ? wave_mask(C.n_time_bins > 0) : 0ull;
    uint64_t time = 0;
    R tnext = R(0);
    if (timed != 0) {
        if (C.n_time_bins > 0) tnext = F32 ? C.tedge[p.tb] : C.tedge[p.tb + 1];
        const R st = tnext - p.t;
        time = timed & wave_mask(st < s);
        s = sel(time, st, s);   // (steady lanes of a mixed wave keep theirs)
        edge &= ~time;
    }
    edge &= G;
    const uint32_t noff = off + sel_or_zero(edge, static_cast<uint32_t>(p.step));
    GeomOut o;
    o.leak = G & wave_mask(noff >= C.n_off);   // -1 wraps past n_off
    o.census = 0;
    uint64_t last = 0;
    if (timed != 0) {
        last = wave_mask(p.tb + 1 == C.n_time_bins);
        o.census = G & time & last;
    }
    o.coll = G & ~(edge | time);
    if (in_mask(G)) {
        tally.add((TIMED ? __umul24(static_cast<uint32_t>(p.tb), 8u * static_cast<uint32_t>(C.n_space_bins)) : 0u) +
                      C.bin8(off),
                  static_cast<double>(s));
        p.tau = __builtin_fmax(p.tau - static_cast<double>(sig) * static_cast<double>(s), 0.0);
        const R moved = min_num(max_num(p.x + p.mu * s, e_lo), e_hi);
        const R entry = F32 ? (in_mask(up) ? R(0) : e0) : e_to;
        p.x = sel(edge, entry, moved);
        p.off = noff;
        if (timed != 0) {
            p.t = sel(time, F32 ? R(0) : tnext, min_num(p.t + s, tnext));
            p.tb += static_cast<int32_t>(sel_const<1, 0>(time & ~last));
        }
    }
    return o;
}

// The cell step of the direction: sizeof(R) with the sign bit of mu (of no
// meaning when mu == 0, which meets no edge).
template <bool F32>
__device__ __forceinline__ void set_step(Particle<F32>& p) {
    int32_t top;
    if constexpr (F32)
        top = static_cast<int32_t>(__float_as_uint(p.mu));
    else
        top = static_cast<int32_t>(static_cast<uint64_t>(__double_as_longlong(p.mu)) >> 32);
    p.step = static_cast<int32_t>(sizeof(typename Particle<F32>::R)) ^ (top >> 31);
    p.step -= top >> 31;
}

// Collision of the lanes in W at their sites: u1 decides absorption (the
// state against the cell's bound), u2 the new direction mu = R(2 u2 - 1)
// (computed in double, exact, then rounded once).  Returns the scattered
// lanes, which sample their next flight with sample_tau (the others of W are
// absorbed), and updates the lanes with mu > 0.
template <bool F32, class Cells>
__device__ __forceinline__ uint64_t collide_pass(Particle<F32>& p, const Cells& C, const LcgDev& L, uint64_t W,
                                                 uint64_t& up) {
    using R = typename Particle<F32>::R;
    const uint64_t z1 = lcg_next_z(L, p.Z);
    const uint64_t go = wave_mask(z1 < C.below(p.off)) & W;
    const uint64_t z2 = lcg_next_z(L, z1);
    const R mu = static_cast<R>(__builtin_fma(uniform_z(z2), 2.0, -1.0));
    up = (up & ~go) | (go & wave_mask(mu > R(0)));
    if (in_mask(go)) {
        p.Z = z2;
        p.mu = mu;
        p.rmu = recip_refined(mu);
        set_step<F32>(p);
    }
    return go;
}

// A new history whose stream starts at state Z: source at the left face
// moving right, at the first time edge; its first flight is sampled before
// its first geometry step.
template <bool F32, bool TIMED, class Cells>
__device__ __forceinline__ void init_particle_at(Particle<F32>& p, const Cells& C, uint64_t Z) {
    using R = typename Particle<F32>::R;
    p.Z = Z;
    if constexpr (F32) {
        p.x = 0.0f;
        p.t = 0.0f;
    } else {
        p.x = *C.edge(0);
        p.t = (TIMED && C.n_time_bins > 0) ? C.tedge[0] : 0.0;
    }
    p.mu = R(1);
    p.rmu = R(1);   // recip_refined(1) is exactly 1
    p.tau = 0.0;
    p.off = 0;
    p.step = static_cast<int32_t>(sizeof(R));
    p.tb = 0;
}

}  // namespace mcrng
