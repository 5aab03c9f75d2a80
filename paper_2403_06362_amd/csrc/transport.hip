// Fixed-source 1-D slab transport kernels for gfx950 (history-based schedule).
//
// k_transport (history-based, persistent).  A block takes work units (a run
// of histories of one batch of one problem) from a global counter.  For each
// unit it stages the problem's cells in LDS, zeroes an LDS tally slice and
// runs the unit's histories one per lane; a wave's empty lanes take the next
// histories from the wave's ring, seeded 64 at a time.  Every track length is
// scored as the integer q = round-half-even(s 2^56) into the LDS slice (two
// 64-bit LDS atomics, one per 32-bit limb, exact while fewer than 2^32 of the
// unit's scores fall in one bin), so the unit's partial tally is an exact
// integer whatever order the lanes score in.  At the end of the unit the block
// adds its tally copies (carrying a wrap of the low limb) and writes the slice
// to the unit's own partial-tally slot in HBM.  (Carrying every score's wrap,
// with a returning low-word atomic, measured 5-6% slower.)
//
// k_transport_chain holds two units of one problem per block, so that lanes
// go on without a pause between units.
//
// k_reduce sums the partial slots of each (problem, batch) in unit order
// (a fixed order; integer addition makes any order give the same bits),
// converts the 128-bit sums to double with round-half-even, normalises the
// flux and reduces per-problem diagnostics.
//
// The per-history arithmetic (flight sampling, cell / time marching,
// collision, scoring) follows the same fixed IEEE operation sequence in FP64
// mode and in FP32-flight mode; it is spelled out in particle.hpp.
#include <algorithm>

#include "particle.hpp"

namespace mcrng {

__global__ void k_fill_u32(uint32_t* p, uint64_t n, uint32_t v) {
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<uint64_t>(gridDim.x) * blockDim.x)
        p[i] = v;
}

__global__ void k_fill_u64(uint64_t* p, uint64_t n, uint64_t v) {
    for (uint64_t i = static_cast<uint64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < n;
         i += static_cast<uint64_t>(gridDim.x) * blockDim.x)
        p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, uint64_t n, uint32_t v, hipStream_t st) {
    if (n == 0) return hipSuccess;
    uint64_t b = (n + 255) / 256;
    if (b > 4096) b = 4096;
    hipLaunchKernelGGL(k_fill_u32, dim3(static_cast<unsigned>(b)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

hipError_t launch_fill_u64(uint64_t* p, uint64_t n, uint64_t v, hipStream_t st) {
    if (n == 0) return hipSuccess;
    uint64_t b = (n + 255) / 256;
    if (b > 4096) b = 4096;
    hipLaunchKernelGGL(k_fill_u64, dim3(static_cast<unsigned>(b)), dim3(256), 0, st, p, n, v);
    return hipGetLastError();
}

// LDS layout: [tally: copies x (low limbs, high limbs) x max_slice u64][edges]
// [sig][rsig][below u64][bin i32][tedges]; with one region per problem the
// four per-cell arrays after the edges are left out (registers hold them).
__host__ __device__ inline size_t align16(size_t v) { return (v + 15) & ~static_cast<size_t>(15); }

size_t transport_lds_bytes(const TransportParams& p, int f32) {
    const size_t rs = f32 ? sizeof(float) : sizeof(double);
    size_t b = align16(static_cast<size_t>(p.tally_copies) * p.max_slice * 2 * sizeof(uint64_t));
    b += align16((p.max_cells + 1) * rs);
    if (!p.one_region) {
        b += align16(p.max_cells * rs);
        b += align16(p.max_cells * rs);
        b += align16(p.max_cells * sizeof(uint64_t));
        b += align16(p.max_cells * sizeof(int32_t));
    }
    b += align16((p.max_tedges > 0 ? p.max_tedges : 1) * rs);
    return b;
}

size_t transport_static_lds_bytes(int block) {
    // skip table, rings, ring slice tags (k_transport_chain), block words
    return static_cast<size_t>(kStrideDigits) * kStrideRadix * 2 * sizeof(uint64_t) +
           static_cast<size_t>(block / 64) * 128 * (sizeof(uint64_t) + 1) + 512;
}

// A record that is the same on every lane, in scalar registers: the compiler
// loads one through an address it cannot prove unchanged into vector registers
// (24 of them here, and one wave per SIMD fewer).
template <class T>
__device__ __forceinline__ T uniform_record(const T& v) {
    static_assert(sizeof(T) % 4 == 0, "whole words");
    uint32_t w[sizeof(T) / 4];
    __builtin_memcpy(w, &v, sizeof(T));
#pragma unroll
    for (uint32_t& x : w) x = __builtin_amdgcn_readfirstlane(x);
    T r;
    __builtin_memcpy(&r, w, sizeof(T));
    return r;
}

// The block's LDS arrays after the tally slices.
template <bool F32, bool ONE>
struct CellArrays {
    using R = typename Particle<F32>::R;
    R *edge, *sig, *rsig, *tedge;
    uint64_t* below;
    int32_t* bin8;
    __device__ __forceinline__ CellArrays(const TransportParams& P, unsigned char* smem) {
        size_t off = align16(static_cast<size_t>(P.tally_copies) * P.max_slice * 2 * sizeof(uint64_t));
        edge = reinterpret_cast<R*>(smem + off);
        off += align16((P.max_cells + 1) * sizeof(R));
        sig = rsig = nullptr;
        below = nullptr;
        bin8 = nullptr;
        if constexpr (!ONE) {
            sig = reinterpret_cast<R*>(smem + off);
            off += align16(P.max_cells * sizeof(R));
            rsig = reinterpret_cast<R*>(smem + off);
            off += align16(P.max_cells * sizeof(R));
            below = reinterpret_cast<uint64_t*>(smem + off);
            off += align16(P.max_cells * sizeof(uint64_t));
            bin8 = reinterpret_cast<int32_t*>(smem + off);
            off += align16(P.max_cells * sizeof(int32_t));
        }
        tedge = reinterpret_cast<R*>(smem + off);
    }
};

// Stages problem PR's cells, time edges and stride skip table (all threads of
// the block; the caller synchronises).
template <bool F32, bool TIMED, bool ONE, int BLOCK>
__device__ __forceinline__ void stage_problem(const TransportParams& P, const DevProblem& PR,
                                              const CellArrays<F32, ONE>& A, uint64_t* skip, uint32_t tid) {
    using R = typename Particle<F32>::R;
    const R *g_edge, *g_sig, *g_tedge;
    if constexpr (F32) {
        g_edge = P.edges32;
        g_sig = P.sig32;
        g_tedge = P.tedges32;
    } else {
        g_edge = P.edges64;
        g_sig = P.sig64;
        g_tedge = P.tedges64;
    }
    // FP32: widths from entry 1 on
    for (uint32_t i = tid; i <= PR.n_cells; i += BLOCK)
        A.edge[i] = F32 ? (i == 0 ? R(0) : g_edge[PR.edge_off + i - 1]) : g_edge[PR.edge_off + i];
    if constexpr (!ONE)
        for (uint32_t i = tid; i < PR.n_cells; i += BLOCK) {
            const R sg = g_sig[PR.cell_off + i];
            A.sig[i] = sg;
            A.rsig[i] = recip_refined(sg);
            A.below[i] = uniform_below(P.scat64[PR.cell_off + i]);
            A.bin8[i] = 8 * P.cbin[PR.cell_off + i];
        }
    if (TIMED)
        for (uint32_t i = tid; i <= PR.n_time_bins; i += BLOCK) A.tedge[i] = g_tedge[PR.tedge_off + i];
    if (PR.seed_kind == SEED_STRIDE)
        for (uint32_t i = tid; i < PR.stride_digits * kStrideRadix * 2u; i += BLOCK) skip[i] = PR.table[i];
}

template <bool F32, bool ONE>
__device__ __forceinline__ LdsCells<F32, ONE> staged_cells(const TransportParams& P, const DevProblem& PR,
                                                           const CellArrays<F32, ONE>& A) {
    using R = typename Particle<F32>::R;
    LdsCells<F32, ONE> C;
    C.edge_base = reinterpret_cast<const char*>(A.edge);
    C.sig_base = reinterpret_cast<const char*>(A.sig);
    C.rsig_base = reinterpret_cast<const char*>(A.rsig);
    C.below_base = reinterpret_cast<const char*>(A.below);
    C.bin_base = reinterpret_cast<const char*>(A.bin8);
    C.tedge = A.tedge;
    C.sig1 = C.rsig1 = R(0);
    C.below1 = 0;
    if constexpr (ONE) {
        R sg;
        if constexpr (F32)
            sg = P.sig32[PR.cell_off];
        else
            sg = P.sig64[PR.cell_off];
        C.sig1 = uniform_value(sg);
        C.rsig1 = uniform_value(recip_refined(sg));
        C.below1 = uniform_value(uniform_below(P.scat64[PR.cell_off]));
    }
    C.n_off = PR.n_cells * static_cast<uint32_t>(sizeof(R));
    C.n_time_bins = static_cast<int32_t>(PR.n_time_bins);
    C.n_space_bins = static_cast<int32_t>(PR.n_space_bins);
    return C;
}

__device__ __forceinline__ SeedDev problem_seed(const DevProblem& PR, const uint64_t* skip) {
    SeedDev S;
    S.kind = static_cast<int>(PR.seed_kind);
    S.stride_digits = PR.stride_digits;
    S.base = PR.seed_base;
    S.first_index = PR.first_index;
    S.table = skip;
    return S;
}

// The limbs of one LDS tally bin as a word pair low + 2^32 high, 0 <= low < 2^32
// (the low limbs' sum is signed; the bin's total is not negative).
__device__ __forceinline__ void add_limbs(uint64_t lo, uint64_t hi, uint64_t* plo, uint64_t* phi) {
    *plo += lo & 0xffffffffull;
    *phi += hi + static_cast<uint64_t>(static_cast<int64_t>(lo) >> 32);
}

// Waiting lanes at which a wave's collision pass runs: `full` of `all` slots,
// and the same share of the live ones once lanes stay empty (a wave's last
// histories would otherwise wait for each other at every collision), at
// least one and at most all of them.
__device__ __forceinline__ uint32_t wave_batch(uint32_t full, uint32_t live, uint32_t all) {
    const uint32_t b = (live * full + all - 1u) / all;
    return b < live ? b : live;
}

// Empty lanes at which a wave takes new histories (about one history ends per
// collision pass of the long-chain slab, and a refill costs a seventh of one).
constexpr uint32_t kRefill = 3;

// A lane's history slot is flying (its bit in G: takes geometry steps),
// waiting at a collision site (W), or empty.
//   Bound by vector issue where histories are many: an instruction of a wave
// takes a SIMD 4.3 cycles on average and the vector units are 93-98% busy, so
// the bookkeeping lives in scalar registers and a geometry pass has no branch
// per outcome.  With phases in vector registers: 512 slabs of 1.3e8 histories
// 22.2 ms, now 9.2 (with the units in order of expected time); 2e7
// time-dependent histories of ten regions 1588 us, now 1184; the long chain of
// 1e8 histories on the chained kernel 35.2 ms, now 25.8 (173 vector
// instructions per event, now 121).  A run of 1e6 thick-slab histories ends
// with its longest histories' serial chains: 3.5 ms, now 1.5.
template <bool F32, bool TIMED, bool ONE, int H, int BLOCK>
__global__ void __launch_bounds__(BLOCK, (H == 1) ? 7 : 1) k_transport(TransportParams P) {
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint32_t s_unit;
    __shared__ uint32_t s_next;
    __shared__ unsigned long long s_diag[kNDiag];
    // the current problem's stride skip table: a history's start is a chain
    // of dependent table reads, cheaper from LDS than from the cache
    __shared__ uint64_t s_skip[kStrideDigits * kStrideRadix * 2];
    // per wave: start states of the next histories, seeded 64 at a time
    __shared__ uint64_t s_ring[BLOCK / 64][128];

    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const CellArrays<F32, ONE> A(P, smem);
    const uint32_t copy = (P.tally_copies > 1) ? (wid % P.tally_copies) : 0u;
    const uint32_t copy_bytes = P.max_slice * 16u;
    LimbTally tally;
    tally.lo = reinterpret_cast<char*>(smem) + static_cast<size_t>(copy) * copy_bytes;
    tally.hi_off = P.max_slice * 8u;
    int32_t cur_problem = -1;

    for (;;) {
        if (tid == 0) {
            s_unit = atomicAdd(P.unit_counter, 1u);
            s_next = 0;
        }
        if (tid < kNDiag) s_diag[tid] = 0;
        __syncthreads();
        const uint32_t pos = __builtin_amdgcn_readfirstlane(s_unit);
        if (pos >= P.n_units) break;
        const uint32_t ui = __builtin_amdgcn_readfirstlane(P.order[pos]);
        const WorkUnit U = uniform_record(P.units[ui]);
        const DevProblem PR = uniform_record(P.problems[U.problem]);
        const uint32_t slice = PR.slice_bins;

        for (uint32_t c = 0; c < P.tally_copies; ++c) {
            uint64_t* const t = reinterpret_cast<uint64_t*>(smem) + static_cast<size_t>(c) * P.max_slice * 2;
            for (uint32_t i = tid; i < slice; i += BLOCK) {
                t[i] = 0;
                t[P.max_slice + i] = 0;
            }
        }
        if (static_cast<int32_t>(U.problem) != cur_problem) {
            stage_problem<F32, TIMED, ONE, BLOCK>(P, PR, A, s_skip, tid);
            cur_problem = static_cast<int32_t>(U.problem);
        }
        __syncthreads();
        const LdsCells<F32, ONE> C = staged_cells<F32, ONE>(P, PR, A);
        const SeedDev S = problem_seed(PR, s_skip);
        const uint64_t stride_q = PR.stride_q;

        Particle<F32> p[H];
        uint32_t draws[H];   // numbers drawn by the lane's history, before an absorption's one
        uint64_t G[H], W[H], up[H];
#pragma unroll
        for (int h = 0; h < H; ++h) {
            init_particle_at<F32, TIMED>(p[h], C, 0ull);
            draws[h] = 0;
            G[h] = W[h] = 0;
            up[h] = ~0ull;
        }
        // wave-uniform counts of the unit (scalar registers)
        uint64_t w_events = 0, w_colls = 0;
        uint32_t w_leak = 0, w_lr = 0, w_abs = 0, w_cen = 0;
        // per lane, over the histories this lane ended (their total draws
        // follow from the wave counts: one for each history's first flight,
        // one per collision for the absorption test and two more per scatter)
        uint32_t l_maxd = 0, l_over = 0;
        bool exhausted = false;   // wave-uniform: no history of the unit left for this wave
        // the wave's ring of seeded histories (positions & 127): [r_next, r_filled)
        uint64_t* ring = s_ring[wid];
        uint32_t r_next = 0, r_filled = 0;   // wave-uniform
        bool unit_taken = false;             // wave-uniform: s_next has passed the unit's end
        auto ended = [&](uint64_t m, uint32_t d) {
            if (in_mask(m)) {
                l_maxd = d > l_maxd ? d : l_maxd;
                if (stride_q != 0 && d > stride_q) l_over++;
            }
        };

        // Geometry steps for every lane with a flight until enough lanes wait
        // at a collision site (or stand empty while histories remain), or
        // none can move; then the collision pass: empty lanes take new
        // histories, and every waiting particle runs its collision draws and
        // samples its next flight.  Every particle still runs its own
        // operations in its own order.
        for (;;) {
            uint64_t fresh[H], live = 0;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                fresh[h] = 0;
                const uint64_t need = ~(G[h] | W[h]);
                if (!exhausted && need != 0) {
                    const uint32_t nneed = mask_count(need);
                    if (r_filled - r_next < nneed && !unit_taken) {
                        // seed the next 64 histories of the unit at once (one per
                        // lane), so that a refill is an LDS read
                        uint32_t base = 0;
                        if (lane == 0) base = atomicAdd(&s_next, 64u);
                        base = __builtin_amdgcn_readfirstlane(base);
                        if (base + 64u >= U.count) unit_taken = true;
                        const uint32_t got = base < U.count ? (U.count - base < 64u ? U.count - base : 64u) : 0u;
                        if (lane < got) ring[(r_filled + lane) & 127u] = stream_start_z(P.lcg, S, U.j0 + base + lane);
                        r_filled += got;
                        __builtin_amdgcn_wave_barrier();
                    }
                    const uint32_t avail = r_filled - r_next;
                    const uint32_t take = avail < nneed ? avail : nneed;
                    const uint32_t rank = mask_rank(need);
                    fresh[h] = need & wave_mask(rank < take);
                    if (in_mask(fresh[h])) {
                        init_particle_at<F32, TIMED>(p[h], C, ring[(r_next + rank) & 127u]);
                        draws[h] = 1;
                    }
                    up[h] |= fresh[h];
                    r_next += take;
                    if (unit_taken && r_next == r_filled) exhausted = true;
                    __builtin_amdgcn_wave_barrier();
                }
                live |= G[h] | W[h] | fresh[h];
            }
            if (live == 0) break;
#pragma unroll
            for (int h = 0; h < H; ++h) {
                uint64_t fly = fresh[h];
                if (W[h] != 0) {
                    w_colls += mask_count(W[h]);
                    const uint64_t scat = collide_pass<F32>(p[h], C, P.lcg, W[h], up[h]);
                    const uint64_t absorbed = W[h] & ~scat;
                    w_abs += mask_count(absorbed);
                    ended(absorbed, draws[h] + 1u);
                    draws[h] += sel_const<3, 0>(scat);
                    fly |= scat;
                    W[h] = 0;
                }
                if (in_mask(fly)) sample_tau<F32>(p[h], P.lcg);
                G[h] |= fly;
            }
            // idle[h]: the lanes that stay empty; at `batch` waiting lanes the
            // geometry steps end (all live ones wait then at the latest)
            uint64_t idle[H];
            uint32_t nidle = 0, batch = 0, nwait = 0;
            auto set_batch = [&]() {
                nidle = 0;
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    idle[h] = exhausted ? ~(G[h] | W[h]) : 0ull;
                    nidle += mask_count(idle[h]);
                }
                batch = wave_batch(P.coll_batch, 64u * H - nidle, 64u * H);
            };
            set_batch();
            do {
                nwait = 0;
                uint64_t any_end = 0;
#pragma unroll
                for (int h = 0; h < H; ++h) {
                    if (H == 1 || G[h] != 0) {
                        w_events += mask_count(G[h]);
                        const GeomOut o = geom_pass<F32, TIMED>(p[h], C, G[h], up[h], tally);
                        const uint64_t end = o.leak | o.census;
                        G[h] &= ~(o.coll | end);
                        W[h] |= o.coll;
                        if (end != 0) {
                            w_leak += mask_count(o.leak);
                            w_lr += mask_count(o.leak & up[h]);
                            if (TIMED) w_cen += mask_count(o.census);
                            ended(end, draws[h]);
                        }
                        any_end |= end;
                    }
                }
                if (any_end != 0) set_batch();
#pragma unroll
                for (int h = 0; h < H; ++h) nwait += mask_count(~(G[h] | idle[h]));
            } while (nwait < batch);
        }

        // unit diagnostics: the wave's counts and the lanes' into LDS
        if (lane == 0) {
            const unsigned long long ends = static_cast<unsigned long long>(w_leak) + w_abs + w_cen;
            atomicAdd(&s_diag[D_HISTORIES], ends);
            atomicAdd(&s_diag[D_LEAK_LEFT], static_cast<unsigned long long>(w_leak - w_lr));
            atomicAdd(&s_diag[D_LEAK_RIGHT], static_cast<unsigned long long>(w_lr));
            atomicAdd(&s_diag[D_ABSORBED], static_cast<unsigned long long>(w_abs));
            atomicAdd(&s_diag[D_CENSUS], static_cast<unsigned long long>(w_cen));
            atomicAdd(&s_diag[D_EVENTS], static_cast<unsigned long long>(w_events));
            atomicAdd(&s_diag[D_COLLISIONS], static_cast<unsigned long long>(w_colls));
            atomicAdd(&s_diag[D_DRAWS], ends + 3ull * w_colls - 2ull * w_abs);
        }
        atomicMax(&s_diag[D_MAX_DRAWS], static_cast<unsigned long long>(l_maxd));
        atomicAdd(&s_diag[D_OVER_STRIDE], static_cast<unsigned long long>(l_over));
        __syncthreads();

        uint64_t* dst = P.partial + U.slot;
        for (uint32_t i = tid; i < slice; i += BLOCK) {
            uint64_t lo = 0, hi = 0;
            for (uint32_t c = 0; c < P.tally_copies; ++c) {
                const uint64_t* t = reinterpret_cast<uint64_t*>(smem) + static_cast<size_t>(c) * P.max_slice * 2;
                add_limbs(t[i], t[P.max_slice + i], &lo, &hi);
            }
            dst[2 * i] = lo;
            dst[2 * i + 1] = hi;
        }
        if (tid < kNDiag) P.unit_diag[static_cast<size_t>(ui) * kNDiag + tid] = s_diag[tid];
        __syncthreads();
    }
}

// Chained units (a set of one problem, one history per lane).  In k_transport
// a block's lanes fall idle while the slowest histories of its unit finish
// (history lengths are heavy-tailed: the long-chain slab has a median of 23
// events and a longest of about 1750), and the block's next unit starts only
// after a barrier.  Here a block holds two units at once, each
// with its own LDS tally slice: once every history of the feeding unit has
// been handed out, the block takes its next unit into the other slice and
// the lanes go on without a pause.  A unit's slice is written to the unit's
// HBM slot by the wave that ends its last history, and the slice is then free
// for the block's next unit.  Each particle still runs its own operations in
// its own order and the counts are integer sums, so every output equals
// k_transport's.  The problem's diagnostics are summed over the block's
// units and written to the block's last unit (the per-unit words start at
// zero; the reduction sums a problem's units).
//
// Block state in LDS (only lane 0 of a wave touches it, with
// workgroup-scope atomics):
//   s_w     bit s (s = 0, 1): slice s holds a unit; kWant: the feeding unit
//           has been handed out and the block wants its next unit; kNoMore:
//           the launch's counter has passed its last unit
//   s_feed  (claim number << 1) | slice of the unit handed out now, or kNone
//   s_cs[s] the unit in slice s: first index, HBM slot, the histories not
//           yet ended, and the hand-out word (claim number, size, handed
//           out)
// Claims are serial: kWant is set once per unit, by the wave that hands out
// its last histories, and cleared by the compare-exchange that takes a free
// slice, so exactly one wave claims; that wave is the one that finds both
// conditions (kWant set, a slice free), whichever of the two came last.
// A wave with nothing to run waits only while no unit is being handed out
// and the counter is not exhausted: then kWant is set and both slices are
// busy (or a claim is under way), a busy slice's live histories run in other
// waves' lanes, the last of them frees the slice and that wave claims.  So
// every wave ends once the counter has passed the last unit and its own
// lanes and ring are empty.
namespace chain {
constexpr uint32_t kWant = 4u, kNoMore = 8u, kNone = 0xffffffffu;
// A slice's hand-out word: claim number (24 bits, mod 2^24) | the unit's
// histories (20 bits) | histories handed out (20 bits).  A wave takes
// histories by compare-exchange on the whole word, so a wave that read a
// stale feed word (its unit replaced in the meantime) fails the exchange and
// changes nothing, and a unit's size is read with the word, never from a
// field a new claim could have overwritten.
constexpr int kWordCount = 20, kWordGen = 40;
constexpr uint64_t kWordMask = (1ull << kWordCount) - 1ull;
static_assert(kMaxUnitHistories + 64u < (1u << kWordCount), "a unit's size and hand-out count fit their fields");
struct Slot {
    uint64_t j0;
    uint64_t hslot;
    uint64_t word;
    uint32_t alive;
    uint32_t pad;
};
}  // namespace chain

#define CH_ACQ_REL(op, p, v) __hip_atomic_##op((p), (v), __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_WORKGROUP)

// Seven waves per SIMD (72 VGPRs), six (80) with time bins in FP64, which would
// spill: 20 x 20 space-time bins, units of 8192: 2e7 histories 1091 us at seven,
// 1047 at six, 6e7 2746 and 2641.  k_transport holds seven there (952 and
// 2468 us; six within 1%), so such runs stay on it (transport_chain_fits).
template <bool F32, bool TIMED, bool ONE, int BLOCK>
__global__ void __launch_bounds__(BLOCK, (F32 || !TIMED) ? 7 : 6) k_transport_chain(TransportParams P) {
    using chain::kNone;
    using chain::kNoMore;
    using chain::kWant;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ uint64_t s_skip[kStrideDigits * kStrideRadix * 2];
    __shared__ uint64_t s_ring[BLOCK / 64][128];
    __shared__ uint8_t s_rslice[BLOCK / 64][128];   // the slice of each ring entry's unit
    __shared__ chain::Slot s_cs[2];
    __shared__ uint32_t s_w, s_feed, s_seq, s_last_ui;
    __shared__ unsigned long long s_diag[kNDiag];

    const uint32_t tid = threadIdx.x;
    const uint32_t lane = tid & 63u;
    const uint32_t wid = __builtin_amdgcn_readfirstlane(tid >> 6);
    const CellArrays<F32, ONE> A(P, smem);
    const DevProblem PR = P.problems[0];
    const uint32_t slice = PR.slice_bins;
    const uint32_t slice1_off = P.max_slice * 16u;   // bytes from slice 0 to slice 1
    stage_problem<F32, TIMED, ONE, BLOCK>(P, PR, A, s_skip, tid);
    for (uint32_t i = tid; i < 4u * P.max_slice; i += BLOCK) reinterpret_cast<uint64_t*>(smem)[i] = 0ull;
    if (tid < kNDiag) s_diag[tid] = 0;

    // lane 0 of a wave: puts the launch's next unit into free slice f
    auto take_unit = [&](uint32_t f) {
        const uint32_t pos = atomicAdd(P.unit_counter, 1u);
        if (pos >= P.n_units) {
            CH_ACQ_REL(fetch_or, &s_w, kNoMore);
            CH_ACQ_REL(fetch_and, &s_w, ~(1u << f));
            return;
        }
        const uint32_t ui = P.order[pos];
        const WorkUnit U = P.units[ui];
        const uint32_t seq = s_seq + 1u;
        s_seq = seq;
        s_last_ui = ui;
        s_cs[f].j0 = U.j0;
        s_cs[f].hslot = U.slot;
        s_cs[f].alive = U.count;
        __hip_atomic_store(&s_cs[f].word,
                           (static_cast<uint64_t>(seq & 0xffffffu) << chain::kWordGen) |
                               (static_cast<uint64_t>(U.count) << chain::kWordCount),
                           __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&s_feed, (seq << 1) | f, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
    };
    // lane 0 of a wave: claims a free slice if the block wants a unit
    auto try_claim = [&]() {
        uint32_t old = __hip_atomic_load(&s_w, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
        for (;;) {
            if (!(old & kWant) || (old & kNoMore)) return;
            const int f = !(old & 1u) ? 0 : (!(old & 2u) ? 1 : -1);
            if (f < 0) return;
            if (__hip_atomic_compare_exchange_strong(&s_w, &old, (old & ~kWant) | (1u << f), __ATOMIC_ACQ_REL,
                                                     __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP)) {
                take_unit(static_cast<uint32_t>(f));
                return;
            }
        }
    };
    if (tid == 0) {
        s_w = 1u;
        s_seq = 0;
        s_last_ui = kNone;
        s_feed = kNone;
        take_unit(0);
    }
    __syncthreads();

    const LdsCells<F32, ONE> C = staged_cells<F32, ONE>(P, PR, A);
    const SeedDev S = problem_seed(PR, s_skip);
    const uint64_t stride_q = PR.stride_q;
    uint64_t* const ring = s_ring[wid];
    uint8_t* const rsl = s_rslice[wid];

    // The lanes in `ended` have ended their histories.  A wave counts its
    // ended histories per slice and subtracts them from the unit's live
    // count once none of its lanes runs a history of that slice (so about
    // once per unit and wave, not at every end); the wave whose subtraction
    // reaches zero writes the unit's slice to HBM, clears it and frees it.
    uint64_t live = 0;     // wave-uniform: lanes running a history
    uint64_t s1mask = 0;   // wave-uniform: lanes whose history is in slice 1
    uint32_t acc0 = 0, acc1 = 0;
    auto report = [&](uint32_t sl, uint32_t n) {
        uint32_t old = 0;
        if (lane == 0) old = CH_ACQ_REL(fetch_sub, &s_cs[sl].alive, n);
        old = __builtin_amdgcn_readfirstlane(old);
        if (old != n) return;
        uint64_t* t = reinterpret_cast<uint64_t*>(smem) + (sl ? static_cast<size_t>(P.max_slice) * 2 : 0);
        uint64_t* dst = P.partial + s_cs[sl].hslot;
        for (uint32_t i = lane; i < slice; i += 64u) {
            uint64_t lo = 0, hi = 0;
            add_limbs(t[i], t[P.max_slice + i], &lo, &hi);
            dst[2 * i] = lo;
            dst[2 * i + 1] = hi;
            t[i] = 0ull;
            t[P.max_slice + i] = 0ull;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        if (lane == 0) {
            CH_ACQ_REL(fetch_and, &s_w, ~(1u << sl));
            try_claim();
        }
        __builtin_amdgcn_wave_barrier();
    };
    auto ends = [&](uint64_t ended) {
        const uint32_t e1 = static_cast<uint32_t>(__popcll(ended & s1mask));
        acc1 += e1;
        acc0 += static_cast<uint32_t>(__popcll(ended)) - e1;
        live &= ~ended;
        s1mask &= ~ended;
        if (acc0 != 0 && (live & ~s1mask) == 0) {
            report(0, acc0);
            acc0 = 0;
        }
        if (acc1 != 0 && (live & s1mask) == 0) {
            report(1, acc1);
            acc1 = 0;
        }
    };
    // seeds up to 64 histories of the feeding unit into the ring; returns
    // false when no unit is feeding or it has been handed out
    uint32_t r_next = 0, r_filled = 0;   // wave-uniform: the ring holds [r_next, r_filled)
    auto fetch = [&]() -> bool {
        // lane 0: takes up to 64 histories of the feeding unit, if it has any left
        uint32_t fd = kNone, base = 0, cnt = 0;
        if (lane == 0) {
            fd = __hip_atomic_load(&s_feed, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
            if (fd != kNone) {
                uint64_t* w = &s_cs[fd & 1u].word;
                const uint64_t gen = (fd >> 1) & 0xffffffu;
                uint64_t cur = __hip_atomic_load(w, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
                for (;;) {
                    const uint32_t c = static_cast<uint32_t>(cur >> chain::kWordCount) & chain::kWordMask;
                    const uint32_t h = static_cast<uint32_t>(cur) & chain::kWordMask;
                    if ((cur >> chain::kWordGen) != gen || h >= c) {   // replaced, or handed out
                        fd = kNone;
                        break;
                    }
                    if (__hip_atomic_compare_exchange_strong(w, &cur, cur + 64u, __ATOMIC_ACQ_REL, __ATOMIC_ACQUIRE,
                                                             __HIP_MEMORY_SCOPE_WORKGROUP)) {
                        base = h;
                        cnt = c;
                        break;
                    }
                }
            }
        }
        fd = __builtin_amdgcn_readfirstlane(fd);
        if (fd == kNone) return false;
        const uint32_t f = fd & 1u;
        base = __builtin_amdgcn_readfirstlane(base);
        cnt = __builtin_amdgcn_readfirstlane(cnt);
        const uint32_t got = cnt - base < 64u ? cnt - base : 64u;
        if (lane < got) {
            ring[(r_filled + lane) & 127u] = stream_start_z(P.lcg, S, s_cs[f].j0 + base + lane);
            rsl[(r_filled + lane) & 127u] = static_cast<uint8_t>(f);
        }
        r_filled += got;
        if (base + 64u >= cnt && lane == 0) {
            // this wave took the unit's last histories
            __hip_atomic_store(&s_feed, kNone, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_WORKGROUP);
            CH_ACQ_REL(fetch_or, &s_w, kWant);
            try_claim();
        }
        __builtin_amdgcn_wave_barrier();
        return true;
    };

    Particle<F32> p;
    init_particle_at<F32, TIMED>(p, C, 0ull);
    uint32_t draws = 0;         // numbers drawn by the lane's history, before an absorption's one
    uint64_t G = 0, W = 0;      // flying, waiting (`live` also covers them)
    uint64_t up = ~0ull;        // lanes with mu > 0
    uint32_t tl = 0;            // byte offset of the slice of the lane's history
    uint64_t w_events = 0, w_colls = 0;
    uint32_t w_leak = 0, w_lr = 0, w_abs = 0, w_cen = 0;
    uint32_t l_maxd = 0, l_over = 0;
    bool starved = false;   // wave-uniform: the last refill found no history to take
    uint64_t done = 0;      // lanes whose ended histories are not reported yet
    auto note_end = [&](uint64_t m, uint32_t d) {
        if (in_mask(m)) {
            l_maxd = d > l_maxd ? d : l_maxd;
            if (stride_q != 0 && d > stride_q) l_over++;
        }
    };

    for (;;) {
        // report the histories that ended since the last pass (here only: one
        // copy of that code keeps the scalar registers of the loops below)
        if (done != 0) {
            ends(done);
            done = 0;
        }
        // collision pass: refill the empty lanes first
        uint64_t fresh = 0;
        const uint64_t need = ~(G | W);
        if (mask_count(need) >= kRefill || (G | W) == 0) {
            const uint32_t nneed = mask_count(need);
            starved = false;
            while (r_filled - r_next < nneed) {
                if (!fetch()) {
                    starved = true;
                    break;
                }
            }
            const uint32_t avail = r_filled - r_next;
            const uint32_t take = avail < nneed ? avail : nneed;
            const uint32_t rank = mask_rank(need);
            fresh = need & wave_mask(rank < take);
            const uint32_t e = (r_next + rank) & 127u;
            const uint64_t in1 = fresh & wave_mask(rsl[e] != 0);
            if (in_mask(fresh)) {
                init_particle_at<F32, TIMED>(p, C, ring[e]);
                tl = sel_or_zero(in1, slice1_off);
                draws = 1;
            }
            up |= fresh;
            s1mask |= in1;
            live = G | W | fresh;
            r_next += take;
            __builtin_amdgcn_wave_barrier();
        }
        if (live == 0) {
            // nothing to run: done once the launch has no unit left, else
            // wait for a unit (another wave frees a slice or is claiming)
            uint32_t w = 0;
            if (lane == 0) w = __hip_atomic_load(&s_w, __ATOMIC_ACQUIRE, __HIP_MEMORY_SCOPE_WORKGROUP);
            w = __builtin_amdgcn_readfirstlane(w);
            if ((w & kNoMore) && r_next == r_filled) break;
            __builtin_amdgcn_s_sleep(4);
            continue;
        }
        uint64_t fly = fresh;
        if (W != 0) {
            w_colls += mask_count(W);
            const uint64_t scat = collide_pass<F32>(p, C, P.lcg, W, up);
            const uint64_t absorbed = W & ~scat;
            W = 0;
            draws += sel_const<3, 0>(scat);
            if (absorbed != 0) {
                w_abs += mask_count(absorbed);
                note_end(absorbed, draws + 1u);
                done |= absorbed;
            }
            fly |= scat;
        }
        if (in_mask(fly)) sample_tau<F32>(p, P.lcg);
        G |= fly;
        if (G == 0) continue;

        // geometry steps until `batch` lanes wait (empty lanes count while
        // there may be histories for them)
        uint64_t idle = starved ? ~(G | W) : 0ull;
        uint32_t batch = wave_batch(P.coll_batch, 64u - mask_count(idle), 64u);
        LimbTally tally;
        tally.lo = reinterpret_cast<char*>(smem) + tl;
        tally.hi_off = P.max_slice * 8u;
        do {
            w_events += mask_count(G);
            const GeomOut o = geom_pass<F32, TIMED>(p, C, G, up, tally);
            const uint64_t end = o.leak | o.census;
            G &= ~(o.coll | end);
            W |= o.coll;
            if (end != 0) {
                w_leak += mask_count(o.leak);
                w_lr += mask_count(o.leak & up);
                if (TIMED) w_cen += mask_count(o.census);
                note_end(end, draws);
                done |= end;
                if (starved) {
                    idle |= end;
                    batch = wave_batch(P.coll_batch, 64u - mask_count(idle), 64u);
                }
            }
        } while (mask_count(~(G | idle)) < batch);
    }

    // the problem's diagnostics: the block's sums, into its last unit's words
    if (lane == 0) {
        const unsigned long long nend = static_cast<unsigned long long>(w_leak) + w_abs + w_cen;
        atomicAdd(&s_diag[D_HISTORIES], nend);
        atomicAdd(&s_diag[D_LEAK_LEFT], static_cast<unsigned long long>(w_leak - w_lr));
        atomicAdd(&s_diag[D_LEAK_RIGHT], static_cast<unsigned long long>(w_lr));
        atomicAdd(&s_diag[D_ABSORBED], static_cast<unsigned long long>(w_abs));
        atomicAdd(&s_diag[D_CENSUS], static_cast<unsigned long long>(w_cen));
        atomicAdd(&s_diag[D_EVENTS], static_cast<unsigned long long>(w_events));
        atomicAdd(&s_diag[D_COLLISIONS], static_cast<unsigned long long>(w_colls));
        atomicAdd(&s_diag[D_DRAWS], nend + 3ull * w_colls - 2ull * w_abs);
    }
    atomicMax(&s_diag[D_MAX_DRAWS], static_cast<unsigned long long>(l_maxd));
    atomicAdd(&s_diag[D_OVER_STRIDE], static_cast<unsigned long long>(l_over));
    __syncthreads();
    if (tid < kNDiag && s_last_ui != kNone) P.unit_diag[static_cast<size_t>(s_last_ui) * kNDiag + tid] = s_diag[tid];
}
#undef CH_ACQ_REL

template <bool F32, bool TIMED, bool ONE, int H, int BLOCK>
static hipError_t launch_t(const TransportParams& p, int grid, size_t lds, hipStream_t st, int* used) {
    auto kern = k_transport<F32, TIMED, ONE, H, BLOCK>;
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern),
                                           hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    if (grid <= 0) {
        int dev = 0, cus = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, reinterpret_cast<const void*>(kern), BLOCK, lds);
        if (e != hipSuccess) return e;
        if (per_cu < 1) per_cu = 1;
        grid = cus * per_cu;
    }
    if (static_cast<uint32_t>(grid) > p.n_units) grid = static_cast<int>(p.n_units);
    if (grid < 1) grid = 1;
    if (used) *used = grid;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(BLOCK), lds, st, p);
    return hipGetLastError();
}

template <bool F32, bool TIMED, bool ONE, int H>
static hipError_t launch_b(const TransportParams& p, int block, int grid, size_t lds, hipStream_t st, int* used) {
    switch (block) {
        case 64: return launch_t<F32, TIMED, ONE, H, 64>(p, grid, lds, st, used);
        case 128: return launch_t<F32, TIMED, ONE, H, 128>(p, grid, lds, st, used);
        case 512: return launch_t<F32, TIMED, ONE, H, 512>(p, grid, lds, st, used);
        case 1024: return launch_t<F32, TIMED, ONE, H, 1024>(p, grid, lds, st, used);
        default: return launch_t<F32, TIMED, ONE, H, 256>(p, grid, lds, st, used);
    }
}

template <bool F32, bool TIMED, bool ONE>
static hipError_t launch_h(const TransportParams& p, const LaunchShape& s, size_t lds, hipStream_t st, int* used) {
    switch (s.hist_per_lane) {
        // (several histories per lane: only the general form is built)
        case 2: return launch_b<F32, TIMED, false, 2>(p, s.block, s.grid, lds, st, used);
        case 4: return launch_b<F32, TIMED, false, 4>(p, s.block, s.grid, lds, st, used);
        default: return launch_b<F32, TIMED, ONE, 1>(p, s.block, s.grid, lds, st, used);
    }
}

// Blocks of `kern` that fit on one CU with `lds` bytes of dynamic LDS.
static hipError_t blocks_per_cu(const void* kern, int block, size_t lds, int* out) {
    if (lds > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
        if (e != hipSuccess) return e;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(out, kern, block, lds);
}

template <bool F32, bool TIMED, bool ONE, int BLOCK>
static hipError_t launch_chain_t(const TransportParams& p, int grid, size_t lds, hipStream_t st, int* used) {
    auto kern = k_transport_chain<F32, TIMED, ONE, BLOCK>;
    if (grid <= 0) {
        int dev = 0, cus = 0, per_cu = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        if (e != hipSuccess) return e;
        e = blocks_per_cu(reinterpret_cast<const void*>(kern), BLOCK, lds, &per_cu);
        if (e != hipSuccess) return e;
        if (per_cu < 1) per_cu = 1;
        grid = cus * per_cu;
    } else if (lds > 64 * 1024) {
        int per_cu = 0;
        hipError_t e = blocks_per_cu(reinterpret_cast<const void*>(kern), BLOCK, lds, &per_cu);
        if (e != hipSuccess) return e;
    }
    if (static_cast<uint32_t>(grid) > p.n_units) grid = static_cast<int>(p.n_units);
    if (grid < 1) grid = 1;
    if (used) *used = grid;
    hipLaunchKernelGGL(kern, dim3(grid), dim3(BLOCK), lds, st, p);
    return hipGetLastError();
}

template <bool F32, bool TIMED, bool ONE>
static hipError_t launch_chain_b(const TransportParams& p, const LaunchShape& s, size_t lds, hipStream_t st,
                                 int* used) {
    switch (s.block) {
        case 64: return launch_chain_t<F32, TIMED, ONE, 64>(p, s.grid, lds, st, used);
        case 128: return launch_chain_t<F32, TIMED, ONE, 128>(p, s.grid, lds, st, used);
        case 512: return launch_chain_t<F32, TIMED, ONE, 512>(p, s.grid, lds, st, used);
        case 1024: return launch_chain_t<F32, TIMED, ONE, 1024>(p, s.grid, lds, st, used);
        default: return launch_chain_t<F32, TIMED, ONE, 256>(p, s.grid, lds, st, used);
    }
}

template <bool F32, bool TIMED, bool ONE, int BLOCK>
static hipError_t chain_fits_t(const TransportParams& a, const TransportParams& b, int f32, bool* fits) {
    int na = 0, nb = 0;
    hipError_t e = blocks_per_cu(reinterpret_cast<const void*>(k_transport<F32, TIMED, ONE, 1, BLOCK>), BLOCK,
                                 transport_lds_bytes(a, f32), &na);
    if (e != hipSuccess) return e;
    e = blocks_per_cu(reinterpret_cast<const void*>(k_transport_chain<F32, TIMED, ONE, BLOCK>), BLOCK,
                      transport_lds_bytes(b, f32), &nb);
    if (e != hipSuccess) return e;
    // seven waves per SIMD are as many as help (eight measured 3% slower on
    // the long-chain slab: 28.2 against 27.3 ms), so fewer are not missed
    const int enough = std::max(1, 7 * 4 / (BLOCK / 64));
    *fits = nb >= 1 && nb >= std::min(na, enough);
    return hipSuccess;
}

template <bool F32, bool TIMED, bool ONE>
static hipError_t chain_fits_b(const TransportParams& a, const TransportParams& b, const LaunchShape& s, bool* fits) {
    switch (s.block) {
        case 64: return chain_fits_t<F32, TIMED, ONE, 64>(a, b, s.f32, fits);
        case 128: return chain_fits_t<F32, TIMED, ONE, 128>(a, b, s.f32, fits);
        case 512: return chain_fits_t<F32, TIMED, ONE, 512>(a, b, s.f32, fits);
        case 1024: return chain_fits_t<F32, TIMED, ONE, 1024>(a, b, s.f32, fits);
        default: return chain_fits_t<F32, TIMED, ONE, 256>(a, b, s.f32, fits);
    }
}

// Calls f with the precision, time-dependence and one-region flags of a launch
// as compile-time constants.
template <class F>
static hipError_t with_flags(int f32, int timed, int one, F f) {
    using T = std::true_type;
    using N = std::false_type;
    if (f32) {
        if (timed) return one ? f(T(), T(), T()) : f(T(), T(), N());
        return one ? f(T(), N(), T()) : f(T(), N(), N());
    }
    if (timed) return one ? f(N(), T(), T()) : f(N(), T(), N());
    return one ? f(N(), N(), T()) : f(N(), N(), N());
}

hipError_t transport_chain_fits(const TransportParams& single, const TransportParams& chained, const LaunchShape& s,
                                bool* fits) {
    *fits = false;
    // (asking for more LDS than there is would leave an error behind for the
    // next launch to report)
    int dev = 0, lds = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev);
    if (e != hipSuccess) return e;
    if (transport_lds_bytes(chained, s.f32) + transport_static_lds_bytes(s.block) > static_cast<size_t>(lds))
        return hipSuccess;
    return with_flags(s.f32, s.timed, static_cast<int>(single.one_region), [&](auto f, auto t, auto o) {
        return chain_fits_b<f.value, t.value, o.value>(single, chained, s, fits);
    });
}

hipError_t launch_transport(const TransportParams& p, const LaunchShape& s, hipStream_t st, int* grid_used) {
    if (p.n_units == 0) return hipSuccess;
    const size_t lds = transport_lds_bytes(p, s.f32);
    return with_flags(s.f32, s.timed, static_cast<int>(p.one_region), [&](auto f, auto t, auto o) {
        if (s.chain) return launch_chain_b<f.value, t.value, o.value>(p, s, lds, st, grid_used);
        return launch_h<f.value, t.value, o.value>(p, s, lds, st, grid_used);
    });
}

// ------------------------------------------------------------------ reduction

// Round-half-even conversion of the 128-bit integer (hi, lo) to double:
// keep the top 53 bits, round on the dropped bits, scale back exactly.
__device__ __forceinline__ double u128_to_double(uint64_t lo, uint64_t hi) {
    typedef unsigned __int128 u128;
    const u128 v = (static_cast<u128>(hi) << 64) | lo;
    if ((v >> 53) == 0) return static_cast<double>(lo);
    const int nbits = (hi != 0) ? 128 - __clzll(static_cast<long long>(hi)) : 64 - __clzll(static_cast<long long>(lo));
    const int sh = nbits - 53;
    u128 mant = v >> sh;
    const u128 rem = v - (mant << sh);
    const u128 half = static_cast<u128>(1) << (sh - 1);
    if (rem > half || (rem == half && (mant & 1))) mant += 1;
    return __builtin_ldexp(static_cast<double>(static_cast<uint64_t>(mant)), sh);
}

// One launch: blocks (tile, group) reduce a group's bins, blocks (0, n_groups +
// p) problem p's diagnostics.
// Bins: a tile of 8 bins, 32 unit lanes per bin.  A group's units are
// consecutive with consecutive partial slots (2 x slice_bins words each), so
// unit u's words for bin i sit at slot0 + (u - u0) 2 slice + 2 i.  Unit lane l
// sums units u0 + l, u0 + l + 32, ..., several loads in flight; the partial sums
// are then added in lane order (integers: any order gives the same bits).  The
// kernel waits for HBM: with 32 bins per tile and 8 unit lanes a group of 1000
// bins and 4096 units was 32 blocks of 512 dependent steps, 169 us.
constexpr int kRedBins = 8, kRedLanes = 32, kRedAhead = 8;

__device__ __forceinline__ void reduce_bins(const ReduceParams& P) {
    typedef unsigned __int128 u128;
    __shared__ uint64_t part[kRedLanes][kRedBins][2];
    const ReduceGroup G = P.groups[blockIdx.y];
    const uint32_t bl = threadIdx.x % kRedBins, ul = threadIdx.x / kRedBins;
    const uint32_t i = blockIdx.x * kRedBins + bl;
    if (blockIdx.x * kRedBins >= G.slice_bins) return;
    u128 acc = 0;
    if (i < G.slice_bins && G.unit_end > G.unit_begin) {
        const uint64_t stride = 2ull * G.slice_bins;
        const uint64_t* s = P.partial + P.units[G.unit_begin].slot + 2ull * i;
        const uint32_t n = G.unit_end - G.unit_begin;
        uint32_t u = ul;
        for (; u + (kRedAhead - 1) * kRedLanes < n; u += kRedAhead * kRedLanes) {
            ulonglong2 v[kRedAhead];
#pragma unroll
            for (int k = 0; k < kRedAhead; ++k)
                v[k] = *reinterpret_cast<const ulonglong2*>(s + (u + k * kRedLanes) * stride);
#pragma unroll
            for (int k = 0; k < kRedAhead; ++k) acc += static_cast<u128>(v[k].x) + (static_cast<u128>(v[k].y) << 32);
        }
        for (; u < n; u += kRedLanes) {
            const ulonglong2 v = *reinterpret_cast<const ulonglong2*>(s + u * stride);
            acc += static_cast<u128>(v.x) + (static_cast<u128>(v.y) << 32);
        }
    }
    part[ul][bl][0] = static_cast<uint64_t>(acc);
    part[ul][bl][1] = static_cast<uint64_t>(acc >> 64);
    __syncthreads();
    if (ul != 0 || i >= G.slice_bins) return;
    u128 tot = 0;
    for (int l = 0; l < kRedLanes; ++l)
        tot += (static_cast<u128>(part[l][bl][1]) << 64) | part[l][bl][0];
    const uint64_t lo = static_cast<uint64_t>(tot), hi = static_cast<uint64_t>(tot >> 64);
    const uint64_t o = G.out_off + i;
    P.raw[2 * o] = lo;
    P.raw[2 * o + 1] = hi;
    const uint32_t sb = i % G.n_space_bins;
    const uint32_t tb = i / G.n_space_bins;
    const double r = u128_to_double(lo, hi) * 0x1p-56;
    double d = static_cast<double>(G.n_hist) * P.dx[G.dx_off + sb];
    if (G.n_time_bins > 0) d = d * P.dt[G.dt_off + tb];
    P.flux[o] = (d != 0.0) ? r / d : 0.0;
}

// The words of a problem's units, each thread's units first, then across the
// wave by exchanges, then across the waves in LDS.
__device__ __forceinline__ void reduce_diag(const ReduceParams& P, uint32_t pb) {
    __shared__ unsigned long long acc[4][kNDiag];
    const uint32_t u0 = P.pu_begin[pb], u1 = P.pu_begin[pb + 1];
    unsigned long long loc[kNDiag];
#pragma unroll
    for (int k = 0; k < kNDiag; ++k) loc[k] = 0;
    for (uint32_t u = u0 + threadIdx.x; u < u1; u += 256) {
#pragma unroll
        for (int k = 0; k < kNDiag; ++k) {
            const unsigned long long v = P.unit_diag[static_cast<size_t>(u) * kNDiag + k];
            if (k == D_MAX_DRAWS)
                loc[k] = v > loc[k] ? v : loc[k];
            else
                loc[k] += v;
        }
    }
#pragma unroll
    for (int m = 32; m != 0; m >>= 1)
#pragma unroll
        for (int k = 0; k < kNDiag; ++k) {
            const unsigned long long v = __shfl_xor(loc[k], m);
            loc[k] = k == D_MAX_DRAWS ? (v > loc[k] ? v : loc[k]) : loc[k] + v;
        }
    if ((threadIdx.x & 63u) == 0)
#pragma unroll
        for (int k = 0; k < kNDiag; ++k) acc[threadIdx.x >> 6][k] = loc[k];
    __syncthreads();
    if (threadIdx.x < kNDiag) {
        unsigned long long v = acc[0][threadIdx.x];
        for (int w = 1; w < 4; ++w) {
            const unsigned long long o = acc[w][threadIdx.x];
            v = threadIdx.x == D_MAX_DRAWS ? (o > v ? o : v) : v + o;
        }
        P.diag[static_cast<size_t>(pb) * kNDiag + threadIdx.x] = v;
    }
}

__global__ void __launch_bounds__(256) k_reduce(ReduceParams P) {
    if (blockIdx.y < P.n_groups)
        reduce_bins(P);
    else if (blockIdx.x == 0)
        reduce_diag(P, blockIdx.y - P.n_groups);
}

__global__ void __launch_bounds__(256) k_reduce_diag(ReduceParams P) { reduce_diag(P, blockIdx.x); }

hipError_t launch_reduce(const ReduceParams& p, hipStream_t st) {
    uint32_t bx = (p.max_slice + kRedBins - 1) / kRedBins;
    if (bx < 1) bx = 1;
    const uint32_t nd = p.diag != nullptr ? p.n_problems : 0;
    // (a grid's second extent is at most 65535)
    const bool one = static_cast<uint64_t>(p.n_groups) + nd <= 65535;
    const uint32_t rows = p.n_groups + (one ? nd : 0);
    if (rows > 0) {
        hipLaunchKernelGGL(k_reduce, dim3(bx, rows), dim3(256), 0, st, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (!one) {
        hipLaunchKernelGGL(k_reduce_diag, dim3(nd), dim3(256), 0, st, p);
        return hipGetLastError();
    }
    return hipSuccess;
}

}  // namespace mcrng
