// Uniform random numbers of many streams, for gfx950.
//
// k_uniforms: stream i (grid-stride) starts at its seed (stride skip-ahead
// or hash seed, or a state loaded from HBM), takes k LCG steps (eq. 1) and
// writes the uniform of its j-th output to u[(j - 1) n + i].  The layout is
// draw-major, so a wave's 64 stores of one draw are one contiguous 512-byte
// run; the stores are non-temporal (the output is not read back by the
// kernel).  The kernel is bound by HBM writes: 8 bytes per number against
// about a dozen VALU operations.
#include "internal.hpp"
#include "uniforms.hpp"

namespace mcrng {

// NT: non-temporal stores.
template <int MODE, bool NT>
__global__ void __launch_bounds__(256) k_uniforms(LcgDev L, SeedDev S, uint64_t n, uint32_t k, uint64_t* state,
                                                  double* u) {
    const uint64_t stride = static_cast<uint64_t>(gridDim.x) * 256;
    const uint64_t b0 = static_cast<uint64_t>(blockIdx.x) * 256;
    // stride seeding: stream b0 + t + j stride starts at A_{Q t} of the
    // block's base, which moves on by A_{Q stride} (one affine step each)
    uint64_t lg = 1, lc = 0, jg = 1, jc = 0, base = 0;
    if (MODE == SEED_STRIDE && b0 < n) {
        const uint64_t* a = S.table + 2 * (threadIdx.x & (kStrideRadix - 1));
        const uint64_t* b = S.table + 2 * (kStrideRadix + (threadIdx.x >> kStrideRadixBits));
        lg = a[0] * b[0];
        lc = a[0] * b[1] + a[1];
        for (uint32_t d = 0; d < kStrideDigits && (stride >> (kStrideRadixBits * d)) != 0; ++d) {
            const uint32_t v = static_cast<uint32_t>(stride >> (kStrideRadixBits * d)) & (kStrideRadix - 1);
            const uint64_t* e = S.table + 2 * (d * kStrideRadix + v);
            jc = e[0] * jc + e[1];
            jg = e[0] * jg;
        }
        base = stream_start(L, S, b0);
    }
    for (uint64_t i = b0 + threadIdx.x; i < n; i += stride) {
        uint64_t x;   // the state, top-aligned while it is stepped
        if (MODE == SEED_LOAD) {
            x = state[i];
        } else if (MODE == SEED_STRIDE) {
            x = affine_apply(lg, lc, L.mask, base);
            base = affine_apply(jg, jc, L.mask, base);
        } else {
            x = stream_start(L, S, i);
        }
        x <<= L.up;
        double* out = u + i;
        for (uint32_t j = 0; j < k; ++j) {
            x = lcg_next_z(L, x);
            if (NT)
                __builtin_nontemporal_store(uniform_z(x), out);
            else
                *out = uniform_z(x);
            out += n;
        }
        if (state) state[i] = x >> L.up;
    }
}

// The same for rows that do not start on 128-byte lines (n not a multiple of 16,
// more than one row).  A wave's 64 numbers of a row then begin and end inside
// lines, which the non-temporal stores send to HBM in parts: 4194301 streams x 16
// took 193 us where 4194304 take 118.  Here a block takes runs of 1024 streams,
// passes each row of a run through LDS and stores it from line to line, so that
// only a run's first and last line are split (137 us).
constexpr uint32_t kRunStreams = 1024, kRunPer = kRunStreams / 256;

template <int MODE>
__global__ void __launch_bounds__(256) k_uniforms_runs(LcgDev L, SeedDev S, uint64_t n, uint32_t k, uint64_t* state,
                                                       double* u) {
    __shared__ double row[2][kRunStreams];
    const uint32_t tid = threadIdx.x;
    uint64_t lg = 1, lc = 0;
    if (MODE == SEED_STRIDE) {
        const uint64_t* a = S.table + 2 * (tid & (kStrideRadix - 1));
        const uint64_t* b = S.table + 2 * (kStrideRadix + (tid >> kStrideRadixBits));
        lg = a[0] * b[0];
        lc = a[0] * b[1] + a[1];
    }
    for (uint64_t b0 = static_cast<uint64_t>(blockIdx.x) * kRunStreams; b0 < n;
         b0 += static_cast<uint64_t>(gridDim.x) * kRunStreams) {
        uint64_t x[kRunPer];   // the states, top-aligned while they are stepped
        uint64_t base = MODE == SEED_STRIDE ? stream_start(L, S, b0) : 0ull;
#pragma unroll
        for (uint32_t q = 0; q < kRunPer; ++q) {
            const uint64_t i = b0 + q * 256u + tid;
            if (MODE == SEED_LOAD) {
                x[q] = i < n ? state[i] : 0ull;
            } else if (MODE == SEED_STRIDE) {
                x[q] = affine_apply(lg, lc, L.mask, base);
                const uint64_t* e = S.table + 2 * (2 * kStrideRadix + 1);   // A_{256 Q}
                base = affine_apply(e[0], e[1], L.mask, base);
            } else {
                x[q] = stream_start(L, S, i);
            }
            x[q] <<= L.up;
        }
        const uint32_t cnt = n - b0 < kRunStreams ? static_cast<uint32_t>(n - b0) : kRunStreams;
        for (uint32_t j = 0; j < k; ++j) {
            double* const r = row[j & 1u];   // (two rows: the next is filled while this one is stored)
#pragma unroll
            for (uint32_t q = 0; q < kRunPer; ++q) {
                x[q] = lcg_next_z(L, x[q]);
                r[q * 256u + tid] = uniform_z(x[q]);
            }
            __syncthreads();
            const uint64_t first = j * n + b0;
            const uint32_t skew = static_cast<uint32_t>((reinterpret_cast<uintptr_t>(u + first) >> 3) & 15u);
            double* const out = u + first;
#pragma unroll
            for (uint32_t q = 0; q <= kRunPer; ++q) {
                const uint32_t i = q * 256u + tid - skew;   // wraps below the run's start
                if (i < cnt) __builtin_nontemporal_store(r[i], out + i);
            }
        }
        if (state)
#pragma unroll
            for (uint32_t q = 0; q < kRunPer; ++q) {
                const uint64_t i = b0 + q * 256u + tid;
                if (i < n) state[i] = x[q] >> L.up;
            }
        __syncthreads();   // the next run fills row 0 again
    }
}

hipError_t launch_uniforms(const LcgDev& L, const SeedDev& S, int mode, uint64_t n, uint32_t k, uint64_t* state,
                           double* u, hipStream_t st) {
    if (n == 0 || k == 0) return hipSuccess;
    int dev = 0, cus = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (e != hipSuccess) return e;
    // Rows that start inside lines: up to about what the last-level cache holds,
    // ordinary stores (split lines meet there: 2000003 x 16, 256 MB, 57 us
    // against 92 non-temporal and 73 by runs; 8388607 x 4, 268 MB, 83, 89 and
    // 87); beyond, line by line in runs (4194301 x 16, 537 MB: 146, ordinary
    // 171, non-temporal 193; 30000001 x 3, 720 MB: 212, 294, 234).
    const bool split = k > 1 && n % 16 != 0;
    const bool big = static_cast<double>(n) * k * 8.0 > 384e6;
    if (split && big && n >= 64ull * kRunStreams) {
        uint64_t runs = (n + kRunStreams - 1) / kRunStreams;
        if (runs > (1u << 20)) runs = 1u << 20;
        const dim3 g(static_cast<unsigned>(runs)), b(256);
        switch (mode) {
            case SEED_LOAD: hipLaunchKernelGGL(k_uniforms_runs<SEED_LOAD>, g, b, 0, st, L, S, n, k, state, u); break;
            case SEED_HASH: hipLaunchKernelGGL(k_uniforms_runs<SEED_HASH>, g, b, 0, st, L, S, n, k, state, u); break;
            default: hipLaunchKernelGGL(k_uniforms_runs<SEED_STRIDE>, g, b, 0, st, L, S, n, k, state, u); break;
        }
        return hipGetLastError();
    }
    // many short-lived blocks: 256 per CU wrote 5.3 TB/s, 16 per CU 4.6 TB/s
    uint64_t blocks = (n + 255) / 256;
    const uint64_t cap = static_cast<uint64_t>(cus > 0 ? cus : 256) * 256;
    if (blocks > cap) blocks = cap;
    const dim3 grid(static_cast<unsigned>(blocks)), block(256);
    const bool nt = !split || big;
    switch (mode) {
        case SEED_LOAD:
            if (nt) hipLaunchKernelGGL((k_uniforms<SEED_LOAD, true>), grid, block, 0, st, L, S, n, k, state, u);
            else hipLaunchKernelGGL((k_uniforms<SEED_LOAD, false>), grid, block, 0, st, L, S, n, k, state, u);
            break;
        case SEED_HASH:
            if (nt) hipLaunchKernelGGL((k_uniforms<SEED_HASH, true>), grid, block, 0, st, L, S, n, k, state, u);
            else hipLaunchKernelGGL((k_uniforms<SEED_HASH, false>), grid, block, 0, st, L, S, n, k, state, u);
            break;
        default:
            if (nt) hipLaunchKernelGGL((k_uniforms<SEED_STRIDE, true>), grid, block, 0, st, L, S, n, k, state, u);
            else hipLaunchKernelGGL((k_uniforms<SEED_STRIDE, false>), grid, block, 0, st, L, S, n, k, state, u);
            break;
    }
    return hipGetLastError();
}

}  // namespace mcrng
