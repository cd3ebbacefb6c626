// Small device/host helpers shared by libbsr's kernels.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>

#include "bsr_internal.h"

namespace bsr {

inline hipStream_t as_stream(void *s) { return reinterpret_cast<hipStream_t>(s); }

// Status of the launch just enqueued (records the HIP error text on failure).
inline bsr_status launch_status() {
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) return BSR_OK;
    set_last_hip_error(hipGetErrorString(e));
    return BSR_ERR_HIP;
}

// Launch `kernel`, through hipExtLaunchKernel when an event pair is given so that the events
// mark the kernel's own start and end on the device.
template <typename... Params, typename... Args>
inline void launch_kernel(void (*kernel)(Params...), dim3 grid, dim3 block, size_t lds,
                          hipStream_t st, const LaunchEvents &ev, Args... args) {
    if (ev.start != nullptr || ev.stop != nullptr)
        hipExtLaunchKernelGGL(kernel, grid, block, static_cast<uint32_t>(lds), st,
                              static_cast<hipEvent_t>(ev.start),
                              static_cast<hipEvent_t>(ev.stop), 0u, static_cast<Params>(args)...);
    else
        hipLaunchKernelGGL(kernel, grid, block, static_cast<uint32_t>(lds), st,
                           static_cast<Params>(args)...);
}

__device__ __forceinline__ int64_t clamp64(int64_t v, int64_t lo, int64_t hi) {
    return v < lo ? lo : (v > hi ? hi : v);
}

__device__ __forceinline__ int clampi(int v, int lo, int hi) {
    return v < lo ? lo : (v > hi ? hi : v);
}

// A value the compiler may treat as uniform across the wave (lane 0's copy).
__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

// Raw buffer resource over [base, base + bytes): loads past the end return 0 and stores past
// it are dropped.  The check covers the vector, instruction and scalar offsets together, word by
// word, also where the scalar offset alone is past the end (MI355X, a range inside a larger
// allocation, 16-byte loads and 4-byte stores at scalar offsets from 0 to 64 times the range).  Word
// 3 is the default raw-buffer configuration for gfx9-family chips.  The launch plans keep every range
// below 2^31 bytes.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_rsrc(const void *base, unsigned bytes) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), 0, int(bytes), 0x00020000);
}

// A slice's units are shared out over the 16 waves by weights that depend on a wave's place
// among the four waves of its SIMD (wave w runs on SIMD w % 4, after waves w - 4, w - 8, ...).
// The SIMDs' instruction arbitration favours older waves: with equal shares the first wave of
// every SIMD finished its stream about 30% before the last (per-wave timestamps on MI355X, the
// BERT-large 32x1 stack), and the item waits for the last.  Weights 48:38:31:27 made that
// launch 2% faster than equal shares (same box, A/B).  Start of wave l's units (l = 16: the end
// of the range).
constexpr unsigned kShareWeight[4] = {48, 38, 31, 27};
constexpr unsigned kShareTotal = 4 * (kShareWeight[0] + kShareWeight[1] + kShareWeight[2] +
                                      kShareWeight[3]);
__device__ __forceinline__ int wave_start(int64_t Q0, unsigned span, unsigned l) {
    const unsigned a = l >> 2, b = l & 3;
    unsigned cum = 0;
#pragma unroll
    for (unsigned i = 0; i < 4; ++i) cum += i < a ? 4 * kShareWeight[i] : 0u;
#pragma unroll
    for (unsigned i = 0; i < 4; ++i) cum += i == a ? b * kShareWeight[i] : 0u;
    return int(Q0) + int(uint64_t(span) * cum / kShareTotal);
}

// Inclusive prefix sum over the 64 lanes of a wave: row shifts by 1, 2, 4 and 8 lanes sum each
// row of 16 lanes, then the last lane of row 0 is added to row 1 and of row 2 to row 3, and
// the last lane of row 1 (now rows 0 and 1) to rows 2 and 3.  Lanes a shift reads from
// outside their row contribute 0.
__device__ __forceinline__ int wave_scan_incl(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);   // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);   // row_bcast:31
    return v;
}

// bf16 bit pattern -> fp32 value (exact widening).
__device__ __forceinline__ float bf16_bits_to_float(unsigned short h) {
    return __uint_as_float(static_cast<unsigned int>(h) << 16);
}

// Grid size for a grid-stride loop over `n` items with `threads` per block.
inline unsigned grid_for(int64_t n, int threads, int64_t cap = int64_t(1) << 20) {
    int64_t g = (n + threads - 1) / threads;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return static_cast<unsigned>(g);
}

}  // namespace bsr
