// Key of a block for pruning (prune.hip), in plain C++ so that it also runs where no GPU exists.
#pragma once

#include <cstdint>

#ifdef __HIP__
#define BSR_HOST_DEVICE __host__ __device__
#else
#define BSR_HOST_DEVICE
#endif

namespace bsr {

constexpr unsigned long long kNaNKey = 0x7FF8000000000000ull;

// The fp64 l1 or squared l2 norm of a block as a bit pattern.  The elements are visited in the
// sequential order of the definition, sixteen loads issued before the sixteen dependent fp64
// operations that use them: with one load per operation a 32 x 32 block waited 1024 times for
// memory.  A block may have 2^32 elements and more, so the batches are counted in 64 bits (counted
// down: a comparison with zero is one scalar instruction).
template <bool kL1>
BSR_HOST_DEVICE inline unsigned long long block_key(const float *__restrict__ base, int64_t ldw,
                                                    int32_t R, int32_t C) {
    constexpr unsigned kAhead = 16;
    const uint64_t n = uint64_t(R) * uint64_t(C);
    double s = 0.0;
    const float *row = base;
    int c = 0;
    auto next = [&]() -> float {
        const float x = row[c];
        if (++c == C) {
            c = 0;
            row += ldw;
        }
        return x;
    };
    auto add = [&](float v) {
        const double x = static_cast<double>(v);
        if constexpr (kL1) s += __builtin_fabs(x);
        else s = __builtin_fma(x, x, s);
    };
    for (uint64_t batch = n / kAhead; batch != 0; --batch) {
        float v[kAhead];
#pragma unroll
        for (unsigned q = 0; q < kAhead; ++q) v[q] = next();
#pragma unroll
        for (unsigned q = 0; q < kAhead; ++q) add(v[q]);
    }
    for (unsigned e = unsigned(n % kAhead); e != 0; --e) add(next());
    return s != s ? kNaNKey : __builtin_bit_cast(unsigned long long, s);
}

}  // namespace bsr
