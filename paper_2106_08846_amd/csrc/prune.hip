// Block-magnitude pruning on the GPU: dense fp32 W -> BSR keeping the top-k blocks.
//
// Sec. 2.1, Eq. 3 partitions W into blocks scored by a per-block norm (l2, or l1: the p = 1 case
// of Eq. 1 and Eq. 2); Eq. 2 bounds the number of nonzero groups, whose projection keeps the k
// blocks of largest norm (globally, or k / Nb in every block-row); Sec. 2.2 stores the result
// as SciPy-style data / indices / indptr.
//
// On the caller's stream:
//   1. Keys: fp64, summed sequentially (row r outer, column c inner).  Each fp32 square and each
//      |x| is exact in fp64, so fma(x, x, s) and s + |x| round exactly like the CPU's sequential
//      loop: the key is bit-identical.
//   2. Selection: the k-th largest key tau (keys are >= +0.0, so bit order is value order; NaN is
//      canonicalised above +inf) and the last id kept among the keys equal to it, then every
//      kept block's place in id order.  One workgroup (prune_select_kernel) up to 32768 blocks,
//      five launches over the whole chip (prune_*_kernel from prune_keys_range_kernel on) above.
//      Integer atomics count histogram bins and candidates are ordered by (key, id), so the
//      result is deterministic.
//      Per-row selection (prune_select_rows_kernel) runs a radix select and an id-order sweep
//      inside each block-row, one workgroup per row; indptr is then i * k_row.
//   3. prune_copy_kernel: one thread per output element copies the kept blocks' bits (the chip-
//      wide selection copies them where it places them).
#include <mutex>

#include "device_common.h"
#include "prune_key.h"

namespace bsr {

namespace {

// The workspace of bsr_prune_from_dense_noalloc: a fixed device array, one copy per GPU.  In
// host code its name is only a stand-in for the symbol; the device address of each GPU's copy
// comes from hipGetSymbolAddress, looked up once per device with that device current.
__device__ __align__(256) unsigned char scratch[kNoallocScratchBytes];

constexpr int kScratchDevices = 64;
void *g_scratch_ptr[kScratchDevices] = {};
std::mutex g_scratch_mutex;

constexpr int kKeyThreads = 256;
constexpr int kSelThreads = 1024;
constexpr int kSelWaves = kSelThreads / 64;

// Blocks' keys, one thread per block.
template <bool kL1>
__global__ __launch_bounds__(kKeyThreads) void prune_keys_kernel(
    const float *__restrict__ W, int64_t ldw, int32_t R, int32_t C, int64_t Kb, int64_t nb,
    unsigned long long *__restrict__ keybits) {
    const int64_t b = int64_t(blockIdx.x) * kKeyThreads + threadIdx.x;
    if (b >= nb) return;
    const int64_t i = b / Kb, j = b - i * Kb;
    keybits[b] = block_key<kL1>(W + (i * R) * ldw + j * C, ldw, R, C);
}

// The keys of blocks that are wide and few: a workgroup copies G consecutive blocks to LDS with
// coalesced loads, then G lanes walk one block each in the sequential order.  A thread per block
// read its rows through loads 4 C bytes apart, at most nine waves of them on a 768 x 768 weight in
// 32 x 32 blocks, and waited on memory (111 us there).  Blocks are kPitch = R C + 1 words
// apart, so the walking lanes stay on different banks.
constexpr int kStageWords = 6144;
constexpr int kStageBlocks = 32;
constexpr int kStageMinWords = 32;   // smaller blocks, and one-column ones, take a thread each

template <bool kL1>
__global__ __launch_bounds__(kKeyThreads) void prune_keys_staged_kernel(
    const float *__restrict__ W, int64_t ldw, int32_t R, int32_t C, unsigned Kb, unsigned nb,
    int G, unsigned long long *__restrict__ keybits) {
    extern __shared__ float s_blk[];
    const unsigned tid = threadIdx.x, RC = unsigned(R) * unsigned(C), pitch = RC + 1;
    const unsigned b0 = blockIdx.x * unsigned(G);
    const unsigned g = min(unsigned(G), nb - b0), words = g * RC;
    constexpr int kAhead = 8;
    for (unsigned e0 = tid; e0 < words; e0 += kKeyThreads * kAhead) {
        float v[kAhead];
        unsigned at[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            // Word e: row r of the blocks, block p, column c -- a row's blocks side by side.
            const unsigned e = e0 + q * kKeyThreads;
            const unsigned ec = e < words ? e : 0u;
            const unsigned r = ec / (g * unsigned(C)), rest = ec - r * (g * unsigned(C));
            const unsigned p = rest / unsigned(C), c = rest - p * unsigned(C);
            const unsigned b = b0 + p, i = b / Kb, j = b - i * Kb;
            at[q] = p * pitch + r * unsigned(C) + c;
            v[q] = W[(int64_t(i) * R + r) * ldw + int64_t(j) * C + c];
        }
#pragma unroll
        for (int q = 0; q < kAhead; ++q)
            if (e0 + q * kKeyThreads < words) s_blk[at[q]] = v[q];
    }
    __syncthreads();
    if (tid < g)
        keybits[b0 + tid] = block_key<kL1>(s_blk + tid * pitch, C, R, C);
}

// Exclusive prefix count of `pred` over the workgroup of NWAVES waves (thread order) and its
// total.
template <int NWAVES = kSelWaves>
__device__ __forceinline__ void wg_scan(bool pred, unsigned &excl, unsigned &total,
                                        unsigned *wave_tot) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long m = __ballot(pred);
    const unsigned long long below = lane ? (m & ((1ull << lane) - 1ull)) : 0ull;
    const unsigned in_wave = static_cast<unsigned>(__popcll(below));
    if (lane == 0) wave_tot[wave] = static_cast<unsigned>(__popcll(m));
    __syncthreads();
    unsigned before = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) {
        const unsigned c = wave_tot[w];
        before += (w < wave) ? c : 0u;
        tot += c;
    }
    __syncthreads();
    excl = before + in_wave;
    total = tot;
}

// One radix step of the selection, by the first wave, lane l holding the counts c of bins
// 4 l .. 4 l + 3 (the bins of this digit of the keys that match the prefix so far): the digit
// of the key with rank `remaining` (1-based, descending), i.e. the largest v whose bins
// v .. 255 hold at least `remaining` keys.  Suffix sums over the lanes give each bin's count
// of keys at or above it.  Writes the extended prefix and the rank within bin v.
__device__ __forceinline__ void pick_digit_counts(const unsigned (&c)[4], long long remaining,
                                                  unsigned long long prefix, int shift,
                                                  unsigned long long *s_prefix,
                                                  long long *s_remaining) {
    const int lane = threadIdx.x & 63;
    const unsigned t = c[0] + c[1] + c[2] + c[3];
    unsigned sfx = t;   // keys in the bins of lanes >= lane
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned y = __shfl_down(sfx, d);
        sfx += lane + d < 64 ? y : 0u;
    }
    long long at[4];    // keys in bins >= 4 lane + q
    at[3] = static_cast<long long>(sfx - t) + c[3];
    at[2] = at[3] + c[2];
    at[1] = at[2] + c[1];
    at[0] = at[1] + c[0];
    const int qb = at[3] >= remaining ? 3 : at[2] >= remaining ? 2
                 : at[1] >= remaining ? 1 : at[0] >= remaining ? 0 : -1;
    const unsigned long long m = __ballot(qb >= 0);
    if (m == 0ull) {   // fewer keys than the rank (not reached for 1 <= k <= nb)
        if (lane == 0) {
            *s_prefix = prefix;
            *s_remaining = remaining - static_cast<long long>(sfx);
        }
        return;
    }
    const int L = 63 - __clzll(static_cast<long long>(m));
    if (lane == L) {
        const int digit = 4 * lane + qb;
        *s_prefix = prefix | (static_cast<unsigned long long>(digit) << shift);
        *s_remaining = remaining - (at[qb] - static_cast<long long>(c[qb]));
    }
}

__device__ __forceinline__ void pick_digit(const unsigned *hist, long long remaining,
                                           unsigned long long prefix, int shift,
                                           unsigned long long *s_prefix,
                                           long long *s_remaining) {
    const int lane = threadIdx.x & 63;
    unsigned c[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) c[q] = hist[4 * lane + q];
    pick_digit_counts(c, remaining, prefix, shift, s_prefix, s_remaining);
}

// ------------------------------------------------------------------ global selection, helpers
// The k-th largest key tau, and the last id kept among the keys equal to tau, are found by range
// histograms: kBins equal bins over a range of key bit patterns, the bin that holds the wanted
// rank, then the same inside that bin, until at most kRankMax keys are left, which are ranked
// directly by (key descending, id ascending), or the range is a single value.
constexpr int kBins = 4096;      // four bins per thread of a 1024-thread workgroup
constexpr int kRankMax = 64;     // keys ranked directly, each against all the others

// Right shift that puts the offsets 0 .. range into kBins bins.
__device__ __forceinline__ int bin_shift(unsigned long long range) {
    const int bits = 64 - __clzll(static_cast<long long>(range | 1ull));
    return bits > 12 ? bits - 12 : 0;
}

struct Picked {
    int bin;
    unsigned count;   // keys in the bin
    long long rank;   // the wanted rank within the bin (1-based, descending)
};

// The bin of the key with rank `remaining` (1-based, descending) of a histogram held four bins
// per thread (c: bins 4 tid .. 4 tid + 3), by all threads of a kSelThreads workgroup.
__device__ __forceinline__ Picked pick_bin(const unsigned (&c)[4], long long remaining,
                                           unsigned *wave_tot, Picked *s_picked) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned t = c[0] + c[1] + c[2] + c[3];
    unsigned sfx = t;   // keys in the bins of this wave's lanes >= lane
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned y = __shfl_down(sfx, d);
        sfx += lane + d < 64 ? y : 0u;
    }
    if (lane == 0) wave_tot[wave] = sfx;
    __syncthreads();
    long long above = static_cast<long long>(sfx - t);   // keys in bins above this thread's
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) above += w > wave ? wave_tot[w] : 0u;
    if (above < remaining && remaining <= above + static_cast<long long>(t)) {
#pragma unroll
        for (int q = 3; q >= 0; --q) {
            if (remaining > above && remaining <= above + static_cast<long long>(c[q]))
                *s_picked = Picked{4 * tid + q, c[q], remaining - above};
            above += c[q];
        }
    }
    __syncthreads();
    return *s_picked;
}

// Smallest and largest of every thread's (kmin, kmax), in every thread.
__device__ __forceinline__ void wg_min_max(unsigned long long &kmin, unsigned long long &kmax,
                                           unsigned long long *s_min, unsigned long long *s_max) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const unsigned long long x = __shfl_xor(kmin, d), y = __shfl_xor(kmax, d);
        kmin = x < kmin ? x : kmin;
        kmax = y > kmax ? y : kmax;
    }
    if (lane == 0) {
        s_min[wave] = kmin;
        s_max[wave] = kmax;
    }
    __syncthreads();
#pragma unroll
    for (int w = 0; w < kSelWaves; ++w) {
        kmin = s_min[w] < kmin ? s_min[w] : kmin;
        kmax = s_max[w] > kmax ? s_max[w] : kmax;
    }
    __syncthreads();
}

// tau and the last kept id among n <= kRankMax candidates in LDS: the candidate that `rank` - 1
// others precede in the order (key descending, id ascending).
__device__ __forceinline__ void rank_candidates(const unsigned long long *ck, const int *cid,
                                                int n, long long rank, unsigned long long *s_tau,
                                                int *s_last) {
    for (int i = threadIdx.x; i < n; i += kSelThreads) {
        const unsigned long long u = ck[i];
        const int id = cid[i];
        int before = 0;
        for (int j = 0; j < n; ++j)
            before += (ck[j] > u || (ck[j] == u && cid[j] < id)) ? 1 : 0;
        if (before == int(rank) - 1) {
            *s_tau = u;
            *s_last = id;
        }
    }
}

__device__ __forceinline__ bool is_kept(unsigned long long u, int id, unsigned long long tau,
                                        int last_eq) {
    return u > tau || (u == tau && id <= last_eq);
}

// --------------------------------------------------------------- nb <= kSelThreads * kRegKeys
// One workgroup holding a 32-bit code of every key in LDS (e.g. a 1024 x 1024 weight in 32 x 1
// blocks: 32768 keys, 128 KB): thread t holds ids t + kSelThreads e, e < kRegKeys ("round" e).
//   * The code is the 32 bits of the key under the highest bit in which the keys differ (counted
//     from the smallest high word), so it orders the keys up to equal codes, and every step over
//     the keys costs a few full-rate 32-bit instructions.
//   * Selection: range histograms from [smallest code, largest code].  The keys of one matrix lie
//     within a few octaves, so 4096 bins over their own range leave a few tens of candidates
//     after one pass; radix passes over the key's bytes took six or seven.  When more than
//     kRankMax keys share the wanted code, the passes go on over the 64-bit keys, in memory.
//   * Placement: per round and wave, the count of kept keys goes to a table of
//     kRegKeys x kSelWaves entries whose exclusive prefix, in (round, wave) order, is id order; a
//     key's position is its table entry plus the kept lanes below it in its wave.
// What bounds it is one CU: its share of memory bandwidth for the keys, its LDS atomics and its
// barriers.  32768 keys: 25 us, against 34 us for byte-wise radix passes over 64-bit keys in
// registers (MI355X); with the codes in registers the fully unrolled steps spilled about 180
// scalar masks and took 32 us.
constexpr int kRegKeys = 32;
constexpr int kTab = kRegKeys * kSelWaves;   // 512

// Exclusive prefix, in place, of tab[kTab] by the first wave (8 entries per lane).
__device__ __forceinline__ void tab_excl_scan(unsigned *tab) {
    const int lane = threadIdx.x & 63;
    unsigned v[8], t = 0;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        v[q] = tab[8 * lane + q];
        t += v[q];
    }
    unsigned incl = t;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned y = __shfl_up(incl, d);
        incl += lane >= d ? y : 0u;
    }
    unsigned run = incl - t;
#pragma unroll
    for (int q = 0; q < 8; ++q) {
        tab[8 * lane + q] = run;
        run += v[q];
    }
}

__global__ __launch_bounds__(kSelThreads) void prune_select_kernel(
    const unsigned long long *__restrict__ keybits, int64_t nb, int64_t Kb, int64_t Nb,
    int64_t k, int32_t *__restrict__ indptr, int32_t *__restrict__ indices,
    int32_t *__restrict__ src) {
    extern __shared__ unsigned s_code[];   // [rounds * kSelThreads]
    __shared__ __align__(16) unsigned hist[kBins];
    __shared__ unsigned tab[kTab];
    __shared__ unsigned s_min[kSelWaves], s_max[kSelWaves];
    __shared__ unsigned wave_tot[kSelWaves];
    __shared__ unsigned long long ck[kRankMax];
    __shared__ int cid[kRankMax];
    __shared__ Picked s_picked;
    __shared__ unsigned long long s_tau;
    __shared__ int s_last, s_n;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;

    if (k <= 0) {
        for (int64_t i = tid; i <= Nb; i += kSelThreads) indptr[i] = 0;
        return;
    }
    // Rounds, in whole batches of kBatch (the loops below take a batch's LDS reads at a time).
    constexpr int kBatch = 8;
    static_assert(kRegKeys % kBatch == 0, "whole batches");
    const int n = int(nb);
    const int rounds = (n + kSelThreads * kBatch - 1) / (kSelThreads * kBatch) * kBatch;
    const __amdgpu_buffer_rsrc_t rk = buffer_rsrc(keybits, unsigned(n) * 8u);
    auto load_key = [&](int e) -> unsigned long long {   // key e of this thread (0 past nb)
        const auto w = __builtin_amdgcn_raw_buffer_load_b64(rk, tid * 8 + kSelThreads * 8 * e, 0, 0);
        return (static_cast<unsigned long long>(w[1]) << 32) | w[0];
    };
    auto clear_hist = [&]() {
        *reinterpret_cast<uint4 *>(&hist[4 * tid]) = make_uint4(0u, 0u, 0u, 0u);
    };
    int shift;         // low key bits under the code
    unsigned hmin = ~0u;
    {
        // All loads are issued before any is used: range-checked buffer loads (ids past nb read
        // 0 and touch no memory) need no branch per key.
        unsigned klo[kRegKeys], khi[kRegKeys];
#pragma unroll
        for (int e = 0; e < kRegKeys; ++e) {
            const unsigned long long u = load_key(e);
            klo[e] = unsigned(u);
            khi[e] = unsigned(u >> 32);
        }
        clear_hist();
        if (tid == 0) s_n = 0;
        unsigned hmax = 0u;
#pragma unroll
        for (int e = 0; e < kRegKeys; ++e) {
            hmin = min(hmin, tid + kSelThreads * e < n ? khi[e] : ~0u);
            hmax = max(hmax, khi[e]);   // past nb: 0
        }
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) {
            hmin = min(hmin, __shfl_xor(hmin, d));
            hmax = max(hmax, __shfl_xor(hmax, d));
        }
        if (lane == 0) {
            s_min[wave] = hmin;
            s_max[wave] = hmax;
        }
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w) {
            hmin = min(hmin, s_min[w]);
            hmax = max(hmax, s_max[w]);
        }
        shift = hmax == hmin ? 0 : 32 - __clz(int(hmax - hmin));
#pragma unroll
        for (int e = 0; e < kRegKeys; ++e) {
            const unsigned long long d =
                (static_cast<unsigned long long>(khi[e] - hmin) << 32) | klo[e];
            if (e < rounds) s_code[tid + kSelThreads * e] = unsigned(d >> shift);
        }
    }
    // From here on a thread reads only the codes it wrote.

    long long remaining = k;
    unsigned cand = unsigned(n);   // keys with codes in [lo, hi]
    unsigned lo = 0, hi = ~0u;
    bool clear = true;             // hist holds zeros
    while (cand > unsigned(kRankMax) && lo < hi) {
        const unsigned range = hi - lo;
        const int sh = range >= unsigned(kBins) ? 20 - __clz(int(range)) : 0;
        if (!clear) {
            clear_hist();
            __syncthreads();
        }
        clear = false;
        for (int e0 = 0; e0 < rounds; e0 += kBatch) {
#pragma unroll
            for (int q = 0; q < kBatch; ++q) {
                const int id = tid + kSelThreads * (e0 + q);
                const unsigned d = s_code[id] - lo;
                if (d <= range && id < n) atomicAdd(&hist[d >> sh], 1u);
            }
        }
        __syncthreads();
        const uint4 h4 = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
        const unsigned c[4] = {h4.x, h4.y, h4.z, h4.w};
        const Picked p = pick_bin(c, remaining, wave_tot, &s_picked);
        lo += unsigned(p.bin) << sh;
        const unsigned top = lo + ((1u << sh) - 1u);
        hi = top < hi ? top : hi;
        remaining = p.rank;
        cand = p.count;
        __syncthreads();   // hist and s_picked are free again
    }
    const unsigned code_lo = lo, range = hi - lo;
    // The candidates' keys: those with codes in [code_lo, code_lo + range], in [klo, khi] once
    // the codes do not tell them apart.
    unsigned long long klo = 0ull, khi = ~0ull;
    if (cand > unsigned(kRankMax) && shift > 0) {
        klo = (static_cast<unsigned long long>(hmin) << 32) +
              (static_cast<unsigned long long>(code_lo) << shift);
        khi = klo + ((1ull << shift) - 1ull);
        while (cand > unsigned(kRankMax) && klo < khi) {
            const int sh = bin_shift(khi - klo);
            clear_hist();
            __syncthreads();
            for (int e = 0; e < rounds; ++e) {
                const unsigned long long u = load_key(e);
                if (tid + kSelThreads * e < n && u >= klo && u <= khi)
                    atomicAdd(&hist[(u - klo) >> sh], 1u);
            }
            __syncthreads();
            const uint4 h4 = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
            const unsigned c[4] = {h4.x, h4.y, h4.z, h4.w};
            const Picked p = pick_bin(c, remaining, wave_tot, &s_picked);
            klo += static_cast<unsigned long long>(p.bin) << sh;
            const unsigned long long top = klo + ((1ull << sh) - 1ull);
            khi = top < khi ? top : khi;
            remaining = p.rank;
            cand = p.count;
            __syncthreads();
        }
    }
    if (cand <= unsigned(kRankMax)) {
#pragma unroll kBatch
        for (int e = 0; e < rounds; ++e) {
            const int id = tid + kSelThreads * e;
            if (s_code[id] - code_lo <= range && id < n) {
                const unsigned long long u = load_key(e);
                if (u >= klo && u <= khi) {
                    const int at = atomicAdd(&s_n, 1);
                    ck[at] = u;
                    cid[at] = id;
                }
            }
        }
        __syncthreads();
        rank_candidates(ck, cid, int(cand), remaining, &s_tau, &s_last);
    } else {
        // More than kRankMax equal keys: the last kept one by their ranks in id order.
        const unsigned long long tie =
            shift > 0 ? klo : (static_cast<unsigned long long>(hmin) << 32) + code_lo;
        for (int e = 0; e < rounds; ++e) {
            const unsigned long long b =
                __ballot(tid + kSelThreads * e < n && load_key(e) == tie);
            if (lane == 0) tab[e * kSelWaves + wave] = unsigned(__popcll(b));
        }
        for (int i = rounds * kSelWaves + tid; i < kTab; i += kSelThreads) tab[i] = 0;
        __syncthreads();
        if (wave == 0) tab_excl_scan(tab);
        __syncthreads();
        for (int e = 0; e < rounds; ++e) {
            const int id = tid + kSelThreads * e;
            const bool eq = id < n && load_key(e) == tie;
            const unsigned long long b = __ballot(eq);
            const long long before = static_cast<long long>(tab[e * kSelWaves + wave]) +
                                     __popcll(b & ((1ull << lane) - 1ull));
            if (eq && before == remaining - 1) {
                s_tau = tie;
                s_last = id;
            }
        }
    }
    __syncthreads();
    const unsigned long long tau = s_tau;
    const int last_eq = s_last;

    const unsigned long long below = (1ull << lane) - 1ull;   // lanes under this one
    unsigned keepm = 0;   // bit e: key e is kept
    for (int e0 = 0; e0 < rounds; e0 += kBatch) {
        unsigned code[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) code[q] = s_code[tid + kSelThreads * (e0 + q)];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            const int e = e0 + q, id = tid + kSelThreads * e;
            bool keep = id < n && code[q] > code_lo;
            if (id < n && code[q] - code_lo <= range) keep = is_kept(load_key(e), id, tau, last_eq);
            keepm |= keep ? 1u << e : 0u;
            const unsigned long long b = __ballot(keep);
            if (lane == 0) tab[e * kSelWaves + wave] = unsigned(__popcll(b));
        }
    }
    for (int i = rounds * kSelWaves + tid; i < kTab; i += kSelThreads) tab[i] = 0;
    __syncthreads();
    if (wave == 0) tab_excl_scan(tab);
    __syncthreads();
    // Row and column of the thread's ids: one division, then steps of kSelThreads ids.
    const unsigned kb = unsigned(Kb);
    const unsigned di = unsigned(kSelThreads) / kb, dj = unsigned(kSelThreads) - di * kb;
    unsigned i = unsigned(tid) / kb, j = unsigned(tid) - i * kb;
    for (int e0 = 0; e0 < rounds; e0 += kBatch) {
        unsigned first[kBatch];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) first[q] = tab[(e0 + q) * kSelWaves + wave];
#pragma unroll
        for (int q = 0; q < kBatch; ++q) {
            const int e = e0 + q, id = tid + kSelThreads * e;
            const bool keep = (keepm >> e) & 1u;
            const unsigned long long b = __ballot(keep);
            const int pos = int(first[q]) + __popcll(b & below);
            if (id < n && j == 0) indptr[i] = pos;
            if (keep) {
                indices[pos] = int32_t(j);
                src[pos] = int32_t(id);
            }
            i += di;
            j += dj;
            if (j >= kb) {
                j -= kb;
                ++i;
            }
        }
    }
    if (tid == 0) indptr[Nb] = static_cast<int32_t>(k);
}

// Dynamic LDS of prune_select_kernel: the codes, in whole batches of eight rounds.
size_t select_lds_bytes(int64_t nb) {
    constexpr int64_t kPer = int64_t(kSelThreads) * 8;
    return size_t((nb + kPer - 1) / kPer * kPer) * 4;
}

// ---------------------------------------------------------------- nb > kSelThreads * kRegKeys
// The selection spread over the chip, in five launches (one workgroup streaming every key nine
// times took 10.2 ms on a 3072 x 768 weight in 1 x 1 blocks):
//   1. prune_keys_range_kernel: the keys, each workgroup's smallest and largest finite key, and
//      the clearing of the histogram;
//   2. prune_hist_kernel: a histogram of the keys over a window around the k-th key.  Every
//      workgroup takes the same window from the same sample of kSamples keys: the values whose
//      ranks in the sample lie four standard deviations on either side of the wanted rank.  About
//      4% of the keys fall into it (at a density of 0.1), so few bins of a workgroup are non-zero
//      and few global atomics add them up; the keys above it are counted per workgroup;
//   3. prune_collect_kernel: the bin of the k-th key; per chunk of ids, the number of keys above
//      that bin and the bin's keys and ids, listed in the chunk's own segment;
//   4. prune_finish_kernel: one workgroup resolves the listed keys to tau and the last kept id
//      among its equals, and turns the chunks' kept counts into their first positions;
//   5. prune_place_kernel: every chunk writes its part of indptr, indices and data.
// On that weight the five take 12, 25, 15, 11 and 13 us (the whole call 10.25 ms -> 76 us); with
// the list appended through one global counter and the last workgroup of step 3 doing step 4,
// step 3 alone took 340 us (its atomics and release fences).  Chunks of 4096 ids (576 workgroups
// where 256 run at once), 1024 ids per pass of step 5 and the k-th key's bin searched again in
// step 4 cost 20, 18 and 15 us (88 us).  At 36864 blocks (768 x 768 in 4 x 4) the call went from
// 131 to 34 us; below the one-workgroup limit (32768 blocks, 33 us) the five launches would cost
// more than they save.
// A k-th key outside the window (the sample misled), or a bin with more keys than a segment
// holds, is resolved from all keys by the one workgroup of step 4 (a bin of equal keys needs
// only one chunk's).  Ordering between the steps is the stream's: no workgroup waits for another.
// The arrays between them live in the workspace's source-id array, which this path has no
// other use for.
constexpr int kSamples = 4 * kSelThreads;
constexpr int kMaxRanges = 1024;          // workgroups of the key kernel
constexpr int kMaxHists = 256;            // workgroups of the histogram kernel
constexpr int kMinChunkShift = 11;        // ids per chunk (log2), raised until
constexpr int kWantChunks = 512;          // kWantChunks suffice: about one round of workgroups
constexpr unsigned long long kInfKey = 0x7FF0000000000000ull;

// The histogram's window: kBins bins of 2^shift bit patterns from lo on; hi is its last value.
struct Window {
    unsigned long long lo, hi;
    int shift;
};

// The range of key values that holds the k-th key, the keys in it and the wanted rank among
// them: a bin of the window, or everything above or below the window.
struct Target {
    unsigned long long lo, hi;
    long long count, rank;
};

struct SelectCtrl {
    Window win;
    Target target;
    unsigned long long tau;
    int32_t last_eq;
};

// What a chunk of ids holds: keys above the picked bin (after the finish kernel: the chunk's
// first position), keys in the bin, and their smallest and largest.
struct Chunk {
    unsigned above, in_bin;
    unsigned long long kmin, kmax;
};

// The workspace's source-id array (4 nb bytes) as the selection's arrays.
struct SelectArrays {
    SelectCtrl *ctrl;
    unsigned long long *range;   // [2 * kMaxRanges]: smallest and largest finite key per workgroup
    unsigned *hist;              // [kBins]
    unsigned *above;             // [kMaxHists]: keys above the window, per workgroup
    Chunk *chunk;                // [kWantChunks] at most
    unsigned long long *list_key;
    int32_t *list_id;
    unsigned cap;                // list entries per chunk
    unsigned chunks;
    int chunk_shift;
};

constexpr int64_t kSelectFixed = 256 + int64_t(kMaxRanges) * 16 + int64_t(kBins) * 4 +
                                 int64_t(kMaxHists) * 4;
constexpr int kSelectAlign = 16;   // a caller's workspace may start at any address
static_assert(sizeof(SelectCtrl) <= 256 && sizeof(Chunk) == 24 && kSelectFixed % 16 == 0);

SelectArrays select_arrays(void *src, int64_t nb) {
    char *p = reinterpret_cast<char *>((reinterpret_cast<uintptr_t>(src) + kSelectAlign - 1) &
                                       ~uintptr_t(kSelectAlign - 1));
    SelectArrays a;
    a.chunk_shift = kMinChunkShift;
    while (((nb - 1) >> a.chunk_shift) + 1 > kWantChunks) ++a.chunk_shift;
    a.chunks = unsigned(((nb - 1) >> a.chunk_shift) + 1);
    a.ctrl = reinterpret_cast<SelectCtrl *>(p);
    a.range = reinterpret_cast<unsigned long long *>(p + 256);
    a.hist = reinterpret_cast<unsigned *>(p + 256 + kMaxRanges * 16);
    a.above = a.hist + kBins;
    a.chunk = reinterpret_cast<Chunk *>(p + kSelectFixed);
    const int64_t fixed = kSelectAlign + kSelectFixed + int64_t(a.chunks) * int64_t(sizeof(Chunk));
    const int64_t cap = (nb * 4 - fixed) / 12 / a.chunks;   // > 400 (nb > 32768)
    const int64_t ids = int64_t(1) << a.chunk_shift;
    a.cap = unsigned(cap < ids ? cap : ids);
    a.list_key = reinterpret_cast<unsigned long long *>(a.chunk + a.chunks);
    a.list_id = reinterpret_cast<int32_t *>(a.list_key + int64_t(a.cap) * a.chunks);
    return a;
}

template <bool kL1>
__global__ __launch_bounds__(kKeyThreads) void prune_keys_range_kernel(
    const float *__restrict__ W, int64_t ldw, int32_t R, int32_t C, unsigned Kb, unsigned nb,
    unsigned long long *__restrict__ keybits, SelectArrays A) {
    __shared__ unsigned long long s_min[kKeyThreads / 64], s_max[kKeyThreads / 64];
    const unsigned tid = threadIdx.x, g = blockIdx.x;
    for (unsigned i = g * kKeyThreads + tid; i < unsigned(kBins); i += gridDim.x * kKeyThreads)
        A.hist[i] = 0;
    unsigned long long kmin = ~0ull, kmax = 0ull;
    for (uint64_t b = uint64_t(g) * kKeyThreads + tid; b < nb;
         b += uint64_t(gridDim.x) * kKeyThreads) {
        const unsigned i = unsigned(b) / Kb, j = unsigned(b) - i * Kb;
        const unsigned long long u =
            block_key<kL1>(W + (int64_t(i) * R) * ldw + int64_t(j) * C, ldw, R, C);
        keybits[b] = u;
        if (u < kInfKey) {
            kmin = u < kmin ? u : kmin;
            kmax = u > kmax ? u : kmax;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const unsigned long long x = __shfl_xor(kmin, d), y = __shfl_xor(kmax, d);
        kmin = x < kmin ? x : kmin;
        kmax = y > kmax ? y : kmax;
    }
    if ((tid & 63) == 0) {
        s_min[tid >> 6] = kmin;
        s_max[tid >> 6] = kmax;
    }
    __syncthreads();
    if (tid == 0) {
        for (int w = 1; w < kKeyThreads / 64; ++w) {
            kmin = s_min[w] < kmin ? s_min[w] : kmin;
            kmax = s_max[w] > kmax ? s_max[w] : kmax;
        }
        A.range[2 * g] = kmin;
        A.range[2 * g + 1] = kmax;
    }
}

// The window: from the sample's range histogram over [smallest, largest finite key], the bins of
// the ranks four standard deviations above and below the wanted rank's place in the sample.
__device__ __forceinline__ Window sample_window(const unsigned long long *__restrict__ keybits,
                                                unsigned nb, long long k,
                                                const unsigned long long *range, int ranges,
                                                unsigned *hist, unsigned *wave_tot,
                                                unsigned long long *s_min,
                                                unsigned long long *s_max, Picked *s_picked) {
    const int tid = threadIdx.x;
    unsigned long long u[kSamples / kSelThreads];
#pragma unroll
    for (int s = 0; s < kSamples / kSelThreads; ++s) {
        // Spread over all ids without a period that a weight's rows could share (multiples of
        // the golden ratio, modulo 2^32, scaled to nb).
        const unsigned h = unsigned(tid + s * kSelThreads) * 2654435769u;
        u[s] = keybits[(uint64_t(h) * nb) >> 32];
    }
    unsigned long long kmin = ~0ull, kmax = 0ull;
    for (int i = tid; i < ranges; i += kSelThreads) {
        const unsigned long long a = range[2 * i], b = range[2 * i + 1];
        kmin = a < kmin ? a : kmin;
        kmax = b > kmax ? b : kmax;
    }
    *reinterpret_cast<uint4 *>(&hist[4 * tid]) = make_uint4(0u, 0u, 0u, 0u);
    wg_min_max(kmin, kmax, s_min, s_max);   // ends with a barrier
    if (kmin > kmax) kmin = kmax = 0ull;    // no finite key
    const int shift = bin_shift(kmax - kmin);
#pragma unroll
    for (int s = 0; s < kSamples / kSelThreads; ++s) {
        const unsigned long long v = u[s] < kmax ? u[s] : kmax;   // infinities and NaN: the top
        atomicAdd(&hist[(v - kmin) >> shift], 1u);
    }
    __syncthreads();
    const uint4 h4 = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
    const unsigned c[4] = {h4.x, h4.y, h4.z, h4.w};
    const float p = float(k) / float(nb);
    const int margin = int(4.0f * sqrtf(float(kSamples) * p * (1.0f - p))) + 4;
    const int at = int(float(kSamples) * p);
    const int r_hi = at - margin, r_lo = at + margin;   // ranks count from the largest key
    Window w;
    w.lo = 0ull;
    w.hi = ~0ull;
    if (r_hi >= 1) {
        const int b = pick_bin(c, r_hi, wave_tot, s_picked).bin;
        __syncthreads();
        const unsigned long long top =
            kmin + ((static_cast<unsigned long long>(b) + 1ull) << shift) - 1ull;
        w.hi = top;
    }
    if (r_lo <= kSamples) {
        const int b = pick_bin(c, r_lo, wave_tot, s_picked).bin;
        __syncthreads();
        w.lo = kmin + (static_cast<unsigned long long>(b) << shift);
    }
    // An open end stops at the finite keys' range, so that the bins stay fine.
    if (w.lo < kmin) w.lo = kmin;
    if (w.hi > kmax) w.hi = kmax > w.lo ? kmax : w.lo;
    w.shift = bin_shift(w.hi - w.lo);
    return w;
}

__global__ __launch_bounds__(kSelThreads) void prune_hist_kernel(
    const unsigned long long *__restrict__ keybits, unsigned nb, long long k, int ranges,
    SelectArrays A) {
    __shared__ __align__(16) unsigned hist[kBins];
    __shared__ unsigned long long s_min[kSelWaves], s_max[kSelWaves];
    __shared__ unsigned wave_tot[kSelWaves];
    __shared__ Picked s_picked;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const Window w = sample_window(keybits, nb, k, A.range, ranges, hist, wave_tot, s_min, s_max,
                                   &s_picked);
    if (blockIdx.x == 0 && tid == 0) A.ctrl->win = w;
    *reinterpret_cast<uint4 *>(&hist[4 * tid]) = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const uint64_t stride = uint64_t(gridDim.x) * kSelThreads;
    constexpr int kAhead = 8;
    unsigned above = 0;
    for (uint64_t b = uint64_t(blockIdx.x) * kSelThreads + tid; b < nb; b += stride * kAhead) {
        unsigned long long u[kAhead];
#pragma unroll
        for (int q = 0; q < kAhead; ++q) u[q] = b + stride * q < nb ? keybits[b + stride * q] : 0ull;
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const bool valid = b + stride * q < nb;
            above += valid && u[q] > w.hi ? 1u : 0u;
            if (valid && u[q] >= w.lo && u[q] <= w.hi) atomicAdd(&hist[(u[q] - w.lo) >> w.shift], 1u);
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) above += __shfl_xor(above, d);
    if (lane == 0) wave_tot[wave] = above;
    __syncthreads();
    if (tid == 0) {
        unsigned t = 0;
        for (int i = 0; i < kSelWaves; ++i) t += wave_tot[i];
        A.above[blockIdx.x] = t;
    }
    const uint4 h4 = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
    const unsigned c[4] = {h4.x, h4.y, h4.z, h4.w};
#pragma unroll
    for (int q = 0; q < 4; ++q)
        if (c[q]) atomicAdd(&A.hist[4 * tid + q], c[q]);
}

__device__ __forceinline__ Target find_target(unsigned nb, long long k, int hists,
                                              const SelectArrays &A, unsigned *wave_tot,
                                              Picked *s_picked) {
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const Window w = A.ctrl->win;
    const uint4 h4 = *reinterpret_cast<const uint4 *>(&A.hist[4 * tid]);
    const unsigned c[4] = {h4.x, h4.y, h4.z, h4.w};
    unsigned a = tid < hists ? A.above[tid] : 0u, inside = c[0] + c[1] + c[2] + c[3];
    static_assert(kMaxHists <= kSelThreads, "one count per thread");
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        a += __shfl_xor(a, d);
        inside += __shfl_xor(inside, d);
    }
    if (lane == 0) wave_tot[wave] = a;
    __syncthreads();
    long long above = 0, in = 0;
    for (int i = 0; i < kSelWaves; ++i) above += wave_tot[i];
    __syncthreads();
    if (lane == 0) wave_tot[wave] = inside;
    __syncthreads();
    for (int i = 0; i < kSelWaves; ++i) in += wave_tot[i];
    __syncthreads();
    if (k <= above) return Target{w.hi + 1ull, ~0ull, above, k};
    if (k > above + in)
        return Target{0ull, w.lo - 1ull, static_cast<long long>(nb) - above - in, k - above - in};
    const Picked p = pick_bin(c, k - above, wave_tot, s_picked);
    __syncthreads();
    Target t;
    t.lo = w.lo + (static_cast<unsigned long long>(p.bin) << w.shift);
    t.hi = t.lo + ((1ull << w.shift) - 1ull);
    t.hi = t.hi < w.hi ? t.hi : w.hi;
    t.count = p.count;
    t.rank = p.rank;
    return t;
}

// Two workgroups per CU: 64 registers.
__global__ __launch_bounds__(kSelThreads) void prune_collect_kernel(
    const unsigned long long *__restrict__ keybits, unsigned nb, long long k, int hists,
    SelectArrays A) {
    __shared__ unsigned wave_tot[kSelWaves];
    __shared__ unsigned long long s_min[kSelWaves], s_max[kSelWaves];
    __shared__ Picked s_picked;
    __shared__ unsigned s_n;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int64_t b0 = int64_t(blockIdx.x) << A.chunk_shift;
    const int64_t bmax = b0 + (int64_t(1) << A.chunk_shift);
    const int64_t b1 = bmax < int64_t(nb) ? bmax : int64_t(nb);
    constexpr int kAhead = 2;
    unsigned long long u[kAhead];
    auto load = [&](int64_t base) {
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int64_t b = base + q * kSelThreads + tid;
            u[q] = b < b1 ? keybits[b] : 0ull;
        }
    };
    load(b0);   // under the target's reductions
    if (tid == 0) s_n = 0;
    const Target t = find_target(nb, k, hists, A, wave_tot, &s_picked);   // ends with a barrier
    if (blockIdx.x == 0 && tid == 0) A.ctrl->target = t;

    unsigned above = 0;
    unsigned long long kmin = ~0ull, kmax = 0ull;
    const int64_t seg = int64_t(blockIdx.x) * A.cap;
    for (int64_t base = b0; base < b1; base += kSelThreads * kAhead) {
        if (base != b0) load(base);
#pragma unroll
        for (int q = 0; q < kAhead; ++q) {
            const int64_t b = base + q * kSelThreads + tid;
            if (b < b1 && u[q] >= t.lo) {
                if (u[q] > t.hi) {
                    ++above;
                } else {
                    kmin = u[q] < kmin ? u[q] : kmin;
                    kmax = u[q] > kmax ? u[q] : kmax;
                    const unsigned at = atomicAdd(&s_n, 1u);
                    if (at < A.cap) {
                        A.list_key[seg + at] = u[q];
                        A.list_id[seg + at] = int32_t(b);
                    }
                }
            }
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) above += __shfl_xor(above, d);
    if (lane == 0) wave_tot[wave] = above;
    wg_min_max(kmin, kmax, s_min, s_max);   // two barriers
    if (tid == 0) {
        unsigned s = 0;
        for (int i = 0; i < kSelWaves; ++i) s += wave_tot[i];
        A.chunk[blockIdx.x] = Chunk{s, s_n, kmin, kmax};
    }
}

__global__ __launch_bounds__(kSelThreads) void prune_finish_kernel(
    const unsigned long long *__restrict__ keybits, unsigned nb, SelectArrays A) {
    constexpr int kList = 4096;   // candidates held in LDS; more are read from the segments
    __shared__ __align__(16) unsigned hist[kBins];
    __shared__ unsigned long long s_list[kList];
    __shared__ int s_list_id[kList];
    __shared__ unsigned long long s_min[kSelWaves], s_max[kSelWaves];
    __shared__ unsigned wave_tot[kSelWaves];
    __shared__ unsigned long long ck[kRankMax];
    __shared__ int cid[kRankMax];
    __shared__ Picked s_picked;
    __shared__ unsigned long long s_tau;
    __shared__ int s_last_eq, s_n, s_chunk;
    __shared__ long long s_run;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int chunks = int(A.chunks);
    static_assert(kWantChunks <= 2 * kSelThreads, "at most two chunks per thread");
    Chunk mine[2];
#pragma unroll
    for (int q = 0; q < 2; ++q)
        mine[q] = 2 * tid + q < chunks ? A.chunk[2 * tid + q] : Chunk{0u, 0u, ~0ull, 0ull};
    const Target t = A.ctrl->target;

    unsigned long long lo = mine[0].kmin < mine[1].kmin ? mine[0].kmin : mine[1].kmin;
    unsigned long long hi = mine[0].kmax > mine[1].kmax ? mine[0].kmax : mine[1].kmax;
    wg_min_max(lo, hi, s_min, s_max);   // the candidates' own range
    const unsigned most = mine[0].in_bin > mine[1].in_bin ? mine[0].in_bin : mine[1].in_bin;
    const bool listed = __syncthreads_and(most <= A.cap);

    // Exclusive prefix over the chunks (two per thread) of a count; every thread gets the place
    // of its first chunk.
    auto chunk_prefix = [&](unsigned a0, unsigned a1) -> unsigned {
        unsigned incl = a0 + a1;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const unsigned y = __shfl_up(incl, d);
            incl += lane >= d ? y : 0u;
        }
        __syncthreads();
        if (lane == 63) wave_tot[wave] = incl;
        __syncthreads();
        unsigned first = incl - (a0 + a1);
#pragma unroll
        for (int i = 0; i < kSelWaves; ++i) first += i < wave ? wave_tot[i] : 0u;
        return first;
    };

    long long remaining = t.rank;
    if (tid == 0) s_n = 0;
    const unsigned first_in = chunk_prefix(mine[0].in_bin, mine[1].in_bin);
    if (lo == hi) {
        // Equal keys only (ties, zero blocks): the chunk of the last kept one by the chunks'
        // counts, then its place in the chunk.
        unsigned at = first_in;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            if (static_cast<long long>(at) < remaining &&
                remaining <= static_cast<long long>(at) + mine[q].in_bin) {
                s_chunk = 2 * tid + q;
                s_run = at;
            }
            at += mine[q].in_bin;
        }
        __syncthreads();
        const int64_t b0 = int64_t(s_chunk) << A.chunk_shift;
        const int64_t bmax = b0 + (int64_t(1) << A.chunk_shift);
        const int64_t b1 = bmax < int64_t(nb) ? bmax : int64_t(nb);
        long long run = s_run;
        for (int64_t base = b0; base < b1; base += kSelThreads) {
            const int64_t b = base + tid;
            const bool eq = b < b1 && keybits[b] == lo;
            unsigned ex, tot;
            wg_scan(eq, ex, tot, wave_tot);
            if (eq && run + static_cast<long long>(ex) == remaining - 1) {
                s_tau = lo;
                s_last_eq = int(b);
            }
            run += tot;
        }
        __syncthreads();
        // Kept keys per chunk: the equal ones up to that place.
        const int last_chunk = s_chunk;
        unsigned kept[2];
        at = first_in;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int c = 2 * tid + q;
            kept[q] = mine[q].above + (c < last_chunk ? mine[q].in_bin
                                       : c == last_chunk ? unsigned(remaining - at) : 0u);
            at += mine[q].in_bin;
        }
        const unsigned first = chunk_prefix(kept[0], kept[1]);
        if (2 * tid < chunks) A.chunk[2 * tid].above = first;
        if (2 * tid + 1 < chunks) A.chunk[2 * tid + 1].above = first + kept[0];
        if (tid == 0) {
            A.ctrl->tau = s_tau;
            A.ctrl->last_eq = s_last_eq;
        }
        return;
    }

    // Candidates: in LDS when they fit, else all keys (of which those in [lo, hi] count).
    const bool in_lds = listed && t.count <= kList;
    if (in_lds) {
        unsigned at = first_in;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int64_t seg = int64_t(2 * tid + q) * A.cap;
            for (unsigned i = 0; i < mine[q].in_bin; ++i, ++at) {
                s_list[at] = A.list_key[seg + i];
                s_list_id[at] = A.list_id[seg + i];
            }
        }
    }
    __syncthreads();
    const unsigned n = in_lds ? unsigned(t.count) : nb;
    auto each = [&](auto &&f) {   // f(key, id) of every key in [lo, hi]
        if (in_lds) {
            for (unsigned i = tid; i < n; i += kSelThreads) {
                const unsigned long long u = s_list[i];
                if (u >= lo && u <= hi) f(u, s_list_id[i]);
            }
        } else {
            constexpr int kAhead = 8;
            for (uint64_t b = tid; b < n; b += uint64_t(kSelThreads) * kAhead) {
                unsigned long long u[kAhead];
#pragma unroll
                for (int q = 0; q < kAhead; ++q) {
                    const uint64_t i = b + uint64_t(q) * kSelThreads;
                    u[q] = i < n ? keybits[i] : ~0ull;   // ~0: above every key
                }
#pragma unroll
                for (int q = 0; q < kAhead; ++q)
                    if (u[q] >= lo && u[q] <= hi) f(u[q], int(b + uint64_t(q) * kSelThreads));
            }
        }
    };
    const unsigned long long bin_lo = lo, bin_hi = hi;
    long long cand = t.count;
    while (cand > kRankMax && lo < hi) {
        const int shift = bin_shift(hi - lo);
        *reinterpret_cast<uint4 *>(&hist[4 * tid]) = make_uint4(0u, 0u, 0u, 0u);
        __syncthreads();
        each([&](unsigned long long u, int) { atomicAdd(&hist[(u - lo) >> shift], 1u); });
        __syncthreads();
        const uint4 h4 = *reinterpret_cast<const uint4 *>(&hist[4 * tid]);
        const unsigned c[4] = {h4.x, h4.y, h4.z, h4.w};
        const Picked r = pick_bin(c, remaining, wave_tot, &s_picked);
        const unsigned long long base = lo + (static_cast<unsigned long long>(r.bin) << shift);
        const unsigned long long top = base + ((1ull << shift) - 1ull);
        hi = top < hi ? top : hi;
        lo = base;
        remaining = r.rank;
        cand = r.count;
        __syncthreads();
    }
    if (cand <= kRankMax) {
        each([&](unsigned long long u, int id) {
            const int at = atomicAdd(&s_n, 1);
            ck[at] = u;
            cid[at] = id;
        });
        __syncthreads();
        rank_candidates(ck, cid, int(cand), remaining, &s_tau, &s_last_eq);
    } else {
        // More than kRankMax keys equal to lo: walk all keys in id order to the last kept one.
        long long run = 0;
        for (uint64_t base = 0; base < nb && run < remaining; base += kSelThreads) {
            const uint64_t b = base + tid;
            const bool eq = b < nb && keybits[b] == lo;
            unsigned ex, tot;
            wg_scan(eq, ex, tot, wave_tot);
            if (eq && run + static_cast<long long>(ex) == remaining - 1) {
                s_tau = lo;
                s_last_eq = int(b);
            }
            run += tot;
        }
    }
    __syncthreads();
    const unsigned long long tau = s_tau;
    const int last_eq = s_last_eq;

    // Kept keys per chunk (those above the bin, plus the bin's kept ones), then their prefix.
    unsigned *cnt = hist;
    cnt[2 * tid] = mine[0].above;
    cnt[2 * tid + 1] = mine[1].above;
    __syncthreads();
    lo = bin_lo;
    hi = bin_hi;
    each([&](unsigned long long u, int id) {
        if (is_kept(u, id, tau, last_eq)) atomicAdd(&cnt[unsigned(id) >> A.chunk_shift], 1u);
    });
    __syncthreads();
    const unsigned a0 = cnt[2 * tid], a1 = cnt[2 * tid + 1];
    const unsigned first = chunk_prefix(a0, a1);
    if (2 * tid < chunks) A.chunk[2 * tid].above = first;
    if (2 * tid + 1 < chunks) A.chunk[2 * tid + 1].above = first + a0;
    if (tid == 0) {
        A.ctrl->tau = tau;
        A.ctrl->last_eq = last_eq;
    }
}

// One chunk of ids: the kept ones' columns, row starts and data, kPlaceIds ids at a time (four per
// thread, so that two barriers place 4096 ids).
constexpr int kPlacePer = 4;
constexpr int kPlaceIds = kPlacePer * kSelThreads;

__global__ __launch_bounds__(kSelThreads) void prune_place_kernel(
    const float *__restrict__ W, int64_t ldw, int32_t R, int32_t C, unsigned Kb, unsigned nb,
    long long k, unsigned Nb, const unsigned long long *__restrict__ keybits, SelectArrays A,
    int32_t *__restrict__ indptr, int32_t *__restrict__ indices, float *__restrict__ data) {
    __shared__ unsigned s_cnt[kPlacePer * kSelWaves];   // kept ids per (part, wave), in id order
    __shared__ unsigned s_id[kPlaceIds];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned long long tau = A.ctrl->tau;
    const int last_eq = A.ctrl->last_eq;
    const int64_t b0 = int64_t(blockIdx.x) << A.chunk_shift;
    const int64_t bmax = b0 + (int64_t(1) << A.chunk_shift);
    const int64_t b1 = bmax < int64_t(nb) ? bmax : int64_t(nb);
    const unsigned *Wu = reinterpret_cast<const unsigned *>(W);
    unsigned *Du = reinterpret_cast<unsigned *>(data);
    const unsigned RC = unsigned(R) * unsigned(C);
    int64_t pos0 = A.chunk[blockIdx.x].above;
    unsigned long long u[kPlacePer];
    auto load = [&](int64_t base) {
#pragma unroll
        for (int q = 0; q < kPlacePer; ++q) {
            const int64_t b = base + q * kSelThreads + tid;
            u[q] = b < b1 ? keybits[b] : 0ull;
        }
    };
    load(b0);
    for (int64_t base = b0; base < b1; base += kPlaceIds) {
        bool keep[kPlacePer];
        unsigned below[kPlacePer];
#pragma unroll
        for (int q = 0; q < kPlacePer; ++q) {
            const int64_t b = base + q * kSelThreads + tid;
            keep[q] = b < b1 && is_kept(u[q], int(b), tau, last_eq);
            const unsigned long long m = __ballot(keep[q]);
            below[q] = unsigned(__popcll(m & ((1ull << lane) - 1ull)));
            if (lane == 0) s_cnt[q * kSelWaves + wave] = unsigned(__popcll(m));
        }
        load(base + kPlaceIds);   // the next ids, under the placement
        __syncthreads();
        // Kept ids before each of this wave's parts, and in all: one entry per lane.
        static_assert(kPlacePer * kSelWaves == 64, "one count per lane");
        const unsigned mine = s_cnt[lane];
        const unsigned incl = unsigned(wave_scan_incl(int(mine)));
        const unsigned tot = unsigned(__builtin_amdgcn_readlane(int(incl), 63));
#pragma unroll
        for (int q = 0; q < kPlacePer; ++q) {
            const int64_t b = base + q * kSelThreads + tid;
            const unsigned ex =
                unsigned(__builtin_amdgcn_readlane(int(incl - mine), q * kSelWaves + uniform(wave))) +
                below[q];
            if (b < b1) {
                const unsigned id = unsigned(b), i = id / Kb, j = id - i * Kb;
                if (j == 0) indptr[i] = int32_t(pos0 + ex);
                if (keep[q]) {
                    indices[pos0 + ex] = int32_t(j);
                    if (RC == 1) Du[pos0 + ex] = Wu[int64_t(i) * ldw + j];
                    else s_id[ex] = id;
                }
            }
        }
        __syncthreads();   // s_cnt is read; the kept ids are in s_id
        if (RC > 1) {
            const uint64_t total = uint64_t(tot) * RC;
            auto copy = [&](auto index) {   // 32-bit divisions where the element count allows
                using I = decltype(index);
                for (I e = I(tid); e < I(total); e += kSelThreads) {
                    const unsigned p = unsigned(e / RC), rc = unsigned(e - I(p) * RC);
                    const unsigned r = rc / unsigned(C), c = rc - r * unsigned(C);
                    const unsigned id = s_id[p], i = id / Kb, j = id - i * Kb;
                    Du[pos0 * RC + e] = Wu[(int64_t(i) * R + r) * ldw + int64_t(j) * C + c];
                }
            };
            if (total < (uint64_t(1) << 31)) copy(0u);
            else copy(uint64_t(0));
            __syncthreads();   // s_id is free again
        }
        pos0 += tot;
    }
    if (blockIdx.x == 0 && tid == 0) indptr[Nb] = static_cast<int32_t>(k);
}

constexpr int kRowThreads = 256;
constexpr int kRowWaves = kRowThreads / 64;

// Per-row selection: workgroup i keeps the k_row blocks of block-row i that come first in the
// order (key descending, column ascending).  A radix select over the row's keys, eight bits a pass
// from the top, gives the k_row-th largest key and how many of its equals are kept; a sweep over the
// columns then counts equals and kept blocks and writes the kept ones in place.  Every row keeps k_row
// blocks, so indptr[i] is i * k_row and the kept blocks of row i occupy positions i * k_row ..
// (i + 1) * k_row - 1.
__global__ __launch_bounds__(kRowThreads) void prune_select_rows_kernel(
    const unsigned long long *__restrict__ keybits, int64_t Kb, int64_t Nb, int64_t k_row,
    int32_t *__restrict__ indptr, int32_t *__restrict__ indices, int32_t *__restrict__ src) {
    __shared__ unsigned hist[256];
    __shared__ unsigned wave_tot[kRowWaves];
    __shared__ unsigned long long s_prefix;
    __shared__ long long s_remaining;
    const int tid = threadIdx.x;
    const int64_t i = blockIdx.x;
    if (tid == 0) {
        indptr[i] = static_cast<int32_t>(i * k_row);
        if (i == Nb - 1) indptr[Nb] = static_cast<int32_t>(Nb * k_row);
    }
    if (k_row <= 0) return;   // uniform: a kernel argument
    const unsigned long long *key = keybits + i * Kb;

    unsigned long long prefix = 0, pmask = 0;
    long long remaining = k_row;
    for (int pass = 0; pass < 8; ++pass) {
        const int shift = 56 - 8 * pass;
        hist[tid] = 0;   // kRowThreads == 256 bins
        __syncthreads();
        for (int64_t b = tid; b < Kb; b += kRowThreads) {
            const unsigned long long u = key[b];
            if ((u & pmask) == prefix) atomicAdd(&hist[(u >> shift) & 255ull], 1u);
        }
        __syncthreads();
        if (tid < 64) pick_digit(hist, remaining, prefix, shift, &s_prefix, &s_remaining);
        __syncthreads();
        prefix = s_prefix;
        remaining = s_remaining;
        pmask |= 0xFFull << shift;
        __syncthreads();
    }
    const unsigned long long tau = prefix;
    const long long need_eq = remaining;

    long long run_eq = 0, run_keep = 0;
    for (int64_t base = 0; base < Kb; base += kRowThreads) {
        const int64_t j = base + tid;
        const bool valid = j < Kb;
        const unsigned long long u = valid ? key[j] : 0ull;
        const bool gt = valid && u > tau;
        const bool eq = valid && u == tau;
        unsigned eq_ex, eq_tot;
        wg_scan<kRowWaves>(eq, eq_ex, eq_tot, wave_tot);
        const bool keep = gt || (eq && (run_eq + static_cast<long long>(eq_ex)) < need_eq);
        unsigned keep_ex, keep_tot;
        wg_scan<kRowWaves>(keep, keep_ex, keep_tot, wave_tot);
        const long long pos = i * k_row + run_keep + static_cast<long long>(keep_ex);
        if (keep) {
            indices[pos] = static_cast<int32_t>(j);
            src[pos] = static_cast<int32_t>(i * Kb + j);
        }
        run_eq += eq_tot;
        run_keep += keep_tot;
    }
}

__global__ __launch_bounds__(256) void prune_copy_kernel(
    const float *__restrict__ W, int64_t ldw, int32_t R, int32_t C, int64_t Kb, int64_t nb,
    int64_t k, const int32_t *__restrict__ src, float *__restrict__ data) {
    const int64_t RC = int64_t(R) * C;
    const int64_t total = k * RC;
    const unsigned *Wu = reinterpret_cast<const unsigned *>(W);
    unsigned *Du = reinterpret_cast<unsigned *>(data);
    for (int64_t e = int64_t(blockIdx.x) * 256 + threadIdx.x; e < total;
         e += int64_t(gridDim.x) * 256) {
        const int64_t p = e / RC, rc = e - p * RC;
        const int64_t r = rc / C, c = rc - r * C;
        const int64_t b = clamp64(src[p], 0, nb - 1);
        const int64_t i = b / Kb, j = b - i * Kb;
        Du[e] = Wu[(i * R + r) * ldw + j * C + c];
    }
}

bsr_status launch_prune_wide(const float *W, int64_t ldw, int32_t R, int32_t C, int64_t Kb,
                             int64_t Nb, int64_t nb, int64_t k, unsigned long long *keybits,
                             int32_t *src, int32_t *indptr, int32_t *indices, float *data,
                             int norm, hipStream_t st) {
    const SelectArrays A = select_arrays(src, nb);
    const int64_t want = (nb + kKeyThreads - 1) / kKeyThreads;
    const int ranges = int(want < kMaxRanges ? want : kMaxRanges);
    const int cus = device_cu_count() > 0 ? device_cu_count() : 256;
    const int64_t hist_want = (nb + kSelThreads - 1) / kSelThreads;
    const int64_t hist_most = cus < kMaxHists ? cus : kMaxHists;
    const int hists = int(hist_want < hist_most ? hist_want : hist_most);
    auto keys = norm == BSR_NORM_L1 ? prune_keys_range_kernel<true> : prune_keys_range_kernel<false>;
    hipLaunchKernelGGL(keys, dim3(ranges), dim3(kKeyThreads), 0, st, W, ldw, R, C, unsigned(Kb),
                       unsigned(nb), keybits, A);
    bsr_status s = launch_status();
    if (s != BSR_OK) return s;
    const long long kk = k;
    const unsigned n = unsigned(nb);
    hipLaunchKernelGGL(prune_hist_kernel, dim3(hists), dim3(kSelThreads), 0, st, keybits, n, kk,
                       ranges, A);
    if ((s = launch_status()) != BSR_OK) return s;
    hipLaunchKernelGGL(prune_collect_kernel, dim3(A.chunks), dim3(kSelThreads), 0, st, keybits, n,
                       kk, hists, A);
    if ((s = launch_status()) != BSR_OK) return s;
    hipLaunchKernelGGL(prune_finish_kernel, dim3(1), dim3(kSelThreads), 0, st, keybits, n, A);
    if ((s = launch_status()) != BSR_OK) return s;
    hipLaunchKernelGGL(prune_place_kernel, dim3(A.chunks), dim3(kSelThreads), 0, st, W, ldw, R, C,
                       unsigned(Kb), n, kk, unsigned(Nb), keybits, A, indptr, indices, data);
    return launch_status();
}

}  // namespace

bsr_status noalloc_scratch(void **ptr) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) {
        set_last_hip_error(hipGetErrorString(e));
        return BSR_ERR_HIP;
    }
    if (dev < 0 || dev >= kScratchDevices) return BSR_ERR_UNSUPPORTED;
    std::lock_guard<std::mutex> lock(g_scratch_mutex);
    if (g_scratch_ptr[dev] == nullptr) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) {
            set_last_hip_error(e != hipSuccess ? hipGetErrorString(e)
                                               : "hipGetSymbolAddress returned NULL");
            return BSR_ERR_HIP;
        }
        g_scratch_ptr[dev] = p;
    }
    *ptr = g_scratch_ptr[dev];
    return BSR_OK;
}

bsr_status launch_prune(const float *W, int64_t N, int64_t K, int64_t ldw, int32_t R, int32_t C,
                        int64_t k, int32_t *indptr, int32_t *indices, float *data,
                        void *workspace, int norm, int select, void *stream) {
    const int64_t Nb = N / R, Kb = K / C, nb = Nb * Kb;
    const PruneWorkspace ws = prune_workspace_layout(nb);
    char *base = static_cast<char *>(workspace);
    auto *keybits = reinterpret_cast<unsigned long long *>(base + ws.key_offset);
    auto *src = reinterpret_cast<int32_t *>(base + ws.src_offset);
    hipStream_t st = as_stream(stream);

    // Global selection over more keys than one workgroup's LDS holds codes of: spread over the chip.
    if (select == BSR_SELECT_GLOBAL && k > 0 && nb > int64_t(kSelThreads) * kRegKeys)
        return launch_prune_wide(W, ldw, R, C, Kb, Nb, nb, k, keybits, src, indptr, indices, data,
                                 norm, st);
    if (k > 0) {
        const int64_t RC = int64_t(R) * C;
        if (C > 1 && RC >= kStageMinWords && RC <= kStageWords) {
            const int G = int(kStageWords / RC < kStageBlocks ? kStageWords / RC : kStageBlocks);
            auto keys =
                norm == BSR_NORM_L1 ? prune_keys_staged_kernel<true> : prune_keys_staged_kernel<false>;
            hipLaunchKernelGGL(keys, dim3(static_cast<unsigned>((nb + G - 1) / G)),
                               dim3(kKeyThreads), size_t(G) * size_t(RC + 1) * 4, st, W, ldw, R, C,
                               unsigned(Kb), unsigned(nb), G, keybits);
        } else {
            const unsigned g = static_cast<unsigned>((nb + kKeyThreads - 1) / kKeyThreads);
            auto keys = norm == BSR_NORM_L1 ? prune_keys_kernel<true> : prune_keys_kernel<false>;
            hipLaunchKernelGGL(keys, dim3(g), dim3(kKeyThreads), 0, st, W, ldw, R, C, Kb, nb,
                               keybits);
        }
        bsr_status s = launch_status();
        if (s != BSR_OK) return s;
    }
    if (select == BSR_SELECT_PER_ROW)
        hipLaunchKernelGGL(prune_select_rows_kernel, dim3(static_cast<unsigned>(Nb)),
                           dim3(kRowThreads), 0, st, keybits, Kb, Nb, k / Nb, indptr, indices,
                           src);
    else
        hipLaunchKernelGGL(prune_select_kernel, dim3(1), dim3(kSelThreads),
                           k > 0 ? select_lds_bytes(nb) : 0, st, keybits, nb, Kb, Nb, k, indptr,
                           indices, src);
    bsr_status s = launch_status();
    if (s != BSR_OK || k == 0) return s;
    hipLaunchKernelGGL(prune_copy_kernel, dim3(grid_for(k * R * C, 256)), dim3(256), 0, st, W,
                       ldw, R, C, Kb, nb, k, src, data);
    return launch_status();
}

}  // namespace bsr
