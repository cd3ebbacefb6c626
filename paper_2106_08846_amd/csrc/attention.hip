// Scaled dot-product attention of the BERT attention block whose projections are the pruned
// BSR products (Sec. 2.3 prunes BERT's attention weights; Table 1 times the whole model):
//
//   ctx[b, s, head h] = sum_j softmax_j(scale * <Q[b,s,h], K[b,j,h]>) V[b,j,h]
//
// Tokens are rows t = b * seq + s of Q, K, V and ctx; head h owns columns h*64 .. h*64 + 63.
// No mask: every token attends to every token of its sequence.  fp32 inputs, sums and outputs; the
// products are fp32, or exact cross terms of bf16 pieces in the matrix-core version below.
//
// Short sequences with few queries run on the vector ALUs: one workgroup of 64 threads computes
// 8 queries of one (sequence, head).  The keys are
// visited in blocks of 64: the block's K and V rows are staged in LDS (row pitch 68 floats, so
// rows start 4 banks apart and the 16-byte reads below are conflict-free), and the softmax is
// kept online (running maximum m, running sum l, output rescaled by exp(m_old - m_new)), so no
// score matrix is stored.  Thread t serves query t / 8; its 8 lanes split the block's keys for
// the scores (lane u takes keys u, u + 8, ...) and the 64 output columns for P V (lane u takes
// columns 8u .. 8u + 7); the row's maximum and sum are combined across the 8 lanes with xor
// shuffles, and the row's weights pass from the score lanes to the output lanes through LDS.
#include <cmath>

#include "device_common.h"

namespace bsr {

namespace {

constexpr int kKB = 64;       // keys per block
constexpr int kD = 64;        // head width
constexpr int kPitch = 68;    // LDS row pitch, floats
constexpr int kMfmaMinSeq = 256;   // sequences that always take the matrix-core kernel
constexpr int kSplitBelow = 2;     // key-split 8-query tiles below this many tiles per CU

typedef float floatx4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ floatx4 load4(const float *p) {
    return *reinterpret_cast<const floatx4 *>(p);
}

__device__ __forceinline__ float row_max8(float x) {
    x = fmaxf(x, __shfl_xor(x, 1));
    x = fmaxf(x, __shfl_xor(x, 2));
    return fmaxf(x, __shfl_xor(x, 4));
}

__device__ __forceinline__ float row_sum8(float x) {
    x += __shfl_xor(x, 1);
    x += __shfl_xor(x, 2);
    return x + __shfl_xor(x, 4);
}

__global__ __launch_bounds__(64) void attention_kernel(
    const float *__restrict__ Q, int64_t ldq, const float *__restrict__ K, int64_t ldk,
    const float *__restrict__ V, int64_t ldv, float *__restrict__ O, int64_t ldo, int seq,
    float scale) {
    constexpr int kQT = 8, kThreads = kQT * 8;
    __shared__ float Ks[kKB * kPitch];
    __shared__ float Vs[kKB * kPitch];
    __shared__ float Ps[kQT * kPitch];
    const int tid = threadIdx.x, qi = tid >> 3, u = tid & 7;
    const int q0 = blockIdx.x * kQT, h = blockIdx.y;
    const int64_t tok0 = int64_t(blockIdx.z) * seq;
    const int qrow = q0 + qi;
    const bool qvalid = qrow < seq;

    // This thread's query row, pre-scaled (rows past the sequence read row 0; never stored).
    float q[kD];
    {
        const float *qp = Q + (tok0 + (qvalid ? qrow : 0)) * ldq + h * kD;
#pragma unroll
        for (int d = 0; d < kD; d += 4) {
            const floatx4 v = load4(qp + d);
#pragma unroll
            for (int e = 0; e < 4; ++e) q[d + e] = v[e] * scale;
        }
    }
    float m = -INFINITY, l = 0.0f, acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;

    for (int k0 = 0; k0 < seq; k0 += kKB) {
        __syncthreads();   // the previous block's LDS reads are done
        // Stage K and V rows k0 .. k0 + 63 of this head (rows past the sequence are zero).
        // Four 16-byte pieces of K and of V per thread in flight, then their LDS stores.
        constexpr int kPer = kKB * (kD / 4) / kThreads;   // pieces per thread
        constexpr int kBatch = kPer < 4 ? kPer : 4;
#pragma unroll
        for (int n0 = 0; n0 < kPer; n0 += kBatch) {
            floatx4 kst[kBatch], vst[kBatch];
#pragma unroll
            for (int n = 0; n < kBatch; ++n) {
                const int i = tid + (n0 + n) * kThreads;
                const int r = i >> 4, c4 = (i & 15) * 4;
                const int key = k0 + r < seq ? k0 + r : seq - 1;   // past the end: zeroed below
                kst[n] = load4(K + (tok0 + key) * ldk + h * kD + c4);
                vst[n] = load4(V + (tok0 + key) * ldv + h * kD + c4);
            }
#pragma unroll
            for (int n = 0; n < kBatch; ++n) {
                const int i = tid + (n0 + n) * kThreads;
                const int r = i >> 4, c4 = (i & 15) * 4;
                const floatx4 z = {0.0f, 0.0f, 0.0f, 0.0f};
                *reinterpret_cast<floatx4 *>(&Ks[r * kPitch + c4]) = k0 + r < seq ? kst[n] : z;
                *reinterpret_cast<floatx4 *>(&Vs[r * kPitch + c4]) = k0 + r < seq ? vst[n] : z;
            }
        }
        __syncthreads();

        // Scores of keys u + 8j (j < 8), the eight dot products advanced together (eight
        // independent FMA chains); keys past the sequence get -inf (weight 0).
        float s[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) s[j] = 0.0f;
#pragma unroll
        for (int d = 0; d < kD; d += 4) {
            floatx4 kv[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) kv[j] = load4(&Ks[(u + 8 * j) * kPitch + d]);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < 8; ++j) s[j] = __builtin_fmaf(q[d + e], kv[j][e], s[j]);
        }
#pragma unroll
        for (int j = 0; j < 8; ++j)
            if (k0 + u + 8 * j >= seq) s[j] = -INFINITY;
        float bm = s[0];
#pragma unroll
        for (int j = 1; j < 8; ++j) bm = fmaxf(bm, s[j]);
        const float mn = fmaxf(m, row_max8(bm));   // finite: key k0 exists
        const float corr = expf(m - mn);           // 0 on the first block (m = -inf)
        float ps = 0.0f;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const float p = expf(s[j] - mn);
            ps += p;
            Ps[qi * kPitch + u + 8 * j] = p;
        }
        l = l * corr + row_sum8(ps);
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= corr;
        m = mn;
        __syncthreads();   // the row's weights are in LDS

        const float *pr = &Ps[qi * kPitch];
#pragma unroll 8
        for (int r = 0; r < kKB; ++r) {
            const float p = pr[r];
            const floatx4 v0 = load4(&Vs[r * kPitch + 8 * u]);
            const floatx4 v1 = load4(&Vs[r * kPitch + 8 * u + 4]);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                acc[e] = __builtin_fmaf(p, v0[e], acc[e]);
                acc[4 + e] = __builtin_fmaf(p, v1[e], acc[4 + e]);
            }
        }
    }
    if (qvalid) {
        float *op = O + (tok0 + qrow) * ldo + h * kD + 8 * u;
#pragma unroll
        for (int e = 0; e < 8; ++e) op[e] = acc[e] / l;
    }
}

// Short sequences with few (sequence, head) pairs: kKS groups of 8 queries x 8 lanes (one wave
// each) serve the same queries; group ks takes the key blocks ks, ks + kKS, ... with the online
// softmax above, and the groups' partial results are merged at the end.  Each group has its own
// K, V and P buffers in (dynamic) LDS.
template <int kKS>
__global__ __launch_bounds__(64 * kKS) void attention_split_kernel(
    const float *__restrict__ Q, int64_t ldq, const float *__restrict__ K, int64_t ldk,
    const float *__restrict__ V, int64_t ldv, float *__restrict__ O, int64_t ldo, int seq,
    float scale) {
    constexpr int kQT = 8;
    constexpr int kThreads = kQT * 8;             // threads per group
    constexpr int kGroupFloats = 2 * kKB * kPitch + kQT * kPitch;
    extern __shared__ float smem[];
    const int ks = threadIdx.x / kThreads, tid = threadIdx.x % kThreads;
    float *Ks = smem + ks * kGroupFloats;
    float *Vs = Ks + kKB * kPitch;
    float *Ps = Vs + kKB * kPitch;
    const int qi = tid >> 3, u = tid & 7;
    const int q0 = blockIdx.x * kQT, h = blockIdx.y;
    const int64_t tok0 = int64_t(blockIdx.z) * seq;
    const int qrow = q0 + qi;
    const bool qvalid = qrow < seq;

    // This thread's query row, pre-scaled (rows past the sequence read row 0; never stored).
    float q[kD];
    {
        const float *qp = Q + (tok0 + (qvalid ? qrow : 0)) * ldq + h * kD;
#pragma unroll
        for (int d = 0; d < kD; d += 4) {
            const floatx4 v = load4(qp + d);
#pragma unroll
            for (int e = 0; e < 4; ++e) q[d + e] = v[e] * scale;
        }
    }
    float m = -INFINITY, l = 0.0f, acc[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] = 0.0f;

    // Every group runs the same number of rounds (and barriers); a group whose block is past
    // the end of the sequence idles through its round.
    const int nblk = (seq + kKB - 1) / kKB;
    const int rounds = (nblk + kKS - 1) / kKS;
    for (int it = 0; it < rounds; ++it) {
        const int k0 = (ks + kKS * it) * kKB;
        const bool active = k0 < seq;
        __syncthreads();   // the previous block's LDS reads are done
        // Stage K and V rows k0 .. k0 + 63 of this head (rows past the sequence are zero).
        // Four 16-byte pieces of K and of V per thread in flight, then their LDS stores.
        constexpr int kPer = kKB * (kD / 4) / kThreads;   // pieces per thread
        constexpr int kBatch = kPer < 4 ? kPer : 4;
        if (active) {
#pragma unroll
            for (int n0 = 0; n0 < kPer; n0 += kBatch) {
                floatx4 kst[kBatch], vst[kBatch];
#pragma unroll
                for (int n = 0; n < kBatch; ++n) {
                    const int i = tid + (n0 + n) * kThreads;
                    const int r = i >> 4, c4 = (i & 15) * 4;
                    const int key = k0 + r < seq ? k0 + r : seq - 1;   // past the end: zeroed
                    kst[n] = load4(K + (tok0 + key) * ldk + h * kD + c4);
                    vst[n] = load4(V + (tok0 + key) * ldv + h * kD + c4);
                }
#pragma unroll
                for (int n = 0; n < kBatch; ++n) {
                    const int i = tid + (n0 + n) * kThreads;
                    const int r = i >> 4, c4 = (i & 15) * 4;
                    const floatx4 z = {0.0f, 0.0f, 0.0f, 0.0f};
                    *reinterpret_cast<floatx4 *>(&Ks[r * kPitch + c4]) = k0 + r < seq ? kst[n] : z;
                    *reinterpret_cast<floatx4 *>(&Vs[r * kPitch + c4]) = k0 + r < seq ? vst[n] : z;
                }
            }
        }
        __syncthreads();

        if (active) {
            // Scores of keys u + 8j (j < 8), the eight dot products advanced together (eight
            // independent FMA chains); keys past the sequence get -inf (weight 0).
            float s[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] = 0.0f;
#pragma unroll
            for (int d = 0; d < kD; d += 4) {
                floatx4 kv[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) kv[j] = load4(&Ks[(u + 8 * j) * kPitch + d]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int j = 0; j < 8; ++j) s[j] = __builtin_fmaf(q[d + e], kv[j][e], s[j]);
            }
#pragma unroll
            for (int j = 0; j < 8; ++j)
                if (k0 + u + 8 * j >= seq) s[j] = -INFINITY;
            float bm = s[0];
#pragma unroll
            for (int j = 1; j < 8; ++j) bm = fmaxf(bm, s[j]);
            const float mn = fmaxf(m, row_max8(bm));   // finite: key k0 exists
            const float corr = expf(m - mn);           // 0 on the group's first block
            float ps = 0.0f;
#pragma unroll
            for (int j = 0; j < 8; ++j) {
                const float p = expf(s[j] - mn);
                ps += p;
                Ps[qi * kPitch + u + 8 * j] = p;
            }
            l = l * corr + row_sum8(ps);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] *= corr;
            m = mn;
        }
        __syncthreads();   // the row's weights are in LDS

        if (active) {
            const float *pr = &Ps[qi * kPitch];
#pragma unroll 8
            for (int r = 0; r < kKB; ++r) {
                const float p = pr[r];
                const floatx4 v0 = load4(&Vs[r * kPitch + 8 * u]);
                const floatx4 v1 = load4(&Vs[r * kPitch + 8 * u + 4]);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    acc[e] = __builtin_fmaf(p, v0[e], acc[e]);
                    acc[4 + e] = __builtin_fmaf(p, v1[e], acc[4 + e]);
                }
            }
        }
    }
    {
        // Merge the groups in group order: with M the largest running maximum,
        // out = sum_g acc_g exp(m_g - M) / sum_g l_g exp(m_g - M).  A group that saw no key
        // has m = -inf, l = 0 and adds nothing; group 0 always saw key 0.
        constexpr int kSlot = 8 * 8 + 2;   // per thread: acc, then m and l
        __syncthreads();
        float *C = smem + (ks * kThreads + tid) * kSlot;
#pragma unroll
        for (int e = 0; e < 8; ++e) C[e] = acc[e];
        C[64] = m;
        C[65] = l;
        __syncthreads();
        if (ks != 0) return;
        float M = m;
#pragma unroll
        for (int g = 1; g < kKS; ++g) M = fmaxf(M, smem[(g * kThreads + tid) * kSlot + 64]);
        const float w0 = expf(m - M);
        l *= w0;
#pragma unroll
        for (int e = 0; e < 8; ++e) acc[e] *= w0;
#pragma unroll
        for (int g = 1; g < kKS; ++g) {
            const float *Cg = smem + (g * kThreads + tid) * kSlot;
            const float w = expf(Cg[64] - M);   // 0 for a group without keys
            l = __builtin_fmaf(Cg[65], w, l);
#pragma unroll
            for (int e = 0; e < 8; ++e) acc[e] = __builtin_fmaf(Cg[e], w, acc[e]);
        }
    }
    if (qvalid) {
        float *op = O + (tok0 + qrow) * ldo + h * kD + 8 * u;
#pragma unroll
        for (int e = 0; e < 8; ++e) op[e] = acc[e] / l;
    }
}

// ------------------------------------------------------------------- matrix-core version
// One wave computes 32 queries of one (sequence, head); kWQ query tiles of a workgroup share the
// staged keys and values (blocks of 64, as above), and with kKS = 2 two waves serve each tile, one
// taking the first 32 keys of every block and the other the second 32, merged at the end.  Lane l
// serves query l % 32 as half hh = l / 32.
//   Scores, transposed: S^T = K Q^T for each group of 32 keys.  Register v of lane l then holds
//   the score of query l % 32 and key 8(v/4) + 4hh + v%4 of the group, so a query's 32 scores sit
//   in the lane pair (l, l ^ 32): the group maximum and sum take 15 register operations and one
//   exchange.
//   Output, transposed: O^T += V^T P^T: the weights of a lane are its own B operand, so they never
//   leave their registers.
// The online softmax is the one above (running maximum and sum per query, output rescaled by
// exp(m_old - m_new)); each query's running values are kept, identical, in both its lanes.
//
// Arithmetic.  fp32 matrix instructions share the vector ALUs: 147 thousand of a CU's 236 thousand
// cycles went to them and 64 thousand to vector instructions on 16 x 16 heads x 384 tokens
// (MI355X counters), with next to nothing left to overlap.  So both products run on bf16 matrix
// instructions with every fp32 operand x as three bf16 pieces, x = x0 + x1 + x2 exactly, each the
// remainder rounded to nearest (|x1| <= 2^-9 |x|, |x2| <= 2^-18 |x|).  Of the nine cross terms the
// six with i + j <= 2 are formed, each exact in fp32; the three left out are below 2^-25 |x y|
// together, half an ulp of the fp32 product that they belong to.  The weights are carried as
// 2^24 exp(s - m), as is their sum, and the values as 2^24 V: the last bit of any fp32 number, 2^-149,
// is then a normal bf16 number, so the pieces of a weight or a value are exact down to the smallest
// one.  (Pieces of a query or a key below 2^-102 may lose their last bits: less than 2^-126 of an
// operand, times one below 2^48, changes a score by less than 2^-70.)
// Every group's output is summed from zero and then added to the running output, so the long sum
// is rounded once per 32 keys.  Against fp64, 384 tokens x 16 heads, normal inputs: 2-norm error
// 2.4e-7, where fp32 matrix instructions with one running sum gave 4.5e-7.
// 16 x 384 tokens, 16 heads: 104 -> 66 us; 8 x 512, 12 heads: 76 -> 53 us (MI355X); what bounds it
// now is vector instructions (softmax and splitting) and matrix instructions in turn.
// kAhead: the next block's keys and values are loaded under this block's products, in registers that
// two waves per SIMD leave free.  With few tiles a workgroup has a SIMD nearly to itself, and waiting
// for K and then for V in every block made it slower than the fp32 kernel, which loaded both at once
// (inputs not in the L2: 3 x 262 tokens, 8 heads 25.5 us, fp32 23.3; now 18.9; 1 x 508, 12 heads 38.7,
// 35.1 and 27.4).
// Operands have to lie below 2^48, so that no score and no sum over 2^31 keys overflows.  A workgroup
// that stages any other element (infinities and NaN among them) goes on from that block of keys on
// fp32 matrix instructions.
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int kPieces = 3;
constexpr int kPlane = kKB * kD;   // elements of a plane: 64 rows of 64 bf16, 8-element chunks
                                   // of a row swizzled by its row so that equal chunks of eight
                                   // consecutive rows lie in different banks
constexpr float kWeightExp = 24.0f, kWeightScale = 0x1p24f, kValueScale = 0x1p24f;

__device__ __forceinline__ unsigned cvt_pair(float a, float b) {   // round to nearest even
    const floatx2 v = {a, b};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}

// The pieces of a pair of values, packed.
__device__ __forceinline__ void split_pair(float a, float b, unsigned (&u)[kPieces]) {
#pragma unroll
    for (int p = 0; p < kPieces; ++p) {
        u[p] = cvt_pair(a, b);
        a -= __uint_as_float(u[p] << 16);
        b -= __uint_as_float(u[p] & 0xffff0000u);
    }
}

__device__ __forceinline__ void split8(const float (&v)[8], uintx4 (&out)[kPieces]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        unsigned u[kPieces];
        split_pair(v[2 * i], v[2 * i + 1], u);
#pragma unroll
        for (int p = 0; p < kPieces; ++p) out[p][i] = u[p];
    }
}

// The largest magnitude seen, as a bit pattern (infinities and NaN above all numbers).
struct Range {
    unsigned hi = 0u;
    __device__ __forceinline__ void add(float x) {
        hi = max(hi, __float_as_uint(x) & 0x7fffffffu);
    }
    __device__ __forceinline__ bool outside() const { return hi >= 0x57800000u; }   // 2^48
};

// Byte offset of chunk c of row r in a plane.
__device__ __forceinline__ int plane_at(int r, int c) { return r * 128 + ((c ^ (r & 7)) << 4); }

__device__ __forceinline__ floatx16 mfma_bf16(const uintx4 &a, const uintx4 &b, floatx16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                   __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The six cross terms, smallest first.
__device__ __forceinline__ floatx16 mfma_split(const uintx4 (&a)[kPieces],
                                               const uintx4 (&b)[kPieces], floatx16 c) {
    c = mfma_bf16(a[2], b[0], c);
    c = mfma_bf16(a[1], b[1], c);
    c = mfma_bf16(a[0], b[2], c);
    c = mfma_bf16(a[1], b[0], c);
    c = mfma_bf16(a[0], b[1], c);
    return mfma_bf16(a[0], b[0], c);
}

// 2^24 exp(x) for x <= 0: 2^u of u = x log2(e) + 24, rounded to z + 24 with z = u - 24 exact, times
// 1 + r ln 2 for what the roundings and log2(e)'s low bits left out (r < 2^-16 where exp(x) is not
// negligible).  About half of expf's instructions: x is never positive and above -2^121, so nothing
// overflows (where 2^u is 0, r is finite).  The 2^24 inside the hardware's 2^u, which is never a
// subnormal number, keep the smallest weights.
__device__ __forceinline__ float exp_scaled(float x) {
#pragma clang fp contract(off)
    constexpr float kLog2e = 0x1.715476p+0f, kLog2eLo = 0x1.4ae0bfp-26f, kLn2 = 0x1.62e430p-1f;
    const float t = x * kLog2e, u = t + kWeightExp, z = u - kWeightExp;
    float r = __builtin_fmaf(x, kLog2e, -z);
    r = __builtin_fmaf(x, kLog2eLo, r);
    return __builtin_amdgcn_exp2f(u) * __builtin_fmaf(r, kLn2, 1.0f);
}

// A tile's running state, by lane: query l % 32, outputs as documented at the stores.
struct TileState {
    float m, l;
    floatx16 o0, o1;
};

__device__ __forceinline__ void tile_reset(TileState &st) {
    st.m = -INFINITY;
    st.l = 0.0f;
#pragma unroll
    for (int v = 0; v < 16; ++v) st.o0[v] = st.o1[v] = 0.0f;
}

// Keys past the sequence get a score of weight 0: -inf, or -2^120 for exp_scaled, which is below every
// score of operands under 2^48.  A group's first key exists.
template <bool kSplit>
__device__ __forceinline__ void mask_keys(floatx16 &s, int kg, int hh, int seq) {
    if (kg + 32 > seq) {
#pragma unroll
        for (int v = 0; v < 16; ++v)
            if (kg + 8 * (v >> 2) + 4 * hh + (v & 3) >= seq) s[v] = kSplit ? -0x1p120f : -INFINITY;
    }
}

// Running maximum, weights (in s; kSplit: times 2^24) and running sum; the factor by which the
// outputs so far are to be rescaled is returned.
template <bool kSplit>
__device__ __forceinline__ float online_softmax(TileState &st, floatx16 &s) {
    float mx = s[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float mn = fmaxf(st.m, mx);
    const float corr = expf(st.m - mn);   // 0 on the first group (m = -inf)
    float ps = 0.0f;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        s[v] = kSplit ? exp_scaled(s[v] - mn) : expf(s[v] - mn);
        ps += s[v];
    }
    ps += __shfl_xor(ps, 32);
    st.l = st.l * corr + ps;
    st.m = mn;
    return corr;
}

// A tile's keys on bf16 pieces.  At the first block with an operand out of the pieces' range (a query
// counts with the first) it stops and returns false, the block's first key in `left`, in every thread
// of the workgroup.  The state carries the scales of the weights and the values.
template <int kWQ, int kKS, bool kAhead>
__device__ __forceinline__ bool tile_split(TileState &st, const float *qp, const float *Kh,
                                           int64_t ldk, const float *Vh, int64_t ldv, int seq,
                                           float scale, char *smem, int *s_bad, int &left) {
    constexpr int kThreads = kWQ * kKS * 64;
    char *Kp = smem, *Vp = smem + kPieces * kPlane * 2;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ks = wave / kWQ;
    const int ql = lane & 31, hh = lane >> 5;
    Range range;
    // The lane's pre-scaled query pieces: step s contracts dimensions 16 s + 8 hh + e.
    uintx4 q[4][kPieces];
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const floatx4 a = load4(qp + 16 * s + 8 * hh), b = load4(qp + 16 * s + 8 * hh + 4);
        float v[8];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = a[e] * scale;
            v[4 + e] = b[e] * scale;
        }
#pragma unroll
        for (int e = 0; e < 8; ++e) range.add(v[e]);
        split8(v, q[s]);
    }
    // A block's planes, in chunks of eight elements, one or more of each per thread.  K: row = key, chunk = 8
    // dimensions.  V: row = output column d, chunk = the 8 keys that one half contracts in one step,
    // in its registers' order: keys 16 s + 4 h + (0 .. 3) and 16 s + 8 + 4 h + (0 .. 3).  Rows past the
    // sequence are zero.  With one chunk of each per thread (eight tiles) K and V are loaded together
    // (8 x 512 tokens, 12 heads 55.3 -> 53.4 us); elsewhere that spilled.
    constexpr bool kBoth = kAhead || kThreads == kKB * 8;   // K and V in registers at once
    constexpr int kPer = kBoth ? kKB * 8 / kThreads : 1;
    static_assert(!kBoth || kPer * kThreads == kKB * 8, "every thread holds kPer chunks of each");
    float kv[kPer][8], vv[kPer][8];
    auto each_chunk = [&](auto f) {
        if constexpr (kBoth) {
#pragma unroll
            for (int n = 0; n < kPer; ++n) f(n, tid + n * kThreads);
        } else {
            for (int i = tid; i < kKB * 8; i += kThreads) f(0, i);
        }
    };
    auto v_key = [](int c, int e) { return 16 * (c >> 1) + 4 * (c & 1) + (e & 3) + 8 * (e >> 2); };
    auto load_k = [&](int n, int i, int k0) {
        const int key = k0 + (i >> 3);
        const float *kp = Kh + int64_t(key < seq ? key : seq - 1) * ldk + 8 * (i & 7);
        const floatx4 a = load4(kp), b = load4(kp + 4);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            kv[n][e] = a[e];
            kv[n][4 + e] = b[e];
        }
    };
    auto load_v = [&](int n, int i, int k0) {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const int key = k0 + v_key(i >> 6, e);
            vv[n][e] = Vh[int64_t(key < seq ? key : seq - 1) * ldv + (i & 63)];
        }
    };
    auto store = [&](const float (&v)[8], char *planes, int r, int c) {
        uintx4 u[kPieces];
        split8(v, u);
#pragma unroll
        for (int p = 0; p < kPieces; ++p)
            *reinterpret_cast<uintx4 *>(planes + p * kPlane * 2 + plane_at(r, c)) = u[p];
    };
    auto store_k = [&](int n, int i, int k0) {
        const int r = i >> 3;
#pragma unroll
        for (int e = 0; e < 8; ++e) kv[n][e] = k0 + r < seq ? kv[n][e] : 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) range.add(kv[n][e]);
        store(kv[n], Kp, r, i & 7);
    };
    auto store_v = [&](int n, int i, int k0) {
        const int c = i >> 6;
#pragma unroll
        for (int e = 0; e < 8; ++e) vv[n][e] = k0 + v_key(c, e) < seq ? vv[n][e] : 0.0f;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            range.add(vv[n][e]);
            vv[n][e] *= kValueScale;
        }
        store(vv[n], Vp, i & 63, c);
    };
    auto load_block = [&](int k0) {
        each_chunk([&](int n, int i) { load_k(n, i, k0); });
        each_chunk([&](int n, int i) { load_v(n, i, k0); });
    };
    if (tid == 0) *s_bad = 0;
    if constexpr (kAhead) load_block(0);
    for (int k0 = 0; k0 < seq; k0 += kKB) {
        __syncthreads();   // the previous block's LDS reads are done
        if constexpr (kBoth && !kAhead) load_block(k0);
        each_chunk([&](int n, int i) {
            if constexpr (!kBoth) load_k(n, i, k0);
            store_k(n, i, k0);
        });
        each_chunk([&](int n, int i) {
            if constexpr (!kBoth) load_v(n, i, k0);
            store_v(n, i, k0);
        });
        if (range.outside()) *s_bad = 1;
        __syncthreads();
        if (*s_bad) {   // the same word in every thread
            left = k0;
            return false;
        }
        // The next block's loads, under this block's products.
        if (kAhead && k0 + kKB < seq) load_block(k0 + kKB);

#pragma unroll
        for (int gi = 0; gi < kKB / 32 / kKS; ++gi) {
            const int g = gi * kKS + ks;
            const int kg = k0 + 32 * g;
            if (kg >= seq) break;   // the whole group is past the end
            floatx16 s;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = 0.0f;
#pragma unroll
            for (int st4 = 0; st4 < 4; ++st4) {
                uintx4 a[kPieces];
#pragma unroll
                for (int p = 0; p < kPieces; ++p)
                    a[p] = *reinterpret_cast<const uintx4 *>(
                        Kp + p * kPlane * 2 + plane_at(32 * g + ql, 2 * st4 + hh));
                s = mfma_split(a, q[st4], s);
            }
            mask_keys<true>(s, kg, hh, seq);
            const float corr = online_softmax<true>(st, s);
            uintx4 w2[2][kPieces];
#pragma unroll
            for (int h16 = 0; h16 < 2; ++h16) {
                auto &w = w2[h16];
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    unsigned u[kPieces];
                    split_pair(s[8 * h16 + 2 * i], s[8 * h16 + 2 * i + 1], u);
#pragma unroll
                    for (int p = 0; p < kPieces; ++p) w[p][i] = u[p];
                }
            }
            // The group's output from zero, then added to the rescaled sum: one rounding of the
            // long sum per group.
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                floatx16 o;
#pragma unroll
                for (int v = 0; v < 16; ++v) o[v] = 0.0f;
#pragma unroll
                for (int h16 = 0; h16 < 2; ++h16) {
                    uintx4 a[kPieces];
#pragma unroll
                    for (int p = 0; p < kPieces; ++p)
                        a[p] = *reinterpret_cast<const uintx4 *>(
                            Vp + p * kPlane * 2 + plane_at(32 * t + ql, 4 * g + 2 * h16 + hh));
                    o = mfma_split(a, w2[h16], o);
                }
                floatx16 &sum = t == 0 ? st.o0 : st.o1;
#pragma unroll
                for (int v = 0; v < 16; ++v) sum[v] = __builtin_fmaf(sum[v], corr, o[v]);
            }
        }
    }
    return true;
}

// A tile's keys from k0 on, on v_mfma_f32_32x32x2_f32, for operands of any value.  Scores: step s
// (s < 32) contracts dimension s + 32hh in slot hh: A = K[key l%32][s + 32hh] (LDS), B = the lane's
// pre-scaled q[s + 32hh].  Output: step v contracts the two keys that register v holds in the two
// halves: A = V[that key][32t + l%32] (LDS; output column tile t = 0, 1), B = the lane's weight p[v].
template <int kWQ, int kKS>
__device__ __forceinline__ void tile_fp32(TileState &st, const float *qp, const float *Kh,
                                          int64_t ldk, const float *Vh, int64_t ldv, int seq,
                                          float scale, char *smem, int k0) {
    constexpr int kThreads = kWQ * kKS * 64;
    float *Ks = reinterpret_cast<float *>(smem), *Vs = Ks + kKB * kPitch;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, ks = wave / kWQ;
    const int ql = lane & 31, hh = lane >> 5;
    float q[32];
#pragma unroll
    for (int d = 0; d < 32; d += 4) {
        const floatx4 v = load4(qp + 32 * hh + d);
#pragma unroll
        for (int e = 0; e < 4; ++e) q[d + e] = v[e] * scale;
    }
    for (; k0 < seq; k0 += kKB) {
        __syncthreads();   // the previous block's LDS reads are done
        for (int i = tid; i < kKB * (kD / 4); i += kThreads) {
            const int r = i >> 4, c4 = (i & 15) * 4, key = k0 + r;
            const floatx4 z = {0.0f, 0.0f, 0.0f, 0.0f};
            const int64_t row = key < seq ? key : seq - 1;
            const floatx4 kv = load4(Kh + row * ldk + c4), vv = load4(Vh + row * ldv + c4);
            *reinterpret_cast<floatx4 *>(&Ks[r * kPitch + c4]) = key < seq ? kv : z;
            *reinterpret_cast<floatx4 *>(&Vs[r * kPitch + c4]) = key < seq ? vv : z;
        }
        __syncthreads();
#pragma unroll 1
        for (int gi = 0; gi < kKB / 32 / kKS; ++gi) {
            const int g = gi * kKS + ks;
            const int kg = k0 + 32 * g;
            if (kg >= seq) break;   // the whole group is past the end
            floatx16 s;
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = 0.0f;
            const float *kr = &Ks[(32 * g + ql) * kPitch + 32 * hh];
#pragma unroll
            for (int d = 0; d < 32; d += 4) {
                const floatx4 kv = load4(kr + d);
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    s = __builtin_amdgcn_mfma_f32_32x32x2f32(kv[e], q[d + e], s, 0, 0, 0);
            }
            mask_keys<false>(s, kg, hh, seq);
            const float corr = online_softmax<false>(st, s);
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                st.o0[v] *= corr;
                st.o1[v] *= corr;
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const float *vr = &Vs[(32 * g + 8 * (v >> 2) + 4 * hh + (v & 3)) * kPitch + ql];
                st.o0 = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[0], s[v], st.o0, 0, 0, 0);
                st.o1 = __builtin_amdgcn_mfma_f32_32x32x2f32(vr[32], s[v], st.o1, 0, 0, 0);
            }
        }
    }
}

// LDS of a workgroup: the piece planes of K and V, or K and V in fp32, or the merge buffer.
constexpr int kMfmaLds = 2 * kPieces * kPlane * 2;
static_assert(2 * kKB * kPitch * 4 <= kMfmaLds, "the fp32 tiles fit");

template <int kWQ, int kKS, bool kAhead = false>
__global__ __launch_bounds__(kWQ * kKS * 64) __attribute__((amdgpu_waves_per_eu(kAhead ? 2 : 3)))
void attention_mfma_kernel(
    const float *__restrict__ Q, int64_t ldq, const float *__restrict__ K, int64_t ldk,
    const float *__restrict__ V, int64_t ldv, float *__restrict__ O, int64_t ldo, int seq,
    float scale) {
    static_assert(kKS == 1 || kKS == 2, "one or two waves per query tile");
    __shared__ __align__(16) char smem[kMfmaLds];
    __shared__ int s_bad;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int qw = wave % kWQ, ks = wave / kWQ;
    const int ql = lane & 31, hh = lane >> 5;
    const int qrow = (blockIdx.x * kWQ + qw) * 32 + ql, h = blockIdx.y;
    const int64_t tok0 = int64_t(blockIdx.z) * seq;
    const bool qvalid = qrow < seq;
    // This lane's query row (rows past the sequence read row 0; never stored).
    const float *qp = Q + (tok0 + (qvalid ? qrow : 0)) * ldq + h * kD;
    const float *Kh = K + tok0 * ldk + h * kD, *Vh = V + tok0 * ldv + h * kD;
    TileState st;
    tile_reset(st);
    int left = 0;
    if (!tile_split<kWQ, kKS, kAhead>(st, qp, Kh, ldk, Vh, ldv, seq, scale, smem, &s_bad, left)) {
        st.l *= 1.0f / kWeightScale;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            st.o0[v] *= 1.0f / (kWeightScale * kValueScale);
            st.o1[v] *= 1.0f / (kWeightScale * kValueScale);
        }
        tile_fp32<kWQ, kKS>(st, qp, Kh, ldk, Vh, ldv, seq, scale, smem, left);
    } else {
        // Outputs are quotients, so a common scale does not show.  (With this line before the return
        // above, the compiler spilled 26 registers.)
        st.l *= kValueScale;
    }
    float &m = st.m, &l = st.l;
    floatx16 &o0 = st.o0, &o1 = st.o1;
    if constexpr (kKS == 2) {
        // Merge the two key halves: the second wave of each tile leaves its running maximum,
        // sum and output in LDS (the planes are free after the barrier); the first adds
        // them, both rescaled to the larger maximum.  A wave that saw no key (sequences of at
        // most 32) has m = -inf, l = 0 and adds nothing.
        constexpr int kSlot = 34;   // floats per lane: o0, o1, m, l
        static_assert(kWQ * 64 * kSlot * 4 <= kMfmaLds, "the merge buffer fits");
        __syncthreads();
        float *C = reinterpret_cast<float *>(smem) + (qw * 64 + lane) * kSlot;
        if (ks == 1) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                C[v] = o0[v];
                C[16 + v] = o1[v];
            }
            C[32] = m;
            C[33] = l;
        }
        __syncthreads();
        if (ks == 1) return;
        const float m1 = C[32], M = fmaxf(m, m1);
        const float w0 = expf(m - M), w1 = expf(m1 - M);
        l = l * w0 + C[33] * w1;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            o0[v] = o0[v] * w0 + C[v] * w1;
            o1[v] = o1[v] * w0 + C[16 + v] * w1;
        }
    }
    // Register v of tile t holds O[query][32t + 8(v/4) + 4hh + v%4]: four consecutive columns
    // per group of four registers, stored as 16 bytes.
    if (qvalid) {
        float *op = O + (tok0 + qrow) * ldo + h * kD + 4 * hh;
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            floatx4 a, b;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                a[e] = o0[4 * v4 + e] / l;
                b[e] = o1[4 * v4 + e] / l;
            }
            *reinterpret_cast<floatx4 *>(op + 8 * v4) = a;
            *reinterpret_cast<floatx4 *>(op + 32 + 8 * v4) = b;
        }
    }
}

}  // namespace

bsr_status launch_attention(const float *Q, int64_t ldq, const float *K, int64_t ldk,
                            const float *V, int64_t ldv, float *O, int64_t ldo, int batch,
                            int seq, int heads, float scale, void *stream) {
    const int64_t nt = (seq + 31) / 32, pairs = int64_t(heads) * batch, tiles32 = nt * pairs;
    const int64_t cus = device_cu_count() > 0 ? device_cu_count() : 256;
    // The matrix-core kernel from 256 keys on, and for shorter sequences when there are enough
    // 32-query tiles (its one-wave chain of key groups is longer than the vector kernels' waves).
    // Vector / matrix kernel in us, 12 heads: 2 x 128 tokens (96 tiles) 9.9 / 11.4, 1 x 200 (84)
    // 17.0 / 17.9, 4 x 128 (192) 13.8 / 11.6, 16 x 40 (384) 10.4 / 9.5, 4 x 200 (336) 31.4 / 18.7.
    if (seq >= kMfmaMinSeq || 8 * tiles32 >= 5 * cus) {
        auto go = [&](auto kernel, int wq, int ks) {
            const dim3 grid(unsigned((nt + wq - 1) / wq), unsigned(heads), unsigned(batch));
            hipLaunchKernelGGL(kernel, grid, dim3(64 * wq * ks), 0, as_stream(stream), Q, ldq, K,
                               ldk, V, ldv, O, ldo, seq, scale);
            return launch_status();
        };
        // Under three tiles per CU (or tiles too few to share staged keys) two waves split each
        // tile's keys: 1 x 512 tokens 32 us against 43 with one wave per tile.  Loading ahead takes
        // registers for at most 1.5 workgroups per CU, all that there are below three tiles.
        if (tiles32 < 3 * cus) return go(attention_mfma_kernel<2, 2, true>, 2, 2);
        if (nt < 4) return go(attention_mfma_kernel<2, 2>, 2, 2);
        // Else 12, 8 or 4 tiles share a workgroup's staged keys, whichever leaves the fewest waves
        // on the busiest SIMD; staging costs about a tenth and three tenths more for 8 and 4 tiles
        // (12 / 8 / 4 tiles: 16 x 384 tokens, 16 heads 70 / 92 / 80 us; 8 x 512, 12 heads
        // 77 / 61 / 73; 32 x 128, 12 heads 41 / 33 / 23).
        auto rounds = [&](int64_t wq) { return ((nt + wq - 1) / wq * pairs + cus - 1) / cus; };
        const int64_t c12 = 30 * rounds(12), c8 = 22 * rounds(8), c4 = 13 * rounds(4);
        if (c12 <= c8 && c12 <= c4) return go(attention_mfma_kernel<12, 1>, 12, 1);
        if (c8 <= c4) return go(attention_mfma_kernel<8, 1>, 8, 1);
        return go(attention_mfma_kernel<4, 1>, 4, 1);
    }
    // Vector-ALU kernels: 8-query tiles; when they give fewer than kSplitBelow waves per CU, two
    // or four waves split the keys of each tile.
    const int nblk = (seq + kKB - 1) / kKB;
    const int64_t tiles8 = int64_t((seq + 7) / 8) * pairs;
    const dim3 grid(unsigned((seq + 7) / 8), unsigned(heads), unsigned(batch));
    const int ks = tiles8 >= kSplitBelow * cus || nblk < 2 ? 1 : (nblk < 4 ? 2 : 4);
    const size_t lds = size_t(ks) * (2 * kKB * kPitch + 8 * kPitch) * sizeof(float);
    if (ks == 1)
        hipLaunchKernelGGL(attention_kernel, grid, dim3(64), 0, as_stream(stream), Q, ldq, K,
                           ldk, V, ldv, O, ldo, seq, scale);
    else if (ks == 2)
        hipLaunchKernelGGL(attention_split_kernel<2>, grid, dim3(128), lds, as_stream(stream), Q,
                           ldq, K, ldk, V, ldv, O, ldo, seq, scale);
    else
        hipLaunchKernelGGL(attention_split_kernel<4>, grid, dim3(256), lds, as_stream(stream), Q,
                           ldq, K, ldk, V, ldv, O, ldo, seq, scale);
    return launch_status();
}

}  // namespace bsr
