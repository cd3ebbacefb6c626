// BSR product for small blocks of 4 or 8 rows (4x1, 8x1, 4x4, 8x8; fp32 or bf16 inputs, fp32
// accumulate) on gfx950 matrix cores.
//
// Y[t][n] = bias[n] + sum over stored blocks p of block-row i = n / R of
//           sum over c < C of X[t][indices[p] * C + c] * data[p][n - iR][c]          (Sec. 2.2)
//
// v_mfma_f32_4x4x1 multiplies sixteen independent 4x1 by 1x4 products; with its A operand
// broadcast inside groups of products (CBSZ/ABID) it becomes four multiply-adds per lane whose
// weights are the same for every lane of a group: four rows of one block column times one X value
// per lane.  So a lane is a token, as on the vector ALUs, but an instruction does four
// multiply-adds in eight cycles where four vector instructions take sixteen, and the weights need
// no broadcast of their own.  bf16 blocks of 4 or 8 columns take v_mfma_f32_4x4x4 (four columns,
// sixteen multiply-adds per lane); other bf16 blocks are widened, exactly, to fp32.
//
//   * One workgroup = TT tokens x a slice of block-rows; the X tile [TT][columns] is staged in LDS.
//     fp32 tiles hold 32 tokens, and the two halves of a wave take alternate blocks of a row (A
//     broadcast inside each half); bf16 tiles hold 64 tokens and a wave takes every block.
//   * A block-row is cut into units of UB consecutive stored blocks (the last one partial, and at
//     least one per row); the slice's units are split evenly over the 16 waves, each walking its
//     share as one stream with the operands of the next kDepth units in flight, row ends included.
//     A row cut by a wave boundary is finished by the wave that starts it, in wave order.
//   * Inputs too wide for one tile are staged in column chunks.  A row's part of a chunk is found
//     by binary search over its ascending indices (all chunks at once, under the first chunk's
//     loads), and its running sum stays in LDS between chunks.
//   * Slots of a partial unit past the row's end read zero weights and the tile's zero columns, so
//     no infinite X element meets a padding weight.
// The order of every sum depends only on the launch shape: results are bitwise reproducible.
#include <utility>

#include "device_common.h"
#include "mtile_plan.h"
#include "spmm_tiled.h"

namespace bsr {

namespace {

using namespace mtile;

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef short shortx4 __attribute__((ext_vector_type(4)));
typedef unsigned uintx2 __attribute__((ext_vector_type(2)));
typedef unsigned uintx4 __attribute__((ext_vector_type(4)));

constexpr int kDepth = 3;    // units in flight ahead of the one being multiplied
constexpr int kRing = kDepth + 1;

struct MtileItem {
    const void *X;
    int64_t T, ldx;
    const int32_t *indptr;
    const int32_t *indices;
    const void *data;
    const float *bias;
    float *Y;
    int64_t ldy;
    int nnzb, Nb, Kb;
    int num_tiles, slices, XP, chunk_blocks, nchunks;
    int acc_words, bias_words, bound_words, up_words;   // LDS words to each array from the tile
    int stage_words;
};

struct MtileBatch {
    int n;
    MtileItem item[kMaxItems];
};

template <class S>
struct MOps {
    int j;   // column of slot lane % 16 of this half's blocks
    std::conditional_t<S::kBf, shortx4, float> w[S::WL][S::LE];
};

template <int B, int ABID>
__device__ __forceinline__ floatx4 mfma_bcast(float a, float x, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_4x4x1f32(a, x, c, B, ABID, 0);
}
template <int B, int ABID>
__device__ __forceinline__ floatx4 mfma_bcast(shortx4 a, shortx4 x, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(a, x, c, B, ABID, 0);
}

// f(0), f(1), ..., f(N - 1) with constant arguments (ABID is an instruction field).
template <class Fn, int... I>
__device__ __forceinline__ void static_for_each(Fn &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class Fn>
__device__ __forceinline__ void static_for(Fn &&f) {
    static_for_each(f, std::make_integer_sequence<int, N>{});
}

// Lane L of v's 16-lane row, in every lane of the row.
template <int L>
__device__ __forceinline__ unsigned row_bcast(unsigned v) {
    return unsigned(__builtin_amdgcn_mov_dpp(int(v), 0x150 + L, 0xf, 0xf, true));
}

// Y staging.  A finished row is 16 or 32 bytes per token, and the L2 sends such pieces on to memory
// one by one (at 3072 outputs and 4096 tokens in bf16 4x4 blocks, 143 MB of write requests for 50
// MB of Y), so a wave collects kGroup = 16 consecutive outputs per token in LDS and stores 64
// bytes of a token with four adjacent lanes.  The buffer holds 32 tokens at a pitch of 20 words.
// CH: several column chunks (else the tile holds whole rows of X); ST: staged Y stores.
template <int R, int C, bool BF, bool CH, bool ST>
__global__ __launch_bounds__(kNW * 64) void spmm_mtile_kernel(const MtileBatch batch) {
    using S = MShape<R, C, BF>;
    constexpr int TT = S::TT, H = S::H, F = S::F, UB = S::UB, PV = S::PV, RC = S::RC;
    constexpr int CB = H == 2 ? 3 : 4;   // CBSZ: A broadcast over 8 products (a half) or all 16
    extern __shared__ float smem[];
    constexpr int kThreads = kNW * 64;
    const int lane = threadIdx.x & 63, wave = uniform(threadIdx.x >> 6);
    const int t = lane % TT, h = lane / TT;

    const MtileItem &I = batch.item[blockIdx.y];
    const void *__restrict__ X = I.X;
    const int64_t T = I.T, ldx = I.ldx, ldy = I.ldy;
    const int32_t *__restrict__ indptr = I.indptr;
    const int32_t *__restrict__ indices = I.indices;
    const void *__restrict__ data = I.data;
    const float *__restrict__ bias = I.bias;
    float *__restrict__ Y = I.Y;
    const int nnzb = I.nnzb, Nb = I.Nb, Kb = I.Kb, num_tiles = I.num_tiles, slices = I.slices,
              XP = I.XP, kcb = I.chunk_blocks, nchunks = CH ? I.nchunks : 1;

    // Workgroup -> (token tile, slice), in contiguous ranges per XCD as in the other kernels.
    const int g = blockIdx.x, xcd = g & 7, rank = g >> 3;
    const int pairs = num_tiles * slices, per_xcd = (pairs + 7) >> 3;
    const int q = xcd * per_xcd + rank;
    if (rank >= per_xcd || q >= pairs) return;
    const int tile = q / slices, s = q - tile * slices;
    const int64_t t0 = int64_t(tile) * TT;
    const int rows = int(T - t0 < TT ? T - t0 : TT);
    const int row_lo = int(int64_t(s) * Nb / slices), row_hi = int(int64_t(s + 1) * Nb / slices);
    const int nr = row_hi - row_lo;

    // LDS: X tile (between chunks: the waves' head partials); running sums (several chunks);
    // the slice's bias; bounds[c][r], where row r's part of chunk c begins; up[c][r], the units
    // of chunk c before row r; the waves' Y staging buffers.
    unsigned *Xs = reinterpret_cast<unsigned *>(smem);
    float *s_acc = smem + I.acc_words;
    float *s_bias = smem + I.bias_words;
    int *s_bound = reinterpret_cast<int *>(smem) + I.bound_words;
    int *s_up = reinterpret_cast<int *>(smem) + I.up_words;

    // ------------------------------------------------------------------------------- X tile
    // Wave w moves token rows w + 16 r, SW words per lane and load, all loads of up to 1024
    // columns before their LDS stores.  Rows past T read an empty range (zeros).
    constexpr int kXBytes = BF ? 2 : 4;
    constexpr bool kWiden = BF && !S::kBf;
    constexpr int kRows = TT / kNW, SW = S::VW;
    constexpr int kG = 1024 * S::kXs / 4 / 64 / SW;
    typedef unsigned piece __attribute__((ext_vector_type(SW == 1 ? 2 : SW)));
    using XRegs = unsigned[kRows][kG][SW];
    auto x_load = [&](XRegs &v, int jlo, int cols, int w0) {
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            const int tr = wave + kNW * r;
            const __amdgpu_buffer_rsrc_t rx = buffer_rsrc(
                static_cast<const char *>(X) +
                    ((t0 + (tr < rows ? tr : 0)) * ldx + int64_t(jlo) * C) * kXBytes,
                tr < rows ? unsigned(cols) * kXBytes : 0u);
#pragma unroll
            for (int m = 0; m < kG; ++m) {
                const int w = w0 + (64 * m + lane) * SW;
                if constexpr (kWiden) {
                    v[r][m][0] = unsigned(__builtin_amdgcn_raw_buffer_load_b16(rx, w * 2, 0, 0));
                } else if constexpr (SW == 1) {
                    v[r][m][0] = __builtin_amdgcn_raw_buffer_load_b32(rx, w * 4, 0, 0);
                } else if constexpr (SW == 2) {
                    const uintx2 x = __builtin_amdgcn_raw_buffer_load_b64(rx, w * 4, 0, 0);
                    v[r][m][0] = x[0];
                    v[r][m][1] = x[1];
                } else {
                    const uintx4 x = __builtin_amdgcn_raw_buffer_load_b128(rx, w * 4, 0, 0);
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[r][m][e] = x[e];
                }
            }
        }
    };
    auto x_store = [&](const XRegs &v, int words, int w0) {   // words: of a whole row
#pragma unroll
        for (int r = 0; r < kRows; ++r) {
            unsigned *dst = Xs + (wave + kNW * r) * XP;
#pragma unroll
            for (int m = 0; m < kG; ++m) {
                const int w = w0 + (64 * m + lane) * SW;
                if (w < words) {   // whole pieces: words is a multiple of SW
                    if constexpr (SW == 1) {
                        dst[w] = kWiden ? v[r][m][0] << 16 : v[r][m][0];
                    } else {
                        piece x;
#pragma unroll
                        for (int e = 0; e < SW; ++e) x[e] = v[r][m][e];
                        *reinterpret_cast<piece *>(dst + w) = x;
                    }
                }
            }
        }
    };
    // Columns jlo C .. jlo C + cols: the first batch is in v, wider tiles take more passes; then
    // the zero columns that padding slots read.
    auto stage = [&](XRegs &v, int jlo, int cols) {
        const int words = cols * S::kXs / 4;
        x_store(v, words, 0);
        for (int w0 = 64 * SW * kG; w0 < words; w0 += 64 * SW * kG) {
            x_load(v, jlo, cols, w0);
            x_store(v, words, w0);
        }
        constexpr int kZero = C * S::kXs / 4;
        for (int i = threadIdx.x; i < TT * kZero; i += kThreads)
            Xs[(i / kZero) * XP + words + i % kZero] = 0u;
    };

    // --------------------------------------------------------------------------- row tables
    const int cols0 = (CH ? kcb : Kb) * C;
    XRegs xv;
    x_load(xv, 0, cols0, 0);   // in flight under the tables
    for (int i = threadIdx.x; i < nr; i += kThreads) {
        const int p0 = clampi(indptr[row_lo + i], 0, nnzb);
        s_bound[i] = p0;
        s_bound[nchunks * nr + i] = clampi(indptr[row_lo + i + 1], p0, nnzb);
    }
    for (int i = threadIdx.x; i < nr * R; i += kThreads)
        s_bias[i] = bias ? bias[int64_t(row_lo) * R + i] : 0.0f;
    stage(xv, 0, cols0);
    __syncthreads();
    if constexpr (CH) {
        // First position of row r at or past column c kcb, for every boundary between chunks.
        for (int i = threadIdx.x; i < nr * (nchunks - 1); i += kThreads) {
            const int c = i / nr + 1, r = i - (c - 1) * nr, jc = c * kcb;
            int lo = s_bound[r], hi = s_bound[nchunks * nr + r];
            while (lo < hi) {
                const int mid = (lo + hi) >> 1;
                if (indices[mid] < jc) lo = mid + 1; else hi = mid;
            }
            s_bound[c * nr + r] = lo;
        }
        __syncthreads();
    }
    for (int c = wave; c < nchunks; c += kNW) {
        int carry = 0;
        int *up = s_up + c * (nr + 1);
        for (int base = 0; base < nr; base += 64) {
            const int r = base + lane;
            int n = 0;
            if (r < nr) {
                const int len = s_bound[(c + 1) * nr + r] - s_bound[c * nr + r];
                n = len > UB ? (len + UB - 1) / UB : 1;
            }
            const int incl = wave_scan_incl(n) + carry;
            if (r < nr) up[r] = incl - n;
            carry = __builtin_amdgcn_readlane(incl, 63);
        }
        if (lane == 0) up[nr] = carry;
    }
    __syncthreads();

    const int ldy4 = int(ldy) * 4;
    const __amdgpu_buffer_rsrc_t ry = buffer_rsrc(Y + t0 * ldy, unsigned(rows) * unsigned(ldy4));
    [[maybe_unused]] const int vy = t * ldy4 + h * PV * 4;
    // Per-lane byte offsets of the unit's operands from the unit's first block.
    const int vj = (H * (lane & 15) + h) * 4;
    int vw[S::WL];
#pragma unroll
    for (int k = 0; k < S::WL; ++k) {
        const int gi = S::GV * k + (lane % (64 / H)) / 4, i4 = lane & 3;
        const int u = gi / S::GP, f = gi % F, cq = gi % S::GP / F;
        vw[k] = ((H * u + h) * RC + (4 * f + i4) * C + 4 * cq) * S::kEs;
    }
    const char *xrow = reinterpret_cast<const char *>(Xs + t * XP);

    // Staged stores: rows r of the wave that are finished in row order, GR to a group.  Halves
    // (H = 2) write their part of a row to the buffer at once; whole-token lanes keep the group
    // in registers and pass the buffer 32 tokens at a time.
    constexpr int GR = kGroup / R;
    [[maybe_unused]] float *s_y = smem + I.stage_words + wave * kYWords;
    [[maybe_unused]] float pend[H == 1 ? kGroup : 1] = {};
    [[maybe_unused]] int pend_lo = -1, pend_hi = -1;   // pending rows of one group; -1: none
    [[maybe_unused]] auto flush = [&]() {
        const int g0 = pend_lo / GR * GR;
        const int quad = lane & 3, rq = g0 + 4 * quad / R;   // the row of this lane's 16 bytes
        const bool mine = rq >= pend_lo && rq < pend_hi;
#pragma unroll
        for (int part = 0; part < TT / 32; ++part) {
            if constexpr (H == 1) {
                if (lane / 32 == part) {
#pragma unroll
                    for (int e = 0; e < kGroup; e += 4)
                        *reinterpret_cast<floatx4 *>(s_y + (lane & 31) * kYPitch + e) =
                            floatx4{pend[e], pend[e + 1], pend[e + 2], pend[e + 3]};
                }
            }
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int tk = 16 * j + (lane >> 2);
                const uintx4 o =
                    *reinterpret_cast<const uintx4 *>(s_y + tk * kYPitch + 4 * quad);
                if (mine)
                    __builtin_amdgcn_raw_buffer_store_b128(
                        o, ry, (32 * part + tk) * ldy4 + ((row_lo + g0) * R + 4 * quad) * 4, 0, 0);
            }
        }
        pend_lo = -1;
    };
    [[maybe_unused]] auto put = [&](int r, const float (&y)[PV]) {
        const int slot = r % GR;
        if (pend_lo < 0) pend_lo = r;
        pend_hi = r + 1;
        if constexpr (H == 1) {
#pragma unroll
            for (int k = 0; k < GR; ++k) {
#pragma unroll
                for (int e = 0; e < R; ++e) pend[k * R + e] = slot == k ? y[e] : pend[k * R + e];
            }
        } else {
            float *d = s_y + t * kYPitch + slot * R + h * PV;
            if constexpr (PV == 4)
                *reinterpret_cast<floatx4 *>(d) = floatx4{y[0], y[1], y[2], y[3]};
            else
                *reinterpret_cast<floatx2 *>(d) = floatx2{y[0], y[1]};
        }
        if (slot == GR - 1) flush();
    };

    for (int c = 0; c < nchunks; ++c) {
        const int jlo = c * kcb;
        const int kbw = (c + 1 == nchunks ? Kb : jlo + kcb) - jlo;
        const unsigned zoff = unsigned(kbw * C * S::kXs);   // the zero columns
        if (CH && c > 0) {
            x_load(xv, jlo, kbw * C, 0);
            stage(xv, jlo, kbw * C);
            __syncthreads();
        }
        const int *up = s_up + c * (nr + 1);
        const int *b0 = s_bound + c * nr, *b1 = b0 + nr;
        const bool last = !CH || c + 1 == nchunks;

        // A row's sum over this chunk, y (the lane's PV outputs): added to the running sum, and
        // in the last chunk to the bias and stored.
        auto finish = [&](int r, float (&y)[PV]) {
            typedef float pvec __attribute__((ext_vector_type(PV == 2 ? 2 : 4)));
            constexpr int PN = PV == 2 ? 1 : PV / 4, PE = PV == 2 ? 2 : 4;
            float *a = s_acc + (r * 64 + lane) * PV;
            if (CH && c > 0) {
#pragma unroll
                for (int n = 0; n < PN; ++n) {
                    const pvec p = *reinterpret_cast<const pvec *>(a + PE * n);
#pragma unroll
                    for (int e = 0; e < PE; ++e) y[PE * n + e] += p[e];
                }
            }
            if (last) {
                const float *bp = s_bias + r * R + h * PV;
#pragma unroll
                for (int n = 0; n < PN; ++n) {
                    const pvec p = *reinterpret_cast<const pvec *>(bp + PE * n);
#pragma unroll
                    for (int e = 0; e < PE; ++e) y[PE * n + e] += p[e];
                }
                if constexpr (ST) {
                    put(r, y);
                    return;
                }
#pragma unroll
                for (int n = 0; n < PN; ++n) {
                    // The whole offset in the vector offset: with a scalar register in the store's
                    // offset field the compiler leaves out the wait state between a 16-byte store
                    // and the next write of its data registers, and such stores have written the
                    // next row's values (MI355X, last lanes of the last two words).
                    const int vo = vy + ((row_lo + r) * R + PE * n) * 4;
                    if constexpr (PE == 2) {
                        const uintx2 o = {__float_as_uint(y[0]), __float_as_uint(y[1])};
                        __builtin_amdgcn_raw_buffer_store_b64(o, ry, vo, 0, 0);
                    } else {
                        const uintx4 o = {__float_as_uint(y[4 * n]), __float_as_uint(y[4 * n + 1]),
                                          __float_as_uint(y[4 * n + 2]),
                                          __float_as_uint(y[4 * n + 3])};
                        __builtin_amdgcn_raw_buffer_store_b128(o, ry, vo, 0, 0);
                    }
                }
            } else {
#pragma unroll
                for (int n = 0; n < PN; ++n) {
                    pvec p;
#pragma unroll
                    for (int e = 0; e < PE; ++e) p[e] = y[PE * n + e];
                    *reinterpret_cast<pvec *>(a + PE * n) = p;
                }
            }
        };

        // The wave's share [Pw, Pw1) of the chunk's units (lane l: wave l's start ws, and wsn the
        // next wave's), and the rows r0 .. r1 it touches (every row has a unit, so `up` ascends
        // strictly).
        const int total = uniform(up[nr]);
        const int ws = wave_start(0, unsigned(total), unsigned(lane));
        const int wsn = wave_start(0, unsigned(total), unsigned(lane) + 1);
        const int Pw = __builtin_amdgcn_readlane(ws, wave);
        const int Pw1 = __builtin_amdgcn_readlane(wsn, wave);
        auto rows_before = [&](int v) {   // rows whose first unit is < v
            int n = 0;
            for (int base = 0; base < nr; base += 64) {
                const int k = __popcll(__ballot(base + lane < nr && up[min(base + lane, nr)] < v));
                n += k;
                if (k < 64) break;
            }
            return uniform(n);
        };
        float head[PV], tail[PV];
        int head_row = -1, tail_row = -1;
#pragma unroll
        for (int i = 0; i < PV; ++i) head[i] = tail[i] = 0.0f;
        if (Pw < Pw1) {
            const int r0 = rows_before(Pw + 1) - 1, r1 = rows_before(Pw1) - 1;
            if (uniform(up[r0]) < Pw) head_row = r0;
            const bool cut_end = uniform(up[r1 + 1]) > Pw1;
#pragma unroll 1
            for (int gr = r0; gr <= r1; gr += 64) {
                // Rows gr + k, k < ng: lane k holds row k's blocks in the wave's share.
                const int ng = min(64, r1 - gr + 1);
                int pb, pe;
                {
                    const int r = gr + min(lane, ng - 1);
                    const int u0 = up[r], first = b0[r];
                    pb = first + (u0 < Pw ? (Pw - u0) * UB : 0);
                    pe = b1[r];
                    const int cut = first + (Pw1 - u0) * UB;
                    pe = r == r1 && cut < pe ? cut : pe;
                }
                // Load cursor.
                int kl = 0, lp = __builtin_amdgcn_readlane(pb, 0),
                    lend = __builtin_amdgcn_readlane(pe, 0);
                auto load_next = [&](MOps<S> &o) {
                    const __amdgpu_buffer_rsrc_t ri = buffer_rsrc(indices, unsigned(lend) * 4u);
                    const __amdgpu_buffer_rsrc_t rd =
                        buffer_rsrc(data, unsigned(lend) * unsigned(RC * S::kEs));
                    // lp goes into the vector offsets; in the scalar offset, which is range-checked as
                    // well, it measured within 2% either way (3072 x 768, 4096 tokens, 8x1 fp32 42.0
                    // / 41.4 us, bf16 39.0 / 39.3).  A range that starts at lp was slower.
                    o.j = __builtin_amdgcn_raw_buffer_load_b32(ri, vj + lp * 4, 0, 0);
                    const int so = lp * (RC * S::kEs);
#pragma unroll
                    for (int k = 0; k < S::WL; ++k) {
                        if constexpr (S::kBf && S::LE == 2) {
                            const uintx4 v = __builtin_amdgcn_raw_buffer_load_b128(rd, vw[k] + so, 0, 0);
                            o.w[k][0] = __builtin_bit_cast(shortx4, uintx2{v[0], v[1]});
                            o.w[k][1] = __builtin_bit_cast(shortx4, uintx2{v[2], v[3]});
                        } else if constexpr (S::kBf) {
                            o.w[k][0] = __builtin_bit_cast(
                                shortx4, __builtin_amdgcn_raw_buffer_load_b64(rd, vw[k] + so, 0, 0));
                        } else if constexpr (S::LE == 4) {
                            const floatx4 v = __builtin_bit_cast(
                                floatx4, __builtin_amdgcn_raw_buffer_load_b128(rd, vw[k] + so, 0, 0));
#pragma unroll
                            for (int e = 0; e < 4; ++e) o.w[k][e] = v[e];
                        } else if constexpr (BF) {
                            o.w[k][0] = __uint_as_float(
                                unsigned(__builtin_amdgcn_raw_buffer_load_b16(rd, vw[k] + so, 0, 0))
                                << 16);
                        } else {
                            o.w[k][0] = __uint_as_float(
                                __builtin_amdgcn_raw_buffer_load_b32(rd, vw[k] + so, 0, 0));
                        }
                    }
                    lp += UB;
                    if (lp >= lend) {   // the next row; past the last one nothing is read
                        ++kl;
                        lp = kl < ng ? __builtin_amdgcn_readlane(pb, min(kl, 63)) : 0;
                        lend = kl < ng ? __builtin_amdgcn_readlane(pe, min(kl, 63)) : 0;
                    }
                };
                MOps<S> ring[kRing];
#pragma unroll
                for (int d = 0; d < kDepth; ++d) load_next(ring[d]);
                int kc = 0, cp = __builtin_amdgcn_readlane(pb, 0),
                    cend = __builtin_amdgcn_readlane(pe, 0);
                floatx4 acc[F];
#pragma unroll
                for (int f = 0; f < F; ++f) acc[f] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};

                // Slot u's products, for every slot (FULL) or while it has a block in some half.
                auto multiply = [&](const MOps<S> &o, int left, auto full) {
                    constexpr bool FULL = decltype(full)::value;
                    unsigned col =
                        min(unsigned(o.j - jlo), unsigned(kbw - 1)) * unsigned(C * S::kXs);
                    if (!FULL) col = H * (lane & 15) + h < left ? col : zoff;
                    static_for<S::NB>([&](auto uu) {
                        constexpr int u = decltype(uu)::value;
                        if (FULL || H * u < left) {
                            const char *xp = xrow + row_bcast<u>(col);
                            if constexpr (S::kBf) {
                                shortx4 x[C / 4];
                                if constexpr (C == 8) {
                                    const uintx4 v = *reinterpret_cast<const uintx4 *>(xp);
                                    x[0] = __builtin_bit_cast(shortx4, uintx2{v[0], v[1]});
                                    x[1] = __builtin_bit_cast(shortx4, uintx2{v[2], v[3]});
                                } else {
                                    x[0] = *reinterpret_cast<const shortx4 *>(xp);
                                }
                                static_for<C / 4 * F>([&](auto gg) {
                                    constexpr int cq = decltype(gg)::value / F,
                                                  f = decltype(gg)::value % F;
                                    constexpr int gi = u * S::GP + f;
                                    acc[f] = mfma_bcast<CB, gi % S::GV>(o.w[gi / S::GV][cq], x[cq],
                                                                        acc[f]);
                                });
                            } else {
                                float x[C];
#pragma unroll
                                for (int c4 = 0; c4 < C; c4 += 4) {
                                    if constexpr (C >= 4) {
                                        const floatx4 v =
                                            *reinterpret_cast<const floatx4 *>(xp + 4 * c4);
#pragma unroll
                                        for (int e = 0; e < 4; ++e) x[c4 + e] = v[e];
                                    } else {
                                        x[0] = *reinterpret_cast<const float *>(xp);
                                    }
                                }
                                static_for<C * F>([&](auto gg) {
                                    constexpr int cc = decltype(gg)::value / F,
                                                  f = decltype(gg)::value % F;
                                    constexpr int gi = u * S::GP + cc / 4 * F + f;
                                    acc[f] = mfma_bcast<CB, gi % S::GV>(o.w[gi / S::GV][cc % 4],
                                                                        x[cc], acc[f]);
                                });
                            }
                        }
                    });
                };
#pragma unroll 1
                while (kc < ng) {
#pragma unroll
                    for (int ph = 0; ph < kRing; ++ph) {
                        load_next(ring[(ph + kDepth) % kRing]);
                        __builtin_amdgcn_sched_barrier(0);
                        if (kc < ng) {
                            const int left = cend - cp;
                            if (left >= UB) multiply(ring[ph], left, std::true_type{});
                            else multiply(ring[ph], left, std::false_type{});
                            cp += UB;
                            if (cp >= cend) {
                                // The row's end: sum the halves (half 0 + half 1; the swap leaves
                                // half 0's totals of the first outputs on half 0 and of the rest
                                // on half 1), then the row's end or the share's head or tail.
                                float y[PV];
                                if constexpr (H == 2) {
#pragma unroll
                                    for (int i = 0; i < PV; ++i) {
                                        const float P = acc[0][i],
                                                    Q = F == 2 ? acc[F - 1][i] : acc[0][(PV + i) & 3];
                                        const auto sw = __builtin_amdgcn_permlane32_swap(
                                            __float_as_uint(P), __float_as_uint(Q), false, false);
                                        y[i] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
                                    }
                                } else {
#pragma unroll
                                    for (int i = 0; i < PV; ++i) y[i] = acc[i / 4][i % 4];
                                }
                                const int r = gr + kc;
                                if (r == head_row) {
#pragma unroll
                                    for (int i = 0; i < PV; ++i) head[i] = y[i];
                                } else if (r == r1 && cut_end) {
                                    tail_row = r;
#pragma unroll
                                    for (int i = 0; i < PV; ++i) tail[i] = y[i];
                                } else {
                                    finish(r, y);
                                }
#pragma unroll
                                for (int f = 0; f < F; ++f)
                                    acc[f] = floatx4{0.0f, 0.0f, 0.0f, 0.0f};
                                ++kc;
                                cp = kc < ng ? __builtin_amdgcn_readlane(pb, min(kc, 63)) : 0;
                                cend = kc < ng ? __builtin_amdgcn_readlane(pe, min(kc, 63)) : 0;
                            }
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
            }
        }

        if constexpr (ST) {
            if (pend_lo >= 0) flush();
        }

        // Rows cut by wave boundaries: the later waves' head partials go through the dead X
        // tile to the wave that starts the row, which adds them in wave order.
        __syncthreads();
        float *P = smem;
        if (head_row >= 0) {
#pragma unroll
            for (int i = 0; i < PV; ++i) P[(wave * PV + i) * 64 + lane] = head[i];
        }
        __syncthreads();
        if (tail_row >= 0) {
            const int e = uniform(up[tail_row + 1]);
            for (unsigned m = unsigned(__ballot(lane > wave && lane < kNW && ws < e && wsn != ws)); m;
                 m &= m - 1) {
                const int w2 = __ffs(m) - 1;
#pragma unroll
                for (int i = 0; i < PV; ++i) tail[i] += P[(w2 * PV + i) * 64 + lane];
            }
            finish(tail_row, tail);
            if constexpr (ST) {
                if (pend_lo >= 0) flush();
            }
        }
        if (CH && !last) __syncthreads();   // the partials are read; the next chunk may be staged
    }
}

// Least multiply-adds (stored weights x tokens) of a product for this kernel, by the plan that it
// would have in a launch of its own; smaller ones keep the vector-ALU kernels, whose prologue is
// shorter (no unit tables, shares or combine).  Measured on MI355X at a density of 0.1, vector-ALU /
// this kernel in us, 8x8 and 4x4 blocks:
//   fp32  768x768, 777 tokens (46 M): 7.8 / 8.3, 7.4 / 8.4;  3072x768, 777 tokens (183 M):
//         15.8 / 13.8, 17.2 / 15.8;  768x3072 (chunked, 183 M): 21.0 / 20.6, 19.8 / 20.9;
//         3072x768, 4096 tokens: 52.8 / 36.8, 66.3 / 46.1;  768x3072: 76.6 / 45.6, 84.2 / 55.6.
//   bf16  768x768, 128 tokens (7.5 M): 7.6 / 6.6, 6.0 / 7.6;  3072x768, 128 tokens (30 M):
//         9.0 / 7.4, 8.7 / 8.3;  3072x768, 4096 tokens: 93.5 / 18.8, 122 / 25.4.
constexpr int64_t kMinWork = int64_t(128) << 20;
constexpr int64_t kMinWorkChunked = int64_t(192) << 20;
constexpr int64_t kMinWorkBf16 = int64_t(16) << 20;

template <int R, int C, bool BF>
bsr_status launch_shape(const MtileBatch &b, bool chunked, bool staged, dim3 grid, size_t lds,
                        hipStream_t st, const LaunchEvents &ev) {
    const dim3 block(kNW * 64);
    if (chunked)
        launch_kernel(spmm_mtile_kernel<R, C, BF, true, false>, grid, block, lds, st, ev, b);
    else if (staged)
        launch_kernel(spmm_mtile_kernel<R, C, BF, false, true>, grid, block, lds, st, ev, b);
    else
        launch_kernel(spmm_mtile_kernel<R, C, BF, false, false>, grid, block, lds, st, ev, b);
    return launch_status();
}

template <int RR, int CC, bool BB>
struct ShapeTag {
    static constexpr int R = RR, C = CC;
    static constexpr bool BF = BB;
};

// f(tag) for the instantiated shape of a product; nothing for any other.
template <class Fn>
void with_shape(int R, int C, bool bf, Fn &&f) {
#define BSR_MTILE(RR, CC)                     \
    if (R == RR && C == CC) {                 \
        if (bf) f(ShapeTag<RR, CC, true>{});  \
        else f(ShapeTag<RR, CC, false>{});    \
    }
    BSR_MTILE(8, 8)
    BSR_MTILE(4, 4)
    BSR_MTILE(8, 1)
    BSR_MTILE(4, 1)
#undef BSR_MTILE
}

}  // namespace

// The product's launch plan; ok depends on the layer and its arrays, never on the slices.
MtilePlan plan_mtile(const void *X, int64_t T, int64_t ldx, const bsr_matrix_t *W, int64_t ldy,
                     int slices, size_t lds_limit) {
    const int R = W->R, C = W->C;
    const bool bf = W->dtype == BSR_BF16;
    if (W->dtype != BSR_F32 && !bf) return MtilePlan{};
    // 32-bit buffer ranges: the block data, one X row and a tile of Y.
    if (W->nnzb * R * C >= (int64_t(1) << 29)) return MtilePlan{};
    if (ldy >= (int64_t(1) << 23) || W->n_cols >= (int64_t(1) << 24)) return MtilePlan{};
    // bf16 tiles move X in words and weights in 8-byte pieces.
    if (bf && C > 1 &&
        ((reinterpret_cast<uintptr_t>(X) & 3) != 0 || (ldx & 1) != 0 ||
         (reinterpret_cast<uintptr_t>(W->data) & 7) != 0))
        return MtilePlan{};
    MtilePlan p{};
    with_shape(R, C, bf, [&](auto tag) {
        using G = decltype(tag);
        p = plan_shape<G::R, G::C, G::BF>(T, W, slices, lds_limit);
    });
    return p;
}

MtilePlan route_mtile(const bsr_spmm_item_t &it, int slices, int cus, size_t lds_limit) {
    const bool bf = it.W->dtype == BSR_BF16;
    // Too little work whatever the plan: nothing is planned.  (Small calls are bound by the host: eight
    // products of 368 x 133 in 8x1 blocks with 2 tokens took 7.5 us with a trial plan each.)
    const double macs = double(it.W->nnzb) * it.W->R * it.W->C * double(it.T);
    static_assert(kMinWork <= kMinWorkChunked, "the least work of an fp32 product");
    if (macs < double(bf ? kMinWorkBf16 : kMinWork)) return MtilePlan{};
    MtilePlan p = plan_mtile(it.X, it.T, it.ldx, it.W, it.ldy, 1, lds_limit);
    if (!p.ok) return p;
    const int64_t tiles = (it.T + p.tokens - 1) / p.tokens;
    p = plan_mtile(it.X, it.T, it.ldx, it.W, it.ldy,
                   slices > 0 ? slices : auto_slices(&tiles, 1, cus), lds_limit);
    if (!bf && p.nchunks > 1 && macs < double(kMinWorkChunked)) return MtilePlan{};
    return p;
}

bsr_status launch_spmm_mtile(const MtileWork *work, int n, void *stream, const LaunchEvents &ev) {
    if (n < 1 || n > kMaxItems) return BSR_ERR_ARG;
    for (int i = 0; i < n; ++i)
        if (!work[i].plan.ok) return BSR_ERR_UNSUPPORTED;
    const int R = work[0].W->R, C = work[0].W->C, dtype = work[0].W->dtype;
    MtileBatch batch{};
    batch.n = n;
    int gx = 0;
    size_t lds = 0;
    bool chunked = false;   // whole-row products of a mixed launch run as one chunk
    bool staged = true;
    for (int i = 0; i < n; ++i) {
        const MtileWork &w = work[i];
        chunked = chunked || w.plan.nchunks > 1;
        staged = staged && w.plan.stage_words > 0;
        if (w.W->R != R || w.W->C != C || w.W->dtype != dtype) return BSR_ERR_ARG;
        MtileItem &it = batch.item[i];
        it.X = w.X;
        it.T = w.T;
        it.ldx = w.ldx;
        it.indptr = w.W->indptr;
        it.indices = w.W->indices;
        it.data = w.W->data;
        it.bias = w.bias;
        it.Y = w.Y;
        it.ldy = w.ldy;
        it.nnzb = int(w.W->nnzb);
        it.Nb = int(w.W->n_rows / R);
        it.Kb = int(w.W->n_cols / C);
        it.num_tiles = w.plan.num_tiles;
        it.slices = w.plan.slices;
        it.XP = w.plan.x_pitch;
        it.chunk_blocks = w.plan.chunk_blocks;
        it.nchunks = w.plan.nchunks;
        it.acc_words = w.plan.acc_words;
        it.bias_words = w.plan.bias_words;
        it.bound_words = w.plan.bound_words;
        it.up_words = w.plan.up_words;
        it.stage_words = w.plan.stage_words;
        const int wgs = ((w.plan.num_tiles * w.plan.slices + 7) / 8) * 8;
        if (wgs > gx) gx = wgs;
        if (w.plan.lds_bytes > lds) lds = w.plan.lds_bytes;
    }
    bsr_status s = BSR_ERR_UNSUPPORTED;
    with_shape(R, C, dtype == BSR_BF16, [&](auto tag) {
        using G = decltype(tag);
        s = launch_shape<G::R, G::C, G::BF>(batch, chunked, staged, dim3(gx, n), lds, as_stream(stream), ev);
    });
    return s;
}

}  // namespace bsr
