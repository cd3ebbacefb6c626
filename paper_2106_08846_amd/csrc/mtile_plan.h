// Launch planning of the small-block matrix kernel (spmm_mtile.hip): pure C++, so that it also runs
// where no GPU exists.
#pragma once

#include "spmm_tiled.h"

namespace bsr {

namespace mtile {

constexpr int kNW = 16;      // waves per workgroup

template <int R, int C, bool BF>
struct MShape {
    static constexpr bool kBf = BF && C % 4 == 0;   // bf16 matrix instructions, bf16 tile
    static constexpr int TT = kBf ? 64 : 32;        // tokens per tile
    static constexpr int H = 64 / TT;               // halves of a wave, on alternate blocks
    static constexpr int F = R / 4;                 // groups of four rows
    // A lane's weight load: LE instruction operands of one row, 16 bytes of it where a block's
    // rows are that long (with 4-byte loads of 32-byte strided words the fp32 8x8 kernel waited
    // on the texture addresser).  GP groups of 4 lanes (rows 4 f .. 4 f + 3) load a block.
    static constexpr int LE = kBf ? C / 4 : (C >= 4 ? 4 : 1);
    static constexpr int GP = (!kBf && C > 4 ? C / 4 : 1) * F;
    static constexpr int GV = 16 / H;               // groups per half in one load
    static constexpr int WL = C == 1 ? 2 : 1;       // weight loads per unit
    static constexpr int NB = GV * WL / GP;         // blocks per half and unit
    static constexpr int UB = H * NB;               // blocks per unit
    static constexpr int RC = R * C;
    static constexpr int kEs = BF ? 2 : 4;          // bytes per stored weight
    static constexpr int kXs = kBf ? 2 : 4;         // bytes per X element in the tile
    static constexpr int VW = C * kXs >= 16 ? 4 : C * kXs / 4;   // words per LDS read of X
    static constexpr int PV = R * TT / 64;          // outputs per lane once the halves are summed
    static_assert(NB <= 16 && NB * GP == GV * WL && (R == 4 || R == 8));
};

// Words (4 bytes) between token rows of a tile of `cols` columns: the columns and C zero ones,
// rounded so that reads of VW words by consecutive tokens start VW banks apart (mod 2 VW).
template <class S>
int64_t tile_words(int64_t cols, int C) {
    const int64_t w = ((cols + C) * S::kXs + 3) / 4;
    return w + (((S::VW - w) % (2 * S::VW)) + 2 * S::VW) % (2 * S::VW);
}

// Y staging: a wave collects kGroup consecutive outputs of 32 tokens at a pitch of kYPitch words.
constexpr int kGroup = 16;
constexpr int kYPitch = 20;
constexpr int kYWords = 32 * kYPitch;   // per wave

// The layout of a product for `slices` wanted slices: as few chunks as fit with them; more slices
// (smaller tables and running sums), doubling up to one block-row each, only when no chunk count
// fits.  Every array shrinks with the rows per slice and one block-row per slice is always tried, so
// whether a product fits (p.ok) does not depend on the wanted slices: a kernel chosen with one count
// can be launched with another.
template <int R, int C, bool BF>
MtilePlan plan_shape(int64_t T, const bsr_matrix_t *W, int slices, size_t lds_limit) {
    using S = MShape<R, C, BF>;
    MtilePlan p{};
    p.tokens = S::TT;
    const int64_t K = W->n_cols, Nb = W->n_rows / R, Kb = K / C;
    constexpr int64_t kPartials = int64_t(kNW) * S::PV * 64;   // words
    auto a4 = [](int64_t w) { return (w + 3) & ~int64_t(3); };
    constexpr int kMaxChunks = 16;
    const int64_t wanted = slices > 0 ? slices : 1;
    for (int64_t Su = wanted < Nb ? wanted : Nb;; Su = 2 * Su < Nb ? 2 * Su : Nb) {
        const int64_t nr = (Nb + Su - 1) / Su;
        for (int64_t nch = 1; nch <= kMaxChunks && nch <= Kb; ++nch) {
            const int64_t kcb = (Kb + nch - 1) / nch;
            if (kcb * (nch - 1) >= Kb) continue;   // the last chunk would be empty
            const int64_t xp = tile_words<S>(kcb * C, C);
            // Running sums take at most a third of LDS (more slices rather than narrower chunks).
            if (nch > 1 && nr * 64 * S::PV * 4 > int64_t(lds_limit) / 3) break;
            int64_t w = a4(S::TT * xp > kPartials ? S::TT * xp : kPartials);
            const int64_t acc = w;
            if (nch > 1) w += nr * 64 * S::PV;
            const int64_t bias = w;
            w += a4(nr * R);
            const int64_t bound = w;
            w += a4(nr * (nch + 1));
            const int64_t up = w;
            w = a4(w + nch * (nr + 1));
            if (w * 4 > int64_t(lds_limit)) continue;
            // Staging buffers where the rest leaves room (they do
            // beside tiles of 768 columns, fp32 or bf16).
            if (nch == 1 && (w + kNW * kYWords) * 4 <= int64_t(lds_limit)) {
                p.stage_words = int(w);
                w += kNW * kYWords;
            }
            p.x_pitch = int(xp);
            p.chunk_blocks = int(kcb);
            p.nchunks = int(nch);
            p.acc_words = int(acc);
            p.bias_words = int(bias);
            p.bound_words = int(bound);
            p.up_words = int(up);
            p.lds_bytes = size_t(w) * 4;
            p.slices = int(Su);
            p.num_tiles = int((T + S::TT - 1) / S::TT);
            p.ok = true;
            return p;
        }
        if (Su == Nb) return MtilePlan{};
    }
}

}  // namespace mtile

}  // namespace bsr
