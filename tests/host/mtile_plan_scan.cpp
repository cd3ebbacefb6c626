// Scan of the small-block matrix kernel's planner over layer sizes and slice counts: a layer that
// fits with one wanted slice fits with any, the search ends for every wanted count, and a plan's LDS
// arrays follow each other inside the limit and its chunks cover the columns.
#include <cstdio>
#include <cstdlib>
#include <set>

#include "mtile_plan.h"

static long plans = 0;

static void fail(const char *what, int R, int C, bool bf, int64_t N, int64_t K, int S) {
    std::printf("%s: %dx%d %s N=%lld K=%lld slices=%d\n", what, R, C, bf ? "bf16" : "f32",
                (long long)N, (long long)K, S);
    std::exit(1);
}

template <int R, int C, bool BF>
static void layer(int64_t N, int64_t K, int64_t T) {
    using S = bsr::mtile::MShape<R, C, BF>;
    const size_t limit = 160 * 1024;
    const int64_t Nb = N / R, Kb = K / C;
    bsr_matrix_t W{};
    W.n_rows = N;
    W.n_cols = K;
    W.R = R;
    W.C = C;
    W.nnzb = Nb * Kb / 20 > 0 ? Nb * Kb / 20 : 1;
    W.dtype = BF ? BSR_BF16 : BSR_F32;
    std::set<int> counts = {1, 2, 3, 5, 6, 7, 12, 23, 48, 200, int(Nb), int(Nb) + 1, int(2 * Nb)};
    if (Nb > 1) counts.insert(int(Nb) - 1);
    const bool fits = bsr::mtile::plan_shape<R, C, BF>(T, &W, 1, limit).ok;
    for (int s : counts) {
        const bsr::MtilePlan p = bsr::mtile::plan_shape<R, C, BF>(T, &W, s, limit);
        ++plans;
        if (p.ok != fits) fail(fits ? "fits with one slice only" : "does not fit with one slice",
                               R, C, BF, N, K, s);
        if (!p.ok) continue;
        const int64_t nr = (Nb + p.slices - 1) / p.slices;
        if (p.slices < 1 || p.slices > Nb || p.slices < (s < Nb ? s : Nb) ||
            int64_t(p.num_tiles) * S::TT < T)
            fail("slices or tiles", R, C, BF, N, K, s);
        if (p.nchunks < 1 || int64_t(p.chunk_blocks) * p.nchunks < Kb ||
            int64_t(p.chunk_blocks) * (p.nchunks - 1) >= Kb)
            fail("chunks do not cover the columns", R, C, BF, N, K, s);
        // Words: the X tile (with the zero columns) or the partials, running sums, bias, bounds,
        // units before each row, Y staging.
        const int64_t tile = int64_t(S::TT) * p.x_pitch, part = int64_t(bsr::mtile::kNW) * S::PV * 64;
        if (int64_t(p.x_pitch) * 4 < (int64_t(p.chunk_blocks) + 1) * C * S::kXs)
            fail("pitch", R, C, BF, N, K, s);
        int64_t end = tile > part ? tile : part;
        const int64_t need[][2] = {{p.acc_words, p.nchunks > 1 ? nr * 64 * S::PV : 0},
                                   {p.bias_words, nr * R},
                                   {p.bound_words, nr * (p.nchunks + 1)},
                                   {p.up_words, p.nchunks * (nr + 1)},
                                   {p.stage_words, int64_t(bsr::mtile::kNW) * bsr::mtile::kYWords}};
        for (int i = 0; i < (p.stage_words > 0 ? 5 : 4); ++i) {
            if (need[i][0] < end) fail("arrays overlap", R, C, BF, N, K, s);
            end = need[i][0] + need[i][1];
        }
        if (end * 4 > int64_t(p.lds_bytes) || p.lds_bytes > limit)
            fail("LDS bytes", R, C, BF, N, K, s);
    }
}

template <int R, int C>
static void shape() {
    for (int64_t nb : {1, 3, 4, 5, 7, 32, 96, 112, 128, 130, 140, 256, 384, 768})
        for (int64_t k : {8, 96, 768, 1024, 1232, 1240, 1248, 1256, 1264, 1272, 1280, 1536, 2304, 2520,
                          3072, 4096, 6144, 16384, 19720, 19728, 19744, 19976, 20000, 20136, 20160,
                          39000, 40000, 100000}) {
            layer<R, C, false>(nb * R, k, 2560);
            layer<R, C, true>(nb * R, k, 700);
            if (C == 1) {
                layer<R, C, false>(nb * R, k + 3, 2560);
                layer<R, C, true>(nb * R, k + 2, 700);
            }
        }
}

int main() {
    shape<8, 8>();
    shape<4, 4>();
    shape<8, 1>();
    shape<4, 1>();
    std::printf("ok %ld plans\n", plans);
    return 0;
}
