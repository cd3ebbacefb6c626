// Keys of blocks by plain sums, and of one block of 2^32 elements (one row of ones, pitch 0).
#include <cmath>
#include <cstdio>
#include <cstring>
#include <vector>

#include "prune_key.h"

static double value(unsigned long long bits) {
    double d;
    std::memcpy(&d, &bits, 8);
    return d;
}

int main() {
    for (int R : {1, 2, 3, 8, 32})
        for (int C : {1, 2, 5, 16, 33}) {
            const int64_t ldw = C + 3;
            std::vector<float> w(size_t(ldw) * R);
            for (size_t i = 0; i < w.size(); ++i) w[i] = float(int(i * 37 % 101) - 50) * 0.37f;
            double l1 = 0.0, l2 = 0.0;
            for (int r = 0; r < R; ++r)
                for (int c = 0; c < C; ++c) {
                    const double x = w[size_t(r * ldw + c)];
                    l1 += std::fabs(x);
                    l2 = std::fma(x, x, l2);
                }
            if (value(bsr::block_key<true>(w.data(), ldw, R, C)) != l1 ||
                value(bsr::block_key<false>(w.data(), ldw, R, C)) != l2) {
                std::printf("key of a %dx%d block\n", R, C);
                return 1;
            }
        }
    const std::vector<float> ones(65536, 1.0f);
    const double sum = value(bsr::block_key<true>(ones.data(), 0, 65536, 65536));
    if (sum != 4294967296.0) {
        std::printf("a block of 2^32 ones has the key %.1f\n", sum);
        return 1;
    }
    std::printf("ok\n");
    return 0;
}
