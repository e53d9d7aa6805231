// Which fully connected layers XNOR_ALGO_AUTO gives to linear_popcount_kernel.  Plain integers, no HIP headers: a host
// compiler can check the rule against measurements.
#pragma once
#include <stdint.h>

namespace xnor {

// Packed words per load, and words of a row that one pass of the 16 lanes covers (linear_popcount_kernel).
constexpr int linear_words_per_load(int cw) { return cw % 4 == 0 ? 4 : cw % 2 == 0 ? 2 : 1; }
constexpr int linear_words_per_pass(int v) { return v == 4 ? 320 : v == 2 ? 256 : 128; }

// n rows of c features (cw words), k filters; matrix_image: the caller gave the images of the matrix-core forms.
//
// A workgroup holds two rows (one if there is only one) and 16 filters whether they exist or not, so the time follows the
// padded product: 2.5 us + rows * filters * passes over the row * 0.052 ns with 4 words per load (0.083 ns with 2, 0.032 ns
// with 1; measured from 8192 to 2^20 padded products, 32 to 131072 features).
// With an image, rows of up to three words are against the matrix-core convolution, 4 to 5 us whatever rows and filters (rows x filters, c,
// us back to back): 2048 x 8, 96 3.2 / 4.3, 300 x 100, 96 3.6 / 4.3, 64 x 512, 32 3.3 / 4.2, 1000 x 30, 40 5.1 / 4.2, 9000 x 3, 96 7.1 / 4.7.  One or
// two rows, where nothing is padded, are ahead but for 1 x 32768, 64: 6.0 / 5.0.  Longer rows come here only where the images pass what
// linear_words_kernel and the convolution address (2 GiB).
inline bool linear_popcount_route(int n, int k, int c, int cw, bool matrix_image)
{
    // rows times filters: beyond these no shape was measured ahead
    const int64_t pairs = (int64_t)n * k;
    if (n > 65535 || pairs > (c >= 4096 ? 131072 : c >= 2048 ? 65536 : 32768)) return false;       // (n: grid limit)
    if (n <= 2) return true;
    const int v = linear_words_per_load(cw), pass = linear_words_per_pass(v);
    const int64_t padded = ((int64_t)n + 1) / 2 * 2 * (((int64_t)k + 15) / 16 * 16);
    const int64_t cost = padded * ((cw + pass - 1) / pass) * (v == 4 ? 8 : v == 2 ? 13 : 5) / 8;
    // against the vector-ALU convolution (5.3 us + 6.5 ns per feature: 32768 x 1, 512: 30.8 / 7.4, 2048: 31.0 / 18.7,
    // 4096: 30.6 / 32.1)
    if (!matrix_image) return cost <= 53500 + 124 * (int64_t)c;
    return cw > 320 || cost <= 40960 + 15 * (int64_t)c;
}

// Rows of four packed words and more with a matrix image have a third form, linear_words_kernel.  Its tiles (filters, rows of 32): what a
// CU's rounds of workgroups cost, in fifths of a round of 1 x 1 (rows x filters, c: 1 x 1 / 2 x 1 / 2 x 2, us back to back: 64 x 4096,
// 9216 4.9 / 6.0 / 7.8; 128 x 4096, 9216 7.3 / 6.5 / 8.3; 256 x 4096, 9216 11.9 / 10.4 / 9.1; 256 x 4096, 4096 7.3 / 6.7 / 6.5; 256 x 1000,
// 4096 4.2 / 4.6 / 5.7).
struct LinearWordsTile { int filters, rows; int64_t cost; };
inline LinearWordsTile linear_words_tile(int n, int k)
{
    const LinearWordsTile tiles[] = {{1, 1, 5}, {2, 1, 8}, {2, 2, 12}};
    LinearWordsTile best{0, 0, INT64_MAX};
    for (const LinearWordsTile &t : tiles) {
        const int64_t wgs = (((int64_t)k + 32 * t.filters - 1) / (32 * t.filters)) * (((int64_t)n + 32 * t.rows - 1) / (32 * t.rows));
        const int64_t cost = (wgs + 255) / 256 * t.cost;
        if (cost < best.cost) best = {t.filters, t.rows, cost};
    }
    return best;
}
// Few rows against it, both in graphs of one kernel: the few-rows kernel 2.1 us + padded product * passes * 0.055 ns (as above), the other
// 2.4 us and 0.2 us per 1024 features for a round of 1 x 1, 1.1 us and as many features' worth for every further one.  us, few rows /
// words: 8 x 4096, 4096 features 3.8 / 3.2, 9216 3.8 / 4.1; 4 x 4096, 4096 2.9 / 3.2; 16 x 1000, 1024 2.9 / 2.6; 256 x 100, 4096 3.8 / 3.4,
// 9216 3.8 / 4.3; 32 x 4096, 9216 9.4 / 4.3; 1 x 4096, 9216 2.3 / 4.1; 64 x 1000, 25088 12.8 / 7.4.  Timed again on 252 shapes of 1 to 65535 rows and
// 97 to 131072 features, one of them is chosen more than 10 % behind (5 x 3237, 34701 10.4 / 9.3), 0.3 % in the mean.
inline bool linear_few_rows_ahead_of_words(int n, int k, int c, int cw)
{
    if (n > 65535) return false;                                   // (grid limit)
    const int v = linear_words_per_load(cw), pass = linear_words_per_pass(v);
    const int64_t padded = (n == 1 ? 1 : ((int64_t)n + 1) / 2 * 2) * (((int64_t)k + 15) / 16 * 16);
    if (padded > (1ll << 32)) return false;
    const int64_t cost = padded * ((cw + pass - 1) / pass) * (v == 4 ? 8 : v == 2 ? 13 : 5) / 8;
    const int64_t r = linear_words_tile(n, k).cost;
    return cost <= 3978 * r - 14466 + (int64_t)c * r * 706 / 1000;
}

}  // namespace xnor
