// Host-side check of csrc/fastdiv.h: SmallDiv::div against x / d for every x up to the bound it was made for, over the
// divisors and bounds of the kernels' tiles; prints the mismatches and the refusals.  Run by tests/test_fastdiv_small.py.
#include "fastdiv.h"
#include <cstdio>
#include <initializer_list>

int main()
{
    using xnor::SmallDiv;
    unsigned long long bad = 0, made = 0;
    for (uint32_t d = 1; d < 3000; d += d < 70 ? 1 : 37)
        for (uint64_t max : {0ull, 10ull, 100ull, 857ull, 5000ull, 60000ull, 1000000ull, 16000000ull}) {
            SmallDiv s;
            if (!SmallDiv::make(d, max, &s)) continue;
            ++made;
            for (uint64_t x = 0; x <= max; x += max > 100000 && x < max - 3000 ? 101 : 1) bad += s.div((uint32_t)x) != x / d;
        }
    SmallDiv s;
    // the planes of the benchmark layers with a tile beyond them are never refused; what cannot be exact is
    for (uint32_t w : {1u, 2u, 7u, 13u, 14u, 27u, 28u, 56u, 112u, 224u})
        if (!SmallDiv::make(w, (uint64_t)w * w + 256, &s)) ++bad;
    if (SmallDiv::make(3, 1u << 24, &s) || SmallDiv::make(0, 5, &s)) ++bad;
    std::printf("made %llu mismatches %llu\n", made, bad);
    return bad != 0 || made < 500;
}
