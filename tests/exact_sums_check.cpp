// Host check of sum_of_words (logfx_bits.h): totals below 2^96 split into a
// low and a high word in many ways, as different tilings of one image split
// them, give one double each, within one part in 2^52 of the total.  Exit
// status 0 when all agree.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <random>

#include "logfx_bits.h"

int main() {
    std::mt19937_64 rng(7);
    long bad = 0;
    for (int i = 0; i < 200000; ++i) {
        const uint64_t high = rng() >> (4 + rng() % 40), low = rng() >> 32;
        const double want = logfx::kern::sum_of_words(low, high);
        const long double exact = (long double)high * 4294967296.0L + (long double)low;
        bad += std::fabs((double)((want - exact) / exact)) > 0x1p-52;
        for (int k = 0; k < 8; ++k) {
            // move up to 2^29 units of 2^32 (or all there are) back to the low word
            const uint64_t move = std::min(high, rng() >> (35 + rng() % 20));
            bad += logfx::kern::sum_of_words(low + (move << 32), high - move) != want;
        }
    }
    std::printf("%ld mismatches\n", bad);
    return bad == 0 ? 0 : 1;
}
