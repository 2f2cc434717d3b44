// Checks tl::join_rows (csrc/tl_unpack.hpp) on rows of every short length and of lengths up to the largest there is.
#include "tl_unpack.hpp"

#include <cstdio>

static uint32_t code(uint64_t row, uint64_t k) { return uint32_t((row * 7 + k * 5 + (k >> 3)) % 3); }

int main()
{
    for (uint64_t span = 0; span < 80; ++span) {
        const uint64_t K = span < 48 ? span + 1 : 0x7fffffffull - (span - 48);
        for (uint32_t left = 1; left < 16 && left <= K; ++left) {
            // rows the 16 codes reach beyond the first, in 64 bits
            const uint64_t reach = (16 - left + K - 1) / K;
            uint32_t want = 0;
            for (uint32_t j = 0; j < 16; ++j) {
                const uint64_t at = K - left + j;
                want |= code(at / K, at % K) << (2 * j);
            }
            auto sixteen = [&](uint64_t row, uint64_t k0) {        // past the row: anything
                uint32_t c = 0;
                for (uint32_t j = 0; j < 16; ++j) c |= (k0 + j < K ? code(row, k0 + j) : 3u) << (2 * j);
                return c;
            };
            uint64_t asked = 0;
            bool outside = false;
            const uint32_t got = tl::join_rows(sixteen(0, K - left), left, uint32_t(K), [&](int i) {
                ++asked;
                if (uint64_t(i) > reach) { outside = true; return 0u; }
                return sixteen(uint64_t(i), 0);
            });
            if (got != want || outside || asked != reach) {
                std::printf("K = %llu, left = %u: %08x instead of %08x, %llu rows asked for instead of %llu\n", (unsigned long long)K, left, got, want,
                            (unsigned long long)asked, (unsigned long long)reach);
                return 1;
            }
        }
    }
    std::puts("ok");
    return 0;
}
