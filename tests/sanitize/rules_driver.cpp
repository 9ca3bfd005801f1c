// rules_driver.cpp -- the launch rules that are plain functions of sizes
// (csrc/nn_kernels.hpp and its neighbours), on the CPU: what a rule promises
// over its whole range, checked at both sides of every line it draws.  Built by
// tests/test_launch_rules.py with a host compiler only; test infrastructure.
#include <stdint.h>
#include <stdio.h>

#include "nn_kernels.hpp"

static int fails = 0;
#define CHECK(c)                                                                  \
    do {                                                                          \
        if (!(c)) {                                                               \
            if (fails < 20) fprintf(stderr, "FAIL %s:%d: %s\n", __FILE__, __LINE__, #c); \
            ++fails;                                                              \
        }                                                                         \
    } while (0)

// Workgroups per compute unit of the fused consumer: each ends in one atomic
// on the same address, about 12 ns one after another.
static void consume_workgroups() {
    for (uint32_t block = 64; block <= 1024; block += 64) {
        for (uint64_t count : {1ull, 32769ull, 10000019ull, (1ull << 27) - 1}) {
            const uint32_t per = nn::consume_per_cu(block, count);
            CHECK(per >= 1 && per * block <= 1024);
            // 8 per compute unit with 256 CUs are 25 us of atomics
            CHECK(per <= 8);
        }
        for (uint64_t count : {1ull << 27, 1ull << 30, 1ull << 40}) {
            const uint32_t per = nn::consume_per_cu(block, count);
            CHECK(per >= 2 && per * block <= 2048);
        }
    }
    CHECK(nn::consume_per_cu(1024, 1) == 1 && nn::consume_per_cu(1024, 1ull << 27) == 2);
}

int main() {
    consume_workgroups();
    if (fails) {
        fprintf(stderr, "%d check(s) failed\n", fails);
        return 1;
    }
    printf("rules driver ok\n");
    return 0;
}
