// rules_driver.cpp -- the launch rules that are plain functions of sizes
// (csrc/nn_kernels.hpp and its neighbours), on the CPU: what a rule promises
// over its whole range, checked at both sides of every line it draws.  Built by
// tests/test_launch_rules.py with a host compiler only; test infrastructure.
#include <stdint.h>
#include <stdio.h>

#include "nn_batch.hpp"
#include "nn_e40.hpp"
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

// Plans that name no kernel: a workgroup per record fits one launch, whose
// threads are counted in 32 bits, and the records of both slots stay within 512
// MiB; every launch of the chunked kernels fits as well.
static void batch_capacity() {
    const uint64_t outs[] = {0, 2047, 2048, 1ull << 32, (1ull << 35) - (1 << 16), 1ull << 35,
                             1ull << 40, 1ull << 45};
    const uint64_t descs[] = {1, 10000, 1ull << 22, (1ull << 23) - 1, 1ull << 23, 0xffffffffull};
    for (uint64_t o : outs)
        for (uint64_t d : descs)
            if (nn::chunks_implied(o, d)) {
                CHECK(nn::chunk_records(o, d) * 256 < 1ull << 32);
                CHECK(nn::chunk_records(o, d) * 2 * sizeof(nn::RowRec) < 1ull << 29);
            }
    CHECK(nn::chunks_implied(1ull << 32, 10000 + 257));
    CHECK(!nn::chunks_implied(1ull << 40, 1) && !nn::chunks_implied(1ull << 45, 1));
    CHECK(!nn::chunks_implied(1, 1ull << 23));
    for (uint64_t r : {1ull, 2ull, (1ull << 24) - 1, 1ull << 24, (1ull << 24) + 5, 1ull << 33}) {
        CHECK(nn::chunk_grid(r) >= 1 && nn::chunk_grid(r) <= r);
        CHECK((uint64_t)nn::chunk_grid(r) * 256 < 1ull << 32);
        CHECK(r >= 1ull << 24 || nn::chunk_grid(r) == r);
    }
}

// Windows out of order are sorted on the host only where the kernel's time is
// long beside it: never with non-temporal stores, nor for short windows.
static void batch_order() {
    for (uint64_t n : {129ull, 9999ull, 1ull << 20}) {
        CHECK(!nn::batch_sorts(true, n * 1000, n));
        CHECK(!nn::batch_sorts(false, n * 4, n));
        CHECK(!nn::batch_sorts(false, n * 32 - 1, n) && nn::batch_sorts(false, n * 32, n));
    }
}

// Modulus 3^40, flat layout: the residency cap goes with the rows actually taken
// (a caller's or the size rule's), fewer workgroups the longer their chunks.
static void e40_shapes() {
    namespace e = nn::e40;
    for (int kind = 0; kind < 2; ++kind)
        for (bool nt : {false, true})
            for (uint32_t rows = 2; rows <= 32; rows *= 2) {
                CHECK(e::flat_occupancy(0, kind, nt, rows) == 4);
                const uint32_t cap = e::flat_occupancy(1, kind, nt, rows);
                CHECK(cap >= 2 && cap <= 16 && cap * rows >= 12 && cap * rows <= 64);
                CHECK(rows == 2 || cap <= e::flat_occupancy(1, kind, nt, rows / 2));
            }
    for (int kind = 0; kind < 2; ++kind)
        for (uint64_t count : {1ull, 200003ull, 3000017ull, (1ull << 22) - 1, 1ull << 22,
                               1ull << 23, 1ull << 30}) {
            const uint32_t most = e::flat_rows(kind, 1), rows = e::flat_rows_for(most, count, 256);
            CHECK(rows >= 2 && rows <= most);
            CHECK(rows == 2 || count / (512 * rows) >= 512);
            CHECK(rows == most || count / (1024 * rows) < 512);
        }
}

int main() {
    e40_shapes();
    batch_order();
    consume_workgroups();
    batch_capacity();
    if (fails) {
        fprintf(stderr, "%d check(s) failed\n", fails);
        return 1;
    }
    printf("rules driver ok\n");
    return 0;
}
