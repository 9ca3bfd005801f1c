// steps_driver.cpp -- the two FP64 steps that the default kernels run,
// chained as the kernels chain them: balanced states modulo 3^33 (mm_bal,
// csrc/nn_arith.hpp) and three balanced limbs modulo 3^40 (mul40t,
// csrc/nn_e40.hpp).  Their proofs rest on bounds of states that only chaining
// produces (beyond m/2 at 3^33), so every step checks the bounds as well as
// the value, against 128-bit integer products and the oracle.  Built by
// tests/test_steps_sanitized.py under AddressSanitizer and
// UndefinedBehaviorSanitizer with a host compiler only; test infrastructure.
#include <math.h>
#include <stdint.h>
#include <stdio.h>

#include "nn_e40.hpp"
#include "nn_host.hpp"

extern "C" {
#include "nn_oracle.h"
}

typedef __int128 i128;

static int fails = 0;
#define CHECK(c)                                                                  \
    do {                                                                          \
        if (!(c)) {                                                               \
            if (fails < 20) fprintf(stderr, "FAIL %s:%d: %s\n", __FILE__, __LINE__, #c); \
            ++fails;                                                              \
        }                                                                         \
    } while (0)

static uint64_t rng = 0x9E3779B97F4A7C15ULL;
static uint64_t next64() {  // xorshift64*
    rng ^= rng >> 12;
    rng ^= rng << 25;
    rng ^= rng >> 27;
    return rng * 0x2545F4914F6CDD1DULL;
}

static uint64_t unit(uint64_t m) {  // a random unit modulo a power of 3
    for (;;) {
        const uint64_t z = 1 + next64() % (m - 1);
        if (z % 3) return z;
    }
}

// ------------------------------------------------------------ modulo 3^33 --

static const double kM = (double)ORC_MOD;

static bool is_int(double x) { return x == rint(x); }

// One balanced step of any admissible r: exact, and its bound closes.
static void check_bal(double r, uint64_t v) {
    const nn::BalMult f = nn::make_bal(v);
    CHECK(is_int(f.v) && fabs(f.v) < 0.5 * kM && fabs(f.q) < 0.5);
    const double out = nn::mm_bal(r, f);
    CHECK(is_int(out) && fabs(out) < 0.593 * kM);
    const i128 m = ORC_MOD;
    CHECK(((i128)(int64_t)r * (i128)v - (i128)(int64_t)out) % m == 0);
}

static void balanced_steps() {
    const uint64_t m = ORC_MOD;
    // multipliers at the ends of the balanced range, and states at the ends of
    // theirs (0.6 m in magnitude, where a chain's never come)
    uint64_t vs[40];
    int nv = 0;
    for (uint64_t d = 0; d < 8; ++d) {
        vs[nv++] = m / 2 - d;
        vs[nv++] = m / 2 + 1 + d;
        vs[nv++] = 1 + d;
        vs[nv++] = m - 1 - d;
    }
    vs[nv++] = nn::kMult;
    vs[nv++] = m / 4;
    vs[nv++] = m - m / 4;
    const int64_t top = (int64_t)(0.6 * kM) - 1;
    for (int i = 0; i < nv; ++i) {
        for (int64_t d = 0; d < 8; ++d)
            for (int64_t at : {top, (int64_t)(m / 2), (int64_t)(0.593 * kM), (int64_t)9})
                for (int sign : {1, -1}) check_bal((double)(sign * (at - d)), vs[i]);
        for (int k = 0; k < 20000; ++k)
            check_bal((double)((int64_t)(next64() % (2 * (uint64_t)top)) - top), vs[i]);
    }
    // chains, with the outputs at every step
    for (int c = 0; c < 400; ++c) {
        const uint64_t v = c < nv ? vs[c] : c < 300 ? unit(m) : nn::MultPowers::get().pow(next64());
        if (v % 3 == 0) continue;
        const nn::BalMult f = nn::make_bal(v);
        uint64_t want = unit(m);
        double r = nn::VarBal::load(want);
        for (int k = 0; k < 5000; ++k) {
            r = nn::VarBal::mul(r, f);
            want = orc_mulmod(want, v, m);
            CHECK(is_int(r) && fabs(r) < 0.593 * kM);
            CHECK(nn::VarBal::to_u64(r) == want && nn::VarBal::to_f64(r) == orc_to_f64(want));
        }
    }
    // the generator itself
    uint64_t z = 0;
    CHECK(orc_seed(ORC_INDEX_MIN + 4242, &z) == 0);
    double r = nn::VarBal::load(z);
    const nn::BalMult m1 = nn::make_bal(nn::kMult);
    for (int k = 0; k < 200000; ++k) {
        r = nn::VarBal::mul(r, m1);
        z = orc_step(z);
        CHECK(nn::VarBal::to_u64(r) == z && nn::VarBal::to_f64(r) == orc_to_f64(z));
    }
}

// ------------------------------------------------------------ modulo 3^40 --

static void check_limbs(nn::e40::L3 z, uint64_t want) {
    CHECK(is_int(z.x0) && is_int(z.x1) && is_int(z.x2));
    CHECK(fabs(z.x0) <= 0.5 * (nn::e40::kB3 - 1) && fabs(z.x1) <= 0.5 * (nn::e40::kB3 - 1));
    CHECK(fabs(z.x2) <= 0.5 * (nn::e40::kD - 1));
    CHECK(nn::e40::to_u64(z) == want);
    CHECK(nn::e40::to_f64(z) == orc_e40_to_f64(want));
}

static void limb_steps() {
    const uint64_t m = ORC_E40_MOD, B = nn::e40::kLimb3, D = nn::e40::kTopLimb;
    // states and multipliers at the ends of every digit's range
    uint64_t edge[64];
    int n = 0;
    for (uint64_t s : {(uint64_t)1, (uint64_t)2, B - 1, B + 1, B * B - 1, B * B + 1, B / 2, B / 2 + 1,
                       (B / 2) * B + B / 2, (D / 2) * B * B + (B / 2) * B + B / 2, m / 2, m / 2 + 1,
                       (uint64_t)nn::e40::kMult, (uint64_t)nn::e40::kHalf, (uint64_t)1 << 63})
        for (uint64_t x : {s, m - s})
            if (x % 3) edge[n++] = x;
    for (int i = 0; i < n; ++i) check_limbs(nn::e40::limbs3(edge[i]), edge[i]);
    for (int i = 0; i < 20000; ++i) {
        const uint64_t s = unit(m);
        check_limbs(nn::e40::limbs3(s), s);
    }
    for (int i = 0; i < n; ++i)
        for (int k = 0; k < n; ++k)
            check_limbs(nn::e40::mul40t(nn::e40::limbs3(edge[k]), nn::e40::make_mult40t(edge[i])),
                        (uint64_t)(((nn::u128)edge[k] * edge[i]) % m));
    // chains, with the outputs at every step
    for (int c = 0; c < 300; ++c) {
        const uint64_t v = c < n ? edge[c] : c < 200 ? unit(m) : orc_e40_skip(1, next64());
        const nn::e40::Mult40T f = nn::e40::make_mult40t(v);
        uint64_t want = c & 1 ? edge[c % n] : unit(m);
        nn::e40::L3 z = nn::e40::limbs3(want);
        for (int k = 0; k < 5000; ++k) {
            z = nn::e40::mul40t(z, f);
            want = (uint64_t)(((nn::u128)want * v) % m);
            check_limbs(z, want);
        }
    }
    // the generator itself
    uint64_t want = 0;
    CHECK(orc_e40_seed(ORC_E40_INDEX_MIN + 4242, &want) == 0);
    nn::e40::L3 z = nn::e40::limbs3(want);
    const nn::e40::Mult40T m1 = nn::e40::make_mult40t(nn::e40::kMult);
    for (int k = 0; k < 100000; ++k) {
        z = nn::e40::mul40t(z, m1);
        want = orc_e40_step(want);
        check_limbs(z, want);
    }
}

int main() {
    balanced_steps();
    limb_steps();
    if (fails) {
        fprintf(stderr, "%d check(s) failed\n", fails);
        return 1;
    }
    printf("steps driver ok\n");
    return 0;
}
