// nn_e40.hpp -- the generator at the larger modulus 3^40 that Section 2
// names for a longer period (2*3^39): Eq. 3 with m = 3^40 and the same
// multiplier 2^53 (still 53 bits of alpha_{2,3} per step), Eq. 2 with 3^40
// in place of 3^33.  m > 2^63, so states need all 64 bits and the product
// of two of them 128: the FP64 reduction of the 3^33 path does not apply.
// The default step runs on FP64 limbs; the other is Montgomery's reduction with
// R = 2^64 and multipliers kept in Montgomery form (v R mod m), so its states stay
// in standard form.
#pragma once

#include <stdint.h>

#include "nn_arith.hpp"

namespace nn {
namespace e40 {

constexpr uint64_t kMod = 12157665459056928801ULL;  // 3^40
constexpr uint64_t kPeriod = 2ULL * (kMod / 3ULL);   // 2*3^39
constexpr uint64_t kMult = 1ULL << 53;               // 2^53 < 3^40
constexpr uint64_t kHalf = kMod / 2ULL;              // floor(3^40/2) (Eq. 2)
constexpr uint64_t kIndexMin = kMod + 100ULL;
constexpr double kRecip = 1.0 / 12157665459056928801.0;  // RN(1/3^40)

constexpr uint64_t neg_inv() {
    uint64_t x = kMod;
    for (int i = 0; i < 6; ++i) x *= 2ULL - kMod * x;
    return 0ULL - x;
}
constexpr uint64_t kNInv = neg_inv();  // -m^{-1} mod 2^64
static_assert(kMod * (0ULL - kNInv) == 1ULL, "Montgomery inverse");
static_assert(kMod > (1ULL << 63), "3^40 needs the full 64 bits");

// A fixed multiplier v and its Montgomery form v 2^64 mod m.
struct Mult40 {
    uint64_t v;
    uint64_t mont;
};

// REDC(z * vmont) = v z mod m for z < m.  With T = z vmont < m^2 and
// u = (T mod 2^64) (-1/m) mod 2^64, T + u m is a multiple of 2^64 and
// S = (T + u m) / 2^64 < 2m; 2m > 2^64, so S is formed in 128 bits: the
// low words of T and u m sum to 0 or 2^64, a carry of (T mod 2^64 != 0).
NN_HD uint64_t mm40(uint64_t z, uint64_t vmont) {
    const u128 t = (u128)z * vmont;
    const uint64_t tl = (uint64_t)t;
    const uint64_t u = tl * kNInv;
    const u128 um = (u128)u * kMod;
    const u128 s = (t >> 64) + (um >> 64) + (tl != 0);
    return (uint64_t)(s >= kMod ? s - kMod : s);
}

NN_HD double to_f64(uint64_t z) { return (double)z * kRecip; }

// The step on two limbs, an exact form of its own against which the host build
// checks the kernels' (below): base-B limbs, B = 3^20 < 2^32, m = B^2.  For a state
// z = x1 B + x0 and a multiplier v = j1 B + j0 the term x1 j1 B^2 is a
// multiple of m, so
//     v z = (x1 j0 + x0 j1 + c) B + r   (mod m),   x0 j0 = c B + r,
// three products of integers below 2^33, each reduced modulo B exactly in
// FP64: the product as ph + pl (two-product, exact), a quotient rounded
// from ph/B (off by at most one from the nearest), the remainder formed by
// one FMA and one add, both exact because it is an integer below 2^34.
// States stay redundant (limbs() starts them so): x0 = r in about
// [-B/2, B/2] and x1 the unreduced sum, below 2.01 B in magnitude; the
// output takes z from them directly (top() below).  Multipliers are
// canonical: 0 <= j0, j1 < B.
constexpr uint64_t kLimb = 3486784401ULL;  // 3^20
constexpr double kB = 3486784401.0;
constexpr double kRB = 1.0 / 3486784401.0;      // RN(1/B)
constexpr double kHalfRB = 0.5 / 3486784401.0;  // RN(1/(2B)) = RN(1/B)/2
static_assert(kLimb * kLimb == kMod, "3^40 = (3^20)^2");

struct L2 {
    double lo;  // x0
    double hi;  // x1
};

struct Mult40L {
    double j0;  // v mod B
    double j1;  // v div B
};

// x j - q B for q the rounded quotient: x j mod B up to one B either way.
NN_HD double rem_b(double x, double j, double* q_out) {
    const double ph = x * j;
    const double pl = __builtin_fma(x, j, -ph);
    const double q = __builtin_rint(ph * kRB);
    *q_out = q;
    return __builtin_fma(-q, kB, ph) + pl;
}

NN_HD L2 mul40l(L2 z, Mult40L v) {
    double c, qa, qb;
    const double r = rem_b(z.lo, v.j0, &c);
    const double ta = rem_b(z.hi, v.j0, &qa);
    const double tb = rem_b(z.lo, v.j1, &qb);
    return L2{r, ta + tb + c};
}

// A state's limbs in the form the step keeps: z = x1 B + x0 with
// |x0| <= B/2 (x0 = z mod B, less B above B/2) and 0 <= x1 <= B.
NN_HD L2 limbs(uint64_t z) {
    const uint64_t q = z / kLimb, r = z % kLimb;
    return r > kLimb / 2 ? L2{(double)r - kB, (double)(q + 1)} : L2{(double)r, (double)q};
}

// The output needs z = x1 B + x0 mod m in [0, m), not canonical limbs:
// z = (x1 - f B) B + x0 for f = floor((x1 + x0/B) / B).  x0 is a nonzero
// integer in (-B, B) (a state is a unit, so x0 is not a multiple of B), so
// x1 + x0/B lies strictly between x1 and x1 + 1 for x0 > 0 and between
// x1 - 1 and x1 for x0 < 0, and neither open interval holds a multiple of
// B: f = floor((x1 + 1/2) / B) or floor((x1 - 1/2) / B), the half taking
// x0's sign.  That quotient is at least 1/(2B) away from an integer, far
// beyond the rounding of the one FMA that forms it, so its floor is exact.
// top() returns x1 - f B, in [0, B) for x0 > 0 and [1, B] for x0 < 0, and
// z = top B + x0 lies in (0, m).
NN_HD double top(L2 z) {
    const double f = __builtin_floor(__builtin_fma(z.hi, kRB, __builtin_copysign(kHalfRB, z.lo)));
    return __builtin_fma(-f, kB, z.hi);
}

// top < 2^32 and |x0| < 2^31: z formed modulo 2^64, where it is exact.
NN_HD uint64_t to_u64(L2 z) {
    return (uint64_t)(uint32_t)top(z) * kLimb + (uint64_t)(int64_t)(int32_t)z.lo;
}

// RN(z) is one FMA: top B + x0 formed exactly and rounded once.
NN_HD double to_f64(L2 z) { return __builtin_fma(top(z), kB, z.lo) * kRecip; }

inline Mult40L make_mult40l(uint64_t v) { return Mult40L{(double)(v % kLimb), (double)(v / kLimb)}; }

// The kernels' FP64 step: three balanced limbs.  With B = 3^14 and D = 3^12, m = B^2 D, and
// a state z stands as z = (x2 B + x1) B + x0 (mod m) with |x0|, |x1| < B/2 and
// |x2| < D/2, the balanced residue of z in its balanced digits.  The product
// with a multiplier's limbs j needs only what stays below B^2 D:
//     t0 = x0 j0,                        x0' = t0 mod B, carry q0;
//     t1 = x0 j1 + x1 j0 + q0,           x1' = t1 mod B, carry q1;
//     t2 = x0 j2 + x1 j1 + x2 j0 + q1,   x2' = t2 mod D,
// six products as FMAs and three reductions of three instructions each, 15 where
// two limbs of 3^20 take 20 (their products have 64 bits and need the two-product
// and a quotient each).  Every t is an integer below 2^43.4, so all of this is
// exact, and a quotient's fused multiply-add onto 1.5 * 2^52 rounds t/B to the
// nearest integer: t/B is at least 1/(2B) = 2^-23 away from a half (B is odd),
// its error below 2^-30.  So limbs are unique, whatever led to them.
constexpr uint64_t kLimb3 = 4782969ULL;    // 3^14
constexpr uint64_t kTopLimb = 531441ULL;  // 3^12
constexpr double kB3 = 4782969.0;
constexpr double kRB3 = 1.0 / 4782969.0;  // RN(1/B)
constexpr double kD = 531441.0;
constexpr double kRD = 1.0 / 531441.0;  // RN(1/D)
constexpr double kBD = 2541865828329.0;  // B D = 3^26
constexpr double kRBD = 1.0 / 2541865828329.0;
constexpr double kHalfRBD = 0.5 / 2541865828329.0;
static_assert(kLimb3 * kLimb3 * kTopLimb == kMod, "3^40 = (3^14)^2 3^12");

struct L3 {
    double x0, x1, x2;
};

struct Mult40T {
    double j0, j1, j2;  // a multiplier's balanced limbs
};

// The integer nearest to t/base for the base's reciprocal rb (kBalRound in
// nn_arith.hpp: 1.5 * 2^52).
NN_HD double near_quot(double t, double rb) {
    return __builtin_fma(t, rb, kBalRound) - kBalRound;
}

NN_HD L3 mul40t(L3 z, Mult40T v) {
    const double t0 = z.x0 * v.j0;
    const double q0 = near_quot(t0, kRB3);
    const double t1 = __builtin_fma(z.x0, v.j1, __builtin_fma(z.x1, v.j0, q0));
    const double q1 = near_quot(t1, kRB3);
    const double t2 = __builtin_fma(
        z.x0, v.j2, __builtin_fma(z.x1, v.j1, __builtin_fma(z.x2, v.j0, q1)));
    const double q2 = near_quot(t2, kRD);
    return L3{__builtin_fma(-q0, kB3, t0), __builtin_fma(-q1, kB3, t1), __builtin_fma(-q2, kD, t2)};
}

// A state's limbs: its balanced residue, digit by digit.
NN_HD L3 limbs3(uint64_t z) {
    const int64_t b = (int64_t)(z > kMod / 2 ? z - kMod : z);  // |b| < 2^63
    const int64_t n = (int64_t)kLimb3, h = n / 2;
    int64_t x0 = b % n;
    x0 += x0 < -h ? n : x0 > h ? -n : 0;
    const int64_t r = (b - x0) / n;
    int64_t x1 = r % n;
    x1 += x1 < -h ? n : x1 > h ? -n : 0;
    return L3{(double)x0, (double)x1, (double)((r - x1) / n)};
}

// The output's z in [0, m) is T B + x0 for T = x2 B + x1, or with T + B D where
// that is negative: for T < 0, or T = 0 and x0 < 0 (x0 is never 0, a state being
// a unit).  (T + 1/2) / (B D), the half taking x0's sign, lies in (-1, 1) and
// at least 1/(2 B D) from 0 and 1, far beyond the one rounding that forms it, so its
// floor, 0 or -1, tells.  Returns that T, in [0, B D).
NN_HD double top(L3 z) {
    const double t = __builtin_fma(z.x2, kB3, z.x1);
    const double f =
        __builtin_floor(__builtin_fma(t, kRBD, __builtin_copysign(kHalfRBD, z.x0)));
    return __builtin_fma(-f, kBD, t);
}

NN_HD uint64_t to_u64(L3 z) {
    // top < 2^41.3 lies in the low bits of top + 2^52, x0 (below 2^22 in
    // magnitude) in the low word of x0 + 1.5 * 2^52
    const uint64_t t = __builtin_bit_cast(uint64_t, top(z) + 4503599627370496.0);
    const int32_t x0 = (int32_t)(uint32_t)__builtin_bit_cast(uint64_t, z.x0 + kBalRound);
    const uint64_t lo = (uint64_t)(uint32_t)t * (uint32_t)kLimb3 + (uint64_t)(int64_t)x0;
    return lo + ((uint64_t)(((uint32_t)(t >> 32) & 0x3ffu) * (uint32_t)kLimb3) << 32);
}

// RN(z) is one FMA: top B + x0 formed exactly and rounded once.
NN_HD double to_f64(L3 z) { return __builtin_fma(top(z), kB3, z.x0) * kRecip; }

inline Mult40T make_mult40t(uint64_t v) {
    const L3 x = limbs3(v);
    return Mult40T{x.x0, x.x1, x.x2};
}

// ------------------------------------------------ the flat layout's shape --
// Rows of 512 outputs per chunk and resident workgroups per CU, one chunk per
// workgroup in XCD runs.  What bounds the FP64 step's kernels is how the stores of
// a compute unit's workgroups are spaced, more than the arithmetic, and that is a
// matter of rows times residency: the best residency falls as the rows grow, for
// both kinds and store policies.  Medians, 2^28 and 100,000,007 outputs, us:
//   rows           cap 2       3           4           6           8
//    2  f64        478 183     386 147     368 134     345 134     336 132
//    4             384 153     332 127     316 122     313 127     315 131
//    8             330 125     311 124     332 129     341 132     345 133
//   16             327 129     349 136     351 140     353 140     355 141
//    2  u64        475 190     407 154     405 142     377 147     368 145
//    4             393 154     355 131     335 124     346 129     343 131
//    8             346 133     312 122     319 128     327 130     325 131
//   16             328 122     326 136     353 138     365 142     364 143
// 32 rows: 357 140 (f64) and 357 136 (u64) at 2, 364 144 and 373 143 at 4.
// Non-temporal stores follow the same line but for f64 with 8 rows, whose outputs
// take the fewest instructions: 305 120 at 2, 326 130 at 3, 339 131 at 4 (u64 331 126,
// 322 119 and 326 124).  One cap
// for every row count would cost up to a third: u64, 2^24 outputs, two rows 32.8
// us at 2 and 23.9 at 6.  Montgomery's step, bound by its arithmetic, keeps 4.
inline uint32_t flat_occupancy(int mm, int kind, bool nontemporal, uint32_t rows) {
    if (mm == 0) return 4;
    if (rows == 8) return kind == 1 && nontemporal ? 2 : 3;
    return rows <= 2 ? 6 : rows == 4 ? 4 : 2;
}

// The default rows (kind 0 u64, 1 f64).  f64 (25.8 VALU instructions an output)
// is fastest with 8; u64 (30.8) with 8 or 16 alike within the spread of machines
// (2^26 + 5 outputs 83.8 and 84.2 us, 2^28 312-331 and 325-330).
inline uint32_t flat_rows(int kind, int mm) { return mm == 1 && kind == 1 ? 8 : 16; }

// An output too short to give every CU two such chunks takes shorter ones
// (halved down to 2 rows): its time is a workgroup's own chain of rows.  Kernel
// times, f64 (u64): 200,003 outputs with 16 rows 3.84 (4.34) us, by this rule 2.70
// (2.74); 2^20 4.66 (5.16) and 4.08 (4.28).
inline uint32_t flat_rows_for(uint32_t rows, uint64_t count, uint32_t cus) {
    while (rows > 2 && count / (512ull * rows) < 2ull * cus) rows /= 2;
    return rows;
}

}  // namespace e40
}  // namespace nn
