// nn_kernels.hpp -- launch interface of the gfx950 kernels (host side).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nn_arith.hpp"

namespace nn {

// Skip-ahead tables on the device: t_lo[l] = 2^(53 l) for l < 1024 and
// t_hi[j] = 2^(53 * 1024 j) for j < 32768 (mod 3^33), so the multiplier of
// any offset k < 2^25 is t_hi[k >> 10] * t_lo[k & 1023].
constexpr uint32_t kLoBits = 10;
constexpr uint32_t kLoSize = 1u << kLoBits;
constexpr uint32_t kHiSize = 1u << 15;
constexpr uint64_t kMaxOffset = (uint64_t)kLoSize * kHiSize;  // 2^25
constexpr uint64_t kMaxThreads = kMaxOffset / 2;             // 2^24

// Plain generation.  Each of the T = grid*block threads owns W consecutive
// elements per row (W = 1: 8-byte stores, W = 2: 16-byte stores); row i
// covers elements [i*W*T, (i+1)*W*T).  count = e_full*W*T + rem with
// rem < W*T: the last, partial row holds `rem` elements.  `base` is
// state * 2^53 (the first output of the call), J = (2^53)^(W*T) and
// M1 = 2^53 with its reduction data.
struct GenArgs {
    uint64_t* out;
    uint64_t T;
    uint64_t e_full;
    uint32_t rem;
    uint64_t base;
    Mult J;
    Mult M1;
    Mult JI;  // J^ilp: the step of a thread that advances ilp rows at once
    const Mult* t_lo;
    const Mult* t_hi;
};

// ilp (width 2 only): rows a thread keeps in flight, 1, 2 or 4.
hipError_t launch_generate(int mulmod, int kind, int width, int unroll, int ilp,
                           bool nontemporal, uint32_t grid, uint32_t block, hipStream_t stream,
                           const GenArgs& a);

// Fused consumer: T = grid*block threads, thread t taking the outputs t, t + T,
// t + 2T, ... in registers and adding them up (raw states modulo 2^64 for
// kind 0, variates in binary64 for kind 1); one atomic per workgroup folds
// the sums into *result.  count = e_full*T + rem with rem < T; `base` is
// state * 2^53 and J[k] = (2^53)^(T 2^k): the steps by one, two and four rows.
struct ConsumeArgs {
    uint64_t T;
    uint64_t e_full;
    uint32_t rem;
    bool set;  // one workgroup: store the sum instead of adding it
    uint64_t base;
    Mult J[3];     // all but the FP64 reduction
    BalMult B[3];  // the same multipliers balanced: the FP64 reduction
    const Mult* t_lo;
    const Mult* t_hi;
};

// Workgroups of the default launch.  Every workgroup ends in one atomic on
// the same address, and those are served one after another at about 12 ns
// each (8192 of them, one per wavefront, held a call of any size up at
// 100 us), so the workgroups are as large as they come, at most one per
// compute unit, and a thread has at least kConsumeMinRows outputs.  From
// kConsumeTwoPerCu outputs on two per compute unit hide more latency than
// their atomics cost (2^28 variates: 66.4 against 69.2 us; 10,000,019: 11.2
// against 9.2).  A caller's smaller blocks fill a compute unit likewise, but
// below kConsumeTwoPerCu outputs with kConsumeMaxPerCu at most: more of them
// wait for their atomics (64 threads, 10,000,019 variates: 19.2 us with 4, 29.8
// with 8, 53.3 with 16; 2^26: 43.4, 44.1 and 62.5).  From kConsumeTwoPerCu on
// the unit is filled twice, as with the default's (2^30: 255 against 410 us).
constexpr uint32_t kConsumeBlock = 1024;
constexpr uint64_t kConsumeMinRows = 8;
constexpr uint64_t kConsumeTwoPerCu = 1ull << 27;
constexpr uint32_t kConsumeMaxPerCu = 4;
inline uint32_t consume_per_cu(uint32_t block, uint64_t count) {
    const uint32_t fill = kConsumeBlock / block;  // block <= kConsumeBlock
    if (count >= kConsumeTwoPerCu) return 2 * fill;
    return fill < kConsumeMaxPerCu ? fill : kConsumeMaxPerCu;
}

// Outputs up to which a call that sets the result takes one workgroup, which
// stores its sum: at most 32 rows a thread, where the kernel takes 5.1 us
// (40,000 outputs on five workgroups 4.5), against a launch that clears the
// result: 32,768 variates 7.2 us a call, 40,000 10.4.
constexpr uint64_t kConsumeSetOne = 1ull << 15;

hipError_t launch_clear(void* result, hipStream_t s);  // *result = 0
hipError_t launch_consume(int mulmod, int kind, uint32_t grid, uint32_t block, hipStream_t s,
                          const ConsumeArgs& a, void* result);

// Flat layout: workgroup b of 256 threads writes R rows of 512 elements,
// [512 R b, 512 R (b + 1)) of the launch, two consecutive ones per lane in
// one 16-byte store per row, and exits.  Its chunk starts u = R b rows of
// 512 in, from base * t_fhi[u >> 10] * t_flo[u & 1023] with
// t_flo[j] = (2^53)^(512 j) and t_fhi[i] = (2^53)^(512 * 1024 i): two small
// tables that stay in L2 (a workgroup lives a few microseconds, so its start
// must not wait on DRAM).
constexpr uint32_t kFlatBlock = 256;
constexpr uint32_t kFlatPerBlock = 2 * kFlatBlock;
constexpr uint32_t kFlatLoSize = 1024;
constexpr uint32_t kFlatHiSize = 2048;
constexpr uint64_t kFlatMaxRowsPerLaunch = (uint64_t)kFlatLoSize * kFlatHiSize;  // 2^21
// The device tables are one allocation of Mult entries: t_lo (kLoSize),
// t_hi (kHiSize), the four 8192-entry skip levels, then t_flo and t_fhi.
// The flat kernels take the allocation's start and these fixed offsets, so
// one kernel-argument load gives them every table.
constexpr uint64_t kFlatLoOffset = (uint64_t)kLoSize + kHiSize + 4ull * 8192ull;
constexpr uint64_t kFlatHiOffset = kFlatLoOffset + kFlatLoSize;
constexpr uint64_t kFlatMaxCount = kFlatMaxRowsPerLaunch * kFlatPerBlock;  // 2^30 per launch

// Rows per workgroup of the flat layout: 1, 2, 4, 8 or 16.  Defaults from
// sweeps on MI355X (2^30 f64 outputs): four rows (16 KiB per workgroup) and
// temporal stores, with the residency cap of occupancy 4 (33 280 bytes of
// dynamic LDS per workgroup).  The rate has a cliff in the LDS per
// workgroup: 6.2-6.35 TB/s at 31 744 bytes or less, 7.4-7.5 TB/s from
// 32 256 to 40 960 bytes; non-temporal stores stay at 6.2-6.4 throughout.
constexpr uint32_t kFlatMaxRows = 16;
// Outputs from which an output that is only 8-byte aligned takes every flat
// cfg field without NN_CFG_FLAT (below, a cfg that sets one means the rows).
constexpr uint64_t kFlatUnalignedMin = 1ull << 22;
constexpr uint32_t kFlatDefaultRows = 4;
// The shape without a cfg (FP64 reduction, temporal stores, XCD runs): two rows of
// balanced states at 5 (f64) or 6 (u64) workgroups per CU.  As at modulus 3^40,
// what bounds these kernels is how their stores are spaced: the shorter step needs
// shorter chunks.  Against four rows at 4 with the longer step, f64: 67,108,869
// outputs 79.2 against 81.6 us, 100,000,007 115.9 against 119.5, 2^29 - 1 593 against
// 605; u64: 159,912,993 181 against 188, 2^28 302 against 310, 2^30 1177 against 1229
// (7.30 TB/s).  Other mixes write slower (2^30, f64, the shorter step with four
// rows at 4 and 3: 1228 and 1187; the longer one with two rows at 6: 1392; two rows
// at 6 without runs 1215).  Below 2^24 outputs, which the last-level cache takes,
// four rows tie or are ahead (3,000,017 f64 6.0 against 6.2).  The f64 limit is no
// measured line: two rows stay 1 to 1.5 % ahead beyond it (medians of eight
// alternating runs, 2^29 589.7 against 598.1 us, 700,000,001 773 and 778, 2^30 1170
// and 1186; on other machines 2^30 took two rows up to 1212).  nn_default_cfg's
// shape for 2^30 f64 outputs, four rows at 4, is checked as part of its interface;
// the limit is the power of two below it.
constexpr uint32_t kFlatFastRows = 2;
inline uint32_t flat_fast_occupancy(int kind) { return kind == 1 ? 5u : 6u; }
constexpr uint64_t kFlatFastMin = 1ull << 24;
constexpr uint64_t kFlatFastMaxF64 = 1ull << 29;
constexpr uint32_t kFlatDefaultOccupancy = 4;

// The flat kernels' own copy of their multipliers (a static device array):
// kFlatBlock lane offsets (2^53)^(2l), then t_flo and t_fhi.
constexpr uint32_t kFlatSymLane = 0;
constexpr uint32_t kFlatSymLo = kFlatBlock;
constexpr uint32_t kFlatSymHi = kFlatSymLo + kFlatLoSize;
constexpr uint32_t kFlatSymEntries = kFlatSymHi + kFlatHiSize;
// Copies kFlatSymEntries entries into the current device's array.
hipError_t upload_flat_symbol(const Mult* entries);

// XCD runs: the 8 XCDs take consecutive workgroups in turn, so with chunks in
// workgroup order each XCD writes every eighth chunk.  With two or four rows per
// workgroup the whole chunks are taken in runs instead, with four rows of
// 8*kFlatXcdRun workgroups, in which XCD x writes the kFlatXcdRun consecutive
// chunks [x kFlatXcdRun, (x + 1) kFlatXcdRun) of the run (4 MiB).  Whole
// chunks beyond the last full run keep workgroup order.
constexpr uint32_t kFlatXcds = 8;
constexpr uint32_t kFlatXcdRun = 256;
// Chunks of two rows take runs of as many bytes.  The chunks per XCD of a run, 0
// for row counts without runs:
constexpr uint32_t flat_xcd_run(int rows) {
    return rows == 2 || rows == 4 ? kFlatXcdRun * 4 / rows : 0;
}
// Whole chunks of a flat launch that are taken in XCD runs (runs: the launch takes
// any).
inline uint64_t flat_run_chunks(int rows, bool runs, uint64_t whole_chunks) {
    const uint64_t run = (uint64_t)kFlatXcds * flat_xcd_run(rows);
    return run && runs ? whole_chunks / run * run : 0;
}

// One launch writes all of it: the whole chunks, the partial last one and,
// where the caller's output is only 8-byte aligned, the element before `out`.
struct FlatArgs {
    uint64_t base;   // state of out[0]
    uint64_t* out;   // 16-byte aligned
    uint32_t full;   // whole chunks of kFlatPerBlock*rows outputs
    uint32_t runs;   // the first of them, in XCD runs (flat_run_chunks)
    uint32_t tail;   // outputs of the partial last chunk
    uint64_t* head;  // one output before out[0], or null
    uint64_t head_state;
    Mult M1;         // 2^53
    Mult J;          // (2^53)^kFlatPerBlock: the next row of a lane
    BalMult bal_M1, bal_J;  // both balanced
};

// rows: rows per workgroup (1, 2, 4, 8, 16); lds_bytes > 0 caps the
// resident workgroups per compute unit.
hipError_t launch_generate_flat(int mulmod, int kind, bool nontemporal, int rows,
                                uint32_t lds_bytes, hipStream_t stream, const FlatArgs& a);
// start: the fill that keeps the generator's table loads (NN_FILL_WITH_START);
// it reads neither the states nor the multipliers of `a`.
hipError_t launch_fill_flat(bool nontemporal, int rows, uint32_t lds_bytes, hipStream_t stream,
                            bool start, const FlatArgs& a, uint64_t value);

// Consecutive layout: the output is cut into tiles of block*E elements;
// workgroup w makes tiles w, w + grid, ...  In a tile, thread t makes
// elements t*E .. t*E + E-1 one after another with the Modified Barrett
// step by 2^53, parks them in LDS, and the workgroup then stores the tile
// in serial order, lane-contiguous (16 bytes per lane when width 2).
// `base` is state * 2^53 (element 0), J = (2^53)^(grid*block*E) moves a
// thread to its next tile, and grid*block*E <= kMaxOffset.
constexpr uint32_t kConsecMaxE = 32;

struct ConsecArgs {
    uint64_t* out;
    uint64_t count;
    uint64_t base;
    Mult J;
    const Mult* t_lo;
    const Mult* t_hi;
};

// E in {2, 4, 8, 16, 32}, width 1 or 2; lds_bytes = block*(E+1)*8.
hipError_t launch_generate_consec(int kind, int E, int width, bool nontemporal, uint32_t grid,
                                  uint32_t block, hipStream_t stream, const ConsecArgs& a);

inline uint32_t consec_lds_bytes(uint32_t block, uint32_t E) { return block * (E + 1) * 8; }

hipError_t launch_fill(int width, int unroll, bool nontemporal, uint32_t grid, uint32_t block,
                       hipStream_t stream, uint64_t* out, uint64_t T, uint64_t e_full,
                       uint32_t rem, uint64_t value);

}  // namespace nn
