// nn_kernels.hip -- gfx950 kernels of the alpha_{2,3} generator.
//
// Layout (serial order in memory, coalesced stores): with T = grid*block
// threads, each owning W consecutive elements per row, row i covers
// elements [i*W*T, (i+1)*W*T) and thread t writes elements
// i*W*T + W*t .. + W-1.  A thread starts at element W*t by skip-ahead and
// then moves one row per step with the jump multiplier J = (2^53)^(W*T):
// Eq. 3 applied W*T times is one multiplication by J (Section 2: any iterate
// is reachable directly).  A wavefront's 64 lanes therefore store 64*W
// consecutive elements (512 or 1024 contiguous bytes) per row, and memory
// order equals sequence order, unlike the paper's strided layout of
// Section 3.2.
#include <hip/hip_runtime.h>

#include <vector>

#include "nn_device.hpp"
#include "nn_host.hpp"

namespace nn {

// W = 1: one element per thread and row.
template <class V, int KIND, int UNROLL, bool NT>
__global__ __launch_bounds__(1024) void k_generate1(uint64_t* __restrict__ out, uint64_t T,
                                                    uint64_t e_full, uint32_t rem, uint64_t base,
                                                    Mult J, Mult M1,
                                                    const Mult* __restrict__ t_lo,
                                                    const Mult* __restrict__ t_hi) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    const bool extra = t < rem;
    if (e_full == 0 && !extra) return;
    typename V::S z = thread_start<V>(base, t, t_lo, t_hi);
    uint64_t* row = out;  // uniform: row i starts at element i*T
#pragma unroll UNROLL
    for (uint64_t i = 0; i < e_full; ++i) {
        put<NT>(row + t, out_bits<V, KIND>(z));
        row += T;
        z = V::mul(z, J);
    }
    if (extra) put<NT>(row + t, out_bits<V, KIND>(z));
}

// W = 2: two consecutive elements per thread and row, one 16-byte store.
// Requires a 16-byte aligned output.
template <class V, int KIND, int UNROLL, bool NT>
__global__ __launch_bounds__(1024) void k_generate2(uint64_t* __restrict__ out, uint64_t T,
                                                    uint64_t e_full, uint32_t rem, uint64_t base,
                                                    Mult J, Mult M1,
                                                    const Mult* __restrict__ t_lo,
                                                    const Mult* __restrict__ t_hi) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t rem_pairs = rem >> 1;
    const bool extra_pair = t < rem_pairs;
    const bool extra_one = (rem & 1u) && t == rem_pairs;
    if (e_full == 0 && !extra_pair && !extra_one) return;
    typename V::S za = thread_start<V>(base, 2ull * t, t_lo, t_hi);
    typename V::S zb = V::mul(za, M1);
    u64x2* row = reinterpret_cast<u64x2*>(out);
#pragma unroll UNROLL
    for (uint64_t i = 0; i < e_full; ++i) {
        u64x2 v;
        v.x = out_bits<V, KIND>(za);
        v.y = out_bits<V, KIND>(zb);
        put<NT>(row + t, v);
        row += T;
        za = V::mul(za, J);
        zb = V::mul(zb, J);
    }
    if (extra_pair) {
        u64x2 v;
        v.x = out_bits<V, KIND>(za);
        v.y = out_bits<V, KIND>(zb);
        put<NT>(row + t, v);
    } else if (extra_one) {
        put<NT>(reinterpret_cast<uint64_t*>(row + t), out_bits<V, KIND>(za));
    }
}

// W = 2 with IL rows in flight per thread: 2*IL independent multiplication
// chains per lane, each advanced by JI = J^IL per trip.
template <class V, int KIND, int UNROLL, bool NT, int IL>
__global__ __launch_bounds__(1024) void k_generate2_ilp(uint64_t* __restrict__ out, uint64_t T,
                                                        uint64_t e_full, uint32_t rem,
                                                        uint64_t base, Mult J, Mult M1, Mult JI,
                                                        const Mult* __restrict__ t_lo,
                                                        const Mult* __restrict__ t_hi) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    const uint32_t rem_pairs = rem >> 1;
    const bool extra_pair = t < rem_pairs;
    const bool extra_one = (rem & 1u) && t == rem_pairs;
    if (e_full == 0 && !extra_pair && !extra_one) return;
    typename V::S za[IL], zb[IL];
    za[0] = thread_start<V>(base, 2ull * t, t_lo, t_hi);
    zb[0] = V::mul(za[0], M1);
#pragma unroll
    for (int r = 1; r < IL; ++r) {
        za[r] = V::mul(za[r - 1], J);
        zb[r] = V::mul(zb[r - 1], J);
    }
    u64x2* row = reinterpret_cast<u64x2*>(out);
    uint64_t i = 0;
#pragma unroll UNROLL
    for (; i + IL <= e_full; i += IL) {
#pragma unroll
        for (int r = 0; r < IL; ++r) {
            u64x2 v;
            v.x = out_bits<V, KIND>(za[r]);
            v.y = out_bits<V, KIND>(zb[r]);
            put<NT>(row + r * T + t, v);
            za[r] = V::mul(za[r], JI);
            zb[r] = V::mul(zb[r], JI);
            // Each row's store stays next to its own two multiplications:
            // left to itself the scheduler bunches the stores of a trip
            // together, which writes about 8 % slower on MI355X.
            __builtin_amdgcn_sched_barrier(0);
        }
        row += IL * T;
    }
    // Fewer than IL full rows remain, then the partial row; za[r], zb[r]
    // hold rows i + r.
    const uint32_t left = (uint32_t)(e_full - i);
    typename V::S pa = za[0], pb = zb[0];
#pragma unroll
    for (int r = 0; r < IL; ++r) {
        if ((uint32_t)r < left) {
            u64x2 v;
            v.x = out_bits<V, KIND>(za[r]);
            v.y = out_bits<V, KIND>(zb[r]);
            put<NT>(row + r * T + t, v);
        }
        if ((uint32_t)r == left) {
            pa = za[r];
            pb = zb[r];
        }
    }
    row += left * T;
    if (extra_pair) {
        u64x2 v;
        v.x = out_bits<V, KIND>(pa);
        v.y = out_bits<V, KIND>(pb);
        put<NT>(row + t, v);
    } else if (extra_one) {
        put<NT>(reinterpret_cast<uint64_t*>(row + t), out_bits<V, KIND>(pa));
    }
}

// Fused consumer (the paper's point that variates usually feed a simulation
// directly, Section 3.2; its Table 2 removes the memory traffic): the outputs
// are summed in registers and never stored.  Kind 0 sums raw states modulo
// 2^64 (exact in any order).

// The sum of v over a workgroup, valid in thread 0 (every thread calls it, once
// per type: a second call would write the LDS that the first still reads).
template <class X>
__device__ __forceinline__ X block_sum(X v) {
    __shared__ X part[16];
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    const uint32_t w = threadIdx.x >> 6;
    if ((threadIdx.x & 63) == 0) part[w] = v;
    __syncthreads();
    v = threadIdx.x < (blockDim.x >> 6) ? part[threadIdx.x] : X(0);
    if (w == 0)
        for (int off = 8; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// A workgroup's sum to *result: set where it is the only one of a call that
// sets the result, else added.
template <class X>
__device__ __forceinline__ void give(X* result, X sum, bool set) {
    if (threadIdx.x) return;
    if (set)
        *result = sum;
    else
        atomicAdd(result, sum);
}

// Clears the result of a call that sets it with several workgroups (both kinds'
// zero is the same 64 bits).
__global__ void k_clear(uint64_t* result) { *result = 0; }

hipError_t launch_clear(void* result, hipStream_t s) {
    k_clear<<<1, 1, 0, s>>>(static_cast<uint64_t*>(result));
    return hipGetLastError();
}

// The integer reductions, four rows in flight per thread.
template <class V, int KIND>
__global__ __launch_bounds__(1024) void k_consume(ConsumeArgs a, void* result) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    typename V::S z[4];
    z[0] = thread_start<V>(a.base, t, a.t_lo, a.t_hi);
    z[1] = V::mul(z[0], a.J[0]);
    z[2] = V::mul(z[0], a.J[1]);
    z[3] = V::mul(z[1], a.J[1]);
    unsigned long long su = 0;
    double sf = 0.0;
    auto take = [&](typename V::S x) {
        if constexpr (KIND == 0)
            su += V::to_u64(x);
        else
            sf += V::to_f64(x);
    };
    uint64_t i = 0;
    for (; i + 4 <= a.e_full; i += 4) {
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            take(z[c]);
            z[c] = V::mul(z[c], a.J[2]);
        }
    }
    const uint32_t left = (uint32_t)(a.e_full - i);  // full rows left, then the partial row
#pragma unroll
    for (uint32_t c = 0; c < 4; ++c)
        if (c < left || (c == left && t < a.rem)) take(z[c]);
    if constexpr (KIND == 0) {
        give(static_cast<unsigned long long*>(result), block_sum(su), a.set);
    } else {
        give(static_cast<double*>(result), block_sum(sf), a.set);
    }
}

// The FP64 reduction on balanced states (mm_bal): a state z is r or r + m, so
// the sum of the states is the sum of the r plus m for every negative one.
// Bound by the VALU: per output six instructions for the step, one compare
// whose mask the scalar unit counts, and the sum's:
//  * kind 1: one add.  The partial sums of balanced states stay near zero, so
//    they round less than sums of variates do, and the conversion is one
//    product per workgroup.
//  * kind 0: the exact sum, one add per pair (|r + r'| < 1.2 m < 2^53) and
//    three that split it into multiples of 2^26 (added to hi, which starts at
//    1.5 * 2^78 where the unit is 2^26) and the rest (below 2^26, added to
//    lo): exact for 2^24 pairs, so hi and lo are emptied every 2^20 trips.
// Four rows in flight per thread: four independent chains.  2^30 variates back to
// back: 246-258 us, 4.2-4.4e12 a second (85-89 % of the VALU's rate for eight
// instructions an output at 2.4 GHz), against 402-421 us with nn_dev_mulmod's step
// and a conversion per variate; 2^30 raw states 300-304 us against 532-600.  After
// a minute of launches bound by HBM, at the clock these leave, 278-283 and
// 350-360 us (before: 427 and 604).
template <int KIND>
__global__ __launch_bounds__(1024) void k_consume_bal(ConsumeArgs a, void* result) {
    constexpr double kSplit = 453347182355485940514816.0;  // 1.5 * 2^78
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    double z[4];
    z[0] = balanced(thread_start<VarFP64>(a.base, t, a.t_lo, a.t_hi));
    z[1] = mm_bal(z[0], a.B[0]);
    z[2] = mm_bal(z[0], a.B[1]);
    z[3] = mm_bal(z[1], a.B[1]);
    double hi[2] = {kSplit, kSplit}, lo[2] = {0.0, 0.0};  // kind 0
    double sf[4] = {0.0, 0.0, 0.0, 0.0};                  // kind 1
    unsigned long long su = 0;
    uint64_t negative = 0;  // of the whole wavefront; neg: since the last emptying
    uint32_t neg = 0;
    auto split = [&](int k, double x) {
        const double h = hi[k] + x;
        lo[k] += x - (h - hi[k]);
        hi[k] = h;
    };
    auto empty = [&] {
        negative += neg;
        neg = 0;
#pragma unroll
        for (int k = 0; k < 2 && KIND == 0; ++k) {
            su += ((unsigned long long)(long long)((hi[k] - kSplit) * 0x1p-26) << 26) +
                  (unsigned long long)(long long)lo[k];
            hi[k] = kSplit;
            lo[k] = 0.0;
        }
    };
    auto count = [&](double r) {
        neg += (uint32_t)__builtin_popcountll(__builtin_amdgcn_ballot_w64(r < 0.0));
    };
    uint64_t trips = a.e_full >> 2;
    while (trips) {
        const uint32_t n = trips < (1u << 20) ? (uint32_t)trips : 1u << 20;
        trips -= n;
        for (uint32_t i = 0; i < n; ++i) {
            if constexpr (KIND == 0) {
                split(0, z[0] + z[1]);
                split(1, z[2] + z[3]);
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if constexpr (KIND == 1) sf[c] += z[c];
                count(z[c]);
                z[c] = mm_bal(z[c], a.B[2]);
            }
        }
        empty();
    }
    const uint32_t left = (uint32_t)a.e_full & 3u;  // full rows left, then the partial row
#pragma unroll
    for (uint32_t c = 0; c < 4; ++c) {
        if (c < left || (c == left && t < a.rem)) {
            count(z[c]);
            if constexpr (KIND == 0)
                su += (unsigned long long)(long long)z[c];
            else
                sf[c] += z[c];
        }
    }
    negative = (threadIdx.x & 63) == 0 ? negative + neg : 0;  // the wavefront's count, once
    if constexpr (KIND == 0) {
        give(static_cast<unsigned long long*>(result), block_sum(su + negative * kMod), a.set);
    } else {
        negative = block_sum(negative);
        const double s = block_sum((sf[0] + sf[1]) + (sf[2] + sf[3]));
        give(static_cast<double*>(result), __builtin_fma((double)negative, kModD, s) * kRecip,
             a.set);
    }
}

template <class V>
static hipError_t consume_v(int kind, uint32_t grid, uint32_t block, hipStream_t s,
                            const ConsumeArgs& a, void* result) {
    if (kind == 0)
        k_consume<V, 0><<<grid, block, 0, s>>>(a, result);
    else
        k_consume<V, 1><<<grid, block, 0, s>>>(a, result);
    return hipGetLastError();
}

hipError_t launch_consume(int mulmod, int kind, uint32_t grid, uint32_t block, hipStream_t s,
                          const ConsumeArgs& a, void* result) {
    switch (mulmod) {
        case 1:
            if (kind == 0)
                k_consume_bal<0><<<grid, block, 0, s>>>(a, result);
            else
                k_consume_bal<1><<<grid, block, 0, s>>>(a, result);
            return hipGetLastError();
        case 2: return consume_v<VarBarrett>(kind, grid, block, s, a, result);
        case 3: return consume_v<VarShoup>(kind, grid, block, s, a, result);
        case 4: return consume_v<VarMontgomery>(kind, grid, block, s, a, result);
        default: return hipErrorInvalidValue;
    }
}

// The paper's "Constant" kernel (Section 4.2): the same stores, a fixed value.
template <int W, int UNROLL, bool NT>
__global__ __launch_bounds__(1024) void k_fill(uint64_t* __restrict__ out, uint64_t T,
                                               uint64_t e_full, uint32_t rem, uint64_t value) {
    const uint32_t t = blockIdx.x * blockDim.x + threadIdx.x;
    if constexpr (W == 1) {
        uint64_t* row = out;
#pragma unroll UNROLL
        for (uint64_t i = 0; i < e_full; ++i) {
            put<NT>(row + t, value);
            row += T;
        }
        if (t < rem) put<NT>(row + t, value);
    } else {
        u64x2 v;
        v.x = value;
        v.y = value;
        u64x2* row = reinterpret_cast<u64x2*>(out);
#pragma unroll UNROLL
        for (uint64_t i = 0; i < e_full; ++i) {
            put<NT>(row + t, v);
            row += T;
        }
        if (t < (rem >> 1))
            put<NT>(row + t, v);
        else if ((rem & 1u) && t == (rem >> 1))
            put<NT>(reinterpret_cast<uint64_t*>(row + t), value);
    }
}

// The flat kernels' multipliers in a static device array of this module:
// the lane offsets (2^53)^(2l) for l < kFlatBlock, then t_flo and t_fhi.
// Its address is a link-time constant of the code, so a workgroup issues
// its table loads at once instead of after the load of a table pointer
// from its arguments.  Filled per device at set-up (upload_flat_symbol).
// flat_bal: the same multipliers balanced.
__device__ Mult flat_sym[kFlatSymEntries];
__device__ BalMult flat_bal[kFlatSymEntries];

template <class V>
__device__ __forceinline__ const typename V::M* flat_tab() {
    if constexpr (std::is_same<typename V::M, BalMult>::value)
        return flat_bal;
    else
        return flat_sym;
}

// flat_start over flat_tab: the states of lane l's pair (outputs 2l and
// 2l + 1) of the chunk that begins u = b*R rows after the output whose state
// is `base`.  b*R < kFlatMaxRowsPerLaunch.
template <class V>
__device__ __forceinline__ void flat_start_sym(uint64_t b, uint32_t l, int R, uint64_t base,
                                               const typename V::M& M1, typename V::S& za,
                                               typename V::S& zb) {
    const uint64_t u = b * (uint64_t)R;
    const typename V::M hi = flat_tab<V>()[kFlatSymHi + u / kFlatLoSize];
    const typename V::M lo = flat_tab<V>()[kFlatSymLo + u % kFlatLoSize];
    const typename V::M lane = flat_tab<V>()[kFlatSymLane + l];
    za = V::mul(V::mul(V::mul(V::load(base), hi), lo), lane);
    zb = V::mul(za, M1);
}

hipError_t upload_flat_symbol(const Mult* entries) {
    std::vector<BalMult> bal;
    for (uint32_t k = 0; k < kFlatSymEntries; ++k) bal.push_back(make_bal(entries[k].vi));
    const hipError_t e =
        hipMemcpyToSymbol(HIP_SYMBOL(flat_bal), bal.data(), sizeof(BalMult) * kFlatSymEntries, 0,
                          hipMemcpyHostToDevice);
    if (e != hipSuccess) return e;
    return hipMemcpyToSymbol(HIP_SYMBOL(flat_sym), entries, sizeof(Mult) * kFlatSymEntries, 0,
                             hipMemcpyHostToDevice);
}

// The chunk that workgroup w writes: w itself (G = 0), or its XCD-run chunk (runs
// of G chunks per XCD, in launches of whole runs).
template <int G>
__device__ __forceinline__ uint64_t flat_chunk(uint64_t w) {
    if constexpr (G == 0)
        return w;
    else
        return xcd_run_index<G>(w);
}
// In a launch whose first `runs` chunks are in XCD runs.
template <int R>
__device__ __forceinline__ uint32_t flat_chunk_any(uint32_t w, uint32_t runs) {
    if constexpr (flat_xcd_run(R) != 0)
        if (w < runs) return (uint32_t)xcd_run_index<flat_xcd_run(R)>(w);
    return w;
}

// Flat layout (see launch_generate_flat).  Workgroup w writes the R rows of
// kFlatPerBlock outputs of chunk b = flat_chunk<G>(w), from element
// kFlatPerBlock*R*b on, lane l the pair 2l of each row, and exits.  Its start is two multiplications by uniform
// table entries (scalar loads that hit L2), then one by the lane's offset;
// after that one multiplication per output.  Each row: its store, then the
// two multiplications to the next.
//
// A workgroup lives a few microseconds, so its start must not wait on more
// round trips of scalar-load latency than needed: the tables sit at a fixed
// address (flat_sym), so their loads go out with the load of the base, the
// whole-chunk kernel takes no count and tests nothing, and the table
// indices are in range for every lane.  It takes whole chunks only, all of
// them in XCD runs or none; every other output goes to k_generate_flat_any.
template <class V, int KIND, bool NT, int R, int G>
__global__ __launch_bounds__(kFlatBlock) void k_generate_flat(uint64_t base,
                                                              uint64_t* __restrict__ out,
                                                              typename V::M M1,
                                                              typename V::M J) {
    extern __shared__ char occupancy_cap[];  // dynamic LDS only limits residency
    (void)occupancy_cap;
    const uint64_t b = flat_chunk<G>(blockIdx.x);
    const uint32_t l = threadIdx.x;
    typename V::S za, zb;
    flat_start_sym<V>(b, l, R, base, M1, za, zb);
    u64x2* p = reinterpret_cast<u64x2*>(out + (uint64_t)kFlatPerBlock * R * b + 2u * l);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        u64x2 v;
        v.x = out_bits<V, KIND>(za);
        v.y = out_bits<V, KIND>(zb);
        put<NT>(p + r * kFlatBlock, v);
        if (r + 1 < R) {
            za = V::mul(za, J);
            zb = V::mul(zb, J);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
}

// Any other output in one launch: its whole chunks (the first `runs` in XCD
// runs), the partial last chunk, which the last workgroup writes pair by
// pair, and the element before `out` of an output that is only 8-byte
// aligned, which workgroup 0 adds.  The partial chunk and that element cost
// nothing of their own, where each launch of their own (one workgroup, after
// or before the others) took 3-4 us: 2^28 - 3 variates 308 -> 303 us,
// 20,000,003 into an 8-byte aligned output 31.5 -> 24.9 us, 3,000,017 12.8 ->
// 9.8 us.  The tests on `runs` and `full` hold a workgroup's table loads back
// until its arguments are there, which the whole-chunk kernel avoids: on whole
// runs that one stays ahead (2^23 variates 11.7 against 12.1 us, 2^30 1187
// against 1193).
template <class V>
__host__ __device__ __forceinline__ typename V::M flat_m1(const FlatArgs& a) {
    if constexpr (std::is_same<typename V::M, BalMult>::value)
        return a.bal_M1;
    else
        return a.M1;
}
template <class V>
__host__ __device__ __forceinline__ typename V::M flat_j(const FlatArgs& a) {
    if constexpr (std::is_same<typename V::M, BalMult>::value)
        return a.bal_J;
    else
        return a.J;
}

template <class V, int KIND, bool NT, int R>
__global__ __launch_bounds__(kFlatBlock) void k_generate_flat_any(FlatArgs a) {
    extern __shared__ char occupancy_cap[];
    (void)occupancy_cap;
    const uint32_t w = blockIdx.x;
    const uint32_t b = flat_chunk_any<R>(w, a.runs);
    const uint32_t l = threadIdx.x;
    const typename V::M M1 = flat_m1<V>(a), J = flat_j<V>(a);
    typename V::S za, zb;
    flat_start_sym<V>(b, l, R, a.base, M1, za, zb);
    const global_ptr<uint64_t> p = as_global(a.out) + ((uint64_t)kFlatPerBlock * R * b + 2u * l);
    if (b < a.full) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            u64x2 v;
            v.x = out_bits<V, KIND>(za);
            v.y = out_bits<V, KIND>(zb);
            put<NT>(reinterpret_cast<global_ptr<u64x2>>(p + r * kFlatPerBlock), v);
            if (r + 1 < R) {
                za = V::mul(za, J);
                zb = V::mul(zb, J);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        uint32_t k = 2u * l;
        for (int r = 0; r < R && k < a.tail; ++r, k += kFlatPerBlock) {
            if (k + 1 < a.tail) {
                u64x2 v;
                v.x = out_bits<V, KIND>(za);
                v.y = out_bits<V, KIND>(zb);
                put<NT>(reinterpret_cast<global_ptr<u64x2>>(p + r * kFlatPerBlock), v);
            } else {
                put<NT>(p + r * kFlatPerBlock, out_bits<V, KIND>(za));
            }
            za = V::mul(za, J);
            zb = V::mul(zb, J);
        }
    }
    if (w == 0 && a.head && l == 0)
        put<NT>(as_global(a.head), out_bits<V, KIND>(V::load(a.head_state)));
}

// The paper's "Constant" kernel (Section 4.2) for the flat layout: exactly
// k_generate_flat's stores with the arithmetic taken out -- whole chunks of
// R rows of kFlatPerBlock outputs, no count test, each row's store followed
// by the same scheduling barrier (k_fill_flat), and k_generate_flat_any's for
// every other output (k_fill_flat_any).
//
// START: also the generator's start -- its three table loads (the chunk's
// two row multipliers and the lane's offset) -- with only a comparison in
// place of its multiplications, so the stores wait for the same loads:
// the generator minus its arithmetic.  (The entries are positive, so the
// comparison always keeps `value`.)
template <int R, bool START>
__device__ __forceinline__ u64x2 fill_pair(uint64_t b, uint64_t value) {
    u64x2 v;
    v.x = value;
    if constexpr (START) {
        const uint64_t u = b * R;
        const double hi = flat_sym[kFlatSymHi + u / kFlatLoSize].v;
        const double lo = flat_sym[kFlatSymLo + u % kFlatLoSize].v;
        const double lane = flat_sym[kFlatSymLane + threadIdx.x].v;
        v.x = hi + lo + lane > 0.0 ? value : 0;
    }
    v.y = v.x;
    return v;
}

template <bool NT, int R, bool START, int G>
__global__ __launch_bounds__(kFlatBlock) void k_fill_flat(uint64_t* __restrict__ out,
                                                          uint64_t value) {
    extern __shared__ char occupancy_cap[];
    (void)occupancy_cap;
    const uint64_t b = flat_chunk<G>(blockIdx.x);
    const u64x2 v = fill_pair<R, START>(b, value);
    u64x2* p = reinterpret_cast<u64x2*>(out + (uint64_t)kFlatPerBlock * R * b + 2u * threadIdx.x);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        put<NT>(p + r * kFlatBlock, v);
        __builtin_amdgcn_sched_barrier(0);
    }
}

template <bool NT, int R, bool START>
__global__ __launch_bounds__(kFlatBlock) void k_fill_flat_any(FlatArgs a, uint64_t value) {
    extern __shared__ char occupancy_cap[];
    (void)occupancy_cap;
    const uint32_t w = blockIdx.x;
    const uint32_t b = flat_chunk_any<R>(w, a.runs);
    const uint32_t l = threadIdx.x;
    const u64x2 v = fill_pair<R, START>(b, value);
    const global_ptr<uint64_t> p = as_global(a.out) + ((uint64_t)kFlatPerBlock * R * b + 2u * l);
    if (b < a.full) {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            put<NT>(reinterpret_cast<global_ptr<u64x2>>(p + r * kFlatPerBlock), v);
            __builtin_amdgcn_sched_barrier(0);
        }
    } else {
        uint32_t k = 2u * l;
        for (int r = 0; r < R && k < a.tail; ++r, k += kFlatPerBlock) {
            if (k + 1 < a.tail)
                put<NT>(reinterpret_cast<global_ptr<u64x2>>(p + r * kFlatPerBlock), v);
            else
                put<NT>(p + r * kFlatPerBlock, value);
        }
    }
    if (w == 0 && a.head && l == 0) put<NT>(as_global(a.head), value);
}

// Whole chunks only, all in XCD runs or none: the kernel without tests.
static bool flat_whole(const FlatArgs& a) {
    return a.full && !a.tail && !a.head && (a.runs == 0 || a.runs == a.full);
}
// Workgroups of the other: one for the partial chunk, or for the lone head.
static uint32_t flat_grid(const FlatArgs& a) {
    const uint32_t chunks = a.full + (a.tail ? 1u : 0u);
    return chunks ? chunks : 1u;
}

template <class V, int KIND, bool NT, int R>
static hipError_t flat_one(uint32_t lds, hipStream_t s, const FlatArgs& a) {
    if (flat_whole(a)) {
        if constexpr (flat_xcd_run(R) != 0) {
            if (a.runs) {
                hipLaunchKernelGGL((k_generate_flat<V, KIND, NT, R, flat_xcd_run(R)>),
                                   dim3(a.full), dim3(kFlatBlock), lds, s, a.base, a.out,
                                   flat_m1<V>(a), flat_j<V>(a));
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((k_generate_flat<V, KIND, NT, R, 0>), dim3(a.full), dim3(kFlatBlock),
                           lds, s, a.base, a.out, flat_m1<V>(a), flat_j<V>(a));
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_generate_flat_any<V, KIND, NT, R>), dim3(flat_grid(a)), dim3(kFlatBlock),
                       lds, s, a);
    return hipGetLastError();
}

// Chunks of two rows with temporal stores take the FP64 reduction's balanced
// form (kFlatFastRows).  Non-temporal ones are spaced better by the longer step:
// two rows at cap 4, u64 2^26 + 5 outputs 81.0 against 83.7 us, 2^28 295 against
// 317, 2^30 1207 against 1251; f64 2^28 314 against 318, 2^30 1242 against 1248.
template <class V, bool NT>
struct TwoRows {
    typedef V T;
};
template <>
struct TwoRows<VarFP64, false> {
    typedef VarBal T;
};

template <class V, int KIND, bool NT>
static hipError_t flat_r(int rows, uint32_t lds, hipStream_t s, const FlatArgs& a) {
    switch (rows) {
        case 1: return flat_one<V, KIND, NT, 1>(lds, s, a);
        case 2: return flat_one<typename TwoRows<V, NT>::T, KIND, NT, 2>(lds, s, a);
        case 4: return flat_one<V, KIND, NT, 4>(lds, s, a);
        case 8: return flat_one<V, KIND, NT, 8>(lds, s, a);
        case 16: return flat_one<V, KIND, NT, 16>(lds, s, a);
        default: return hipErrorInvalidValue;
    }
}

template <class V>
static hipError_t flat_v(int kind, bool nt, int rows, uint32_t lds, hipStream_t s,
                         const FlatArgs& a) {
    if (kind == 0)
        return nt ? flat_r<V, 0, true>(rows, lds, s, a) : flat_r<V, 0, false>(rows, lds, s, a);
    return nt ? flat_r<V, 1, true>(rows, lds, s, a) : flat_r<V, 1, false>(rows, lds, s, a);
}

hipError_t launch_generate_flat(int mulmod, int kind, bool nt, int rows, uint32_t lds,
                                hipStream_t s, const FlatArgs& a) {
    switch (mulmod) {
        case 1: return flat_v<VarFP64>(kind, nt, rows, lds, s, a);
        case 2: return flat_v<VarBarrett>(kind, nt, rows, lds, s, a);
        case 3: return flat_v<VarShoup>(kind, nt, rows, lds, s, a);
        case 4: return flat_v<VarMontgomery>(kind, nt, rows, lds, s, a);
        default: return hipErrorInvalidValue;
    }
}

template <bool NT, int R, bool START>
static hipError_t fill_flat_one(uint32_t lds, hipStream_t s, const FlatArgs& a, uint64_t value) {
    if (flat_whole(a)) {
        if constexpr (flat_xcd_run(R) != 0) {
            if (a.runs) {
                hipLaunchKernelGGL((k_fill_flat<NT, R, START, flat_xcd_run(R)>), dim3(a.full),
                                   dim3(kFlatBlock), lds, s, a.out, value);
                return hipGetLastError();
            }
        }
        hipLaunchKernelGGL((k_fill_flat<NT, R, START, 0>), dim3(a.full), dim3(kFlatBlock), lds, s,
                           a.out, value);
        return hipGetLastError();
    }
    hipLaunchKernelGGL((k_fill_flat_any<NT, R, START>), dim3(flat_grid(a)), dim3(kFlatBlock), lds,
                       s, a, value);
    return hipGetLastError();
}

template <bool NT, bool START>
static hipError_t fill_flat_r(int rows, uint32_t lds, hipStream_t s, const FlatArgs& a,
                              uint64_t value) {
    switch (rows) {
        case 1: return fill_flat_one<NT, 1, START>(lds, s, a, value);
        case 2: return fill_flat_one<NT, 2, START>(lds, s, a, value);
        case 4: return fill_flat_one<NT, 4, START>(lds, s, a, value);
        case 8: return fill_flat_one<NT, 8, START>(lds, s, a, value);
        case 16: return fill_flat_one<NT, 16, START>(lds, s, a, value);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_fill_flat(bool nt, int rows, uint32_t lds, hipStream_t s, bool start,
                            const FlatArgs& a, uint64_t value) {
    if (start)
        return nt ? fill_flat_r<true, true>(rows, lds, s, a, value)
                  : fill_flat_r<false, true>(rows, lds, s, a, value);
    return nt ? fill_flat_r<true, false>(rows, lds, s, a, value)
              : fill_flat_r<false, false>(rows, lds, s, a, value);
}

// Kernel selector: W = 1, W = 2, or W = 2 with IL = 2 or 4 rows in flight.
// ------------------------------------------------------- consecutive --
// The paper's per-thread loop (Section 3.2) with its Modified Barrett step
// (Section 3.1), kept in serial memory order by an LDS transpose.  Element
// j = t*E + e of a tile sits at LDS word j + j/E (one pad word per thread,
// so the E-strided writes of a wavefront spread over the banks).
template <int KIND, int E, int W, bool NT>
__global__ __launch_bounds__(1024) void k_generate_consec(ConsecArgs a) {
    extern __shared__ uint64_t tile[];
    const uint32_t B = blockDim.x;
    const uint32_t t = threadIdx.x;
    const uint64_t per_tile = (uint64_t)B * E;
    const uint64_t n_tiles = (a.count + per_tile - 1) / per_tile;
    uint64_t ti = blockIdx.x;
    if (ti >= n_tiles) return;
    // The state of this thread's first element in tile ti.
    uint64_t z0 = thread_start<VarShoup>(a.base, ti * per_tile + (uint64_t)t * E, a.t_lo, a.t_hi);
    const global_ptr<uint64_t> out = as_global(a.out);
    for (; ti < n_tiles; ti += gridDim.x) {
        uint64_t z = z0;
#pragma unroll
        for (int e = 0; e < E; ++e) {
            const uint64_t bits = KIND == 0 ? z : (uint64_t)__double_as_longlong((double)z * kRecip);
            tile[t * (E + 1) + e] = bits;
            z = mm_modbarrett_step(z);
        }
        z0 = VarShoup::mul(z0, a.J);
        __syncthreads();
        const uint64_t first = ti * per_tile;
        const uint64_t here = a.count - first < per_tile ? a.count - first : per_tile;
        if (W == 2 && here == per_tile) {
#pragma unroll
            for (int i = 0; i < E / 2; ++i) {
                const uint32_t j = 2 * (i * B + t);  // even, so j and j+1 share a thread
                const uint32_t w = j + j / E;
                u64x2 v;
                v.x = tile[w];
                v.y = tile[w + 1];
                put<NT>(reinterpret_cast<global_ptr<u64x2>>(out + first + j), v);
            }
        } else {
            for (uint32_t j = t; j < here; j += B) put<NT>(out + first + j, tile[j + j / E]);
        }
        __syncthreads();  // the next tile reuses the LDS
    }
}

template <int KIND, int E, int W>
static hipError_t consec_one(bool nt, uint32_t grid, uint32_t block, hipStream_t s,
                             const ConsecArgs& a) {
    const uint32_t lds = consec_lds_bytes(block, E);
    if (nt) {
        k_generate_consec<KIND, E, W, true><<<grid, block, lds, s>>>(a);
    } else {
        k_generate_consec<KIND, E, W, false><<<grid, block, lds, s>>>(a);
    }
    return hipGetLastError();
}

template <int KIND, int W>
static hipError_t consec_e(int E, bool nt, uint32_t grid, uint32_t block, hipStream_t s,
                           const ConsecArgs& a) {
    switch (E) {
        case 2: return consec_one<KIND, 2, W>(nt, grid, block, s, a);
        case 4: return consec_one<KIND, 4, W>(nt, grid, block, s, a);
        case 8: return consec_one<KIND, 8, W>(nt, grid, block, s, a);
        case 16: return consec_one<KIND, 16, W>(nt, grid, block, s, a);
        case 32: return consec_one<KIND, 32, W>(nt, grid, block, s, a);
        default: return hipErrorInvalidValue;
    }
}

hipError_t launch_generate_consec(int kind, int E, int width, bool nt, uint32_t grid,
                                  uint32_t block, hipStream_t s, const ConsecArgs& a) {
    if (kind == 0)
        return width == 2 ? consec_e<0, 2>(E, nt, grid, block, s, a)
                          : consec_e<0, 1>(E, nt, grid, block, s, a);
    return width == 2 ? consec_e<1, 2>(E, nt, grid, block, s, a)
                      : consec_e<1, 1>(E, nt, grid, block, s, a);
}

template <class V, int KIND, int W, int IL, int U, bool NT>
static hipError_t gen_one(uint32_t grid, uint32_t block, hipStream_t s, const GenArgs& a) {
    if constexpr (W == 1)
        hipLaunchKernelGGL((k_generate1<V, KIND, U, NT>), dim3(grid), dim3(block), 0, s, a.out,
                           a.T, a.e_full, a.rem, a.base, a.J, a.M1, a.t_lo, a.t_hi);
    else if constexpr (IL == 1)
        hipLaunchKernelGGL((k_generate2<V, KIND, U, NT>), dim3(grid), dim3(block), 0, s, a.out,
                           a.T, a.e_full, a.rem, a.base, a.J, a.M1, a.t_lo, a.t_hi);
    else
        hipLaunchKernelGGL((k_generate2_ilp<V, KIND, U, NT, IL>), dim3(grid), dim3(block), 0, s,
                           a.out, a.T, a.e_full, a.rem, a.base, a.J, a.M1, a.JI, a.t_lo,
                           a.t_hi);
    return hipGetLastError();
}

template <class V, int KIND, int W, int IL, bool NT>
static hipError_t gen_u(int unroll, uint32_t grid, uint32_t block, hipStream_t s,
                        const GenArgs& a) {
    switch (unroll) {
        case 1: return gen_one<V, KIND, W, IL, 1, NT>(grid, block, s, a);
        case 2: return gen_one<V, KIND, W, IL, 2, NT>(grid, block, s, a);
        case 4: return gen_one<V, KIND, W, IL, 4, NT>(grid, block, s, a);
        case 8: return gen_one<V, KIND, W, IL, 8, NT>(grid, block, s, a);
        default: return hipErrorInvalidValue;
    }
}

template <class V, int KIND, int W, int IL>
static hipError_t gen_n(int unroll, bool nt, uint32_t grid, uint32_t block, hipStream_t s,
                        const GenArgs& a) {
    return nt ? gen_u<V, KIND, W, IL, true>(unroll, grid, block, s, a)
              : gen_u<V, KIND, W, IL, false>(unroll, grid, block, s, a);
}

template <class V, int KIND>
static hipError_t gen_k(int width, int unroll, int ilp, bool nt, uint32_t grid, uint32_t block,
                        hipStream_t s, const GenArgs& a) {
    if (width == 1 && ilp == 1) return gen_n<V, KIND, 1, 1>(unroll, nt, grid, block, s, a);
    if (width == 2 && ilp == 1) return gen_n<V, KIND, 2, 1>(unroll, nt, grid, block, s, a);
    if (width == 2 && ilp == 2) return gen_n<V, KIND, 2, 2>(unroll, nt, grid, block, s, a);
    if (width == 2 && ilp == 4) return gen_n<V, KIND, 2, 4>(unroll, nt, grid, block, s, a);
    return hipErrorInvalidValue;
}

template <class V>
static hipError_t gen_v(int kind, int width, int unroll, int ilp, bool nt, uint32_t grid,
                        uint32_t block, hipStream_t s, const GenArgs& a) {
    return kind == 0 ? gen_k<V, 0>(width, unroll, ilp, nt, grid, block, s, a)
                     : gen_k<V, 1>(width, unroll, ilp, nt, grid, block, s, a);
}

hipError_t launch_generate(int mulmod, int kind, int width, int unroll, int ilp, bool nt,
                           uint32_t grid, uint32_t block, hipStream_t s, const GenArgs& a) {
    switch (mulmod) {
        case 1: return gen_v<VarFP64>(kind, width, unroll, ilp, nt, grid, block, s, a);
        case 2: return gen_v<VarBarrett>(kind, width, unroll, ilp, nt, grid, block, s, a);
        case 3: return gen_v<VarShoup>(kind, width, unroll, ilp, nt, grid, block, s, a);
        case 4: return gen_v<VarMontgomery>(kind, width, unroll, ilp, nt, grid, block, s, a);
        default: return hipErrorInvalidValue;
    }
}

template <int W, int U, bool NT>
static hipError_t fill_one(uint32_t grid, uint32_t block, hipStream_t s, uint64_t* out,
                           uint64_t T, uint64_t e_full, uint32_t rem, uint64_t value) {
    hipLaunchKernelGGL((k_fill<W, U, NT>), dim3(grid), dim3(block), 0, s, out, T, e_full, rem,
                       value);
    return hipGetLastError();
}

template <int W>
static hipError_t fill_w(int unroll, bool nt, uint32_t grid, uint32_t block, hipStream_t s,
                         uint64_t* out, uint64_t T, uint64_t e_full, uint32_t rem,
                         uint64_t value) {
#define NN_FILL_CASE(U)                                                              \
    case U:                                                                          \
        return nt ? fill_one<W, U, true>(grid, block, s, out, T, e_full, rem, value) \
                  : fill_one<W, U, false>(grid, block, s, out, T, e_full, rem, value);
    switch (unroll) {
        NN_FILL_CASE(1)
        NN_FILL_CASE(2)
        NN_FILL_CASE(4)
        NN_FILL_CASE(8)
        default: return hipErrorInvalidValue;
    }
#undef NN_FILL_CASE
}

hipError_t launch_fill(int width, int unroll, bool nt, uint32_t grid, uint32_t block,
                       hipStream_t s, uint64_t* out, uint64_t T, uint64_t e_full, uint32_t rem,
                       uint64_t value) {
    if (width == 1) return fill_w<1>(unroll, nt, grid, block, s, out, T, e_full, rem, value);
    if (width == 2) return fill_w<2>(unroll, nt, grid, block, s, out, T, e_full, rem, value);
    return hipErrorInvalidValue;
}

}  // namespace nn
