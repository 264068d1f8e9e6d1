// device.hpp -- gfx950 device building blocks shared by the library's kernels:
// storage/compute type traits, 16-byte packed global loads and stores,
// error-free transformations, and wave64 and work-group float64 reductions.
//
// Cross-work-group combines are done by a second, small kernel rather than by
// a "last work-group" ticket inside the first: on gfx950 every agent-scope
// fence that such a ticket needs writes back and invalidates the XCD's L2,
// which serialises badly across thousands of work-groups.  The kernel
// boundary gives the visibility for free and keeps the combine order fixed.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace bwla {

using bf16_t = __bf16;

// Compute precision of a storage type: double for f64, float for f32/bf16.
template <typename T> struct Compute;
template <> struct Compute<double> { using type = double; };
template <> struct Compute<float> { using type = float; };
template <> struct Compute<bf16_t> { using type = float; };
template <typename T> using compute_t = typename Compute<T>::type;

template <typename T> __device__ __forceinline__ compute_t<T> widen(T v) { return (compute_t<T>)v; }
// float -> bf16 conversion is an LLVM fptrunc, round to nearest even (a single
// v_cvt_pk_bf16_f32 on gfx950).
template <typename T> __device__ __forceinline__ T narrow(compute_t<T> v) { return (T)v; }

__device__ __forceinline__ double fma_c(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_c(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// ---------------------------------------------------------------------------
// Packed global memory access: V consecutive elements per thread.  Packs of
// 16 bytes or more are moved as 16-byte (dwordx4) accesses; smaller packs as
// one 8/4/2-byte access.  A pack may start on any element: the word types
// below claim the smallest element's alignment only, and the compiler still issues
// one dwordx4 for them, because gfx950 runs with unaligned global access enabled.
// What a misaligned pack costs is the extra cache line that a wave's 1 KiB
// then touches; element-wide accesses, to which a misaligned operand once fell
// back, cost 2 (f64) to 8 (bf16) times the instructions.  Measured, element
// accesses against packs: slices of 10^7 bf16, axpby 32.0 -> 12.3 us, copy 15.4
// -> 8.8, dot 14.6 -> 8.3, nrm2 9.3 -> 4.8; y = A x with rows of an odd length,
// 8001 x 8003 bf16 32.2 -> 24.9 us, 5001 x 5003 f64 38.5 -> 34.5 us, and the
// transposed bf16 product 41.8 -> 29.0 us.
// ---------------------------------------------------------------------------
typedef uint32_t word4 __attribute__((ext_vector_type(4), aligned(2)));
typedef uint32_t word2 __attribute__((ext_vector_type(2), aligned(2)));
typedef uint32_t word1 __attribute__((aligned(2)));

template <typename T, int V> struct Pack {
    T v[V];
};

// NT: the nontemporal hint, for data touched exactly once -- vector operands,
// the matrix of a GEMV, outputs.  It keeps once-read streams from displacing
// reusable lines in the caches; measured on MI355X, copy goes from ~6.0 to
// ~6.6 TB/s and a read-only stream from ~6.3 to ~7.0 TB/s.
// (A function each: a template parameter would drop the type's alignment.)
#define BWLA_WORD(W)                                                                                   \
    template <bool NT> __device__ __forceinline__ W load_##W(const W *p)                               \
    {                                                                                                  \
        if constexpr (NT)                                                                              \
            return __builtin_nontemporal_load(p);                                                      \
        else                                                                                           \
            return *p;                                                                                 \
    }                                                                                                  \
    __device__ __forceinline__ void store_nt_##W(W *p, W v) { __builtin_nontemporal_store(v, p); }
BWLA_WORD(word4)
BWLA_WORD(word2)
BWLA_WORD(word1)
BWLA_WORD(uint16_t)
#undef BWLA_WORD

template <typename T, int V, bool NT = false>
__device__ __forceinline__ Pack<T, V> load_pack(const T *p)
{
    constexpr int B = V * (int)sizeof(T);
    Pack<T, V> r;
    if constexpr (B >= 16) {
        const auto *s = reinterpret_cast<const word4 *>(p);
        word4 tmp[B / 16];
#pragma unroll
        for (int i = 0; i < B / 16; ++i)
            tmp[i] = load_word4<NT>(s + i);
        __builtin_memcpy(&r, tmp, B);
    } else if constexpr (B == 8) {
        const word2 tmp = load_word2<NT>(reinterpret_cast<const word2 *>(p));
        __builtin_memcpy(&r, &tmp, B);
    } else if constexpr (B == 4) {
        const word1 tmp = load_word1<NT>(reinterpret_cast<const word1 *>(p));
        __builtin_memcpy(&r, &tmp, B);
    } else {
        const uint16_t tmp = load_uint16_t<NT>(reinterpret_cast<const uint16_t *>(p));
        __builtin_memcpy(&r, &tmp, B);
    }
    return r;
}
template <typename T, int V>
__device__ __forceinline__ Pack<T, V> load_pack_nt(const T *p)
{
    return load_pack<T, V, true>(p);
}

// Ends the load phase of an unrolled trip: no instruction moves across it,
// so every load issued above is in flight before the arithmetic below starts.
// Without it the machine scheduler sinks part of a trip's loads into the
// arithmetic (to shorten register live ranges) and waits on each at once,
// which cuts the bytes a wave keeps in flight -- on gfx950 down to one or two
// packs for some compensated instantiations, halving their bandwidth.
__device__ __forceinline__ void end_of_loads() { __builtin_amdgcn_sched_barrier(0); }

// Streaming (nontemporal) store of a pack.
template <typename T, int V>
__device__ __forceinline__ void store_pack_nt(T *p, const Pack<T, V> &r)
{
    constexpr int B = V * (int)sizeof(T);
    if constexpr (B >= 16) {
        word4 tmp[B / 16];
        __builtin_memcpy(tmp, &r, B);
        auto *d = reinterpret_cast<word4 *>(p);
#pragma unroll
        for (int i = 0; i < B / 16; ++i)
            store_nt_word4(d + i, tmp[i]);
    } else if constexpr (B == 8) {
        word2 tmp;
        __builtin_memcpy(&tmp, &r, B);
        store_nt_word2(reinterpret_cast<word2 *>(p), tmp);
    } else if constexpr (B == 4) {
        word1 tmp;
        __builtin_memcpy(&tmp, &r, B);
        store_nt_word1(reinterpret_cast<word1 *>(p), tmp);
    } else {
        uint16_t tmp;
        __builtin_memcpy(&tmp, &r, B);
        store_nt_uint16_t(reinterpret_cast<uint16_t *>(p), tmp);
    }
}

// The elements of a vector outside its packs: `head` before the first pack
// (negative indices from it, fewer than 64) and the last n - packed, all taken
// by the first threads of work-group 0.  n and the indices count from the
// first pack.
template <typename F>
__device__ __forceinline__ void edge_elements(int head, int64_t packed, int64_t n, F &&f)
{
    if (blockIdx.x != 0)
        return;
    const int t = (int)threadIdx.x;
    if (t < head)
        f((int64_t)t - head);
    if (t < n - packed)
        f(packed + t);
}

// ---------------------------------------------------------------------------
// XCD-aware work-group numbering.  The hardware hands consecutive work-group
// ids to the 8 XCDs in turn; renumbering so that each XCD's work-groups
// cover one contiguous range of the logical index space keeps each XCD on
// its own stretch of memory.  A bijection on [0, gridDim.x) for any grid size.
// ---------------------------------------------------------------------------
// In 32 bits (a grid has fewer than 2^31 work-groups), so that no branch of a
// 64-bit division splits a kernel's first block and all of its arguments are
// loaded at once: each such split was one more serial load of arguments before
// the first load of data (with the slice index and length done alike, columns
// of 4096 x 4096 f32 16.8 -> 16.0 us, rows of 1453 x 116 3.2 -> 2.8).
constexpr int kXcds = 8;
__device__ __forceinline__ int64_t xcd_block()
{
    const unsigned g = gridDim.x, b = blockIdx.x;
    const unsigned xcd = b % kXcds, idx = b / kXcds;
    const unsigned q = g / kXcds, r = g % kXcds;
    return xcd * q + (xcd < r ? xcd : r) + idx;
}

// ---------------------------------------------------------------------------
// Error-free transformations (exact for finite values without overflow).
// ---------------------------------------------------------------------------
// s + e == a + b, s = RN(a + b)   (Knuth)
template <typename C> __device__ __forceinline__ void two_sum(C a, C b, C &s, C &e)
{
    s = a + b;
    C bv = s - a;
    e = (a - (s - bv)) + (b - bv);
}
// s + e == a + b given |a| >= |b| or a == 0   (Dekker)
template <typename C> __device__ __forceinline__ void fast_two_sum(C a, C b, C &s, C &e)
{
    s = a + b;
    e = b - (s - a);
}

// |a| in the compute precision (clears the sign bit: |-0| = +0).
__device__ __forceinline__ float abs_c(float a) { return __builtin_fabsf(a); }
__device__ __forceinline__ double abs_c(double a) { return __builtin_fabs(a); }

// A float64 value carried with its rounding error (hi + lo, |lo| <= ulp(hi)/2).
struct DD {
    double hi, lo;
};

// Once the sum is infinite or NaN the error terms are meaningless (inf - inf)
// and the IEEE value of the sum is the plain sum, which is kept with lo = 0.
__device__ __forceinline__ DD dd_add(DD a, DD b)
{
    double s, e;
    two_sum(a.hi, b.hi, s, e);
    DD r;
    if (!__builtin_isfinite(s)) {
        r.hi = s;
        r.lo = 0.0;
        return r;
    }
    e += a.lo + b.lo;
    fast_two_sum(s, e, r.hi, r.lo);
    return r;
}

// Accumulator of a reduction.  PLAIN keeps one running sum; COMPENSATED keeps
// the running sum and the gathered rounding errors of products and sums.
template <typename C, bool COMP> struct Acc {
    C s = 0, e = 0;
    // s += a*b.  EXACT_PROD: a*b is exact in C (bf16 operands in float), so
    // no product error is gathered.
    template <bool EXACT_PROD>
    __device__ __forceinline__ void add_prod(C a, C b)
    {
        if constexpr (!COMP) {
            s = fma_c(a, b, s);
        } else {
            C h = a * b;
            C q, t;
            two_sum(s, h, t, q);
            s = t;
            if constexpr (EXACT_PROD) {
                e += q;
            } else {
                C r = fma_c(a, b, -h);
                e += q + r;
            }
        }
    }
    __device__ __forceinline__ void merge(const Acc &o)
    {
        if constexpr (!COMP) {
            s += o.s;
        } else {
            C t, q;
            two_sum(s, o.s, t, q);
            s = t;
            e += q + o.e;
        }
    }
    __device__ __forceinline__ void fold() {}
    // Leave the thread as a float64 pair.
    __device__ __forceinline__ DD to_dd() const
    {
        DD r;
        if constexpr (!COMP) {
            r.hi = (double)s;
            r.lo = 0.0;
        } else if (!__builtin_isfinite(s)) { // see dd_add
            r.hi = (double)s;
            r.lo = 0.0;
        } else {
            fast_two_sum((double)s, (double)e, r.hi, r.lo);
        }
        return r;
    }
};

// Compensated accumulator of bf16 storage: a float64 sum.  The products of two
// bf16 values are exact in float64, so one fma per term is all, and its error
// (2^-53 per term) is below that of a float32 sum that carries its error (2^-48).
// On gfx950 float64 fma issues at the float32 rate, so a term costs a conversion
// and an fma where the TwoSum of the float32 form took seven adds and a product:
// y = A x 16384 x 16384 89.7 -> 84.8 us, 3001 x 4099 9.7 -> 9.0, transposed 300 x 300 6.3 ->
// 5.4, dot of 2^26 44.9 -> 43.8, the uneven batch's GEMV tiles 216 -> 204.
struct AccF64 {
    double s = 0;
    template <bool EXACT_PROD>
    __device__ __forceinline__ void add_prod(float a, float b)
    {
        s = __builtin_fma((double)a, (double)b, s);
    }
    __device__ __forceinline__ void fold() {}
    __device__ __forceinline__ DD to_dd() const { return DD{s, 0.0}; }
};

// Plain accumulator of a sum in short runs, so that the error does not grow with
// the terms of a thread, and the number of threads that share a sum can follow
// speed alone: a run is summed in the compute precision, and fold() adds it to the
// thread's sum, in float64 also for float32 (S).  A run is one pack of f32, two of bf16,
// four of f64, or a trip's lines.  Error of GEMV rows before the output is rounded
// (root mean square, in units of 2^-24 or 2^-53 of a random sum's size), one running sum
// per thread -> this: 4096 x 4096 f32 2.5 -> 0.67, bf16 0.74 -> 0.31, f64 2.7 -> 1.8; 2048 x
// 16384 f32 3.3 -> 0.67; 100 x 640000 f64 11 -> 2.3.  GPU time within 2 %.
template <typename C, typename S = double> struct AccFold {
    C t = 0;
    S s = 0;
    template <bool EXACT_PROD> __device__ __forceinline__ void add_prod(C a, C b) { t = fma_c(a, b, t); }
    __device__ __forceinline__ void fold()
    {
        s += (S)t;
        t = 0;
    }
    __device__ __forceinline__ DD to_dd() const { return DD{(double)s + (double)t, 0.0}; }
};
template <typename T> constexpr int kRunPacks = sizeof(T) == 8 ? 4 : sizeof(T) == 4 ? 1 : 2;
constexpr int kRunLines = 4;

template <typename T, bool COMP>
using acc_t = std::conditional_t<!COMP, AccFold<compute_t<T>>,
                                 std::conditional_t<std::is_same_v<T, bf16_t>, AccF64, Acc<compute_t<T>, true>>>;
// The compensated CG update keeps the float32 form: four streams per term, and
// the conversions would sit between a trip's loads.
template <typename C, bool COMP> using cg_acc_t = std::conditional_t<COMP, Acc<C, true>, AccFold<C>>;
// The cols kernel with several lines per access adds a trip's lines to a sum in the compute
// precision: its 4 or 8 outputs per lane would take as many conversions per trip, with one
// wave per SIMD to hide them (4096 x 4096 f32 15.9 us, 15.7 so; error 0.67 and 1.3 of the
// units above, 2.4 as one running sum).
template <typename T, bool COMP>
using trip_acc_t = std::conditional_t<!COMP, AccFold<compute_t<T>, compute_t<T>>, acc_t<T, COMP>>;
// The cols kernel with one line per access, where one wave may take all lines:
// a float64 sum of exact products for float32.
template <typename T, bool COMP>
using line_acc_t = std::conditional_t<!COMP && !std::is_same_v<T, double>, AccF64, acc_t<T, COMP>>;

template <bool COMP> __device__ __forceinline__ DD combine(DD a, DD b)
{
    if constexpr (COMP) {
        return dd_add(a, b);
    } else {
        DD r;
        r.hi = a.hi + b.hi;
        r.lo = 0.0;
        return r;
    }
}

// ---------------------------------------------------------------------------
// Wave64 reduction.  Butterfly exchanges: DPP quad permutations and row
// mirrors inside each 16-lane row, then cross-row exchanges.  Partners
// compute a+b and b+a, which round identically, so every lane ends with the
// bitwise same total and the pattern is fixed (deterministic).
// ---------------------------------------------------------------------------
template <int CTRL> __device__ __forceinline__ double dpp_f64(double v)
{
    int2 b = __builtin_bit_cast(int2, v);
    int lo = __builtin_amdgcn_update_dpp(0, b.x, CTRL, 0xF, 0xF, false);
    int hi = __builtin_amdgcn_update_dpp(0, b.y, CTRL, 0xF, 0xF, false);
    return __builtin_bit_cast(double, make_int2(lo, hi));
}
constexpr int kDppXor1 = 0xB1;       // quad_perm [1,0,3,2]
constexpr int kDppXor2 = 0x4E;       // quad_perm [2,3,0,1]
constexpr int kDppHalfMirror = 0x141; // lane i <-> 7-i within 8 lanes
constexpr int kDppMirror = 0x140;     // lane i <-> 15-i within 16 lanes
constexpr int kDppXor8 = 0x128;       // row_ror 8: lane i <-> i^8 within 16 lanes

template <int CTRL> __device__ __forceinline__ DD dpp_dd(DD v)
{
    DD r;
    r.hi = dpp_f64<CTRL>(v.hi);
    r.lo = dpp_f64<CTRL>(v.lo);
    return r;
}
__device__ __forceinline__ DD shfl_xor_dd(DD v, int m)
{
    DD r;
    r.hi = __shfl_xor(v.hi, m);
    r.lo = __shfl_xor(v.lo, m);
    return r;
}

template <bool COMP> __device__ __forceinline__ DD wave_sum(DD v)
{
    v = combine<COMP>(v, dpp_dd<kDppXor1>(v));
    v = combine<COMP>(v, dpp_dd<kDppXor2>(v));
    v = combine<COMP>(v, dpp_dd<kDppHalfMirror>(v));
    v = combine<COMP>(v, dpp_dd<kDppMirror>(v));
    v = combine<COMP>(v, shfl_xor_dd(v, 16));
    v = combine<COMP>(v, shfl_xor_dd(v, 32));
    return v;
}

// The halves (M = 32) or the odd and even 16-lane rows (M = 16) of two values
// exchanged and added: lanes with bit M clear end with a summed over the lane
// pair, the others with b.  One gfx950 lane swap per 32-bit word and no LDS.
template <int M> __device__ __forceinline__ void swap_lanes(uint32_t &a, uint32_t &b)
{
    const auto r = M == 32 ? __builtin_amdgcn_permlane32_swap(a, b, false, false)
                           : __builtin_amdgcn_permlane16_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}
template <int M> __device__ __forceinline__ void swap_lanes(double &a, double &b)
{
    uint2 x = __builtin_bit_cast(uint2, a), y = __builtin_bit_cast(uint2, b);
    swap_lanes<M>(x.x, y.x);
    swap_lanes<M>(x.y, y.y);
    a = __builtin_bit_cast(double, x);
    b = __builtin_bit_cast(double, y);
}
template <bool COMP, int M> __device__ __forceinline__ DD pair_sum(DD a, DD b)
{
    swap_lanes<M>(a.hi, b.hi);
    if constexpr (COMP)
        swap_lanes<M>(a.lo, b.lo);
    return combine<COMP>(a, b);
}

// Sums of 2 N values over the lane pairs that differ in bit BIT: each lane is
// left with N of them in d[0 .. N - 1], the upper half where its bit is set.  (Below
// bit 4 the pair is exchanged by selects and one DPP move; the half mirror
// pairs lanes 7 apart from the other end, which a sum over all 8 may use.)
template <bool COMP, int BIT, int N> __device__ __forceinline__ void halve(DD *d, int lane)
{
#pragma unroll
    for (int e = 0; e < N; ++e) {
        if constexpr (BIT >= 4) {
            d[e] = pair_sum<COMP, 1 << BIT>(d[e], d[e + N]);
        } else {
            constexpr int CTRL = BIT == 3 ? kDppXor8 : BIT == 2 ? kDppHalfMirror : BIT == 1 ? kDppXor2 : kDppXor1;
            const bool up = lane & (1 << BIT);
            const DD keep = up ? d[e + N] : d[e], give = up ? d[e] : d[e + N];
            d[e] = combine<COMP>(keep, dpp_dd<CTRL>(give));
        }
    }
}

// Sum over one work-group (blockDim.x a multiple of 64, at most 1024).  `lds`
// holds at least 16 DD.  The result is valid in every thread.  Contains
// barriers: every thread of the block must call it.
template <bool COMP> __device__ __forceinline__ DD block_sum(DD v, DD *lds)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nw = blockDim.x >> 6;
    v = wave_sum<COMP>(v);
    if (lane == 0)
        lds[wave] = v;
    __syncthreads();
    DD t = {0.0, 0.0};
    if (lane < nw)
        t = lds[lane];
    t = wave_sum<COMP>(t);
    __syncthreads(); // lds may be reused by the caller afterwards
    return t;
}

// Rounds a float64 result to the output element type.
__device__ __forceinline__ void store_out(void *out, int64_t i, int out_f64, double v)
{
    if (out_f64)
        reinterpret_cast<double *>(out)[i] = v;
    else
        reinterpret_cast<float *>(out)[i] = (float)v;
}

} // namespace bwla
