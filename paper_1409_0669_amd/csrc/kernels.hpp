// kernels.hpp -- host-side launchers of the gfx950 kernels (internal).  Each
// kernel source is compiled once per storage type; the API layer validates
// arguments and resolves the configuration before calling these.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

namespace bwla {

// Resolved kernel configuration (no zero fields left).
struct Cfg {
    int block, vec, unroll, grid, inc, rows, split;
    int head = 0; // vector operations: elements before the first pack (see pack_head in api.cpp)
};

// The workspace of a reduction holds its float64 partials (DD pairs).
constexpr size_t kColsXchgBytes = 32768; // largest dynamic LDS of the cols kernel's wave combine
// The cols kernel keeps 16 or 32 lines in flight per wave only while the
// bytes of A each lane holds in flight stay within this (32 VGPRs): beyond
// it the loads would spill.  Up to 8 lines are always allowed.
constexpr size_t kColsLoadBytes = 128;

// Map a runtime value onto a compile-time constant for template dispatch.
template <typename F> hipError_t with_vec(int v, F &&f)
{
    switch (v) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 8: return f(std::integral_constant<int, 8>{});
    case 16: return f(std::integral_constant<int, 16>{});
    }
    return hipErrorInvalidValue;
}
template <typename F> hipError_t with_unroll(int u, F &&f)
{
    switch (u) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 4: return f(std::integral_constant<int, 4>{});
    }
    return hipErrorInvalidValue;
}
template <typename F> hipError_t with_rows(int r, F &&f)
{
    switch (r) {
    case 1: return f(std::integral_constant<int, 1>{});
    case 2: return f(std::integral_constant<int, 2>{});
    case 4: return f(std::integral_constant<int, 4>{});
    case 8: return f(std::integral_constant<int, 8>{});
    }
    return hipErrorInvalidValue;
}
template <typename F> hipError_t with_bool(bool b, F &&f)
{
    if (b)
        return f(std::integral_constant<bool, true>{});
    return f(std::integral_constant<bool, false>{});
}

// --- streaming: copy, axpby, fused CG update --------------------------------
template <typename T>
hipError_t launch_copy(int64_t n, const void *y, void *x, const Cfg &c, hipStream_t s);
template <typename T>
hipError_t launch_scal(int64_t n, double alpha, const void *adev, const void *y, void *x, const Cfg &c,
                       hipStream_t s);
template <typename T>
hipError_t launch_axpby(int64_t n, double alpha, const void *adev, const void *y, double beta,
                        const void *bdev, const void *z, void *x, const Cfg &c, hipStream_t s);
template <typename T>
hipError_t launch_cg(int64_t n, bool comp, double alpha, const void *adev, void *x, const void *p,
                     void *r, const void *q, int out_f64, void *out, void *ws, const Cfg &c,
                     hipStream_t s);

// --- reductions: dot, nrm2, asum (mode kRedDot, kRedSq, kRedAbs) -----------
// Partials needed: c.grid DD pairs.
template <typename T>
hipError_t launch_dot(int64_t n, bool comp, int mode, const void *x, const void *y, int out_f64,
                      void *out, void *ws, const Cfg &c, hipStream_t s);

// --- vectors with an increment (BLAS convention; see strided.hip) ----------
enum { kElemCopy = 0, kElemAxpby = 1, kElemScal = 2 };
enum { kRedDot = 0, kRedSq = 1, kRedAbs = 2 };
constexpr int kStridedBlock = 256; // threads per work-group
constexpr int kStridedUnroll = 4;  // elements in flight per thread
// x = copy(y) / RN(fma(a, y, RN(b z))) / RN(a y) with a, b the effective
// factors (host value times *adev / *bdev when given).
template <typename T>
hipError_t launch_strided_elem(int mode, int64_t n, double alpha, const void *adev, double beta,
                               const void *bdev, const void *y, int64_t incy, const void *z, int64_t incz,
                               void *x, int64_t incx, int grid, hipStream_t s);
// <x, y>, sqrt(sum x_i^2) or sum |x_i|; `grid` DD partials in ws when grid > 1.
template <typename T>
hipError_t launch_strided_reduce(int mode, int64_t n, bool comp, const void *x, int64_t incx, const void *y,
                                 int64_t incy, int out_f64, void *out, void *ws, int grid, hipStream_t s);

// --- matrix-vector ---------------------------------------------------------
// Where and how a GEMV stores its results: s_i = RN(result i) in the output type
// O, then y[i * inc] = s_i, RN(a s_i), or RN(fma(a, s_i, RN(b y[i * inc]))) with a
// and b rounded to O.  y points at logical entry 0 (a negative increment walks
// backwards from it).
enum { kOutStore = 0, kOutScale = 1, kOutUpdate = 2 };
struct GemvOut {
    void *y;
    int f64, mode;
    int64_t inc;
    double a, b;
};
inline GemvOut gemv_store(void *y, int f64) { return GemvOut{y, f64, kOutStore, 1, 1.0, 0.0}; }
// A line is a contiguous run of K elements; lines are ld apart.
//   rows kernel:  out[l] = sum_k A[l*ld + k] * v[k]     (l < L)
//   cols kernel:  out[k] = sum_l A[l*ld + k] * v[l]     (k < K)
// ws holds the split partials from offset 0.  With w != NULL (same element
// type as out, one entry per output) the launch also writes
// *dot = sum_o w[o] * out[o], using gemv_dot_parts() float64 pairs at byte
// offset dparts_offset of ws.
// The cols kernels read v[l] at v[l * incv].
template <typename T>
hipError_t launch_gemv_rows(int64_t L, int64_t K, bool comp, const void *A, int64_t ld,
                            const void *v, const GemvOut &out, void *ws, const Cfg &c,
                            hipStream_t s, const void *w = nullptr, size_t dparts_offset = 0,
                            int dot_f64 = 1, void *dot = nullptr);
template <typename T>
hipError_t launch_gemv_cols(int64_t L, int64_t K, bool comp, const void *A, int64_t ld,
                            const void *v, int64_t incv, const GemvOut &out, void *ws, const Cfg &c,
                            hipStream_t s, const void *w = nullptr, size_t dparts_offset = 0,
                            int dot_f64 = 1, void *dot = nullptr);
// The line combine's work-groups: 256 outputs for a split of up to kCombineOne
// (one thread each), else kCombineRuns threads per output.
constexpr int kCombineOne = 8, kCombineRuns = 8;
inline int64_t combine_lines_outputs(int64_t split) { return split <= kCombineOne ? 256 : 256 / kCombineRuns; }
// Outputs of one work-group of the cols kernel (c.rows: lines per wave access).
inline int64_t cols_tile(const Cfg &c) { return (int64_t)(64 / c.rows) * c.vec; }
// Number of float64 pairs the dot epilogue writes: one per work-group of the
// kernel that stores y (the rows or cols kernel, or the line combine when
// split > 1).
inline int64_t gemv_dot_parts(bool rows, int64_t L, int64_t K, const Cfg &c)
{
    const int64_t outputs = rows ? L : K;
    if (c.split > 1)
        return (outputs + combine_lines_outputs(c.split) - 1) / combine_lines_outputs(c.split);
    return rows ? (L + c.rows - 1) / c.rows : (K + cols_tile(c) - 1) / cols_tile(c);
}
// --- rank-1 overwrite: A[l*ld + k] = a[l] * b[k] ---------------------------
template <typename T>
hipError_t launch_ger(int64_t L, int64_t K, const void *a, const void *b, void *A, int64_t ld,
                      const Cfg &c, hipStream_t s);

// --- zero fill of `count` outputs of float64 or float32 ---------------------
hipError_t launch_fill_zero(void *out, int64_t count, int out_f64, hipStream_t s);

// --- second stage of the reductions (type independent) ----------------------
// out = sum of `count` DD partials in index order (sqrt applied if asked).
hipError_t launch_combine_scalar(const void *partials, int64_t count, bool comp, bool do_sqrt,
                                 int out_f64, void *out, hipStream_t s);
// out[o] = sum over q < split of partials[((o / G) * split + q) * G + o % G],
// for o < outputs: the slices of a split GEMV combined in slice order.  With
// w != NULL, work-group b also writes dparts[b] = sum of w[o] * out[o] over
// its combine_lines_outputs(split) outputs.
hipError_t launch_combine_lines(const void *partials, int64_t outputs, int64_t G, int64_t split,
                                bool comp, const GemvOut &out, const void *w, void *dparts,
                                hipStream_t s);

// --- batched persistent kernel ----------------------------------------------
struct BatchItem {
    int32_t kind;   // 0 = GEMV row tile, 1 = dot chunk
    int32_t prob;   // problem index within its kind
    int64_t begin;  // first row (GEMV) or first element (dot)
    int64_t end;    // one past the last row / element
    int32_t chunk;  // chunk index within the dot
    int32_t pad;
};
// How the grouped launch reads one problem (the persistent kernel uses the
// plan-wide BatchArgs::vec instead).
enum {
    kModePacked = 0, // 16-byte packs of every operand (elements aligned to their size)
    kModeScalar = 1, // one element per access
    kModeLong = 2    // GEMV: packs, a work-group shares rows of more than long_from() entries
};
// Where a tile of 2^16 entries has too few rows for the waves to have their own
// (8 GEMVs of 300 rows, own -> shared: f64 2500 entries 18.2 -> 20.6 us, 3000 21.3 -> 18.6, f32 9.9 ->
// 13.0, 11.9 -> 10.7, bf16 3000 9.1 -> 9.4, 4096 10.7 -> 10.0), for elements of `es` bytes.
inline int64_t long_from(size_t es) { return es >= 4 ? 2816 : 4096; }
// Rows that a work-group shares at once: a tile of 2^16 entries holds 8 of up
// to 2^13 entries; longer rows, fewer, so that few rows still make many tiles.
inline int long_rows(int64_t n) { return n <= 8192 ? 8 : n <= 32768 ? 4 : 1; }
constexpr int kTileRows = 8;  // rows a lane group of a packed GEMV tile carries at once
// Default packs of a row each lane of a packed tile owns (sets its row-group size; plans take
// more than 8 as 8).
constexpr int kRowPacks = 16;
struct BatchGemv {
    const void *A;
    int64_t m, n, lda;
    const void *x;
    void *y;
    int32_t lanes; // lanes per row (power of two, <= 64; grouped launch, packs: 8 at least); kModeLong: long_rows
    int32_t mode;  // kMode*
};
struct BatchDot {
    const void *x, *y;
    int64_t n;
    void *out;
    int64_t slot0;  // first partial slot of this dot
    int32_t chunks; // number of chunks
    int32_t mode;   // kModePacked or kModeScalar
};
struct BatchArgs {
    const BatchItem *items;
    int64_t n_items;
    const BatchGemv *gemv;
    const BatchDot *dots;
    double *partials;       // 2 doubles per dot chunk
    unsigned *work_counter; // next item to take
    int out_f64;
    int vec;                // elements per pack: 1 or 16 bytes' worth
};
template <typename T>
hipError_t launch_batched(const BatchArgs &a, bool comp, int grid, int block, hipStream_t s);
hipError_t launch_batch_reset(unsigned *counters, int64_t count, hipStream_t s);
// One work-group per item (a.n_items work-groups of `block` threads).
template <typename T>
hipError_t launch_grouped(const BatchArgs &a, bool comp, int block, hipStream_t s);
// Combines the chunk partials of every multi-chunk dot: each lane of a wave every 64th in chunk
// order, then the lanes.
hipError_t launch_batch_finalize(const BatchDot *dots, int64_t nd, const double *partials, bool comp,
                                 int out_f64, hipStream_t s);

} // namespace bwla
