// batched.hip -- many uneven row-major GEMVs and dots, batched.
//
// Two designs share the work-item list.  The grouped launch (k_grouped, below
// the persistent kernel) runs one work-group per item; it is the one plans
// use.  The persistent kernel (k_batched) keeps a grid sized to the machine
// busy from an atomic work queue; it has not been validated on hardware and
// plan creation refuses it (see api.cpp).
//
// The host flattens every problem into work items -- row tiles of a GEMV
// (full row length) and fixed-size chunks of a dot -- ordered by decreasing
// cost.  The persistent kernel would launch a grid sized to the machine and
// be wave-persistent: each wave64 repeatedly takes the next item from an atomic
// counter (lane 0 draws, readfirstlane broadcasts) until the list is
// exhausted, and reduces its item within the wave, so the kernel has no LDS
// traffic and no work-group barriers -- waves never wait for each other and
// every wave reaches the exit.  GEMV rows are handled by groups of G lanes (G
// a power of two sized to the row length), reduced by butterfly exchanges
// inside the group.  A dot chunk is reduced across the wave; a single-chunk
// dot writes its result directly, otherwise the chunk's float64 partial goes
// to a slot of the dot and a small finalize kernel combines each dot's slots
// in a fixed order.  Every result depends only on its own problem's sizes, never
// on the batch order or on which wave ran which item.
#include "device.hpp"
#include "kernels.hpp"

namespace bwla {

template <typename T, int V, bool COMP>
__device__ __forceinline__ void gemv_tile(const BatchGemv &g, int64_t rb, int64_t re, int out_f64)
{
    using C = compute_t<T>;
    constexpr bool EXACT = std::is_same<T, bf16_t>::value;
    const int lane = threadIdx.x & 63;
    const int G = g.lanes;
    const int rpw = 64 / G;
    const int sub = lane / G, gl = lane - sub * G;
    const T *A = (const T *)g.A;
    const T *x = (const T *)g.x;
    const int64_t K = g.n, kpack = K / V;
    for (int64_t base = rb; base < re; base += rpw) {
        const int64_t r = base + sub;
        const int64_t rr = r < re ? r : re - 1;
        const T *row = A + rr * g.lda;
        acc_t<T, COMP> acc;
        for (int64_t p = gl; p < kpack; p += G) {
            Pack<T, V> av = load_pack<T, V>(row + p * V), xv = load_pack<T, V>(x + p * V);
#pragma unroll
            for (int e = 0; e < V; ++e)
                acc.template add_prod<EXACT>(widen(av.v[e]), widen(xv.v[e]));
        }
        for (int64_t k = kpack * V + gl; k < K; k += G)
            acc.template add_prod<EXACT>(widen(row[k]), widen(x[k]));
        DD d = acc.to_dd();
        for (int m = G >> 1; m >= 1; m >>= 1)
            d = combine<COMP>(d, shfl_xor_dd(d, m));
        if (gl == 0 && r < re)
            store_out(g.y, r, out_f64, d.hi + d.lo);
    }
}

template <typename T, int V, bool COMP>
__device__ __forceinline__ void dot_chunk(const BatchArgs &a, const BatchItem &w)
{
    using C = compute_t<T>;
    constexpr bool EXACT = std::is_same<T, bf16_t>::value;
    const int lane = threadIdx.x & 63;
    const BatchDot &d = a.dots[w.prob];
    const T *x = (const T *)d.x, *y = (const T *)d.y;
    acc_t<T, COMP> acc[2];
    const int64_t pb = w.begin / V, pe = w.end / V; // chunk starts are pack-aligned
    int64_t p = pb + lane;
    for (; p + 64 < pe; p += 128) {
        Pack<T, V> x0 = load_pack<T, V>(x + p * V), y0 = load_pack<T, V>(y + p * V);
        Pack<T, V> x1 = load_pack<T, V>(x + (p + 64) * V), y1 = load_pack<T, V>(y + (p + 64) * V);
#pragma unroll
        for (int e = 0; e < V; ++e) {
            acc[0].template add_prod<EXACT>(widen(x0.v[e]), widen(y0.v[e]));
            acc[1].template add_prod<EXACT>(widen(x1.v[e]), widen(y1.v[e]));
        }
    }
    for (; p < pe; p += 64) {
        Pack<T, V> x0 = load_pack<T, V>(x + p * V), y0 = load_pack<T, V>(y + p * V);
#pragma unroll
        for (int e = 0; e < V; ++e)
            acc[0].template add_prod<EXACT>(widen(x0.v[e]), widen(y0.v[e]));
    }
    const int64_t tail = w.end - pe * V; // < V, only in a dot's last chunk
    if (lane < tail)
        acc[0].template add_prod<EXACT>(widen(x[pe * V + lane]), widen(y[pe * V + lane]));
    DD v = wave_sum<COMP>(combine<COMP>(acc[0].to_dd(), acc[1].to_dd()));
    if (lane == 0) {
        if (d.chunks == 1)
            store_out(d.out, 0, a.out_f64, v.hi + v.lo);
        else
            reinterpret_cast<DD *>(a.partials)[d.slot0 + w.chunk] = v;
    }
}

template <typename T, int V, bool COMP>
__global__ __launch_bounds__(1024) void k_batched(BatchArgs a)
{
    const int lane = threadIdx.x & 63;
    // Each trip takes a distinct item from the counter, so no wave can make
    // more than n_items trips; the bound ends the loop even if a draw went
    // wrong.
    for (int64_t trip = 0; trip <= a.n_items; ++trip) {
        // Every lane takes part in the draw (lane 0 adds 1, the others 0) and
        // readfirstlane then returns lane 0's value.  No branch here depends on
        // the lane: with the draw under `if (lane == 0)` the compiler may split
        // the loop on that condition, so that lanes 1..63 re-enter it without
        // lane 0 and readfirstlane returns their stale value instead.
        const unsigned got = atomicAdd(a.work_counter, lane == 0 ? 1u : 0u);
        const int64_t it = (int64_t)__builtin_amdgcn_readfirstlane(got);
        if (it >= a.n_items)
            break;
        const BatchItem w = a.items[it];
        if (w.kind == 0)
            gemv_tile<T, V, COMP>(a.gemv[w.prob], w.begin, w.end, a.out_f64);
        else
            dot_chunk<T, V, COMP>(a, w);
    }
}

// ---------------------------------------------------------------------------
// Grouped launch: one work-group per work item, no work queue.  Items are
// ordered largest first and the hardware dispatcher hands work-groups to CUs
// in index order as they free up, which schedules the items the way a
// largest-first queue would -- without a software loop over items, without
// atomics, and with barriers only in straight-line code.
// ---------------------------------------------------------------------------
// Rows of one GEMV tile, one element per access (operands not aligned to their
// elements, rows shorter than a pack): one G-lane group per row as in
// gemv_tile, but each group carries kTileRowsInFlight rows at once and each
// lane kTileElemsInFlight elements of each row.  Loop control is wave-uniform
// up to the last trip; rows past the tile re-read its last row and are not stored.
constexpr int kTileRowsInFlight = 4;
constexpr int kTileElemsInFlight = 2;

template <typename T, bool COMP>
__device__ __forceinline__ void gemv_tile_scalar(const BatchGemv &g, int64_t rb, int64_t re, int out_f64)
{
    using C = compute_t<T>;
    constexpr bool EXACT = std::is_same<T, bf16_t>::value;
    constexpr int RB = kTileRowsInFlight, U = kTileElemsInFlight;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int G = g.lanes;
    const int rpw = 64 / G;
    const int sub = lane / G, gl = lane - sub * G;
    const T *A = (const T *)g.A;
    const T *x = (const T *)g.x;
    const int64_t K = g.n;
    const int64_t slots = (int64_t)nw * rpw; // rows the work-group holds per row batch
    for (int64_t base = rb + (int64_t)wave * rpw; base < re; base += RB * slots) {
        const T *row[RB];
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            const int64_t r = base + j * slots + sub;
            row[j] = A + (r < re ? r : re - 1) * g.lda;
        }
        acc_t<T, COMP> acc[RB];
        int64_t k = gl;
        for (; k + (int64_t)(U - 1) * G < K; k += (int64_t)U * G) {
            T xv[U], av[RB][U];
#pragma unroll
            for (int u = 0; u < U; ++u)
                xv[u] = x[k + (int64_t)u * G];
#pragma unroll
            for (int j = 0; j < RB; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    av[j][u] = row[j][k + (int64_t)u * G];
#pragma unroll
            for (int j = 0; j < RB; ++j)
#pragma unroll
                for (int u = 0; u < U; ++u)
                    acc[j].template add_prod<EXACT>(widen(av[j][u]), widen(xv[u]));
        }
        for (; k < K; k += G) {
            const C xk = widen(x[k]);
#pragma unroll
            for (int j = 0; j < RB; ++j)
                acc[j].template add_prod<EXACT>(widen(row[j][k]), xk);
        }
#pragma unroll
        for (int j = 0; j < RB; ++j) {
            DD d = acc[j].to_dd();
            for (int m = G >> 1; m >= 1; m >>= 1)
                d = combine<COMP>(d, shfl_xor_dd(d, m));
            const int64_t r = base + j * slots + sub;
            if (gl == 0 && r < re)
                store_out(g.y, r, out_f64, d.hi + d.lo);
        }
    }
}

// Rows of one GEMV tile in 16-byte packs from any element: a row belongs to a
// group of G lanes (a compile-time constant), and a wave carries R = 8 rows
// per group, 512 / G rows, with one pack of each in flight per trip, so that a
// pack of x (from the caches) is read and widened once for 8 rows.  The last
// trip is masked: its packs end with the row, and entries that an earlier pack
// covered, or past the end, count as 0 on both sides.  No LDS and no
// barrier; loop control is wave-uniform; rows past the tile re-read its last
// row and are not stored.
//
// Bound by HBM once a row is some KiB long, below that by the work per row
// beside its packs.  The 8 sums of a group are reduced together, each of the
// first three exchanges leaving a lane with half of them: 4 + 2 + 1 sums and
// one per further lane bit, 10 for 8 rows of 64 lanes where a butterfly of
// each takes 48.  With fewer than 64 lanes a trip covers 128 to 512 bytes of a
// row, whose lines the next trip reads on where rows start anywhere: those
// loads are not marked as streaming, so that the line is still there (rows of
// 257 bf16 2.9 -> 3.8 TB/s, of 513 f32 4.65 -> 4.84; with 64 lanes streaming
// loads are the faster, 513 f64 5.36 -> 5.57).
//
// The form this replaced staged x in LDS and read a row as head, aligned packs
// and tail.  GEMV kernels of uneven batches (rows and columns 32 to 4096),
// before -> after: 512 compensated bf16, 765 MB, 212 -> 142 us (5.4 TB/s); 256 f32,
// 699 MB, 146 -> 122; 128 f64, 912 MB, 185 -> 153; 20 f64, 120 MB, 74 -> 33; 40
// compensated bf16, 75 MB, 35 -> 21.
template <typename T, bool COMP, int G>
__device__ __forceinline__ void gemv_tile_rows(const BatchGemv &g, int64_t rb, int64_t re, int out_f64)
{
    constexpr bool EXACT = std::is_same<T, bf16_t>::value;
    constexpr int V = 16 / (int)sizeof(T), R = kTileRows, RPW = 64 / G;
    constexpr bool NT = G == 64;
    // Plain sums of rows that share a wave have 8 packs per lane at most: one running sum. Up to
    // long_from entries, one for the even and one for the odd elements of a pack.
    constexpr int H = !COMP && G == 64 ? 2 : 1;
    using Sum = std::conditional_t<!COMP, Acc<compute_t<T>, false>, acc_t<T, COMP>>;
    const int64_t n = g.n;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int sub = lane / G, gl = lane % G;
    const T *A = (const T *)g.A;
    const T *x = (const T *)g.x;
    const int64_t whole = n / (G * V) * (G * V); // entries of the unmasked trips
    // the masked trip: this lane's pack starts at `last`, its first `skip`
    // entries (all of them past the end) are another pack's
    const int64_t want = whole + gl * V;
    const int64_t last = want + V <= n ? want : n - V;
    const int skip = want - last < V ? (int)(want - last) : V;
    for (int64_t base = rb + (int64_t)wave * (R * RPW); base < re; base += (int64_t)nw * (R * RPW)) {
        const T *row[R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            const int64_t r = base + j * RPW + sub;
            row[j] = A + (r < re ? r : re - 1) * g.lda;
        }
        Sum acc[H][R];
        for (int64_t k = gl * V; k < whole; k += G * V) {
            Pack<T, V> a[R];
            const Pack<T, V> xv = load_pack<T, V>(x + k);
#pragma unroll
            for (int j = 0; j < R; ++j)
                a[j] = load_pack<T, V, NT>(row[j] + k);
            end_of_loads();
#pragma unroll
            for (int e = 0; e < V; ++e)
#pragma unroll
                for (int j = 0; j < R; ++j)
                    acc[e % H][j].template add_prod<EXACT>(widen(a[j].v[e]), widen(xv.v[e]));
        }
        if (whole < n) {
            Pack<T, V> a[R];
            const Pack<T, V> xv = load_pack<T, V>(x + last);
#pragma unroll
            for (int j = 0; j < R; ++j)
                a[j] = load_pack<T, V, NT>(row[j] + last);
            end_of_loads();
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const T xe = e >= skip ? xv.v[e] : T(0);
#pragma unroll
                for (int j = 0; j < R; ++j)
                    acc[e % H][j].template add_prod<EXACT>(widen(e >= skip ? a[j].v[e] : T(0)), widen(xe));
            }
        }
        DD d[R];
#pragma unroll
        for (int j = 0; j < R; ++j)
            d[j] = H == 2 ? combine<COMP>(acc[0][j].to_dd(), acc[H - 1][j].to_dd()) : acc[0][j].to_dd();
        constexpr int B = G == 64 ? 5 : G == 32 ? 4 : G == 16 ? 3 : 2; // highest lane bit of a group
        halve<COMP, B, 4>(d, lane);
        halve<COMP, B - 1, 2>(d, lane);
        halve<COMP, B - 2, 1>(d, lane);
        if constexpr (B > 4)
            d[0] = combine<COMP>(d[0], dpp_dd<kDppHalfMirror>(d[0]));
        if constexpr (B > 3)
            d[0] = combine<COMP>(d[0], dpp_dd<kDppXor2>(d[0]));
        if constexpr (B > 2)
            d[0] = combine<COMP>(d[0], dpp_dd<kDppXor1>(d[0]));
        const int j = gl / (G / 8); // the row this lane's sum belongs to
        const int64_t r = base + j * RPW + sub;
        if (gl % (G / 8) == 0 && r < re)
            store_out(g.y, r, out_f64, d[0].hi + d[0].lo);
    }
}

// Rows of more than long_from entries: the work-group shares R of them, each
// thread U packs of each in flight (R * U = 8), and the waves' sums are added in wave order
// through LDS.  A tile of such rows has too few of them to give every wave 8 of
// its own: with one wave's 8 rows per tile three of four waves were idle and each row
// was one serial chain.  GPU time of 8 GEMVs of 300
// rows, a wave's rows -> this: 4099 f32 14.9 -> 11.9 us, 16384 f32 47 -> 28, 10^5 f32 294 ->
// 173, 5000 compensated bf16 14.3 -> 11, 16384 f64 97 -> 58; of 4 of 40 rows of 10^6 f32 2620 -> 159.
template <typename T, bool COMP, int R>
__device__ __forceinline__ void gemv_tile_long(const BatchGemv &g, int64_t rb, int64_t re, int out_f64, DD *lds)
{
    constexpr bool EXACT = std::is_same<T, bf16_t>::value;
    constexpr int V = 16 / (int)sizeof(T), U = 8 / R;
    const int64_t n = g.n, kpack = n / V, tail = n - kpack * V;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int64_t step = blockDim.x;
    const T *A = (const T *)g.A;
    const T *x = (const T *)g.x;
    for (int64_t base = rb; base < re; base += R) {
        const T *row[R];
#pragma unroll
        for (int r = 0; r < R; ++r) // rows past the tile re-read its last one and are not stored
            row[r] = A + (base + r < re ? base + r : re - 1) * g.lda;
        acc_t<T, COMP> acc[R];
        int taken = 0; // packs of a row by this thread
        auto fold = [&](int packs) {
            taken += packs;
            if (taken % kRunPacks<T> == 0)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[r].fold();
        };
        int64_t p = threadIdx.x;
        for (; p + (U - 1) * step < kpack; p += U * step) {
            Pack<T, V> a[U][R], xv[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                xv[u] = load_pack<T, V>(x + (p + u * step) * V);
#pragma unroll
                for (int r = 0; r < R; ++r)
                    a[u][r] = load_pack_nt<T, V>(row[r] + (p + u * step) * V);
            }
            end_of_loads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int e = 0; e < V; ++e)
#pragma unroll
                    for (int r = 0; r < R; ++r)
                        acc[r].template add_prod<EXACT>(widen(a[u][r].v[e]), widen(xv[u].v[e]));
                fold(1);
            }
        }
        for (; p < kpack; p += step) {
            Pack<T, V> a[R];
            const Pack<T, V> xv = load_pack<T, V>(x + p * V);
#pragma unroll
            for (int r = 0; r < R; ++r)
                a[r] = load_pack_nt<T, V>(row[r] + p * V);
#pragma unroll
            for (int e = 0; e < V; ++e)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[r].template add_prod<EXACT>(widen(a[r].v[e]), widen(xv.v[e]));
            fold(1);
        }
        if (threadIdx.x < tail) {
            const int64_t k = kpack * V + threadIdx.x;
#pragma unroll
            for (int r = 0; r < R; ++r)
                acc[r].template add_prod<EXACT>(widen(row[r][k]), widen(x[k]));
        }
        // the rows' sums over the wave together, as in gemv_tile_rows: lanes of
        // one R-th of the wave end with one row's
        DD d[R];
#pragma unroll
        for (int r = 0; r < R; ++r)
            d[r] = acc[r].to_dd();
        if constexpr (R > 1) {
            halve<COMP, 5, R / 2>(d, lane);
            halve<COMP, 4, R / 4>(d, lane);
            if constexpr (R == 8)
                halve<COMP, 3, 1>(d, lane);
            else
                d[0] = combine<COMP>(d[0], dpp_dd<kDppXor8>(d[0]));
            d[0] = combine<COMP>(d[0], dpp_dd<kDppHalfMirror>(d[0]));
            d[0] = combine<COMP>(d[0], dpp_dd<kDppXor2>(d[0]));
            d[0] = combine<COMP>(d[0], dpp_dd<kDppXor1>(d[0]));
        } else {
            d[0] = wave_sum<COMP>(d[0]);
        }
        if (lane % (64 / R) == 0)
            lds[wave * R + lane / (64 / R)] = d[0];
        __syncthreads();
        if (threadIdx.x < R) {
            DD t = lds[threadIdx.x];
            for (int w = 1; w < nw; ++w)
                t = combine<COMP>(t, lds[w * R + threadIdx.x]);
            if (base + threadIdx.x < re)
                store_out(g.y, base + threadIdx.x, out_f64, t.hi + t.lo);
        }
        __syncthreads(); // lds is written again by the next rows
    }
}

// One dot chunk reduced by a whole work-group: each thread keeps U packs of
// both operands in flight per trip, two accumulators, then the work-group
// tree (block_sum, barriers in straight-line code).  U is 8, and 4 in the
// compensated bf16 form, which then fits 4 waves per SIMD (512 GEMVs and 4096 dots
// 485 us with 8, 473 with 4; the f32 form loses, 471 and 476).

template <typename T, int V, bool COMP>
__device__ __forceinline__ void dot_chunk_block(const BatchArgs &a, const BatchItem &w, DD *lds)
{
    using C = compute_t<T>;
    constexpr bool EXACT = std::is_same<T, bf16_t>::value;
    constexpr int U = EXACT && COMP ? 4 : 8;
    const BatchDot &d = a.dots[w.prob];
    const T *x = (const T *)d.x, *y = (const T *)d.y;
    acc_t<T, COMP> acc[2];
    const int64_t pb = w.begin / V, pe = w.end / V; // chunk starts are pack-aligned
    const int64_t step = blockDim.x;
    int64_t p = pb + threadIdx.x;
    for (; p + (U - 1) * step < pe; p += U * step) {
        Pack<T, V> xs[U], ys[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            xs[u] = load_pack_nt<T, V>(x + (p + u * step) * V);
            ys[u] = load_pack_nt<T, V>(y + (p + u * step) * V);
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < V; ++e)
                acc[u & 1].template add_prod<EXACT>(widen(xs[u].v[e]), widen(ys[u].v[e]));
    }
    for (; p < pe; p += step) {
        const Pack<T, V> x0 = load_pack_nt<T, V>(x + p * V), y0 = load_pack_nt<T, V>(y + p * V);
#pragma unroll
        for (int e = 0; e < V; ++e)
            acc[0].template add_prod<EXACT>(widen(x0.v[e]), widen(y0.v[e]));
    }
    const int64_t tail = w.end - pe * V; // < V, only in a dot's last chunk
    if (threadIdx.x < tail)
        acc[0].template add_prod<EXACT>(widen(x[pe * V + threadIdx.x]), widen(y[pe * V + threadIdx.x]));
    DD v = block_sum<COMP>(combine<COMP>(acc[0].to_dd(), acc[1].to_dd()), lds);
    if (threadIdx.x == 0) {
        if (d.chunks == 1)
            store_out(d.out, 0, a.out_f64, v.hi + v.lo);
        else
            reinterpret_cast<DD *>(a.partials)[d.slot0 + w.chunk] = v;
    }
}

// Every item of a plan in one launch: GEMV tiles first, whose rows are the
// longer serial chains, then dot chunks, which fill the CUs the tiles leave.
// With a launch per kind each kind's last work-groups ran alone.  GEMV and dot
// kernels -> this one, with dot chunks of 64 KiB for 128 and more: 20 GEMVs and 20 dots f32
// 18.2 + 15.0 -> 18.7 us, 20 and 80 f64 32.7 + 33.1 -> 51.8, 8 and 32 bf16 9.2 + 12.4 -> 9.6,
// 512 and 4096 compensated bf16 144 + 339 -> 473 (3.07 GB, 6.5 TB/s).
template <typename T, bool COMP>
__global__ __launch_bounds__(512) void k_grouped(BatchArgs a)
{
    constexpr int NATIVE = 16 / (int)sizeof(T);
    __shared__ DD lds[64]; // block_sum's, or 8 waves' sums of 8 rows
    // the item is the same for every thread of the work-group
    const BatchItem w = a.items[blockIdx.x];
    if (__builtin_amdgcn_readfirstlane(w.kind) == 1) { // block_sum holds barriers
        if (__builtin_amdgcn_readfirstlane(a.dots[w.prob].mode) == kModePacked)
            dot_chunk_block<T, NATIVE, COMP>(a, w, lds);
        else
            dot_chunk_block<T, 1, COMP>(a, w, lds);
        return;
    }
    const BatchGemv &g = a.gemv[w.prob];
    const int mode = __builtin_amdgcn_readfirstlane(g.mode);
    if (mode == kModeScalar) {
        gemv_tile_scalar<T, COMP>(g, w.begin, w.end, a.out_f64);
        return;
    }
    if (mode == kModeLong) { // holds barriers: begin and end are the work-group's
        switch (__builtin_amdgcn_readfirstlane(g.lanes)) {
        case 8: gemv_tile_long<T, COMP, 8>(g, w.begin, w.end, a.out_f64, lds); break;
        case 4: gemv_tile_long<T, COMP, 4>(g, w.begin, w.end, a.out_f64, lds); break;
        default: gemv_tile_long<T, COMP, 1>(g, w.begin, w.end, a.out_f64, lds); break;
        }
        return;
    }
    switch (__builtin_amdgcn_readfirstlane(g.lanes)) {
    case 8: gemv_tile_rows<T, COMP, 8>(g, w.begin, w.end, a.out_f64); break;
    case 16: gemv_tile_rows<T, COMP, 16>(g, w.begin, w.end, a.out_f64); break;
    case 32: gemv_tile_rows<T, COMP, 32>(g, w.begin, w.end, a.out_f64); break;
    default: gemv_tile_rows<T, COMP, 64>(g, w.begin, w.end, a.out_f64); break;
    }
}

#if BWLA_T_IS_F64 // type-independent kernels live in the f64 object only
__global__ void k_zero_counters(unsigned *c, int64_t count)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < count;
         i += (int64_t)gridDim.x * blockDim.x)
        c[i] = 0u;
}

// One wave per dot: combine the chunk partials of multi-chunk dots, each
// lane's in chunk order and then the lanes (single-chunk dots were written by
// the chunk's work-group).  Bound by the chain of loads and sums: one thread
// per dot took 0.5 us per chunk beyond 8.
template <bool COMP>
__global__ __launch_bounds__(256) void k_batch_finalize(const BatchDot *dots, int64_t nd, const DD *partials,
                                                        int out_f64)
{
    const int lane = threadIdx.x & 63;
    const int64_t i = ((int64_t)blockIdx.x * blockDim.x + threadIdx.x) >> 6;
    if (i >= nd)
        return;
    const BatchDot d = dots[i];
    if (d.chunks <= 1)
        return;
    const DD *p = partials + d.slot0;
    DD t = {0.0, 0.0};
    if (lane < d.chunks)
        t = p[lane];
    for (int c = lane + 64; c < d.chunks; c += 64)
        t = combine<COMP>(t, p[c]);
    t = wave_sum<COMP>(t);
    if (lane == 0)
        store_out(d.out, 0, out_f64, t.hi + t.lo);
}
#endif

template <typename T>
hipError_t launch_batched(const BatchArgs &a, bool comp, int grid, int block, hipStream_t s)
{
    constexpr int NATIVE = 16 / (int)sizeof(T);
    auto go = [&](auto V) {
        return with_bool(comp, [&](auto CP) {
            hipLaunchKernelGGL((k_batched<T, V.value, CP.value>), dim3(grid), dim3(block), 0, s, a);
            return hipGetLastError();
        });
    };
    if (a.vec == 1)
        return go(std::integral_constant<int, 1>{});
    return go(std::integral_constant<int, NATIVE>{});
}

template hipError_t launch_batched<BWLA_T>(const BatchArgs &, bool, int, int, hipStream_t);

template <typename T>
hipError_t launch_grouped(const BatchArgs &a, bool comp, int block, hipStream_t s)
{
    return with_bool(comp, [&](auto CP) {
        hipLaunchKernelGGL((k_grouped<T, CP.value>), dim3((unsigned)a.n_items), dim3(block), 0, s, a);
        return hipGetLastError();
    });
}

template hipError_t launch_grouped<BWLA_T>(const BatchArgs &, bool, int, hipStream_t);

#if BWLA_T_IS_F64
hipError_t launch_batch_reset(unsigned *counters, int64_t count, hipStream_t s)
{
    int64_t blocks = (count + 255) / 256;
    if (blocks > 1024)
        blocks = 1024;
    if (blocks < 1)
        blocks = 1;
    hipLaunchKernelGGL(k_zero_counters, dim3((unsigned)blocks), dim3(256), 0, s, counters, count);
    return hipGetLastError();
}

hipError_t launch_batch_finalize(const BatchDot *dots, int64_t nd, const double *partials, bool comp,
                                 int out_f64, hipStream_t s)
{
    if (nd <= 0)
        return hipSuccess;
    const int64_t blocks = (nd + 3) / 4;
    return with_bool(comp, [&](auto CP) {
        hipLaunchKernelGGL((k_batch_finalize<CP.value>), dim3((unsigned)blocks), dim3(256), 0, s, dots, nd,
                           (const DD *)partials, out_f64);
        return hipGetLastError();
    });
}
#endif

} // namespace bwla
