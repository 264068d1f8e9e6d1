// gemv.hip -- dense matrix-vector products (paper Section 2: each output
// entry is the inner product of one row with the right-hand side; the paper
// notes other blockings are possible, and these kernels use two).
//
// A matrix is viewed as L "lines" of K contiguous elements, ld elements apart.
// A row-major A has its rows as lines, a column-major A its columns, so:
//   row-major  y = A x    and column-major y = A^T x  -> rows kernel
//   row-major  y = A^T x  and column-major y = A x    -> cols kernel
//
// rows kernel: out[l] = sum_k A[l*ld + k] v[k].  A work-group owns R lines
//   (and, with split > 1, one of `split` slices of their length).  Each
//   thread loads a pack of v once into registers and reuses it for the R
//   lines, so v is read from cache once per R lines of A; A itself is read
//   with nontemporal loads (touched once), U packs per line in flight.  The R sums are
//   reduced across the wave (DPP) and across waves through LDS.  With split >
//   1 each slice writes float64 partials and a second kernel combines them in
//   slice order.
//
// cols kernels: out[k] = sum_l A[l*ld + k] v[l], with one line per wave access
//   (k_gemv_cols) or several (k_gemv_cols_grouped, below; the default).  With
//   one, a work-group owns a tile of
//   64*V consecutive outputs (V per lane, so each wave access is 64*V
//   contiguous elements) and one of `split` slices of the lines; its waves
//   take interleaved lines of the slice, U lines in flight (up to 32).  Each
//   v[l] is one scalar load per wave, issued with the loads of its line, so
//   the first loads of A start without a staging pass or a barrier.  Per-wave
//   partial sums are combined through LDS in wave order; with split > 1 the
//   slices' partials are combined in slice order by a second kernel.
//
// Dot epilogue (w != NULL): the caller also wants s = <w, y> over the
// outputs, with y as stored (the storage type equals the compute type
// here).  Whichever kernel stores an output also forms w_o * y_o and reduces
// those products over its outputs to one float64 pair per work-group:
// the rows or cols kernel when split == 1, the line combine otherwise.  The
// scalar second stage then sums the pairs in work-group order.  This saves
// re-reading y and w and one launch of the separate inner product.
#include "device.hpp"
#include "kernels.hpp"

namespace bwla {

// The prior value of output i (read only when it is updated), and the store
// of result v in its place.  The rows kernel fetches the prior value before its
// main loop, the grouped cols kernel before its sums across lanes and waves, and the line
// combine with its partials; the one-line cols kernel at the store.
__device__ __forceinline__ double out_prior(const GemvOut &o, int64_t i)
{
    if (o.mode != kOutUpdate)
        return 0.0;
    return o.f64 ? reinterpret_cast<const double *>(o.y)[i * o.inc]
                 : (double)reinterpret_cast<const float *>(o.y)[i * o.inc];
}
template <typename O> __device__ __forceinline__ O out_value(const GemvOut &o, O s, O prior)
{
    if (o.mode == kOutScale)
        return (O)o.a * s;
    if (o.mode == kOutUpdate)
        return fma_c((O)o.a, s, (O)o.b * prior);
    return s;
}
__device__ __forceinline__ void out_put(const GemvOut &o, int64_t i, double v, double prior)
{
    if (o.f64)
        reinterpret_cast<double *>(o.y)[i * o.inc] = out_value<double>(o, v, prior);
    else
        reinterpret_cast<float *>(o.y)[i * o.inc] = out_value<float>(o, (float)v, (float)prior);
}

// One product of the dot epilogue, left as a float64 pair.
template <typename C, bool COMP> __device__ __forceinline__ DD epilogue_term(C w, C y)
{
    Acc<C, COMP> a;
    a.template add_prod<false>(w, y);
    return a.to_dd();
}

// per: packs of a slice, divided on the host (a 64-bit division here branches).
template <typename T, int V, int R, int U, bool COMP>
__global__ __launch_bounds__(1024) void k_gemv_rows(int64_t L, int64_t K, const T *A, int64_t ld,
                                                    const T *v, DD *partials, GemvOut out,
                                                    int split, int64_t per, const T *w, DD *dparts)
{
    using C = compute_t<T>;
    constexpr bool EXACT = std::is_same<T, bf16_t>::value;
    const unsigned lb = (unsigned)xcd_block();
    const int64_t group = lb / (unsigned)split;
    const int s = (int)(lb % (unsigned)split);
    const int64_t l0 = group * R;
    const int nr = (int)(L - l0 < R ? L - l0 : R);
    const T *row[R];
#pragma unroll
    for (int r = 0; r < R; ++r)
        row[r] = A + (l0 + (r < nr ? r : nr - 1)) * ld; // rows past L re-read the last one

    const int64_t kpack = K / V;
    const int64_t pb = (int64_t)s * per;
    const int64_t pe = pb + per < kpack ? pb + per : kpack;
    // the dot epilogue's weight and the prior output of this thread's line,
    // fetched before the main loop: read at the end they would be one more
    // memory latency in every work-group's tail
    C wl = C(0);
    double prior = 0.0;
    if (split == 1 && (int)threadIdx.x < nr) {
        if (w != nullptr)
            wl = widen(w[l0 + threadIdx.x]);
        prior = out_prior(out, l0 + threadIdx.x);
    }

    // U trips of the pack loop per iteration, all loads first: R * U packs of
    // A in flight per thread.  Each row's sum still takes the packs in the
    // order p, p + blockDim, ..., and ends its runs at the same packs, so U does
    // not change any result.
    acc_t<T, COMP> acc[R];
    int taken = 0; // packs of a row by this thread
    auto fold_rows = [&](int n) {
        if constexpr (!COMP && kRunPacks<T> > 1) {
            taken += n;
            if (taken % kRunPacks<T> == 0)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[r].fold();
        }
    };
    int64_t p = pb + threadIdx.x;
    for (; p + (int64_t)(U - 1) * blockDim.x < pe; p += (int64_t)U * blockDim.x) {
        Pack<T, V> xv[U], av[U][R];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            xv[u] = load_pack<T, V>(v + (p + (int64_t)u * blockDim.x) * V);
#pragma unroll
            for (int r = 0; r < R; ++r)
                av[u][r] = load_pack_nt<T, V>(row[r] + (p + (int64_t)u * blockDim.x) * V);
        }
        end_of_loads();
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int r = 0; r < R; ++r) {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    acc[r].template add_prod<EXACT>(widen(av[u][r].v[e]), widen(xv[u].v[e]));
                if (kRunPacks<T> == 1)
                    acc[r].fold();
            }
        fold_rows(U);
    }
    for (; p < pe; p += blockDim.x) {
        Pack<T, V> xv = load_pack<T, V>(v + p * V);
        Pack<T, V> av[R];
#pragma unroll
        for (int r = 0; r < R; ++r)
            av[r] = load_pack_nt<T, V>(row[r] + p * V);
#pragma unroll
        for (int r = 0; r < R; ++r) {
#pragma unroll
            for (int e = 0; e < V; ++e)
                acc[r].template add_prod<EXACT>(widen(av[r].v[e]), widen(xv.v[e]));
            if (kRunPacks<T> == 1)
                acc[r].fold();
        }
        fold_rows(1);
    }
    const int64_t tail = K - kpack * V; // < V elements, taken by the last slice
    if (s == split - 1 && threadIdx.x < tail) {
        const int64_t k = kpack * V + threadIdx.x;
        C xk = widen(v[k]);
#pragma unroll
        for (int r = 0; r < R; ++r)
            acc[r].template add_prod<EXACT>(widen(row[r][k]), xk);
    }

    __shared__ DD lds[16 * R];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        DD d = wave_sum<COMP>(acc[r].to_dd());
        if (lane == 0)
            lds[wave * R + r] = d;
    }
    __syncthreads();
    DD t = {0.0, 0.0};
    if (threadIdx.x < R) {
        t = lds[threadIdx.x];
        for (int wv = 1; wv < nw; ++wv)
            t = combine<COMP>(t, lds[wv * R + threadIdx.x]);
        if (split == 1) {
            if ((int)threadIdx.x < nr)
                out_put(out, l0 + threadIdx.x, t.hi + t.lo, prior);
        } else {
            partials[(group * split + s) * R + threadIdx.x] = t;
        }
    }
    if (w != nullptr && split == 1 && wave == 0) { // the whole first wave
        DD d = {0.0, 0.0};
        if ((int)threadIdx.x < nr)
            d = epilogue_term<C, COMP>(wl, (C)(t.hi + t.lo));
        d = wave_sum<COMP>(d);
        if (lane == 0)
            dparts[group] = d;
    }
}

template <typename T, int V, int U, bool COMP>
__global__ __launch_bounds__(1024) void k_gemv_cols(int64_t L, int64_t K, const T *A, int64_t ld,
                                                    const T *__restrict__ v, int64_t incv, DD *partials,
                                                    GemvOut out, int split, int64_t per, const T *w, DD *dparts,
                                                    int xchg)
{
    using C = compute_t<T>;
    constexpr bool EXACT = std::is_same<T, bf16_t>::value;
    constexpr int TK = 64 * V;
    const unsigned blk = (unsigned)xcd_block();
    const int64_t tile = blk / (unsigned)split;
    const int s = (int)(blk % (unsigned)split);
    const int lane = threadIdx.x & 63, nw = blockDim.x >> 6;
    // the wave index as a wave-uniform (scalar) value, so that every v[l]
    // below is one scalar load shared by the wave
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t k0 = tile * TK + (int64_t)lane * V;
    // The lane whose pack runs past the end of the lines takes the last V
    // columns instead and keeps those from k0 on: the same loads and the same
    // loop as its neighbours.  Taken element by element, that one lane made
    // its waves three times as long (8001 x 8003 bf16: 107 us in all).
    const int64_t kb = k0 + V <= K ? k0 : K - V;
    const int64_t lb = (int64_t)s * per;
    const int64_t le = lb + per < L ? lb + per : L;

    // LDS for the cross-wave combine (the hand-over path).
    __shared__ __attribute__((aligned(16))) DD red[TK];
    line_acc_t<T, COMP> acc[V];
    int taken = 0; // lines by this wave
    auto fold_cols = [&](int n) { // (runs of lines end where they do for every U and V)
        if constexpr (!COMP && std::is_same_v<T, double>) {
            taken += n;
            if (taken % kRunLines == 0)
#pragma unroll
                for (int e = 0; e < V; ++e)
                    acc[e].fold();
        }
    };

    // v[l] is read with the U lines' loads (no staging pass and no barrier
    // before the first loads of A).
    const T *vt = v + lb * incv;
    const T *base = A + lb * ld + kb;
    const int64_t tn = le - lb;
    int64_t j = wave;
    if (k0 < K && kb >= 0) {
        for (; j + (int64_t)(U - 1) * nw < tn; j += (int64_t)U * nw) {
            Pack<T, V> a[U];
            T xv[U]; // widened after the loads: a conversion among them would wait
#pragma unroll
            for (int u = 0; u < U; ++u) {
                a[u] = load_pack_nt<T, V>(base + (j + (int64_t)u * nw) * ld);
                xv[u] = vt[(j + (int64_t)u * nw) * incv];
            }
            end_of_loads();
#pragma unroll
            for (int u = 0; u < U; ++u) {
#pragma unroll
                for (int e = 0; e < V; ++e)
                    acc[e].template add_prod<EXACT>(widen(a[u].v[e]), widen(xv[u]));
                if (U > kRunLines && u % kRunLines == kRunLines - 1 && u < U - 1)
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        acc[e].fold();
            }
            fold_cols(U);
        }
        for (; j < tn; j += nw) {
            Pack<T, V> a = load_pack_nt<T, V>(base + j * ld);
            const C xl = widen(vt[j * incv]);
#pragma unroll
            for (int e = 0; e < V; ++e)
                acc[e].template add_prod<EXACT>(widen(a.v[e]), xl);
            fold_cols(1);
        }
    } else if (k0 < K) { // lines shorter than a pack
        for (; j < tn; j += nw) {
            const C xl = widen(vt[j * incv]);
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (kb + e >= 0)
                    acc[e].template add_prod<EXACT>(widen(base[j * ld + e]), xl);
            fold_cols(1);
        }
    }

    // Combine the waves' partial sums in wave order through LDS.  With xchg
    // the launch gave every wave but the first (nw - 1) * TK pairs of dynamic
    // LDS: all waves write at once and wave 0 adds them in wave order after
    // one barrier.  Otherwise the waves hand over one at a time through a
    // buffer of one tile of pairs.  Both orders of addition are the same.
    DD d[V];
#pragma unroll
    for (int e = 0; e < V; ++e)
        d[e] = acc[e].to_dd();
    if (xchg) {
        extern __shared__ DD xs[];
        if (wave > 0)
#pragma unroll
            for (int e = 0; e < V; ++e)
                xs[(wave - 1) * TK + lane * V + e] = d[e];
        __syncthreads();
        if (wave == 0)
            for (int wv = 1; wv < nw; ++wv)
#pragma unroll
                for (int e = 0; e < V; ++e)
                    d[e] = combine<COMP>(d[e], xs[(wv - 1) * TK + lane * V + e]);
    } else {
        for (int wv = 1; wv < nw; ++wv) {
            if (wave == wv)
#pragma unroll
                for (int e = 0; e < V; ++e)
                    red[lane * V + e] = d[e];
            __syncthreads();
            if (wave == 0)
#pragma unroll
                for (int e = 0; e < V; ++e)
                    d[e] = combine<COMP>(d[e], red[lane * V + e]);
            __syncthreads();
        }
    }
    if (wave == 0) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            if (kb + e < k0 || k0 >= K)
                continue;
            if (split == 1)
                out_put(out, kb + e, d[e].hi + d[e].lo, out_prior(out, kb + e));
            else
                partials[(tile * split + s) * TK + (kb + e - tile * TK)] = d[e];
        }
        if (w != nullptr && split == 1) {
            DD t = {0.0, 0.0};
#pragma unroll
            for (int e = 0; e < V; ++e)
                if (kb + e >= k0 && k0 < K)
                    t = combine<COMP>(t, epilogue_term<C, COMP>(widen(w[kb + e]), (C)(d[e].hi + d[e].lo)));
            t = wave_sum<COMP>(t);
            if (lane == 0)
                dparts[tile] = t;
        }
    }
}

// ---------------------------------------------------------------------------
// cols kernel with P lines per wave access: the 64 lanes are P groups of G =
// 64 / P, each lane loads a 16-byte pack, so an access covers G * V
// consecutive outputs (128 to 512 bytes) of P lines, and a group's U lines are
// consecutive, so that v is one pack per trip.
//
// Bound by the bytes of A in flight over all CUs.  One line per access needs
// 8-byte or narrower lanes to keep the tile at 64 columns, and with wider
// lanes its tiles are too few to fill the chip without deep splitting.  Groups
// give 16-byte lanes and 16- to 128-column tiles at once: a wave moves 1 KiB
// per load, 4096 columns make 64 to 128 tiles instead of 16 to 32, and small
// matrices need no split and no second kernel.  Before -> after, GPU time:
// 300 x 300 f32 6.8 -> 3.2 us, 1200 x 1501 f32 11.2 -> 6.7, 16000 x 100 f32 17.7 -> 7.6
// (with the wider line combine), 3001 x 4099 compensated bf16 30.7 -> 12.3, 16384 x
// 20001 bf16 229 -> 112; from 64 MiB on with aligned lines both are at the rate of
// HBM (f32 16384 x 2048 29.0 -> 27.9, 4096 x 4096 16.2 -> 16.0).
//
// The groups of a wave are summed by lane swaps that halve the values each
// time (V / 2 + V / 4 exchanges, no LDS; a butterfly of every value took as
// many vector instructions as a small matrix's products), the waves through
// LDS with one thread per output.
// ---------------------------------------------------------------------------
// UNIT: v has unit increment and is read in packs (a run-time choice between the
// two inside the loop made its loads wait: 16384 x 16384 bf16 79 -> 107 us).
template <typename T, int P, int U, bool COMP, bool UNIT>
__global__ __launch_bounds__(1024) void k_gemv_cols_grouped(int64_t L, int64_t K, const T *A, int64_t ld,
                                                            const T *v, int64_t incv, DD *partials, GemvOut out,
                                                            int split, int64_t per, const T *w, DD *dparts)
{
    using C = compute_t<T>;
    using Part = std::conditional_t<COMP, DD, double>;
    constexpr bool EXACT = std::is_same<T, bf16_t>::value;
    constexpr int V = 16 / (int)sizeof(T), G = 64 / P, TK = G * V;
    const unsigned blk = (unsigned)xcd_block();
    const int64_t tile = blk / (unsigned)split;
    const int s = (int)(blk % (unsigned)split);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
    const int gl = lane % G;
    const int64_t k0 = tile * TK + gl * V;
    // the last lane's pack is the last whole one of the lines (its columns
    // from k0 on are kept), and lanes past the end repeat it
    const int64_t kb = k0 + V <= K ? k0 : K - V;
    const int64_t lb = (int64_t)s * per;
    const int64_t tn = lb + per < L ? per : (lb < L ? L - lb : 0);

    // slot t of the tile holds column kb + e of its pack; -1: the column is
    // another lane's, or past the end
    auto column = [&](int t) -> int64_t {
        const int64_t q0 = tile * TK + (t / V) * V;
        const int64_t k = (q0 + V <= K ? q0 : K - V) + t % V;
        return k < q0 || q0 >= K ? -1 : k;
    };
    trip_acc_t<T, COMP> acc[V];
    if constexpr (UNIT)
        incv = 1;
    const T *vt = v + lb * incv;
    const T *base = A + lb * ld + kb;
    const int64_t step = (int64_t)nw * (P * U);
    int64_t j = (int64_t)(wave * P + lane / G) * U; // this group's U lines of the trip
    int64_t done = 0;
    for (; done + step <= tn; done += step, j += step) {
        Pack<T, V> a[U];
        Pack<T, U> xv;
        if constexpr (UNIT) {
            xv = load_pack<T, U>(vt + j);
        } else {
#pragma unroll
            for (int u = 0; u < U; ++u)
                xv.v[u] = vt[(j + u) * incv];
        }
        const T *row = base + j * ld;
#pragma unroll
        for (int u = 0; u < U; ++u)
            a[u] = load_pack_nt<T, V>(row + u * ld);
        end_of_loads();
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int e = 0; e < V; ++e) {
                acc[e].template add_prod<EXACT>(widen(a[u].v[e]), widen(xv.v[u]));
                if (u == U - 1)
                    acc[e].fold();
            }
    }
    if (j < tn) { // the last trip: lines past the end re-read the last one and are not added
        Pack<T, V> a[U];
        T xv[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t l = j + u < tn ? j + u : tn - 1;
            xv[u] = vt[l * incv];
            a[u] = load_pack_nt<T, V>(base + l * ld);
        }
        end_of_loads();
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (j + u < tn)
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    acc[e].template add_prod<EXACT>(widen(a[u].v[e]), widen(xv[u]));
                    if (u == U - 1)
                        acc[e].fold();
                }
    }

    // This thread's prior output, in flight during the sums below.
    const int64_t own = split == 1 && (int)threadIdx.x < TK ? column(threadIdx.x) : -1;
    const double prior = own >= 0 ? out_prior(out, own) : 0.0;

    // Sum the P groups of the wave: each exchange of halves leaves a lane with
    // half of its values, summed over twice the lines.
    DD d[V];
#pragma unroll
    for (int e = 0; e < V; ++e)
        d[e] = acc[e].to_dd();
    constexpr int R1 = V / 2, R2 = P >= 4 && V >= 4 ? V / 4 : R1; // values left per lane
    int e0 = lane & 32 ? R1 : 0;                                  // the first of them
#pragma unroll
    for (int e = 0; e < R1; ++e)
        d[e] = pair_sum<COMP, 32>(d[e], d[e + R1]);
    if constexpr (P >= 4) {
        if constexpr (V >= 4) {
            e0 += lane & 16 ? R2 : 0;
#pragma unroll
            for (int e = 0; e < R2; ++e)
                d[e] = pair_sum<COMP, 16>(d[e], d[e + R2]);
        } else {
            d[0] = pair_sum<COMP, 16>(d[0], d[0]);
        }
    }
    if constexpr (P >= 8) {
#pragma unroll
        for (int e = 0; e < R2; ++e)
            d[e] = combine<COMP>(d[e], dpp_dd<kDppXor8>(d[e]));
    }

    // Sum the waves in wave order through LDS, one thread per output.
    extern __shared__ __attribute__((aligned(16))) char grouped_lds[];
    Part *red = reinterpret_cast<Part *>(grouped_lds);
    // (where a step above left both lanes of a pair with the same value, one writes)
    if (!(P >= 8 && (lane & 8)) && !(P >= 4 && V == 2 && (lane & 16))) {
#pragma unroll
        for (int e = 0; e < R2; ++e) {
            if constexpr (COMP)
                red[wave * TK + gl * V + e0 + e] = d[e];
            else
                red[wave * TK + gl * V + e0 + e] = d[e].hi;
        }
    }
    __syncthreads();
    DD dot = {0.0, 0.0};
    for (int t = threadIdx.x; t < TK; t += blockDim.x) {
        DD r = {0.0, 0.0};
        for (int wv = 0; wv < nw; ++wv) {
            DD x = {0.0, 0.0};
            if constexpr (COMP)
                x = red[wv * TK + t];
            else
                x.hi = red[wv * TK + t];
            r = wv == 0 ? x : combine<COMP>(r, x);
        }
        const int64_t k = column(t);
        if (k < 0)
            continue;
        const double y = r.hi + r.lo;
        if (split == 1) {
            out_put(out, k, y, t == (int)threadIdx.x ? prior : out_prior(out, k));
            if (w != nullptr)
                dot = combine<COMP>(dot, epilogue_term<C, COMP>(widen(w[k]), (C)y));
        } else {
            partials[(tile * split + s) * TK + (k - tile * TK)] = r;
        }
    }
    if (w != nullptr && split == 1) {
        __shared__ DD lds[16];
        dot = block_sum<COMP>(dot, lds);
        if (threadIdx.x == 0)
            dparts[tile] = dot;
    }
}

#if BWLA_T_IS_F64 // type-independent kernels live in the f64 object only
// Second stage of a split GEMV: S threads per output, each summing a run of
// consecutive slices' float64 partials in slice order, then the S runs in
// order through LDS.  Consecutive threads take consecutive outputs, so they
// read consecutive partials.  With w (same element type as out), the
// work-group also reduces w_o * y_o over its outputs into dparts[blockIdx.x].
// B partials in flight per round trip: the smallest power of two (2 to 8)
// that holds a thread's run.
template <bool COMP, int B, int S>
__global__ __launch_bounds__(256) void k_combine_lines(const DD *partials, int64_t outputs, int64_t G,
                                                       int64_t split, GemvOut out, const void *w,
                                                       DD *dparts)
{
    constexpr int O = 256 / S; // outputs of the work-group
    __shared__ DD lds[S > 1 ? 256 : 16];
    const int run = threadIdx.x / O;
    const int64_t o = (int64_t)blockIdx.x * O + threadIdx.x % O;
    const bool live = o < outputs;
    DD t = {0.0, 0.0};
    const double prior = live && run == 0 ? out_prior(out, o) : 0.0;
    if (live) {
        const int64_t per = S > 1 ? (split + S - 1) / S : split;
        const int64_t q0 = run * per, q1 = q0 + per < split ? q0 + per : split;
        const int64_t g = o / G, r = o - g * G;
        const DD *p = partials + g * split * G + r;
        // slice order as written, B partials in flight at a time: one at a
        // time, a split of 128 cost 32 us of load latency.  The last batch
        // re-reads the last partial in its unused places (no branch between
        // the loads) and adds only the first nb.
        for (int64_t q = q0; q < q1; q += B) {
            const int64_t nb = q1 - q < B ? q1 - q : B;
            DD v[B];
#pragma unroll
            for (int b = 0; b < B; ++b)
                v[b] = p[(q + (b < nb ? b : nb - 1)) * G];
            end_of_loads();
#pragma unroll
            for (int b = 0; b < B; ++b)
                if (b < nb)
                    t = q + b == q0 ? v[0] : combine<COMP>(t, v[b]);
        }
    }
    if constexpr (S > 1) {
        lds[threadIdx.x] = t;
        __syncthreads();
        if (run == 0)
#pragma unroll
            for (int k = 1; k < S; ++k) // a run past the last slice holds zero
                t = combine<COMP>(t, lds[k * O + threadIdx.x]);
    }
    double y = 0.0;
    const bool store = live && run == 0;
    if (store) {
        y = t.hi + t.lo;
        out_put(out, o, y, prior);
    }
    if (w == nullptr)
        return;
    DD d = {0.0, 0.0};
    if (store) {
        if (out.f64)
            d = epilogue_term<double, COMP>(reinterpret_cast<const double *>(w)[o], y);
        else
            d = epilogue_term<float, COMP>(reinterpret_cast<const float *>(w)[o], (float)y);
    }
    if constexpr (S > 1)
        __syncthreads(); // lds is reused
    d = block_sum<COMP>(d, lds);
    if (threadIdx.x == 0)
        dparts[blockIdx.x] = d;
}

hipError_t launch_combine_lines(const void *partials, int64_t outputs, int64_t G, int64_t split,
                                bool comp, const GemvOut &out, const void *w, void *dparts,
                                hipStream_t s)
{
    const int64_t blocks = (outputs + combine_lines_outputs(split) - 1) / combine_lines_outputs(split);
    return with_bool(comp, [&](auto CP) {
        auto go = [&](auto B, auto S) {
            hipLaunchKernelGGL((k_combine_lines<CP.value, B.value, S.value>), dim3((unsigned)blocks), dim3(256), 0, s,
                               (const DD *)partials, outputs, G, split, out, w, (DD *)dparts);
            return hipGetLastError();
        };
        constexpr std::integral_constant<int, 1> one{};
        if (split <= 2)
            return go(std::integral_constant<int, 2>{}, one);
        if (split <= 4)
            return go(std::integral_constant<int, 4>{}, one);
        if (split <= kCombineOne)
            return go(std::integral_constant<int, 8>{}, one);
        return go(std::integral_constant<int, 8>{}, std::integral_constant<int, kCombineRuns>{});
    });
}
#endif


// Workspace: [split partials of the GEMV][dot-epilogue pairs].  With w the
// epilogue pairs are then summed into *dot by the scalar combine.
template <typename T>
hipError_t launch_gemv_rows(int64_t L, int64_t K, bool comp, const void *A, int64_t ld,
                            const void *v, const GemvOut &out, void *ws, const Cfg &c,
                            hipStream_t s, const void *w, size_t dparts_offset, int dot_f64,
                            void *dot)
{
    DD *partials = (DD *)ws;
    DD *dparts = w ? (DD *)((char *)ws + dparts_offset) : nullptr;
    hipError_t e = with_vec(c.vec, [&](auto V) {
        return with_rows(c.rows, [&](auto R) {
            return with_bool(comp, [&](auto CP) {
                auto go = [&](auto U) {
                    const int64_t groups = (L + R.value - 1) / R.value;
                    hipLaunchKernelGGL((k_gemv_rows<T, V.value, R.value, U.value, CP.value>),
                                       dim3((unsigned)(groups * c.split)), dim3(c.block), 0, s, L, K,
                                       (const T *)A, ld, (const T *)v, partials, out, c.split,
                                       (K / V.value + c.split - 1) / c.split, (const T *)w, dparts);
                    return hipGetLastError();
                };
                if (c.unroll == 2)
                    return go(std::integral_constant<int, 2>{});
                return go(std::integral_constant<int, 1>{});
            });
        });
    });
    if (e == hipSuccess && c.split > 1)
        e = launch_combine_lines(partials, L, c.rows, c.split, comp, out, w, dparts, s);
    if (e != hipSuccess || !w)
        return e;
    return launch_combine_scalar(dparts, gemv_dot_parts(true, L, K, c), comp, false, dot_f64, dot, s);
}

template <typename T>
hipError_t launch_cols_grouped(int64_t L, int64_t K, bool comp, const T *A, int64_t ld, const T *v, int64_t incv,
                               DD *partials, const GemvOut &out, const Cfg &c, hipStream_t s, const T *w, DD *dparts)
{
    const int64_t tiles = (K + cols_tile(c) - 1) / cols_tile(c);
    const size_t lds = (size_t)(c.block / 64) * cols_tile(c) * (comp ? sizeof(DD) : sizeof(double));
    return with_bool(comp, [&](auto CP) {
        return with_rows(c.rows, [&](auto P) -> hipError_t {
            if constexpr (P.value == 1) {
                return hipErrorInvalidValue; // one line per access: the other kernel
            } else {
                auto go = [&](auto U, auto unit) {
                    hipLaunchKernelGGL((k_gemv_cols_grouped<T, P.value, U.value, CP.value, unit.value>),
                                       dim3((unsigned)(tiles * c.split)), dim3(c.block), (unsigned)lds, s, L, K, A,
                                       ld, v, incv, partials, out, c.split, (L + c.split - 1) / c.split, w,
                                       dparts);
                    return hipGetLastError();
                };
                // (the trip's lines decide the order of a sum, so x's increment may not)
                return with_bool(incv == 1, [&](auto unit) {
                    if (c.unroll >= 8)
                        return go(std::integral_constant<int, 8>{}, unit);
                    return go(std::integral_constant<int, 4>{}, unit);
                });
            }
        });
    });
}

template <typename T>
hipError_t launch_gemv_cols(int64_t L, int64_t K, bool comp, const void *A, int64_t ld,
                            const void *v, int64_t incv, const GemvOut &out, void *ws, const Cfg &c,
                            hipStream_t s, const void *w, size_t dparts_offset, int dot_f64,
                            void *dot)
{
    DD *partials = (DD *)ws;
    DD *dparts = w ? (DD *)((char *)ws + dparts_offset) : nullptr;
    // lines in flight per wave: 1, 2, 4, 8, 16 or 32 (16 and 32 only within
    // kColsLoadBytes per lane; the configuration resolution keeps to that)
    auto with_unroll_cols = [](int u, auto &&f) -> hipError_t {
        switch (u) {
        case 32: return f(std::integral_constant<int, 32>{});
        case 16: return f(std::integral_constant<int, 16>{});
        case 8: return f(std::integral_constant<int, 8>{});
        }
        return with_unroll(u, f);
    };
    hipError_t e = c.rows > 1 ? launch_cols_grouped<T>(L, K, comp, (const T *)A, ld, (const T *)v, incv, partials,
                                                       out, c, s, (const T *)w, dparts)
                              : with_vec(c.vec, [&](auto V) {
        return with_unroll_cols(c.unroll, [&](auto U) -> hipError_t {
            if constexpr (U.value > 8 && (size_t)U.value * V.value * sizeof(T) > kColsLoadBytes) {
                return hipErrorInvalidValue;
            } else {
                return with_bool(comp, [&](auto CP) {
                    const int64_t tiles = (K + 64 * V.value - 1) / (64 * V.value);
                    // the one-barrier wave combine when its exchange area is
                    // small enough not to limit how many work-groups share a CU
                    const size_t xbytes = (size_t)(c.block / 64 - 1) * 64 * V.value * sizeof(DD);
                    const int xchg = xbytes > 0 && xbytes <= kColsXchgBytes;
                    hipLaunchKernelGGL((k_gemv_cols<T, V.value, U.value, CP.value>),
                                       dim3((unsigned)(tiles * c.split)), dim3(c.block),
                                       (unsigned)(xchg ? xbytes : 0), s, L, K, (const T *)A, ld,
                                       (const T *)v, incv, partials, out, c.split,
                                       (L + c.split - 1) / c.split, (const T *)w, dparts, xchg);
                    return hipGetLastError();
                });
            }
        });
    });
    if (e == hipSuccess && c.split > 1)
        e = launch_combine_lines(partials, K, cols_tile(c), c.split, comp, out, w, dparts, s);
    if (e != hipSuccess || !w)
        return e;
    return launch_combine_scalar(dparts, gemv_dot_parts(false, L, K, c), comp, false, dot_f64, dot, s);
}

template hipError_t launch_gemv_rows<BWLA_T>(int64_t, int64_t, bool, const void *, int64_t,
                                             const void *, const GemvOut &, void *, const Cfg &,
                                             hipStream_t, const void *, size_t, int, void *);
template hipError_t launch_gemv_cols<BWLA_T>(int64_t, int64_t, bool, const void *, int64_t,
                                             const void *, int64_t, const GemvOut &, void *, const Cfg &,
                                             hipStream_t, const void *, size_t, int, void *);

} // namespace bwla
