// Canonical chunked inclusive scan on the GPU.
//
// The association order is fixed: chunk c covers [c*1024, min((c+1)*1024, n)); one
// thread runs the chunk's left-to-right chain; the chunk totals are scanned the same
// way, recursively; element i of chunk c > 0 becomes combine(inc[c-1], loc[i]).  For
// the binary64 compensated sum this order is part of the definition of the alias
// tables' normalisation and prefix sums, so the GPU result is bitwise reproducible
// against any implementation of the same definition.  For max and for integer sums
// the order does not matter, and the same code is reused.
//
// This header is compiled only into translation units built with -ffp-contract=off.
#pragma once

#include "common.hpp"

namespace lh {

constexpr int SCAN_CHUNK = 1024;

// Neumaier-compensated running sum; the chunk value is s + comp after each element.
struct OpNeumaier {
    using T = double;
    struct State {
        double s, c;
    };
    __device__ static State init() { return State{0.0, 0.0}; }
    __device__ static double step(State &st, double x)
    {
        double t = st.s + x;
        if (fabs(st.s) >= fabs(x))
            st.c += (st.s - t) + x;
        else
            st.c += (x - t) + st.s;
        st.s = t;
        return st.s + st.c;
    }
    __device__ static double combine(double off, double loc) { return off + loc; }
};

struct OpMax {
    using T = double;
    struct State {
        double m;
    };
    __device__ static State init() { return State{-__builtin_huge_val()}; }
    __device__ static double step(State &st, double x)
    {
        st.m = x > st.m ? x : st.m;
        return st.m;
    }
    __device__ static double combine(double off, double loc) { return loc > off ? loc : off; }
};

template <class I>
struct OpAdd {
    using T = I;
    struct State {
        I s;
    };
    __device__ static State init() { return State{I(0)}; }
    __device__ static I step(State &st, I x)
    {
        st.s += x;
        return st.s;
    }
    __device__ static I combine(I off, I loc) { return off + loc; }
};

// ---------------------------------------------------------------------------
// The chains of up to 16 consecutive chunks of one array of non-negative binary64 values, by one
// workgroup of 256 threads.
//
// Written out, a Neumaier step is nine dependent operations, and one thread per chunk waits
// for each of them: about 110 cycles an element, 27-70 us a scan however small.  Only two
// additions of a step really follow from the step before it: s_k = s_(k-1) + x_k and
// c_k = c_(k-1) + e_k.  The error e_k = (s_(k-1) + x_k) - s_k is exact and comes from three
// values that are known by then, so it is taken for all elements at once (Knuth's TwoSum; the
// ordered form of OpNeumaier gives the same value, since both are exact).  So the work is cut
// into 32-element tiles that pass through the workgroup's wavefronts like a pipeline:
//   wavefront 0   lanes 0-15 add up s of tile t, lanes 16-31 add up c of tile t - 1
//   wavefront 1   lanes 0-15 take the running maximum of tile t - 2 (WHAT 2)
//   wavefronts 2, 3  move tile t + 1 from registers to LDS and load tile t + 5
//   all           e of tile t, s + c of tile t - 1, results of tile t - 2 to memory
// A tile takes 0.9 us, so a scan's chains take 30 us whatever its length up to 16.8 M elements
// (C2's two weight scans together 55 us, its four deficit and excess scans 92 us).
// (roles rotate with the workgroup's number, so that the chains of several resident ones do not
// share a SIMD).  16 chunks, not 64, spread small arrays over more compute units.
//
// Elements past the end read as 0, which changes neither s, c nor the maximum.
// WHAT: 0 only the chunk totals, 1 store s + c after each element, 2 store its running maximum.
// tiles: 32-element tiles per chunk to run (uniform).  total(c, s + c) is called for every chunk
// of the 16, maximum(c, m) too for WHAT 2; chunks past the end included.  load(i) only fetches
// (any index it is given is in range) and the value becomes binary64 a tile later, so that
// nothing waits for a load in flight; n >= 1.
constexpr int WAVE_CHUNKS = 16;
constexpr int CHAIN_TILE = 32;
constexpr int CHAIN_ROW = CHAIN_TILE + 1;
constexpr int CHAIN_BUF = WAVE_CHUNKS * CHAIN_ROW;
constexpr int CHAIN_LDS = 6 * CHAIN_BUF + WAVE_CHUNKS;  // doubles per workgroup

static inline __host__ __device__ int chain_tiles(long long rest)
{
    return rest >= SCAN_CHUNK ? SCAN_CHUNK / CHAIN_TILE : (int)LH_CDIV(rest, CHAIN_TILE);
}

template <int WHAT, class Raw, class Load, class Store, class Total, class Maximum>
__device__ __forceinline__ void block_chains(double *lds, long long n, long long c0, int tiles, Load load, Store store,
                                             Total total, Maximum maximum)
{
    double *const X = lds, *const S = lds + 2 * CHAIN_BUF, *const E = lds + 4 * CHAIN_BUF, *const O = lds + 5 * CHAIN_BUF,
                  *const carry = lds + 6 * CHAIN_BUF;
    const int lane = threadIdx.x & 63, role = ((threadIdx.x >> 6) + blockIdx.x) & 3;
    // the loaders' elements of a tile: four each
    const int l0 = (role & 1) * 64 + lane;
    Raw r[4][4];
    auto at = [&](int t, int q) {
        const int e = l0 + q * 128;
        return (c0 + (e >> 5)) * SCAN_CHUNK + t * CHAIN_TILE + (e & 31);
    };
    auto fetch = [&](int t, Raw(&d)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const long long i = at(t, q);
            d[q] = load(i < n ? i : n - 1);
        }
    };
    auto place = [&](int t, const Raw(&d)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int e = l0 + q * 128;
            X[(t & 1) * CHAIN_BUF + (e >> 5) * CHAIN_ROW + (e & 31)] = at(t, q) < n ? (double)d[q] : 0.0;
        }
    };
    if (role >= 2) {
#pragma unroll
        for (int p = 0; p < 4; ++p) fetch(p, r[p]);
        place(0, r[0]);
        fetch(4, r[0]);
    }
    __syncthreads();
    double acc = 0.0, mx = -__builtin_huge_val();
    const int its = tiles + (WHAT == 2 ? 2 : 1);
    for (int it0 = 0; it0 < its; it0 += 4) {
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int it = it0 + u;
            if (it >= its) break;
            const bool cur = it < tiles, prev = it >= 1 && it - 1 < tiles, third = WHAT == 2 && it >= 2 && it - 2 < tiles;
            const int buf = (it & 1) * CHAIN_BUF, last = CHAIN_BUF - buf;
            if (role == 0) {
                const bool isC = lane >= WAVE_CHUNKS;
                const int row = (lane & (WAVE_CHUNKS - 1)) * CHAIN_ROW;
                if (lane < 2 * WAVE_CHUNKS && (isC ? prev : cur)) {
                    const double *in = isC ? E + row : X + buf + row;
                    double *out = isC ? E + row : S + buf + row;
                    if (!isC) carry[lane] = acc;
#pragma unroll
                    for (int k0 = 0; k0 < CHAIN_TILE; k0 += 16) {
                        double x[16];
#pragma unroll
                        for (int k = 0; k < 16; ++k) x[k] = in[k0 + k];
#pragma unroll
                        for (int k = 0; k < 16; ++k) x[k] = acc = acc + x[k];
#pragma unroll
                        for (int k = 0; k < 16; ++k) out[k0 + k] = x[k];
                    }
                }
            } else if (role == 1) {
                if (third && lane < WAVE_CHUNKS) {
                    double *row = O + lane * CHAIN_ROW;
#pragma unroll
                    for (int k0 = 0; k0 < CHAIN_TILE; k0 += 16) {
                        double x[16];
#pragma unroll
                        for (int k = 0; k < 16; ++k) x[k] = row[k0 + k];
#pragma unroll
                        for (int k = 0; k < 16; ++k) x[k] = mx = __builtin_fmax(mx, x[k]);
#pragma unroll
                        for (int k = 0; k < 16; ++k) row[k0 + k] = x[k];
                    }
                }
            } else if (it + 1 < tiles) {
                place(it + 1, r[(u + 1) & 3]);
                fetch(it + 5, r[(u + 1) & 3]);
            }
            __syncthreads();
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const int e = (int)threadIdx.x + q * 256, col = e & 31, a = (e >> 5) * CHAIN_ROW + col;
                const long long i = (c0 + (e >> 5)) * SCAN_CHUNK + it * CHAIN_TILE + col;
                if (third && i - 2 * CHAIN_TILE < n) store(i - 2 * CHAIN_TILE, O[a]);
                if (WHAT != 0 && prev) {
                    const double v = S[last + a] + E[a];
                    if (WHAT == 2) O[a] = v;
                    else if (i - CHAIN_TILE < n) store(i - CHAIN_TILE, v);
                }
                if (cur) {
                    const double s = S[buf + a], p = col ? S[buf + a - 1] : carry[e >> 5], b = s - p;
                    E[a] = (p - (s - b)) + (X[buf + a] - b);
                }
            }
            __syncthreads();
        }
    }
    if (role == 0) {
        const double c = __shfl(acc, (lane & (WAVE_CHUNKS - 1)) + WAVE_CHUNKS);
        if (lane < WAVE_CHUNKS) total(c0 + lane, acc + c);
    }
    if (WHAT == 2 && role == 1 && lane < WAVE_CHUNKS) maximum(c0 + lane, mx);
}

// Elements a chain loads ahead of its arithmetic: the chain itself is one dependent
// sequence, but its loads are not, so they are issued in blocks of this many.
constexpr int CHAIN_BLOCK = 64;

// The left-to-right chain of one chunk [lo, hi), in place or not (each block is loaded
// before any of its results is stored).
template <class Op>
__device__ __forceinline__ typename Op::T chain(const typename Op::T *x, typename Op::T *out, long long lo,
                                                long long hi)
{
    typename Op::State st = Op::init();
    typename Op::T last{};
    long long i = lo;
    for (; i + CHAIN_BLOCK <= hi; i += CHAIN_BLOCK) {
        typename Op::T v[CHAIN_BLOCK];
#pragma unroll
        for (int k = 0; k < CHAIN_BLOCK; ++k) v[k] = x[i + k];
#pragma unroll
        for (int k = 0; k < CHAIN_BLOCK; ++k) {
            last = Op::step(st, v[k]);
            out[i + k] = last;
        }
    }
    for (; i < hi; ++i) {
        last = Op::step(st, x[i]);
        out[i] = last;
    }
    return last;
}

template <class Op>
__global__ void __launch_bounds__(256) k_chunk_chain(const typename Op::T *x, typename Op::T *out,
                                                     long long n, typename Op::T *tot)
{
    long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    long long nch = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    if (c >= nch) return;
    long long lo = c * SCAN_CHUNK, hi = lo + SCAN_CHUNK < n ? lo + SCAN_CHUNK : n;
    tot[c] = chain<Op>(x, out, lo, hi);
}

template <class Op>
__global__ void __launch_bounds__(256) k_chunk_offset(typename Op::T *out, long long n,
                                                      const typename Op::T *inc)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    long long c = i / SCAN_CHUNK;
    if (c == 0) return;
    out[i] = Op::combine(inc[c - 1], out[i]);
}

// Elements of level storage needed for a scan of n items.
static inline long long scan_levels_size(long long n)
{
    long long total = 0;
    while (n > 1) {
        n = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
        total += n;
    }
    return total + 8;
}

// Inclusive scan of x[0..n) into out (out may equal x).  levels must hold
// scan_levels_size(n) elements.
template <class Op>
static void chunk_scan(const typename Op::T *x, typename Op::T *out, long long n,
                       typename Op::T *levels, hipStream_t s)
{
    if (n <= 0) return;
    long long nch = (n + SCAN_CHUNK - 1) / SCAN_CHUNK;
    hipLaunchKernelGGL(k_chunk_chain<Op>, dim3((unsigned)LH_CDIV(nch, 256)), dim3(256), 0, s, x, out,
                       n, levels);
    if (nch > 1) {
        chunk_scan<Op>(levels, levels, nch, levels + nch, s);
        hipLaunchKernelGGL(k_chunk_offset<Op>, dim3((unsigned)LH_CDIV(n, 256)), dim3(256), 0, s, out,
                           n, levels);
    }
}

}  // namespace lh
