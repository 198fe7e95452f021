// Canonical chunked scans of binary64 values on the GPU.
//
// The association order is fixed: chunk c covers [c*1024, min((c+1)*1024, n)); the chunk's values
// are one left-to-right chain; the chunk totals are scanned the same way, recursively; element i
// of chunk c > 0 becomes combine(inc[c-1], loc[i]).  For the binary64 compensated sum this order is
// part of the definition of the alias tables' normalisation and prefix sums, so the GPU result is
// bitwise reproducible against any implementation of the same definition.
//
// The constructions read their prefix sums only through searches, so no scan is ever written out
// element by element with its offsets: a scan is the chains' values within each chunk and, per
// chunk, the offset of the chunk (the canonical scan of the totals before it).  They use its
// running maximum; rounding is monotone, so the running maximum of off + x within a chunk is
// off + (the running maximum of x), and across chunks it is enough to keep the largest value
// before the chunk:  value(i) = max(before[c], off[c] + loc[i]),  c = i / 1024.
//
// This header is compiled only into translation units built with -ffp-contract=off.
#pragma once

#include "common.hpp"

namespace lh {

constexpr int SCAN_CHUNK = 1024;

// Neumaier-compensated running sum; the chunk value is s + comp after each element.
struct OpNeumaier {
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

// ---------------------------------------------------------------------------
// The chains of up to 16 chunks of non-negative binary64 values, anywhere in one array, by one
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
// (16.8 M arcs and 1.05 M nodes: the two weight scans together 55 us, the four deficit and excess
// scans 92 us).  Roles rotate with the workgroup's number, so that the chains of several resident
// ones do not share a SIMD.  16 chunks, not 64, spread small arrays over more compute units.
//
// Elements past a chunk's end read as 0, which changes neither s, c nor the maximum.
// WHAT: 0 only the chunk totals, 1 store s + c after each element, 2 store its running maximum.
// segs: the chunks (in LDS, visible to the workgroup; length 0: none).  total(r, s + c) is called
// for every r < 16, maximum(r, m) too for WHAT 2.  load(i) only fetches (any index it is given is
// in range) and the value becomes binary64 a tile later, so that nothing waits for a load in flight.
constexpr int WAVE_CHUNKS = 16;
constexpr int CHAIN_TILE = 32;
constexpr int CHAIN_ROW = CHAIN_TILE + 1;
constexpr int CHAIN_BUF = WAVE_CHUNKS * CHAIN_ROW;
constexpr int CHAIN_LDS = 6 * CHAIN_BUF + WAVE_CHUNKS;  // doubles per workgroup

struct ChainSegs {
    long long start[WAVE_CHUNKS];
    int len[WAVE_CHUNKS];  // at most SCAN_CHUNK
};

// Chunks c0 .. c0 + 15 of an array of n elements (threads below 16; no barrier here).
__device__ __forceinline__ void chunk_segs(ChainSegs &sg, long long c0, long long n)
{
    if (threadIdx.x >= WAVE_CHUNKS) return;
    const long long lo = (c0 + threadIdx.x) * SCAN_CHUNK, left = n - lo;
    sg.start[threadIdx.x] = lo;
    sg.len[threadIdx.x] = left <= 0 ? 0 : left < SCAN_CHUNK ? (int)left : SCAN_CHUNK;
}

template <int WHAT, class Raw, class Load, class Store, class Total, class Maximum>
__device__ __forceinline__ void block_chains(double *lds, const ChainSegs &segs, Load load, Store store, Total total,
                                             Maximum maximum)
{
    double *const X = lds, *const S = lds + 2 * CHAIN_BUF, *const E = lds + 4 * CHAIN_BUF, *const O = lds + 5 * CHAIN_BUF,
                  *const carry = lds + 6 * CHAIN_BUF;
    const int lane = threadIdx.x & 63, role = ((threadIdx.x >> 6) + blockIdx.x) & 3;
    int most = 0;
#pragma unroll
    for (int k = 0; k < WAVE_CHUNKS; ++k) most = segs.len[k] > most ? segs.len[k] : most;
    const int tiles = LH_CDIV(most, CHAIN_TILE);
    // the loaders' elements of a tile: four each, in chunks (l0 >> 5) + 4 q
    const int l0 = (role & 1) * 64 + lane, lcol = l0 & 31;
    Raw r[4][4];
    long long lstart[4];
    int llen[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        lstart[q] = segs.start[(l0 >> 5) + 4 * q];
        llen[q] = segs.len[(l0 >> 5) + 4 * q];
    }
    auto fetch = [&](int t, Raw(&d)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = t * CHAIN_TILE + lcol;
            d[q] = load(llen[q] > 0 ? lstart[q] + (k < llen[q] ? k : llen[q] - 1) : segs.start[0]);
        }
    };
    auto place = [&](int t, const Raw(&d)[4]) {
#pragma unroll
        for (int q = 0; q < 4; ++q)
            X[(t & 1) * CHAIN_BUF + ((l0 >> 5) + 4 * q) * CHAIN_ROW + lcol] =
                t * CHAIN_TILE + lcol < llen[q] ? (double)d[q] : 0.0;
    };
    // the elements of a tile whose errors, sums and stores this thread takes: two
    long long estart[2];
    int elen[2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        estart[q] = segs.start[((int)threadIdx.x + q * 256) >> 5];
        elen[q] = segs.len[((int)threadIdx.x + q * 256) >> 5];
    }
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
                const int i = it * CHAIN_TILE + col;
                if (third && i - 2 * CHAIN_TILE < elen[q]) store(estart[q] + (i - 2 * CHAIN_TILE), O[a]);
                if (WHAT != 0 && prev) {
                    const double v = S[last + a] + E[a];
                    if (WHAT == 2) O[a] = v;
                    else if (i - CHAIN_TILE < elen[q]) store(estart[q] + (i - CHAIN_TILE), v);
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
        if (lane < WAVE_CHUNKS) total(lane, acc + c);
    }
    if (WHAT == 2 && role == 1 && lane < WAVE_CHUNKS) maximum(lane, mx);
}

struct Scan {
    const double *loc;     // [n] per element, within its chunk
    const double *off;     // [chunks] canonical scan of the totals before the chunk (0 for the first)
    const double *before;  // [chunks] largest value before the chunk (-inf for the first)
    const double *end;     // [chunks] value of the chunk's last element
    long long n;

    __device__ __forceinline__ double at(long long i) const
    {
        const long long c = i / SCAN_CHUNK;
        return __builtin_fmax(before[c], off[c] + loc[i]);
    }
};

// The levels above the chunks, one workgroup per scan: the canonical scan of the chunk totals (its
// own chains as above, the totals of those, at most 4,096 for 2^32 items, by one thread), which
// becomes each chunk's offset.  tot is left with the chains' values.
constexpr int LEVEL_THREADS = 256, LEVEL_TOP = 4096;

struct LevelLds {
    double chains[CHAIN_LDS];
    double top[LEVEL_TOP];
    ChainSegs segs;
};

__device__ __forceinline__ void scan_levels(double *tot, double *off, long long nch, LevelLds &l)
{
    double *const top = l.top;
    const long long n1 = LH_CDIV(nch, SCAN_CHUNK);
    for (long long c0 = 0; c0 < n1; c0 += WAVE_CHUNKS) {
        chunk_segs(l.segs, c0, nch);
        __syncthreads();
        block_chains<1, double>(l.chains, l.segs, [&](long long i) { return tot[i]; },
                                [&](long long i, double v) { tot[i] = v; },
                                [&](int r, double v) { if (c0 + r < n1) top[c0 + r] = v; }, [](int, double) {});
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        // chunks of 1,024 again: at most four, offset by the totals before them (the totals of
        // their totals are one chunk)
        OpNeumaier::State up = OpNeumaier::init();
        double base = 0.0;
        for (long long lo = 0; lo < n1; lo += SCAN_CHUNK) {
            OpNeumaier::State st = OpNeumaier::init();
            double v = 0.0;
            for (long long i = lo; i < n1 && i < lo + SCAN_CHUNK; ++i) {
                v = OpNeumaier::step(st, top[i]);
                top[i] = lo ? OpNeumaier::combine(base, v) : v;
            }
            base = OpNeumaier::step(up, v);
        }
    }
    __syncthreads();
    if (threadIdx.x == 0) off[0] = 0.0;
    // (eight loads at a time: the compiler keeps each behind the store before it otherwise)
    for (long long i0 = threadIdx.x; i0 + 1 < nch; i0 += 8 * LEVEL_THREADS) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = i0 + k * LEVEL_THREADS + 1 < nch ? tot[i0 + k * LEVEL_THREADS] : 0.0;
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const long long i = i0 + k * LEVEL_THREADS, c = i / SCAN_CHUNK;
            if (i + 1 < nch) off[i + 1] = c ? OpNeumaier::combine(top[c - 1], v[k]) : v[k];
        }
    }
    __syncthreads();
}

// Prefix maxima of a scan's chunks: end[c] (the chunk's own maximum) becomes the largest value up to
// the chunk's last element, before[c] the largest before the chunk.
__device__ __forceinline__ void scan_maxima(const double *off, double *before, double *end, long long nch, LevelLds &l)
{
    double *const top = l.top;
    // a consecutive quarter of the chunks per wavefront, 4 x 64 of them at a time
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const long long per = LH_CDIV(nch, LEVEL_THREADS) * 64;
    const long long lo = wave * per, hi = lo + per < nch ? lo + per : nch;
    const double none = -__builtin_huge_val();
    auto four = [&](long long c, double(&v)[4]) {
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const long long i = c + k * 64 + lane;
            v[k] = i < hi ? off[i] + end[i] : none;
        }
    };
    double m = none, v[4];
    for (long long c = lo; c < hi; c += 256) {
        four(c, v);
        m = __builtin_fmax(m, __builtin_fmax(__builtin_fmax(v[0], v[1]), __builtin_fmax(v[2], v[3])));
    }
    for (int d = 32; d >= 1; d >>= 1) m = __builtin_fmax(m, __shfl_xor(m, d));
    if (lane == 0) top[wave] = m;
    __syncthreads();
    double run = none;
    for (int w = 0; w < wave; ++w) run = __builtin_fmax(run, top[w]);
    for (long long c = lo; c < hi; c += 256) {
        four(c, v);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            double inc = v[k];
            for (int d = 1; d < 64; d <<= 1) {
                const double y = __shfl_up(inc, d);
                if (lane >= d) inc = __builtin_fmax(inc, y);
            }
            double exc = __shfl_up(inc, 1);
            if (lane == 0) exc = none;
            const long long i = c + k * 64 + lane;
            if (i < hi) {
                before[i] = __builtin_fmax(run, exc);
                end[i] = __builtin_fmax(run, inc);
            }
            run = __builtin_fmax(run, __shfl(inc, 63));
        }
    }
}

}  // namespace lh
