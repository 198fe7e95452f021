// The sweeping construction of alias tables, for tables of any length: the two tables of a graph
// (alias.hip) and the rows of the walk graph that are too long for one workgroup (walk.hip).
//
// A set of tables is built by one sequence of launches; Set says which table a workgroup works on:
//   of(b)      the table of this workgroup (Table below with its q and its records' writer), and in
//              b the workgroup's number within it, which may lie beyond the table's end
//   whole(k)   table k
//
// Compiled only into translation units built with -ffp-contract=off.
#pragma once

#include "scan.hpp"

namespace lh {

__device__ __forceinline__ unsigned long long prob_to_thr(double prob)
{
    if (prob >= 1.0) return ~0ull;
    return (unsigned long long)__dmul_rn(prob, 18446744073709551616.0);
}

constexpr int SPLIT_ITEMS = 1024;  // items a wavefront splits

struct Table {
    long long N;
    const float *w;        // item weights, or NULL (a table's own matter)
    double *dx;            // [N] deficits of the lights, then excesses of the heavies
    uint32_t *idx;         // [N] the heavies' items, in index order
    uint32_t *blk;         // [N / 1024 + 2] lights before each 1,024 items; last: all of them
    double *tot, *mxl;     // [N / 1024 + 2] chunk totals and chunk maxima, then (in place)
                           // the totals' own chains and the chunks' last values
    double *off, *before;  // [N / 1024 + 2]
    double *W;             // total weight

    __device__ __forceinline__ long long lights() const { return blk[LH_CDIV(N, SPLIT_ITEMS)]; }
    // The scan of one half (false: lights, true: heavies), its chunks after the lights' ones.
    __device__ __forceinline__ Scan half(bool heavy, long long nL) const
    {
        const long long c0 = heavy ? LH_CDIV(nL, SCAN_CHUNK) : 0;
        return Scan{dx + (heavy ? nL : 0), off + c0, before + c0, mxl + c0, heavy ? N - nL : nL};
    }
};

// q_i = fl(fl(w_i N) / W).  A total that is not a positive finite number makes every item heavy
// (prob 1, self).
__device__ __forceinline__ double alias_q(double w, long long N, double W)
{
    return W > 0.0 && !isinf(W) ? __ddiv_rn(__dmul_rn(w, (double)N), W) : 1.0;
}

// Total weight of a table: off[last chunk] + that chunk's total (thread 0 gets it and stores it).
__device__ __forceinline__ double levels_weight(const Table &t, LevelLds &l)
{
    const long long nch = LH_CDIV(t.N, SCAN_CHUNK);
    const double last = t.tot[nch - 1];  // before the totals become their chains
    __syncthreads();
    scan_levels(t.tot, t.off, nch, l);
    const double W = nch > 1 ? OpNeumaier::combine(t.off[nch - 1], last) : last;
    if (threadIdx.x == 0) *t.W = W;
    return W;
}

// Offsets and prefix maxima of the deficit and excess scans (workgroup: table, half).
template <class Set>
__global__ void __launch_bounds__(LEVEL_THREADS) k_levels_dx(Set T)
{
    __shared__ LevelLds l;
    const auto &t = T.whole(blockIdx.x >> 1);
    const bool heavy = (blockIdx.x & 1) != 0;
    const long long nL = t.lights(), n = heavy ? t.N - nL : nL;
    if (n == 0) return;
    const long long c0 = heavy ? LH_CDIV(nL, SCAN_CHUNK) : 0, nch = LH_CDIV(n, SCAN_CHUNK);
    double *off = t.off + c0, *before = t.before + c0, *end = t.mxl + c0;
    scan_levels(t.tot + c0, off, nch, l);
    scan_maxima(off, before, end, nch, l);
}

// Lights (q < 1) among 1,024 consecutive items, per wavefront.
template <class Set>
__global__ void __launch_bounds__(256) k_split_count(Set T)
{
    long long b;
    const auto &t = T.of(b);
    const int lane = threadIdx.x & 63;
    const long long part = b * 4 + (threadIdx.x >> 6), lo = part * SPLIT_ITEMS;
    if (lo >= t.N) return;
    const double W = *t.W;
    uint32_t cnt = 0;
#pragma unroll 4
    for (int r = 0; r < SPLIT_ITEMS / 64; ++r) {
        const long long i = lo + r * 64 + lane;
        cnt += __popcll(__ballot(i < t.N && t.q(i < t.N ? i : 0, W) < 1.0));
    }
    if (lane == 0) t.blk[part] = cnt;
}

// Exclusive prefix sums of the light counts, in place, with the total behind them; one workgroup
// per table, a run of counts per thread.
template <class Set>
__global__ void __launch_bounds__(1024) k_split_scan(Set T)
{
    __shared__ uint32_t ws[16];
    const auto &t = T.whole(blockIdx.x);
    const long long nt = LH_CDIV(t.N, SPLIT_ITEMS), per = LH_CDIV(nt, 1024);
    const long long lo = threadIdx.x * per, hi = lo + per < nt ? lo + per : nt;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    uint32_t s = 0;
#pragma unroll 8
    for (long long i = lo; i < hi; ++i) s += t.blk[i];
    uint32_t inc = s;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d);
        if (lane >= d) inc += y;
    }
    if (lane == 63) ws[wave] = inc;
    __syncthreads();
    uint32_t run = inc - s;
    for (int v = 0; v < wave; ++v) run += ws[v];
#pragma unroll 8
    for (long long i = lo; i < hi; ++i) {
        const uint32_t c = t.blk[i];
        t.blk[i] = run;
        run += c;
    }
    if (threadIdx.x == 1023) t.blk[nt] = run;
}

// Split into lights (deficits 1 - q, prefix of dx) and heavies (excesses q - 1, suffix, and their
// items), each in index order.  q is computed again from the weight: cheaper than a pass that
// stores it.
template <class Set>
__global__ void __launch_bounds__(256) k_split(Set T)
{
    long long b;
    const auto &t = T.of(b);
    const int lane = threadIdx.x & 63;
    const long long part = b * 4 + (threadIdx.x >> 6), lo = part * SPLIT_ITEMS;
    if (lo >= t.N) return;
    const double W = *t.W;
    const long long nL = t.lights();
    long long a = t.blk[part];
#pragma unroll 4
    for (int r = 0; r < SPLIT_ITEMS / 64; ++r) {
        const long long i = lo + r * 64 + lane;
        const double q = i < t.N ? t.q(i, W) : 1.0;
        const unsigned long long mask = __ballot(q < 1.0);
        const long long before = a + __popcll(mask & ((1ull << lane) - 1ull));  // lights before item i
        if (i < t.N) {
            if (q < 1.0) {
                t.dx[before] = __dsub_rn(1.0, q);
            } else {
                t.dx[nL + (i - before)] = __dsub_rn(q, 1.0);
                t.idx[i - before] = (uint32_t)i;
            }
        }
        a += __popcll(mask);
    }
}

// First position in [lo, hi) whose value is not `below` (values are monotone), by a whole
// wavefront: 64 probes at a time.
template <class Below>
__device__ __forceinline__ long long wave_search(long long lo, long long hi, Below below)
{
    const int lane = threadIdx.x & 63;
    while (lo < hi) {
        const long long step = LH_CDIV(hi - lo, 64);
        const long long pos = lo + (lane + 1) * step - 1;  // last position of this lane's part
        const long long parts = __popcll(__ballot(pos < hi && below(pos)));
        lo += parts * step;
        if (step == 1) break;
        if (lo + step - 1 < hi) hi = lo + step - 1;  // its part's last position is not below
    }
    return lo;
}

// The same over a scan: first among the chunks' last values, then inside the chunk.
template <class Less>
__device__ __forceinline__ long long wave_search_scan(const Scan &x, long long n, Less less)
{
    // n <= x.n positions; the chunk's `end` stands for its last position, which may lie past n
    const long long nch = LH_CDIV(n, SCAN_CHUNK);
    const long long c = wave_search(0, nch, [&](long long k) { return less(x.end[k]); });
    if (c >= nch) return n;
    const long long lo = c * SCAN_CHUNK, hi = lo + SCAN_CHUNK < n ? lo + SCAN_CHUNK : n;
    const double before = x.before[c], off = x.off[c];
    return wave_search(lo, hi, [&](long long i) { return less(__builtin_fmax(before, off + x.loc[i])); });
}

// Records: light a with start S_a = D[a-1] (S_0 = 0) aliases heavy #{X[k] <= S_a}; heavy k finds
// the last light that starts before X[k].  A workgroup writes 1,024 consecutive items, whose
// lights and whose heavies are each a consecutive run: whole lines are written, and the item's
// own weight and endpoints are read in order.  Both sequences are monotone, so the answers of a
// run lie between those of its two ends, which one wavefront each searches for; the stretch of
// the other sequence between them is staged in LDS when it fits (it is about as long as the run
// times the ratio of the halves), and the items' own searches touch no memory.  A graph's two
// tables (16.8 M arcs, 1.05 M nodes): 0.51 ms, 0.87 ms with a thread per light and per heavy that
// searched all of the other half and wrote every second record of a line.  What is left is 0.24 ms
// of traffic at a copy's rate and 0.14 ms of heat bytes (67 M scattered reads).
constexpr int REC_ITEMS = 1024, REC_STAGE = 1024;
static_assert(REC_ITEMS == SPLIT_ITEMS, "a workgroup's first light is its split count");

// The two halves' scans lie one behind the other: position p of half `heavy` is element
// (heavy ? nL : 0) + p, in chunk (heavy ? cL : 0) + p / 1024.
// A run of 256 RS items at most takes RS per thread: rows of a few hundred items are common.
struct RecLds {
    double sx[REC_STAGE], sd[REC_STAGE + 1];
    long long ends[4];
    int32_t wc[4];
};

template <int RS, class T>
__device__ __forceinline__ void records_run(const T &t, long long b, RecLds &lds)
{
    double *const sx = lds.sx, *const sd = lds.sd;
    long long *const ends = lds.ends;
    int32_t *const wc = lds.wc;
    const long long N = t.N, nL = t.lights(), nH = N - nL, cL = LH_CDIV(nL, SCAN_CHUNK), i0 = b * REC_ITEMS;
    const long long i1 = i0 + REC_ITEMS < N ? i0 + REC_ITEMS : N;
    const long long a0 = t.blk[b], a1 = t.blk[b + 1], h0 = i0 - a0, h1 = i1 - a1;  // the runs
    const Scan D = t.half(false, nL), X = t.half(true, nL);
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double W = *t.W;
    // lights: count of X <= S_a; heavies: count of D < X[k] over the lights but the last (the
    // start of light a >= 1 is D[a - 1])
    const long long nD = nL > 0 ? nL - 1 : 0;
    {
        long long k = 0;
        if (N <= REC_ITEMS) {  // one run: the whole of both sequences
            k = wave == 1 ? nH : wave == 3 ? nD : 0;
        } else if (wave < 2) {
            const long long a = wave == 0 ? a0 : a1 - 1;
            if (a1 > a0 && nH > 0) {
                const double s = a == 0 ? 0.0 : D.at(a - 1);
                k = wave_search_scan(X, nH, [&](double v) { return v <= s; });
            }
        } else {
            const long long p = wave == 2 ? h0 : h1 - 1;
            if (h1 > h0 && nD > 0) {
                const double x = X.at(p);
                k = wave_search_scan(D, nD, [&](double v) { return v < x; });
            }
        }
        if (lane == 0) ends[wave] = k;
    }
    // item r of this thread: i0 + wave * 64 RS + r * 64 + lane.  Each step below is taken for all
    // its items before the next, so that their loads are in flight together.
    const long long first = i0 + wave * (64 * RS) + lane;
    double q[RS];
    unsigned long long mask[RS];
    int32_t cnt = 0;
#pragma unroll
    for (int r = 0; r < RS; ++r) {
        const long long i = first + r * 64;
        const double qi = t.q(i < i1 ? i : i1 - 1, W);
        q[r] = i < i1 ? qi : 1.0;
        mask[r] = __ballot(q[r] < 1.0);
        cnt += __popcll(mask[r]);
    }
    if (lane == 0) wc[wave] = cnt;
    __syncthreads();
    const long long x0 = ends[0], d0 = ends[2];
    const int xn = (int)(ends[1] - x0), dn = (int)(ends[3] - d0), dr = dn + (nL > 0 ? 1 : 0);
    const bool staged = xn <= REC_STAGE && dr <= REC_STAGE + 1;
    if (staged) {
        for (int i = threadIdx.x; i < xn; i += 256) sx[i] = X.at(x0 + i);
        for (int i = threadIdx.x; i < dr; i += 256) sd[i] = D.at(d0 + i);  // heavies read D at their answer too
    }
    long long a = a0;
    for (int v = 0; v < wave; ++v) a += wc[v];
    long long pos[RS];  // lights before the item, or its place among the heavies
    double key[RS];     // S_a, or X[k]
#pragma unroll
    for (int r = 0; r < RS; ++r) {
        const long long i = first + r * 64;
        const long long before = a + __popcll(mask[r] & ((1ull << lane) - 1ull));
        a += __popcll(mask[r]);
        const bool light = q[r] < 1.0;
        pos[r] = light ? before : (i < i1 ? i - before : 0);
        const long long p = light ? (before > 0 ? before - 1 : 0) : pos[r];
        const long long c = (light ? 0 : cL) + p / SCAN_CHUNK;
        const double v = nH == 0 && !light ? 0.0 : __builtin_fmax(t.before[c], t.off[c] + t.dx[(light ? 0 : nL) + p]);
        key[r] = light && before == 0 ? 0.0 : v;
    }
    __syncthreads();
    int lo[RS] = {};
    if (staged) {
        int hi[RS];
#pragma unroll
        for (int r = 0; r < RS; ++r) hi[r] = q[r] < 1.0 ? xn : dn;
        for (int left = xn > dn ? xn : dn; left > 0; left >>= 1) {
#pragma unroll
            for (int r = 0; r < RS; ++r) {
                const bool light = q[r] < 1.0;
                const int mid = (lo[r] + hi[r]) >> 1;
                const double y = light ? sx[mid < xn ? mid : 0] : sd[mid];
                const bool up = lo[r] < hi[r] && (light ? y <= key[r] : y < key[r]);
                if (up) lo[r] = mid + 1;
                else if (lo[r] < hi[r]) hi[r] = mid;
            }
        }
    } else {
#pragma unroll 1
        for (int r = 0; r < RS; ++r) {
            const bool light = q[r] < 1.0;
            int l = 0, h = light ? xn : dn;
            while (l < h) {
                const int mid = l + ((h - l) >> 1);
                const double y = light ? X.at(x0 + mid) : D.at(d0 + mid);
                if (light ? y <= key[r] : y < key[r]) l = mid + 1;
                else h = mid;
            }
            lo[r] = l;
        }
    }
    unsigned long long thr[RS];
    uint32_t al[RS];
#pragma unroll
    for (int r = 0; r < RS; ++r) {
        const bool light = q[r] < 1.0;
        long long k = -1;  // the heavy that the item aliases (-1: itself)
        thr[r] = ~0ull;
        if (light) {
            if (nH > 0) {
                k = x0 + lo[r] < nH - 1 ? x0 + lo[r] : nH - 1;
                thr[r] = prob_to_thr(q[r]);
            }
        } else if (pos[r] < nH - 1 && nL > 0 && 0.0 < key[r]) {
            // light d0 + lo is the last that starts before X[k]; its deficit sum past X[k] is
            // what overflows to the next heavy
            double ov = __dsub_rn(staged ? sd[lo[r]] : D.at(d0 + lo[r]), key[r]);
            if (ov < 0.0) ov = 0.0;
            if (ov > 0.0) {
                const double pr = __dsub_rn(1.0, ov);
                thr[r] = prob_to_thr(pr < 0.0 ? 0.0 : pr);
                k = pos[r] + 1;
            }
        }
        const uint32_t item = t.idx[k < 0 ? 0 : k];
        al[r] = k < 0 ? (uint32_t)(first + r * 64) : item;
    }
    t.template write<RS>(first, i1, thr, al);
}

}  // namespace lh
