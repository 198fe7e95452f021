// Random-walk positive pairs (Sec. IV-B: Algorithm 2, RandomWalk, and Algorithm 3,
// GeneratePairs) on one GPU, where every vertex is local: the walks never stop at a
// remote vertex (the paper's "Local" variant over the whole graph).  Built with
// -ffp-contract=off: the per-row alias tables are binary64 and bitwise reproducible.
//
// Walk graph: the undirected graph of the arcs.  Entry e < m is arc e forwards (tail
// src[e], head dst[e]), entry m + e arc e backwards; both weigh w[e].  Row x (the
// neighbourhood N(x)) lists the entries with tail x in increasing entry index: a stable
// radix sort of the entries by tail.  discrete(N(x)) is the alias table of the row's
// weights, built exactly as the edge and negative tables are (table.hpp) but per row:
// the canonical scans restart at every row, and items are numbered within the row.
//
// Walk k: Philox4x64-10 key (seed, 5 * 2^32 | graph_id).  Block (k, 0, 0, 0) draws the
// root arc from the edge table (Algorithm 3's weight-normalised edge distribution):
// w_0 = its tail, w_1 = its head.  Block (k, t, 0, 0), t = 1 .. L - 2, draws w_{t+1}
// from row w_t.  A walk visits L vertices (Algorithm 2 counts visited vertices, root
// pair included, up to the walk length).  Pairs: (w_i, w_{i+delta}), delta = 1 .. W - 1
// (window W; W = 2 gives the consecutive pairs Algorithm 2 collects), numbered
// p = sum_{delta' < delta} (L - delta') + i.  Sample order (Algorithm 3 shuffles a
// batch's pairs): sample s = b Bw P + p Bw + j is pair p of walk b Bw + j.
#include <algorithm>
#include <cmath>

#include "handle.hpp"
#include "sort.hpp"
#include "table.hpp"
#include "tile.hpp"

#pragma clang fp contract(off)

namespace lh {

constexpr unsigned long long kWalkTag = 5ull;
constexpr int kWalkMaxWindow = 8;
constexpr int kWalkMaxLength = 4096;
// Pairs one buffer fill aims at (the chunk holds whole walk batches).
constexpr long long kWalkChunkPairs = 1ll << 24;

static size_t carve(size_t &off, size_t bytes)
{
    size_t at = off;
    off = lh_align_up(off + bytes, 256);
    return at;
}

WalkLayout walk_layout(long long n, long long m, int L, int W, long long Bw)
{
    WalkLayout w;
    w.P = 0;
    for (int dl = 1; dl < W; ++dl) w.P += L - dl;
    const long long per = Bw * w.P;
    const long long batches = per >= kWalkChunkPairs ? 1 : kWalkChunkPairs / per;
    w.chunk_walks = Bw * batches;
    size_t off = 0;
    w.off = carve(off, 8 * (size_t)(n + 1));
    w.rec = carve(off, sizeof(WalkRec) * (size_t)(2 * m > 0 ? 2 * m : 1));
    w.pairs = carve(off, 8 * (size_t)w.chunk_walks * (size_t)w.P);
    w.total = off;
    return w;
}

namespace {

// A row longer than ROW_SHORT, as a table of its own (table.hpp).
constexpr int ROW_SHORT = 256, ROW_HUGE = 64 * SCAN_CHUNK;

struct LongRow {
    long long lo, len;  // its entries
    long long slot;     // its first word in the arrays of chunk values: len / 1024 + 2 of them at most
    double W;
};

struct WalkScratch {
    size_t k0, w0, h0, k1, w1, h1, dx, hist, part, cnt, rows, huge, slot_row, blk, tot, mxl, off, before, total;
};

WalkScratch walk_scratch_layout(long long n, long long m)
{
    (void)n;
    WalkScratch L;
    const long long E = 2 * m > 0 ? 2 * m : 1;
    const long long rows = E / (ROW_SHORT + 1) + 1, slots = E / SCAN_CHUNK + 2 * rows;
    size_t off = 0;
    L.k0 = carve(off, 4 * (size_t)E);
    L.w0 = carve(off, 4 * (size_t)E);
    L.h0 = carve(off, 4 * (size_t)E);
    L.k1 = carve(off, 4 * (size_t)E);
    L.w1 = carve(off, 4 * (size_t)E);
    L.h1 = carve(off, 4 * (size_t)E);
    L.dx = carve(off, 8 * (size_t)E);
    L.hist = carve(off, 4 * (size_t)sort_hist_size(E));
    L.part = carve(off, 4 * (size_t)sort_part_size(E));
    L.cnt = carve(off, 3 * sizeof(unsigned long long));
    L.rows = carve(off, sizeof(LongRow) * (size_t)rows);
    L.huge = carve(off, 4 * (size_t)(E / ROW_HUGE + 1));
    L.slot_row = carve(off, 4 * (size_t)slots);
    L.blk = carve(off, 4 * (size_t)slots);
    L.tot = carve(off, 8 * (size_t)slots);
    L.mxl = carve(off, 8 * (size_t)slots);
    L.off = carve(off, 8 * (size_t)slots);
    L.before = carve(off, 8 * (size_t)slots);
    L.total = off;
    return L;
}

// The entries as the sort's first pass reads them: the tail, and as payloads the weight and the
// head, which the rows need and which would otherwise be gathered by entry afterwards (a
// scattered 4-byte read per entry and array: 0.6 ms each on C2's 33.6 M entries).
struct WalkEntries {
    static constexpr int PAY = 2;
    const int32_t *src, *dst;
    const float *w;
    unsigned long long m;
    __device__ __forceinline__ uint32_t key(unsigned long long e) const { return (uint32_t)(e < m ? src[e] : dst[e - m]); }
    __device__ __forceinline__ uint32_t pay(unsigned long long e, int which) const
    {
        const unsigned long long a = e < m ? e : e - m;
        if (which == 0) return __float_as_uint(w[a]);
        return (uint32_t)(e < m ? dst[a] : src[a]);
    }
};

}  // namespace

// ---------------------------------------------------------------------------
// Rows of the walk graph.
// ---------------------------------------------------------------------------
// off[x] = the first sorted position whose tail is >= x; off[n] = E.  Clears the counters of k_rows.
__global__ void __launch_bounds__(256) k_row_offsets(const uint32_t *ks, long long E, long long n, long long *off,
                                                     unsigned long long *cnt)
{
    if (blockIdx.x == 0 && threadIdx.x < 3) cnt[threadIdx.x] = 0ull;
    const long long i0 = (long long)blockIdx.x * 1024 + threadIdx.x;
    long long k[4], prev[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const long long i = i0 + r * 256 < E ? i0 + r * 256 : E - 1;
        k[r] = ks[i];
        prev[r] = i == 0 ? -1 : (long long)ks[i - 1];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const long long i = i0 + r * 256;
        if (i >= E) break;
        for (long long x = prev[r] + 1; x <= k[r]; ++x) off[x] = i;
        if (i == E - 1)
            for (long long x = k[r] + 1; x <= n; ++x) off[x] = E;
    }
}

// The chain of one short row (values in LDS, one chunk) by one thread, eight values at a time; the
// errors as in block_chains.  SCAN: each value becomes the running maximum of s + c; otherwise only
// the total s + c is wanted, and returned.
struct RowChain {
    double s, c, m;

    template <bool SCAN>
    __device__ __forceinline__ void eight(double (&v)[8])
    {
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const double p = s;
            s = p + v[k];
            const double b = s - p;
            c += (p - (s - b)) + (v[k] - b);
            if (SCAN) v[k] = m = __builtin_fmax(m, s + c);
        }
    }
};

template <bool SCAN>
__device__ __forceinline__ double row_chain(double *x, int n)
{
    RowChain r{0.0, 0.0, -__builtin_huge_val()};
    int k0 = 0;
    for (; k0 + 8 <= n; k0 += 8) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = x[k0 + k];
        r.eight<SCAN>(v);
        if (SCAN) {
#pragma unroll
            for (int k = 0; k < 8; ++k) x[k0 + k] = v[k];
        }
    }
    if (k0 < n) {
        double v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            v[k] = x[k0 + k < n ? k0 + k : k0];
            if (k0 + k >= n) v[k] = 0.0;
        }
        r.eight<SCAN>(v);
        if (SCAN) {
#pragma unroll
            for (int k = 0; k < 8; ++k)
                if (k0 + k < n) x[k0 + k] = v[k];
        }
    }
    return r.s + r.c;
}

// Items of 256 threads' flags, 8 per thread (thread t has items t, 256 + t, ..): flags before each
// group of 64 items go to at[r][wave]; the total is returned.
constexpr int ROW_WINDOW = 2048, ROW_TILE = ROW_WINDOW - ROW_SHORT, ROW_PER = ROW_WINDOW / 256;

__device__ __forceinline__ int flag_groups(const unsigned long long (&mask)[ROW_PER], uint16_t *at)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r)
        if (lane == r) at[r * 4 + wave] = (uint16_t)__popcll(mask[r]);
    __syncthreads();
    // (every wavefront for itself: lane g sums the groups up to g)
    const int own = lane < 4 * ROW_PER ? at[lane] : 0;
    int inc = own;
#pragma unroll
    for (int d = 1; d < 4 * ROW_PER; d <<= 1) {
        const int y = __shfl_up(inc, d);
        if (lane >= d) inc += y;
    }
    __syncthreads();
    if (wave == 0 && lane < 4 * ROW_PER) at[lane] = (uint16_t)(inc - own);
    __syncthreads();
    return __shfl(inc, 4 * ROW_PER - 1);
}

// Records of the rows that start among this workgroup's ROW_TILE sorted entries and are at most
// ROW_SHORT long, in LDS from the weights to the records, which are written in order; longer rows are only
// listed.  A thread runs a row's chain, then a light or heavy half's.
//
// What bounds it is the instructions of the chains (a wavefront runs as long as its longest row) and
// of the entries' divisions and searches.  The limit of 256 entries and the tile of 1,792 (a window
// of 2,048) keep the one small and fill the lanes: 33.6 M entries in 0.57 ms, with rows of up to
// 1,024 and tiles of 1,024 in 0.96 ms.  The longer rows, which need 0.95 ms there, took 1.5 ms a
// workgroup each.  A kernel per step over all rows (a thread per chain in memory, three scans with
// their offsets written out) took 4.1 ms for all rows.
__global__ void __launch_bounds__(256) k_rows(const uint32_t *ks, const float *ws, const uint32_t *hs, const long long *off,
                                              long long E, WalkRec *rec, LongRow *rows, uint32_t *huge,
                                              uint32_t *slot_row, unsigned long long *cnt)
{
    __shared__ double v[ROW_WINDOW];      // weights, then per row deficits and excesses, then their scans
    __shared__ uint16_t idx[ROW_WINDOW];  // at a heavy's place in the split: its entry
    __shared__ uint16_t start[ROW_TILE], len[ROW_TILE], lights[ROW_TILE + 1];  // per row; lights before it
    __shared__ uint16_t at[4 * ROW_PER];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long below = (1ull << lane) - 1ull;
    const long long p0 = (long long)blockIdx.x * ROW_TILE;
    const int owned = (int)(E - p0 < ROW_TILE ? E - p0 : ROW_TILE), here = (int)(E - p0 < ROW_WINDOW ? E - p0 : ROW_WINDOW);
    // entry r of this thread: r * 256 + threadIdx.x
    float w[ROW_PER];
    uint32_t key[ROW_PER], prev[ROW_PER];
    unsigned long long mask[ROW_PER];
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r) {
        const int i = r * 256 + (int)threadIdx.x;
        const long long p = p0 + (i < here ? i : here - 1);
        w[r] = ws[p];
        key[r] = ks[p];
        prev[r] = ks[p > 0 ? p - 1 : 0];
    }
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r) {
        const int i = r * 256 + (int)threadIdx.x;
        mask[r] = __ballot(i < owned && (p0 + i == 0 || prev[r] != key[r]));
        v[i] = (double)w[r];
    }
    const int nrows = flag_groups(mask, at);
    int row[ROW_PER];
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r) {
        const int i = r * 256 + (int)threadIdx.x;
        const bool head = (mask[r] >> lane) & 1ull;
        row[r] = at[r * 4 + wave] + __popcll(mask[r] & below) + (head ? 1 : 0) - 1;
        if (!head) continue;
        const long long lo = p0 + i, n = off[key[r] + 1] - lo;
        start[row[r]] = (uint16_t)i;
        len[row[r]] = n <= ROW_SHORT ? (uint16_t)n : (uint16_t)0;
        if (n > ROW_SHORT) {
            const unsigned long long slots = LH_CDIV(n, SCAN_CHUNK) + 1;
            const unsigned long long k = atomicAdd(&cnt[0], 1ull), s = atomicAdd(&cnt[1], slots);
            rows[k] = LongRow{lo, n, (long long)s, 0.0};
            if (n > ROW_HUGE) huge[atomicAdd(&cnt[2], 1ull)] = (uint32_t)k;
            for (unsigned long long j = 0; j < slots; ++j) slot_row[s + j] = (uint32_t)k;
        }
    }
    __syncthreads();
    for (int x = threadIdx.x; x < nrows; x += 256) {
        const int n = len[x];
        if (n > 0) {
            const double W = row_chain<false>(v + start[x], n);
            v[start[x]] = W;  // (the weights are in registers)
        }
    }
    __syncthreads();
    double q[ROW_PER];
    bool mine[ROW_PER];
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r) {
        const int i = r * 256 + (int)threadIdx.x;
        const int x = row[r] < 0 ? 0 : row[r], n = len[x], j = i - start[x];
        mine[r] = row[r] >= 0 && j < n;
        q[r] = mine[r] ? alias_q((double)w[r], n, v[start[x]]) : 1.0;
        mask[r] = __ballot(q[r] < 1.0);
    }
    const int nlights = flag_groups(mask, at);
    if (threadIdx.x == 0) lights[nrows] = (uint16_t)nlights;
    int a[ROW_PER];  // lights before the entry
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r) {
        const int i = r * 256 + (int)threadIdx.x;
        a[r] = at[r * 4 + wave] + __popcll(mask[r] & below);
        if (row[r] >= 0 && i == start[row[r]]) lights[row[r]] = (uint16_t)a[r];
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r) {
        if (!mine[r]) continue;
        const int i = r * 256 + (int)threadIdx.x, s = start[row[r]], l0 = lights[row[r]], nL = lights[row[r] + 1] - l0;
        a[r] -= l0;
        if (q[r] < 1.0) {
            v[s + a[r]] = __dsub_rn(1.0, q[r]);
        } else {
            const int p = s + nL + (i - s - a[r]);
            v[p] = __dsub_rn(q[r], 1.0);
            idx[p] = (uint16_t)i;
        }
    }
    __syncthreads();
    for (int x = threadIdx.x; x < 2 * nrows; x += 256) {
        const int n = len[x >> 1], nL = n > 0 ? lights[(x >> 1) + 1] - lights[x >> 1] : 0;
        double *const d = v + start[x >> 1] + (x & 1 ? nL : 0);
        (void)row_chain<true>(d, x & 1 ? n - nL : nL);
    }
    __syncthreads();
    // Searches, in step for all of a thread's entries: a light's start S = D[a - 1] among the row's
    // excesses, a heavy's X[k] among its deficits but the last.
    int lo[ROW_PER], hi[ROW_PER], base[ROW_PER], most = 0;
    double s[ROW_PER];
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r) {
        lo[r] = hi[r] = base[r] = 0;
        s[r] = 0.0;
        if (!mine[r]) continue;
        const int i = r * 256 + (int)threadIdx.x, st = start[row[r]], n = len[row[r]],
                  nL = lights[row[r] + 1] - lights[row[r]];
        const bool light = q[r] < 1.0;
        base[r] = light ? st + nL : st;
        if (light) {
            hi[r] = n - nL;
            s[r] = a[r] > 0 ? v[st + a[r] - 1] : 0.0;
        } else {
            s[r] = v[st + nL + (i - st - a[r])];
            hi[r] = nL > 0 && 0.0 < s[r] ? nL - 1 : 0;
        }
        most = hi[r] > most ? hi[r] : most;
    }
    for (; most > 0; most >>= 1) {
#pragma unroll
        for (int r = 0; r < ROW_PER; ++r) {
            const int mid = (lo[r] + hi[r]) >> 1;
            const double y = v[base[r] + mid];
            const bool open = lo[r] < hi[r], up = q[r] < 1.0 ? y <= s[r] : y < s[r];
            if (open && up) lo[r] = mid + 1;
            else if (open) hi[r] = mid;
        }
    }
    unsigned long long thr[ROW_PER];
    int alias[ROW_PER];
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r) {
        thr[r] = ~0ull;
        alias[r] = r * 256 + (int)threadIdx.x;
        if (!mine[r]) continue;
        const int i = alias[r], st = start[row[r]], n = len[row[r]], nL = lights[row[r] + 1] - lights[row[r]], nH = n - nL;
        if (q[r] < 1.0) {
            if (nH > 0) {
                thr[r] = prob_to_thr(q[r]);
                alias[r] = idx[st + nL + (lo[r] < nH - 1 ? lo[r] : nH - 1)];
            }
        } else {
            const int k = i - st - a[r];
            if (k < nH - 1 && nL > 0 && 0.0 < s[r]) {
                double ov = __dsub_rn(v[st + lo[r]], s[r]);
                if (ov < 0.0) ov = 0.0;
                if (ov > 0.0) {
                    const double p = __dsub_rn(1.0, ov);
                    thr[r] = prob_to_thr(p < 0.0 ? 0.0 : p);
                    alias[r] = idx[st + nL + k + 1];
                }
            }
        }
    }
    int32_t keep[ROW_PER], other[ROW_PER];
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r) {
        const int i = r * 256 + (int)threadIdx.x;
        keep[r] = (int32_t)hs[p0 + (i < here ? i : 0)];
        other[r] = (int32_t)hs[p0 + (i < here ? alias[r] : 0)];
    }
#pragma unroll
    for (int r = 0; r < ROW_PER; ++r)
        if (mine[r]) rec[p0 + r * 256 + threadIdx.x] = WalkRec{thr[r], keep[r], other[r]};
}

// The long rows as a set of tables (table.hpp): a workgroup per slot, so a row has one for each
// chunk of its entries and one more.
struct RowTable : Table {
    const uint32_t *heads;
    WalkRec *rec;

    __device__ __forceinline__ double q(long long i, double Wt) const { return alias_q((double)w[i], N, Wt); }
    template <int RS>
    __device__ __forceinline__ void write(long long first, long long end, const unsigned long long (&thr)[RS],
                                          const uint32_t (&al)[RS]) const
    {
        int32_t keep[RS], other[RS];
#pragma unroll
        for (int r = 0; r < RS; ++r) {
            const long long i = first + r * 64;
            keep[r] = (int32_t)heads[i < end ? i : end - 1];
            other[r] = (int32_t)heads[i < end ? (long long)al[r] : end - 1];
        }
#pragma unroll
        for (int r = 0; r < RS; ++r)
            if (first + r * 64 < end) rec[first + r * 64] = WalkRec{thr[r], keep[r], other[r]};
    }
};

struct LongRows {
    LongRow *rows;
    const uint32_t *huge;
    const uint32_t *slot_row;
    const float *ws;
    const uint32_t *hs;
    WalkRec *rec;
    double *dx;
    uint32_t *idx, *blk;
    double *tot, *mxl, *off, *before;

    __device__ __forceinline__ RowTable whole(unsigned k) const
    {
        const long long lo = rows[k].lo, s = rows[k].slot;
        RowTable t;
        t.N = rows[k].len;
        t.w = ws + lo;
        t.dx = dx + lo;
        t.idx = idx + lo;
        t.blk = blk + s;
        t.tot = tot + s;
        t.mxl = mxl + s;
        t.off = off + s;
        t.before = before + s;
        t.W = &rows[k].W;
        t.heads = hs + lo;
        t.rec = rec + lo;
        return t;
    }
    __device__ __forceinline__ RowTable of(long long &b) const
    {
        const uint32_t k = slot_row[blockIdx.x];
        b = (long long)blockIdx.x - rows[k].slot;
        return whole(k);
    }
};

__global__ void __launch_bounds__(256) k_row_records(LongRows T)
{
    __shared__ RecLds lds;
    long long b;
    const RowTable t = T.of(b);
    const long long left = t.N - b * REC_ITEMS;
    if (left <= 0) return;
    if (left <= 256) records_run<1>(t, b, lds);
    else if (left <= 512) records_run<2>(t, b, lds);
    else if (left <= 768) records_run<3>(t, b, lds);
    else records_run<4>(t, b, lds);
}

// The rows longer than ROW_HUGE alone, for what takes a workgroup a row or half a row.
struct HugeRows {
    LongRows T;
    __device__ __forceinline__ RowTable whole(unsigned k) const { return T.whole(T.huge[k]); }
};

__global__ void __launch_bounds__(LEVEL_THREADS) k_huge_weights(HugeRows T)
{
    __shared__ LevelLds l;
    (void)levels_weight(T.whole(blockIdx.x), l);
}

// Chains of 16 slots' chunks, of whatever rows: most long rows have one or two chunks, so a
// workgroup to a row would run one chain where it can run 16 in the same time.  Chunk j of a row's
// weights is in its slot j; of its deficits too, with the excesses' chunks behind them.
__global__ void __launch_bounds__(256) k_row_chain_weights(LongRows T, long long slots)
{
    __shared__ double lds[CHAIN_LDS];
    __shared__ ChainSegs segs;
    const long long s0 = (long long)blockIdx.x * WAVE_CHUNKS, s = s0 + threadIdx.x;
    if (threadIdx.x < WAVE_CHUNKS) {
        long long at = 0, left = 0;
        if (s < slots) {
            const LongRow &r = T.rows[T.slot_row[s]];
            at = (s - r.slot) * SCAN_CHUNK;
            left = r.len - at;
            at = r.lo + (left > 0 ? at : 0);
        }
        segs.start[threadIdx.x] = at;
        segs.len[threadIdx.x] = left <= 0 ? 0 : left < SCAN_CHUNK ? (int)left : SCAN_CHUNK;
    }
    __syncthreads();
    const float *ws = T.ws;
    double *tot = T.tot;
    block_chains<0, float>(lds, segs, [&](long long i) { return ws[i]; }, [](long long, double) {},
                           [&](int r, double v) { if (segs.len[r]) tot[s0 + r] = v; }, [](int, double) {});
}

__global__ void __launch_bounds__(256, 4) k_row_chain_dx(LongRows T, long long slots)
{
    __shared__ double lds[CHAIN_LDS];
    __shared__ ChainSegs segs;
    const long long s0 = (long long)blockIdx.x * WAVE_CHUNKS, s = s0 + threadIdx.x;
    if (threadIdx.x < WAVE_CHUNKS) {
        long long at = 0, left = 0;
        if (s < slots) {
            const LongRow &r = T.rows[T.slot_row[s]];
            const long long nL = T.blk[r.slot + LH_CDIV(r.len, SPLIT_ITEMS)], cL = LH_CDIV(nL, SCAN_CHUNK), j = s - r.slot;
            const long long first = j < cL ? j * SCAN_CHUNK : nL + (j - cL) * SCAN_CHUNK;
            left = (j < cL ? nL : r.len) - first;
            at = r.lo + (left > 0 ? first : 0);
        }
        segs.start[threadIdx.x] = at;
        segs.len[threadIdx.x] = left <= 0 ? 0 : left < SCAN_CHUNK ? (int)left : SCAN_CHUNK;
    }
    __syncthreads();
    double *x = T.dx, *tot = T.tot, *mxl = T.mxl;
    block_chains<2, double>(lds, segs, [&](long long i) { return x[i]; }, [&](long long i, double v) { x[i] = v; },
                            [&](int r, double v) { if (segs.len[r]) tot[s0 + r] = v; },
                            [&](int r, double v) { if (segs.len[r]) mxl[s0 + r] = v; });
}

// What levels_weight, k_split_scan and k_levels_dx do, for rows of at most 64 chunks: a wavefront
// a row or half a row, lane l has chunk l.
__device__ __forceinline__ double lane_chain(double x, int n)
{
    OpNeumaier::State st = OpNeumaier::init();
    double mine = 0.0;
    for (int i = 0; i < n; ++i) {
        const double v = OpNeumaier::step(st, __shfl(x, i));
        if ((int)(threadIdx.x & 63) == i) mine = v;
    }
    return mine;
}

__global__ void __launch_bounds__(256) k_row_weights(LongRows T, unsigned rows)
{
    const unsigned k = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (k >= rows || T.rows[k].len > ROW_HUGE) return;
    const RowTable t = T.whole(k);
    const int nch = (int)LH_CDIV(t.N, SCAN_CHUNK);
    const double x = lane < nch ? t.tot[lane] : 0.0;
    const double before = __shfl(lane_chain(x, nch - 1), nch > 1 ? nch - 2 : 0), last = __shfl(x, nch - 1);
    if (lane == 0) *t.W = nch > 1 ? OpNeumaier::combine(before, last) : last;
}

__global__ void __launch_bounds__(256) k_row_split_scan(LongRows T, unsigned rows)
{
    const unsigned k = blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (k >= rows || T.rows[k].len > ROW_HUGE) return;
    const RowTable t = T.whole(k);
    const int nt = (int)LH_CDIV(t.N, SPLIT_ITEMS);
    const uint32_t c = lane < nt ? t.blk[lane] : 0u;
    uint32_t inc = c;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d);
        if (lane >= d) inc += y;
    }
    if (lane < nt) t.blk[lane] = inc - c;
    if (lane == 63) t.blk[nt] = inc;
}

__global__ void __launch_bounds__(256) k_row_levels_dx(LongRows T, unsigned rows)
{
    const unsigned g = blockIdx.x * 4 + (threadIdx.x >> 6), k = g >> 1;
    const int lane = threadIdx.x & 63;
    if (k >= rows || T.rows[k].len > ROW_HUGE) return;
    const RowTable t = T.whole(k);
    const bool heavy = (g & 1u) != 0;
    const long long nL = t.lights(), c0 = heavy ? LH_CDIV(nL, SCAN_CHUNK) : 0;
    const int nch = (int)LH_CDIV(heavy ? t.N - nL : nL, SCAN_CHUNK);
    if (nch == 0) return;
    const double x = lane < nch ? t.tot[c0 + lane] : 0.0, none = -__builtin_huge_val();
    double off = __shfl_up(lane_chain(x, nch - 1), 1);
    if (lane == 0) off = 0.0;
    double m = lane < nch ? off + t.mxl[c0 + lane] : none;
    for (int d = 1; d < 64; d <<= 1) {
        const double y = __shfl_up(m, d);
        if (lane >= d) m = __builtin_fmax(m, y);
    }
    double before = __shfl_up(m, 1);
    if (lane == 0) before = none;
    if (lane >= nch) return;
    t.off[c0 + lane] = off;
    t.before[c0 + lane] = before;
    t.mxl[c0 + lane] = m;
}

// ---------------------------------------------------------------------------
// Walks: one thread per walk of a chunk.
// ---------------------------------------------------------------------------
__global__ void __launch_bounds__(256) k_walk(const EdgeRec *erec, long long m, const long long *off,
                                              const WalkRec *rec, unsigned long long seed, unsigned long long key1,
                                              int L, int W, long long Bw, long long P, unsigned long long k0,
                                              long long nwalks, int2 *pairs)
{
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= nwalks) return;
    const unsigned long long k = k0 + (unsigned long long)t;
    int2 *out = pairs + (t / Bw) * Bw * P + (t % Bw);
    const u64x4 x0 = philox4x64_10(seed, key1, k, 0ull, 0ull, 0ull);
    uint4 r0, r1;
    load_edge_rec(erec, draw_column(x0.x, m), r0, r1);
    int u = 0, v = 0;
    (void)edge_pick(r0, r1, x0.y, u, v);
    // ring of the last W - 1 vertices: ring[pos % (W - 1)] holds w_pos
    int ring[kWalkMaxWindow - 1];
    ring[0] = u;
    out[0] = make_int2(u, v);  // pair (w_0, w_1): delta 1, i 0
    int cur = v;
    if (W > 2) ring[1 % (W - 1)] = v;
    for (int pos = 2; pos < L; ++pos) {
        const u64x4 x = philox4x64_10(seed, key1, k, (unsigned long long)(pos - 1), 0ull, 0ull);
        const long long lo = off[cur], len = off[cur + 1] - lo;
        int nxt = cur;  // a row without entries is never reached (every step leaves along an entry)
        if (len > 0) {
            const WalkRec r = rec[lo + draw_column(x.x, len)];
            nxt = x.y < r.thr ? r.keep : r.alias;
        }
        // pairs (w_{pos - delta}, w_pos), delta = 1 .. min(W - 1, pos)
        long long pbase = 0;
        for (int dl = 1; dl < W && dl <= pos; ++dl) {
            const int prev = dl == 1 ? cur : ring[(pos - dl) % (W - 1)];
            out[(pbase + pos - dl) * Bw] = make_int2(prev, nxt);
            pbase += L - dl;
        }
        if (W > 2) ring[pos % (W - 1)] = nxt;
        cur = nxt;
    }
}

__global__ void k_pairs_out(const int2 *pairs, long long from, long long count, int32_t *u, int32_t *v)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    const int2 p = pairs[from + i];
    u[i] = p.x;
    v[i] = p.y;
}

__global__ void k_walk_export(const WalkRec *rec, long long E, unsigned long long *thr, int32_t *keep, int32_t *alias)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= E) return;
    const WalkRec r = rec[i];
    thr[i] = r.thr;
    keep[i] = r.keep;
    alias[i] = r.alias;
}

// ---------------------------------------------------------------------------
// Host side.
// ---------------------------------------------------------------------------
static lh_status walk_args_ok(long long n, long long m, int L, int W, long long Bw)
{
    if (n < 1 || m < 1 || 2 * m >= (1ll << 32) || n >= (1ll << 31)) return LH_ERR_INVALID_ARG;
    if (L < 2 || L > kWalkMaxLength || W < 2 || W > kWalkMaxWindow || W > L) return LH_ERR_INVALID_ARG;
    if (Bw < 1 || Bw > (1ll << 24)) return LH_ERR_INVALID_ARG;
    long long P = 0;
    for (int dl = 1; dl < W; ++dl) P += L - dl;
    if (Bw * P > (1ll << 27)) return LH_ERR_INVALID_ARG;
    return LH_OK;
}

static lh_status build_walk(lh_handle *h, char *persist, char *scratch, const WalkLayout &WL, const WalkScratch &S)
{
    hipStream_t st = h->stream;
    const long long n = h->n, m = h->m, E = 2 * m;
    WalkState &w = h->walk;
    w.off = (long long *)(persist + WL.off);
    w.rec = (WalkRec *)(persist + WL.rec);
    w.pairs = (int2 *)(persist + WL.pairs);
    const auto words = [&](size_t at) { return (uint32_t *)(scratch + at); };
    const SortBuffers b0{words(S.k0), words(S.w0), words(S.h0)}, b1{words(S.k1), words(S.w1), words(S.h1)};
    int bits = 1;
    while (bits < 31 && (1ll << bits) < n) ++bits;
    const SortBuffers rows = radix_sort(WalkEntries{h->src, h->dst, h->w, (unsigned long long)m}, E, bits, b0, b1,
                                        words(S.hist), words(S.part), st);
    const SortBuffers rest = rows.k == b0.k ? b1 : b0;
    const uint32_t *ks = rows.k, *hs = rows.p1;
    const float *ws = (const float *)rows.p0;
    unsigned long long *cnt = (unsigned long long *)(scratch + S.cnt);
    LongRows T;
    T.rows = (LongRow *)(scratch + S.rows);
    T.huge = words(S.huge);
    T.slot_row = words(S.slot_row);
    T.ws = ws;
    T.hs = hs;
    T.rec = w.rec;
    T.dx = (double *)(scratch + S.dx);
    T.idx = rest.k;  // (the sort is done)
    T.blk = words(S.blk);
    T.tot = (double *)(scratch + S.tot);
    T.mxl = (double *)(scratch + S.mxl);
    T.off = (double *)(scratch + S.off);
    T.before = (double *)(scratch + S.before);

    hipLaunchKernelGGL(k_row_offsets, dim3((unsigned)LH_CDIV(E, 1024)), dim3(256), 0, st, ks, E, n, w.off, cnt);
    hipLaunchKernelGGL(k_rows, dim3((unsigned)LH_CDIV(E, ROW_TILE)), dim3(256), 0, st, ks, ws, hs, w.off, E, w.rec, T.rows,
                       words(S.huge), words(S.slot_row), cnt);
    unsigned long long listed[3];  // long rows, their slots, huge rows
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(listed, cnt, sizeof(listed), hipMemcpyDeviceToHost, st);
    if (e == hipSuccess) e = hipStreamSynchronize(st);
    if (e != hipSuccess) return hip_fail(h, e, "walk rows");
    if (listed[0] == 0) return LH_OK;
    const unsigned nr = (unsigned)listed[0], nh = (unsigned)listed[2];
    const long long slots = (long long)listed[1];
    const HugeRows H{T};
    const dim3 gs((unsigned)slots), gc((unsigned)LH_CDIV(slots, WAVE_CHUNKS)), gr((unsigned)LH_CDIV(nr, 4)), blk(256);
    hipLaunchKernelGGL(k_row_chain_weights, gc, blk, 0, st, T, slots);
    hipLaunchKernelGGL(k_row_weights, gr, blk, 0, st, T, nr);
    if (nh) hipLaunchKernelGGL(k_huge_weights, dim3(nh), blk, 0, st, H);
    hipLaunchKernelGGL(k_split_count<LongRows>, gs, blk, 0, st, T);
    hipLaunchKernelGGL(k_row_split_scan, gr, blk, 0, st, T, nr);
    if (nh) hipLaunchKernelGGL(k_split_scan<HugeRows>, dim3(nh), dim3(1024), 0, st, H);
    hipLaunchKernelGGL(k_split<LongRows>, gs, blk, 0, st, T);
    hipLaunchKernelGGL(k_row_chain_dx, gc, blk, 0, st, T, slots);
    hipLaunchKernelGGL(k_row_levels_dx, dim3((unsigned)LH_CDIV(nr, 2)), blk, 0, st, T, nr);
    if (nh) hipLaunchKernelGGL(k_levels_dx<HugeRows>, dim3(2 * nh), blk, 0, st, H);
    hipLaunchKernelGGL(k_row_records, gs, blk, 0, st, T);
    e = hipStreamSynchronize(st);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(h, e, "walk rows");
    return LH_OK;
}

static hipError_t generate_chunk(lh_handle *h, long long chunk)
{
    const WalkState &w = h->walk;
    const unsigned long long k0 = (unsigned long long)chunk * (unsigned long long)w.chunk_walks;
    const unsigned long long key1 = (kWalkTag << 32) | (unsigned long long)(uint32_t)h->p.graph_id;
    hipLaunchKernelGGL(k_walk, dim3((unsigned)LH_CDIV(w.chunk_walks, 256)), dim3(256), 0, h->stream, h->erec, h->m,
                       w.off, w.rec, h->p.seed, key1, w.L, w.W, w.Bw, w.P, k0, w.chunk_walks, w.pairs);
    return hipGetLastError();
}

lh_status walk_each_chunk(lh_handle *h, unsigned long long first, unsigned long long count,
                          const std::function<lh_status(unsigned long long, unsigned long long, const int2 *,
                                                        unsigned long long)> &body)
{
    WalkState &w = h->walk;
    if (w.pool > 0) {
        // Pair pool: the collected pairs are chunk 0's first R; every sample draws from them.
        if (w.loaded != 0) {
            w.loaded = -1;
            hipError_t e = generate_chunk(h, 0);
            if (e != hipSuccess) return hip_fail(h, e, "walk generation");
            w.loaded = 0;
        }
        return count > 0 ? body(first, count, w.pairs, 0) : LH_OK;
    }
    const unsigned long long cs = (unsigned long long)w.chunk_walks * (unsigned long long)w.P;
    const unsigned long long end = first + count;
    for (unsigned long long s = first; s < end;) {
        const unsigned long long c = s / cs, c0 = c * cs;
        const unsigned long long stop = std::min(end, c0 + cs);
        if (w.loaded != (long long)c) {
            w.loaded = -1;
            hipError_t e = generate_chunk(h, (long long)c);
            if (e != hipSuccess) return hip_fail(h, e, "walk generation");
            w.loaded = (long long)c;
        }
        lh_status st = body(s, stop - s, w.pairs, c0);
        if (st != LH_OK) return st;
        s = stop;
    }
    return LH_OK;
}

}  // namespace lh

using namespace lh;

extern "C" {

lh_status lh_walk_size(int64_t n, int64_t m, int32_t walk_length, int32_t window, int64_t walks_per_batch,
                       size_t *persist, size_t *scratch)
{
    if (!persist || !scratch) return LH_ERR_INVALID_ARG;
    lh_status st = walk_args_ok(n, m, walk_length, window, walks_per_batch);
    if (st != LH_OK) return st;
    *persist = walk_layout(n, m, walk_length, window, walks_per_batch).total;
    *scratch = walk_scratch_layout(n, m).total;
    return LH_OK;
}

lh_status lh_walk_build(lh_handle *h, int32_t walk_length, int32_t window, int64_t walks_per_batch, void *persist,
                        size_t persist_bytes, void *scratch, size_t scratch_bytes)
{
    if (!h) return LH_ERR_INVALID_ARG;
    if (!h->graph_set || !h->edge_ready) return fail(h, LH_ERR_NOT_BUILT, "lh_set_graph and lh_build_alias first");
    if (walk_args_ok(h->n, h->m, walk_length, window, walks_per_batch) != LH_OK)
        return fail(h, LH_ERR_INVALID_ARG, "walk length, window or walks per batch out of range");
    if (!persist || ((uintptr_t)persist & 255u) || !scratch || ((uintptr_t)scratch & 255u))
        return fail(h, LH_ERR_INVALID_ARG, "walk memory must be 256-byte aligned device memory");
    const WalkLayout WL = walk_layout(h->n, h->m, walk_length, window, walks_per_batch);
    const WalkScratch S = walk_scratch_layout(h->n, h->m);
    if (persist_bytes < WL.total || scratch_bytes < S.total)
        return fail(h, LH_ERR_WORKSPACE_TOO_SMALL, "walk memory smaller than lh_walk_size");
    if (h->p.mode == LH_SNAPSHOT && ((unsigned long long)walks_per_batch * (unsigned long long)WL.P) %
                                            (unsigned long long)h->p.batch != 0)
        return fail(h, LH_ERR_INVALID_ARG, "SNAPSHOT with walk pairs needs the batch to divide a walk batch's pairs");
    int prev = -1;
    (void)hipGetDevice(&prev);
    if (prev != h->device) (void)hipSetDevice(h->device);
    WalkState &w = h->walk;
    w = WalkState();
    w.L = walk_length;
    w.W = window;
    w.Bw = walks_per_batch;
    w.P = WL.P;
    w.chunk_walks = WL.chunk_walks;
    lh_status st = build_walk(h, (char *)persist, (char *)scratch, WL, S);
    w.ready = st == LH_OK;
    w.loaded = -1;
    if (prev >= 0 && prev != h->device) (void)hipSetDevice(prev);
    return st;
}

lh_status lh_walk_detach(lh_handle *h)
{
    if (!h) return LH_ERR_INVALID_ARG;
    h->walk = WalkState();
    return LH_OK;
}

lh_status lh_walk_pool_size(uint64_t total_samples, uint64_t *pairs)
{
    if (!pairs || total_samples == 0) return LH_ERR_INVALID_ARG;
    // least R >= 2 with R (R - 1) / 2 >= T: start from the binary64 root and correct it
    unsigned long long R = (unsigned long long)std::ceil(0.5 * (1.0 + std::sqrt(1.0 + 8.0 * (double)total_samples)));
    if (R < 2) R = 2;
    auto tri = [](unsigned long long r) { return (unsigned __int128)r * (unsigned __int128)(r - 1) / 2; };
    while (R > 2 && tri(R - 1) >= (unsigned __int128)total_samples) --R;
    while (tri(R) < (unsigned __int128)total_samples) ++R;
    *pairs = R;
    return LH_OK;
}

lh_status lh_walk_pool(lh_handle *h, uint64_t pairs)
{
    if (!h) return LH_ERR_INVALID_ARG;
    if (!h->walk.ready) return fail(h, LH_ERR_NOT_BUILT, "lh_walk_build first");
    WalkState &w = h->walk;
    const unsigned long long cap = (unsigned long long)w.chunk_walks * (unsigned long long)w.P;
    if (pairs > cap) return fail(h, LH_ERR_OUT_OF_RANGE, "pool larger than the walk pair buffer");
    w.pool = pairs;
    if (pairs == 0) return LH_OK;
    int prev = -1;
    (void)hipGetDevice(&prev);
    if (prev != h->device) (void)hipSetDevice(h->device);
    lh_status st = LH_OK;
    if (w.loaded != 0) {
        w.loaded = -1;
        hipError_t e = generate_chunk(h, 0);
        if (e != hipSuccess) {
            w.pool = 0;
            st = hip_fail(h, e, "walk generation");
        } else {
            w.loaded = 0;
        }
    }
    if (prev >= 0 && prev != h->device) (void)hipSetDevice(prev);
    return st;
}

lh_status lh_walk_pairs(lh_handle *h, uint64_t first, uint64_t count, int32_t *u, int32_t *v)
{
    if (!h) return LH_ERR_INVALID_ARG;
    if (!h->walk.ready) return fail(h, LH_ERR_NOT_BUILT, "lh_walk_build first");
    if (h->walk.pool > 0) return fail(h, LH_ERR_UNSUPPORTED, "a pair pool is on: lh_sample gives its pairs");
    if (count > 0 && (!u || !v)) return fail(h, LH_ERR_INVALID_ARG, "NULL output");
    if (first + count < first || count >= (1ull << 40)) return fail(h, LH_ERR_INVALID_ARG, "sample range out of range");
    int prev = -1;
    (void)hipGetDevice(&prev);
    if (prev != h->device) (void)hipSetDevice(h->device);
    lh_status st = walk_each_chunk(h, first, count,
                                   [&](unsigned long long sf, unsigned long long sc, const int2 *pairs,
                                       unsigned long long pf) -> lh_status {
                                       const unsigned long long o = sf - first;
                                       hipLaunchKernelGGL(k_pairs_out, dim3((unsigned)LH_CDIV(sc, 256)), dim3(256), 0,
                                                          h->stream, pairs, (long long)(sf - pf), (long long)sc, u + o,
                                                          v + o);
                                       hipError_t e = hipGetLastError();
                                       return e == hipSuccess ? LH_OK : hip_fail(h, e, "walk pairs");
                                   });
    if (prev >= 0 && prev != h->device) (void)hipSetDevice(prev);
    return st;
}

lh_status lh_walk_export(lh_handle *h, int64_t *offsets, uint64_t *thr, int32_t *keep, int32_t *alias)
{
    if (!h) return LH_ERR_INVALID_ARG;
    if (!h->walk.ready) return fail(h, LH_ERR_NOT_BUILT, "lh_walk_build first");
    if (!offsets || !thr || !keep || !alias) return fail(h, LH_ERR_INVALID_ARG, "NULL output");
    int prev = -1;
    (void)hipGetDevice(&prev);
    if (prev != h->device) (void)hipSetDevice(h->device);
    const long long E = 2 * h->m;
    hipError_t e = hipMemcpyAsync(offsets, h->walk.off, 8 * (size_t)(h->n + 1), hipMemcpyDeviceToDevice, h->stream);
    if (e == hipSuccess) {
        hipLaunchKernelGGL(k_walk_export, dim3((unsigned)LH_CDIV(E, 256)), dim3(256), 0, h->stream, h->walk.rec, E,
                           (unsigned long long *)thr, keep, alias);
        e = hipStreamSynchronize(h->stream);
    }
    if (e == hipSuccess) e = hipGetLastError();
    if (prev >= 0 && prev != h->device) (void)hipSetDevice(prev);
    return e == hipSuccess ? LH_OK : hip_fail(h, e, "walk export");
}

}  // extern "C"
