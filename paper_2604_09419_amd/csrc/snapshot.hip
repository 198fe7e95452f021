// SNAPSHOT mode: a deterministic form of the batch update of Eq. (4).
//
// For batch [b0, b1) every sample's increments are computed from the tables as they
// were at b0 and written out as entries (key = table * n + row, a d-vector).  A stable radix
// sort on the keys (equal keys keep the order in which they were emitted: by sample, then
// order, then slot) groups the entries of each row.  A row's entries are summed in that order, 16
// (rows over 256 elements: 8) at a time by a fixed binary32 tree and these parts in binary64, and
// the sum is added to the row and rounded once: a hub has thousands of entries, and a binary32
// chain of them loses digits that the row has (2.3e-5 of it after 35,000) and is a latency each.
// No atomics touch the numbers, so the result is the same on every run.
//
// What bounds it: a large batch writes and reads its entries once besides reading the rows (65,536
// samples at d = 128, both orders: 0.47 GB each way); a small one its launches and the chain of
// the row with the most entries.  2^20 nodes, d = 128, both orders, four batches of 65,536: 1.64
// ms; with a row's entries followed a load at a time (a hub's 700 took 0.9 ms), 4-bit sort passes
// and the increments computed by 1,024 wavefronts, 64 samples each, 4.74 ms.  10,000 nodes,
// d = 16, bfloat16, sixteen batches of 4,096: 0.63 against 3.04 ms.
#include "handle.hpp"
#include "sort.hpp"
#include "tile.hpp"

namespace lh {

namespace {

// Tables of order oi of a sample: both orders, the second first; else the one there is.
__device__ __forceinline__ void order_tables(int orders, int oi, int &tabA, int &tabB)
{
    const bool first = orders == LH_ORDER1 || oi == 1;
    tabA = first ? LH_TABLE_U1 : LH_TABLE_U;
    tabB = first ? LH_TABLE_U1 : LH_TABLE_C;
}

// V consecutive elements of a row as binary32, from a 4 V-byte (bfloat16: 2 V) boundary.
template <typename TT, int V>
__device__ __forceinline__ void load_elems(const TT *p, float (&x)[V])
{
    if constexpr (sizeof(TT) == 4) {
#pragma unroll
        for (int q = 0; q < V / 4; ++q) {
            const float4 y = reinterpret_cast<const float4 *>(p)[q];
            x[4 * q] = y.x, x[4 * q + 1] = y.y, x[4 * q + 2] = y.z, x[4 * q + 3] = y.w;
        }
    } else {
#pragma unroll
        for (int q = 0; q < V / 4; ++q) {
            const uint2 y = reinterpret_cast<const uint2 *>(p)[q];
            x[4 * q] = val<TT>(y.x, 0), x[4 * q + 1] = val<TT>(y.x, 1);
            x[4 * q + 2] = val<TT>(y.y, 0), x[4 * q + 3] = val<TT>(y.y, 1);
        }
    }
}

}  // namespace

// The batch's tuples as the entries' keys: a thread per sample and slot (slot 0 draws the pair,
// its vertex row and its context row), so that the Philox blocks of a sample run side by side.
__global__ void __launch_bounds__(256) k_snap_draw(GraphDev g, int orders, unsigned long long first,
                                                   unsigned long long count, uint32_t *keys)
{
    const unsigned long long t = (unsigned long long)blockIdx.x * blockDim.x + threadIdx.x;
    const unsigned K1 = (unsigned)g.K + 1u;
    if (t >= count * K1) return;
    const unsigned long long i = t / K1;
    const int j = (int)(t - i * K1);
    const unsigned long long s = first + i;
    int a = 0, b = 0;
    if (j == 0) {
        const SlotDraw de = draw_slot(g, s, 0, slot0_columns(g));
        uint4 r0, r1;
        load_pair_rec(g, s, de.col, de.x1, r0, r1);
        (void)edge_pick(r0, r1, de.x1, a, b);
    } else {
        const SlotDraw dn = draw_slot(g, s, j, g.n);
        const uint4 nr = *reinterpret_cast<const uint4 *>(g.nrec + dn.col);
        (void)neg_pick(nr, dn, b);
    }
    const int nord = orders == LH_ORDER12 ? 2 : 1;
    for (int oi = 0; oi < nord; ++oi) {
        int tabA, tabB;
        order_tables(orders, oi, tabA, tabB);
        uint32_t *k = keys + (i * nord + oi) * (unsigned long long)(g.K + 2);
        if (j == 0) k[0] = (uint32_t)((long long)tabA * g.n + a);
        k[1 + j] = (uint32_t)((long long)tabB * g.n + b);
    }
}

// The increments of one sample and order, by G lanes of V elements each: slot 0 the vertex row's,
// slots 1 .. K + 1 the context rows'.  One group per sample and order (the batch of 65,536 samples:
// 131,072 groups of 32 lanes), all of a group's rows loaded before any arithmetic.
template <typename TT, int G, int V, int KMAX>
__global__ void __launch_bounds__(256) k_snap_contrib(GraphDev g, int orders, unsigned long long first,
                                                      unsigned long long count, const uint32_t *keys, float *contrib)
{
    const int nord = orders == LH_ORDER12 ? 2 : 1, gl = threadIdx.x % G, K = g.K, d = g.d, c = gl * V;
    const unsigned long long q = (unsigned long long)blockIdx.x * (256 / G) + threadIdx.x / G;
    if (q >= count * nord) return;
    int tabA, tabB;
    order_tables(orders, nord == 2 ? (int)(q & 1) : 0, tabA, tabB);
    const unsigned long long i = nord == 2 ? q >> 1 : q, e0 = q * (unsigned long long)(K + 2);
    const bool in = c < d;
    float a[V], b[KMAX + 1][V];
    uint32_t row[KMAX + 2];
#pragma unroll
    for (int j = 0; j <= KMAX + 1; ++j) row[j] = j <= K + 1 ? keys[e0 + j] : 0u;
#pragma unroll
    for (int j = 0; j <= KMAX + 1; ++j) {
        float(&x)[V] = j == 0 ? a : b[j > 0 ? j - 1 : 0];
#pragma unroll
        for (int k = 0; k < V; ++k) x[k] = 0.f;
        if (j <= K + 1 && in) {
            const int t = j == 0 ? tabA : tabB;
            load_elems<TT, V>((const TT *)g.tab[t] + ((long long)row[j] - (long long)t * g.n) * d + c, x);
        }
    }
    float gj[KMAX + 1];
#pragma unroll
    for (int j = 0; j <= KMAX; ++j) {
        float x = 0.f;
#pragma unroll
        for (int k = 0; k < V; ++k) x = fmaf(a[k], b[j][k], x);
        gj[j] = x;
    }
#pragma unroll
    for (int j = 0; j <= KMAX; ++j) gj[j] = group_sum<G>(gj[j]);
    const unsigned long long s = first + i;
    const float eta = (float)(g.eta0 * (1.0 - (double)s / (double)g.T));
    const float el = eta * g.lambda, decayA = (float)(K + 1) * el;
#pragma unroll
    for (int j = 0; j <= KMAX; ++j) {
        const float sg = __builtin_amdgcn_rcpf(1.0f + __expf(-gj[j]));
        const float gg = j == 0 ? eta * (1.0f - sg) : -eta * g.alpha * sg;
        gj[j] = j <= K ? gg : 0.f;
    }
    if (!in) return;
    float *out = contrib + e0 * (unsigned long long)d + c;
#pragma unroll
    for (int k0 = 0; k0 < V; k0 += 4) {
        float y[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            y[k] = -decayA * a[k0 + k];
#pragma unroll
            for (int j = 0; j <= KMAX; ++j) y[k] = fmaf(gj[j], b[j][k0 + k], y[k]);
        }
        *reinterpret_cast<float4 *>(out + k0) = make_float4(y[0], y[1], y[2], y[3]);
    }
#pragma unroll
    for (int j = 0; j <= KMAX; ++j) {
        if (j <= K) {
            float *o = out + (unsigned long long)(j + 1) * d;
#pragma unroll
            for (int k0 = 0; k0 < V; k0 += 4) {
                float y[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) y[k] = gj[j] * a[k0 + k] - el * b[j][k0 + k];
                *reinterpret_cast<float4 *>(o + k0) = make_float4(y[0], y[1], y[2], y[3]);
            }
        }
    }
}

// Each touched row: its entries summed in order, added once.  A wavefront looks at 64 consecutive
// sorted entries and takes the rows that begin among them, a group of G lanes each (the row at the
// end may run on past the 64).  A group has 16 entries in flight (V = 8: 8) and their indices the
// step before.
template <typename TT, int G, int V>
__global__ void __launch_bounds__(256) k_snap_apply(GraphDev g, const uint32_t *keys, const uint32_t *vals, long long E,
                                                    const float *contrib, unsigned long long batch_idx)
{
    constexpr int GROUPS = 64 / G, STEP = V == 4 ? 16 : 8;
    const int lane = threadIdx.x & 63, grp = lane / G, gl = lane % G, c = gl * V;
    const long long w0 = ((long long)blockIdx.x * 4 + (threadIdx.x >> 6)) * 64, p = w0 + lane;
    if (w0 >= E) return;
    const uint32_t key = keys[p < E ? p : E - 1];
    const uint32_t prev = p > 0 ? keys[(p < E ? p : E) - 1] : ~key;
    unsigned long long heads = __ballot(p < E && key != prev);
    if (!heads) return;
    // where the last row of the 64 ends
    const int last = 63 - __clzll((long long)heads);
    const uint32_t lastkey = (uint32_t)__builtin_amdgcn_readlane((int)key, last);
    long long end = E < w0 + 64 ? E : w0 + 64;
    while (end < E) {
        unsigned long long off[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const long long x = end + k * 64 + lane;
            off[k] = __ballot(x >= E || keys[x < E ? x : E - 1] != lastkey);
        }
        int run = 256;
#pragma unroll
        for (int k = 3; k >= 0; --k)
            if (off[k]) run = k * 64 + __ffsll((long long)off[k]) - 1;
        end += run;
        if (run < 256) break;
    }
    const int d = g.d;
    const bool in = c < d;
    while (heads) {
        // the next GROUPS rows: this group's first entry, and the entry after its last
        long long p0 = -1, p1 = 0;
#pragma unroll 1
        for (int k = 0; k < GROUPS && heads; ++k) {
            const int at = __ffsll((long long)heads) - 1;
            heads &= heads - 1;
            if (k == grp) {
                p0 = w0 + at;
                p1 = heads ? w0 + __ffsll((long long)heads) - 1 : end;
            }
        }
        if (p0 < 0 || !in) continue;
        const uint32_t rk = keys[p0];
        double acc[V];
#pragma unroll
        for (int k = 0; k < V; ++k) acc[k] = 0.0;
        uint32_t idx[STEP];
#pragma unroll
        for (int k = 0; k < STEP; ++k) idx[k] = vals[p0 + k < p1 ? p0 + k : p1 - 1];
        for (long long q = p0; q < p1; q += STEP) {
            float x[STEP][V];
#pragma unroll
            for (int k = 0; k < STEP; ++k) {
                if (k == 0 || q + k < p1) {  // (uniform over the group)
                    load_elems<float, V>(contrib + (unsigned long long)idx[k] * d + c, x[k]);
                } else {
#pragma unroll
                    for (int v = 0; v < V; ++v) x[k][v] = 0.f;
                }
            }
#pragma unroll
            for (int k = 0; k < STEP; ++k) idx[k] = vals[q + STEP + k < p1 ? q + STEP + k : p1 - 1];
#pragma unroll
            for (int w = STEP / 2; w >= 1; w /= 2)
#pragma unroll
                for (int k = 0; k < w; ++k)
#pragma unroll
                    for (int v = 0; v < V; ++v) x[k][v] += x[k + w][v];
#pragma unroll
            for (int v = 0; v < V; ++v) acc[v] += (double)x[0][v];
        }
        const int table = (int)(rk / (uint32_t)g.n);
        const long long row = (long long)(rk % (uint32_t)g.n);
        TT *X = (TT *)g.tab[table] + row * d + c;
        float x[V];
        load_elems<TT, V>(X, x);
#pragma unroll
        for (int v = 0; v < V; ++v) x[v] = (float)((double)x[v] + acc[v]);
        if constexpr (sizeof(TT) == 4) {
#pragma unroll
            for (int k0 = 0; k0 < V; k0 += 4)
                *reinterpret_cast<float4 *>(X + k0) = make_float4(x[k0], x[k0 + 1], x[k0 + 2], x[k0 + 3]);
        } else {
            // Stochastic rounding bits: Philox4x64-10 keyed by (batch, table, row); block un / 8
            // holds 32 bits for each of 8 units (un: the unit's number in the row).
            const int un = c / 2;
            const u64x4 r = philox4x64_10(g.seed, g.sr_key, batch_idx, (unsigned long long)table, (unsigned long long)row,
                                          (unsigned long long)(un / 8));
            const unsigned long long w[4] = {r.x, r.y, r.z, r.w};
#pragma unroll
            for (int k0 = 0; k0 < V; k0 += 4) {
                const int z = ((un + k0 / 2) % 8) / 2;
                const unsigned long long wd = z == 0 ? w[0] : z == 1 ? w[1] : z == 2 ? w[2] : w[3];
                uint2 y;
                y.x = bf16x2_sr(x[k0], x[k0 + 1], (uint32_t)wd);
                y.y = bf16x2_sr(x[k0 + 2], x[k0 + 3], (uint32_t)(wd >> 32));
                *reinterpret_cast<uint2 *>(X + k0) = y;
            }
        }
    }
}

namespace {

struct SnapBatch {
    int orders;
    unsigned long long first, count, index;
    long long entries;
    const uint32_t *drawn, *keys, *vals;  // the tuples' keys in order of emission, and sorted
    float *contrib;
};

template <typename TT, int G, int V>
void launch_contrib(const GraphDev &g, const SnapBatch &b, hipStream_t s)
{
    const unsigned long long groups = b.count * (b.orders == LH_ORDER12 ? 2 : 1);
    const dim3 grid((unsigned)LH_CDIV(groups, 256 / G)), blk(256);
    if (g.K <= 5)
        hipLaunchKernelGGL((k_snap_contrib<TT, G, V, 5>), grid, blk, 0, s, g, b.orders, b.first, b.count, b.drawn, b.contrib);
    else
        hipLaunchKernelGGL((k_snap_contrib<TT, G, V, 8>), grid, blk, 0, s, g, b.orders, b.first, b.count, b.drawn, b.contrib);
}

template <typename TT, int G, int V>
void launch_apply(const GraphDev &g, const SnapBatch &b, hipStream_t s)
{
    hipLaunchKernelGGL((k_snap_apply<TT, G, V>), dim3((unsigned)LH_CDIV(b.entries, 256)), dim3(256), 0, s, g, b.keys,
                       b.vals, b.entries, b.contrib, b.index);
}

// Lanes and elements per lane by width: four elements (16 bytes of an entry) over up to 64 lanes.
#define LH_SNAP_WIDTH(fn, TT)                                     \
    if (g.d <= 8) fn<TT, 2, 4>(g, b, s);                  \
    else if (g.d <= 16) fn<TT, 4, 4>(g, b, s);            \
    else if (g.d <= 32) fn<TT, 8, 4>(g, b, s);            \
    else if (g.d <= 64) fn<TT, 16, 4>(g, b, s);           \
    else if (g.d <= 128) fn<TT, 32, 4>(g, b, s);          \
    else if (g.d <= 256) fn<TT, 64, 4>(g, b, s);          \
    else fn<TT, 64, 8>(g, b, s);

void contrib(const GraphDev &g, int dtype, const SnapBatch &b, hipStream_t s)
{
    if (dtype == LH_FP32) {
        LH_SNAP_WIDTH(launch_contrib, float)
    } else {
        LH_SNAP_WIDTH(launch_contrib, uint16_t)
    }
}

void apply(const GraphDev &g, int dtype, const SnapBatch &b, hipStream_t s)
{
    if (dtype == LH_FP32) {
        LH_SNAP_WIDTH(launch_apply, float)
    } else {
        LH_SNAP_WIDTH(launch_apply, uint16_t)
    }
}
#undef LH_SNAP_WIDTH

}  // namespace

lh_status train_snapshot(lh_handle *h, unsigned long long first, unsigned long long count, const int2 *pairs,
                         unsigned long long pairs_first)
{
    const lh_params &p = h->p;
    const WsLayout &L = h->lay;
    GraphDev g = graph_dev(h);
    g.pairs = pairs;
    g.pairs_first = pairs_first;
    g.pool_n = pairs ? h->walk.pool : 0;
    hipStream_t s = h->stream;
    const unsigned long long B = (unsigned long long)p.batch;
    const unsigned long long per = (unsigned long long)(p.orders == LH_ORDER12 ? 2 : 1) * (unsigned long long)(p.K + 2);
    // The drawn keys stay as they are (the contributions read them); the sort's first pass goes
    // to the second buffers and the others between those and the first values' neighbour.
    uint32_t *drawn = (uint32_t *)(h->ws + L.keys0);
    const SortBuffers one{(uint32_t *)(h->ws + L.keys1), (uint32_t *)(h->ws + L.vals1), nullptr};
    const SortBuffers two{(uint32_t *)(h->ws + L.keys2), (uint32_t *)(h->ws + L.vals0), nullptr};
    uint32_t *hist = (uint32_t *)(h->ws + L.hist), *part = (uint32_t *)(h->ws + L.part);
    int bits = 1;  // keys < 3 n
    while (bits < 32 && (1ull << bits) < 3ull * (unsigned long long)h->n) ++bits;
    const unsigned long long end = first + count;
    for (unsigned long long b0 = first; b0 < end;) {
        unsigned long long b1 = (b0 / B + 1) * B;
        if (b1 > end) b1 = end;
        SnapBatch b{p.orders, b0, b1 - b0, b0 / B, (long long)((b1 - b0) * per), drawn, nullptr, nullptr, (float *)(h->ws + L.contrib)};
        hipLaunchKernelGGL(k_snap_draw, dim3((unsigned)LH_CDIV(b.count * (unsigned long long)(p.K + 1), 256)), dim3(256), 0, s, g,
                           p.orders, b.first, b.count, drawn);
        const SortBuffers sorted = radix_sort(SortArrays<1>{drawn, nullptr, nullptr, true}, b.entries, bits, two, one, hist,
                                              part, s);
        b.keys = sorted.k;
        b.vals = sorted.p0;
        contrib(g, p.dtype, b, s);
        apply(g, p.dtype, b, s);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return hip_fail(h, e, "snapshot");
        b0 = b1;
    }
    return LH_OK;
}

}  // namespace lh
