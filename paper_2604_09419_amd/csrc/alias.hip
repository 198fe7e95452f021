// Graph validation and alias-table construction (binary64, built with -ffp-contract=off).
//
// The two discrete distributions of the method are encoded as alias tables (Walker
// 1977 / Vose 1991): the edge distribution of Algorithm 3's root-edge selection
// (weights w over arcs) and the negative distribution of Eq. (1) (weights
// out-degree^0.75 over nodes).  The construction is the closed form of the sweeping
// construction (Huebschle-Schneider and Sanders, "Parallel Weighted Random Sampling"):
//   W = last element of the canonical scan of w; q_i = fl(fl(w_i N) / W)
//   lights L = {q < 1}, heavies H = {q >= 1}, each in index order
//   D = monotone canonical scan of (1 - q) over L, X = the same of (q - 1) over H
//   light a (start S_a = D[a-1], S_0 = 0): prob q, alias H[min(#{X[k] <= S_a}, |H|-1)]
//   heavy k < |H|-1: j = #{S_a < X[k]} - 1, overflow o = D[j] - X[k] (0 when j < 0,
//   clamped at 0); o > 0 gives prob max(0, 1 - o), alias H[k+1]; else prob 1, self
//   last heavy, or every item when H is empty: prob 1, self
//   thr = prob >= 1 ? 2^64 - 1 : (uint64)(prob 2^64)
// Every step is a single correctly rounded binary64 operation in a fixed order, so
// the tables are bitwise reproducible.
#include <algorithm>
#include <cstring>
#include <mutex>
#include <vector>

#include "handle.hpp"
#include "scan.hpp"

#pragma clang fp contract(off)

// Build scratch of lh_build_alias_noalloc, for callers that cannot allocate: one array
// per GPU, held from the library's load to the end of the process.  Host code never uses
// this name as an address (in host code it names a host-side stand-in); it uses the
// device address hipGetSymbolAddress returns for the current device, kept per device.
static __device__ __align__(256) unsigned char scratch[lh::kNoAllocScratchBytes];

namespace lh {

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void *g_scratch_ptr[kMaxDevices] = {};
hipError_t g_scratch_err[kMaxDevices] = {};
bool g_scratch_done[kMaxDevices] = {};
}  // namespace

// Once per device, with that device current: the device address of `scratch` there.
hipError_t noalloc_scratch_setup(int device)
{
    if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_done[device]) {
        void *ptr = nullptr;
        hipError_t e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        g_scratch_err[device] = e;
        g_scratch_ptr[device] = e == hipSuccess ? ptr : nullptr;
        g_scratch_done[device] = true;
    }
    return g_scratch_err[device];
}

static void *noalloc_scratch(int device)
{
    if (device < 0 || device >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    return g_scratch_done[device] ? g_scratch_ptr[device] : nullptr;
}

// ---------------------------------------------------------------------------
// Validation of the arcs: endpoints in [0, n), weights finite and >= 0.
// ---------------------------------------------------------------------------
__global__ void k_validate(const int32_t *src, const int32_t *dst, const float *w, long long m,
                           long long n, unsigned int *status)
{
    long long a = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (a >= m) return;
    int32_t s = src[a], t = dst[a];
    float x = w[a];
    unsigned int f = 0;
    if (s < 0 || (long long)s >= n || t < 0 || (long long)t >= n) f |= ST_OUT_OF_RANGE;
    if (!(x >= 0.0f) || isinf(x)) f |= ST_BAD_WEIGHT;
    if (f) atomicOr(status, f);
}

__global__ void k_clear_status(unsigned int *status) { status[0] = 0u; }

lh_status validate_graph(lh_handle *h)
{
    hipStream_t s = h->stream;
    hipLaunchKernelGGL(k_clear_status, dim3(1), dim3(1), 0, s, h->status);
    if (h->m > 0)
        hipLaunchKernelGGL(k_validate, dim3((unsigned)LH_CDIV(h->m, 256)), dim3(256), 0, s, h->src,
                           h->dst, h->w, h->m, h->n, h->status);
    unsigned int st = 0;
    hipError_t e = hipMemcpyAsync(&st, h->status, sizeof(st), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(h, e, "graph validation");
    if (st & ST_OUT_OF_RANGE) return fail(h, LH_ERR_OUT_OF_RANGE, "an arc endpoint is outside [0, n)");
    if (st & ST_BAD_WEIGHT) return fail(h, LH_ERR_ZERO_WEIGHT, "a weight is negative, NaN or infinite");
    return LH_OK;
}

// ---------------------------------------------------------------------------
// Out- and in-degrees.  Counting with one global atomic per arc end runs at the rate of single
// scattered atomics (21 G/s; C2's 2 x 16.8 M ends: 1.59 ms), and a hub's counter takes one at
// a time, which alone costs 90 us on a graph of 10,000 nodes and 200,000 arcs.  So the ends are
// counted in LDS and each workgroup adds its counters once.
//
//   n <= 2^15         a counter per node fits in LDS (128 of 160 KB): k_degrees_lds, 7 us on
//                     the graph of 10,000 nodes
//   up to 2^21, m >= n   k_degree_parts sorts tiles of 16,384 ends by ranges of 2^15 nodes
//                     (2 bytes an end, tile by tile, so no tile waits for another), and
//                     k_degree_ranges counts a range's parts of many tiles in LDS: C2 81 us
//   else              k_degrees, an atomic per run of equal ends: with more ranges a tile's parts
//                     are too short, and with few arcs the counters cost more than the arcs
// ---------------------------------------------------------------------------
constexpr int DEG_RANGE_BITS = 15, DEG_RANGE = 1 << DEG_RANGE_BITS;
constexpr int DEG_MAX_RANGES = 64, DEG_TILE = 16384, DEG_THREADS = 1024;
constexpr long long DEG_MAX_NODES = (long long)DEG_RANGE * DEG_MAX_RANGES;

// The lanes whose key differs from the lane before it count the run that starts there: arc lists
// are often grouped by an end, and equal LDS addresses are taken one lane at a time.  The valid
// lanes are a prefix of the wavefront.
__device__ __forceinline__ int run_length(int key, bool ok)
{
    const int lane = threadIdx.x & 63;
    const int prev = __shfl_up(key, 1);
    const bool head = ok && (lane == 0 || prev != key);
    const unsigned long long heads = __ballot(head);
    const int nvalid = __popcll(__ballot(ok));
    const unsigned long long above = lane == 63 ? 0ull : heads & (~0ull << (lane + 1));
    const int next = above ? __ffsll((long long)above) - 1 : nvalid;
    return head ? next - lane : 0;
}

// blockIdx.y: 0 the sources, 1 the destinations.
__global__ void __launch_bounds__(256) k_degrees(const int32_t *src, const int32_t *dst, long long m, int32_t *deg,
                                                 int32_t *indeg)
{
    const long long a = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const int32_t *end = blockIdx.y ? dst : src;
    int32_t *cnt = blockIdx.y ? indeg : deg;
    const int x = a < m ? end[a] : -1;
    const int len = run_length(x, a < m);
    if (len) atomicAdd(&cnt[x], len);
}

__global__ void __launch_bounds__(DEG_THREADS) k_degrees_lds(const int32_t *src, const int32_t *dst, long long m,
                                                             int n, int32_t *deg, int32_t *indeg)
{
    __shared__ int32_t cnt[DEG_RANGE];
    const int32_t *end = blockIdx.y ? dst : src;
    int32_t *out = blockIdx.y ? indeg : deg;
    for (int i = threadIdx.x; i < n; i += DEG_THREADS) cnt[i] = 0;
    __syncthreads();
    const long long step = (long long)gridDim.x * DEG_THREADS;
    for (long long a0 = (long long)blockIdx.x * DEG_THREADS; a0 < m; a0 += 4 * step) {
        int x[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const long long a = a0 + r * step + threadIdx.x;
            x[r] = a < m ? end[a] : -1;
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int len = run_length(x[r], x[r] >= 0);
            if (len) atomicAdd(&cnt[x[r]], len);
        }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < n; i += DEG_THREADS)
        if (cnt[i]) atomicAdd(&out[i], cnt[i]);
}

// part[y][tile][16384]: the tile's ends (low 15 bits) by range; off[y][tile][ranges + 1].
__global__ void __launch_bounds__(DEG_THREADS) k_degree_parts(const int32_t *src, const int32_t *dst, long long m,
                                                              int ranges, uint16_t *part, int32_t *off)
{
    __shared__ __align__(16) uint16_t buf[DEG_TILE];
    __shared__ int32_t cnt[DEG_MAX_RANGES], base[DEG_MAX_RANGES];
    const long long ntiles = gridDim.x, tile = blockIdx.x;
    const int32_t *end = blockIdx.y ? dst : src;
    const long long lo = tile * DEG_TILE;
    const int len = (int)(m - lo < DEG_TILE ? m - lo : DEG_TILE);
    if (threadIdx.x < DEG_MAX_RANGES) cnt[threadIdx.x] = 0;
    __syncthreads();
    int x[DEG_TILE / DEG_THREADS], at[DEG_TILE / DEG_THREADS];
#pragma unroll
    for (int r = 0; r < DEG_TILE / DEG_THREADS; ++r) {
        const int k = r * DEG_THREADS + (int)threadIdx.x;
        x[r] = k < len ? end[lo + k] : -1;
    }
#pragma unroll
    for (int r = 0; r < DEG_TILE / DEG_THREADS; ++r)
        at[r] = x[r] >= 0 ? atomicAdd(&cnt[x[r] >> DEG_RANGE_BITS], 1) : 0;
    __syncthreads();
    if (threadIdx.x < 64) {
        const int lane = threadIdx.x, c = lane < ranges ? cnt[lane] : 0;
        int inc = c;
        for (int d = 1; d < 64; d <<= 1) {
            const int y = __shfl_up(inc, d);
            if (lane >= d) inc += y;
        }
        base[lane] = inc - c;
        int32_t *o = off + ((long long)blockIdx.y * ntiles + tile) * (ranges + 1);
        if (lane < ranges) o[lane] = inc - c;
        if (lane == ranges - 1) o[ranges] = inc;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < DEG_TILE / DEG_THREADS; ++r)
        if (x[r] >= 0) buf[base[x[r] >> DEG_RANGE_BITS] + at[r]] = (uint16_t)(x[r] & (DEG_RANGE - 1));
    __syncthreads();
    // (the end of a short tile copies words that no part covers)
    uint4 *out = reinterpret_cast<uint4 *>(part + ((long long)blockIdx.y * ntiles + tile) * DEG_TILE);
    for (int i = threadIdx.x; i * 8 < len; i += DEG_THREADS) out[i] = reinterpret_cast<const uint4 *>(buf)[i];
}

// Workgroup (range, slice of the tiles, end): a wavefront takes a tile's part at a time.
__global__ void __launch_bounds__(DEG_THREADS) k_degree_ranges(const uint16_t *part, const int32_t *off, long long ntiles,
                                                               int ranges, long long n, int32_t *deg, int32_t *indeg)
{
    __shared__ int32_t cnt[DEG_RANGE];
    const int range = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long first = (long long)range * DEG_RANGE;
    const int nodes = (int)(n - first < DEG_RANGE ? n - first : DEG_RANGE);
    for (int i = threadIdx.x; i < nodes; i += DEG_THREADS) cnt[i] = 0;
    __syncthreads();
    const int32_t *o = off + (long long)blockIdx.z * ntiles * (ranges + 1) + range;
    const uint16_t *p = part + (long long)blockIdx.z * ntiles * DEG_TILE;
    for (long long t = (long long)blockIdx.y * (DEG_THREADS / 64) + wave; t < ntiles;
         t += (long long)gridDim.y * (DEG_THREADS / 64)) {
        const int lo = o[t * (ranges + 1)], hi = o[t * (ranges + 1) + 1];
        const uint16_t *q = p + t * DEG_TILE;
        for (int k0 = lo; k0 < hi; k0 += 512) {
            int x[8];
#pragma unroll
            for (int r = 0; r < 8; ++r) {
                const int k = k0 + r * 64 + lane;
                x[r] = k < hi ? (int)q[k] : -1;
            }
#pragma unroll
            for (int r = 0; r < 8; ++r)
                if (x[r] >= 0) atomicAdd(&cnt[x[r]], 1);
        }
    }
    __syncthreads();
    int32_t *out = (blockIdx.z ? indeg : deg) + first;
    for (int i = threadIdx.x; i < nodes; i += DEG_THREADS)
        if (cnt[i]) atomicAdd(&out[i], cnt[i]);
}

// deg and indeg are zero; work: at least 8 m bytes of scratch.
static void count_degrees(const int32_t *src, const int32_t *dst, long long n, long long m, int32_t *deg, int32_t *indeg,
                          char *work, hipStream_t s)
{
    if (n <= DEG_RANGE) {
        const long long wanted = LH_CDIV(m, 16 * DEG_THREADS);
        hipLaunchKernelGGL(k_degrees_lds, dim3((unsigned)std::min(wanted, 64ll), 2), dim3(DEG_THREADS), 0, s, src, dst, m,
                           (int)n, deg, indeg);
    } else if (n <= DEG_MAX_NODES && m >= n) {
        const int ranges = (int)LH_CDIV(n, DEG_RANGE);
        const long long ntiles = LH_CDIV(m, DEG_TILE);
        uint16_t *part = (uint16_t *)work;  // 4 bytes an arc (and less than 64 KB of a last tile),
        int32_t *off = (int32_t *)(work + 4 * ntiles * DEG_TILE);  // then at most 520 a tile
        hipLaunchKernelGGL(k_degree_parts, dim3((unsigned)ntiles, 2), dim3(DEG_THREADS), 0, s, src, dst, m, ranges, part,
                           off);
        const long long slices = std::max(1ll, std::min((long long)LH_CDIV(128, ranges), LH_CDIV(ntiles, 16)));
        hipLaunchKernelGGL(k_degree_ranges, dim3((unsigned)ranges, (unsigned)slices, 2), dim3(DEG_THREADS), 0, s, part, off,
                           ntiles, ranges, n, deg, indeg);
    } else {
        hipLaunchKernelGGL(k_degrees, dim3((unsigned)LH_CDIV(m, 256), 2), dim3(256), 0, s, src, dst, m, deg, indeg);
    }
}

// ---------------------------------------------------------------------------
// Weights of the two tables, binary64.
// ---------------------------------------------------------------------------
// Eq. (1) numerator: d^0.75 = sqrt(d) * sqrt(sqrt(d)), each step correctly rounded.
__device__ __forceinline__ double neg_weight(int32_t deg)
{
    const double s = __dsqrt_rn((double)deg);
    return __dmul_rn(s, __dsqrt_rn(s));
}

__global__ void __launch_bounds__(256) k_neg_weights(const int32_t *deg, long long n, double *w)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) w[i] = neg_weight(deg[i]);
}

// Words of the build's small result block: what the host reads back in one copy.
enum { CNT_ACTIVE = 0, CNT_HEAT = 1, CNT_STATUS = 257, CNT_PMAX = 258, CNT_WORDS = 259 };

// The degrees and the result block of a build start at zero.
__global__ void __launch_bounds__(256) k_build_zero(int32_t *deg, int32_t *indeg, long long n, unsigned long long *cnt)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) deg[i] = indeg[i] = 0;
    if (i < CNT_WORDS) cnt[i] = 0ull;
}

// Heat of node r (see common.hpp): floor(-log2 p_r), p_r = (out + in) / m + K nu_r / W_nu.
// It only chooses between the write paths of the training kernel, so it is computed in
// ordinary binary64 arithmetic.  cnt[CNT_PMAX] is the largest p_r (the bits of a non-negative
// binary64 number order like the number), cnt[CNT_ACTIVE] counts the nodes with an arc, cnt[CNT_HEAT + h]
// the nodes of heat h (a histogram in LDS per workgroup, then one atomic per bin; the grid
// is at most 256 workgroups, since every one of them ends with atomics on the same few words).
__global__ void __launch_bounds__(256) k_heat(const int32_t *deg, const int32_t *indeg, const double *Wnu, long long n,
                                              long long m, int K, uint8_t *heat, unsigned long long *cnt)
{
    __shared__ unsigned int hist[256];
    __shared__ unsigned int active;
    __shared__ unsigned long long pmax;
    hist[threadIdx.x] = 0u;
    if (threadIdx.x == 0) active = 0u, pmax = 0ull;
    __syncthreads();
    const double Wn = *Wnu;
    unsigned mine = 0u;
    double top = 0.0;
    for (long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (long long)gridDim.x * blockDim.x) {
        const int32_t od = deg[r], both = od + indeg[r];
        if (both > 0) ++mine;
        double p = (double)both / (double)m;
        if (Wn > 0.0) p += (double)K * neg_weight(od) / Wn;
        if (p > top) top = p;
        int hv = 255;
        if (p > 0.0) {
            const double t = floor(-log2(p));
            hv = t < 0.0 ? 0 : (t > 254.0 ? 254 : (int)t);
        }
        heat[r] = (uint8_t)hv;
        atomicAdd(&hist[hv], 1u);
    }
    if (mine) atomicAdd(&active, mine);
    atomicMax(&pmax, (unsigned long long)__double_as_longlong(top));
    __syncthreads();
    if (hist[threadIdx.x]) atomicAdd(&cnt[CNT_HEAT + threadIdx.x], (unsigned long long)hist[threadIdx.x]);
    if (threadIdx.x == 0) {
        if (active) atomicAdd(&cnt[CNT_ACTIVE], (unsigned long long)active);
        atomicMax(&cnt[CNT_PMAX], pmax);
    }
}

__global__ void k_fill_u8(uint8_t *p, long long n, uint8_t v)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__device__ __forceinline__ unsigned long long prob_to_thr(double prob)
{
    if (prob >= 1.0) return ~0ull;
    return (unsigned long long)__dmul_rn(prob, 18446744073709551616.0);
}

struct RecOut {
    EdgeRec *erec;  // edge table, or
    NegRec *nrec;   // negative table
    const int32_t *src, *dst;
    const uint8_t *heat;  // per node; NULL: every node 255 (never hot)
};

// Without a heat array (imported alias tables carry no degrees) every row is taken as hot:
// the coherent atomic update is correct for any row, only slower.
__device__ __forceinline__ uint32_t heat_of(const RecOut &o, long long v) { return o.heat ? o.heat[v] : 0u; }

__device__ __forceinline__ void write_rec(const RecOut &o, long long i, unsigned long long thr,
                                          int32_t al)
{
    if (o.erec) {
        EdgeRec r;
        r.thr = thr;
        r.alias = al;
        r.src_c = o.src[i];
        r.dst_c = o.dst[i];
        r.src_a = o.src[al];
        r.dst_a = o.dst[al];
        r.heat = heat_of(o, r.src_c) | (heat_of(o, r.dst_c) << 8) | (heat_of(o, r.src_a) << 16) |
                 (heat_of(o, r.dst_a) << 24);
        o.erec[i] = r;
    } else {
        NegRec r;
        r.thr = thr;
        r.alias = al;
        r.heat = heat_of(o, i) | (heat_of(o, al) << 8);
        o.nrec[i] = r;
    }
}

// ---------------------------------------------------------------------------
// One table's build.  Both tables are built by the same launches: a kernel's first workgroups
// take table 0, the rest table 1, and every count that a later kernel needs stays on the device,
// so the host waits once, at the end.  (C2: checks, degrees, both tables and their export 5.46 ms
// with a table at a time and three waits, 1.23 ms so.)
//
// The construction reads its prefix sums only through searches, so no scan is ever written out
// element by element with its offsets: a scan is the chains' values within each chunk and, per
// chunk, the offset of the chunk (the canonical scan of the totals before it).  Rounding is
// monotone, so the running maximum of off + x within a chunk is off + (the running maximum of
// x), and across chunks it is enough to keep the largest value before the chunk:
//   value(i) = max(before[c], off[c] + loc[i]),  c = i / 1024.
// ---------------------------------------------------------------------------
struct Scan {
    const double *loc;   // [n] per element, within its chunk
    const double *off;   // [chunks] canonical scan of the totals before the chunk (0 for the first)
    const double *before;  // [chunks] largest value before the chunk (-inf for the first)
    const double *end;   // [chunks] value of the chunk's last element
    long long n;

    __device__ __forceinline__ double at(long long i) const
    {
        const long long c = i / SCAN_CHUNK;
        return __builtin_fmax(before[c], off[c] + loc[i]);
    }
};

constexpr int SPLIT_ITEMS = 1024;  // items a wavefront splits

struct Table {
    long long N;
    const float *w;        // arc weights, or NULL: the weight of item i is neg_weight(deg[i])
    const int32_t *deg;
    double *dx;            // [N] deficits of the lights, then excesses of the heavies
    int32_t *idx;          // [N] the heavies' items, in index order
    int32_t *blk;          // [N / 1024 + 2] lights before each 1,024 items; last: all of them
    double *tot, *mxl;     // [N / 1024 + 2] chunk totals and chunk maxima, then (in place)
                           // the totals' own chains and the chunks' last values
    double *off, *before;  // [N / 1024 + 2]
    double *W;             // total weight
    RecOut out;

    __device__ __forceinline__ double weight(long long i) const { return w ? (double)w[i] : neg_weight(deg[i]); }
    // q_i = fl(fl(w_i N) / W).  A total that is not a positive finite number makes every item
    // heavy (prob 1, self).
    __device__ __forceinline__ double q(long long i, double Wt) const
    {
        return Wt > 0.0 && !isinf(Wt) ? __ddiv_rn(__dmul_rn(weight(i), (double)N), Wt) : 1.0;
    }
    __device__ __forceinline__ long long lights() const { return blk[LH_CDIV(N, SPLIT_ITEMS)]; }
    // The scan of one half (false: lights, true: heavies), its chunks after the lights' ones.
    __device__ __forceinline__ Scan half(bool heavy, long long nL) const
    {
        const long long c0 = heavy ? LH_CDIV(nL, SCAN_CHUNK) : 0;
        return Scan{dx + (heavy ? nL : 0), off + c0, before + c0, mxl + c0, heavy ? N - nL : nL};
    }
};

struct Tables {
    Table t[2];
    unsigned first[3];  // workgroups [first[k], first[k + 1]) take table k
};

__device__ __forceinline__ const Table &table_of(const Tables &T, long long &b)
{
    const int k = blockIdx.x >= T.first[1] ? 1 : 0;
    b = (long long)blockIdx.x - T.first[k];
    return T.t[k];
}

// Chains over the weights, of which only the total is needed: no element is stored.  The node
// weights are in dx (k_neg_weights), which the split overwrites later.
__global__ void __launch_bounds__(256) k_chain_weights(Tables T)
{
    __shared__ double lds[CHAIN_LDS];
    long long b;
    const Table &t = table_of(T, b);
    const long long c0 = b * WAVE_CHUNKS, N = t.N;
    const int tiles = chain_tiles(N - c0 * SCAN_CHUNK);
    const float *w = t.w;
    const double *nw = t.dx;
    double *tot = t.tot;
    const auto total = [&](long long c, double v) { if (c * SCAN_CHUNK < N) tot[c] = v; };
    const auto none = [](long long, double) {};
    if (w)
        block_chains<0, float>(lds, N, c0, tiles, [&](long long i) { return w[i]; }, none, total, none);
    else
        block_chains<0, double>(lds, N, c0, tiles, [&](long long i) { return nw[i]; }, none, total, none);
}

// Chains over the deficits and the excesses (both halves of both tables), storing the running
// maximum of each chunk's prefix sums in place.
__global__ void __launch_bounds__(256) k_chain_dx(Tables T)
{
    __shared__ double lds[CHAIN_LDS];
    long long b;
    const Table &t = table_of(T, b);
    const long long nL = t.lights();
    const long long cL = LH_CDIV(nL, SCAN_CHUNK), gL = LH_CDIV(cL, WAVE_CHUNKS);
    const bool heavy = b >= gL;
    const long long c0 = (heavy ? b - gL : b) * WAVE_CHUNKS;
    const long long n = heavy ? t.N - nL : nL;
    if (c0 * SCAN_CHUNK >= n) return;
    double *x = t.dx + (heavy ? nL : 0), *tot = t.tot + (heavy ? cL : 0), *mxl = t.mxl + (heavy ? cL : 0);
    block_chains<2, double>(lds, n, c0, chain_tiles(n - c0 * SCAN_CHUNK), [&](long long i) { return x[i]; },
                            [&](long long i, double v) { x[i] = v; },
                            [&](long long c, double v) { if (c * SCAN_CHUNK < n) tot[c] = v; },
                            [&](long long c, double v) { if (c * SCAN_CHUNK < n) mxl[c] = v; });
}

// The levels above the chunks, one workgroup per scan: the canonical scan of the chunk totals (its
// own chains as above, the totals of those, at most 2,048 for 2^31 items, by one thread), which
// becomes each chunk's offset.  tot is left with the chains' values.
constexpr int LEVEL_THREADS = 256, LEVEL_TOP = 2048;

__device__ __forceinline__ void scan_levels(double *tot, double *off, long long nch, double *lds, double *top,
                                            double *topinc)
{
    const long long n1 = LH_CDIV(nch, SCAN_CHUNK);
    for (long long c0 = 0; c0 < n1; c0 += WAVE_CHUNKS)
        block_chains<1, double>(lds, nch, c0, chain_tiles(nch - c0 * SCAN_CHUNK), [&](long long i) { return tot[i]; },
                                [&](long long i, double v) { tot[i] = v; },
                                [&](long long c, double v) { if (c < n1) top[c] = v; }, [](long long, double) {});
    __syncthreads();
    if (threadIdx.x == 0) {
        // chunks of 1,024 again: at most two, the second offset by the first one's total
        double base = 0.0;
        for (long long lo = 0; lo < n1; lo += SCAN_CHUNK) {
            OpNeumaier::State st = OpNeumaier::init();
            double v = 0.0;
            for (long long i = lo; i < n1 && i < lo + SCAN_CHUNK; ++i) {
                v = OpNeumaier::step(st, top[i]);
                topinc[i] = lo ? OpNeumaier::combine(base, v) : v;
            }
            base = v;
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
            if (i + 1 < nch) off[i + 1] = c ? OpNeumaier::combine(topinc[c - 1], v[k]) : v[k];
        }
    }
    __syncthreads();
}

// Total weight of each table: off[last chunk] + that chunk's total.  Flags ST_ZERO_TOTAL, in the
// status word and (with what was flagged there before) in the result block.
__global__ void __launch_bounds__(LEVEL_THREADS) k_levels_weights(Tables T, unsigned int *status, unsigned long long *cnt)
{
    __shared__ double lds[CHAIN_LDS];
    __shared__ double top[LEVEL_TOP], topinc[LEVEL_TOP];
    const Table &t = T.t[blockIdx.x];
    const long long nch = LH_CDIV(t.N, SCAN_CHUNK);
    const double last = t.tot[nch - 1];  // before the totals become their chains
    __syncthreads();
    scan_levels(t.tot, t.off, nch, lds, top, topinc);
    if (threadIdx.x == 0) {
        const double W = nch > 1 ? OpNeumaier::combine(t.off[nch - 1], last) : last;
        *t.W = W;
        const unsigned bad = !(W > 0.0) || isinf(W) ? ST_ZERO_TOTAL : 0u;
        if ((atomicOr(status, bad) | bad) & ST_ZERO_TOTAL) atomicOr(&cnt[CNT_STATUS], (unsigned long long)ST_ZERO_TOTAL);
    }
}

// Offsets and prefix maxima of the four deficit and excess scans (workgroup: table, half).
__global__ void __launch_bounds__(LEVEL_THREADS) k_levels_dx(Tables T)
{
    __shared__ double lds[CHAIN_LDS];
    __shared__ double top[LEVEL_TOP], topinc[LEVEL_TOP];
    const Table &t = T.t[blockIdx.x >> 1];
    const bool heavy = (blockIdx.x & 1) != 0;
    const long long nL = t.lights(), n = heavy ? t.N - nL : nL;
    if (n == 0) return;
    const long long c0 = heavy ? LH_CDIV(nL, SCAN_CHUNK) : 0, nch = LH_CDIV(n, SCAN_CHUNK);
    double *off = t.off + c0, *before = t.before + c0, *end = t.mxl + c0;
    scan_levels(t.tot + c0, off, nch, lds, top, topinc);
    // prefix maximum of off[c] + (the chunk's own maximum): a consecutive quarter of the chunks
    // per wavefront, 4 x 64 of them at a time
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

// Lights (q < 1) among 1,024 consecutive items, per wavefront.
__global__ void __launch_bounds__(256) k_split_count(Tables T)
{
    long long b;
    const Table &t = table_of(T, b);
    const int lane = threadIdx.x & 63;
    const long long part = b * 4 + (threadIdx.x >> 6), lo = part * SPLIT_ITEMS;
    if (lo >= t.N) return;
    const double W = *t.W;
    int32_t cnt = 0;
#pragma unroll 4
    for (int r = 0; r < SPLIT_ITEMS / 64; ++r) {
        const long long i = lo + r * 64 + lane;
        cnt += __popcll(__ballot(i < t.N && t.q(i < t.N ? i : 0, W) < 1.0));
    }
    if (lane == 0) t.blk[part] = cnt;
}

// Exclusive prefix sums of the light counts, in place, with the total behind them; one workgroup
// per table, a run of counts per thread.
__global__ void __launch_bounds__(1024) k_split_scan(Tables T)
{
    __shared__ int32_t ws[16];
    const Table &t = T.t[blockIdx.x];
    const long long nt = LH_CDIV(t.N, SPLIT_ITEMS), per = LH_CDIV(nt, 1024);
    const long long lo = threadIdx.x * per, hi = lo + per < nt ? lo + per : nt;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    int32_t s = 0;
#pragma unroll 8
    for (long long i = lo; i < hi; ++i) s += t.blk[i];
    int32_t inc = s;
    for (int d = 1; d < 64; d <<= 1) {
        const int32_t y = __shfl_up(inc, d);
        if (lane >= d) inc += y;
    }
    if (lane == 63) ws[wave] = inc;
    __syncthreads();
    int32_t run = inc - s;
    for (int v = 0; v < wave; ++v) run += ws[v];
#pragma unroll 8
    for (long long i = lo; i < hi; ++i) {
        const int32_t c = t.blk[i];
        t.blk[i] = run;
        run += c;
    }
    if (threadIdx.x == 1023) t.blk[nt] = run;
}

// Split into lights (deficits 1 - q, prefix of dx) and heavies (excesses q - 1, suffix, and their
// items), each in index order.  q is computed again from the weight: cheaper than a pass that
// stores it.
__global__ void __launch_bounds__(256) k_split(Tables T)
{
    long long b;
    const Table &t = table_of(T, b);
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
                t.idx[i - before] = (int32_t)i;
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
// times the ratio of the halves), and the items' own searches touch no memory.  C2's 16.8 M arcs:
// 0.51 ms for both tables, 0.87 ms with a thread per light and per heavy that searched all of the
// other half and wrote every second record of a line.  What is left is 0.24 ms of traffic at a
// copy's rate and 0.14 ms of heat bytes (67 M scattered reads).
constexpr int REC_ITEMS = 1024, REC_STAGE = 1024;
static_assert(REC_ITEMS == SPLIT_ITEMS, "a workgroup's first light is its split count");

// The two halves' scans lie one behind the other: position p of half `heavy` is element
// (heavy ? nL : 0) + p, in chunk (heavy ? cL : 0) + p / 1024.
__global__ void __launch_bounds__(256) k_records(Tables T)
{
    __shared__ double sx[REC_STAGE], sd[REC_STAGE + 1];
    __shared__ long long ends[4];
    __shared__ int32_t wc[4];
    long long b;
    const Table &t = table_of(T, b);
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
        if (wave < 2) {
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
    // item r of this thread: i0 + wave * 256 + r * 64 + lane.  Each step below is taken for all
    // four items before the next, so that their loads are in flight together.
    const long long first = i0 + wave * 256 + lane;
    double q[4];
    unsigned long long mask[4];
    int32_t cnt = 0;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
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
    long long pos[4];  // lights before the item, or its place among the heavies
    double key[4];     // S_a, or X[k]
#pragma unroll
    for (int r = 0; r < 4; ++r) {
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
    int lo[4] = {0, 0, 0, 0};
    if (staged) {
        int hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) hi[r] = q[r] < 1.0 ? xn : dn;
        for (int left = xn > dn ? xn : dn; left > 0; left >>= 1) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
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
        for (int r = 0; r < 4; ++r) {
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
    unsigned long long thr[4];
    int32_t al[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
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
        const int32_t item = t.idx[k < 0 ? 0 : k];
        al[r] = k < 0 ? (int32_t)(first + r * 64) : item;
    }
    if (t.out.erec) {
        int32_t e[4][4];  // endpoints: source and destination, of the item and of its alias
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const long long i = first + r * 64 < i1 ? first + r * 64 : i1 - 1;
            const long long z = first + r * 64 < i1 ? al[r] : i1 - 1;
            e[r][0] = t.out.src[i];
            e[r][1] = t.out.dst[i];
            e[r][2] = t.out.src[z];
            e[r][3] = t.out.dst[z];
        }
        uint32_t heat[4];
#pragma unroll
        for (int r = 0; r < 4; ++r)
            heat[r] = (uint32_t)t.out.heat[e[r][0]] | ((uint32_t)t.out.heat[e[r][1]] << 8) |
                      ((uint32_t)t.out.heat[e[r][2]] << 16) | ((uint32_t)t.out.heat[e[r][3]] << 24);
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (first + r * 64 < i1)
                t.out.erec[first + r * 64] = EdgeRec{thr[r], al[r], e[r][0], e[r][1], e[r][2], e[r][3], heat[r]};
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (first + r * 64 < i1) write_rec(t.out, first + r * 64, thr[r], al[r]);
    }
}

// ---------------------------------------------------------------------------
// Host driver: both tables, no wait before the end.
// ---------------------------------------------------------------------------
static unsigned spread(Tables &T, long long per)
{
    T.first[0] = 0;
    for (int k = 0; k < 2; ++k) T.first[k + 1] = T.first[k] + (unsigned)LH_CDIV(T.t[k].N, per);
    return T.first[2];
}

// Two halves cut separately: at most one part more than the whole.
static unsigned spread_halves(Tables &T, long long per)
{
    T.first[0] = 0;
    for (int k = 0; k < 2; ++k) T.first[k + 1] = T.first[k] + (unsigned)LH_CDIV(T.t[k].N, per) + 1;
    return T.first[2];
}

lh_status build_alias(lh_handle *h, void *scratch, size_t bytes)
{
    const ScratchLayout L = scratch_layout(h->n, h->m);
    if (!scratch) return fail(h, LH_ERR_INVALID_ARG, "scratch is NULL");
    if (bytes < L.total) return fail(h, LH_ERR_WORKSPACE_TOO_SMALL, "alias scratch too small");
    h->edge_ready = h->neg_ready = false;
    h->walk.loaded = -1;  // walk roots come from the edge table: pairs made before are stale
    char *sc = (char *)scratch;
    hipStream_t s = h->stream;
    int32_t *deg = (int32_t *)(sc + L.deg), *indeg = (int32_t *)(sc + L.indeg);
    unsigned long long *cnt = (unsigned long long *)(sc + L.cnt);
    uint8_t *heat = (uint8_t *)(h->ws + h->lay.nheat);
    Tables T;
    for (int k = 0; k < 2; ++k) {
        Table &t = T.t[k];
        t.N = k == 0 ? h->n : h->m;
        t.w = k == 0 ? nullptr : h->w;
        t.deg = deg;
        t.dx = (double *)(sc + L.dx[k]);
        t.idx = (int32_t *)(sc + L.idx[k]);
        t.blk = (int32_t *)(sc + L.blk[k]);
        t.tot = (double *)(sc + L.tot[k]);
        t.mxl = (double *)(sc + L.mxl[k]);
        t.off = (double *)(sc + L.off[k]);
        t.before = (double *)(sc + L.before[k]);
        t.W = (double *)(sc + L.total_weight) + k;
        t.out = RecOut{k == 0 ? nullptr : h->erec, k == 0 ? h->nrec : nullptr, h->src, h->dst, heat};
    }
    const dim3 blk(256);
    // Degrees, the two total weights (the heats need the negative one), the heats.
    const long long zn = h->n > CNT_WORDS ? h->n : CNT_WORDS;
    hipLaunchKernelGGL(k_build_zero, dim3((unsigned)LH_CDIV(zn, 256)), blk, 0, s, deg, indeg, h->n, cnt);
    count_degrees(h->src, h->dst, h->n, h->m, deg, indeg, sc + L.dx[1], s);  // (dx is written after it)
    hipLaunchKernelGGL(k_neg_weights, dim3((unsigned)LH_CDIV(h->n, 256)), blk, 0, s, deg, h->n, T.t[0].dx);
    unsigned g = spread(T, (long long)WAVE_CHUNKS * SCAN_CHUNK);
    hipLaunchKernelGGL(k_chain_weights, dim3(g), blk, 0, s, T);
    hipLaunchKernelGGL(k_levels_weights, dim3(2), blk, 0, s, T, h->status, cnt);
    const unsigned gh = (unsigned)LH_CDIV(h->n, 256);
    hipLaunchKernelGGL(k_heat, dim3(gh < 256 ? gh : 256), blk, 0, s, deg, indeg, T.t[0].W, h->n, h->m, h->p.K, heat,
                       cnt);
    // Lights and heavies, their scans, the records.
    g = spread(T, 4 * SPLIT_ITEMS);
    hipLaunchKernelGGL(k_split_count, dim3(g), blk, 0, s, T);
    hipLaunchKernelGGL(k_split_scan, dim3(2), dim3(1024), 0, s, T);
    hipLaunchKernelGGL(k_split, dim3(g), blk, 0, s, T);
    g = spread_halves(T, (long long)WAVE_CHUNKS * SCAN_CHUNK);
    hipLaunchKernelGGL(k_chain_dx, dim3(g), blk, 0, s, T);
    hipLaunchKernelGGL(k_levels_dx, dim3(4), blk, 0, s, T);
    g = spread(T, REC_ITEMS);
    hipLaunchKernelGGL(k_records, dim3(g), blk, 0, s, T);
    unsigned long long host[CNT_WORDS];
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(h, e, "alias kernels");
    // One wait: the scratch may be released by the caller once this work has run.
    e = hipMemcpyAsync(host, cnt, sizeof(host), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return hip_fail(h, e, "alias build");
    h->n_active = (long long)host[CNT_ACTIVE];
    std::memcpy(&h->p_max, &host[CNT_PMAX], sizeof(double));
    for (int v = 0; v < 256; ++v) h->heat_count[v] = host[CNT_HEAT + v];
    if (host[CNT_STATUS] & ST_ZERO_TOTAL) {
        // with at least one arc some out-degree is positive: it is the arcs' total
        h->neg_ready = true;
        return fail(h, LH_ERR_ZERO_WEIGHT, "total arc weight is zero");
    }
    h->neg_ready = h->edge_ready = true;
    if (!h->cfg_pinned) h->cfg = auto_cfg(h);
    return LH_OK;
}

// ---------------------------------------------------------------------------
// Import / export of (thr, alias) arrays.  Imported alias entries outside [0, N)
// are replaced by the column itself and flagged, so no later kernel reads out of
// bounds.
// ---------------------------------------------------------------------------
__global__ void k_import(const unsigned long long *thr, const int32_t *alias, long long N, RecOut o,
                         unsigned int *status)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    int32_t al = alias[i];
    if (al < 0 || (long long)al >= N) {
        atomicOr(status, ST_OUT_OF_RANGE);
        al = (int32_t)i;
    }
    write_rec(o, i, thr[i], al);
}

__global__ void k_export(const EdgeRec *erec, const NegRec *nrec, long long N, unsigned long long *thr,
                         int32_t *alias)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= N) return;
    if (erec) {
        thr[i] = erec[i].thr;
        alias[i] = erec[i].alias;
    } else {
        thr[i] = nrec[i].thr;
        alias[i] = nrec[i].alias;
    }
}

lh_status import_alias(lh_handle *h, int which, const uint64_t *thr, const int32_t *alias)
{
    if (which == LH_ALIAS_EDGE) h->walk.loaded = -1;  // walk roots come from this table
    long long N = which == LH_ALIAS_EDGE ? h->m : h->n;
    RecOut o{which == LH_ALIAS_EDGE ? h->erec : nullptr, which == LH_ALIAS_EDGE ? nullptr : h->nrec,
             h->src, h->dst, nullptr};
    if (N > 0)
        hipLaunchKernelGGL(k_import, dim3((unsigned)LH_CDIV(N, 256)), dim3(256), 0, h->stream,
                           (const unsigned long long *)thr, alias, N, o, h->status);
    // Imported tables come without degrees: every node is taken as hot (heat 0).
    if (h->n > 0)
        hipLaunchKernelGGL(k_fill_u8, dim3((unsigned)LH_CDIV(h->n, 256)), dim3(256), 0, h->stream,
                           (uint8_t *)(h->ws + h->lay.nheat), h->n, (uint8_t)0);
    h->p_max = 0.0;
    for (int v = 0; v < 256; ++v) h->heat_count[v] = 0;
    h->heat_count[0] = (unsigned long long)h->n;
    if (!h->cfg_pinned) h->cfg = auto_cfg(h);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(h, e, "alias import");
    if (which == LH_ALIAS_EDGE)
        h->edge_ready = true;
    else
        h->neg_ready = true;
    return LH_OK;
}

lh_status export_alias(lh_handle *h, int which, uint64_t *thr, int32_t *alias)
{
    long long N = which == LH_ALIAS_EDGE ? h->m : h->n;
    if (N > 0)
        hipLaunchKernelGGL(k_export, dim3((unsigned)LH_CDIV(N, 256)), dim3(256), 0, h->stream,
                           which == LH_ALIAS_EDGE ? h->erec : nullptr,
                           which == LH_ALIAS_EDGE ? nullptr : h->nrec, N,
                           (unsigned long long *)thr, alias);
    hipError_t e = hipStreamSynchronize(h->stream);
    if (e != hipSuccess) return hip_fail(h, e, "alias export");
    return LH_OK;
}

}  // namespace lh

// The alias build of lh_build_alias with its scratch in the static per-device array
// instead of a caller's workspace: the same kernels, handed the array's device address.
// The kernels clear what they accumulate into (degrees, histogram) themselves, and every
// other scratch word is written before it is read, so the contents a previous call left
// do not matter.  Two such calls that overlap on one GPU (two host threads, two streams)
// race on the array.
extern "C" lh_status lh_build_alias_noalloc(lh_handle *h)
{
    if (!h) return LH_ERR_INVALID_ARG;
    if (!h->graph_set) return lh::fail(h, LH_ERR_NOT_BUILT, "lh_set_graph first");
    if (h->m < 1) return lh::fail(h, LH_ERR_ZERO_WEIGHT, "the graph has no arcs");
    // The documented limits; scratch_layout(2^21, 2^21) is 64.03 MiB, within the array.
    const lh::ScratchLayout L = lh::scratch_layout(h->n, h->m);
    if (h->n > lh::kNoAllocMaxItems || h->m > lh::kNoAllocMaxItems || L.total > lh::kNoAllocScratchBytes)
        return lh::fail(h, LH_ERR_INVALID_ARG,
                        "graph too large for the static build scratch (65 MiB: n and m up to 2^21 each)");
    int prev = -1;
    (void)hipGetDevice(&prev);
    if (prev != h->device) (void)hipSetDevice(h->device);
    lh_status st = LH_OK;
    hipError_t e = lh::noalloc_scratch_setup(h->device);
    void *ptr = lh::noalloc_scratch(h->device);
    if (e != hipSuccess || !ptr)
        st = lh::hip_fail(h, e != hipSuccess ? e : hipErrorInvalidSymbol, "static scratch address");
    else
        st = lh::build_alias(h, ptr, lh::kNoAllocScratchBytes);
    if (prev >= 0 && prev != h->device) (void)hipSetDevice(prev);
    return st;
}
