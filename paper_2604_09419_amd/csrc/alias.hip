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
#include <mutex>
#include <vector>

#include "handle.hpp"
#include "table.hpp"

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
enum { CNT_ACTIVE = 0, CNT_HEAT = 1, CNT_STATUS = 257, CNT_WORDS = 258 };

// The degrees and the result block of a build start at zero.
__global__ void __launch_bounds__(256) k_build_zero(int32_t *deg, int32_t *indeg, long long n, unsigned long long *cnt)
{
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) deg[i] = indeg[i] = 0;
    if (i < CNT_WORDS) cnt[i] = 0ull;
}

// Heat of node r (see common.hpp): floor(-log2 p_r), p_r = (out + in) / m + K nu_r / W_nu.
// It only chooses between the write paths of the training kernel, so it is computed in
// ordinary binary64 arithmetic.  cnt[CNT_ACTIVE] counts the nodes with an arc, cnt[CNT_HEAT + h] the
// nodes of heat h (a histogram in LDS per workgroup, then one atomic per bin; the grid
// is at most 256 workgroups, since every one of them ends with atomics on the same few words).
__global__ void __launch_bounds__(256) k_heat(const int32_t *deg, const int32_t *indeg, const double *Wnu, long long n,
                                              long long m, int K, uint8_t *heat, unsigned long long *cnt)
{
    __shared__ unsigned int hist[256];
    __shared__ unsigned int active;
    hist[threadIdx.x] = 0u;
    if (threadIdx.x == 0) active = 0u;
    __syncthreads();
    const double Wn = *Wnu;
    unsigned mine = 0u;
    for (long long r = (long long)blockIdx.x * blockDim.x + threadIdx.x; r < n; r += (long long)gridDim.x * blockDim.x) {
        const int32_t od = deg[r], both = od + indeg[r];
        if (both > 0) ++mine;
        double p = (double)both / (double)m;
        if (Wn > 0.0) p += (double)K * neg_weight(od) / Wn;
        int hv = 255;
        if (p > 0.0) {
            const double t = floor(-log2(p));
            hv = t < 0.0 ? 0 : (t > 254.0 ? 254 : (int)t);
        }
        heat[r] = (uint8_t)hv;
        atomicAdd(&hist[hv], 1u);
    }
    if (mine) atomicAdd(&active, mine);
    __syncthreads();
    if (hist[threadIdx.x]) atomicAdd(&cnt[CNT_HEAT + threadIdx.x], (unsigned long long)hist[threadIdx.x]);
    if (threadIdx.x == 0 && active) atomicAdd(&cnt[CNT_ACTIVE], (unsigned long long)active);
}

__global__ void k_fill_u8(uint8_t *p, long long n, uint8_t v)
{
    long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

struct RecOut {
    EdgeRec *erec;  // edge table, or
    NegRec *nrec;   // negative table
    const int32_t *src, *dst;
    const uint8_t *heat;  // per node; NULL: every node 0 (always hot)
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
// The two tables of the graph (table.hpp).  Both are built by the same launches: a kernel's first
// workgroups take table 0, the rest table 1, and every count that a later kernel needs stays on
// the device, so the host waits once, at the end.  (C2: checks, degrees, both tables and their
// export 5.46 ms with a table at a time and three waits, 1.23 ms so.)
// ---------------------------------------------------------------------------
struct GraphTable : Table {
    const int32_t *deg;  // without w: the weight of item i is neg_weight(deg[i])
    RecOut out;

    __device__ __forceinline__ double weight(long long i) const { return w ? (double)w[i] : neg_weight(deg[i]); }
    __device__ __forceinline__ double q(long long i, double Wt) const { return alias_q(weight(i), N, Wt); }
    // Items first, first + 64, .., RS of them, those before end.
    template <int RS>
    __device__ __forceinline__ void write(long long first, long long end, const unsigned long long (&thr)[RS],
                                          const uint32_t (&al)[RS]) const
    {
        if (out.erec) {
            int32_t e[RS][4];  // endpoints: source and destination, of the item and of its alias
#pragma unroll
            for (int r = 0; r < RS; ++r) {
                const long long i = first + r * 64 < end ? first + r * 64 : end - 1;
                const long long z = first + r * 64 < end ? (long long)al[r] : end - 1;
                e[r][0] = out.src[i];
                e[r][1] = out.dst[i];
                e[r][2] = out.src[z];
                e[r][3] = out.dst[z];
            }
            uint32_t heat[RS];
#pragma unroll
            for (int r = 0; r < RS; ++r)
                heat[r] = (uint32_t)out.heat[e[r][0]] | ((uint32_t)out.heat[e[r][1]] << 8) |
                          ((uint32_t)out.heat[e[r][2]] << 16) | ((uint32_t)out.heat[e[r][3]] << 24);
#pragma unroll
            for (int r = 0; r < RS; ++r)
                if (first + r * 64 < end)
                    out.erec[first + r * 64] = EdgeRec{thr[r], (int32_t)al[r], e[r][0], e[r][1], e[r][2], e[r][3], heat[r]};
        } else {
#pragma unroll
            for (int r = 0; r < RS; ++r)
                if (first + r * 64 < end) write_rec(out, first + r * 64, thr[r], (int32_t)al[r]);
        }
    }
};

struct Tables {
    GraphTable t[2];
    unsigned first[3];  // workgroups [first[k], first[k + 1]) take table k

    __device__ __forceinline__ const GraphTable &of(long long &b) const
    {
        const int k = blockIdx.x >= first[1] ? 1 : 0;
        b = (long long)blockIdx.x - first[k];
        return t[k];
    }
    __device__ __forceinline__ const GraphTable &whole(unsigned k) const { return t[k]; }
};

// Chains over the weights, of which only the total is needed: no element is stored.  The node
// weights are in dx (k_neg_weights), which the split overwrites later.
__global__ void __launch_bounds__(256) k_chain_weights(Tables T)
{
    __shared__ double lds[CHAIN_LDS];
    __shared__ ChainSegs segs;
    long long b;
    const GraphTable &t = T.of(b);
    const long long c0 = b * WAVE_CHUNKS, N = t.N;
    chunk_segs(segs, c0, N);
    __syncthreads();
    const float *w = t.w;
    const double *nw = t.dx;
    double *tot = t.tot;
    const auto total = [&](int r, double v) { if (segs.len[r]) tot[c0 + r] = v; };
    const auto none = [](long long, double) {};
    if (w)
        block_chains<0, float>(lds, segs, [&](long long i) { return w[i]; }, none, total, none);
    else
        block_chains<0, double>(lds, segs, [&](long long i) { return nw[i]; }, none, total, none);
}

// Chains over the deficits and the excesses (both halves of both tables), storing the running
// maximum of each chunk's prefix sums in place.
__global__ void __launch_bounds__(256) k_chain_dx(Tables T)
{
    __shared__ double lds[CHAIN_LDS];
    __shared__ ChainSegs segs;
    long long b;
    const GraphTable &t = T.of(b);
    const long long nL = t.lights();
    const long long cL = LH_CDIV(nL, SCAN_CHUNK), gL = LH_CDIV(cL, WAVE_CHUNKS);
    const bool heavy = b >= gL;
    const long long c0 = (heavy ? b - gL : b) * WAVE_CHUNKS;
    const long long n = heavy ? t.N - nL : nL;
    if (c0 * SCAN_CHUNK >= n) return;
    double *x = t.dx + (heavy ? nL : 0), *tot = t.tot + (heavy ? cL : 0), *mxl = t.mxl + (heavy ? cL : 0);
    chunk_segs(segs, c0, n);
    __syncthreads();
    block_chains<2, double>(lds, segs, [&](long long i) { return x[i]; }, [&](long long i, double v) { x[i] = v; },
                            [&](int r, double v) { if (segs.len[r]) tot[c0 + r] = v; },
                            [&](int r, double v) { if (segs.len[r]) mxl[c0 + r] = v; });
}

__global__ void __launch_bounds__(256) k_records(Tables T)
{
    __shared__ RecLds lds;
    long long b;
    const GraphTable &t = T.of(b);
    records_run<4>(t, b, lds);
}

// Total weights.  Flags ST_ZERO_TOTAL, in the status word and (with what was flagged there before)
// in the result block.
__global__ void __launch_bounds__(LEVEL_THREADS) k_levels_weights(Tables T, unsigned int *status, unsigned long long *cnt)
{
    __shared__ LevelLds l;
    const double W = levels_weight(T.t[blockIdx.x], l);
    if (threadIdx.x == 0) {
        const unsigned bad = !(W > 0.0) || isinf(W) ? ST_ZERO_TOTAL : 0u;
        if ((atomicOr(status, bad) | bad) & ST_ZERO_TOTAL) atomicOr(&cnt[CNT_STATUS], (unsigned long long)ST_ZERO_TOTAL);
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
        GraphTable &t = T.t[k];
        t.N = k == 0 ? h->n : h->m;
        t.w = k == 0 ? nullptr : h->w;
        t.deg = deg;
        t.dx = (double *)(sc + L.dx[k]);
        t.idx = (uint32_t *)(sc + L.idx[k]);
        t.blk = (uint32_t *)(sc + L.blk[k]);
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
    hipLaunchKernelGGL(k_split_count<Tables>, dim3(g), blk, 0, s, T);
    hipLaunchKernelGGL(k_split_scan<Tables>, dim3(2), dim3(1024), 0, s, T);
    hipLaunchKernelGGL(k_split<Tables>, dim3(g), blk, 0, s, T);
    g = spread_halves(T, (long long)WAVE_CHUNKS * SCAN_CHUNK);
    hipLaunchKernelGGL(k_chain_dx, dim3(g), blk, 0, s, T);
    hipLaunchKernelGGL(k_levels_dx<Tables>, dim3(4), blk, 0, s, T);
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
    for (int v = 0; v < 256; ++v) h->heat_count[v] = host[CNT_HEAT + v];
    if (host[CNT_STATUS] & ST_ZERO_TOTAL) {
        // with at least one arc some out-degree is positive: it is the arcs' total
        h->neg_ready = true;
        return fail(h, LH_ERR_ZERO_WEIGHT, "total arc weight is zero");
    }
    h->neg_ready = h->edge_ready = true;
    choose_cfg(h);
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
    for (int v = 0; v < 256; ++v) h->heat_count[v] = 0;
    h->heat_count[0] = (unsigned long long)h->n;
    choose_cfg(h);
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
    // The documented limits; scratch_layout(2^21, 2^21) is 64.15 MiB, within the array.
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
