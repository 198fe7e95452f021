// Stable LSD radix sort of 32-bit keys with one or two 32-bit payloads, for the SNAPSHOT entries
// and the walk graph's rows.
//
// A pass takes up to 8 bits: digit counts per tile of 4,096 items, their prefix sums (digit by
// digit, tiles in order), then the scatter.  In the scatter a wavefront holds 1,024 consecutive
// items, 64 at a time; the lanes with an equal digit find each other by one ballot per bit, so an
// item's place is its digit's running count plus the equal lanes before it, and equal keys keep
// their order.  The tile is put in order in LDS first, so that each digit's run is written to
// consecutive addresses.
//
// What bounds a pass is memory: 33.6 M items with two payloads move 0.13 GB for the counts and
// 0.8 GB for the scatter.  Four-bit passes with a thread per 16 consecutive items (uncoalesced reads
// and writes, and a scan of 256 threads' counters by 16 lanes) took 1.28 ms each.
#pragma once

#include "common.hpp"

namespace lh {

constexpr int SORT_THREADS = 256, SORT_ITEMS = 16, SORT_TILE = SORT_THREADS * SORT_ITEMS;
constexpr int SORT_MAX_BITS = 8, SORT_MAX_DIGITS = 1 << SORT_MAX_BITS;

// Digit counters of a sort of E items, and the totals of their scan's parts.
static inline long long sort_hist_size(long long E) { return SORT_MAX_DIGITS * LH_CDIV(E > 0 ? E : 1, SORT_TILE); }
static inline long long sort_part_size(long long E) { return LH_CDIV(sort_hist_size(E), SORT_TILE) + 1; }

// Lanes of the wavefront whose digit equals this lane's (valid lanes only).
template <int BITS>
__device__ __forceinline__ unsigned long long equal_lanes(unsigned digit, bool valid)
{
    unsigned long long m = __ballot(valid);
#pragma unroll
    for (int b = 0; b < BITS; ++b) {
        const bool bit = (digit >> b) & 1u;
        const unsigned long long x = __ballot(bit);
        m &= bit ? x : ~x;
    }
    return m;
}

// In: key(i), and pay(i, 0), pay(i, 1) of the first PAY payloads.
template <int BITS, class In>
__global__ void __launch_bounds__(SORT_THREADS) k_sort_count(In in, unsigned long long E, int shift, uint32_t *hist,
                                                             unsigned ntiles)
{
    constexpr int D = 1 << BITS;
    __shared__ uint32_t cnt[4][D];
    for (int i = threadIdx.x; i < 4 * D; i += SORT_THREADS) (&cnt[0][0])[i] = 0u;
    __syncthreads();
    const unsigned long long base = (unsigned long long)blockIdx.x * SORT_TILE;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int s = 0; s < SORT_ITEMS; ++s) {
        const unsigned long long i = base + s * SORT_THREADS + threadIdx.x;
        const bool ok = i < E;
        const int d = ok ? (int)((in.key(i) >> shift) & (D - 1)) : -1;
        // (a run of equal digits counts once: its lanes would take the counter one at a time)
        const int before = __shfl_up(d, 1);
        const unsigned long long heads = __ballot(ok && (lane == 0 || before != d));
        const int nvalid = __popcll(__ballot(ok));
        if ((heads >> lane) & 1ull) {
            const unsigned long long above = lane == 63 ? 0ull : heads & (~0ull << (lane + 1));
            atomicAdd(&cnt[wave][d], (uint32_t)((above ? __ffsll((long long)above) - 1 : nvalid) - lane));
        }
    }
    __syncthreads();
    for (int d = threadIdx.x; d < D; d += SORT_THREADS)
        hist[(unsigned long long)d * ntiles + blockIdx.x] = cnt[0][d] + cnt[1][d] + cnt[2][d] + cnt[3][d];
}

// Exclusive prefix sums of 4,096 counters per workgroup, in place; the workgroup's total to part.
static __global__ void __launch_bounds__(SORT_THREADS) k_sort_scan(uint32_t *x, unsigned long long n, uint32_t *part)
{
    __shared__ uint32_t ws[4];
    const unsigned long long lo = (unsigned long long)blockIdx.x * SORT_TILE + threadIdx.x * SORT_ITEMS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t v[SORT_ITEMS], s = 0u;
#pragma unroll
    for (int k = 0; k < SORT_ITEMS; ++k) v[k] = lo + k < n ? x[lo + k] : 0u;
#pragma unroll
    for (int k = 0; k < SORT_ITEMS; ++k) s += v[k];
    uint32_t inc = s;
    for (int d = 1; d < 64; d <<= 1) {
        const uint32_t y = __shfl_up(inc, d);
        if (lane >= d) inc += y;
    }
    if (lane == 63) ws[wave] = inc;
    __syncthreads();
    uint32_t run = inc - s;
    for (int w = 0; w < wave; ++w) run += ws[w];
#pragma unroll
    for (int k = 0; k < SORT_ITEMS; ++k) {
        if (lo + k < n) x[lo + k] = run;
        run += v[k];
    }
    if (threadIdx.x == SORT_THREADS - 1) part[blockIdx.x] = run;
}

// Exclusive prefix sums of the parts, in place, by one workgroup of 1,024 threads.
static __global__ void __launch_bounds__(1024) k_sort_parts(uint32_t *part, unsigned n)
{
    __shared__ uint32_t ws[16];
    __shared__ uint32_t carry;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (threadIdx.x == 0) carry = 0u;
    __syncthreads();
    for (unsigned i0 = 0; i0 < n; i0 += 1024) {
        const unsigned i = i0 + threadIdx.x;
        const uint32_t v = i < n ? part[i] : 0u;
        uint32_t inc = v;
        for (int d = 1; d < 64; d <<= 1) {
            const uint32_t y = __shfl_up(inc, d);
            if (lane >= d) inc += y;
        }
        if (lane == 63) ws[wave] = inc;
        __syncthreads();
        uint32_t run = carry + inc - v;
        for (int w = 0; w < wave; ++w) run += ws[w];
        if (i < n) part[i] = run;
        __syncthreads();
        if (threadIdx.x == 1023) carry = run + v;
        __syncthreads();
    }
}

template <int BITS, class In>
__global__ void __launch_bounds__(SORT_THREADS) k_sort_scatter(In in, unsigned long long E, int shift,
                                                               const uint32_t *hist, const uint32_t *part,
                                                               unsigned ntiles, uint32_t *kout, uint32_t *out0,
                                                               uint32_t *out1)
{
    constexpr int D = 1 << BITS;
    __shared__ volatile uint32_t run[4][D];  // a wavefront's running counts, then its offset in the digit
    __shared__ uint32_t first[D];            // the digit's first place in the ordered tile
    __shared__ uint32_t dest[D];             // where the digit's run goes, less that place
    __shared__ uint32_t ws[4];
    __shared__ uint32_t sk[SORT_TILE], s0[SORT_TILE], s1[In::PAY > 1 ? SORT_TILE : 1];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const unsigned long long base = (unsigned long long)blockIdx.x * SORT_TILE;
    for (int i = threadIdx.x; i < 4 * D; i += SORT_THREADS) (&run[0][0])[i] = 0u;
    uint32_t key[SORT_ITEMS], p0[SORT_ITEMS], p1[SORT_ITEMS];
    const unsigned long long i0 = base + wave * (SORT_ITEMS * 64) + lane;
#pragma unroll
    for (int s = 0; s < SORT_ITEMS; ++s) {
        const unsigned long long i = i0 + s * 64 < E ? i0 + s * 64 : E - 1;
        key[s] = in.key(i);
        p0[s] = in.pay(i, 0);
        p1[s] = In::PAY > 1 ? in.pay(i, 1) : 0u;
    }
    __syncthreads();
    uint32_t rank[SORT_ITEMS];
#pragma unroll
    for (int s = 0; s < SORT_ITEMS; ++s) {
        const bool ok = i0 + s * 64 < E;
        const unsigned d = (key[s] >> shift) & (D - 1);
        const unsigned long long same = equal_lanes<BITS>(d, ok);
        const int before = __popcll(same & ((1ull << lane) - 1ull));
        const uint32_t c = ok ? run[wave][d] : 0u;
        rank[s] = c + (uint32_t)before;
        if (ok && before == 0) run[wave][d] = c + (uint32_t)__popcll(same);
    }
    __syncthreads();
    {
        // thread d: the digit's wavefronts, its count, and the counts of the digits before it
        const int d = threadIdx.x;
        uint32_t c = 0u;
        if (d < D)
            for (int w = 0; w < 4; ++w) {
                const uint32_t x = run[w][d];
                run[w][d] = c;
                c += x;
            }
        uint32_t inc = c;
        for (int k = 1; k < 64; k <<= 1) {
            const uint32_t y = __shfl_up(inc, k);
            if (lane >= k) inc += y;
        }
        if (lane == 63) ws[wave] = inc;
        __syncthreads();
        uint32_t at = inc - c;
        for (int w = 0; w < wave; ++w) at += ws[w];
        if (d < D) {
            const unsigned long long h = (unsigned long long)d * ntiles + blockIdx.x;
            first[d] = at;
            dest[d] = hist[h] + part[h / SORT_TILE] - at;
        }
    }
    __syncthreads();
#pragma unroll
    for (int s = 0; s < SORT_ITEMS; ++s)
        if (i0 + s * 64 < E) {
            const unsigned d = (key[s] >> shift) & (D - 1);
            const uint32_t at = first[d] + run[wave][d] + rank[s];
            sk[at] = key[s];
            s0[at] = p0[s];
            if constexpr (In::PAY > 1) s1[at] = p1[s];
        }
    __syncthreads();
    const int len = (int)(E - base < SORT_TILE ? E - base : SORT_TILE);
    for (int i = threadIdx.x; i < len; i += SORT_THREADS) {
        const uint32_t k = sk[i];
        const uint32_t pos = dest[(k >> shift) & (D - 1)] + (uint32_t)i;
        kout[pos] = k;
        out0[pos] = s0[i];
        if constexpr (In::PAY > 1) out1[pos] = s1[i];
    }
}

// Keys and payloads in arrays; index: the payload of the first pass is the item's index.
template <int N>
struct SortArrays {
    static constexpr int PAY = N;
    const uint32_t *k, *p0, *p1;
    bool index;
    __device__ __forceinline__ uint32_t key(unsigned long long i) const { return k[i]; }
    __device__ __forceinline__ uint32_t pay(unsigned long long i, int which) const
    {
        if (which) return p1[i];
        return index ? (uint32_t)i : p0[i];
    }
};

struct SortBuffers {
    uint32_t *k, *p0, *p1;
};

template <int BITS, class In>
static void sort_pass(const In &in, long long E, int shift, const SortBuffers &out, uint32_t *hist, uint32_t *part,
                      hipStream_t s)
{
    const unsigned nt = (unsigned)LH_CDIV(E, SORT_TILE);
    const unsigned long long n = (unsigned long long)nt << BITS;
    const unsigned np = (unsigned)LH_CDIV(n, SORT_TILE);
    hipLaunchKernelGGL((k_sort_count<BITS, In>), dim3(nt), dim3(SORT_THREADS), 0, s, in, (unsigned long long)E, shift, hist, nt);
    hipLaunchKernelGGL(k_sort_scan, dim3(np), dim3(SORT_THREADS), 0, s, hist, n, part);
    hipLaunchKernelGGL(k_sort_parts, dim3(1), dim3(1024), 0, s, part, np);
    hipLaunchKernelGGL((k_sort_scatter<BITS, In>), dim3(nt), dim3(SORT_THREADS), 0, s, in, (unsigned long long)E, shift,
                       hist, part, nt, out.k, out.p0, out.p1);
}

template <class In>
static void sort_pass_bits(int bits, const In &in, long long E, int shift, const SortBuffers &out, uint32_t *hist,
                           uint32_t *part, hipStream_t s)
{
    if (bits <= 5) sort_pass<5>(in, E, shift, out, hist, part, s);
    else if (bits == 6) sort_pass<6>(in, E, shift, out, hist, part, s);
    else if (bits == 7) sort_pass<7>(in, E, shift, out, hist, part, s);
    else sort_pass<8>(in, E, shift, out, hist, part, s);
}

// Sort E items (1 <= E < 2^32) by the low `bits` bits (at least 1) of their keys, in passes of
// about equal width.  The first pass reads `in`; a and b are the buffers that the passes write to
// in turn, b first, and the result's are returned.  hist, part: sort_hist_size(E) and
// sort_part_size(E) words.
template <class In>
static SortBuffers radix_sort(const In &in, long long E, int bits, const SortBuffers &a, const SortBuffers &b,
                              uint32_t *hist, uint32_t *part, hipStream_t s)
{
    const int passes = (bits + SORT_MAX_BITS - 1) / SORT_MAX_BITS;
    SortBuffers from = a, to = b;
    for (int p = 0, shift = 0; p < passes; ++p) {
        const int left = passes - p, w = (bits - shift + left - 1) / left;
        if (p == 0)
            sort_pass_bits(w, in, E, shift, to, hist, part, s);
        else
            sort_pass_bits(w, SortArrays<In::PAY>{from.k, from.p0, from.p1, false}, E, shift, to, hist, part, s);
        shift += w;
        const SortBuffers t = from;
        from = to;
        to = t;
    }
    return from;
}

}  // namespace lh
