// Hogwild kernels over a range of sample indices, and their host launchers.  Each (dtype, orders)
// pair is instantiated in its own translation unit so the kernel variants compile in parallel.
#pragma once

#include <algorithm>
#include <cmath>

#include "tile.hpp"

namespace lh {

// Register budget of the one-graph kernel: at least 3 (binary32) or 5 (bfloat16) waves per
// SIMD.  The bfloat16 kernel is latency bound: 5 waves (96 registers, no spills) measured
// 2 % faster than 4 on both hub-heavy and large uniform tables, and 6 (with spills) slower.
// Both orders with several samples a wavefront, and one order with four units a lane or more, do not fit 96
// registers (the hot set is the same with 5 waves and with 3, 10,240 and 6,144 samples in flight or a power
// of two times that): what is spilled is read back in
// every round, and the wait for that also waits for the stores before it to be acknowledged.  With 4
// waves for one unit a lane and 3 for more, nothing is spilled up to four units; graphs without hubs, 5 waves and so:
// 40,000 nodes, 640,000 samples, d = 32 1.25 and 1.09 ms, d = 128 2.73 and 1.27, d = 256 7.0 and 1.93;
// 2^20 nodes, 10^6 samples, d = 128 2.34 and 1.34 (4 waves and 3 spilled registers 1.32); one order, four
// or eight units a lane, 300,000 nodes, 500,000 samples, d = 256 1.4 times as fast, d = 512 2.3 times.
// Fewer than 16 lanes keep 5: graphs with hubs, d = 64 on (8, 4), 3 waves take 1.12-1.17 of that time.
// First order with a wavefront a sample and up to five negatives: 80 registers suffice for 6, and the hot
// set stays.  With up to eight 6 would spill (2 registers) and enlarge the hot set, which follows the
// samples in flight: rows of 2^-13 to 2^-14 a sample are hot with 6,144 of them, not with 5,120.
template <typename TT, int LPS, int UPL, int KMAX, int ORD>
constexpr int hogwild_min_waves()
{
    if (sizeof(TT) == 4) return 3;
    if (ORD == 1 && LPS == 64 && UPL <= 2 && KMAX <= 5) return 6;
    return LPS < 64 && (ORD == 3 || (LPS >= 16 && UPL >= 4)) ? (UPL > 1 ? 3 : 4) : 5;
}

// SH: bfloat16 tables whose hot rows live in a binary32 shadow for the launch.  Each
// wavefront takes tiles of 2^tile_shift samples from the launch's tile counter (g.tiles, zero at
// launch) until none are left, so wavefronts that meet slow rows do not hold up a fixed share of
// the work and the grid is only as large as what is resident.  A launch with no more tiles than
// wavefronts has no counter (g.tiles NULL): wavefront t takes tile t.  With g.streams (binary32),
// 2^q_shift wavefronts share each of so many streams of 64-sample tiles (TileAt), tile t being a share of
// stream (t mod (streams 2^q_shift)) / 2^q_shift; a workgroup takes four tiles at a time, and its
// wavefronts keep step (sgd_tile).
// FULL: the tile shape covers a row exactly (lanes x units == the row's units) and K == KMAX,
// so row accesses need no bounds mask or slot test.
template <typename TT, int LPS, int UPL, int KMAX, int ORD, bool SH, bool FULL = false>
__global__ void __launch_bounds__(256, (hogwild_min_waves<TT, LPS, UPL, KMAX, ORD>())) k_hogwild(GraphDev g,
                                                                                           unsigned long long first,
                                                                                           unsigned long long end)
{
    const unsigned lane = threadIdx.x & 63u;
    __shared__ unsigned long long next;
    const unsigned streams = sizeof(TT) == 4 ? g.streams : 0u;
    const unsigned lap_waves = streams << g.q_shift;  // (a multiple of 4)
    const unsigned long long ntiles = streams ? g.laps * lap_waves : ((end - first - 1) >> g.tile_shift) + 1;
    unsigned long long t = blockIdx.x * 4u + (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    while (true) {
        if (g.tiles) {
            if (streams) {
                if (threadIdx.x == 0) next = atomicAdd(g.tiles, 1ull) * 4u;
                __syncthreads();
                t = next + (threadIdx.x >> 6);
                __syncthreads();
            } else {
                t = 0;
                if (lane == 0) t = atomicAdd(g.tiles, 1ull);
            }
            t = ((unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(t >> 32)) << 32) |
                (unsigned long long)(unsigned)__builtin_amdgcn_readfirstlane((int)(t & 0xffffffffull));
        }
        if (t >= ntiles) break;
        unsigned long long before = t << g.tile_shift;  // samples of the launch before the tile
        TileAt at{0, 0, 0, 0};
        if (streams) {
            constexpr int GS = __builtin_ctz(64 / LPS);
            const unsigned long long lap = t / lap_waves;
            const unsigned w = (unsigned)(t - lap * lap_waves), stream = w >> g.q_shift;
            at.q_shift = g.q_shift;
            at.apart = streams * 64u;
            // 2^tile_shift samples a wavefront: 2^(tile_shift + q_shift) of the stream a lap
            before = ((lap << (g.tile_shift + g.q_shift - 6)) * at.apart) + stream * 64u +
                     ((w & ((1u << g.q_shift) - 1u)) << GS);
        }
        at.first = first + before;
        at.left = before < end - first ? samples_left(end - first - before) : 0u;
        sgd_tile<TT, LPS, UPL, KMAX, ORD, SH, FULL>(g, at, g.tile_shift);
        if (!g.tiles) break;
    }
}

// Zero a launch's tile counter (a kernel, not a memset, so the launch can be captured).
template <int N>
__global__ void k_zero_tiles(unsigned long long *c)
{
    if (threadIdx.x < N) c[threadIdx.x] = 0ull;
}

// Resident workgroups of a kernel on the device (at least 1 per CU).
template <typename KernelT>
inline unsigned resident_blocks(KernelT kernel, int num_cu)
{
    int occ = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kernel, 256, 0) != hipSuccess || occ < 1) occ = 1;
    return (unsigned)num_cu * (unsigned)occ;
}

// Heat threshold for a launch whose rows are exposed to a window of W samples (those in
// flight, or unbounded for tables that fit in one L2): a row is hot when W p_r reaches
// hot_rate, i.e. when floor(-log2 p_r) <= floor(log2(W / hot_rate)).  hot_rate <= 0 makes
// every row hot, hot_rate >= 1e30 none.
inline int hot_heat_for(double W, double hot_rate)
{
    if (!(hot_rate > 0.0)) return 255;
    if (hot_rate >= 1e30 || !(W > 0.0)) return -1;
    if (std::isinf(W)) return 255;
    double t = std::floor(std::log2(W / hot_rate));
    if (t < -1.0) return -1;
    if (t > 255.0) return 255;
    return (int)t;
}

// (lanes per sample, units per lane) of the Hogwild kernels.
#define LH_CFG_LIST(X) \
    X(16, 1)           \
    X(32, 1)           \
    X(64, 1)           \
    X(16, 2)           \
    X(32, 2)           \
    X(64, 2)           \
    X(2, 4)            \
    X(4, 4)            \
    X(8, 4)            \
    X(16, 4)           \
    X(32, 4)           \
    X(64, 4)           \
    X(4, 8)            \
    X(8, 8)            \
    X(16, 8)           \
    X(32, 8)           \
    X(64, 8)

// The grid and the tiles of one Hogwild launch over `count` samples (at least 1) and the samples
// it keeps in flight: the configuration's grid, lowered if the staleness cap asks for fewer.
//
// Tiles have 64 samples, one per lane of phase A; a launch of fewer than kTilesWanted such tiles (two
// wavefronts to a compute unit) takes smaller ones, down to four rounds of phase B (below that phase A,
// which costs the same for any number of samples, is most of a tile's time).  Smaller tiles up to every
// wavefront that may be in flight pay for phase A more often and meet more hot rows: 300,000 nodes,
// d = 128, bfloat16, 65,536 samples 109 us with 1,024 tiles of 64, 146 with 4,096 of 16; at 8,192
// samples 512 tiles of 16 take 31 us, 128 of 64 80, and 256 of 32 45.
//
// Teams (team: wavefronts to a stream, 1: none): four_unit_lanes says why.
constexpr unsigned kTilesWanted = 512;

struct HogwildPlan {
    unsigned grid = 1, streams = 0;
    int tile_shift = 6, q_shift = 0;
    unsigned long long laps = 0;
    bool counter = true;  // more tiles than wavefronts
    double in_flight = 0.0;
};

template <typename KernelT>
inline HogwildPlan plan_launch(KernelT kern, int lps, int team, const GraphDev &g, const TileCfg &c,
                               unsigned long long count, int num_cu)
{
    HogwildPlan p;
    const unsigned resident = resident_blocks(kern, num_cu);
    unsigned most_blocks = std::min((unsigned)num_cu * (unsigned)(c.blocks_per_cu > 0 ? c.blocks_per_cu : 8), resident);
    const double per_block = 4.0 * (64.0 / lps);
    const double most = g.max_in_flight;
    if (team > 1) {
        // streams as the narrow shape has wavefronts: four of its workgroups' at a time
        unsigned sets = std::max(1u, most_blocks / (unsigned)team);
        if (most > 0.0) sets = std::min(sets, (unsigned)std::max(1.0, std::floor(std::min(most / (per_block * team), 1e9))));
        const unsigned long long tiles = ((count - 1) >> 6) + 1;
        p.streams = (unsigned)std::min<unsigned long long>(4ull * sets, tiles);
        p.q_shift = __builtin_ctz((unsigned)team);
        // tiles of the stream that a wavefront draws its share of at a time: two, so that a team that
        // lags does so by few samples (10,000 nodes, d = 16: four 5.8 ms, ending 1.6 times as far from
        // the narrow shape as its own runs from each other; two 6.7 ms and 1.3 times; one 9.4 ms)
        const int m = 2ull * p.streams <= tiles ? 1 : 0;
        p.tile_shift = 6 - p.q_shift + m;
        p.laps = (tiles - 1) / ((unsigned long long)p.streams << m) + 1;
        if (team == 2) p.streams += p.streams & 1u;  // whole workgroups
        const unsigned waves = p.streams << p.q_shift;
        p.grid = waves / 4;
        p.counter = p.laps > 1;
        p.in_flight = (double)waves * (64 / lps);
        return p;
    }
    if (most > 0.0) most_blocks = std::min(most_blocks, (unsigned)std::max(1.0, std::floor(std::min(most / per_block, 1e9))));
    const int gpw_shift = 6 - __builtin_ctz((unsigned)lps);
    const int least = std::min(6, gpw_shift + 2);
    const unsigned long long fill = std::min(4ull * most_blocks, (unsigned long long)kTilesWanted);
    while (p.tile_shift > least && ((count - 1) >> p.tile_shift) + 1 < fill) --p.tile_shift;
    const unsigned long long tiles = ((count - 1) >> p.tile_shift) + 1;
    p.grid = (unsigned)std::min<unsigned long long>(most_blocks, (tiles + 3) / 4);
    p.counter = tiles > 4ull * p.grid;
    p.in_flight = (double)std::min(p.grid, resident) * per_block;
    return p;
}

// The samples in flight that hot rows are chosen by: the launch's, or those that four units a lane would
// have (a tile of 64 samples a wavefront), if more.
inline double hot_window(const GraphDev &g, const HogwildPlan &p, unsigned long long count)
{
    if (!(g.narrow_flight > p.in_flight)) return p.in_flight;
    const double tiles = (double)(((count - 1) >> 8) + 1) * 4.0;  // (whole workgroups)
    return std::max(p.in_flight, std::min(g.narrow_flight, tiles * (64 / four_unit_lanes(g.nunits))));
}

// Samples in flight on the hottest row from which context rows are loaded one at a time.
constexpr double kPacedQueue = 128.0;

// Whether a bfloat16 launch with more than five negatives and one unit a lane waits for each context row
// before it loads the next.  With this many samples in flight wanting the graph's hottest row (by its heat,
// a whole power of two), memory is busy with the queue for it, and loads that are in flight together only
// lengthen it; otherwise rows in flight together take less time.  400,000 nodes, d = 32, both orders, six
// negatives, 10^6 samples, together and one at a time: 177 samples on the hottest row 1.91 and 1.69 ms, 93
// 1.02 and 1.21.  (Five negatives or fewer: rows together.)
template <typename TT>
inline bool paced_loads(const GraphDev &g, const TileCfg &c, const HogwildPlan &p)
{
    if (sizeof(TT) != 2 || !g.heat_count || c.upl != 1) return false;
    int v = 0;
    while (v < 255 && !g.heat_count[v]) ++v;
    return p.in_flight * std::exp2(-(v + 0.5)) > kPacedQueue;
}

// One Hogwild launch with the heat threshold for its concurrency.  With a shadow context
// (bfloat16 tables) the hot rows move into the binary32 shadow for the launch and back
// afterwards; without one no row is read from a shadow.
template <typename TT, typename KernelT>
hipError_t launch_one(KernelT kern, int lps, int team, const GraphDev &g, const TileCfg &c, unsigned long long first,
                      unsigned long long end, int num_cu, const ShadowCtx *sc, hipStream_t s)
{
    const HogwildPlan p = plan_launch(kern, lps, team, g, c, end - first, num_cu);
    GraphDev gl = g;
    gl.hot_heat = hot_heat_for(hot_window(g, p, end - first) + g.resid, g.hot_rate);
    gl.paced = paced_loads<TT>(g, c, p);
    gl.tile_shift = p.tile_shift;
    gl.streams = p.streams;
    gl.q_shift = p.q_shift;
    gl.laps = p.laps;
    if (sc) {
        hipError_t e = shadow_begin(*sc, gl.hot_heat, s);
        if (e != hipSuccess) return e;
    } else {
        gl.slot = nullptr;
    }
    if (!gl.tiles) return hipErrorInvalidValue;
    if (p.counter) hipLaunchKernelGGL(k_zero_tiles<1>, dim3(1), dim3(64), 0, s, gl.tiles);
    else gl.tiles = nullptr;
    hipLaunchKernelGGL(kern, dim3(p.grid), dim3(256), 0, s, gl, first, end);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && sc) e = shadow_end(*sc, gl.hot_heat, first, s);
    return e;
}

// Wavefronts to a stream of a launch (1: no teams): binary32 tables that fit in one L2, a shape that
// was not pinned, and more lanes a sample than four units a lane need.
template <typename TT>
inline int team_waves(const GraphDev &g, const TileCfg &c)
{
    if (sizeof(TT) != 4 || !g.teams || !std::isinf(g.resid)) return 1;
    const int narrow = four_unit_lanes(g.nunits);
    return c.lps > narrow ? c.lps / narrow : 1;
}

// Samples a Hogwild launch of `count` samples would keep in flight (0: no such kernel);
// g.slot set means the kernel with the binary32 shadow (bfloat16 only).
template <typename TT, int ORD, bool SH>
double hogwild_in_flight_sh(const GraphDev &g, const TileCfg &c, unsigned long long count, int num_cu)
{
    const int team = team_waves<TT>(g, c);
#define LH_PLAN_H(L, C)                                                                                  \
    if (c.lps == L && c.upl == C) {                                                                      \
        if (!SH && g.K == 5 && L * C == g.nunits)                                                        \
            return plan_launch(k_hogwild<TT, L, C, 5, ORD, false, true>, L, team, g, c, count, num_cu).in_flight; \
        return plan_launch(g.K <= 5 ? k_hogwild<TT, L, C, 5, ORD, SH> : k_hogwild<TT, L, C, 8, ORD, SH>, L, team, g, c, \
                           count, num_cu).in_flight;                                                     \
    }
    LH_CFG_LIST(LH_PLAN_H)
#undef LH_PLAN_H
    return 0.0;
}

template <typename TT, int ORD>
double hogwild_in_flight_t(const GraphDev &g, const TileCfg &c, unsigned long long count, int num_cu)
{
    if constexpr (sizeof(TT) == 2)
        if (g.slot) return hogwild_in_flight_sh<TT, ORD, true>(g, c, count, num_cu);
    return hogwild_in_flight_sh<TT, ORD, false>(g, c, count, num_cu);
}

template <typename TT, int ORD, bool SH>
hipError_t launch_hogwild_sh(const GraphDev &g, const TileCfg &c, unsigned long long first, unsigned long long end,
                             int num_cu, const ShadowCtx *sc, hipStream_t s)
{
    const bool k5 = g.K <= 5;
    const int team = team_waves<TT>(g, c);
#define LH_LAUNCH_H(L, C)                                                                        \
    if (c.lps == L && c.upl == C) {                                                              \
        if (!SH && g.K == 5 && L * C == g.nunits)                                                \
            return launch_one<TT>(k_hogwild<TT, L, C, 5, ORD, false, true>, L, team, g, c, first, end, num_cu, sc, s); \
        if (k5) return launch_one<TT>(k_hogwild<TT, L, C, 5, ORD, SH>, L, team, g, c, first, end, num_cu, sc, s); \
        return launch_one<TT>(k_hogwild<TT, L, C, 8, ORD, SH>, L, team, g, c, first, end, num_cu, sc, s);        \
    }
    LH_CFG_LIST(LH_LAUNCH_H)
#undef LH_LAUNCH_H
    return hipErrorInvalidConfiguration;
}

// A shadow context selects the kernel built with the shadow path (bfloat16 only).
template <typename TT, int ORD>
hipError_t launch_hogwild_t(const GraphDev &g, const TileCfg &c, unsigned long long first, unsigned long long end,
                            int num_cu, const ShadowCtx *sc, hipStream_t s)
{
    if constexpr (sizeof(TT) == 2)
        if (sc) return launch_hogwild_sh<TT, ORD, true>(g, c, first, end, num_cu, sc, s);
    return launch_hogwild_sh<TT, ORD, false>(g, c, first, end, num_cu, nullptr, s);
}

// Explicit instantiations live in sgd_<dtype>_o<orders>.hip.
#define LH_DECLARE_LAUNCHERS(TT, ORD)                                                                          \
    extern template hipError_t launch_hogwild_t<TT, ORD>(const GraphDev &, const TileCfg &, unsigned long long, \
                                                         unsigned long long, int, const ShadowCtx *, hipStream_t); \
    extern template double hogwild_in_flight_t<TT, ORD>(const GraphDev &, const TileCfg &, unsigned long long, int);

#define LH_DEFINE_LAUNCHERS(TT, ORD)                                                                    \
    template hipError_t launch_hogwild_t<TT, ORD>(const GraphDev &, const TileCfg &, unsigned long long, \
                                                  unsigned long long, int, const ShadowCtx *, hipStream_t); \
    template double hogwild_in_flight_t<TT, ORD>(const GraphDev &, const TileCfg &, unsigned long long, int);

}  // namespace lh
