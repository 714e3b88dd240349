// Choice and launch of the D2Q9 tile passes (tile2d.hpp).
#pragma once

#include <algorithm>
#include <cstring>
#include <utility>
#include <vector>

#include "step_launch.hpp"
#include "tile2d.hpp"

namespace ptrt {

// Steps of a call of ptrt_step or ptrt_batch_step from which on it takes
// tile passes; shorter calls keep the one- and two-step passes, whose kinds
// ptrt_last_pass documents.
constexpr int TILE_MIN_STEPS = 8;

enum { TILE_NONE = -1, TILE_A = 0, TILE_B = 1, TILE_C = 2, TILE_D = 3, TILE_SHAPES = 4 };

// f(SH{}) for a shape id.
template <class F>
inline void with_tile_shape(int shape, F &&f)
{
    if (shape == TILE_A) f(TileA{});
    else if (shape == TILE_B) f(TileB{});
    else if (shape == TILE_C) f(TileC{});
    else if (shape == TILE_D) f(TileD{});
}

struct TilePlan {
    int shape = TILE_NONE; // none: no tile passes on this lattice
    bool thin = false;     // not against passes of two steps (few rows, below)
    int T = 0;             // steps of a full pass
    int cw = 0, ch = 0;    // core of a single lattice's tiles
    int tiles_x = 0, tiles = 0;
};

// Near-equal cores of at most `most` nodes along an axis of n nodes.
inline int tile_core(int n, int most)
{
    const int parts = (n + most - 1) / most;
    return (n + parts - 1) / parts;
}

// The shape and the steps per pass with the least estimated time per step
// for the lattices of one launch, or none where the passes of one and two
// steps are estimated faster.
//
// A tile pass costs a launch (c0) and rounds of the workgroups a CU holds: a
// round takes its issue time (rows of 64 nodes over all steps, q each, and
// mem for the first step's loads), or the dependent chain of one workgroup
// (lat per iteration of its waves, plus beta of its own issue time) if that
// is longer; the bytes it moves add their time at bw. The constants are
// those that choose best among the shapes with T = 3 ... 8 timed on fourteen
// lattices and batches (64^2 ... 4096^2, FP32 and FP64): the fastest pass at
// twelve, within 6 % (700^2) and 2 % of it at the others. The earlier passes
// take about 2 us a launch and run at 113 (FP32), 64 (FP64) and 180 (16
// bits) nodes a ns over rows padded to whole strips.  The 16 bits have not
// been fitted so, and Scheme I and open x use the default forcing's
// constants: timed on thirteen lattices of 97 x 31 to 4096^2, the passes
// chosen gained over the earlier ones 1.14 to 2.92 times in FP16 and BF16 (least at
// 2048^2), 1.08 to 3.0 with Scheme I, open x or walls in FP16, 1.5 to 3.6 in
// FP32 and FP64. For stochastic rounding on large lattices the earlier passes
// stay the faster ones: its nine rounded stores double the issue time (2048^2
// FP16 23 us against 38).
//
// Lattices of few rows: a tile is mostly halo, and both estimates are off by
// up to a quarter, so that long ones take tile passes only if these are
// estimated faster by more than that (earlier -> tile passes, us a step:
// 10000 x 1 FP32 2.08 -> 1.01, 10000 x 3 FP64 3.01 -> 1.40, 70000 x 4 FP32
// 1.7 times faster, 1000000 x 8 FP32 2.0 times; but 100000 x 2 FP32 3.19 ->
// 4.07, 100000 x 3 FP64 5.65 -> 7.81, 1000000 x 6 FP16 34.0 -> 46.9, 1000
// lattices of 200 x 4 and 5 FP64 14.9 -> 18.2). In 16 bits a batch's earlier
// pass is slower and the tile passes gain there (13.1 -> 10.7), so that only
// long rows count.  With Scheme I, and with open x below 2^20 nodes, the
// earlier pass of 32 and 64 bits is one of a single step, and the tile passes
// gain as estimated (100000 x 5 with open x FP32 7.98 -> 5.20, FP64 12.8 ->
// 9.5): TilePlan::thin marks a plan that is for these only.
inline TilePlan choose_tile_plan(int storage, const std::vector<std::pair<int, int>> &sizes)
{
    const size_t elem = storage_bytes(storage);
    const bool f64 = elem == 8, sr = storage == PTRT_F16_SR || storage == PTRT_BF16_SR;
    const bool half = elem == 2;
    const double c0 = f64 ? 3.5 : (half ? 3.0 : 2.5), lat = f64 ? 0.3 : (half ? 0.2 : 0.15),
                 q = f64 ? 0.045 : (sr ? 0.08 : (half ? 0.04 : 0.03)),
                 mem = half ? 0.5 : 0.0, bw = f64 ? 10e6 : (half ? 15e6 : 5e6),
                 beta = f64 || half ? 0.8 : 0.4; // us, bytes per us
    const double earlier_rate = f64 ? 64e3 : (elem == 4 ? 113e3 : 180e3); // nodes per us
    const int strip = elem == 2 ? 64 : Step2Shape2D<float>::BX;
    const int waves_per_cu = f64 || sr ? 16 : 32;
    constexpr long long CUS = 256;
    double nodes = 0.0, padded = 0.0;
    for (const auto &n : sizes) {
        nodes += (double)n.first * n.second;
        padded += (double)((n.first + strip - 1) / strip * strip) * n.second;
    }
    double thin = 0.0, columns = 0.0; // of the lattices of few rows
    int rows = 0;
    for (const auto &n : sizes) {
        rows = std::max(rows, n.second);
        if (n.second >= (half ? 12 : 6) || (half && n.first < 50000)) continue;
        thin += (double)n.first * n.second;
        columns += n.first;
    }
    const bool few_rows =
        columns > (half && rows > 1 ? 99999.0 : 50000.0) && thin > (f64 ? 0.5 : 0.75) * nodes;
    TilePlan best;
    const double earlier = 2.0 + padded / earlier_rate;
    double best_cost = earlier;
    for (int shape = 0; shape < TILE_SHAPES; ++shape) {
        with_tile_shape(shape, [&](auto sh) {
            using SH = decltype(sh);
            const int lds = (int)(SH::elems * elem) + 2 * SH::W * SH::H;
            const int occ = std::min(163840 / lds, waves_per_cu / SH::NW);
            if (occ < 1) return;
            for (int T = 3; T <= 8; ++T) {
                const int mw = SH::W - 2 * (T - 1), mh = SH::H - 2 * (T - 1);
                if (mw < 1 || mh < 1) break;
                long long tiles = 0;
                double wave_rows = 0.0, region = 0.0;
                int chain = 0;
                for (const auto &n : sizes) {
                    const int cw = tile_core(n.first, mw), ch = tile_core(n.second, mh);
                    const long long k = (long long)((n.first + cw - 1) / cw) * ((n.second + ch - 1) / ch);
                    int rows64 = 0, its = 0;
                    for (int s = 0; s < T; ++s) {
                        const int wr = ((ch + 2 * (T - 1 - s)) * SH::W + 63) / 64;
                        rows64 += wr;
                        its += (wr + SH::NW - 1) / SH::NW;
                    }
                    tiles += k;
                    wave_rows += (double)k * rows64;
                    region += (double)k * (cw + 2 * (T - 1)) * (ch + 2 * (T - 1));
                    chain = std::max(chain, its);
                }
                // a launch has fewer than 2^32 threads (rows of hundreds of
                // millions of nodes, few of them)
                if (tiles * 64 * SH::NW >= 1LL << 32) continue;
                const double issue = wave_rows / (double)tiles * q, alone = chain * lat + beta * issue;
                const long long per_cu = (tiles + CUS - 1) / CUS, rounds = (per_cu + occ - 1) / occ;
                const long long last = per_cu - (rounds - 1) * occ;
                const double us = c0 + (double)(rounds - 1) * std::max(alone, occ * issue + mem) +
                                  std::max(alone, (double)last * issue + mem) +
                                  9.0 * (double)elem * (nodes + region) / bw;
                const double cost = us / T;
                if (cost < best_cost) {
                    best_cost = cost;
                    best.shape = shape;
                    best.T = T;
                    best.cw = mw;
                    best.ch = mh;
                }
            }
        });
    }
    best.thin = few_rows && best_cost > earlier * (f64 ? 0.75 : 0.8);
    return best;
}

// The steps of tile pass j of k that share m steps.
inline int tile_pass_steps(int m, int k, int j)
{
    return (int)((long long)m * (j + 1) / k - (long long)m * j / k);
}

// Calls that run in tile passes: all but the last one or two of n steps are
// shared out over the fewest passes of at most plan.T steps, an even call
// ends with a pass of two steps and an odd one with a single step (returned
// as the steps left), so that ptrt_last_pass sees what it documents.
template <class F>
inline int tile_passes(const TilePlan &plan, int n, F &&pass)
{
    const int tail = 2 - (n & 1), m = n - tail, k = (m + plan.T - 1) / plan.T;
    for (int j = 0; j < k; ++j) pass(tile_pass_steps(m, k, j));
    if (tail == 1) return 1;
    pass(2);
    return 0;
}

// Which of the tiles of a row of tiles a solid may be in reach of: the hull
// of the solid columns of the rows in reach.
class SolidReach {
public:
    SolidReach(const uint8_t *mask, int nx, int ny) : nx_(nx), ny_(ny), lo_(ny, nx), hi_(ny, -1)
    {
        for (int y = 0; y < ny; ++y) {
            const uint8_t *row = mask + (size_t)y * nx;
            const void *first = std::memchr(row, 1, nx); // masks hold 0 and 1
            if (!first) continue;
            lo_[y] = (int)((const uint8_t *)first - row);
            for (hi_[y] = nx - 1; row[hi_[y]] == 0;) --hi_[y];
        }
    }
    // take the rows y0 ... y1 - 1 (periodic)
    void rows(int y0, int y1)
    {
        left_ = nx_;
        right_ = -1;
        for (int k = 0; k < std::min(y1 - y0, ny_); ++k) {
            const int y = ((y0 + k) % ny_ + ny_) % ny_;
            left_ = std::min(left_, lo_[y]);
            right_ = std::max(right_, hi_[y]);
        }
    }
    // columns x0 ... x1 - 1 (periodic) of those rows meet their solids' hull
    bool any(int x0, int x1) const
    {
        if (right_ < 0) return false;
        if (x1 - x0 >= nx_) return true;
        for (int shift = -nx_; shift <= nx_; shift += nx_)
            if (x0 + shift <= right_ && x1 - 1 + shift >= left_) return true;
        return false;
    }

private:
    int nx_, ny_, left_ = 0, right_ = -1;
    std::vector<int> lo_, hi_;
};

// One tile pass of T steps (src -> dst of `a`) over a single lattice;
// special: per tile, null without solids and open boundaries.
template <class S>
void launch_tile(const StepLaunch &a, const TilePlan &plan, const uint8_t *special, int T);
template <class S>
void launch_tile_batch(const void *src, void *dst, const uint8_t *mask, const uint8_t *near, const void *inst,
                       const int4 *tasks, int ntasks, int shape, int T, hipStream_t stream);

// Definitions, for the translation units that instantiate them.
template <class S>
void launch_tile_impl(const StepLaunch &a, const TilePlan &plan, const uint8_t *special, int T)
{
    using C = typename Codec<S>::compute;
    const Coef<D2Q9, C> r = make_coef<D2Q9, C>(a.tau_plus, a.Lambda, a.force);
    with_tile_shape(plan.shape, [&](auto sh) {
        using SH = decltype(sh);
        auto go = [&](auto fc, auto oc) {
            hipLaunchKernelGGL((k_tile_2d<S, SH, decltype(fc)::value, decltype(oc)::value>),
                               dim3(plan.tiles), dim3(64 * SH::NW), 0, a.stream, (const S *)a.src,
                               (S *)a.dst, a.mask, a.near, special, a.g, r, T, plan.cw, plan.ch, plan.tiles_x);
        };
        using II = std::integral_constant<int, FORCE_II>;
        using GUO = std::integral_constant<int, FORCE_GUO>;
        if (a.forcing == FORCE_GUO) go(GUO{}, std::false_type{});
        else if (a.open) go(II{}, std::true_type{});
        else go(II{}, std::false_type{});
    });
}

template <class S>
void launch_tile_batch_impl(const void *src, void *dst, const uint8_t *mask, const uint8_t *near, const void *inst,
                            const int4 *tasks, int ntasks, int shape, int T, hipStream_t stream)
{
    using C = typename Codec<S>::compute;
    with_tile_shape(shape, [&](auto sh) {
        using SH = decltype(sh);
        hipLaunchKernelGGL((k_batch_tile<S, SH>), dim3(ntasks), dim3(64 * SH::NW), 0, stream,
                           (const S *)src, (S *)dst, mask, near, (const BInst<C> *)inst, tasks, T);
    });
}

#define PTRT_TILE_INSTANCE(S)                                                                        \
    template <>                                                                                      \
    void launch_tile<S>(const StepLaunch &a, const TilePlan &plan, const uint8_t *special, int T)    \
    {                                                                                                \
        launch_tile_impl<S>(a, plan, special, T);                                                    \
    }                                                                                                \
    template <>                                                                                      \
    void launch_tile_batch<S>(const void *src, void *dst, const uint8_t *mask, const uint8_t *near, const void *inst,     \
                              const int4 *tasks, int ntasks, int shape, int T, hipStream_t stream)   \
    {                                                                                                \
        launch_tile_batch_impl<S>(src, dst, mask, near, inst, tasks, ntasks, shape, T, stream);            \
    }

} // namespace ptrt
