// Launch shape of the step kernel: the LDS a shape needs, and the rule that chooses one.  Host
// arithmetic and constants only, so that the rule can be run without a device.
#pragma once

#include <algorithm>
#include <cmath>
#include <cstddef>

#include "gd.h"

namespace gdk {

constexpr int kWave = 64;
constexpr int kLdsBytes = 160 * 1024 - 1024;  // LDS of one gfx950 CU, less room for static LDS

constexpr int kAgentArrays = 13;  // x y yaw v L W cos sin goal_x goal_y flags coll bound

constexpr int stage_cap(int K) { return (K + 60 + 3) / 4 * 4; }

// per-wave LDS of phase 5:
//   hist  NB ints        histogram of bin(d2), then the first (later: end) slot of each bin;
//                        a 0 before it, the start of bin 0 (16 B)
//   cand  ccap entries   (bin, point) of every point within the radius
//   skey  scap floats    keys of the staged points (bins up to the cut bin)
//   sq    scap indices   their points
constexpr size_t wave_lds_bytes(int NB, int K, int ccap, bool idx16) {
    const size_t ib = idx16 ? 2 : 4, cb = idx16 ? 4 : 8;
    const size_t b = 16 + (size_t)NB * 4 + (size_t)ccap * cb + (size_t)stage_cap(K) * (4 + ib);
    return (b + 15) / 16 * 16;
}

inline size_t step_lds_bytes(int waves, int NB, int K, int ccap, int road_cap, int cell_cap4,
                             int edge_cap, int agent_cap, bool idx16) {
    const bool staged = road_cap > 0;
    const size_t road = staged ? (size_t)road_cap * 16 + (size_t)cell_cap4 * 4 : 0;
    const size_t edges = edge_cap > 0 ? (size_t)edge_cap * 16 + (size_t)cell_cap4 * 4 : 0;
    const size_t per_wave = (size_t)waves * wave_lds_bytes(NB, K, ccap, idx16 || staged);
    return road + (size_t)agent_cap * 4 * kAgentArrays + (edges > per_wave ? edges : per_wave);
}

// Grid of at least `groups` (> 0) workgroups of `threads` threads, x fastest: an axis holds fewer
// than 2^32 threads, and one beyond is cut without an error.
struct Grid2 {
    unsigned x, y;
};
inline Grid2 grid_of(long long groups, int threads) {
    const long long x = std::min(groups, (1ll << 31) / threads);
    return {(unsigned)x, (unsigned)((groups + x - 1) / x)};
}

// Launch shape of the step kernel: waves per workgroup, distance bins, candidate-list
// entries per wave, and whether the road is staged in LDS.  Fields the config fixes are
// kept; of the shapes that fit, the one with the lowest predicted step time is taken.
//
// The prediction (microseconds) was fitted to measured steps of 47 batches (1 to 4096
// worlds, 2 to 128 agents each, even and uneven, 500 to 10 000 road points, K 32 to 960;
// 12 to 24 shapes each): the shape it picks is 0.8 % slower on average than the fastest one
// measured, 6.6 % at most.  A rule that took the most resident waves per compute unit, then
// 512 bins, was 17 % slower on average (512 x 32 agents: 41 against 28.7 us, 1024 x 64 with
// 6000 points: 241 against 175).  Its terms:
//   - a workgroup takes a fixed time for its world phases, more with the square of the agents
//     over its waves (pairs) and with the points it stages, then its share of the agents
//     one after the other, at a time per agent that grows with K;
//   - that time is a latency at few waves per compute unit and grows with their number where
//     the vector units are shared; reading the road through the caches costs more, the more
//     so when the roads of the worlds in flight outgrow an XCD's 4 MB of L2;
//   - the batch takes as many rounds of workgroups as the compute units hold at once.  An
//     uneven batch is dispatched longest world first, so its last round is filled.
// 128 and 256 bins measured alike (512 and more up to 7 % slower: their prefix scan).  The
// candidate list has to hold the points within the K-th distance and what the agent moved in a
// step: an agent with more scans its grid rows again, one load in flight.  Its length costs
// nothing but LDS, so of shapes that are otherwise alike the longest list is taken.  With the
// (up to 512 entries, or 2 K; a longer one keeps other kernels from the LDS).  With the shortest of
// at least 1.2 K (K = 100: 128 entries) agents at speed overflowed it on dense maps: 128 worlds x
// 64 agents, 20 000 points, K = 200: 55.4 us at 15 m/s and 61.8 at 30, with 512 entries 47.8 and
// 50.3; at 5 m/s both take 46.
struct Batch {  // what the prediction needs to know of the worlds
    int compute_units = 256;  // of the device
    int worlds = 0, max_agents = 0, max_road = 0, max_edges = 0, cell_cap4 = 0, agent_cap = 0;
    bool idx16 = true, uneven = false;
    double agents = 0.0, road = 0.0;  // means
    double within = 0.0;              // road points within the observation radius of a place, mean
};

struct Shape {
    double us = INFINITY;
    int waves = 0, bins = 0, cand_cap = 0, edge_cap = 0, road_cap = 0;
};

inline double predict_step(const Batch &b, int K, bool staged, int waves, int per_cu) {
    const int per_unit = (b.worlds + b.compute_units - 1) / b.compute_units;  // workgroups of a compute unit
    const int in_flight = std::min(per_cu, per_unit);
    double fixed = 6.0 + 0.0038 * b.agents * b.agents / waves + (staged ? 0.0144 * b.road / waves : 0.0);
    if (per_unit == 1) fixed *= 1.0 + 0.23 * (16 - waves) / 16;  // (nothing else to overlap it)
    fixed *= 1.0 + 0.02 * in_flight * std::sqrt((double)waves);
    double latency = staged ? 5.8 : 7.2, share = staged ? 0.33 : 0.43;
    if (!staged) {
        const double mb = 32.0 * in_flight * b.road * 16e-6;  // roads in flight per XCD
        const double x = std::max(0.0, std::min(1.0, (mb - 1.9) / 4.1));
        latency *= 1.0 + 0.05 * x;
        share *= 1.0 + 0.45 * x + 0.05 * std::max(0.0, std::log2(std::max(mb, 1e-3) / 6.6));
    }
    share *= in_flight * waves;
    const double agent = std::cbrt(latency * latency * latency + share * share * share) * (0.375 + 0.0025 * K);
    const double slots = (double)b.compute_units * per_cu;
    const double n = b.uneven && b.worlds <= slots ? b.max_agents : b.agents;
    const double each = fixed + std::max(1.0, n / waves + (n > waves ? 0.45 : 0.0)) * agent;
    double rounds = b.uneven ? std::max(1.0, b.worlds / slots + 0.4) : (double)per_unit / per_cu;
    if (!b.uneven && (rounds <= 1.0 || per_cu == 1)) rounds = std::max(1.0, rounds);
    else if (!b.uneven && per_unit % per_cu != 0) rounds += 0.15;
    return each * rounds * (b.agents > 20.0 * waves ? 1.3 : 1.0);
}

template <typename Waves>
Shape best_shape(const gd_config &c, const Batch &b, bool staged, Waves &&waves_per_cu) {
    const int K = c.top_k;
    Shape best;
    // a multiple of 4 points keeps the LDS regions after the road 16-byte aligned
    const int rc = staged ? (std::max(b.max_road, 1) + 3) / 4 * 4 : 0;
    // (agents stand on roads, where the map is about twice as dense as on average)
    const double needed = std::min({1.2 * K, 2.0 * b.within, 1024.0});
    for (int ec : {b.max_edges, 0}) {
        for (int wv : {16, 12, 8, 4, 2, 1}) {
            if (c.obs_waves && wv != c.obs_waves) continue;
            for (int nb : {256, 128, 512, 64, 1024}) {
                if (c.obs_bins ? nb != c.obs_bins : nb == 1024) continue;
                const int per_cu_regs = waves_per_cu(nb, staged, b.idx16) / wv;
                for (int cc : {128, 256, 384, 512, 768, 1024}) {
                    if (c.obs_cands && cc != c.obs_cands) continue;
                    const size_t lds = step_lds_bytes(wv, nb, K, K ? cc : 0, rc, b.cell_cap4, ec, b.agent_cap, b.idx16);
                    if (lds > (size_t)kLdsBytes) continue;
                    const int per_cu = std::min((int)((size_t)kLdsBytes / lds), per_cu_regs);
                    if (per_cu < 1) continue;
                    double us = predict_step(b, K, staged, wv, per_cu);
                    us *= nb == 256 ? 1.0 : nb == 128 ? 1.02 : 1.06;
                    if (K && cc < needed) us *= 1.2;                // the grid scanned again
                    us *= 1.0 - 1e-5 * std::min(cc, std::max(512, 2 * K)) / 128;
                    if (!ec && b.max_edges) us *= 1.01;             // edge segments through the caches
                    if (us < best.us) best = Shape{us, wv, nb, K ? cc : 0, ec, rc};
                }
            }
        }
    }
    return best;
}

// waves_per_cu(bins, staged, idx16): waves that the registers of that kernel allow per compute unit.
// False: no shape fits the LDS.
template <typename Waves>
bool launch_shape(const gd_config &c, const Batch &b, Waves &&waves_per_cu, Shape &pick) {
    const bool can_stage = c.top_k > 0 && b.idx16 && b.max_road <= 60000;
    Shape glob, lds;
    if (c.obs_road != GD_ROAD_LDS) glob = best_shape(c, b, false, waves_per_cu);
    if (c.obs_road != GD_ROAD_GLOBAL && can_stage) lds = best_shape(c, b, true, waves_per_cu);
    pick = lds.us <= glob.us ? lds : glob;
    return pick.waves != 0;
}

}  // namespace gdk
