// Differentiable rollout: forward with checkpoints and backward by recomputation.
//
// Forward: a row of 16 lanes per agent takes 16 steps of the configured model at a time, a
// lane per step: what a step needs from the steps before it is a running sum, everything
// else (trigonometry, nearest edge, reward) is independent and formed by all lanes at once.
// After each step the smooth reward is  r = -|g'| - softplus(s),  g' = R(-yaw)(g - p),
// s = signed distance (in the ego frame, positive on the right of the segment direction,
// i.e. off-road) to the nearest road-edge segment within the observation radius (s = -R when
// there is none).  The reward is an instance of the configurable agent/road-distance
// rewards of Sec. 3.2 "Rewards".  The state before every ckpt_every-th step is saved.
//
// Backward: per block of steps, last block first, the forward is recomputed from its
// checkpoint, a lane per step; each lane forms the reward's derivative and the coefficients
// of the adjoint's recursion at its step, the recursion over (x, y, yaw, v) runs backwards
// with them, and each lane turns the adjoint at its step into dJ/d(accel, steer).  Segment
// choice, side and clip activity are held constant; the result does not depend on
// ckpt_every.
//
// Both are bound by vector instructions (per agent-step, 4096 worlds x 64 agents, 6000 road
// points, T = 91, checkpoints every 10 steps: forward 33, backward 41).  With 8 lanes per
// agent that repeated the dynamics and the reward and shared one nearest-edge search per
// step they took 176 and 185, and the time was 9.45 + 11.4 ms against 1.54 + 1.88 ms now;
// 512 x 32 agents, T = 20: 182 + 190 against 27 + 31 us.
//
// Observation (optional): the forward can log the state after every step, from which
// k_rollout_obs forms the continuous observation of each agent (speed, goal in its frame;
// per partner slot the partner's position in its frame, heading difference, speed --
// Fig. 1, Sec. 3.2 "Sensor modalities").  Partners couple the agents of a world, so the
// observation's gradient is formed from that log in a kernel of its own, world by world.
#include <algorithm>

#include "gd_internal.h"

namespace gdk {

constexpr int kRollThreads = 256;               // threads per workgroup
constexpr int kRow = 16;                        // lanes per agent: one DPP row, a lane per step
constexpr int kRollAgents = kRollThreads / kRow;
constexpr int kMaxCkpt = 32;
constexpr int kEdgeList = 64;                   // candidate segments of a block of steps, per agent
constexpr int kEdgeStride = kEdgeList + 1;      // (odd: the rows of a wave read other LDS banks)

struct EdgeChoice {
    int q;          // cell-sorted position of the segment in the world's edge arrays, -1 = none
    float side;     // +1 off-road (right of the segment direction), -1 on-road
};

// ---- rows of 16 lanes
// value of lane K of the row, on all of its lanes
template <int K>
__device__ __forceinline__ float row_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + K, 0xf, 0xf, true));  // row_newbcast
}
// value of the lane before (lane 0: `first`)
__device__ __forceinline__ float row_before(float v, float first) {
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(first), __float_as_int(v), 0x111, 0xf, 0xf, false));  // row_shr:1
}
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// minimum over the row, on all of its lanes (row rotations)
__device__ __forceinline__ float row_min(float v) {
    v = fminf(v, dpp_f<0x128>(v));
    v = fminf(v, dpp_f<0x124>(v));
    v = fminf(v, dpp_f<0x122>(v));
    return fminf(v, dpp_f<0x121>(v));
}
// ballot of the row's 16 lanes
__device__ __forceinline__ unsigned row_ballot(bool p) {
    return (unsigned)(__ballot(p) >> (threadIdx.x & 48)) & 0xffffu;
}
// f(0), f(1), ... f(15) with constant arguments, in groups of four of which those at or
// beyond the (wave-uniform) count n are left out
template <int K>
struct StepIndex {
    static constexpr int k = K;
};
template <int K0, typename F>
__device__ __forceinline__ void four_up(F &&f) {
    f(StepIndex<K0>{});
    f(StepIndex<K0 + 1>{});
    f(StepIndex<K0 + 2>{});
    f(StepIndex<K0 + 3>{});
}
template <typename F>
__device__ __forceinline__ void each_step(int n, F &&f) {
    four_up<0>(f);
    if (n <= 4) return;
    four_up<4>(f);
    if (n <= 8) return;
    four_up<8>(f);
    if (n <= 12) return;
    four_up<12>(f);
}
template <int K0, typename F>
__device__ __forceinline__ void four_down(F &&f) {
    f(StepIndex<K0 + 3>{});
    f(StepIndex<K0 + 2>{});
    f(StepIndex<K0 + 1>{});
    f(StepIndex<K0>{});
}
template <typename F>
__device__ __forceinline__ void each_step_down(int n, F &&f) {
    if (n > 12) four_down<12>(f);
    if (n > 8) four_down<8>(f);
    if (n > 4) four_down<4>(f);
    four_down<0>(f);
}

// world of agent i: the largest w with agent_off[w] <= i, by a 16-way search of the row
__device__ __forceinline__ int world_of_row(const int *agent_off, int W, int i, int sub) {
    int lo = 0, len = W;
    while (len > 1) {
        const int st = (len + kRow - 1) / kRow;
        const int o = sub * st;
        const bool le = o < len && agent_off[lo + o] <= i;
        const int c = max(__popc(row_ballot(le)), 1) - 1;
        lo += c * st;
        len = min(st, len - c * st);
    }
    return lo;
}

// ---- a block of up to 16 steps of one agent, a lane per step
struct AgentState {  // the state a block starts from, the same on all lanes of the row
    float x, y, yaw, v, sn, cs;  // sn, cs: sine and cosine of yaw
};
struct StepState {   // this lane's step: the state before (0) and after (1) it
    float x0, y0, yaw0, v0, sn0, cs0;
    float x1, y1, yaw1, v1, sn1, cs1;
    float ts, cb, sb, sp, cp;  // bicycle: tan(steer), slip angle, direction of motion
    float vb;                  // bicycle: clipped midpoint speed; simplified model: distance
};

// The n steps of a block from state c.  What a step needs from the steps before it is a sum
// (speed, heading and position in turn), so the only serial part is one or a few additions
// per step, taken on all lanes of the row with the step's increment broadcast from its lane;
// tangents, sines and divisions are formed once per lane.  Every operation is rounded as in a
// step-by-step evaluation.  Bicycle model (App. B): slip angle beta = atan(tan(steer) / 2)
// through cos beta = 1 / sqrt(1 + z^2), sin beta = z cos beta (z = tan(steer) / 2), the
// direction of motion by angle addition.
template <bool DELTA, bool ONE>
__device__ __forceinline__ void run_block(const AgentState &c, float2 u, int n, int sub, float L, float dt,
                                          float vmax, StepState &o) {
#pragma clang fp contract(off)
    const float acc = u.x, h = 0.5f * acc;
    float ix, iy, iw;  // increments of the lane's step
    // speed before the step
    float v = c.v;
    if (!ONE) each_step(n, [&](auto kc) {
        constexpr int k = decltype(kc)::k;
        float w = __builtin_fmaf(row_bcast<k>(acc), dt, v);
        if (!DELTA) w = fminf(fmaxf(w, -vmax), vmax);
        v = sub > k ? w : v;
    });
    o.v0 = v;
    o.v1 = __builtin_fmaf(acc, dt, v);
    if (DELTA) {
        o.vb = __builtin_fmaf(v, dt, h * dt * dt);
        iw = u.y * o.vb;
    } else {
        o.v1 = fminf(fmaxf(o.v1, -vmax), vmax);
        o.vb = fminf(fmaxf(__builtin_fmaf(h, dt, v), -vmax), vmax);
        o.ts = tanf(u.y);
        const float z = 0.5f * o.ts;
        o.cb = __builtin_amdgcn_rsqf(__builtin_fmaf(z, z, 1.0f));
        o.sb = z * o.cb;
        iw = o.vb * o.cb * o.ts / L * dt;
    }
    // heading before the step
    float yaw = c.yaw;
    if (!ONE) each_step(n, [&](auto kc) {
        constexpr int k = decltype(kc)::k;
        const float w = yaw + row_bcast<k>(iw);
        yaw = sub > k ? w : yaw;
    });
    o.yaw0 = yaw;
    o.yaw1 = yaw + iw;
    sincosf(o.yaw1, &o.sn1, &o.cs1);
    o.sn0 = ONE ? c.sn : row_before(o.sn1, c.sn);  // the step before ends with this step's heading
    o.cs0 = ONE ? c.cs : row_before(o.cs1, c.cs);
    if (DELTA) {
        ix = o.vb * o.cs0;
        iy = o.vb * o.sn0;
    } else {
        o.sp = __builtin_fmaf(o.cs0, o.sb, o.sn0 * o.cb);
        o.cp = __builtin_fmaf(o.cs0, o.cb, -(o.sn0 * o.sb));
        ix = o.vb * o.cp * dt;
        iy = o.vb * o.sp * dt;
    }
    // position before the step
    float x = c.x, y = c.y;
    if (!ONE) each_step(n, [&](auto kc) {
        constexpr int k = decltype(kc)::k;
        const float wx = x + row_bcast<k>(ix), wy = y + row_bcast<k>(iy);
        x = sub > k ? wx : x;
        y = sub > k ? wy : y;
    });
    o.x0 = x;
    o.y0 = y;
    o.x1 = x + ix;
    o.y1 = y + iy;
}

// the state after the n steps of a block
__device__ __forceinline__ AgentState after_block(const StepState &o, int n) {
    if (n == kRow)
        return {row_bcast<15>(o.x1), row_bcast<15>(o.y1), row_bcast<15>(o.yaw1),
                row_bcast<15>(o.v1), row_bcast<15>(o.sn1), row_bcast<15>(o.cs1)};
    return {__shfl(o.x1, n - 1, kRow), __shfl(o.y1, n - 1, kRow), __shfl(o.yaw1, n - 1, kRow),
            __shfl(o.v1, n - 1, kRow), __shfl(o.sn1, n - 1, kRow), __shfl(o.cs1, n - 1, kRow)};
}

// ---- nearest road-edge segment
struct EdgeGrid {  // a world's edge segments
    WorldGrid g;
    const int *ecs;
    const float4 *es;
    const int *eid;
};
// the last block's nearest segment q (-1: none yet) at distance d of the point (x, y) of the
// path next to the coming block
struct EdgeBound {
    float x, y, d;
    int q;
};

// Visits, 16 at a time, every segment that can lie within r of (cx, cy): f(q, ok) with the
// segment's cell-sorted position (ok = false: padding).  Segments are keyed by the cell of
// their first point, so the square of cells is widened by the longest segment.
template <typename F>
__device__ __forceinline__ void scan_edges(const EdgeGrid &e, float cx, float cy, float r, int sub, F &&f) {
    const WorldGrid &g = e.g;
    const float rr = r + g.max_seg + 1e-3f * g.cs;
    const int x0 = cell_coord(cx - rr, g.ox, g.inv_cs, g.nx), x1 = cell_coord(cx + rr, g.ox, g.inv_cs, g.nx);
    const int y0 = cell_coord(cy - rr, g.oy, g.inv_cs, g.ny), y1 = cell_coord(cy + rr, g.oy, g.inv_cs, g.ny);
    for (int yb = y0; yb <= y1; yb += kRow) {
        // a lane per grid row: its range of segments
        const int yy = min(yb + sub, y1);
        const int q0 = e.ecs[yy * g.nx + x0], q1 = e.ecs[yy * g.nx + x1 + 1];
        const int m = min(kRow, y1 - yb + 1);
        for (int k = 0; k < m; k++) {
            const int b1 = __shfl(q1, k, kRow);
            for (int q = __shfl(q0, k, kRow); q < b1; q += kRow) f(q + sub, q + sub < b1);
        }
    }
}

// squared distance of (px, py) to the segment from (x0, y0) along (ex, ey); ir = 1 / |e|^2 (0
// for a point)
__device__ __forceinline__ float seg_d2(float x0, float y0, float ex, float ey, float ir, float px, float py) {
    const float ax = x0 - px, ay = y0 - py;
    const float u = fminf(fmaxf(-(ax * ex + ay * ey) * ir, 0.0f), 1.0f);
    const float qx = ax + u * ex, qy = ay + u * ey;
    return qx * qx + qy * qy;
}

// 1 / |e|^2 (the hardware reciprocal: 1 ulp; ties closer than the 1e-4 m band are decided
// alike by the forward and its recompute), 0 for a segment without length
__device__ __forceinline__ float seg_inv(float ex, float ey) {
    const float ee = ex * ex + ey * ey;
    return ee > 0.0f ? __builtin_amdgcn_rcpf(ee) : 0.0f;
}

// The candidate list of one row in LDS.
struct EdgeList {
    float4 *seg;  // x0, y0, ex, ey
    float2 *inv;  // 1 / |e|^2, position (bits)
    float *dc;    // distance from the centre of the row's points
};

// Nearest road-edge segment within R of each lane's point (px, py), by the smallest binary32
// squared distance, ties to the lowest world-local index; `valid`: the lane has a point.
// The row's points lie on one agent's path, rho from their centre c at most.  With D a
// bound on the distance of c to its nearest segment, every point's nearest segment lies
// within D + 2 rho of c:
//   1. D from the segments stored around the last block's nearest one, or, without one,
//      from widening squares of cells;
//   2. the row collects the segments within D + 2 rho in LDS, a lane per segment;
//   3. every lane takes its distance b to each fourth of them: its nearest one lies within
//      b, so within max(b + |p - c|) of c for all lanes; the list shrinks to those;
//   4. every lane takes its minimum over what is left, read by all lanes at once.
// A full list is taken in parts.  Bound by vector instructions: step 4 over the whole list
// of step 2 took about 65 instead of 20 segments per block and half of the kernel's time.
// ONE: a rollout of one step has one point per row, c itself, whose nearest segment the widening
// squares find without a list (4096 x 64 agents, T = 1: forward 178 -> 88 us, backward 189 ->
// 118; 114 and 127 with 8 lanes per agent).
template <bool ONE>
__device__ __forceinline__ EdgeChoice nearest_edges(const EdgeGrid &e, const EdgeList &ls, float px, float py,
                                                    bool valid, float R, int sub, EdgeBound &bd,
                                                    bool last_lane) {
    EdgeChoice ch{-1, -1.0f};
    const WorldGrid &g = e.g;
    valid = valid && fabsf(px) < INFINITY && fabsf(py) < INFINITY;
    const float lox = row_min(valid ? px : INFINITY), hix = -row_min(valid ? -px : INFINITY);
    const float loy = row_min(valid ? py : INFINITY), hiy = -row_min(valid ? -py : INFINITY);
    float best = INFINITY;
    int bq = -1;
    if (g.n_edge > 0 && lox <= hix) {
        const float cx = 0.5f * lox + 0.5f * hix, cy = 0.5f * loy + 0.5f * hiy;
        const float wx = hix - lox, wy = hiy - loy;
        // (slack for the rounding of distances between coordinates of this size)
        const float marg = 1e-2f + 1e-3f * g.cs + 2e-6f * (fabsf(cx) + fabsf(cy));
        const float rho = 0.5f * __builtin_amdgcn_sqrtf(wx * wx + wy * wy) + marg;
        const float far = R + rho;  // nothing beyond it is within R of a point
        auto centre_d2 = [&](int q, bool ok) {
            const float4 s = e.es[ok ? q : 0];
            const float ex = s.z - s.x, ey = s.w - s.y;
            const float d2 = seg_d2(s.x, s.y, ex, ey, seg_inv(ex, ey), cx, cy);
            return ok ? d2 : INFINITY;
        };
        auto nearer = [&](float d2, int q) {
            bool less = d2 < best;
            // (exact ties are rare: the indices are read for them only)
            if (d2 == best && bq >= 0) less = e.eid[q] < e.eid[bq];
            best = less ? d2 : best;
            bq = less ? q : bq;
        };
        if (ONE) {
            for (float r = 0.5f * g.cs;; r *= 3.0f) {
                r = fminf(r, far);
                best = INFINITY;
                bq = -1;
                scan_edges(e, cx, cy, r, sub, [&](int q, bool ok) { nearer(centre_d2(q, ok), q); });
                const float d2 = row_min(best);
                unsigned who = row_ballot(bq >= 0 && best == d2);
                if (who & (who - 1)) {  // equal ones: the lowest index
                    const float id = bq >= 0 && best == d2 ? (float)e.eid[bq] : INFINITY;
                    who = row_ballot(id == row_min(id));
                }
                best = d2;
                bq = who ? __shfl(bq, __ffs(who) - 1, kRow) : -1;
                if (__builtin_amdgcn_sqrtf(best) + marg <= r || !(r < far)) break;
            }
        } else {
            float D;
            if (bd.q >= 0) {
                const int q = bd.q - kRow / 2 + sub;
                const float d = __builtin_amdgcn_sqrtf(row_min(centre_d2(q, q >= 0 && q < g.n_edge)));
                const float hx = cx - bd.x, hy = cy - bd.y;
                D = fminf(d, bd.d + __builtin_amdgcn_sqrtf(hx * hx + hy * hy)) + marg;
            } else {
                for (float r = 0.5f * g.cs;; r *= 3.0f) {
                    r = fminf(r, far);
                    float d2 = INFINITY;
                    scan_edges(e, cx, cy, r, sub, [&](int q, bool ok) { d2 = fminf(d2, centre_d2(q, ok)); });
                    D = __builtin_amdgcn_sqrtf(row_min(d2)) + marg;
                    if (D <= r || !(r < far)) break;
                }
            }
            const float rf = fminf(D + 2.0f * rho, far) + marg;
            const float pcx = px - cx, pcy = py - cy;
            const float pc = __builtin_amdgcn_sqrtf(pcx * pcx + pcy * pcy);
            int cnt = 0;
            auto sync = [] {
                __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
                __builtin_amdgcn_wave_barrier();
            };
            auto distance2 = [&](int k, int &q) {
                const float4 s = ls.seg[k];
                const float2 t = ls.inv[k];
                q = __float_as_int(t.y);
                return seg_d2(s.x, s.y, s.z, s.w, t.x, px, py);
            };
            // the segments of the list pad to a multiple of four with some that are never nearer
            auto pad = [&](int m) {
                const int padded = (m + 3) & ~3;
                if (m + sub < padded) {
                    ls.seg[m + sub] = make_float4(NAN, NAN, 0.f, 0.f);
                    ls.inv[m + sub] = make_float2(0.f, 0.f);
                }
                sync();
                return padded;
            };
            auto take = [&]() {
                sync();
                float b2 = best;
                for (int k = 0; k < cnt; k += 4) {
                    int q;
                    b2 = fminf(b2, distance2(k, q));
                }
                const float reach = valid ? __builtin_amdgcn_sqrtf(b2) + pc : 0.0f;
                const float keep = -row_min(-reach) + marg;
                int m = 0;
                for (int k0 = 0; k0 < cnt; k0 += kRow) {
                    const int k = min(k0 + sub, cnt - 1);
                    const float4 s = ls.seg[k];
                    const float2 t = ls.inv[k];
                    const bool in = k0 + sub < cnt && ls.dc[k] <= keep;
                    const unsigned bits = row_ballot(in);
                    sync();
                    if (in) {
                        const int pos = m + __popc(bits & ((1u << sub) - 1u));
                        ls.seg[pos] = s;
                        ls.inv[pos] = t;
                    }
                    m += __popc(bits);
                    sync();
                }
                const int padded = pad(m);
                for (int k0 = 0; k0 < padded; k0 += 2) {
#pragma unroll
                    for (int k = k0; k < k0 + 2; k++) {
                        int q;
                        const float d2 = distance2(k, q);
                        nearer(d2, q);
                    }
                }
                sync();
                cnt = 0;
            };
            scan_edges(e, cx, cy, rf, sub, [&](int q, bool ok) {
                const float4 s = e.es[ok ? q : 0];
                const float ex = s.z - s.x, ey = s.w - s.y;
                const float ir = seg_inv(ex, ey);
                const float d = __builtin_amdgcn_sqrtf(seg_d2(s.x, s.y, ex, ey, ir, cx, cy));
                const bool in = ok && d <= rf;
                const unsigned bits = row_ballot(in);
                if (cnt + kRow > kEdgeList) take();
                if (in) {
                    const int pos = cnt + __popc(bits & ((1u << sub) - 1u));
                    ls.seg[pos] = make_float4(s.x, s.y, ex, ey);
                    ls.inv[pos] = make_float2(ir, __int_as_float(q));
                    ls.dc[pos] = d;
                }
                cnt += __popc(bits);
            });
            take();
        }
    }
    // the bound for the next block: this block's point next to it
    const float d = sqrtf(best);
    const int qk = valid ? bq : -1;
    bd.x = last_lane ? row_bcast<15>(px) : row_bcast<0>(px);
    bd.y = last_lane ? row_bcast<15>(py) : row_bcast<0>(py);
    bd.d = last_lane ? row_bcast<15>(d) : row_bcast<0>(d);
    bd.q = __float_as_int(last_lane ? row_bcast<15>(__int_as_float(qk)) : row_bcast<0>(__int_as_float(qk)));
    if (!valid || bq < 0 || !(d <= R)) return ch;
    ch.q = bq;
    const float4 s = e.es[bq];
    const float cr = (s.z - s.x) * (py - s.y) - (s.w - s.y) * (px - s.x);
    ch.side = cr < 0.0f ? 1.0f : -1.0f;
    return ch;
}

__device__ __forceinline__ float softplusf(float z) { return fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z))); }
// (the hardware reciprocal: 1 ulp, far inside the gradient tolerance)
__device__ __forceinline__ float sigmoidf(float z) { return __builtin_amdgcn_rcpf(1.0f + expf(-z)); }

// smooth reward at (x, y) and the heading's sine and cosine for a fixed segment choice,
// computed through the ego frame
__device__ __forceinline__ float smooth_reward(float x, float y, float st, float ct, float gx, float gy,
                                               const float4 *es, const EdgeChoice &ch, float R) {
    const float dxg = gx - x, dyg = gy - y;
    const float gpx = ct * dxg + st * dyg, gpy = -st * dxg + ct * dyg;
    const float ng = sqrtf(gpx * gpx + gpy * gpy);
    float s = -R;
    if (ch.q >= 0) {
        const float4 e = es[ch.q];
        const float ax = e.x - x, ay = e.y - y, bx = e.z - x, by = e.w - y;
        const float apx = ct * ax + st * ay, apy = -st * ax + ct * ay;
        const float bpx = ct * bx + st * by, bpy = -st * bx + ct * by;
        const float ex = bpx - apx, ey = bpy - apy;
        const float ee = ex * ex + ey * ey;
        // (the backward forms u with the same expression, so their clamp decisions agree)
        float u = ee > 0.0f ? -(apx * ex + apy * ey) * __builtin_amdgcn_rcpf(ee) : 0.0f;
        u = fminf(fmaxf(u, 0.0f), 1.0f);
        const float qx = apx + u * ex, qy = apy + u * ey;
        s = ch.side * sqrtf(qx * qx + qy * qy);
    }
    return -ng - softplusf(s);
}

// The workgroup of tile number b: consecutive tiles (agents of one world, neighbours in the
// rows of actions and rewards) go to one XCD and share its L2.  Workgroups are handed to the
// 8 XCDs in turn.
__device__ __forceinline__ int xcd_tile(int b, int nb) {
    const int per = nb / 8, rest = nb % 8, x = b % 8, k = b / 8;
    return x * per + min(x, rest) + k;
}

// (four waves per SIMD: 128 registers; one more register costs a quarter of the waves)
template <bool DELTA, bool ONE>
__global__ __launch_bounds__(kRollThreads, 4) void k_rollout_fwd(SimArgs a, const float2 *__restrict__ act,
                                                              int T, int C, float *__restrict__ rewards,
                                                              float *__restrict__ ckpt,
                                                              float *__restrict__ slog) {
    constexpr int kList = ONE ? 1 : kRollAgents * kEdgeStride;
    __shared__ float4 s_seg[kList];
    __shared__ float2 s_inv[kList];
    __shared__ float s_dc[kList];
    const int row = threadIdx.x / kRow, sub = threadIdx.x % kRow;
    const unsigned at = (blockIdx.y * gridDim.x + (unsigned)xcd_tile(blockIdx.x, gridDim.x)) * kRollAgents + row;
    if (at >= (unsigned)a.A) return;
    const int i = (int)at;
    const EdgeList ls{s_seg + row * kEdgeStride, s_inv + row * kEdgeStride, s_dc + row * kEdgeStride};
    const size_t A = (size_t)a.A;
    const float2 none = make_float2(0.f, 0.f);
    float2 next = sub < T ? act[(size_t)sub * A + i] : none;
    AgentState c{a.x[i], a.y[i], a.yaw[i], a.v[i], 0.f, 0.f};
    const float L = a.len[i], gx = a.gx[i], gy = a.gy[i];
    const int w = world_of_row(a.agent_off, a.W, i, sub);
    const int r0 = a.road_off[w];
    const EdgeGrid e{a.grid[w], a.ecell_start + (size_t)w * kCellStride, a.eseg + r0, a.eseg_id + r0};
    sincosf(c.yaw, &c.sn, &c.cs);
    EdgeBound bd{0.f, 0.f, 0.f, -1};
    for (int t0 = 0; t0 < (ONE ? 1 : T); t0 += kRow) {
        const int n = ONE ? 1 : min(kRow, T - t0), t = t0 + sub;
        const bool on = sub < n;
        const float2 u = next;
        next = t + kRow < T ? act[(size_t)(t + kRow) * A + i] : none;
        StepState o;
        run_block<DELTA, ONE>(c, u, n, sub, L, a.dt, a.vmax, o);
        if (n == kRow) c = after_block(o, kRow);
        if (on && t % C == 0) {
            float *ck = ckpt + (size_t)(t / C) * 4 * A;
            ck[i] = o.x0;
            ck[A + i] = o.y0;
            ck[2 * A + i] = o.yaw0;
            ck[3 * A + i] = o.v0;
        }
        const EdgeChoice ch = nearest_edges<ONE>(e, ls, o.x1, o.y1, on, a.R_obs, sub, bd, true);
        const float rw = smooth_reward(o.x1, o.y1, o.sn1, o.cs1, gx, gy, e.es, ch, a.R_obs);
        if (on) {
            rewards[(size_t)t * A + i] = rw;
            if (slog) {
                float *sl = slog + (size_t)t * 4 * A;
                sl[i] = o.x1;
                sl[A + i] = o.y1;
                sl[2 * A + i] = o.yaw1;
                sl[3 * A + i] = o.v1;
            }
        }
    }
}

// Four floats of an observation row (a partner slot; rows start at any multiple of 4 bytes).
struct __attribute__((packed, aligned(4))) Slot4 {
    float x, y, z, w;
};

constexpr int kObsThreads = 256;

// Observation of the rollout from its state log slog [T, 4, A] (the state after each
// step): obs [T, A, 3 + 4P] = (speed, goal x', goal y') then, per partner slot s (the
// s-th other agent of the world in index order), (x', y', wrap(yaw_j - yaw), v_j) when
// the partner lies within the radius (binary32 key, inclusive), zeros otherwise.
// Bound by its writes.  One workgroup per world and `steps` of the rollout's steps, whose
// states are staged in LDS with their sines and cosines; then `lpr` lanes (a power of two)
// per agent, a partner slot per lane, 16 bytes stored at a time.  A wave per agent-step with a
// lane per feature looked up the world and took a sine and cosine for each agent-step:
// 512 x 32 agents, T = 20 (166 MB): 192 us against 30 us now (5.6 TB/s).  Where worlds and
// steps leave the chip idle, `share` agents of the world per workgroup instead of all.
__global__ __launch_bounds__(kObsThreads) void k_rollout_obs(SimArgs a, const float *__restrict__ slog, int tb,
                                                             int T, int steps, int share, int lpr,
                                                             float *__restrict__ obs) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int w = blockIdx.x;
    const int a0 = a.agent_off[w], n = a.agent_off[w + 1] - a0;
    const int i0 = (int)blockIdx.z * share, i1 = min(n, i0 + share);
    if (i0 >= n) return;
    const int t0 = tb + (int)blockIdx.y * steps, m = min(steps, T - t0);
    float4 *pose = reinterpret_cast<float4 *>(smem);  // x, y, yaw, speed of the steps' agents
    const size_t A = (size_t)a.A;
    const int P = a.P;
    const size_t F = 3 + 4 * (size_t)P;
    float2 *turn = reinterpret_cast<float2 *>(pose + (size_t)m * n);  // sine, cosine
    for (int k = threadIdx.x; k < m * n; k += kObsThreads) {
        const int tl = k / n, i = k - tl * n;
        const float *S = slog + (size_t)(t0 + tl) * 4 * A + a0 + i;
        const float x = S[0], y = S[A], yaw = S[2 * A], v = S[3 * A];
        const float gx = a.gx[a0 + i], gy = a.gy[a0 + i];
        float sn, cs;
        sincosf(yaw, &sn, &cs);
        pose[k] = make_float4(x, y, yaw, v);
        turn[k] = make_float2(sn, cs);
        if (i < i0 || i >= i1) continue;
        const float dxg = gx - x, dyg = gy - y;
        float *o = obs + ((size_t)(t0 + tl) * A + a0 + i) * F;
        o[0] = v;
        o[1] = cs * dxg + sn * dyg;
        o[2] = -sn * dxg + cs * dyg;
    }
    __syncthreads();
    const int sub = threadIdx.x & (lpr - 1), per = kObsThreads / lpr;
    for (int tl = 0; tl < m; tl++) {
        for (int i = i0 + threadIdx.x / lpr; i < i1; i += per) {
            const float4 p = pose[tl * n + i];
            const float sn = turn[tl * n + i].x, cs = turn[tl * n + i].y;
            Slot4 *o = reinterpret_cast<Slot4 *>(obs + ((size_t)(t0 + tl) * A + a0 + i) * F + 3);
            for (int sl = sub; sl < P; sl += lpr) {
                const int j = sl < i ? sl : sl + 1;
                const float4 q = pose[tl * n + min(j, n - 1)];
                const bool in = j < n && key32(p.x, p.y, q.x, q.y) <= a.R2_obs;
                const float dx = q.x - p.x, dy = q.y - p.y;
                const float fx = cs * dx + sn * dy, fy = -sn * dx + cs * dy, h = wrap_pi(q.z - p.z);
                o[sl] = in ? Slot4{fx, fy, h, q.w} : Slot4{0.f, 0.f, 0.f, 0.f};
            }
        }
    }
}

// Gradient of the observation terms with respect to the states after the steps: og [steps, A]
// (x, y, yaw, speed) for steps t0 .. t0 + gridDim.y, from grad_obs and the state log (the
// states the observation was formed from, so that the partner masks agree with it).
// Partners couple the agents: the slot of agent j in observer m's row, f = R(-yaw_m)(p_j -
// p_m), wrap(yaw_j - yaw_m), v_j, gives terms to both.  One workgroup per world and step: a
// wave takes an observer (a few of them in small worlds) with a lane per agent j, so that
// grad_obs is read in rows, only where the partner is within the radius; the terms of j stay
// in its lane over all observers, those of m are summed over the row's lanes; both in a
// fixed order.  Where worlds and steps leave the chip idle, `share` agents of the world per
// workgroup: it takes their columns over all observers, then their rows over all agents (each
// pair twice, but nothing to add up between workgroups).  Bound by the latency of those reads.  Gathered by each agent's lanes inside
// the backward kernel instead, row and column read per agent and step, the backward took
// 390 us against 40 + 37 us now (512 x 32 agents, T = 20).
struct ObsGradLds {
    float4 *pose;  // x, y, sine, cosine of each agent
    float4 *mine;  // terms of each of the workgroup's agents from its own row (x, y, yaw)
    float4 *part;  // per wave: terms of each of them from the others' rows
};

// sum over groups of `cols` lanes (a power of two, at least 8), on all of their lanes
__device__ __forceinline__ float group_sum(float v, int cols) {
    v += dpp_f<0xB1>(v);   // quad_perm [1, 0, 3, 2]
    v += dpp_f<0x4E>(v);   // quad_perm [2, 3, 0, 1]
    v += dpp_f<0x141>(v);  // row_half_mirror
    if (cols > 8) v += dpp_f<0x140>(v);  // row_mirror
    if (cols > 16) v += __shfl_xor(v, 16, kWave);
    if (cols > 32) v += __shfl_xor(v, 32, kWave);
    return v;
}

__global__ __launch_bounds__(kObsThreads) void k_rollout_obs_grad(SimArgs a, const float *__restrict__ slog, int t0,
                                                                  int share, const float *__restrict__ grad_obs,
                                                                  float4 *__restrict__ og) {
    extern __shared__ __align__(16) unsigned char smem[];
    const int w = blockIdx.x, t = t0 + blockIdx.y;
    const int a0 = a.agent_off[w], n = a.agent_off[w + 1] - a0;
    const int i0 = (int)blockIdx.z * share, i1 = min(n, i0 + share), ni = i1 - i0;
    if (i0 >= n) return;
    const int lane = threadIdx.x & (kWave - 1), wid = threadIdx.x / kWave, waves = blockDim.x / kWave;
    const ObsGradLds s{reinterpret_cast<float4 *>(smem), reinterpret_cast<float4 *>(smem) + n,
                       reinterpret_cast<float4 *>(smem) + n + ni};
    const size_t A = (size_t)a.A;
    const int P = a.P;
    const size_t F = 3 + 4 * (size_t)P;
    const float *S = slog + (size_t)t * 4 * A + a0;
    const float *G = grad_obs + ((size_t)t * A + a0) * F;
    for (int i = threadIdx.x; i < n; i += blockDim.x) {
        float sn, cs;
        sincosf(S[2 * A + i], &sn, &cs);
        s.pose[i] = make_float4(S[i], S[A + i], sn, cs);
        if (i < ni) s.mine[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    }
    __syncthreads();
    // observers [ma, mb) with agents [ja, jb) in their slots: terms of the agents (COLS), of
    // the observers (ROWS)
    auto pairs = [&](int ma, int mb, int ja, int jb, auto cols_too, auto rows_too) {
        constexpr bool COLS = decltype(cols_too)::k, ROWS = decltype(rows_too)::k;
        // lanes of an observer: as many as agents, a power of two from 8 on; observers of a wave
        const int log = jb - ja <= 8 ? 3 : jb - ja > kWave / 2 ? 6 : 32 - __builtin_clz(jb - ja - 1);
        const int cols = 1 << log, rows = kWave >> log;
        const int col = lane & (cols - 1), row = lane >> log;
        for (int j0 = ja; j0 < jb; j0 += cols) {
            const int j = j0 + col;
            const float4 pj = s.pose[min(j, n - 1)];
            float cx = 0.f, cy = 0.f, ch = 0.f, cv = 0.f;
            // four observers' rows in flight together
            constexpr int U = 4;
            for (int m0 = ma + wid * rows; m0 < mb; m0 += U * waves * rows) {
                Slot4 g[U];
                float4 pm[U];
                bool in[U];
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const int m = m0 + u * waves * rows + row;
                    pm[u] = s.pose[min(m, n - 1)];
                    const int sl = j < m ? j : j - 1;
                    in[u] = j < jb && m < mb && j != m && sl < P && key32(pm[u].x, pm[u].y, pj.x, pj.y) <= a.R2_obs;
                    g[u] = Slot4{0.f, 0.f, 0.f, 0.f};
                    if (in[u]) g[u] = *reinterpret_cast<const Slot4 *>(G + (size_t)m * F + 3 + 4 * (size_t)sl);
                }
#pragma unroll
                for (int u = 0; u < U; u++) {
                    const int m = m0 + u * waves * rows + row;
                    if (__ballot(in[u]) == 0ull) continue;
                    float rx = 0.f, ry = 0.f, rh = 0.f;
                    if (in[u]) {
                        const float sn = pm[u].z, cs = pm[u].w;
                        const float dx = pj.x - pm[u].x, dy = pj.y - pm[u].y;
                        const float fx = cs * dx + sn * dy, fy = -sn * dx + cs * dy;
                        const float wx = cs * g[u].x - sn * g[u].y, wy = sn * g[u].x + cs * g[u].y;
                        cx += wx;
                        cy += wy;
                        ch += g[u].z;
                        cv += g[u].w;
                        rx = -wx;
                        ry = -wy;
                        rh = g[u].x * fy - g[u].y * fx - g[u].z;
                    }
                    if (!ROWS) continue;
                    rx = group_sum(rx, cols);
                    ry = group_sum(ry, cols);
                    rh = group_sum(rh, cols);
                    if (col == 0 && m < mb) {
                        float4 q = s.mine[m - i0];  // (observer m is always taken by this wave)
                        q.x += rx;
                        q.y += ry;
                        q.z += rh;
                        s.mine[m - i0] = q;
                    }
                }
            }
            if (!COLS) continue;
            for (int d = cols; d < kWave; d <<= 1) {
                cx += __shfl_xor(cx, d, kWave);
                cy += __shfl_xor(cy, d, kWave);
                ch += __shfl_xor(ch, d, kWave);
                cv += __shfl_xor(cv, d, kWave);
            }
            if (row == 0 && j < jb) s.part[wid * ni + j - i0] = make_float4(cx, cy, ch, cv);
        }
    };
    if (ni == n) {
        pairs(0, n, 0, n, StepIndex<1>{}, StepIndex<1>{});
    } else {
        pairs(0, n, i0, i1, StepIndex<1>{}, StepIndex<0>{});
        pairs(i0, i1, 0, n, StepIndex<0>{}, StepIndex<1>{});
    }
    __syncthreads();
    for (int k = threadIdx.x; k < ni; k += blockDim.x) {
        const int i = i0 + k;
        const float *go = G + (size_t)i * F;
        const float4 p = s.pose[i];
        const float dxg = a.gx[a0 + i] - p.x, dyg = a.gy[a0 + i] - p.y;
        const float gpx = p.w * dxg + p.z * dyg, gpy = -p.z * dxg + p.w * dyg;
        // own speed, goal in the own frame g' = R(-yaw)(g - p), own slots
        float4 q = s.mine[k];
        q.x += -p.w * go[1] + p.z * go[2];
        q.y += -p.z * go[1] - p.w * go[2];
        q.z += gpy * go[1] - gpx * go[2];
        q.w = go[0];
        for (int v = 0; v < waves; v++) {
            const float4 c = s.part[v * ni + k];
            q.x += c.x;
            q.y += c.y;
            q.z += c.z;
            q.w += c.w;
        }
        og[(size_t)blockIdx.y * A + a0 + i] = q;
    }
}

// The same gradient for one agent (number l of the world's n agents from a0) and step t, gathered
// by one lane: for callers that give no scratch.  The backward takes 80 us so, 62 us with
// k_rollout_obs_grad (512 x 32 agents, T = 20); 40 x 120, T = 91: 638 against 222.
__device__ __forceinline__ float4 gather_obs_grad(const SimArgs &a, const float *slog, const float *grad_obs, int t,
                                                  int a0, int n, int l, float gx, float gy) {
    const size_t A = (size_t)a.A, F = 3 + 4 * (size_t)a.P;
    const float *S = slog + (size_t)t * 4 * A + a0;
    const float *G = grad_obs + ((size_t)t * A + a0) * F;
    const float *go = G + (size_t)l * F;
    const float xi = S[l], yi = S[A + l];
    float si, ci;
    sincosf(S[2 * A + l], &si, &ci);
    // own speed, goal in the own frame g' = R(-yaw)(g - p)
    const float dxg = gx - xi, dyg = gy - yi;
    const float gpx = ci * dxg + si * dyg, gpy = -si * dxg + ci * dyg;
    float4 q = make_float4(-ci * go[1] + si * go[2], -si * go[1] - ci * go[2], gpy * go[1] - gpx * go[2], go[0]);
    for (int j = 0; j < n; j++) {
        const float xj = S[j], yj = S[A + j];
        if (j == l || !(key32(xi, yi, xj, yj) <= a.R2_obs)) continue;
        const float dx = xj - xi, dy = yj - yi;
        // agent j in this agent's row
        const int own = j < l ? j : j - 1;
        if (own < a.P) {
            const Slot4 g = *reinterpret_cast<const Slot4 *>(go + 3 + 4 * (size_t)own);
            const float fx = ci * dx + si * dy, fy = -si * dx + ci * dy;
            q.x -= ci * g.x - si * g.y;
            q.y -= si * g.x + ci * g.y;
            q.z += g.x * fy - g.y * fx - g.z;
        }
        // this agent in the row of agent j
        const int slot = l < j ? l : l - 1;
        if (slot < a.P) {
            const Slot4 g = *reinterpret_cast<const Slot4 *>(G + (size_t)j * F + 3 + 4 * (size_t)slot);
            float sj, cj;
            sincosf(S[2 * A + j], &sj, &cj);
            q.x += cj * g.x - sj * g.y;
            q.y += sj * g.x + cj * g.y;
            q.z += g.z;
            q.w += g.w;
        }
    }
    return q;
}

// Steps of a backward block (at most 16, a lane each).  A block starts from the checkpoint
// before it: whole checkpoint segments need no steps in between, but leave lanes idle (six of
// 16 with checkpoints every 10 steps); blocks of 16 take up to C - 1 steps to their start
// first.  Of 91 steps, blocks of 16 make 6 instead of 10 (4096 x 64 agents: 2.16 -> 1.88 ms);
// of 20, both make 2, and the steps in between are saved.
__host__ inline int roll_block(int T, int C) {
    const int whole = C <= kRow ? kRow / C * C : kRow;
    return (T + kRow - 1) / kRow < (T + whole - 1) / whole ? kRow : whole;
}

// Where the backward has the observation's gradient from.
enum ObsGrad { kObsNone = 0, kObsScratch = 1, kObsGather = 2 };

// Steps [Ts, Te) of the backward: all of them, unless the observation's gradient og, of these
// steps, comes in parts (kObsScratch): then the adjoint of the state before the part is kept in
// `carry`.  kObsGather reads slog and grad_obs instead.
template <bool DELTA, int OBS, bool ONE>
__global__ __launch_bounds__(kRollThreads, 4) void k_rollout_bwd(SimArgs a, const float2 *__restrict__ act,
                                                              const float *__restrict__ ckpt, int T, int C,
                                                              int B, int Ts, int Te,
                                                              const float *__restrict__ grad_r,
                                                              const float4 *__restrict__ og,
                                                              float4 *__restrict__ carry,
                                                              const float *__restrict__ slog,
                                                              const float *__restrict__ grad_obs,
                                                              float2 *__restrict__ grad_a,
                                                              float *__restrict__ grad_s0) {
    constexpr int kList = ONE ? 1 : kRollAgents * kEdgeStride;
    __shared__ float4 s_seg[kList];
    __shared__ float2 s_inv[kList];
    __shared__ float s_dc[kList];
    const int row = threadIdx.x / kRow, sub = threadIdx.x % kRow;
    const unsigned at = (blockIdx.y * gridDim.x + (unsigned)xcd_tile(blockIdx.x, gridDim.x)) * kRollAgents + row;
    if (at >= (unsigned)a.A) return;
    const int i = (int)at;
    const EdgeList ls{s_seg + row * kEdgeStride, s_inv + row * kEdgeStride, s_dc + row * kEdgeStride};
    const size_t A = (size_t)a.A;
    const float L = a.len[i], gxa = a.gx[i], gya = a.gy[i];
    const float iL = 1.0f / L;  // once per agent: the adjoint's divisions by L become products
    const float dt = a.dt, vmax = a.vmax;
    const int w = world_of_row(a.agent_off, a.W, i, sub);
    const int r0 = a.road_off[w];
    const EdgeGrid e{a.grid[w], a.ecell_start + (size_t)w * kCellStride, a.eseg + r0, a.eseg_id + r0};
    float lx = 0.f, ly = 0.f, lth = 0.f, lv = 0.f;  // adjoint of the state after the current step
    if (OBS == kObsScratch && Te < T) {
        const float4 q = carry[i];
        lx = q.x;
        ly = q.y;
        lth = q.z;
        lv = q.w;
    }
    EdgeBound bd{0.f, 0.f, 0.f, -1};
    // blocks of B steps, last one first
    for (int t0 = ONE ? 0 : (Te - 1) / B * B; t0 >= Ts; t0 -= B) {
        const int n = ONE ? 1 : min(B, Te - t0), t = t0 + sub;
        const bool on = sub < n;
        const float gr = on ? grad_r[(size_t)t * A + i] : 0.0f;
        float4 og_t = make_float4(0.f, 0.f, 0.f, 0.f);
        if (OBS == kObsScratch && on) og_t = og[(size_t)(t - Ts) * A + i];
        if (OBS == kObsGather && on) {
            const int a0 = a.agent_off[w];
            og_t = gather_obs_grad(a, slog, grad_obs, t, a0, a.agent_off[w + 1] - a0, i - a0, gxa, gya);
        }
        // states of the block, from the checkpoint before it
        const float *ck = ckpt + (size_t)(t0 / C) * 4 * A;
        AgentState c{ck[i], ck[A + i], ck[2 * A + i], ck[3 * A + i], 0.f, 0.f};
        sincosf(c.yaw, &c.sn, &c.cs);
        StepState o;
        float2 u;
        for (int tb = t0 / C * C;;) {
            const bool own = ONE || tb == t0;
            const int m = own ? n : min(kRow, t0 - tb);
            u = sub < m ? act[(size_t)(tb + sub) * A + i] : make_float2(0.f, 0.f);
            run_block<DELTA, ONE>(c, u, m, sub, L, dt, vmax, o);
            if (own) break;
            c = after_block(o, m);
            tb += m;
        }
        const EdgeChoice ch = nearest_edges<ONE>(e, ls, o.x1, o.y1, on, a.R_obs, sub, bd, false);
        // gradient of the step's reward (and observation) with respect to the state after
        // the step
        float gx = og_t.x, gy = og_t.y, gth = og_t.z, gv = og_t.w;
        const float sn = o.sn1, cs = o.cs1;
        // goal term: r = -|g'|
        {
            const float dxg = gxa - o.x1, dyg = gya - o.y1;
            const float gpx = cs * dxg + sn * dyg, gpy = -sn * dxg + cs * dyg;
            const float ng = sqrtf(gpx * gpx + gpy * gpy);
            if (ng > 0.0f) {
                const float ing = __builtin_amdgcn_rcpf(ng);
                const float bgx = -gpx * ing * gr, bgy = -gpy * ing * gr;
                gx += -cs * bgx + sn * bgy;
                gy += -sn * bgx - cs * bgy;
                gth += gpy * bgx - gpx * bgy;
            }
        }
        // off-road term: r = -softplus(side * |q'|), q' = a' + u e' in the ego frame
        if (ch.q >= 0) {
            const float4 s = e.es[ch.q];
            const float ax = s.x - o.x1, ay = s.y - o.y1, bx = s.z - o.x1, by = s.w - o.y1;
            const float apx = cs * ax + sn * ay, apy = -sn * ax + cs * ay;
            const float bpx = cs * bx + sn * by, bpy = -sn * bx + cs * by;
            const float ex = bpx - apx, ey = bpy - apy;
            const float ee = ex * ex + ey * ey;
            const float iee = __builtin_amdgcn_rcpf(ee);
            float uu = ee > 0.0f ? -(apx * ex + apy * ey) * iee : 0.0f;
            const bool cl = uu <= 0.0f || uu >= 1.0f;
            uu = fminf(fmaxf(uu, 0.0f), 1.0f);
            const float qx = apx + uu * ex, qy = apy + uu * ey;
            const float d = sqrtf(qx * qx + qy * qy);
            const float sdist = ch.side * d;
            const float sbar = -sigmoidf(sdist) * gr;
            const float dbar = ch.side * sbar;
            float bqx = 0.f, bqy = 0.f;
            if (d > 0.0f) {
                const float id = __builtin_amdgcn_rcpf(d);
                bqx = dbar * qx * id;
                bqy = dbar * qy * id;
            }
            float bapx = bqx, bapy = bqy, bex = uu * bqx, bey = uu * bqy;
            if (!cl && ee > 0.0f) {
                const float ubar = bqx * ex + bqy * ey;
                bapx += ubar * (-ex * iee);
                bapy += ubar * (-ey * iee);
                bex += ubar * (-apx * iee - 2.0f * uu * ex * iee);
                bey += ubar * (-apy * iee - 2.0f * uu * ey * iee);
            }
            const float bbpx = bex, bbpy = bey;
            bapx -= bex;
            bapy -= bey;
            const float bax = cs * bapx - sn * bapy, bay = sn * bapx + cs * bapy;
            const float bbx = cs * bbpx - sn * bbpy, bby = sn * bbpx + cs * bbpy;
            gx += -(bax + bbx);
            gy += -(bay + bby);
            gth += bapx * apy - bapy * apx + bbpx * bpy - bbpy * bpx;
        }
        // dynamics s_t -> s_{t+1}: coefficients of the adjoint's recursion
        //   lth <- lth + m1 lx + m2 ly,  lv <- n1 lx + n2 ly + n3 lth + n4 lv
        float m1 = 0.f, m2 = 0.f, n1 = 0.f, n2 = 0.f, n3 = 0.f, n4 = 1.f;
        float c1f = 0.f, c2f = 0.f;
        if (DELTA) {
            // d = v dt + a dt^2/2; x += d cos(yaw); y += d sin(yaw); yaw += s d; v += a dt
            m1 = -o.vb * o.sn0;
            m2 = o.vb * o.cs0;
            n1 = o.cs0 * dt;
            n2 = o.sn0 * dt;
            n3 = u.y * dt;
        } else {
            const float vb_raw = o.v0 + 0.5f * u.x * dt, vn_raw = o.v0 + u.x * dt;
            c1f = (vb_raw > -vmax && vb_raw < vmax) ? 1.0f : 0.0f;
            c2f = (vn_raw > -vmax && vn_raw < vmax) ? 1.0f : 0.0f;
            m1 = -o.vb * o.sp * dt;
            m2 = o.vb * o.cp * dt;
            n1 = c1f * (o.cp * dt);
            n2 = c1f * (o.sp * dt);
            n3 = c1f * (o.cb * o.ts * iL * dt);
            n4 = c2f;
        }
        if (!on) {
            gx = gy = gth = gv = 0.f;
            m1 = m2 = n1 = n2 = n3 = 0.f;
            n4 = 1.f;
        }
        // the recursion, last step first, on all lanes of the row; a lane keeps the adjoint
        // of the state after its step
        float kx = 0.f, ky = 0.f, kth = 0.f, kv = 0.f;
        auto back = [&](auto kc) {
            constexpr int k = decltype(kc)::k;
            lx += row_bcast<k>(gx);
            ly += row_bcast<k>(gy);
            lth += row_bcast<k>(gth);
            if (OBS) lv += row_bcast<k>(gv);
            const bool me = sub == k;
            kx = me ? lx : kx;
            ky = me ? ly : ky;
            kth = me ? lth : kth;
            kv = me ? lv : kv;
            const float v = row_bcast<k>(n4) * lv;
            lv = row_bcast<k>(n1) * lx + v;
            lv = row_bcast<k>(n2) * ly + lv;
            lv = row_bcast<k>(n3) * lth + lv;
            lth = row_bcast<k>(m1) * lx + lth;
            lth = row_bcast<k>(m2) * ly + lth;
        };
        if (ONE) back(StepIndex<0>{});
        else each_step_down(n, back);
        // gradient of the step's action
        float2 ga;
        if (DELTA) {
            const float bdist = kx * o.cs0 + ky * o.sn0 + kth * u.y;
            ga = make_float2(kv * dt + bdist * 0.5f * dt * dt, kth * o.vb);
        } else {
            const float sec2 = 1.0f + o.ts * o.ts;
            const float dbeta = 0.5f * sec2 * __builtin_amdgcn_rcpf(1.0f + 0.25f * o.ts * o.ts);
            const float bvb = kx * o.cp * dt + ky * o.sp * dt + kth * o.cb * o.ts * iL * dt;
            const float bphi = -kx * o.vb * o.sp * dt + ky * o.vb * o.cp * dt;
            const float bbeta = bphi - kth * o.vb * o.sb * o.ts * iL * dt;
            ga = make_float2(bvb * c1f * 0.5f * dt + kv * c2f * dt, kth * o.vb * o.cb * sec2 * iL * dt + bbeta * dbeta);
        }
        if (on) grad_a[(size_t)t * A + i] = ga;
    }
    if (OBS == kObsScratch && Ts > 0) {
        if (sub == 0) carry[i] = make_float4(lx, ly, lth, lv);
        return;
    }
    if (grad_s0 && sub == 0) {
        grad_s0[i] = lx;
        grad_s0[A + i] = ly;
        grad_s0[2 * A + i] = lth;
        grad_s0[3 * A + i] = lv;
    }
}

// Heading difference y1 - y0 wrapped to [-pi, pi), rounded once: the difference is kept
// as an unevaluated sum (two-sum, no multiplication involved), the multiple of 2 pi is
// removed with 2 pi split into a binary32 head (subtracted exactly) and tail.  A plain
// binary32 wrap of a log whose heading crosses +-pi would carry an absolute error of a
// few 1e-7 rad into the curvature command, divided by the distance of the step.
__device__ __forceinline__ float wrap_diff(float y1, float y0) {
    const float two_pi_hi = 6.28318548202514648f;   // binary32 nearest to 2 pi
    const float two_pi_lo = -1.74845553e-07f;       // 2 pi - two_pi_hi
    const float inv_two_pi = 0.159154943091895336f;
    const float pi_f = 3.14159265358979324f;
    const float a = y1 - y0;
    const float bb = a - y1;
    const float err = (y1 - (a - bb)) + (-y0 - bb);
    const float k = floorf((a + pi_f) * inv_two_pi);
    float r = fmaf(-k, two_pi_hi, a);
    r = r + (err - k * two_pi_lo);
    if (r >= pi_f) r = (r - two_pi_hi) - two_pi_lo;
    if (r < -pi_f) r = (r + two_pi_hi) + two_pi_lo;
    return r;
}

// Actions of one step of the simplified model from the heading and speed before (0) and
// after (1) it.
__device__ __forceinline__ float2 invert_step(float y0, float y1, float v0, float v1, float dt) {
    const float acc = (v1 - v0) / dt;
    const float d = 0.5f * (v0 + v1) * dt;
    const float w = wrap_diff(y1, y0);
    return make_float2(acc, fabsf(d) < 1e-3f ? 0.0f : w / d);
}

// Expert-action inversion of the simplified model, HBM-bound (reads heading and speed of
// each state once per chunk, writes each action once): one thread per agent and chunk
// of kInvChunk steps, all of the chunk's rows loaded before any action is formed.  Row
// t0 + kInvChunk is read by two chunks.  (Four agents per thread with 16-byte accesses
// measured slower.)
constexpr int kInvThreads = 256;
constexpr int kInvChunk = 16;

__global__ __launch_bounds__(kInvThreads) void k_invert_actions(const float *__restrict__ st, int T, int A,
                                                                float dt, float2 *__restrict__ act) {
    const int i = blockIdx.x * kInvThreads + threadIdx.x;
    if (i >= A) return;
    const size_t As = (size_t)A;
    const int t0 = blockIdx.y * kInvChunk;
    float yw[kInvChunk + 1], vv[kInvChunk + 1];
#pragma unroll
    for (int k = 0; k <= kInvChunk; k++) {
        const int t = t0 + k;
        yw[k] = 0.f;
        vv[k] = 0.f;
        if (t <= T) {
            const float *row = st + (size_t)t * 4 * As;
            yw[k] = row[2 * As + i];
            vv[k] = row[3 * As + i];
        }
    }
#pragma unroll
    for (int k = 0; k < kInvChunk; k++) {
        const int t = t0 + k;
        if (t < T) act[(size_t)t * As + i] = invert_step(yw[k], yw[k + 1], vv[k], vv[k + 1], dt);
    }
}

hipError_t launch_invert_actions_impl(const float *states, int T, int A, float dt, float *actions,
                                      hipStream_t s) {
    const int chunks = (T + kInvChunk - 1) / kInvChunk;
    if (chunks > 65535) return hipErrorInvalidValue;
    const dim3 grid((A + kInvThreads - 1) / kInvThreads, chunks);
    hipLaunchKernelGGL(k_invert_actions, grid, dim3(kInvThreads), 0, s, states, T, A, dt, (float2 *)actions);
    return hipGetLastError();
}

// launches a rollout kernel k, 16 agents per workgroup
template <typename K, typename... Args>
static hipError_t launch_rows(K k, const SimArgs &a, hipStream_t s, Args... args) {
    const Grid2 g = grid_of(((long long)a.A + kRollAgents - 1) / kRollAgents, kRollThreads);
    hipLaunchKernelGGL(k, dim3(g.x, g.y), dim3(kRollThreads), 0, s, a, args...);
    return hipGetLastError();
}

hipError_t launch_rollout_fwd_impl(const SimArgs &a, const float2 *actions, int T, int C,
                                   float *rewards, float *ckpt, float *states, hipStream_t s) {
    if (C < 1 || C > kMaxCkpt) return hipErrorInvalidValue;
    auto k = a.dyn == GD_DYN_DELTA ? (T == 1 ? k_rollout_fwd<true, true> : k_rollout_fwd<true, false>)
                                   : (T == 1 ? k_rollout_fwd<false, true> : k_rollout_fwd<false, false>);
    return launch_rows(k, a, s, actions, T, C, rewards, ckpt, states);
}

// lanes per agent of k_rollout_obs: the power of two that leaves the fewest lanes without a slot
static int obs_lanes(int P) {
    int best = kWave;
    for (int l = kWave / 2; l >= 8; l /= 2)
        if ((P + l - 1) / l * l < (P + best - 1) / best * best) best = l;
    return best;
}

// Agents per workgroup of the observation kernels: all of a world's, unless the `groups` workgroups
// that gives are fewer than four per compute unit; then a share, at most `most` of them.
// Below that a world's kernels take as long as its agents squared: 4 x 1000 agents, T = 5: forward
// 443 -> 86 us, backward 3641 -> 86; 1 x 128, T = 10: 26 -> 19 and 60 -> 24.
static int agents_per_group(int units, int max_agents, long long groups, int most) {
    const int shares = groups >= 4 * units ? 1 : (int)std::min(8 * units / groups, (long long)most);
    return std::max(1, (max_agents + std::max(shares, 1) - 1) / std::max(shares, 1));
}

hipError_t launch_rollout_obs_impl(const SimArgs &a, const float *states, int T, int max_agents, int units, float *obs,
                                   hipStream_t s) {
    // about 4096 slots per workgroup, 16 per thread; at least one step, states within 48 KB
    const long long slots = (long long)std::max(max_agents, 1) * std::max(a.P, 1);
    const int steps = (int)std::max(1ll, std::min({4096 / slots, (long long)T, 2048ll / std::max(max_agents, 1)}));
    const int share = agents_per_group(units, max_agents, (long long)a.W * ((T + steps - 1) / steps),
                                       (int)std::min((long long)max_agents, (slots + 4095) / 4096));
    const size_t lds = (size_t)steps * max_agents * (sizeof(float4) + sizeof(float2));
    const long long most = 65535ll * steps;  // (grid axis y)
    for (long long t0 = 0; t0 < T; t0 += most) {
        const int m = (int)std::min((long long)T - t0, most);
        hipLaunchKernelGGL(k_rollout_obs, dim3(a.W, (m + steps - 1) / steps, (max_agents + share - 1) / share),
                           dim3(kObsThreads), lds, s, a, states, (int)t0, T, steps, share, obs_lanes(a.P), obs);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <bool DELTA, bool ONE>
static hipError_t launch_bwd(const SimArgs &a, int units, const float2 *actions, const float *ckpt, int T, int C,
                             const float *grad_rewards, const float *grad_obs, const float *states, int max_agents,
                             void *scratch, float2 *grad_actions, float *grad_state0, hipStream_t s) {
    const int B = roll_block(T, C);
    if (!grad_obs || !scratch) {
        auto k = grad_obs ? k_rollout_bwd<DELTA, kObsGather, ONE> : k_rollout_bwd<DELTA, kObsNone, ONE>;
        return launch_rows(k, a, s, actions, ckpt, T, C, B, 0, T, grad_rewards, nullptr, nullptr, states, grad_obs,
                           grad_actions, grad_state0);
    }
    // the observation's gradient in parts of as many whole blocks as the scratch holds
    const ObsGradScratch L = obs_grad_scratch(a.A, T);
    float4 *og = (float4 *)scratch, *carry = (float4 *)((char *)scratch + L.carry);
    const int part = L.steps / B * B;
    const int share = agents_per_group(units, max_agents, (long long)a.W * std::min(T, part), (max_agents + 15) / 16);
    int cols = 8;  // lanes of an observer: as many as agents, a power of two
    while (cols < kWave && cols < max_agents) cols *= 2;
    const int rows = kWave / cols;
    // four observers per wave and pass, up to four waves, within 64 KB of LDS
    const int fit = std::max(1, (64 * 1024 / (int)sizeof(float4) - max_agents) / share - 1);
    const int waves = std::min({kObsThreads / kWave, fit, std::max(1, (max_agents + 4 * rows - 1) / (4 * rows))});
    const size_t lds = ((size_t)max_agents + (size_t)share * (1 + waves)) * sizeof(float4);
    for (int Ts = (T - 1) / part * part; Ts >= 0; Ts -= part) {
        const int Te = std::min(T, Ts + part);
        hipLaunchKernelGGL(k_rollout_obs_grad, dim3(a.W, Te - Ts, (max_agents + share - 1) / share), dim3(waves * kWave),
                           lds, s, a, states, Ts, share, grad_obs, og);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        if ((e = launch_rows(k_rollout_bwd<DELTA, kObsScratch, ONE>, a, s, actions, ckpt, T, C, B, Ts, Te, grad_rewards, og,
                             carry, nullptr, nullptr, grad_actions, grad_state0)) != hipSuccess)
            return e;
    }
    return hipSuccess;
}

hipError_t launch_rollout_bwd_impl(const SimArgs &a, int units, const float2 *actions, const float *ckpt, int T,
                                   int C, const float *grad_rewards, const float *grad_obs,
                                   const float *states, int max_agents, void *scratch, float2 *grad_actions,
                                   float *grad_state0, hipStream_t s) {
    if (C < 1 || C > kMaxCkpt) return hipErrorInvalidValue;
    auto f = a.dyn == GD_DYN_DELTA ? (T == 1 ? launch_bwd<true, true> : launch_bwd<true, false>)
                                   : (T == 1 ? launch_bwd<false, true> : launch_bwd<false, false>);
    return f(a, units, actions, ckpt, T, C, grad_rewards, grad_obs, states, max_agents, scratch, grad_actions, grad_state0, s);
}

}  // namespace gdk
