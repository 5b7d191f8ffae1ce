// Visvalingam-Whyatt decimation of road polylines at ingest (Sec. 3.1: densely sampled
// polylines, mostly straight, are thinned by dropping low-importance points, which cuts
// the point count, the memory and the step time).
//
// The effective area of an interior point is the area of the triangle it forms with its
// current neighbours.  Repeatedly, the interior point of smallest area (ties: lowest
// index) is removed and the areas of its two neighbours recomputed, until every remaining
// interior point has an area of at least min_area; end points always stay.  The areas
// decide which points survive, so they are computed in binary32 with a fixed operation
// order (no contraction).
//
// A polyline is taken by a wave (short ones) or a workgroup, with its points, areas and
// links (a doubly linked list of the surviving points) in LDS; longer ones keep areas and
// links in the caller's workspace.  The removals are sequential by definition, and taking
// them one at a time is a chain of LDS round trips and wave minima (about 1250 cycles
// each).  Here a round takes all the next removals that are certain at once.
//
// A key is (area bits, index): areas are >= 0, so their bit patterns order like the values;
// end points carry +inf and removed points a pattern above it.  Each thread owns every TH-th
// point and offers its smallest key, its level.  If a neighbour's area falls below the
// level once the offered point is gone, that neighbour is the next removal by definition, and so
// on: the thread follows this cascade, which leaves a gap between two surviving points l
// and r.  v is the smallest key that can come after it there: of l and r with their new
// areas, and of the thread's second smallest point.  An offer conflicts with a smaller one
// when the latter removes a point within two places of its own gap (so that gaps of one round
// share no neighbour); then its v is its level.  With T the minimum of all v, the offers
// below T with their cascades are exactly the next removals: what they create and everything
// not offered has a key of at least T, and gaps without a shared neighbour do not change
// each other's areas.  The smallest offer has no conflict and is below T, so every round
// removes a point.
//
// Bound by the vector instructions and the latency of the rounds (about 200 for a polyline of
// 2900 points).  2560 polylines of 2600 points on average (64 maps sampled every 0.1 m, 97 %
// of the points removed): one point at a time 9.2 ms, rounds that stop at the first cascade
// (700 of them) 7.9 ms, with cascades 1.64 ms; 128 or 512 threads per polyline instead of
// 256: 2.3 ms both.  16 B of LDS per point let a compute unit hold three polylines.
#include "gd_internal.h"

namespace gdk {

__device__ __forceinline__ float dec_area(const float *x, const float *y, int a, int b, int c) {
#pragma clang fp contract(off)
    const float ux = x[b] - x[a], uy = y[b] - y[a];
    const float vx = x[c] - x[a], vy = y[c] - y[a];
    const float p = ux * vy, q = uy * vx;
    return 0.5f * fabsf(p - q);
}

// minimum over the wave: row minima by DPP row rotations, then the four rows' minima
// through readlane (all 64 lanes must be active)
__device__ __forceinline__ unsigned wave_min_u32(unsigned v) {
    v = min(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, false));  // row_ror:8
    v = min(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x124, 0xf, 0xf, false));  // row_ror:4
    v = min(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x122, 0xf, 0xf, false));  // row_ror:2
    v = min(v, (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x121, 0xf, 0xf, false));  // row_ror:1
    const unsigned a = __builtin_amdgcn_readlane(v, 0), b = __builtin_amdgcn_readlane(v, 16);
    const unsigned c = __builtin_amdgcn_readlane(v, 32), d = __builtin_amdgcn_readlane(v, 48);
    return min(min(a, b), min(c, d));
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// area bits of a removed point: above every area, +inf (end points) and every NaN
constexpr unsigned kRemoved = 0xffffffffu;

using u64 = unsigned long long;
__device__ __forceinline__ u64 dec_key(float area, int k) { return ((u64)__float_as_uint(area) << 32) | (unsigned)k; }
constexpr int kCascade = 8;    // most removals that follow one offer in a round
constexpr int kDecUnroll = 4;  // points a thread reads together

// Shared by the TH threads of one polyline.
template <int TH>
struct DecShared {
    u64 claim[TH];         // by point modulo TH: the smallest level of a cascade that removes it
    u64 bound[2][TH / kWave];  // each wave's minimum of v, rounds in turn
};

// barrier over the TH threads of one polyline (a wave or a workgroup)
template <int TH>
__device__ __forceinline__ void dec_sync() {
    if (TH == kWave) wave_sync();
    else __syncthreads();
}

// One polyline of n points, X/Y its coordinates, AR/PRV/NXT its areas and links (local
// indices), keep/dir the outputs at its first point; tid = 0 .. TH - 1.  Removed points are
// marked in AR only (kRemoved), so that the removals touch no global memory when AR and the
// links sit in LDS; keep is written at the end.  PADDED: AR has room up to the next multiple of
// kDecUnroll * TH points.
template <int TH, typename Link, bool PADDED>
__device__ void vw_polyline(int n, int tid, DecShared<TH> &sh, const float *X, const float *Y, float *AR, Link *PRV,
                            Link *NXT, float min_area, uint8_t *keep, float *dir) {
    for (int k = tid; k < n; k += TH) {
        PRV[k] = (Link)(k - 1);
        NXT[k] = (Link)(k + 1);
        AR[k] = (k > 0 && k < n - 1) ? dec_area(X, Y, k - 1, k, k + 1) : INFINITY;
    }
    if (PADDED)
        for (int k = n + tid; k < (n + kDecUnroll * TH - 1) / (kDecUnroll * TH) * (kDecUnroll * TH); k += TH)
            AR[k] = __uint_as_float(kRemoved);
    sh.claim[tid] = ~0ull;
    dec_sync<TH>();
    const unsigned lim = __float_as_uint(min_area);  // areas >= 0 order like their bits
    // (every round removes a point: at most n - 2 of them)
    for (int left = n, round = 0; left > 0; left--, round ^= 1) {
        // this thread's smallest point and second smallest area (kDecUnroll loads in flight)
        unsigned m1 = kRemoved, m2 = kRemoved;
        int p = 0;
        for (int k0 = tid; k0 - tid < n; k0 += kDecUnroll * TH) {
            unsigned v[kDecUnroll];
#pragma unroll
            for (int u = 0; u < kDecUnroll; u++) {
                const int k = k0 + u * TH;
                v[u] = PADDED || k < n ? __float_as_uint(AR[k]) : kRemoved;
            }
#pragma unroll
            for (int u = 0; u < kDecUnroll; u++) {
                m2 = min(m2, max(m1, v[u]));
                p = v[u] < m1 ? k0 + u * TH : p;
                m1 = min(m1, v[u]);
            }
        }
        // (never an end point: 0 < p < n - 1; T is at most each thread's second smallest area, so
        // offers above the wave's smallest of those are left for a later round)
        const unsigned most = wave_min_u32(m2);  // (by all lanes)
        const bool offers = m1 < lim && m1 <= most;
        const u64 level = ((u64)m1 << 32) | (unsigned)p;
        int l = 0, r = 0, l2 = 0, r2 = 0;
        float nl = INFINITY, nr = INFINITY;
        u64 v = ~0ull;
        int conflict = 0;
        if (offers) {
            // the surviving neighbours l, r of the gap and the points beyond them (end
            // points stand for what is beyond them; their area is infinite)
            l = (int)PRV[p];
            r = (int)NXT[p];
            l2 = l > 0 ? (int)PRV[l] : l;
            r2 = r < n - 1 ? (int)NXT[r] : r;
            auto smaller = [&](int x) { return (int)(dec_key(AR[x], x) < level); };
            conflict = smaller(l) | smaller(r) | smaller(l2) | smaller(r2);
            for (int c = 0;; c++) {
                nl = dec_area(X, Y, l2, l, r);
                nr = dec_area(X, Y, l, r, r2);
                const u64 kl = dec_key(l > 0 ? nl : INFINITY, l), kr = dec_key(r < n - 1 ? nr : INFINITY, r);
                const u64 next = min(kl, kr);
                v = max(level + 1, min(next, (u64)m2 << 32));
                if (next > level || c == kCascade) break;
                atomicMin(&sh.claim[(kl < kr ? l : r) & (TH - 1)], level);
                if (kl < kr) {
                    l = l2;
                    l2 = l > 0 ? (int)PRV[l] : l;
                    conflict |= smaller(l2);
                } else {
                    r = r2;
                    r2 = r < n - 1 ? (int)NXT[r] : r;
                    conflict |= smaller(r2);
                }
            }
        }
        dec_sync<TH>();
        if (offers) {
            auto claimed = [&](int x) { return (int)(sh.claim[x & (TH - 1)] < level); };
            conflict |= claimed(l) | claimed(r) | claimed(l2) | claimed(r2);
            if (conflict) v = level;
        }
        const unsigned hi = wave_min_u32((unsigned)(v >> 32));
        const unsigned lo = wave_min_u32((unsigned)(v >> 32) == hi ? (unsigned)v : 0xffffffffu);
        u64 T = ((u64)hi << 32) | lo;
        if (TH > kWave) {
            if ((tid & (kWave - 1)) == 0) sh.bound[round][tid / kWave] = T;
            dec_sync<TH>();
#pragma unroll
            for (int w = 0; w < TH / kWave; w++) T = min(T, sh.bound[round][w]);
        }
        if (T == ~0ull) break;  // no offers: what remains spans at least min_area
        sh.claim[tid] = ~0ull;
        if (offers && level < T) {
            for (int x = (int)NXT[l]; x != r; x = (int)NXT[x]) AR[x] = __uint_as_float(kRemoved);
            NXT[l] = (Link)r;
            PRV[r] = (Link)l;
            if (l > 0) AR[l] = nl;
            if (r < n - 1) AR[r] = nr;
        }
        dec_sync<TH>();
    }
    for (int k = tid; k < n; k += TH) {
        const bool kept = __float_as_uint(AR[k]) != kRemoved;
        float d = 0.0f;
        if (kept) {
            const int j = (int)NXT[k];
            if (j < n) {
                d = atan2f(Y[j] - Y[k], X[j] - X[k]);
            } else if (k > 0) {
                const int pk = (int)PRV[k];
                d = atan2f(Y[k] - Y[pk], X[k] - X[pk]);
            }
        }
        keep[k] = kept ? 1 : 0;
        dir[k] = d;
    }
}

struct DecArgs {
    const int *off;
    int n_poly, n_points;
    const float *x, *y;
    float min_area;
    uint8_t *keep;
    float *dir;
    float *area;     // workspace
    int *prv, *nxt;
};

// Polyline pl as [s, e): offsets clamped into [0, n_points] and made non-decreasing: malformed
// offsets give a wrong answer, never an access outside the buffers
__device__ __forceinline__ int dec_range(const DecArgs &a, int pl, int &s) {
    s = min(max(a.off[pl], 0), a.n_points);
    return min(max(a.off[pl + 1], s), a.n_points) - s;
}

constexpr int kDecShort = 512;    // points of a polyline taken by one wave (8 per lane)
constexpr int kDecThreads = 256;  // threads of a longer one
constexpr int kDecPoints = 3072;  // points staged in LDS (16 B each): three workgroups of a compute unit
constexpr int kDecLinks = 6144;   // points whose areas and links fit the same LDS (8 B each)

// Polylines of up to kDecShort points, a wave each.
constexpr int kDecShortWaves = 4;
__global__ __launch_bounds__(kDecShortWaves *kWave) void k_decimate_short(DecArgs a) {
    __shared__ float sx[kDecShortWaves][kDecShort], sy[kDecShortWaves][kDecShort], sa[kDecShortWaves][kDecShort];
    __shared__ unsigned short sp[kDecShortWaves][kDecShort], sn[kDecShortWaves][kDecShort];
    __shared__ DecShared<kWave> shared[kDecShortWaves];
    const int g = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int tid = threadIdx.x % kWave;
    const int pl = blockIdx.x * kDecShortWaves + g;
    if (pl >= a.n_poly) return;
    int s;
    const int n = dec_range(a, pl, s);
    if (n < 1 || n > kDecShort) return;
    for (int k = tid; k < n; k += kWave) {
        sx[g][k] = a.x[s + k];
        sy[g][k] = a.y[s + k];
    }
    wave_sync();
    vw_polyline<kWave, unsigned short, true>(n, tid, shared[g], sx[g], sy[g], sa[g], sp[g], sn[g], a.min_area, a.keep + s,
                                       a.dir + s);
}

// Polylines of up to kDecLinks points, a workgroup each: with their points in LDS when they
// fit, else the points are read through the caches.
__global__ __launch_bounds__(kDecThreads) void k_decimate(DecArgs a) {
    __shared__ float mem[kDecPoints * 4];
    __shared__ DecShared<kDecThreads> shared;
    static_assert(kDecPoints * 4 == kDecLinks * 2, "one block of LDS");
    static_assert(kDecPoints % (kDecUnroll * kDecThreads) == 0 && kDecLinks % (kDecUnroll * kDecThreads) == 0, "padded");
    const int tid = threadIdx.x;
    int s;
    const int n = dec_range(a, blockIdx.x, s);
    if (n <= kDecShort || n > kDecLinks) return;
    if (n <= kDecPoints) {
        float *sx = mem, *sy = mem + kDecPoints, *sa = mem + 2 * kDecPoints;
        unsigned short *sp = reinterpret_cast<unsigned short *>(mem + 3 * kDecPoints);
        for (int k = tid; k < n; k += kDecThreads) {
            sx[k] = a.x[s + k];
            sy[k] = a.y[s + k];
        }
        __syncthreads();
        vw_polyline<kDecThreads, unsigned short, true>(n, tid, shared, sx, sy, sa, sp, sp + kDecPoints, a.min_area, a.keep + s,
                                                 a.dir + s);
    } else {
        unsigned short *sp = reinterpret_cast<unsigned short *>(mem + kDecLinks);
        vw_polyline<kDecThreads, unsigned short, true>(n, tid, shared, a.x + s, a.y + s, mem, sp, sp + kDecLinks, a.min_area,
                                                 a.keep + s, a.dir + s);
    }
}

// Polylines of more than kDecLinks points, areas and links in the workspace.
constexpr int kDecLong = 1024;
__global__ __launch_bounds__(kDecLong) void k_decimate_long(DecArgs a) {
    __shared__ DecShared<kDecLong> shared;
    for (int pl = blockIdx.x; pl < a.n_poly; pl += gridDim.x) {
        int s;
        const int n = dec_range(a, pl, s);
        if (n <= kDecLinks) continue;
        __syncthreads();
        vw_polyline<kDecLong, int, false>(n, threadIdx.x, shared, a.x + s, a.y + s, a.area + s, a.prv + s, a.nxt + s, a.min_area,
                             a.keep + s, a.dir + s);
    }
}

// The lengths are on the device, so each kernel that n_points allows is launched and its
// workgroups leave the other polylines alone.
hipError_t launch_decimate_impl(const int *poly_off, int n_poly, int n_points, const float *x, const float *y,
                                float min_area, uint8_t *keep, float *dir, void *ws, hipStream_t s) {
    if (n_poly <= 0) return hipSuccess;
    char *w = (char *)ws;
    // (-0 is 0: its bits would order above every area)
    const DecArgs a{poly_off, n_poly, n_points, x, y, min_area == 0.0f ? 0.0f : min_area, keep, dir, (float *)w,
                    (int *)(w + decimate_ws_offset(n_points, 1)), (int *)(w + decimate_ws_offset(n_points, 2))};
    const unsigned short_blocks = (unsigned)(((long long)n_poly + kDecShortWaves - 1) / kDecShortWaves);
    hipLaunchKernelGGL(k_decimate_short, dim3(short_blocks), dim3(kDecShortWaves * kWave), 0, s, a);
    if (n_points > kDecShort) hipLaunchKernelGGL(k_decimate, dim3(n_poly), dim3(kDecThreads), 0, s, a);
    if (n_points > kDecLinks)
        hipLaunchKernelGGL(k_decimate_long, dim3(n_poly < 65536 ? n_poly : 65536), dim3(kDecLong), 0, s, a);
    return hipGetLastError();
}

}  // namespace gdk
