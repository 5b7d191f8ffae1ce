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
// The removals are sequential by definition, and taking them one at a time (vw_single) is a chain
// of LDS round trips and wave minima.  Up to 4096 points a polyline is taken by chunks that run
// ahead of each other (vw_chunks: a wave up to 512 points, a workgroup beyond) unless it is short
// or mostly ties, or the chunks took it out of order; longer ones round by round (vw_polyline,
// areas and links in LDS up to 6144 points, else in the caller's workspace).
//
// Rounds: every removal that is certain to be among the next ones is taken at once.
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
// 2560 polylines of 2600 points on average (64 maps sampled every 0.1 m, 97 % of the points
// removed): one point at a time 9.2 ms, rounds 1.64 ms (190 of 4500 cycles), chunks 0.80 to 0.87 ms.
// On straight lines, whose areas are all equal, nothing can be taken at the same time: 512 lines
// of 2600 points 1.19 ms one at a time, 2.2 ms by chunks.  Beyond 4096 points rounds are faster also
// there than one wave that searches everything again (straight 5000 points 19.7 and 34.1 ms,
// 7000 points 51 and 75; 1/4 m raster 15.0 and 29.8, 43 and 68).
#include <algorithm>

#include "gd_internal.h"

namespace gdk {

__device__ __forceinline__ float dec_area(float2 a, float2 b, float2 c) {
#pragma clang fp contract(off)
    const float ux = b.x - a.x, uy = b.y - a.y;
    const float vx = c.x - a.x, vy = c.y - a.y;
    const float p = ux * vy, q = uy * vx;
    return 0.5f * fabsf(p - q);
}
__device__ __forceinline__ float2 dec_point(const float *x, const float *y, int k) {
    return make_float2(x[(unsigned)k], y[(unsigned)k]);  // (32-bit offsets from scalar bases)
}
__device__ __forceinline__ float dec_area(const float *x, const float *y, int a, int b, int c) {
    return dec_area(dec_point(x, y, a), dec_point(x, y, b), dec_point(x, y, c));
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
constexpr unsigned kSign = 0x80000000u;

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

// Outputs of a polyline whose removed points have the sign bit of their area set (areas are
// >= 0, end points +inf).
template <int TH, typename Link>
__device__ __forceinline__ void write_kept(int n, int tid, const float *X, const float *Y, const float *AR,
                                           const Link *PRV, const Link *NXT, uint8_t *keep, float *dir) {
    for (int k = tid; k < n; k += TH) {
        const bool kept = !(__float_as_uint(AR[k]) & kSign);
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

// One polyline of n points, X/Y its coordinates, AR/PRV/NXT its areas and links (local
// indices), keep/dir the outputs at its first point; tid = 0 .. TH - 1.  Removed points are
// marked in AR only (kRemoved), so that the removals touch no global memory when AR and the
// links sit in LDS; keep is written at the end.  PADDED: AR has room up to the next multiple of
// kDecUnroll * TH points.
template <int TH, typename Link, bool PADDED>
__device__ __forceinline__ void vw_polyline(int n, int tid, DecShared<TH> &sh, const float *X, const float *Y, float *AR, Link *PRV,
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
    write_kept<TH>(n, tid, X, Y, AR, PRV, NXT, keep, dir);
}

// ---- the same removals, one at a time, by one wave
// Lane c keeps the smallest key of the 64 points from 64 c on.  A removal takes its own chunk's
// smallest key, so that chunk is searched again; in a neighbour's chunk only if the neighbour
// was its smallest and grew.  Bound by one chain of latencies per removal, about 900 cycles: two
// wave minima, two dependent reads of links, the coordinates, and stores.  AR, PRV and NXT are set; removed points are marked in AR (kRemoved); point(k) gives the coordinates.
constexpr int kDecSingle = kWave * kWave;  // points, at most

template <typename P>
__device__ __forceinline__ void vw_single(int n, int lane, P &&point, float *AR, unsigned short *PRV, unsigned short *NXT,
                                          float min_area) {
    const unsigned lim = __float_as_uint(min_area);  // areas >= 0 order like their bits
    unsigned bb = kRemoved;  // smallest area of this lane's chunk, and its first point
    int bk = 0;
    // searches chunk c, whose point 64 c + lane has area bits v on this lane
    auto search = [&](int c, unsigned v) {
        const unsigned m = wave_min_u32(v);
        const int first = __ffsll((long long)__builtin_amdgcn_ballot_w64(v == m)) - 1;
        bb = lane == c ? m : bb;
        bk = lane == c ? c * kWave + first : bk;
    };
    auto area_bits = [&](int c) {
        const int k = c * kWave + lane;
        const unsigned v = __float_as_uint(AR[min(k, n - 1)]);
        return k < n ? v : kRemoved;
    };
    for (int c = 0; c * kWave < n; c++) search(c, area_bits(c));
    for (;;) {
        const unsigned m = wave_min_u32(bb);
        if (!(m < lim)) break;  // (also when only end points remain)
        // (chunks are in order: the first that holds the minimum has its lowest index)
        const int q = __builtin_amdgcn_readlane(bk, __ffsll((long long)__builtin_amdgcn_ballot_w64(bb == m)) - 1);
        const int cq = q >> 6;
        const unsigned vq = area_bits(cq);
        const int l = PRV[q], r = NXT[q];
        const int bl = PRV[l], br = NXT[r], l2 = l > 0 ? bl : l, r2 = r < n - 1 ? br : r;
        const float2 xl2 = point(l2), xl = point(l), xr = point(r), xr2 = point(r2);
        const float al = dec_area(xl2, xl, xr), ar = dec_area(xl, xr, xr2);
        const unsigned nl = __float_as_uint(l > 0 ? al : INFINITY), nr = __float_as_uint(r < n - 1 ? ar : INFINITY);
        if (lane == 0) {
            NXT[l] = (unsigned short)r;
            PRV[r] = (unsigned short)l;
            AR[q] = __uint_as_float(kRemoved);
            AR[l] = __uint_as_float(nl);
            AR[r] = __uint_as_float(nr);
        }
        wave_sync();
        const int k = cq * kWave + lane;
        search(cq, k == q ? kRemoved : k == l ? nl : k == r ? nr : vq);
        // the neighbours' chunks, where they are others (end points keep their area)
        auto neighbour = [&](int p, unsigned v) {
            const int c = p >> 6;
            if (c == cq) return;
            const bool me = lane == c, less = v < bb || (v == bb && p < bk);
            if (__builtin_amdgcn_ballot_w64(me && bk == p && !less) != 0ull) {
                search(c, area_bits(c));
            } else {
                bb = me && less ? v : bb;
                bk = me && less ? p : bk;
            }
        };
        const int sl = __builtin_amdgcn_readfirstlane(l), sr = __builtin_amdgcn_readfirstlane(r);
        if (sl > 0) neighbour(sl, nl);
        if (sr < n - 1) neighbour(sr, nr);
    }
}

// ---- the same removals, by chunks of the polyline that run ahead of each other
// The order of two removals matters only if they are neighbours.  Each thread owns a chunk of
// consecutive surviving points and takes its own next removals as long as their keys are
// below the smallest keys of the chunks around it, as far as the next four points on each
// side reach: between two chunks that take removals at the same time there are four points
// or more, and each touches two of them.  What a thread cannot know is whether a cascade will
// come through these chunks with smaller keys later.  That is checked instead:
// the time of a removal is its key, or the time of the removal that caused it if that is
// larger (a cascade), and each gap between surviving points knows the time of the last
// removal in it.  A removal reads the point's two gaps and changes the areas of its two
// neighbours, so for it to come in order
//   - the removals in its own two gaps must not be later: they are not, one of them caused it
//     if the point's key is smaller;
//   - the removals in the two gaps beyond its neighbours must not be later;
//   - a neighbour with a key before this time would have gone first, unless it lies, like
//     the point, at the gap of the cascade that this removal belongs to.
// When every removal passes, any two that touch each other's points were taken in the order of
// their times, and no point was passed over at its time, so sorted by their times they are
// the removals of the definition.  When one does not pass, the polyline is taken again with
// larger chunks, then by vw_single: never on straight lines and circles, on 1 of 7000 noisy
// curves, on up to 19 % of random points on a few integer positions.  (5.6 million polylines
// compared with the definition by a host model that interleaves the chunks at random.)  When an eighth of the points is gone the chunks are dealt out anew.
//
// Bound by the latency of a removal (about 1700 cycles: six dependent LDS reads, the
// coordinates through the caches, the chunk's next key) times the 150 or so that follow one
// another on some thread of a polyline of 2600 points in 50 rounds.  12 B of LDS per point let
// a compute unit hold three polylines; with the coordinates in LDS too (20 B) it took as
// long.  Chunks of 4 or 6 points and deals after a quarter or a half of them were 1 to 20 %
// slower, mostly for the few polylines taken again (1 to 5 of the 2560, at the end of the
// launch): those are first taken with chunks of 8, which pass (12 instead: up to 5 % slower).
constexpr int kChunk = 5, kChunkAgain = 8;  // points of a chunk, at least: at first, and when taken again
constexpr int kReach = 4;  // points between two chunks that take removals
constexpr int kNear = 2;   // chunks on each side in which it looks for them
constexpr int kOwn = 16;   // points of its chunk that a thread keeps in registers
constexpr unsigned short kNoGap = 0xffff;

template <int TH>
struct ChunkShared {
    u64 first[TH];  // smallest key of each chunk
    unsigned short count[TH];  // its surviving points
    int part[TH / kWave];
    int removed, wrong;
    int below, ties;  // areas below the limit, and how many of them equal their neighbour's
};

template <int TH>
union DecAnyShared {
    DecShared<TH> rounds;
    ChunkShared<TH> chunks;
};

// Areas, links and the rest that vw_chunks starts from.  Ties are counted among the 16 lanes of a
// row, in 15 of 16 places.
template <int TH>
__device__ __forceinline__ void dec_begin(int n, int tid, ChunkShared<TH> &sh, const float *X, const float *Y, float *AR,
                                          unsigned short *PRV, unsigned short *NXT, unsigned short *G,
                                          unsigned short *LST, float min_area) {
    if (tid == 0) sh.removed = sh.wrong = sh.below = sh.ties = 0;
    dec_sync<TH>();  // (also the polyline or the attempt before)
    int below = 0, ties = 0;  // of the wave
    for (int k0 = 0; k0 < n; k0 += TH) {
        const int k = k0 + tid;
        float area = INFINITY;
        if (k < n) {
            if (k > 0 && k < n - 1) area = dec_area(X, Y, k - 1, k, k + 1);
            PRV[k] = (unsigned short)(k - 1);
            NXT[k] = (unsigned short)(k + 1);
            AR[k] = area;
            G[k] = kNoGap;
            LST[k] = (unsigned short)k;
        }
        const int v = __float_as_int(area), before = __builtin_amdgcn_update_dpp(~v, v, 0x111, 0xf, 0xf, false);  // row_shr:1
        const bool in = area < min_area;
        below += __popcll(__builtin_amdgcn_ballot_w64(in));
        ties += __popcll(__builtin_amdgcn_ballot_w64(in && v == before));
    }
    if ((tid & (kWave - 1)) == 0) {
        atomicAdd(&sh.below, below);
        atomicAdd(&sh.ties, ties);
    }
    dec_sync<TH>();
}

// G: by point, the point whose key is the time of the last removal in the gap after it (its
// area stays in AR, with the sign bit set); LST: the surviving points in order.  False: a
// removal was out of order, nothing is valid.  At most MOST points.
template <int TH, int MOST>
__device__ __forceinline__ bool vw_chunks(int n, int tid, ChunkShared<TH> &sh, const float *X, const float *Y, float *AR,
                          unsigned short *PRV, unsigned short *NXT, unsigned short *G, unsigned short *LST,
                          float min_area, int chunk) {
    const unsigned lim = __float_as_uint(min_area);  // areas >= 0 order like their bits
    auto gap = [&](int k) -> u64 {  // (no branch: the reads of a removal go out together)
        const int g = G[k], h = g == kNoGap ? 0 : g;
        const u64 t = ((u64)(__float_as_uint(AR[h]) & ~kSign) << 32) | (unsigned)g;
        return g == kNoGap ? 0ull : t;
    };
    int gone = 0;  // removals so far
    // (every part but the last removes a point, and every round but the last of a part)
    for (;;) {
        const int m = n - gone, start = gone;
        const int chunks = max(1, min(TH, m / chunk)), per = m / chunks, rest = m % chunks;
        const bool mine = tid < chunks;
        const int c0 = mine ? tid * per + min(tid, rest) : 0, c1 = mine ? c0 + per + (tid < rest) : 0;
        const int lo = mine ? (int)LST[c0] : 0, hi = mine ? (int)LST[c1 - 1] : 0;
        int count = c1 - c0;
        // the chunk's smallest key (removed points have the sign bit, above every limit); its
        // first points are kept in registers
        int own[kOwn];
#pragma unroll
        for (int u = 0; u < kOwn; u++) own[u] = LST[max(min(c0 + u, c1 - 1), 0)];
        auto smallest = [&]() -> u64 {
            unsigned a = lim;
            int p = -1;
            auto take = [&](auto first) {
                unsigned v[kOwn / 2];
#pragma unroll
                for (int u = 0; u < kOwn / 2; u++) v[u] = __float_as_uint(AR[own[first() + u]]);
#pragma unroll
                for (int u = 0; u < kOwn / 2; u++) {
                    p = v[u] < a ? own[first() + u] : p;
                    a = min(a, v[u]);
                }
            };
            take([] { return 0; });
            if (per >= kOwn / 2) {
                take([] { return kOwn / 2; });
                for (int j = c0 + kOwn; j < c1; j++) {
                    const int k = LST[j];
                    const unsigned w = __float_as_uint(AR[k]);
                    p = w < a ? k : p;
                    a = min(a, w);
                }
            }
            return p < 0 ? ~0ull : ((u64)a << 32) | (unsigned)p;
        };
        bool wrong = false;
        for (;;) {
            u64 key = smallest();
            sh.first[tid] = key;
            sh.count[tid] = (unsigned short)count;
            dec_sync<TH>();
            // the chunks around this one, kNear on each side read together; where fewer than
            // kReach points are left in them the thread waits for the next deal
            u64 bound = 0ull;
            if (mine) {
                u64 before[kNear], after[kNear];
                int nb[kNear], na[kNear];
#pragma unroll
                for (int u = 0; u < kNear; u++) {
                    const int cb = max(tid - 1 - u, 0), ca = min(tid + 1 + u, chunks - 1);
                    before[u] = sh.first[cb];
                    nb[u] = sh.count[cb];
                    after[u] = sh.first[ca];
                    na[u] = sh.count[ca];
                }
                bound = ~0ull;
                int seenb = 0, seena = 0;
#pragma unroll
                for (int u = 0; u < kNear; u++) {
                    if (tid - 1 - u >= 0 && seenb < kReach) bound = min(bound, before[u]);
                    if (tid + 1 + u < chunks && seena < kReach) bound = min(bound, after[u]);
                    seenb += nb[u];
                    seena += na[u];
                }
                if ((tid > kNear && seenb < kReach) || (tid + 1 + kNear < chunks && seena < kReach)) bound = 0ull;
            }
            int did = 0;
            while (key < bound) {
                const int p = (int)(unsigned)key;
                const int l = PRV[p], r = NXT[p];
                const bool inl = l > 0, inr = r < n - 1;
                const int bl = PRV[l], br = NXT[r], l2 = inl ? bl : l, r2 = inr ? br : r;
                const float2 xl2 = dec_point(X, Y, l2), xl = dec_point(X, Y, l);
                const float2 xr = dec_point(X, Y, r), xr2 = dec_point(X, Y, r2);
                const float nl = dec_area(xl2, xl, xr), nr = dec_area(xl, xr, xr2);
                const u64 gl = gap(l), gp = gap(p), gl2 = gap(l2), gr = gap(r);
                const u64 time = max(key, max(gl, gp));
                const u64 kl = dec_key(AR[l], l), kr = dec_key(AR[r], r);
                wrong |= (inl & ((time < gl2) | ((kl < time) & (gl != time)))) |
                         (inr & ((time < gr) | ((kr < time) & (gp != time))));
                AR[p] = __uint_as_float((unsigned)(key >> 32) | kSign);
                NXT[l] = (unsigned short)r;
                PRV[r] = (unsigned short)l;
                G[l] = (unsigned short)time;
                if (inl) AR[l] = nl;
                if (inr) AR[r] = nr;
                // a neighbour in another chunk is taken there (keys from the limit on never)
                if (inl && l < lo) bound = min(bound, dec_key(nl, l));
                if (inr && r > hi) bound = min(bound, dec_key(nr, r));
                did++;
                key = smallest();
            }
            count -= did;
            if (did) atomicAdd(&sh.removed, did);
            if (wrong) sh.wrong = 1;
            dec_sync<TH>();
            const bool idle = sh.removed == gone;
            gone = sh.removed;
            if (sh.wrong) return false;
            if (idle || (gone - start) * 8 >= m) break;
        }
        if (gone == start) return true;
        // the surviving points in order: a thread counts those of a stretch of the polyline (of an
        // odd length: lanes read different banks)
        const int len = ((n + TH - 1) / TH) | 1, s0 = tid * len, s1 = min(n, s0 + len);
        constexpr int kStretch = MOST / TH + 1;
        unsigned there = 0;
#pragma unroll
        for (int u = 0; u < kStretch; u++) {
            const int k = min(s0 + u, n - 1);
            there |= (unsigned)(s0 + u < s1 && !(__float_as_uint(AR[k]) & kSign)) << u;
        }
        const int alive = __popc(there);
        const int upto = wave_incl_scan(alive);
        if ((tid & (kWave - 1)) == kWave - 1) sh.part[tid / kWave] = upto;
        dec_sync<TH>();
        int at = upto - alive;
        for (int w = 0; w < tid / kWave; w++) at += sh.part[w];
        for (; there; there &= there - 1) LST[at++] = (unsigned short)(s0 + __ffs((int)there) - 1);
        dec_sync<TH>();
    }
}

constexpr int kDecShort = 512;    // points of a polyline taken by one wave (8 per lane)
constexpr int kDecChunked = 4096;  // points taken by chunks (12 B of LDS each)

// The removals of a polyline of up to MOST points, by chunks or one at a time.  The chunks need
// points that can be removed at the same time, and equal areas leave few: with index order
// among them a run of ties is a chain.  So polylines with ties in more than 3 of 7 places
// (straight lines along an axis, lines on a raster, walks on one) are taken one at a time; with a
// workgroup up to 2048 points more than 5 of 9, as the larger ones mostly come out of order.  And
// short ones: up to 128 points, or 160 where more than a quarter ties (straight lines whose areas
// are rounding).  One at a time and by chunks, us: straight 2600 points 1122 and 2018 (1559 before
// there were chunks), 1/4 m raster 981 and 1241 (1210); walk on integers 300 points 74 and 137
// (88), 1000 points 210 and 126 (257), 4096 points 815 and 1165 (984); oblique line of 150 points
// 71 and 93 (84), of 300 139 and 137; noisy curve of 100 points 47 and 56 (55), of 200 92 and 68.
// mem: areas and links of `stride` points (8 B each), then what the chunks need (4 B) or the
// coordinates of `room` points (8 B).
template <int TH, int MOST>
__device__ __forceinline__ void vw_any(int n, int tid, ChunkShared<TH> &sh, const float *X, const float *Y, float *mem,
                                       int stride, int room, float min_area) {
    static_assert(MOST <= kDecSingle, "one chunk per lane of a wave");
    float *AR = mem;
    unsigned short *PRV = reinterpret_cast<unsigned short *>(mem + stride), *NXT = PRV + stride, *G = NXT + stride;
    dec_begin<TH>(n, tid, sh, X, Y, AR, PRV, NXT, G, G + stride, min_area);
    const int below = sh.below, ties = sh.ties;
    const bool some = ties * 4 > below, half = ties * 7 > below * 3, most = ties * 9 > below * 5;
    if (n > (some ? 160 : 128) && !(n > kDecShort && n <= kDecChunked / 2 ? most : half)) {
        for (int chunk = kChunk; chunk <= kChunkAgain; chunk += kChunkAgain - kChunk) {
            if (vw_chunks<TH, MOST>(n, tid, sh, X, Y, AR, PRV, NXT, G, G + stride, min_area, chunk)) return;
            dec_begin<TH>(n, tid, sh, X, Y, AR, PRV, NXT, G, G + stride, min_area);
            if (some) break;  // (larger chunks would hardly pass)
        }
    }
    if (n <= room) {
        float2 *xy = reinterpret_cast<float2 *>(G);
        for (int k = tid; k < n; k += TH) xy[k] = dec_point(X, Y, k);
        dec_sync<TH>();
        if (tid < kWave) vw_single(n, tid, [&](int k) { return xy[k]; }, AR, PRV, NXT, min_area);
    } else if (tid < kWave) {
        vw_single(n, tid, [&](int k) { return dec_point(X, Y, k); }, AR, PRV, NXT, min_area);
    }
    dec_sync<TH>();
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

constexpr int kDecThreads = 256;   // threads of a longer one
// points taken one at a time with their coordinates in LDS (16 B each) where chunks take 12 B
constexpr int kDecShortStaged = kDecShort * 3 / 4, kDecStaged = 3072;
constexpr int kDecLinks = 6144;   // points whose areas and links fit the LDS (8 B each)

// A workgroup (or wave) takes every kDecMaxBlocks-th group of polylines: grids are limited to
// 2^32 threads, which n_poly with a workgroup each can exceed.
constexpr int kDecMaxBlocks = 1 << 20;

// Polylines of up to kDecShort points, a wave each.
constexpr int kDecShortWaves = 4;
__global__ __launch_bounds__(kDecShortWaves *kWave) void k_decimate_short(DecArgs a) {
    __shared__ __align__(16) float mem[kDecShortWaves][3 * kDecShort];
    static_assert(kDecShortStaged * 4 <= kDecShort * 3, "one block of LDS");
    __shared__ ChunkShared<kWave> shared[kDecShortWaves];
    const int g = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const int tid = threadIdx.x % kWave;
    for (long long pl = (long long)blockIdx.x * kDecShortWaves + g; pl < a.n_poly; pl += (long long)gridDim.x * kDecShortWaves) {
        int s;
        const int n = dec_range(a, (int)pl, s);
        if (n < 1 || n > kDecShort) continue;
        const float *x = a.x + s, *y = a.y + s;
        const int stride = n <= kDecShortStaged ? kDecShortStaged : kDecShort;
        vw_any<kWave, kDecShort>(n, tid, shared[g], x, y, mem[g], stride, kDecShortStaged, a.min_area);
        const unsigned short *prv = reinterpret_cast<unsigned short *>(mem[g] + stride);
        write_kept<kWave>(n, tid, x, y, mem[g], prv, prv + stride, a.keep + s, a.dir + s);
    }
}

// Polylines of up to kDecLinks points, a workgroup each: round by round from kDecChunked points on.
__global__ __launch_bounds__(kDecThreads) void k_decimate(DecArgs a) {
    __shared__ __align__(16) float mem[kDecLinks * 2];
    __shared__ DecAnyShared<kDecThreads> shared;
    static_assert(kDecChunked * 3 <= kDecLinks * 2 && kDecStaged * 4 <= kDecLinks * 2, "one block of LDS");
    static_assert(kDecLinks % (kDecUnroll * kDecThreads) == 0, "padded");
    const int tid = threadIdx.x;
    for (long long pl = blockIdx.x; pl < a.n_poly; pl += gridDim.x) {
        int s;
        const int n = dec_range(a, (int)pl, s);
        if (n <= kDecShort || n > kDecLinks) continue;
        if (n <= kDecChunked) {
            const int stride = n <= kDecStaged ? kDecStaged : kDecChunked;
            vw_any<kDecThreads, kDecChunked>(n, tid, shared.chunks, a.x + s, a.y + s, mem, stride, kDecStaged, a.min_area);
            const unsigned short *prv = reinterpret_cast<unsigned short *>(mem + stride);
            write_kept<kDecThreads>(n, tid, a.x + s, a.y + s, mem, prv, prv + stride, a.keep + s, a.dir + s);
            continue;
        }
        __syncthreads();
        unsigned short *link = reinterpret_cast<unsigned short *>(mem + kDecLinks);
        vw_polyline<kDecThreads, unsigned short, true>(n, tid, shared.rounds, a.x + s, a.y + s, mem, link, link + kDecLinks,
                                                       a.min_area, a.keep + s, a.dir + s);
    }
}

// Polylines of more than kDecLinks points, areas and links in the workspace.  A workgroup looks
// through every gridDim.x-th polyline, a thread each: few workgroups, as there is usually nothing
// to do for them (10 000 polylines of 2 points: 24.0 us a call with a workgroup each, 19.6 so).
constexpr int kDecLong = 1024, kDecLongBlocks = 512;
__global__ __launch_bounds__(kDecLong) void k_decimate_long(DecArgs a) {
    __shared__ DecShared<kDecLong> shared;
    __shared__ int found[kDecLong], count;
    for (long long p0 = blockIdx.x; p0 < a.n_poly; p0 += (long long)gridDim.x * kDecLong) {
        __syncthreads();
        if (threadIdx.x == 0) count = 0;
        __syncthreads();
        const long long pl = p0 + (long long)gridDim.x * threadIdx.x;
        int s = 0;
        if (pl < a.n_poly && dec_range(a, (int)pl, s) > kDecLinks) found[atomicAdd(&count, 1)] = (int)pl;
        __syncthreads();
        const int m = count;
        for (int k = 0; k < m; k++) {
            const int n = dec_range(a, found[k], s);
            __syncthreads();
            vw_polyline<kDecLong, int, false>(n, threadIdx.x, shared, a.x + s, a.y + s, a.area + s, a.prv + s, a.nxt + s,
                                              a.min_area, a.keep + s, a.dir + s);
        }
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
    auto blocks = [&](int per) { return dim3((unsigned)std::min(((long long)n_poly + per - 1) / per, (long long)kDecMaxBlocks)); };
    hipLaunchKernelGGL(k_decimate_short, blocks(kDecShortWaves), dim3(kDecShortWaves * kWave), 0, s, a);
    if (n_points > kDecShort) hipLaunchKernelGGL(k_decimate, blocks(1), dim3(kDecThreads), 0, s, a);
    if (n_points > kDecLinks)
        hipLaunchKernelGGL(k_decimate_long, dim3(std::min(n_poly, kDecLongBlocks)), dim3(kDecLong), 0, s, a);
    return hipGetLastError();
}

}  // namespace gdk
