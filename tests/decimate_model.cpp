// Host model of the decimation by chunks (gd_decimate.hip: dec_begin, the rule of vw_any, vw_chunks),
// with the removals of chunks that run at the same time interleaved at random, and the
// definition: one removal after the other.  Compiled by tests/test_decimate_model.py.
#include <algorithm>
#include <cmath>
#include <cstdint>
#include <cstring>
#include <random>
#include <vector>

namespace {
using u64 = uint64_t;
constexpr int kReach = 4, kNear = 2, kChunk = 5, kChunkAgain = 8, kShort = 512, kChunked = 4096;

unsigned bits(float f) {
    unsigned u;
    memcpy(&u, &f, 4);
    return u;
}
u64 key_of(float a, int k) { return ((u64)bits(a) << 32) | (unsigned)k; }

struct Polyline {
    int n;
    const float *x, *y;
    float area(int a, int b, int c) const {  // (compiled without contraction)
        const float ux = x[b] - x[a], uy = y[b] - y[a], vx = x[c] - x[a], vy = y[c] - y[a];
        const float p = ux * vy, q = uy * vx;
        return 0.5f * std::fabs(p - q);
    }
};

std::vector<uint8_t> definition(const Polyline &pl, float lim) {
    const int n = pl.n;
    std::vector<float> ar(n, INFINITY);
    std::vector<int> prv(n), nxt(n);
    std::vector<uint8_t> keep(n, 1);
    for (int k = 0; k < n; k++) {
        prv[k] = k - 1;
        nxt[k] = k + 1;
        if (k > 0 && k < n - 1) ar[k] = pl.area(k - 1, k, k + 1);
    }
    for (;;) {
        int q = -1;
        for (int k = 1; k < n - 1; k++)
            if (keep[k] && ar[k] < lim && (q < 0 || ar[k] < ar[q])) q = k;
        if (q < 0) return keep;
        const int l = prv[q], r = nxt[q];
        keep[q] = 0;
        nxt[l] = r;
        prv[r] = l;
        if (l > 0) ar[l] = pl.area(prv[l], l, r);
        if (r < n - 1) ar[r] = pl.area(l, r, nxt[r]);
    }
}

struct Chunks {
    const Polyline &pl;
    int threads;
    unsigned lim;
    std::mt19937 &rng;
    std::vector<float> ar;
    std::vector<uint8_t> gone_;
    std::vector<int> prv, nxt, gap, lst;
    bool touched_twice = false;

    void begin() {
        const int n = pl.n;
        ar.assign(n, INFINITY);
        gone_.assign(n, 0);
        prv.resize(n);
        nxt.resize(n);
        gap.assign(n, -1);
        lst.resize(n);
        for (int k = 0; k < n; k++) {
            prv[k] = k - 1;
            nxt[k] = k + 1;
            lst[k] = k;
            if (k > 0 && k < n - 1) ar[k] = pl.area(k - 1, k, k + 1);
        }
    }
    // (an area of a removed point is the time of its removal)
    u64 gap_time(int k) const { return gap[k] < 0 ? 0 : key_of(ar[gap[k]], gap[k]); }

    bool run(int chunk) {
        const int n = pl.n;
        int gone = 0;
        for (;;) {
            const int m = n - gone, start = gone;
            const int chunks = std::max(1, std::min(threads, m / chunk)), per = m / chunks, rest = m % chunks;
            std::vector<int> c0(chunks), c1(chunks), count(chunks);
            for (int t = 0; t < chunks; t++) {
                c0[t] = t * per + std::min(t, rest);
                c1[t] = c0[t] + per + (t < rest);
                count[t] = c1[t] - c0[t];
            }
            auto smallest = [&](int t) {
                u64 best = ~0ull;
                for (int j = c0[t]; j < c1[t]; j++)
                    if (!gone_[lst[j]] && bits(ar[lst[j]]) < lim) best = std::min(best, key_of(ar[lst[j]], lst[j]));
                return best;
            };
            bool wrong = false;
            for (;;) {
                std::vector<u64> first(chunks), bound(chunks);
                for (int t = 0; t < chunks; t++) first[t] = smallest(t);
                const std::vector<int> left = count;
                std::vector<int> acting;
                for (int t = 0; t < chunks; t++) {
                    u64 b = ~0ull;
                    int before = 0, after = 0;
                    for (int u = 1; u <= kNear; u++) {
                        if (t - u >= 0 && before < kReach) b = std::min(b, first[t - u]);
                        if (t + u < chunks && after < kReach) b = std::min(b, first[t + u]);
                        before += left[std::max(t - u, 0)];
                        after += left[std::min(t + u, chunks - 1)];
                    }
                    if ((t > kNear && before < kReach) || (t + 1 + kNear < chunks && after < kReach)) b = 0;
                    bound[t] = b;
                    if (first[t] < b) acting.push_back(t);
                }
                std::vector<int> toucher(n, -1);  // the chunk that wrote a point in this round
                int did = 0;
                while (!acting.empty()) {
                    const size_t i = rng() % acting.size();
                    const int t = acting[i];
                    const u64 key = smallest(t);
                    if (!(key < bound[t])) {
                        acting.erase(acting.begin() + i);
                        continue;
                    }
                    const int p = (int)(unsigned)key, l = prv[p], r = nxt[p];
                    for (int k : {l, p, r}) {
                        if (k > 0 && k < n - 1 && toucher[k] >= 0 && toucher[k] != t) touched_twice = true;
                        toucher[k] = t;
                    }
                    const bool inl = l > 0, inr = r < n - 1;
                    const int l2 = inl ? prv[l] : l, r2 = inr ? nxt[r] : r;
                    const u64 gl = gap_time(l), gp = gap_time(p), time = std::max(key, std::max(gl, gp));
                    const u64 kl = key_of(ar[l], l), kr = key_of(ar[r], r);
                    if (inl && (time < gap_time(l2) || (kl < time && gl != time))) wrong = true;
                    if (inr && (time < gap_time(r) || (kr < time && gp != time))) wrong = true;
                    gone_[p] = 1;
                    nxt[l] = r;
                    prv[r] = l;
                    gap[l] = (int)(unsigned)time;
                    if (inl) {
                        ar[l] = pl.area(l2, l, r);
                        if (l < lst[c0[t]]) bound[t] = std::min(bound[t], key_of(ar[l], l));
                    }
                    if (inr) {
                        ar[r] = pl.area(l, r, r2);
                        if (r > lst[c1[t] - 1]) bound[t] = std::min(bound[t], key_of(ar[r], r));
                    }
                    count[t]--;
                    did++;
                }
                gone += did;
                if (wrong) return false;
                if (did == 0 || (gone - start) * 8 >= m) break;
            }
            if (gone == start) return true;
            lst.clear();
            for (int k = 0; k < n; k++)
                if (!gone_[k]) lst.push_back(k);
        }
    }
};
}  // namespace

extern "C" {
// keep masks of the n_poly polylines by the definition in `keep`; path[p]: 0 one at a time by the
// rule, 1 and 2 by chunks at the first and second attempt, 3 one at a time after them.  Returns the
// number of polylines for which a passed attempt differs from the definition, or 1 000 000 if
// two chunks wrote one point in the same round.
int decimate_model(const int *off, int n_poly, const float *x, const float *y, float min_area, unsigned seed,
                   uint8_t *keep, int *path) {
    std::mt19937 rng(seed);
    int bad = 0;
    for (int p = 0; p < n_poly; p++) {
        const Polyline pl{off[p + 1] - off[p], x + off[p], y + off[p]};
        const int n = pl.n;
        path[p] = 0;
        if (n < 1) continue;
        const std::vector<uint8_t> want = definition(pl, min_area);
        std::copy(want.begin(), want.end(), keep + off[p]);
        Chunks c{pl, n <= kShort ? 64 : 256, bits(min_area), rng, {}, {}, {}, {}, {}, {}};
        c.begin();
        int below = 0, ties = 0;
        for (int k = 0; k < n; k++) {
            const bool in = c.ar[k] < min_area;
            below += in;
            ties += in && k % 16 && bits(c.ar[k]) == bits(c.ar[k - 1]);
        }
        const bool some = ties * 4 > below, half = ties * 7 > below * 3, most = ties * 9 > below * 5;
        if (n > kChunked || !(n > (some ? 160 : 128)) || (n > kShort && n <= kChunked / 2 ? most : half)) continue;
        path[p] = 3;
        for (int attempt = 1; attempt <= (some ? 1 : 2); attempt++) {
            c.begin();
            const bool ok = c.run(attempt == 1 ? kChunk : kChunkAgain);
            if (c.touched_twice) return 1000000;
            if (!ok) continue;
            path[p] = attempt;
            for (int k = 0; k < n; k++)
                if (want[k] == c.gone_[k]) {
                    bad++;
                    break;
                }
            break;
        }
    }
    return bad;
}
}
