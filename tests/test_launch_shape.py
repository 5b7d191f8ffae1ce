"""The rule that chooses the step kernel's launch shape, run on the host: a candidate list with
room for agents at speed (512 entries, or 2 K) unless a shorter one keeps more workgroups on a
compute unit; explicit fields are kept; shapes fit the LDS."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r'''
#include <cstdio>
#include "gd_shape.h"
using namespace gdk;
// waves that the registers allow per compute unit
static int regs(int, bool staged, bool) { return staged ? 20 : 28; }
int main() {
    int cus, W, n, road, K, uneven, waves, bins, cands, mode;
    while (scanf("%d %d %d %d %d %d %d %d %d %d", &cus, &W, &n, &road, &K, &uneven, &waves, &bins, &cands, &mode) == 10) {
        gd_config c{};
        c.num_worlds = W; c.top_k = K; c.obs_radius = 50.f;
        c.obs_waves = waves; c.obs_bins = bins; c.obs_cands = cands; c.obs_road = mode;
        Batch b;
        b.compute_units = cus; b.worlds = W; b.max_agents = n; b.max_road = road; b.max_edges = road / 3; b.cell_cap4 = 488;
        b.agent_cap = (n + 3) / 4 * 4; b.uneven = uneven; b.idx16 = road < 65536;
        b.agents = uneven ? n / 2.0 : n; b.road = road; b.within = road * 0.07;
        Shape s;
        const bool ok = launch_shape(c, b, regs, s);
        auto fits = [&](int cc) {
            const size_t lds = step_lds_bytes(s.waves, s.bins, K, cc, s.road_cap, b.cell_cap4, s.edge_cap, b.agent_cap, b.idx16);
            return lds > (size_t)kLdsBytes ? 0 : std::min((int)((size_t)kLdsBytes / lds), regs(s.bins, s.road_cap > 0, b.idx16) / s.waves);
        };
        printf("%d %d %d %d %d %d", ok, s.waves, s.bins, s.cand_cap, s.road_cap, ok ? fits(s.cand_cap) : 0);
        for (int cc : {128, 256, 384, 512, 768, 1024}) printf(" %d", ok ? fits(cc) : 0);
        printf("\n");
    }
}
'''
LISTS = (128, 256, 384, 512, 768, 1024)


@pytest.fixture(scope="module")
def choose(tmp_path_factory):
    d = tmp_path_factory.mktemp("shape")
    (d / "s.cpp").write_text(PROGRAM)
    subprocess.check_call(["g++", "-std=c++17", "-O1", "-I", os.path.join(ROOT, "include"), "-I",
                           os.path.join(ROOT, "paper_2408_01584_amd", "csrc"), "-o", str(d / "s"), str(d / "s.cpp")])

    def run(batches, compute_units=256):
        text = "\n".join(" ".join(map(str, (compute_units, *b))) for b in batches)
        out = subprocess.check_output([str(d / "s")], input=text, text=True).splitlines()
        return [[int(v) for v in line.split()] for line in out]
    return run


BATCHES = [(W, n, road, K, uneven, 0, 0, 0, 0) for W in (1, 16, 256, 300, 1024, 4096) for n in (8, 32, 64, 128)
           for road in (500, 2700, 10000, 20000) for K in (32, 64, 100, 200, 500, 960) for uneven in (0, 1)]


def test_list_is_long_unless_it_costs_workgroups(choose):
    for b, (ok, waves, bins, cands, road, per_cu, *fits) in zip(BATCHES, choose(BATCHES)):
        K = b[3]
        assert ok and per_cu >= 1, b
        for cc, f in zip(LISTS, fits):
            if cands < cc <= max(512, 2 * K):
                assert f < per_cu, (b, cands, cc)


def test_explicit_fields_are_kept(choose):
    cases = [(256, 64, 4000, 200, 0, 8, 0, 0, 0), (256, 64, 4000, 200, 0, 0, 1024, 0, 0), (256, 64, 4000, 200, 0, 0, 0, 128, 0),
             (256, 64, 4000, 200, 0, 4, 64, 768, 2), (256, 64, 4000, 200, 0, 0, 0, 0, 1)]
    for b, (ok, waves, bins, cands, road, *_) in zip(cases, choose(cases)):
        assert ok
        assert b[5] in (0, waves) and b[6] in (0, bins) and b[7] in (0, cands)
        assert b[8] != 2 or road == 0
        assert b[8] != 1 or road >= 4000


def test_no_road_needs_no_list(choose):
    (ok, waves, bins, cands, *_), = choose([(64, 32, 2000, 0, 0, 0, 0, 0, 0)])
    assert ok and cands == 0


def test_what_does_not_fit_is_refused(choose):
    (ok, *_), = choose([(64, 64, 20000, 960, 0, 0, 0, 0, 1)])  # 320 KB of road in LDS
    assert not ok


def test_compute_units_of_the_device(choose):
    """An eighth of the worlds on an eighth of the compute units: the same shape."""
    whole = [b for b in BATCHES if b[0] >= 256 and b[0] % 8 == 0]
    part = [(b[0] // 8, *b[1:]) for b in whole]
    assert choose(whole) == choose(part, 32)
    assert choose(part) != choose(part, 32)


def test_grids_stay_below_2_to_32_threads(tmp_path):
    """A grid has every workgroup, less than one row too many, and no axis of 2^32 threads."""
    (tmp_path / "g.cpp").write_text(r'''
#include <cstdio>
#include "gd_shape.h"
int main() {
    for (long long groups : {1ll, (1ll << 23) - 1, 1ll << 23, (1ll << 23) + 1, 1ll << 24, (1ll << 27) - 3}) {
        const gdk::Grid2 g = gdk::grid_of(groups, 256);
        const long long all = (long long)g.x * g.y;
        if (g.x * 256ll >= (1ll << 32) || g.y > 65535 || all < groups || all - groups >= g.x) printf("wrong %lld\n", groups);
    }
}
''')
    subprocess.check_call(["g++", "-std=c++17", "-I", os.path.join(ROOT, "include"), "-I",
                           os.path.join(ROOT, "paper_2408_01584_amd", "csrc"), "-o", str(tmp_path / "g"), str(tmp_path / "g.cpp")])
    assert subprocess.check_output([str(tmp_path / "g")], text=True) == ""
