"""Records of the launch-shape tuner (no device): one made with another build of the library is not
used, and the tuner leaves the length of the candidate list to the library."""
import json

from paper_2408_01584_amd import scenes as S
from paper_2408_01584_amd import tune


def test_record_of_another_library_lapses(tmp_path, monkeypatch):
    sc = S.make_scene(0)
    cache = tmp_path / "shapes.json"
    monkeypatch.setattr(tune, "CACHE", str(cache))
    monkeypatch.setattr(tune, "_device_name", lambda: "gfx950:256")
    key = tune.signature(sc, sc.params, False) + "@gfx950:256"
    shape = {"obs_waves": 8, "obs_bins": 256, "cell_size": 15.0, "obs_road": 1}
    for library, want in ((tune._library(), shape), ("0" * 20, None)):
        cache.write_text(json.dumps({key: {"shape": shape, "ms_per_step": 0.01, "candidates": 1, "library": library}}))
        assert tune.cached_shape(sc) == want


def test_candidate_list_is_not_tuned():
    assert tune.DEFAULT_SPACE and all("obs_cands" not in s for s in tune.DEFAULT_SPACE)
