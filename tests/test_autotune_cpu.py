"""Autotuner host logic on the CPU: shape buckets, the candidate set and the
JSON cache (the timing itself needs a device)."""
import json

from paper_2008_00326_amd import autotune


def test_shape_bucket_groups_by_powers_of_two():
    a = autotune.shape_bucket(640 * 480, 9000, 2000, True)
    assert a == autotune.shape_bucket(640 * 480, 8200, 2300, True)
    assert a != autotune.shape_bucket(640 * 480, 9000, 2000, False)
    assert a != autotune.shape_bucket(320 * 240, 9000, 2000, True)
    assert a.startswith("px18-tri13-pose11-")


def test_candidates_are_valid_settings():
    defaults = {"small_block": 512, "small_words": 19440, "grid": [512, 256, 256, 64], "order": 2, "key_bands": 2}
    cands = autotune.candidates(defaults, 256)
    assert cands[0] == {"small_block": 512, "order": 2, "grid": [0, 0, 0, 0], "small_words": 0}   # the default first
    keys = {json.dumps(c, sort_keys=True) for c in cands}
    assert len(keys) == len(cands)                                                            # no duplicates
    for c in cands:
        assert c["small_block"] in (256, 512)
        assert c["order"] in (1, 2)
        assert len(c["grid"]) == 4 and all(g >= 0 for g in c["grid"])
        assert 0 <= c["small_words"] <= defaults["small_words"]
        assert c.get("key_bands", 0) in (0, 1, 2)


def test_cache_round_trip(tmp_path):
    path = str(tmp_path / "sub" / "tune.json")
    assert autotune.load_cache(path) == {}
    rec = {"gfx950|px18": {"tuning": {"small_block": 256}, "ms": 1.5}}
    autotune.save_cache(rec, path)
    assert autotune.load_cache(path) == rec
    (tmp_path / "sub" / "tune.json").write_text("{not json")
    assert autotune.load_cache(path) == {}


def test_a_candidate_must_beat_the_default_by_five_per_cent():
    trials = [{"tuning": "default", "ms": 100.0}, {"tuning": "a", "ms": 97.0}, {"tuning": "b", "ms": 99.0}]
    assert autotune.choose(trials)["tuning"] == "default"       # 3 % is within the spread
    trials.append({"tuning": "c", "ms": 94.0})
    assert autotune.choose(trials)["tuning"] == "c"             # 6 % faster
    assert autotune.choose(trials, min_gain=0.10)["tuning"] == "default"


class _Device:
    """A context whose class kernels take 2 ms by default, 1.8 ms with
    256-thread work-groups and 1 ms untuned."""

    def __init__(self):
        self.set = []

    def set_tuning(self, tuning):
        self.set.append(tuning)

    def tuning(self):
        return {"small_block": 512, "small_words": 19440, "grid": [512, 256, 256, 64], "order": 2, "key_bands": 2}

    def ms(self):
        return 1.0 if self.set[-1] is None else (1.8 if self.set[-1]["small_block"] == 256 else 2.0)


def _tune(monkeypatch, dev, n_poses, path):
    import torch
    monkeypatch.setattr(autotune, "device_arch", lambda device=0: "gfx950")
    monkeypatch.setattr(autotune, "_time", lambda ctx, items, reps, stream: ctx.ms())
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda d: type("Props", (), {"multi_processor_count": 256}))
    return autotune.autotune(dev, [{"poses": torch.zeros(n_poses, 12)}], "bucket", cache_path=path, stream=object())


def test_the_untuned_launch_is_what_a_candidate_has_to_beat(monkeypatch, tmp_path):
    """A class-kernel variant faster than the class kernels' defaults but
    slower than the untuned launch is not kept, timed or from the cache."""
    path = str(tmp_path / "tune.json")
    for cached in (False, True):
        dev = _Device()
        rec = _tune(monkeypatch, dev, 160, path)
        assert rec["cached"] == cached
        assert dev.set[-1] is None
        assert rec["default_ms"] == rec["ms"] == 1.0 and rec["gain_of_fastest"] == 0.0
        assert rec["trials"][0]["tuning"] == autotune.candidates(dev.tuning(), 256)[0]


def test_records_of_another_launch_size_or_base_are_not_applied(monkeypatch, tmp_path):
    path = str(tmp_path / "tune.json")
    old = {"gfx950|bucket": {"tuning": {"small_block": 256, "order": 2, "grid": [0, 0, 0, 0], "small_words": 0}}}
    autotune.save_cache(old, path)
    dev = _Device()
    assert not _tune(monkeypatch, dev, 160, path)["cached"]
    assert dev.set[-1] is None
    assert not _tune(monkeypatch, dev, 32000, path)["cached"]
    assert _tune(monkeypatch, dev, 32100, path)["cached"]
    assert not _tune(monkeypatch, dev, 161, path)["cached"]
