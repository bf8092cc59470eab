"""The autotuner's cache key of a batch (no GPU)."""
from paper_2601_16911_amd import autotune


class Batch:
    def signature(self):
        return "abc"


def test_batch_key_names_the_quantity(tmp_path, monkeypatch):
    """A number tuned as blocks per launch is not taken for blocks per work list."""
    path = str(tmp_path / "tune.json")
    monkeypatch.setattr(autotune, "arch", lambda: "gfx950")
    autotune.store("gfx950|batch|abc", {"grid": 256, "ms": 2.7}, path)
    assert autotune.batch_key(Batch()) not in autotune.load_cache(path)
