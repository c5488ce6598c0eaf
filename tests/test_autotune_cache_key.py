"""A cached choice is taken for the same plate only, and not from a version
whose choices stood for other kernels (no GPU)."""
import json

from paper_2208_13769_amd import autotune


class Plate:
    device = 0

    def __init__(self, kinds=(0, 0, 0, 0), mask=False):
        self.kinds, self.mask = kinds, mask

    def edges(self):
        return self.kinds, self.mask


def test_choices_are_kept_per_edges_and_mask(tmp_path, monkeypatch):
    import torch

    cache = tmp_path / "autotune.json"
    cache.write_text(json.dumps({"card|300x200|fp64|pc|v7": {"tiling": [64, 1, 1]}}))
    monkeypatch.setenv("LBM_AUTOTUNE_CACHE", str(cache))
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda device: "card")
    tuned = []
    monkeypatch.setattr(autotune, "tune", lambda *a: tuned.append(a) or ((256, len(tuned), 2), 0.1, []))

    def best(*plate):
        return tuple(autotune.best_tiling(Plate(*plate), 300, 200, "fp64", "pc"))

    plates = [((0, 0, 0, 0), False), ((0, 0, 1, 2), False), ((0, 0, 2, 2), False), ((2, 2, 2, 2), False),
              ((2, 2, 2, 2), True), ((0, 0, 0, 0), True)]
    first = [best(*p) for p in plates]
    assert len(tuned) == len(plates)  # (the entry of the older version is not taken)
    assert [best(*p) for p in plates] == first and len(tuned) == len(plates)
