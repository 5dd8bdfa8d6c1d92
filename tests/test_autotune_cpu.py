"""The tuner's search and cache without a GPU (timings planted): entries of plans built on
other kernels are timed again, and FFT lines are searched only where they have an effect."""
import json
from types import SimpleNamespace

import pytest
import torch

from paper_2606_01598_amd import autotune


@pytest.fixture
def timed(monkeypatch):
    seen = []

    def fake(cfg, mesh, *rest):
        seen.append((tuple(mesh), cfg))
        return 1.0 + 0.1 * sum(cfg.tile) - 0.01 * cfg.fft_lines
    monkeypatch.setattr(autotune, "_time_candidate", fake)
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda d: SimpleNamespace(gcnArchName="gfx950:sramecc+"))
    return seen


def _box(mesh, n=100):
    return {"mesh": mesh, "pos": torch.zeros(n, 3), "q": None, "mu": None, "box": None, "v": None}


def test_entries_of_earlier_kernels_are_timed_again(timed, tmp_path):
    path = tmp_path / "tiles.json"
    mesh = (27, 27, 27)
    for version in (1, 2):
        key = autotune._key("gfx950", mesh, 6, 100).replace(f"v{autotune.VERSION}|", f"v{version}|")
        path.write_text(json.dumps({key: {"tile": [16, 16, 16], "fft_lines": 4, "ms": 0.1}}))
        configs, n = autotune.tune([_box(mesh)], 6, 0.3, cache_path=str(path))
        assert n == 1 and configs[0].tile == (8, 8, 8) and configs[0].fft_lines == 32
    timed.clear()
    assert autotune.tune([_box(mesh)], 6, 0.3, cache_path=str(path))[1] == 0 and not timed


@pytest.mark.parametrize("mesh,lines", [((64, 64, 64), True), ((100, 100, 100), True),
                                        ((20, 400, 18), True), ((160, 160, 160), False),
                                        ((20, 135, 160), False), ((6, 20, 1024), False)])
def test_lines_are_searched_on_slab_meshes_only(timed, tmp_path, mesh, lines):
    autotune.tune([_box(mesh)], 6, 0.3, cache_path=str(tmp_path / "t.json"))
    tried = [cfg.fft_lines for _, cfg in timed]
    assert tried == [0] * len(autotune.CANDIDATES) + (list(autotune.LINES) if lines else [])
