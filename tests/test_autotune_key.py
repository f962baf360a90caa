"""The autotuner's stored choice belongs to one build of the library and to the settings that select
kernels: under anything else the same window is timed again."""
import dataclasses
import types

import pytest

torch = pytest.importorskip("torch")
from paper_2507_03737_amd import autotune, binding  # noqa: E402


@pytest.fixture
def window(monkeypatch, tmp_path):
    lib = tmp_path / "lib.so"
    lib.write_bytes(b"one build")
    monkeypatch.setattr(binding, "LIB_PATH", str(lib))
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda device=None: "device")
    return types.SimpleNamespace(T_cw=torch.zeros(1, 12), sizes=[(480, 640)]), lib


def test_key_is_stable(window):
    win, _ = window
    cfg = binding.RasterConfig()
    assert autotune.cache_key(win, 100, cfg) == autotune.cache_key(win, 100, dataclasses.replace(cfg, tile=32, pixels_per_lane=2))


def test_key_follows_the_library(window):
    win, lib = window
    before = autotune.cache_key(win, 100, binding.RasterConfig())
    lib.write_bytes(b"another build")
    assert autotune.cache_key(win, 100, binding.RasterConfig()) != before


@pytest.mark.parametrize("change", [{"bwd_lane_reduce": 1}, {"count_work": 1}, {"mark_visible": 1}, {"pointmap_frame": 0}])
def test_key_follows_settings_that_select_kernels(window, change):
    win, _ = window
    cfg = binding.RasterConfig()
    assert autotune.cache_key(win, 100, dataclasses.replace(cfg, **change)) != autotune.cache_key(win, 100, cfg)
