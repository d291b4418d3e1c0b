"""The variant rule on the CPU: small launches split their items over element groups however long the windows are."""

import pytest

import paper_2604_06257_amd as das


@pytest.mark.parametrize("frames,max_window,n_tiles,items", [(4, 200, 300, 50.0), (4, 400, 256, 100.0), (6, 200, 300, 60.0),
                                                             (2, 700, 300, 1300.0), (1, 1500, 300, 1300.0), (16, 180, 64, 70.0)])
def test_small_launches_of_long_windows_are_split(frames, max_window, n_tiles, items, monkeypatch):
    monkeypatch.delenv("DAS_VARIANT", raising=False)
    fc, pitch, groups = das.choose_kernel_variant(frames, max_window, n_tiles, items)
    assert groups > 1 and pitch > max_window
