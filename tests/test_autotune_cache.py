"""The tuning cache without a GPU: what an entry or a plan is valid for."""

import shutil
import types

import pytest
import torch

from paper_1503_07659_amd import autotune, dgvol

ENTRY = {"variant": 0, "tile_cost_s": 1e-7, "by_class_variant": 0, "by_class_tile_cost_s": 1e-7, "single_variant": 0,
         "candidates_s_per_tile": {"0": 1e-7, "1": 2e-7}, "by_class_candidates_s_per_tile": {"0": 1e-7, "1": 3e-7}}


@pytest.fixture
def gpu(monkeypatch, tmp_path):
    """A device to name the cache's entries after, and an empty cache."""
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda d: types.SimpleNamespace(gcnArchName="gfx950:sramecc+", name="x"))
    monkeypatch.setenv("DGVOL_AUTOTUNE_CACHE", str(tmp_path / "cache.json"))
    return torch.device("cuda", 0)


def test_cache_belongs_to_one_build_of_the_library(gpu, monkeypatch, tmp_path):
    key = autotune.device_key(gpu)
    assert key == autotune.device_key(gpu) and key.startswith("gfx950/")
    autotune.save_cache({key: {autotune.entry_key(dgvol.FORM_F64, 35, 3): ENTRY},
                         "gfx950/abi4": {autotune.entry_key(dgvol.FORM_F64, 20, 3): ENTRY}})
    assert autotune.lookup(dgvol.FORM_F64, 35, 3, device=gpu, tune_missing=False) == ENTRY
    # an entry that does not say which build it measured
    assert autotune.lookup(dgvol.FORM_F64, 20, 3, device=gpu, tune_missing=False) is None
    # another build: same ABI version, other contents
    other = str(tmp_path / "libdgvol.so")
    shutil.copy(dgvol.LIB_PATH, other)
    monkeypatch.setattr(dgvol, "LIB_PATH", other)
    assert autotune.device_key(gpu) == key
    other2 = str(tmp_path / "libdgvol2.so")
    with open(dgvol.LIB_PATH, "rb") as src, open(other2, "wb") as dst:
        dst.write(src.read() + b"\0")
    monkeypatch.setattr(dgvol, "LIB_PATH", other2)
    assert autotune.device_key(gpu) != key
    assert autotune.lookup(dgvol.FORM_F64, 35, 3, device=gpu, tune_missing=False) is None
