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


@pytest.mark.parametrize("by_class,cost", [(False, 2e-7), (True, 3e-7)])
def test_plan_keeps_the_default_of_small_calls(gpu, by_class, cost):
    """FP64 order 5: the variant tuned on a large problem (0 here) is not forced on a call below the
    size at which the library's default changes."""
    autotune.save_cache({autotune.device_key(gpu): {autotune.entry_key(dgvol.FORM_F64, Np, 3): ENTRY for Np in (35, 56)}})
    group = lambda Np, K: (None, None, types.SimpleNamespace(shape=(K, 3, Np), device=gpu, numel=lambda: K * 3 * Np))  # noqa: E731
    edge = dgvol.ORDER5_DIRECT_MAX_VALUES // (3 * 56)
    plan = lambda *gr: autotune.plan(list(gr), tune_missing=False, by_class=by_class)  # noqa: E731
    assert plan(group(56, edge)) == ([dgvol.VARIANT_AUTO], [cost])
    assert plan(group(56, edge + 1)) == ([0], [1e-7])
    assert plan(group(56, edge), group(35, 1)) == ([0, 0], [1e-7, 1e-7])  # the call as a whole is past it
    assert plan(group(56, 100), group(35, 1)) == ([dgvol.VARIANT_AUTO, 0], [cost, 1e-7])
    broken = dict(ENTRY, candidates_s_per_tile=["x"], by_class_candidates_s_per_tile={"1": "y"})
    autotune.save_cache({autotune.device_key(gpu): {autotune.entry_key(dgvol.FORM_F64, 56, 3): broken}})
    assert plan(group(56, 100)) == ([dgvol.VARIANT_AUTO], [0.0])
