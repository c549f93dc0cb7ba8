"""A tune-cache entry written for other kernels is not applied: its key lacks
this library's revision, so the autotuner times the shapes again and appends its
own entry, which later lattices take."""

import json

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_1708_09689_amd as pv  # noqa: E402


def lattice():
    return pv.Lattice((17, 13, 11), (1, 0, 1), pv.pv_model_stencil(pv.PV_MODEL_TI, [1.0, 2.0, 0.0, 0.0]))


def test_entries_of_another_revision_are_timed_again(tmp_path):
    cache = tmp_path / "tune.jsonl"
    pv.pv_autotune(lattice(), 2, pv.PV_C128, cache_path=str(cache))
    entry = json.loads(cache.read_text())
    # the entry as the first revision wrote it, and one of a later revision, with
    # a shape that no search returns
    former, rev = entry["key"].rsplit(" rev=", 1)
    shape = {k: v for k, v in entry.items() if k != "key"}
    shape.update(kernel=2, elems_per_lane=1, strip_rows=77)
    later = "%s rev=%d" % (former, int(rev) + 1)
    cache.write_text("".join(json.dumps({"key": k, **shape}) + "\n" for k in (former, later)))
    lat = lattice()
    t, ms = pv.pv_autotune(lat, 2, pv.PV_C128, cache_path=str(cache))
    assert ms > 0.0 and t["strip_rows"] != 77
    lines = cache.read_text().splitlines()
    assert len(lines) == 3 and json.loads(lines[2])["key"] == entry["key"]
    t2, ms2 = pv.pv_autotune(lattice(), 2, pv.PV_C128, cache_path=str(cache))
    assert ms2 == 0.0 and t2 == t
