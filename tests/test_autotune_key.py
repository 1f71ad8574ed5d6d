"""The key under which tuned strip rows are kept (host only): rows tuned for
other kernels, or for rows that the kernel cuts into another number of strips,
are not taken for this batch's."""
import json
from types import SimpleNamespace

import pytest

import paper_1812_04135_amd as R
from paper_1812_04135_amd import autotune

torch = pytest.importorskip("torch")


@pytest.fixture
def device(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda d: "card")


def _batch(boxes, xbc="periodic"):
    cfgs = [{"n": [nx, ny, 1], "bc_lo": [xbc, "reflect"], "form": "pvs"} for nx, ny in boxes]
    b = SimpleNamespace(prec="fp64", cfgs=cfgs, shapes=[(4, ny, nx) for nx, ny in boxes], rows=None)
    b.set_tiles = lambda rows: setattr(b, "rows", list(rows))
    return b


BOXES = [(60, 64), (61, 64), (200, 100), (256, 256)]


def test_key_names_the_library_revision(device, monkeypatch, tmp_path):
    b = _batch(BOXES)
    now = autotune.batch_key(b)
    cache = tmp_path / "tiles.json"
    cache.write_text(json.dumps({now: {"strip_rows": [16, 64, 128, 128], "ms": 1.0, "nsteps": 20}}))
    assert autotune.tune(b, None, cache=str(cache)) == ([16, 64, 128, 128], 1.0, True)
    assert b.rows == [16, 64, 128, 128]
    # another revision: the kept rows are not found (the tuner goes on to
    # measure, which this stand-in cannot)
    monkeypatch.setattr(R, "rsst_version", lambda: "rsst-gfx950 another")
    assert autotune.batch_key(b) != now
    with pytest.raises(AttributeError):
        autotune.tune(b, None, cache=str(cache))


def test_key_tells_rows_of_one_and_two_strips_apart(device):
    assert autotune.batch_key(_batch(BOXES)) != autotune.batch_key(_batch(BOXES, "reflect"))
    assert autotune.batch_key(_batch([(60, 64)])) == autotune.batch_key(_batch([(60, 64)], "reflect"))
    assert [autotune.row_strips(n, True) for n in (4, 64, 65, 120, 121, 256)] == [1, 1, 2, 2, 3, 5]
    assert [autotune.row_strips(n, False) for n in (4, 60, 61, 64, 65)] == [1, 1, 2, 2, 2]
