"""The tile cache keeps a choice for launches of one kernel and one for launches of several (host
only): both survive a file, and a file that holds only one leaves the other to the heuristic."""
import pytest

import paper_2009_07482_amd as psc
from test_persist_host import fnv1a64


@pytest.fixture(autouse=True)
def clean_cache():
    psc.psc_tile_cache_clear()
    yield
    psc.psc_tile_cache_clear()


def _body(path):
    text = open(path).read()
    return sorted(x for x in text.splitlines() if x.split()[0] in ("entry", "shared"))


def _file(path, lines):
    body = "psc-tile-cache 1\nkey k\n" + "".join(x + "\n" for x in lines)
    open(path, "w").write(body + "checksum %016x\n" % fnv1a64(body.encode()))


def test_both_choices_survive_a_file(tmp_path):
    path = str(tmp_path / "tiles")
    _file(path, ["entry 512 64 512 1 1 12", "shared 512 64 512 1 1 6", "shared 8 8 8 0 0 2", "entry 9 9 9 0 0 3"])
    psc.psc_tile_cache_set(9, 9, 9, "f32", "f32", 7)           # replaced whole: no shared choice is left
    assert psc.psc_tile_cache_load(path, "k") == 3
    assert psc.psc_tile_cache_get(512, 64, 512, "bf16", "bf16") == 12
    assert psc.psc_tile_cache_get(8, 8, 8, "f32", "f32") == 0
    again = str(tmp_path / "again")
    psc.psc_tile_cache_save(again, "k")
    assert _body(again) == _body(path)
    assert psc.psc_tile_cache_clear() == 3


def test_a_set_tile_serves_both_and_zero_removes_both(tmp_path):
    path = str(tmp_path / "tiles")
    psc.psc_tile_cache_set(64, 64, 64, "f32", "f32", 4)
    psc.psc_tile_cache_save(path, "k")
    assert _body(path) == ["entry 64 64 64 0 0 4", "shared 64 64 64 0 0 4"]
    psc.psc_tile_cache_set(64, 64, 64, "f32", "f32", 0)
    assert psc.psc_tile_cache_clear() == 0


@pytest.mark.parametrize("line", ["shared 8 8 8 0 0 99", "shared 8 8 8 0 0", "both 8 8 8 0 0 2"])
def test_bad_lines_load_nothing(tmp_path, line):
    path = str(tmp_path / "tiles")
    _file(path, ["entry 4 4 4 0 0 2", line])
    with pytest.raises(psc.PscError) as e:
        psc.psc_tile_cache_load(path, "k")
    assert e.value.status == psc.PSC_ERR_IO
    assert psc.psc_tile_cache_clear() == 0
