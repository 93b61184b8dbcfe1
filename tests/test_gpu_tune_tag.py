"""The tune cache holds picks of several libraries: only those of this one are used."""
import pytest

from paper_2101_07163_amd import snowlb as S
from paper_2101_07163_amd import workloads as W

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")


@pytest.mark.parametrize("batch", [False, True])
def test_picks_of_earlier_kernels_are_not_used(batch, tmp_path, monkeypatch):
    """L7 is the tag of the library before the step kernels with computed tiles: a line with it leaves a new context to tune."""
    path = tmp_path / "tune.txt"
    monkeypatch.setenv("SNOWLB_TUNE_CACHE", str(path))
    monkeypatch.setenv("SNOWLB_TUNE_STEPS", "2")
    c = dict(W.C3)
    c.update(nx=100, ny=60, seed=(30.0, 30.0, 6.0))

    def make():
        return S.Batch([c, c], tile=-1) if batch else S.Sim(c, tile=-1)

    make().init().step(2)
    tag, rest = path.read_text().split(" ", 1)
    key = rest.rsplit(" ", 2)[0]
    path.write_text("L7 %s 4 5\n" % key)
    sim = make().init()
    assert sim.tile != 4
    sim.step(2)
    lines = path.read_text().splitlines()
    assert len(lines) == 2 and lines[1].startswith("%s %s " % (tag, key))  # tuned, and stored under this library's tag
    path.write_text("%s %s 4 0\n" % (tag, key))
    sim = make().init().step(2)
    assert sim.tile == 4
    assert len(path.read_text().splitlines()) == 1
