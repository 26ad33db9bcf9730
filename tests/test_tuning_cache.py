"""The autotuner's on-disk cache (no GPU: the tuner and the device are stood in for):
a result is used again only with the library build that measured it."""
import json
import types

import pytest

import paper_2112_09972_amd as sc


@pytest.fixture
def lat(monkeypatch, tmp_path):
    monkeypatch.setenv("XDG_CACHE_HOME", str(tmp_path / "cache"))
    lib = tmp_path / "lib.so"
    lib.write_bytes(b"one build")
    monkeypatch.setattr(sc, "LIB_PATH", str(lib))
    o = object.__new__(sc.Lattice)
    cuda = types.SimpleNamespace(get_device_properties=lambda d: types.SimpleNamespace(name="gpu"))
    o.torch, o.device, o.ctx = types.SimpleNamespace(cuda=cuda), "cuda:0", None
    o.nx, o.ny, o.nz, o.nbox = 32, 32, 32, 1
    o.cfg = types.SimpleNamespace(prec=0, bc=1)
    o.calls = []

    def tune(ctx, steps):
        o.calls.append("tune")
        return 4, 8, 1, 0.5

    monkeypatch.setattr(sc, "sclbm_autotune", tune)
    monkeypatch.setattr(sc, "sclbm_set_launch", lambda ctx, *shape: o.calls.append(shape))
    monkeypatch.setattr(sc, "sclbm_reset_launch", lambda ctx: o.calls.append("reset"))
    monkeypatch.setattr(sc, "sclbm_get_tiles", lambda ctx: o.tiles)
    monkeypatch.setattr(sc, "sclbm_default_tiles", lambda cfg: {"kind": "planes"})
    o.tiles = {"kind": "fixed"}
    return o, lib, tmp_path / "cache" / "sclbm" / "tuning.json"


def test_result_is_measured_once_per_build(lat):
    o, lib, _ = lat
    assert o.autotune() == (4, 8, 1, 0.5) and o.calls == ["tune"]
    assert o.autotune() == (4, 8, 1, 0.5) and o.calls.count("tune") == 1
    lib.write_bytes(b"another build")
    o.autotune()
    assert o.calls.count("tune") == 2
    o.autotune(cache=False)
    assert o.calls.count("tune") == 3


def test_result_of_an_earlier_build_is_not_used(lat):
    """A file left by a build whose shapes meant something else."""
    o, _, path = lat
    path.parent.mkdir(parents=True)
    stale = {"gpu|32x32x32|1|0|1|rowtiles5": {"tile_rows": 8, "zchunk": 2, "tile_waves": 1, "ms": 0.02}}
    path.write_text(json.dumps(stale))
    assert o.autotune() == (4, 8, 1, 0.5)
    assert "tune" in o.calls
    assert stale.items() <= json.loads(path.read_text()).items()


@pytest.mark.parametrize("kind,expect", [("planes", "reset"), ("fixed", (4, 8, 1))])
def test_the_start_is_set_again_as_the_start(lat, kind, expect):
    """Where the launch a context starts with won, a cached result brings that launch back
    and not the shape it is reported as."""
    o, _, _ = lat
    o.tiles = {"kind": kind}
    o.autotune()
    assert o.calls == ["tune"]
    assert o.autotune() == (4, 8, 1, 0.5)
    assert o.calls == ["tune", expect]
