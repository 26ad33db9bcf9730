"""What the step kernel runs: a shape that is named runs as named, the launch a context
starts with is what sclbm_default_tiles says, and neither changes a bit of the state."""
import numpy as np
import pytest

from paper_2112_09972_amd import workloads as wl

pytestmark = pytest.mark.gpu

PRECS = ["f64", "f32", "f32d", "f16dev", "bf16dev"]


@pytest.fixture(scope="module")
def sc():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2112_09972_amd as sc
    return sc


def droplets(sc, nxyz, nbox, prec, bc):
    """Boxes with a droplet each off the centre, and in ghost mode a changing flow each."""
    nx, ny, nz = nxyz
    lat = sc.Lattice(nx, ny, nz, nbox=nbox, bc=bc, prec=prec, table_len=64, tau=(1.0, 1.2), g_ab=wl.G_AB,
                     rho_b=wl.ghost_densities(8.0))
    rng = np.random.default_rng(nx)
    for b in range(nbox):
        ctr = np.array([nx, ny, nz]) / 2.0 + rng.uniform(-2, 2, 3)
        A = 1e-3 * rng.standard_normal(9)
        A[8] = -A[0] - A[4]
        lat.init_droplet(ctr, 0.3 * min(nxyz), wl.WIDTH, wl.RHO_HI, wl.RHO_LO, A if bc == "ghost" else None, box=b)
        if bc == "ghost":
            lat.set_gradient_table(np.array([A * (1 + 0.1 * t) for t in range(64)]), 0, box=b)
    return lat


@pytest.mark.parametrize("bc", ["ghost", "periodic"])
@pytest.mark.parametrize("prec", PRECS)
@pytest.mark.parametrize("nxyz,nbox", [((32, 32, 32), 1), ((100, 10, 9), 1), ((128, 10, 9), 1), ((150, 40, 90), 1),
                                       ((260, 31, 30), 1)])
def test_named_shapes_run_as_named(sc, nxyz, nbox, prec, bc):
    """The default shape named by its numbers is that march, with streaming stores, on boxes
    that start with planes at once, fitted tiles and cached stores too; the start comes
    back with reset_launch; the captured loop follows each change; the states agree."""
    lat = droplets(sc, nxyz, nbox, prec, bc)
    start, shape = sc.sclbm_default_tiles(lat.cfg), sc.sclbm_default_launch(lat.cfg)
    assert lat.get_tiles() == start and lat.get_launch() == shape
    ref = droplets(sc, nxyz, nbox, prec, bc)
    ref.set_launch(4, 3, 1)
    assert ref.get_tiles() == {"kind": "fixed", "width": 64, "rows": 4, "zchunk": 3, "cached": False}
    for change in (None, "named", "start"):
        if change == "named":
            lat.set_launch(*shape)
            assert lat.get_launch() == shape
            assert lat.get_tiles() == {"kind": "fixed", "width": 64 * shape[2], "rows": shape[0], "zchunk": shape[1],
                                       "cached": False}
        elif change == "start":
            lat.reset_launch()
            assert lat.get_launch() == shape and lat.get_tiles() == start
        lat.step_graph(2)
        lat.step(1)
        lat.step_graph(2)
        lat.step(1)
        ref.step(6)
        assert np.array_equal(lat.save(), ref.save()), change
    with pytest.raises(sc.SclbmError):
        lat.set_launch(5, 3, 1)
    assert lat.get_tiles() == start


@pytest.mark.parametrize("prec,nxyz", [("f64", (32, 32, 32)), ("f32", (97, 40, 33)), ("f16dev", (150, 40, 30))])
def test_autotuner_and_cache_set_what_they_measured(sc, prec, nxyz, tmp_path, monkeypatch):
    """What runs after autotune is the start or a named shape; a second lattice, set from the
    cache, runs the same; the states after it agree with a march."""
    monkeypatch.setenv("XDG_CACHE_HOME", str(tmp_path))
    lat, other, ref = (droplets(sc, nxyz, 1, prec, "ghost") for _ in range(3))
    ty, zc, wx, ms = lat.autotune(trial_steps=5)
    assert ms > 0 and lat.get_launch() == (ty, zc, wx)
    named = {"kind": "fixed", "width": 64 * wx, "rows": ty, "zchunk": zc, "cached": False}
    assert lat.get_tiles() in (named, sc.sclbm_default_tiles(lat.cfg))
    other.set_launch(4, 2, 1)
    assert other.autotune(trial_steps=5) == (ty, zc, wx, ms)
    assert other.get_tiles() == lat.get_tiles() and other.get_launch() == (ty, zc, wx)
    ref.set_launch(4, 3, 1)
    fresh = droplets(sc, nxyz, 1, prec, "ghost")
    lat.load(fresh.save())
    for o in (lat, other, ref):
        o.step(5)
    assert np.array_equal(other.save(), ref.save())
    assert np.array_equal(lat.save(), ref.save())


# What a context starts with, by format: (box, boxes, kind, tiles in a row, cached stores).  Fitted tiles: rows held
# whole (24 rows of a tile among them) and cut in two to seven, with a narrower last one; fixed tiles with cached
# stores: each shape, rows held whole and cut; planes at once: chunks of one and two planes, odd counts
# (a last chunk of one), rows held whole and cut in two to four, four wavefronts a plane.
PLANES = [((3, 3, 3), 1, "planes", 1, False), ((32, 32, 32), 1, "planes", 1, False), ((68, 12, 12), 1, "planes", 2, False),
          ((124, 12, 13), 1, "planes", 3, False), ((128, 13, 14), 1, "planes", 4, False), ((45, 33, 29), 1, "planes", 1, False),
          ((103, 19, 13), 1, "planes", 2, False), ((134, 13, 13), 1, "planes", 3, False), ((202, 13, 13), 1, "planes", 4, False),
          ((40, 57, 33), 1, "planes", 1, False), ((21, 70, 9), 5, "planes", 1, False)]
F32X = [((272, 43, 13), 1, "fixed", 5, True), ((372, 34, 12), 1, "fixed", 3, True)]
DEV = [((13, 118, 99), 2, "fitted", 1, True), ((13, 33, 104), 2, "fitted", 1, False), ((133, 14, 86), 2, "fitted", 2, True),
       ((142, 17, 116), 1, "fitted", 2, False), ((292, 23, 46), 1, "fitted", 3, True), ((413, 13, 20), 2, "fitted", 4, False),
       ((257, 17, 86), 1, "fitted", 5, True), ((406, 21, 26), 2, "fitted", 6, True),
       ((143, 118, 18), 1, "fixed", 3, True), ((55, 48, 115), 1, "fixed", 1, True), ((337, 53, 17), 1, "fixed", 3, True),
       ((124, 34, 24), 3, "fixed", 1, True), ((419, 27, 28), 1, "fixed", 2, True), ((181, 43, 39), 1, "fixed", 1, True),
       ((48, 48, 47), 1, "planes", 1, False)]
STARTS = {
    "f64": PLANES + [((17, 93, 24), 2, "fitted", 1, True), ((13, 19, 62), 3, "fitted", 1, False),
                     ((139, 18, 20), 3, "fitted", 2, True), ((271, 16, 26), 1, "fitted", 3, True),
                     ((410, 13, 24), 1, "fitted", 4, True), ((413, 13, 20), 2, "fitted", 6, True),
                     ((387, 51, 12), 1, "fitted", 7, True), ((154, 13, 38), 1, "fixed", 3, True),
                     ((16, 26, 61), 3, "fixed", 1, True), ((209, 14, 26), 1, "fixed", 2, True),
                     ((97, 22, 36), 1, "fixed", 1, True)],
    "f32": PLANES + F32X + [((48, 48, 47), 1, "planes", 1, False), ((21, 77, 47), 2, "fitted", 1, True),
                            ((12, 25, 92), 2, "fitted", 1, False), ((139, 25, 44), 1, "fitted", 2, True),
                            ((271, 16, 26), 1, "fitted", 3, True), ((404, 24, 20), 1, "fitted", 4, True),
                            ((412, 17, 28), 1, "fitted", 5, True), ((387, 51, 12), 1, "fitted", 7, True),
                            ((55, 20, 69), 2, "fixed", 1, True), ((93, 17, 96), 1, "fixed", 1, True)],
    "f32d": PLANES + F32X + [((15, 115, 64), 2, "fixed", 1, True), ((92, 40, 30), 2, "fixed", 1, True)],
    "f16dev": PLANES + DEV,
    "bf16dev": PLANES + DEV,
}


@pytest.mark.parametrize("bc", ["ghost", "periodic"])
@pytest.mark.parametrize("prec,nxyz,nbox,kind,parts,cached", [(p,) + c for p in PRECS for c in STARTS[p]])
def test_every_start_equals_a_march(sc, prec, nxyz, nbox, kind, parts, cached, bc):
    """The launch a context starts with is the one meant, and gives the same bytes as 64 x 4
    tiles in chunks of three planes after seven steps, of every box."""
    lat, ref = (droplets(sc, nxyz, nbox, prec, bc) for _ in range(2))
    t = lat.get_tiles()
    assert (t["kind"], -(-nxyz[0] // t["width"]), t["cached"]) == (kind, parts, cached), t
    ref.set_launch(4, 3, 1)
    for o in (lat, ref):
        o.step(7)
    a, b = lat.save(), ref.save()
    assert np.array_equal(a, b)
    ra, rb = (v.cpu().numpy() for v in lat.fields(box=nbox - 1, velocity=False))
    assert np.isfinite(ra).all() and np.isfinite(rb).all()


def test_starts_with_the_nan_fill_build(sc):
    """No fitted tile and no planes-at-once workgroup reads an LDS cell that none of its threads
    wrote: with every cell NaN before each plane (libsclbm_debug.so) the states are the
    same bytes (one process per build; the marches that are named: debug_fill_cases.py)."""
    import json
    import os
    import subprocess
    import sys
    pkg = os.path.dirname(sc.__file__)
    out = []
    for lib in ("libsclbm.so", "libsclbm_debug.so"):
        path = os.path.join(pkg, lib)
        assert os.path.exists(path), "build() builds it"
        env = dict(os.environ, SCLBM_LIBRARY=path, PYTHONPATH=os.path.dirname(pkg))
        r = subprocess.run([sys.executable, os.path.abspath(__file__)], env=env, cwd=os.path.dirname(pkg),
                           capture_output=True, text=True, timeout=100)
        assert r.returncode == 0, r.stderr[-3000:]
        out.append(json.loads(r.stdout.strip().splitlines()[-1]))
    assert [o["library"].rsplit("/", 1)[1] for o in out] == ["libsclbm.so", "libsclbm_debug.so"]
    assert len(out[0]["states"]) == sum(len(v) for v in STARTS.values()) * 2
    assert out[0]["states"] == out[1]["states"]


def main():
    """States of every start with the library that SCLBM_LIBRARY names, as one JSON line."""
    import hashlib
    import json
    import paper_2112_09972_amd as sc
    states = {}
    for prec in PRECS:
        for nxyz, nbox, kind, _, _ in STARTS[prec]:
            for bc in ("ghost", "periodic"):
                lat = droplets(sc, nxyz, nbox, prec, bc)
                assert lat.get_tiles()["kind"] == kind
                lat.step(4)
                m, _ = lat.totals(check=False)
                assert np.isfinite(m).all()
                states["%s %s %s" % (prec, nxyz, bc)] = hashlib.sha256(lat.save()[64:].tobytes()).hexdigest()[:16]
                lat.close()
    print(json.dumps({"library": sc.LIB_PATH, "states": states}))


if __name__ == "__main__":
    main()
