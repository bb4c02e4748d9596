"""The 16-atom tiles of the FP64 fitting kernel (and of the FP32 kernel of the descriptors of M values):
species counts at the edges of a tile, a species that is absent, a single atom, a grid with more blocks
than CUs (the shape that shares a CU), and an ensemble. FP64: forces within 1e-10 eV/A, atomic energies
1e-11 eV; mixed (FP32 fitting): forces within 1e-3 eV/A, the bounds of the parity tests."""
import numpy as np
import pytest

from paper_2304_09409_amd import synth

pytestmark = pytest.mark.gpu

SYS = {"se_e2_a": (synth.SERVE_MODEL, synth.serve_params),
       "se_e2_r": (dict(synth.SERVE_MODEL, descriptor="se_e2_r"),
                   lambda: synth.make_params(dict(synth.SERVE_MODEL, descriptor="se_e2_r"), 5, 10.0, 30.0))}


def frame(counts, seed=3):
    n = sum(counts)
    c, _, b = synth.serving_frame(n, seed, 2)
    t = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    np.random.default_rng(seed).shuffle(t)
    return c, t, b


@pytest.mark.parametrize("counts", [(1, 0, 0), (16, 0, 1), (15, 17, 32), (0, 33, 0), (1, 1, 129), (2100, 1, 2005)],
                         ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("descriptor,precision", [("se_e2_a", "fp64"), ("se_e2_r", "fp64"), ("se_e2_r", "mixed")])
def test_tiles(counts, descriptor, precision):
    from oracle import Oracle
    from paper_2304_09409_amd import dpk
    print(f"[case] {descriptor} {precision} {counts}", flush=True)
    spec, params = SYS[descriptor]
    c, t, b = frame(counts)
    if sum(counts) == 1:
        b = None
    ref = Oracle(spec, params()).compute(c, t, b)
    ctx = dpk.Context(dpk.Model(spec, params()), precision=precision)
    got = ctx.compute(c, t, b, atom_energy=True)
    ctx.close()
    ftol, etol = (1e-10, 1e-11) if precision == "fp64" else (1e-3, 1e-4 + 1e-5 * np.abs(ref["atom_energy"]).max())
    np.testing.assert_allclose(got["force"], ref["force"], rtol=0, atol=ftol)
    np.testing.assert_allclose(got["atom_energy"], ref["atom_energy"], rtol=0, atol=etol)


def test_ensemble_tiles():
    from oracle import Oracle
    from paper_2304_09409_amd import dpk
    spec, params = SYS["se_e2_a"]
    c, t, b = frame((15, 17, 32))
    ps = synth.ensemble_params(spec, params(), 3)
    got = dpk.Deviation([dpk.Model(spec, p) for p in ps], precision="fp64").compute(c, t, b)
    for k, p in enumerate(ps):
        ref = Oracle(spec, p).compute(c, t, b)
        np.testing.assert_allclose(got["force"][k], ref["force"], rtol=0, atol=1e-10)
        assert abs(got["energy"][k] - ref["energy"]) <= max(1e-9, 1e-12 * abs(ref["energy"]))
