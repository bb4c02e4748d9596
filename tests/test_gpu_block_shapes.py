"""Block shapes of the embedding kernels: atom counts at which the atoms per block, the waves per block
and the atoms per wave change (256 CUs: up to 4, 5, 9, 13 and 17 atoms per block), against the oracle. The
three-body backward holds the slot gradients of two atoms per wave from nine atoms per block on. Bounds
of the parity tests: FP64 forces 1e-10 eV/A, mixed 1e-3 eV/A; virial 1e-12 of its largest entry + 1e-9
(FP64), 1e-3 eV per atom (mixed)."""
import numpy as np
import pytest

from paper_2304_09409_amd import synth

pytestmark = pytest.mark.gpu

SYS = {"se_e2_a": (synth.WATER_MODEL, synth.water_params), "se_e3": (synth.WATER_E3_MODEL, synth.water_e3_params)}


@pytest.mark.parametrize("mols", [1, 342, 683, 1110, 1400])
@pytest.mark.parametrize("descriptor", list(SYS))
@pytest.mark.parametrize("precision", ["fp64", "mixed"])
def test_shapes(mols, descriptor, precision):
    from oracle import Oracle
    from paper_2304_09409_amd import dpk
    print(f"[case] {descriptor} {precision} {3 * mols} atoms", flush=True)
    spec, params = SYS[descriptor]
    side = int(np.ceil(mols ** (1 / 3) - 1e-9))
    c, t, b = synth.water_box(side, (3 * mols / 0.1) ** (1 / 3), 7, n_mol=mols)
    if mols == 1:
        b = None
    ref = Oracle(spec, params()).compute(c, t, b)
    ctx = dpk.Context(dpk.Model(spec, params()), precision=precision)
    got = ctx.compute(c, t, b)
    ctx.close()
    n = len(t)
    np.testing.assert_allclose(got["force"], ref["force"], rtol=0, atol=1e-10 if precision == "fp64" else 1e-3)
    vtol = 1e-9 + 1e-12 * np.abs(ref["virial"]).max() if precision == "fp64" else 1e-3 * n
    np.testing.assert_allclose(got["virial"], ref["virial"], rtol=0, atol=vtol)
