"""The FP64 embedding passes evaluate tanh from a table of nodes: parity with the oracle where the
pre-activations stay inside the first node's interval, spread over the table, and saturate far past its
end. The embedding weights and biases are scaled; forces within 1e-10 eV/A plus 1e-12 of the largest
force, atomic energies within 1e-11 eV plus 1e-13 of the largest (FP64 sums of about 100 neighbours by
100 features in another order)."""
import numpy as np
import pytest

from paper_2304_09409_amd import synth

pytestmark = pytest.mark.gpu

EMB = 25 + 25 + 25 + 25 * 50 + 2 * 50 + 50 * 100 + 2 * 100   # values of one embedding net


@pytest.mark.parametrize("scale", [1e-3, 0.3, 4.0, 60.0])
@pytest.mark.parametrize("descriptor", ["se_e2_a", "se_e3"])
def test_preactivation_range(scale, descriptor):
    from oracle import Oracle
    from paper_2304_09409_amd import dpk
    print(f"[case] {descriptor} scale {scale}", flush=True)
    spec, base = ((synth.WATER_MODEL, synth.water_params()) if descriptor == "se_e2_a"
                  else (synth.WATER_E3_MODEL, synth.water_e3_params()))
    p = base.copy()
    for net in range(spec["ntypes"] ** 2):
        v = p[net * EMB:(net + 1) * EMB]
        at = 0
        for i, o in ((1, 25), (25, 50), (50, 100)):
            v[at:at + i * o + o] *= scale          # W and b; the timestep vector stays
            at += i * o + 2 * o
    c, t, b = synth.water_192()
    ref = Oracle(spec, p).compute(c, t, b)
    ctx = dpk.Context(dpk.Model(spec, p), precision="fp64")
    got = ctx.compute(c, t, b, atom_energy=True)
    ctx.close()
    fmax = np.abs(ref["force"]).max()
    np.testing.assert_allclose(got["force"], ref["force"], rtol=0, atol=1e-10 + 1e-12 * fmax)
    np.testing.assert_allclose(got["atom_energy"], ref["atom_energy"], rtol=0,
                               atol=1e-11 + 1e-13 * np.abs(ref["atom_energy"]).max())
