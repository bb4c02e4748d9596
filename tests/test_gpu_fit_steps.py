"""The BF16-path fitting net in steps (small frames: the W1 products spread over four blocks per 32-atom
tile). Against the oracle at the edges of a tile and on both sides of the rule that chooses the steps (61
tiles with three species: 1,952 atoms), with the parity tests' bounds for mixed precision; and against the
one-launch kernel: a cluster alone (in steps) and beside a second one 100 A away (one launch) has the same
atomic energies bit for bit, every sum having the same order, and forces within 1e-12 eV/A (FP64 sums of
some 200 terms below 10 eV/A in an order that varies: 200 * 10 * 2^-53 = 2e-13). The FP64 net's steps (16-atom
tiles, up to 128 of them with one per species to spare) against the oracle on both sides of their rule, with the
parity tests' FP64 bounds."""
import numpy as np
import pytest

from paper_2304_09409_amd import synth

pytestmark = pytest.mark.gpu


def frame(counts, seed=3):
    c, _, b = synth.serving_frame(sum(counts), seed, 2)
    t = np.repeat(np.arange(len(counts)), counts).astype(np.int32)
    np.random.default_rng(seed).shuffle(t)
    return c, t, b if sum(counts) > 1 else None


@pytest.mark.parametrize("counts", [(1, 0, 0), (31, 33, 32), (0, 1, 129), (650, 650, 652), (650, 650, 653)],
                         ids=lambda c: "-".join(map(str, c)))
def test_steps_match_oracle(counts):
    from oracle import Oracle
    from paper_2304_09409_amd import dpk
    print(f"[case] {counts}", flush=True)
    c, t, b = frame(counts)
    ref = Oracle(synth.SERVE_MODEL, synth.serve_params()).compute(c, t, b)
    ctx = dpk.Context(dpk.Model(synth.SERVE_MODEL, synth.serve_params()), precision="mixed")
    got = ctx.compute(c, t, b, atom_energy=True)
    ctx.close()
    np.testing.assert_allclose(got["force"], ref["force"], rtol=0, atol=1e-3)
    np.testing.assert_allclose(got["atom_energy"], ref["atom_energy"], rtol=0,
                               atol=1e-4 + 1e-5 * np.abs(ref["atom_energy"]).max())


@pytest.mark.parametrize("precision", ["mixed", "bf16"])
def test_steps_equal_one_launch(precision):
    from paper_2304_09409_amd import dpk
    print(f"[case] {precision}", flush=True)
    ca, ta, _ = frame((300, 333, 200), 5)
    cb, tb, _ = frame((500, 500, 400), 6)
    cb = cb + np.array([ca[:, 0].max() - cb[:, 0].min() + 100.0, 0.0, 0.0])
    ctx = dpk.Context(dpk.Model(synth.SERVE_MODEL, synth.serve_params()), precision=precision)
    one = ctx.compute(ca, ta, None, atom_energy=True)
    two = ctx.compute(np.vstack([ca, cb]), np.concatenate([ta, tb]), None, atom_energy=True)
    ctx.close()
    n = len(ta)
    np.testing.assert_array_equal(two["atom_energy"][:n], one["atom_energy"])
    np.testing.assert_allclose(two["force"][:n], one["force"], rtol=0, atol=1e-12)


@pytest.mark.parametrize("counts", [(1, 0, 0), (15, 17, 32), (0, 1, 129), (670, 640, 650), (700, 720, 700)],
                         ids=lambda c: "-".join(map(str, c)))
def test_fp64_steps_match_oracle(counts):
    from oracle import Oracle
    from paper_2304_09409_amd import dpk
    print(f"[case] fp64 {counts}", flush=True)
    c, t, b = frame(counts, 4)
    ref = Oracle(synth.SERVE_MODEL, synth.serve_params()).compute(c, t, b)
    ctx = dpk.Context(dpk.Model(synth.SERVE_MODEL, synth.serve_params()), precision="fp64")
    got = ctx.compute(c, t, b, atom_energy=True)
    ctx.close()
    np.testing.assert_allclose(got["force"], ref["force"], rtol=0, atol=1e-10)
    np.testing.assert_allclose(got["atom_energy"], ref["atom_energy"], rtol=0, atol=1e-11)
