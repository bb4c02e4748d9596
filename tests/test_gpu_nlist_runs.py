"""The neighbour list's sweep over runs of bins and its ranking, where their cases meet: axes of one or two
bins (several images per row of bins, up to seven), tilted and thin cells, open boundaries, counts of hits on
both sides of each ranking width (64, 128, 192, 256) and past it, distances that differ below the key's high
word, exact ties, and types that drop neighbours. The list and the count of dropped neighbours have to equal
the oracle's exactly (no tolerance: the order is defined by the input's bits)."""
import numpy as np
import pytest

from paper_2304_09409_amd import synth

pytestmark = pytest.mark.gpu


def gas(n, cell, seed):
    rng = np.random.default_rng(seed)
    h = np.asarray(cell, dtype=np.float64)
    h = np.diag(h) if h.ndim == 1 else h
    return rng.random((n, 3)) @ h, rng.integers(0, 2, n).astype(np.int32), h


def shells(n, seed):
    """An atom with n others on a sphere of radius 3, in radii that differ by 1e-10 of it."""
    rng = np.random.default_rng(seed)
    v = rng.normal(size=(n, 3))
    v *= (3.0 * (1.0 + 1e-10 * rng.permutation(n)) / np.linalg.norm(v, axis=1))[:, None]
    return np.vstack([np.zeros((1, 3)), v]), np.arange(n + 1, dtype=np.int32) % 2, None


CASES = {
    "one_atom_all_images": lambda: gas(1, [2.1, 2.1, 2.1], 1),
    "thin_x": lambda: gas(40, [2.1, 13.0, 14.0], 2),
    "thin_y": lambda: gas(40, [13.0, 2.1, 14.0], 3),
    "thin_z": lambda: gas(40, [13.0, 14.0, 2.1], 4),
    "two_bins": lambda: gas(150, [12.1, 11.9, 12.5], 5),
    "one_bin": lambda: gas(60, [7.0, 8.0, 6.1], 6),
    "tilted": lambda: gas(200, [[14.0, 0, 0], [5.0, 12.0, 0], [-4.0, 6.0, 11.0]], 7),
    "open_slab": lambda: gas(300, [60.0, 5.0, 13.0], 8)[:2] + (None,),
    "near_ties": lambda: shells(90, 9),
    "exact_ties": lambda: synth.tie_lattice(6),
    **{f"hits_about_{k}": (lambda k=k: gas(int(k / 904.8 * 14.0 ** 3) + 1, [14.0, 14.0, 14.0], k))
       for k in (3, 60, 124, 188, 250, 330)},
}


@pytest.mark.parametrize("case", list(CASES))
def test_list_equals_oracle(case):
    from oracle import Oracle
    from paper_2304_09409_amd import dpk
    print(f"[case] {case}", flush=True)
    c, t, b = CASES[case]()
    params = synth.water_params()
    ref = Oracle(synth.WATER_MODEL, params).compute(c, t, b, dumps=True)
    ctx = dpk.Context(dpk.Model(synth.WATER_MODEL, params), precision="mixed")
    ctx.compute(c, t, b)
    np.testing.assert_array_equal(ctx.debug_nlist(len(t)), ref["nlist"])
    assert ctx.stats()["nbr_dropped"] == ref["ndrop"]
    ctx.close()


@pytest.mark.parametrize("case", list(CASES))
def test_displacements_give_the_oracle_forces(case):
    """The list's r_ij are rebuilt from the run packed into each key, so a wrong run or image shift would leave
    the indices as they are (most of all where an atom's neighbours are its own images): forces and virial of
    the FP64 path, whose error is within 1e-10 plus 1e-11 of the largest (random pairs come close, and a force
    is a sum of terms up to a few hundred times its size)."""
    from oracle import Oracle
    from paper_2304_09409_amd import dpk
    print(f"[case] {case}", flush=True)
    c, t, b = CASES[case]()
    params = synth.water_params()
    ref = Oracle(synth.WATER_MODEL, params).compute(c, t, b)
    ctx = dpk.Context(dpk.Model(synth.WATER_MODEL, params), precision="fp64")
    got = ctx.compute(c, t, b)
    for key in ("force", "virial"):
        r = np.asarray(ref[key]).reshape(-1)
        assert np.abs(np.asarray(got[key]).reshape(-1) - r).max() <= 1e-10 + 1e-11 * np.abs(r).max(), key
    ctx.close()
