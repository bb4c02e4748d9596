"""Launch shapes of the training pass against the training oracle, every gradient entry: the row GEMMs' 64-wide
tiles (column tiles x ceil(n / 64) >= CUs: layer 0 to D from 641 atoms on with 256 CUs, the layers from 4,033)
and the row ranges of the weight gradients (up to seven below 2,048 rows of the largest type, eight from there
on), on both sides of each rule and with rows that fill no tile, no range and no K-chunk; and the embedding
gradients on 8 and on 1 copy (16 and 25 nets). Sparse frames: about four neighbours per atom, so that the
oracle takes seconds. Tolerances: that of the training tests, every entry within 1e-9 max|dL/dtheta|; and every
entry within 1e-8 of the largest of its own block (a layer's W, b or w_hat of one net), so that an error in a
block of small gradients shows: both sides add up to about 2e4 terms per entry in FP64, an error of some 1e-14
of the terms' absolute sum, which may exceed the block's largest entry by a few hundred."""
import numpy as np
import pytest

from paper_2304_09409_amd import synth

pytestmark = pytest.mark.gpu


def spec_of(ntypes, one_side=False):
    return dict(ntypes=ntypes, sel=[16] * ntypes, rcut=6.0, rcut_smth=0.5, emb=[25, 50, 100], axis=16,
                fit=[240, 240, 240], type_one_side=one_side)


def frame(counts, seed):
    """A jittered cubic lattice of spacing 5.3 with counts[t] atoms of type t at random sites."""
    rng = np.random.default_rng(seed)
    n = sum(counts)
    k = int(np.ceil(n ** (1.0 / 3.0)))
    sites = np.array([[i, j, l] for i in range(k) for j in range(k) for l in range(k)], dtype=np.float64)
    sites = sites[rng.permutation(len(sites))[:n]]
    t = rng.permutation(np.repeat(np.arange(len(counts)), counts)).astype(np.int32)
    return 5.3 * sites + rng.uniform(-1.2, 1.2, (n, 3)), t, np.diag([5.3 * k] * 3)


def blocks(spec):
    """(first, end) of every W, b and w_hat in the parameter blob."""
    nt = spec["ntypes"]
    e, f = [1] + spec["emb"], [spec["emb"][-1] * spec["axis"]] + spec["fit"] + [1]
    nets = [e] * (nt if spec["type_one_side"] else nt * nt) + [f] * nt
    off = 0
    for w in nets:
        for nin, nout in zip(w[:-1], w[1:]):
            for size in (nin * nout, nout, nout):
                yield off, off + size
                off += size


CASES = {
    "639_all_narrow": (spec_of(3), (401, 1, 237)),
    "751_wide_to_D": (spec_of(3), (533, 17, 201)),
    "1990_seven_ranges": (spec_of(1), (1990,)),
    "2047_one_type": (spec_of(1), (2047,)),
    "2049_eight_ranges": (spec_of(1), (2049,)),
    "4031_narrow_layers": (spec_of(2, True), (4030, 1)),
    "4097_wide_layers": (spec_of(2, True), (2063, 2034)),
    "5001_uneven_types": (spec_of(4), (2583, 17, 2401, 0)),
    "16_nets_8_copies": (spec_of(4), (31, 30, 29, 7)),
    "25_nets_1_copy": (spec_of(5), (23, 22, 21, 3, 28)),
}


@pytest.mark.parametrize("case", list(CASES))
def test_gradient_entries(case):
    from oracle.train import TrainOracle
    from paper_2304_09409_amd import dpk
    spec, counts = CASES[case]
    n = sum(counts)
    params = synth.make_params(spec, 41, synth.SERVE_OUT_SCALE, synth.SERVE_FIT_IN, timestep_sigma=0.2)
    c, t, b = frame(counts, n)
    rng = np.random.default_rng(n + 1)
    e, f, v = float(n * rng.normal()), rng.normal(size=(n, 3)), rng.normal(size=(3, 3))
    kw = dict(pe=0.3, pf=2.0, pv=0.1)
    L, _, ref = TrainOracle(spec, params).loss_and_grad(c, t, b, e, f, v, **kw)
    print(f"[case] {case}", flush=True)
    tr = dpk.Trainer(dpk.Model(spec, params))
    got = tr.accumulate(c, t, b, energy=e, force=f, virial=v, **kw)
    assert got["loss"] == pytest.approx(L, rel=1e-10)
    err, top = np.abs(tr.gradient() - ref), np.abs(ref).max()
    assert err.max() <= 1e-9 * top, (int(err.argmax()), err.max() / top)
    for lo, hi in blocks(spec):
        assert err[lo:hi].max() <= 1e-8 * np.abs(ref[lo:hi]).max() + 1e-14 * top, (lo, hi)
    assert hi == len(ref)
