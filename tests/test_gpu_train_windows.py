"""Training of sparse frames with many types, where almost every pair is a chunk of its own (a chunk holds up
to 16 kept neighbours of one atom and type): the embedding reverse pass works on a window of chunks at a time,
so that its memory is bounded. The frame is M copies of one cluster, out of each other's reach, so its gradient
follows from the cluster's: with labels of M times the cluster's energy and virial and the cluster's forces on
every copy, the force term's gradient is the cluster's and the energy and virial terms' are M times the
cluster's (every term of the loss is over the number of atoms). Those come from the training oracle; tolerance
of the training tests, every entry within 1e-9 max|dL/dtheta|."""
import numpy as np
import pytest

from paper_2304_09409_amd import synth

pytestmark = pytest.mark.gpu

SPEC = dict(ntypes=8, sel=[4] * 8, rcut=6.0, rcut_smth=0.5, emb=[25, 50, 100], axis=16, fit=[240, 240, 240],
            type_one_side=True)
GRID = 16                # copies per axis
CELL = 16.0
CHUNK_BYTES, WINDOW = 130 * 64 * 8, 1 << 17


def test_sparse_frame():
    import torch
    from oracle.train import TrainOracle
    from paper_2304_09409_amd import dpk
    params = synth.make_params(SPEC, 11, synth.SERVE_OUT_SCALE, synth.SERVE_FIT_IN, timestep_sigma=0.2)
    rng = np.random.default_rng(2)
    # one atom of each type, all pairs within r_c: seven chunks of one pair per atom
    corners = np.array([[i, j, k] for i in (0, 1) for j in (0, 1) for k in (0, 1)], dtype=np.float64)
    c0 = 3.0 + 2.0 * corners + rng.uniform(-0.2, 0.2, (8, 3))
    t0 = rng.permutation(8).astype(np.int32)
    b0 = np.diag([CELL] * 3)
    e0, f0, v0 = float(rng.normal()), rng.normal(size=(8, 3)), rng.normal(size=(3, 3))
    o = TrainOracle(SPEC, params)
    kw = dict(pe=0.3, pf=2.0, pv=0.1)
    g = {k: o.loss_and_grad(c0, t0, b0, e0 if k == "e" else None, f0 if k == "f" else None, v0 if k == "v" else None,
                            **kw)[2] for k in "efv"}
    M = GRID ** 3
    ref = M * (g["e"] + g["v"]) + g["f"]
    cells = CELL * np.array([[i, j, k] for i in range(GRID) for j in range(GRID) for k in range(GRID)], dtype=np.float64)
    c = (cells[:, None, :] + c0[None]).reshape(-1, 3)
    n, chunks = len(c), 7 * 8 * M
    assert chunks > WINDOW
    print(f"[case] {n} atoms, {chunks} chunks", flush=True)
    free0 = torch.cuda.mem_get_info()[0]
    tr = dpk.Trainer(dpk.Model(SPEC, params))
    tr.accumulate(c, np.tile(t0, M), GRID * b0, energy=M * e0, force=np.tile(f0, (M, 1)), virial=M * v0, **kw)
    used = free0 - torch.cuda.mem_get_info()[0]
    assert np.abs(tr.gradient() - ref).max() <= 1e-9 * np.abs(ref).max()
    # a window of chunks, and what an atom takes in the trainer and its context (about 125 KB), with room
    assert used <= CHUNK_BYTES * WINDOW + 160e3 * n + 5e8, used
