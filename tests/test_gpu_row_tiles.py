"""The row kernel carries 64 consecutive t' per block, one matrix row per wavefront: runs whose last
steps put t' = m on the last lane of a tile, on the first lane of the next and one past it, for
every orbital count, with and without Gregory nodes, with the corrector's change output.

Tolerance: both sides compute in FP64 and differ in summation order only; over these run lengths
the established FP64 bar of 1e-10 relative, and for the row changes (differences of O(1) numbers
that agree to 1e-13) 1e-12 absolute."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2505_19467_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nkx,nky,nb,q,n_corr,nsteps", [(3, 1, 1, 1, 3, 65), (2, 2, 2, 1, 3, 64), (1, 2, 3, 1, 2, 66),
                                                        (2, 1, 4, 1, 2, 65), (1, 2, 1, 4, 2, 129), (2, 1, 2, 3, 3, 128),
                                                        (1, 3, 3, 2, 2, 65), (1, 2, 4, 5, 2, 66)])
def test_runs_across_tile_edges(nkx, nky, nb, q, n_corr, nsteps):
    import torch
    assert torch.cuda.is_available()
    from paper_2505_19467_amd import kbe
    print(f"row tiles nk={nkx}x{nky} nb={nb} q={q} K<={n_corr} steps={nsteps}", flush=True)
    rng = np.random.default_rng(10 * nb + q)
    hop = np.zeros((3, nb, nb), complex)
    z = rng.standard_normal((nb, nb)) + 1j * rng.standard_normal((nb, nb))
    hop[0] = 0.5 * (z + z.conj().T)
    hop[1] = -(0.3 + 0.7 * np.eye(nb))
    hop[2] = hop[1] if nky > 1 else 0
    # a tolerance that no pass meets: every step runs all its passes and reports the changes
    cfg = inputs.Config(name="tiles", nkx=nkx, nky=nky, nb=nb, hop=hop, U=1.2, dt=0.02, nt=nsteps, n_corr=n_corr,
                        corr_tol=1e-300, quad_points=q)
    S = kbe.System(cfg)
    for _ in range(nsteps):
        with pytest.raises(kbe.KbeNotConverged):
            S.step(1)
    obs, row = S.observables(), S.history_row(nsteps).cpu().numpy()
    passes, changes = S.corrector_log(1)
    ref = O.run(cfg.replace(corr_tol=0.0), nsteps)
    _, _, ref_changes = O.run_log(cfg, nsteps)
    assert (passes == n_corr).all()
    assert np.abs(changes - ref_changes).max() < 1e-12
    scale = np.abs(ref["obs"]).max(axis=0)
    scale[scale < 1e-12] = 1.0
    assert (np.abs(obs - ref["obs"]) / scale).max() < 1e-10
    assert np.abs(row - ref["final_row"]).max() < 1e-10 * np.abs(ref["final_row"]).max()
