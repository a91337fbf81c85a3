"""Mean field and propagators (one lane per column of one k): grids beyond one block, a grid that
ends inside a block, the padded lanes of nb = 3, and time steps that need several squarings,
against the oracle's spectral propagators of h0 plus the mean field of the initial density.

Tolerance: the kernel bar of 1e-12 relative; a degree-13 Taylor polynomial at norm <= 1/4 truncates
below 2e-19, each of the s squarings doubles the rounding of the one before (s <= 6 here: 64 x 2e-16)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2505_19467_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("interband", [False, True])
@pytest.mark.parametrize("nkx,nky,nb,dt", [(24, 24, 2, 0.02), (1, 1, 1, 0.02), (19, 15, 1, 0.5), (13, 11, 3, 0.02),
                                           (17, 3, 4, 0.02), (5, 1, 2, 1.5), (5, 1, 3, 1.5), (3, 2, 4, 1.0),
                                           (1024, 1, 2, 0.02)])
def test_mean_field_and_propagators(interband, nkx, nky, nb, dt):
    import torch
    from paper_2505_19467_amd import kbe
    if interband and nb != 2:
        pytest.skip("the interband preset has two bands")
    print(f"propagators nk={nkx}x{nky} nb={nb} dt={dt} interband={interband}", flush=True)
    rng = np.random.default_rng(nkx + nb)
    hop = np.zeros((3, nb, nb), complex)
    z = rng.standard_normal((nb, nb)) + 1j * rng.standard_normal((nb, nb))
    hop[0] = 0.5 * (z + z.conj().T)
    hop[1] = -(0.3 + 0.7 * np.eye(nb))
    hop[2] = hop[1] if nky > 1 else 0
    cfg = inputs.Config(name="props", nkx=nkx, nky=nky, nb=nb, hop=hop, U=1.3, dt=dt, nt=4,
                        interaction=inputs.INTERACTION_INTERBAND if interband else inputs.INTERACTION_HUBBARD,
                        pulse=inputs.Pulse(amp=0.7, omega=1.1, t0=0.2, width=2.0, pol=(0.6, 0.8)))
    S = kbe.System(cfg)
    rho = S.rho(kbe.BUF_RHO_PREV).cpu().numpy()
    other = inputs.random_hermitian(nb, cfg.nk, 5)
    S.rho(kbe.BUF_RHO_CUR).copy_(torch.from_numpy(other))
    t = 2.5 * dt
    pu = cfg.pulse
    A = pu.amp * np.sin(pu.omega * t) * np.exp(-((t - pu.t0) / pu.width) ** 2)
    for mode in (0, 1):
        loc = (rho if mode == 0 else 0.5 * (rho + other)).mean(axis=0)
        if interband:
            field = cfg.U * np.array([[loc[1, 1].real, -loc[0, 1]], [-loc[1, 0], loc[0, 0].real - 1.0]])
        else:
            field = cfg.U * np.diag(np.diag(loc).real)
        S.stage_propagators(3, mode)
        got = S.buffer(kbe.BUF_PROP).view(cfg.nk, 3, nb, nb).cpu().numpy()
        ref = O.propagators(O.h0(cfg, A) + field, dt)
        err = np.abs(got - ref).max() / np.abs(ref).max()
        print(f"  mode {mode}: {err:.2e}", flush=True)
        assert err < 1e-12
