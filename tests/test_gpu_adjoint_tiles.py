"""Reverse sweep where its kernels' splits can go wrong: rows that end on and one past a tile of 64 and
a round of 512, an odd number of k-points (the last pair of lanes of the propagator adjoint), a time
step whose propagators need several doublings, and each compile-time grid of the self-energy adjoint,
against the oracle's tangent-linear derivatives.

Tolerance: the reverse sweep's established bar of 1e-9 relative (both sides compute in FP64; the
difference is rounding carried through the sweep)."""
import numpy as np
import pytest

from oracle import oracle as O
from paper_2505_19467_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nkx,nky,nt,dt,observable", [(3, 1, 64, 0.02, "n_band1"), (3, 1, 65, 0.02, "n_orb0"),
                                                      (1, 1, 513, 0.01, "n_band0"), (5, 3, 9, 0.5, "n_band0"),
                                                      (16, 1, 12, 0.05, "n_band1"), (12, 12, 6, 0.1, "n_orb1"),
                                                      (16, 16, 4, 0.2, "n_band0"), (24, 24, 3, 0.2, "n_band1")])
def test_gradient_at_tile_edges(nkx, nky, nt, dt, observable):
    from paper_2505_19467_amd import kbe
    print(f"gradient nk={nkx}x{nky} nt={nt} dt={dt} {observable}", flush=True)
    hop = np.zeros((3, 2, 2), complex)
    hop[0] = np.diag([0.5, -0.5])
    hop[1] = -np.array([[1.0, 0.3], [0.3, 0.9]])
    hop[2] = hop[1] if nky > 1 else 0
    cfg = inputs.Config(name="adj", nkx=nkx, nky=nky, nb=2, hop=hop, U=1.2, dt=dt, nt=nt,
                        pulse=inputs.Pulse(amp=0.6, omega=1.3, t0=0.4, width=1.0, pol=(1.0, 0.0)))
    S = kbe.System(cfg)
    S.step(nt)
    got = S.adjoint_gradient(observable)
    _, dobs = O.tlm_run(cfg, nt)
    ref = dobs[nt, kbe.OBS[observable]]
    err = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"  {got} relative error {err:.2e}", flush=True)
    assert err < 1e-9
