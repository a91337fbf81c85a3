"""Self-energy rows of run-time grids on either side of the lines between the two unrollings of their
transforms (a launch that needs one round of the chip less with five wavefronts per SIMD takes the shorter one),
for the two-stage, the direct and the power-of-two transforms, against numpy's FFT of the same products.

Tolerance 1e-12 relative, the kernel bar: at most 31 + 31 multiply-adds per output and axis at 2e-16 each."""
import numpy as np
import pytest

from paper_2505_19467_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("interband", [False, True])
@pytest.mark.parametrize("nkx,nky", [(7, 1), (64, 1), (128, 1), (9, 7), (22, 22), (23, 22)])
@pytest.mark.parametrize("m", [255, 256, 319, 320])
def test_sigma_rounds(nkx, nky, m, interband):
    import torch
    from paper_2505_19467_amd import kbe
    print(f"sigma rounds nk={nkx}x{nky} m={m} interband={interband}", flush=True)
    nb = 2
    cfg = inputs.Config(name="rounds", nkx=nkx, nky=nky, nb=nb, hop=np.zeros((3, nb, nb), complex), U=1.3, dt=0.02, nt=m,
                        interaction=inputs.INTERACTION_INTERBAND if interband else inputs.INTERACTION_HUBBARD)
    S = kbe.System(cfg)
    gen = torch.Generator(device="cuda").manual_seed(nkx + m)
    row = torch.view_as_complex(torch.rand(m + 1, cfg.nk, 2, nb, nb, 2, generator=gen, device="cuda", dtype=torch.float64) - 0.5)
    S.set_history_row(m, row)
    S.rebuild_aux(m)
    S.stage_sigma(m)
    got = S.sigma_row(m).cpu().numpy()
    g = np.fft.ifftn(row.cpu().numpy().reshape(m + 1, nkx, nky, 2, nb, nb), axes=(1, 2))
    if interband:
        det = g[..., 0, 0] * g[..., 1, 1] - g[..., 0, 1] * g[..., 1, 0]
        sign = np.array([[1.0, -1.0], [-1.0, 1.0]])
        s = -cfg.U ** 2 * sign * det[..., None, None] * g[:, :, :, ::-1, ::-1, ::-1].conj()
    else:
        s = -cfg.U ** 2 * g * g * g[:, :, :, ::-1].conj()
    ref = np.fft.fftn(s, axes=(1, 2)).reshape(m + 1, cfg.nk, 2, nb, nb)
    err = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"  relative error {err:.2e}", flush=True)
    assert err < 1e-12
