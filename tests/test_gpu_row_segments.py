"""History sums split into row segments (small grids): the collision row at the edges where the
split can go wrong (a segment cut short, a segment that starts inside or past a strip's triangular
rows, one segment, the most segments a column has) for every kernel of the history sums, against
the oracle on random histories; and a split context against the library's own unsplit one.

Tolerances: FP64 kernels differ from the oracle in summation order only (1e-12, the kernel bar); the
FP32 forms round the stored blocks to FP32 (1e-5, the bar of the FP32 forms on random histories)."""
import ctypes

import numpy as np
import pytest

from oracle import oracle as O
from paper_2505_19467_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,tol", [(inputs.PRECISION_FP64, 1e-12), (inputs.PRECISION_FP32, 1e-5),
                                           (inputs.PRECISION_FP32_MFMA, 1e-5)])
@pytest.mark.parametrize("nkx,nky,nb,m", [(2, 1, 2, 17), (3, 1, 2, 80), (2, 2, 2, 145), (7, 1, 2, 300), (3, 2, 1, 97),
                                          (2, 1, 1, 321), (2, 1, 3, 33), (2, 2, 3, 130), (2, 1, 4, 31), (2, 1, 4, 161),
                                          (16, 8, 2, 205)])
def test_collision_row_segments(precision, tol, nkx, nky, nb, m):
    import torch
    from paper_2505_19467_amd import kbe
    print(f"row segments nk={nkx}x{nky} nb={nb} m={m} precision={precision}", flush=True)
    # n_corr = 2: every orbital count splits its rows
    cfg = inputs.Config(name="seg", nkx=nkx, nky=nky, nb=nb, hop=np.zeros((3, nb, nb), complex), U=1.0, dt=0.02,
                        nt=m + 1, n_corr=2, precision=precision)
    S = kbe.System(cfg)
    sampled = list(range(cfg.nk)) if cfg.nk <= 8 else [0, 1, cfg.nk // 2, cfg.nk - 1]
    rows = []
    for j in range(m + 1):
        r = inputs.random_complex((j + 1, cfg.nk, 2, nb, nb), 1000 * m + j, scale=0.3)
        S.set_history_row(j, torch.from_numpy(r).cuda())
        rows.append(r[:, sampled])
    sig = inputs.random_complex((m + 1, cfg.nk, 2, nb, nb), 9 + m, scale=0.4)
    planes = S.sigma_planes()
    t = torch.from_numpy(sig).cuda().reshape(m + 1, cfg.nk, 2, nb * nb).permute(1, 2, 3, 0)
    planes[:, :2, :, :m + 1].copy_(t)
    planes[:, 2, :, :m + 1].copy_(t[:, 1] - t[:, 0])
    S.rebuild_aux(m)
    S.stage_collision(m)
    got = S.collision_row(m)[:, sampled].cpu().numpy()
    few = cfg.replace(nkx=len(sampled), nky=1)
    ref = O.collision_row(few, m, rows, np.ascontiguousarray(sig[:, sampled]))
    err = np.abs(got - ref).max() / np.abs(ref).max()
    print(f"  relative error {err:.2e}", flush=True)
    assert err < tol
    first = S.collision_row(m).clone()
    S.stage_collision(m)
    assert torch.equal(first, S.collision_row(m))   # a fixed order of sums


def test_workspace_slots_stay_within_the_allocation_free_array():
    """The column-sum slots never push a workspace that fits the static array out of it: what the
    sizes come to with one slot per column decides."""
    from paper_2505_19467_amd import kbe
    limit = kbe.NOALLOC_WORKSPACE_MAX
    for cfg in (inputs.c1(), inputs.c4(), inputs.c1().replace(nkx=64), inputs.c4().replace(nkx=11, nky=7),
                inputs.c5().replace(nkx=3, nky=3), inputs.c2().replace(nkx=9, nky=5)):
        for nt in (50, 200, 400, 700, 1000):
            _, w, _ = kbe.workspace_query(cfg, nt)
            Tp, C = 8 * ((nt + 8) // 8), 2 * cfg.nb ** 2
            seg = cfg.nk * C * Tp * 16
            # the buffers every context has: 3/2 C Sigma rows, 2 collision rows, 1 column sum, 2 copies,
            # 2 rows, and Smax / 2 row-partial slots, all [k][C][Tp]
            base = seg * (1.5 + 2 + 1 + 2 + 2 + 0.5 * ((nt + 63) // 64))
            assert w <= base + 23 * seg + (1 << 20)
            if base + (1 << 20) <= limit:
                assert w <= limit
    n = ctypes.c_size_t()
    assert kbe._lib.kbe_adjoint_query(ctypes.byref(kbe._c_config(inputs.c4())), ctypes.byref(n)) == 0
