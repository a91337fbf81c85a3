"""The corrector's stopping rule on a run that has diverged: a row change that is not a number must end
the call with KBE_ERR_NONFINITE and leave the step uncommitted, whether the whole row is lost or a single
entry of it among finite ones, and never count as a change below the tolerance."""
import numpy as np
import pytest

from paper_2505_19467_amd import inputs

pytestmark = pytest.mark.gpu


def _chain(nb, **kw):
    hop = np.zeros((3, nb, nb), complex)
    hop[0] = np.diag(np.linspace(0.5, -0.5, nb))
    hop[1] = -(0.3 + 0.7 * np.eye(nb))
    return inputs.Config(name="lost", nkx=5, nky=1, nb=nb, hop=hop, dt=0.02, **kw)


@pytest.mark.parametrize("quad", [1, 4])
@pytest.mark.parametrize("nb", [1, 2, 3, 4])
def test_diverged_self_energy(nb, quad):
    """U^2 overflows: the predictor's row is finite, the first corrector row is not a number anywhere."""
    from paper_2505_19467_amd import kbe
    print(f"diverged self-energy nb={nb} quad={quad}", flush=True)
    S = kbe.System(_chain(nb, nt=4, U=1e160, hf=0, n_corr=3, corr_tol=1e-6, quad_points=quad))
    with pytest.raises(kbe.KbeError, match="KBE_ERR_NONFINITE"):
        S.step(4)
    assert S.current_step == 0
    assert S.corrector_log(1, 1)[0][0] == 0
    S.close()


@pytest.mark.parametrize("precision", [inputs.PRECISION_FP64, inputs.PRECISION_FP32_MFMA])
@pytest.mark.parametrize("nb,k,c,tp", [(1, 0, 1, 0), (1, 4, 0, 63), (2, 2, 5, 64), (3, 3, 17, 100), (4, 1, 0, 127)])
def test_one_lost_entry(nb, k, c, tp, precision):
    """One entry of the stored collision row is lost (any lane, tile and component) in a run without
    correlation self-energy, where it reaches row entries of its own k only: all other changes are finite."""
    from paper_2505_19467_amd import kbe
    print(f"one lost entry nb={nb} k={k} c={c} t'={tp} precision={precision}", flush=True)
    m = 129
    S = kbe.System(_chain(nb, nt=m + 1, U=1.0, corr=0, n_corr=3, corr_tol=1e30, precision=precision))
    S.step(m)
    S.rowbuf(kbe.BUF_I_PREV)[k, c, tp] = float("nan")
    with pytest.raises(kbe.KbeError, match="KBE_ERR_NONFINITE"):
        S.step(1)
    assert S.current_step == m
    S.close()
