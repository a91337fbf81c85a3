"""Inside one kbe_step call a step's observables are computed in a launch of the next step: a run of
n steps in one call, in calls of one and in uneven calls must give the same bits (the same kernels on
the same inputs), on every way the call can end: the last step, the kick's slice, a step that
reports an unmet tolerance."""
import numpy as np
import pytest

from paper_2505_19467_amd import inputs

pytestmark = pytest.mark.gpu


def _square(nb, **kw):
    hop = np.zeros((3, nb, nb), complex)
    hop[0] = np.diag(np.linspace(0.5, -0.5, nb))
    hop[1] = hop[2] = -(0.3 + 0.7 * np.eye(nb))
    return inputs.Config(name="batch", nkx=3, nky=2, nb=nb, hop=hop, U=1.2, dt=0.02, nt=30, **kw)


@pytest.mark.parametrize("cfg", [_square(1), _square(2), _square(3), _square(4), _square(2, n_corr=0),
                                 _square(3, n_corr=0), _square(2, n_corr=5, corr_tol=1e-8),
                                 _square(2, precision=inputs.PRECISION_FP32_MFMA),
                                 inputs.paper_chain(16, 30)], ids=lambda c: f"{c.name}-nb{c.nb}-K{c.n_corr}-p{c.precision}")
def test_observables_do_not_depend_on_the_calls(cfg):
    from paper_2505_19467_amd import kbe
    out = []
    for calls in ([30], [1] * 30, [7, 1, 18, 0, 4]):
        S = kbe.System(cfg)
        for n in calls:
            S.step(n)
        out.append((S.observables(), S.history_row(30).cpu().numpy()))
    for obs, row in out[1:]:
        assert np.array_equal(obs, out[0][0])
        assert np.array_equal(row, out[0][1])


def test_observables_of_a_step_that_reports():
    from paper_2505_19467_amd import kbe
    cfg = _square(2, n_corr=1, corr_tol=1e-300)
    S, R = kbe.System(cfg), kbe.System(_square(2))
    R.step(5)
    ref = R.observables()
    for m in range(1, 6):
        with pytest.raises(kbe.KbeNotConverged):
            S.step(30 - m)          # each call commits one step and reports
        assert S.current_step == m
        assert np.array_equal(S.observables()[m], ref[m])


@pytest.mark.parametrize("nb,precision", [(1, inputs.PRECISION_FP64), (2, inputs.PRECISION_FP64),
                                          (2, inputs.PRECISION_FP32)])
def test_evaluation_and_predictor_in_one_launch(nb, precision):
    # within a call a row's evaluation and the next row's predictor are one launch: across the edges
    # of its 64-column tiles (rows 63..65, 127..129) the bits are those of the two launches
    from paper_2505_19467_amd import kbe
    hop = np.zeros((3, nb, nb), complex)
    hop[0] = np.diag(np.linspace(0.5, -0.5, nb))
    hop[1] = -(0.3 + 0.7 * np.eye(nb))
    cfg = inputs.Config(name="tiles", nkx=5, nky=1, nb=nb, hop=hop, U=1.2, dt=0.02, nt=130, precision=precision)
    one, many = kbe.System(cfg), kbe.System(cfg)
    for _ in range(130):
        one.step(1)
    many.step(130)
    assert np.array_equal(many.observables(), one.observables())
    for m in (63, 64, 65, 127, 128, 129, 130):
        assert np.array_equal(many.history_row(m).cpu().numpy(), one.history_row(m).cpu().numpy()), m
