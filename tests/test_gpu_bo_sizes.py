"""Born-Oppenheimer states over the forms of the eigensolver: grids whose
transforms take one wave (up to 1024 points; a last pass of 2, 4 or 8 points)
and the work-group, bases of up to 15 columns and above, and a basis of more
columns (36) than the grid has points.  Against the oracle's dense
eigensolver; bars as in test_gpu_bo.py: energies 1e-12 of max(1, |E|),
residuals 1e-10 in the maximum norm."""

import numpy as np
import pytest

from oracle import bo as obo
from oracle import grid, models
from paper_1805_11169_amd import icwf, inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_r,n_states", [(32, 1), (32, 8), (64, 3), (128, 4), (256, 3), (512, 8), (1024, 5), (2048, 2)])
def test_forms(n_r, n_states):
    print(f"[case] BO forms n_r={n_r} states={n_states}", flush=True)
    box = min(75.0, 0.15 * n_r + 5.0)
    R = np.array([-3.1, 0.2, 4.7])
    cfg = icwf.make_config(4, n_r, 32, (-box, box), (-9.0, 9.0), 1.0, 1836.0, 0.1, inputs.MODEL_SHIN_METIU,
                           inputs.SHIN_METIU_PARAMS)
    states, E, info = icwf.bo_states(cfg, R, n_states)
    model = models.make("shin_metiu", inputs.SHIN_METIU_PARAMS)
    r, h = grid.points(-box, box, n_r)
    Eref = obo.bo_states(model, r, h, 1.0, R, n_states)[1]
    T = grid.kinetic_matrix(n_r, h, 1.0)
    assert info["unconverged"] == 0
    assert np.max(np.abs(E - Eref) / np.maximum(1.0, np.abs(Eref))) < 1e-12
    for j, Rj in enumerate(R):
        H = T + np.diag(model.W(r, Rj))
        gram = h * states[j] @ states[j].T
        assert np.max(np.abs(gram - np.eye(n_states))) < 1e-12
        assert np.max(np.abs(states[j] @ H - E[j][:, None] * states[j])) < 1e-10
