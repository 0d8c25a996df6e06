"""Runs in which nothing arrives with step 0 (tracks that come later, or none
at all), from a workspace full of NaN, against the oracle."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_1610_06749_amd as it
    it.lib()
    return it


def poisoned(gpu, ch, n):
    import torch
    size = gpu.it_workspace_size(ch, n)
    return torch.full((size // 8 + 1,), float("nan"), dtype=torch.float64, device="cuda").view(torch.uint8)[:size]


@pytest.mark.parametrize("ex", [None, dict(kernel=1), dict(steps_per_pass=3)], ids=["default", "T1", "T3"])
@pytest.mark.parametrize("absorbing", [0, 1])
@pytest.mark.parametrize("late", [True, False])
def test_nothing_with_step_0(gpu, orc, ex, absorbing, late):
    ch = W.chamber(33, 20, 17, 4e-4, 17 * 4e-4, 60.0, lateral_bc=absorbing, reaction_limit=0.0)
    ch.update(max_steps=30, stop_tol=0.0 if late else 1e-12)
    rows = [[3.0, 1e-3, 5e-3, 4e-3, 0.3, 1.0, 0.0], [2.0, 8e-4, 9e-3, 2e-3, 0.0, 0.0, 0.0]] if late else []
    tr = W.tracks(rows) if late else W.no_tracks()
    dt = orc.dt(ch, tr)
    if late:
        tr[0, 6], tr[1, 6] = 4.5 * dt, 11.5 * dt
    for _ in range(2):
        g = gpu.it_solve(ch, tr, exec=ex, ws=poisoned(gpu, ch, len(tr)), trace=True, fields=ex is None)
        o = orc.solve(ch, tr, with_trace=True)
        assert g["steps"] == o["steps"] and g["flags"] == o["flags"]
        N = max(o["n_released"], 1.0)
        assert np.max(np.abs(g["trace"][:, :9] - o["trace"][:, :9])) <= 1e-9 * N
        assert g["n_released"] == pytest.approx(o["n_released"], rel=1e-9)
        if ex is None:
            for k in ("pos", "neg"):
                assert np.linalg.norm(g[k].cpu().numpy() - o[k]) <= 1e-9 * np.linalg.norm(o[k])
