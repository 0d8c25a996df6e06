"""Grids around the size from which the library chooses blocked passes (three
rows per thread up to 5e6 nodes): the same run a step per launch gives the same
records, results and final fields, also where the run ends inside a pass."""
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


def both(gpu, ch, tr, **kw):
    auto = gpu.it_solve(ch, tr, trace=True, fields=True, **kw)
    plain = gpu.it_solve(ch, tr, trace=True, fields=True, exec=dict(kernel=gpu.IT_KERNEL_PLAIN), **kw)
    return auto, plain


@pytest.mark.parametrize("nx,ny,nz,over", [
    (128, 100, 97, {}), (37, 190, 180, {}), (181, 134, 60, dict(lateral_bc=1, space_charge=1)),
    (200, 180, 141, dict(lateral_bc=1)), (116, 108, 100, {})])
def test_auto_passes_match_single_steps(gpu, nx, ny, nz, over):
    r = np.random.default_rng(nx)
    ch = W.chamber(nx, ny, nz, 4e-4, nz * 4e-4, 150.0, uniform_n0=1e8, **over)
    ch.update(max_steps=20, stop_tol=0.0)
    n = 6
    tr = np.stack([r.uniform(1, 8, n), r.uniform(8e-4, 1.5e-3, n), r.uniform(0, nx * 4e-4, n), r.uniform(0, ny * 4e-4, n),
                   r.uniform(0, 0.5, n), r.uniform(0, 6, n), np.zeros(n)], axis=1)
    dt = gpu.it_dt(ch, tr)
    tr[4, 6], tr[5, 6] = 4.5 * dt, 11.5 * dt  # passes cut short at both
    ch.update(reaction_limit=0.0, dt_safety=dt / gpu.it_dt(dict(ch, reaction_limit=0.0), tr))
    auto, plain = both(gpu, ch, tr)
    assert auto["passes"] < plain["passes"] == 20 and auto["steps"] == plain["steps"] == 20
    N = plain["n_released"]
    assert np.max(np.abs(auto["trace"] - plain["trace"])) <= 1e-12 * N
    for k in ("pos", "neg"):
        a, b = auto[k].cpu().numpy(), plain[k].cpu().numpy()
        assert np.linalg.norm(a - b) <= 1e-13 * np.linalg.norm(b)


def test_fields_of_a_run_that_ends_inside_a_pass(gpu):
    """Nothing released (the run ends with its first step), and a density
    whose product overflows (a non-finite tally ends it): the fields are those
    of the last step itself."""
    for n0, flag in ((0.0, gpu.IT_FLAG_EMPTY), (1e200, gpu.IT_FLAG_NONFINITE)):
        ch = W.chamber(128, 110, 100, 4e-4, 0.04, 150.0, uniform_n0=n0, reaction_limit=0.0)
        ch.update(max_steps=20, stop_tol=0.0)
        auto, plain = both(gpu, ch, np.zeros((0, 7)))
        assert auto["steps"] == plain["steps"] < 20 and auto["flags"] == plain["flags"] and auto["flags"] & flag
        for k in ("pos", "neg"):
            assert np.array_equal(auto[k].cpu().numpy(), plain[k].cpu().numpy(), equal_nan=True)
