"""Batches of narrow periodic chambers (one block per cross-section and chunk
of planes) against the CPU oracle, at the edges of the block shapes: two,
three and four rows per thread, the widest sections, lanes without a node,
the shortest gaps, chunk remainders, and mixed cross-sections."""
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


def chamber(nx, ny, nz, seed, **over):
    rng = np.random.default_rng(seed)
    ch = W.chamber(nx, ny, nz, 3e-4, nz * 3e-4, float(rng.uniform(20, 80)), uniform_n0=float(rng.uniform(1e8, 5e9)))
    ch.update(max_steps=80, **over)
    k = 1 + seed % 3
    th = np.where(np.arange(k) == 1, 0.3, 0.0)  # some tilted
    tr = np.stack([rng.uniform(1, 20, k), rng.uniform(6e-4, 1.5e-3, k), rng.uniform(0, nx * 3e-4, k),
                   rng.uniform(0, ny * 3e-4, k), th, rng.uniform(0, 6, k), np.zeros(k)], axis=1)
    return ch, W.tracks(tr)


def compare(g, o):
    assert g["steps"] == o["steps"] and g["flags"] == o["flags"]
    assert g["f"] == pytest.approx(o["f"], rel=1e-9)
    N = max(o["n_released"], 1.0)
    for k in ("n_released", "n_recombined", "col_pos_anode", "col_pos_cathode", "col_neg_anode", "col_neg_cathode",
              "n_inflight_pos", "n_inflight_neg"):
        assert abs(g[k] - o[k]) <= 1e-9 * N, k
    assert g["max_beta_n"] == pytest.approx(o["max_beta_n"], rel=1e-9)


SHAPES = [(24, 24), (20, 20), (33, 33), (28, 28), (32, 32), (1, 2), (2, 3), (64, 16), (512, 2), (46, 44), (3, 170)]


@pytest.mark.parametrize("nx,ny", SHAPES, ids=[f"{a}x{b}" for a, b in SHAPES])
def test_sections_match_oracle(gpu, orc, nx, ny):
    cells = [chamber(nx, ny, nz, 10 * nz + nx) for nz in (3, 4, 5, 7, 8, 13, 40)]
    res = gpu.it_solve_batch(*zip(*cells))
    for (ch, tr), g in zip(cells, res):
        compare(g, orc.solve(ch, tr, with_fields=False))


def test_mixed_sections_match_oracle(gpu, orc):
    """Cross-sections of different sizes in one batch: blocks sized for the
    largest, idle lanes in the others."""
    shapes = [(24, 24, 30), (20, 18, 9), (30, 24, 17), (24, 21, 12), (16, 24, 25)]
    cells = [chamber(nx, ny, nz, 7 + q) for q, (nx, ny, nz) in enumerate(shapes)]
    for (ch, tr), g in zip(cells, gpu.it_solve_batch(*zip(*cells), exec=dict(check_every=4))):
        compare(g, orc.solve(ch, tr, with_fields=False))


def test_many_sections_match_oracle(gpu, orc):
    """Enough blocks for several on a compute unit (the crowded form), with
    chunks that change as chambers stop."""
    cells = [chamber(24, 24, 40 + 9 * (q % 5), q % 10) for q in range(150)]
    res = gpu.it_solve_batch(*zip(*cells), exec=dict(check_every=2))
    seen = {}
    for q, ((ch, tr), g) in enumerate(zip(cells, res)):
        if q % 10 not in seen:
            seen[q % 10] = orc.solve(ch, tr, with_fields=False)
        compare(g, seen[q % 10])


@pytest.mark.parametrize("period", [3, 4, 5, 11])
def test_section_trains_match_oracle(gpu, orc, period):
    """Pulse trains with the shortest period a pass takes, and longer ones."""
    cells = []
    for q, (nx, ny, nz) in enumerate([(24, 24, 8), (20, 24, 13), (24, 12, 21)]):
        ch, tr = chamber(nx, ny, nz, 3 + q)
        dt = orc.dt(ch, tr)
        ch.update(n_pulses=5, pulse_period_s=period * dt * 0.999, max_steps=100000)
        cells.append((ch, tr))
    for (ch, tr), g in zip(cells, gpu.it_solve_batch(*zip(*cells))):
        o = orc.solve(ch, tr, with_fields=False)
        compare(g, o)
        assert g["pulses"] == o["pulses"] and g["period_collected"] == pytest.approx(o["period_collected"], rel=1e-9)
