"""Every form of the passes over whole cross-sections against the CPU oracle,
the form asserted by the rule's host query: the crowded kernels with two and
three rows per thread at each block size, batches that change from them to the
others as chambers stop, pulse trains in them, and the narrowest wraps."""
import numpy as np
import pytest

from test_gpu_section import chamber, compare, gpu  # noqa: F401
from test_section_forms import batch_form

pytestmark = pytest.mark.gpu


def check(gpu, orc, cells, key, **kw):  # noqa: F811
    seen = {}
    for q, ((ch, tr), g) in enumerate(zip(cells, gpu.it_solve_batch(*zip(*cells), **kw))):
        k = key(q)
        if k not in seen:
            seen[k] = orc.solve(ch, tr, with_fields=False)
        compare(g, seen[k])
        if ch.get("n_pulses", 0) >= 2:
            o = seen[k]
            assert g["pulses"] == o["pulses"] and g["period_collected"] == pytest.approx(o["period_collected"], rel=1e-9)


@pytest.mark.parametrize("nx,ny", [(1, 128), (2, 64), (64, 2), (128, 2), (3, 64), (170, 3)])
def test_narrowest_sections(gpu, orc, nx, ny):  # noqa: F811
    cells = [chamber(nx, ny, nz, 10 * nz + nx) for nz in (3, 4, 5, 7, 8, 13, 40)]
    assert batch_form(cells)[0] > 0
    check(gpu, orc, cells, lambda q: q)


# cross-section, planes and chambers for which the rule takes the crowded form;
# rows per thread, threads
CROWDED = [(24, 24, 140, 192, 3, 192), (20, 14, 140, 192, 2, 192), (16, 10, 100, 400, 2, 128), (30, 24, 140, 192, 3, 256),
           (36, 14, 140, 192, 2, 256)]


@pytest.mark.parametrize("nx,ny,nz,count,rows,threads", CROWDED, ids=[f"{c[0]}x{c[1]}" for c in CROWDED])
@pytest.mark.parametrize("train", [False, True])
def test_crowded_sections(gpu, orc, nx, ny, nz, count, rows, threads, train):  # noqa: F811
    """All chambers run to their own step limit, in ten kinds, and the batch
    goes over to the other form, and to other chunks, while they stop."""
    kinds = []
    for k in range(10):
        ch, tr = chamber(nx, ny, nz + k, k)
        if train:
            ch.update(n_pulses=3, pulse_period_s=(5 + k) * orc.dt(ch, tr) * 0.999, max_steps=100000)
        else:
            ch.update(max_steps=16 + 7 * k)
        kinds.append((ch, tr))
    cells = [kinds[q % 10] for q in range(count)]
    form = batch_form(cells)
    assert form[:3] == (rows, threads, 1), form
    last = [q for q in range(count) if q % 10 == 9]
    assert batch_form(cells, last)[2] == 0
    check(gpu, orc, cells, lambda q: q % 10, exec=dict(check_every=2))
