"""The rule that gives a block a narrow chamber's whole cross-section: which
batches it takes, with how many rows per thread, and in which form (host only)."""
import ctypes

import numpy as np
import pytest

import workloads as W


def batch_form(cells, running=None, ex=None):
    """(rows per thread or 0, threads, crowded, planes per chunk) of a batch
    [(chamber, tracks)] while the chambers `running` (default: all) run."""
    from paper_1610_06749_amd import binding as B
    n, chs, offs, tr = B._batch_args(*zip(*cells))
    run = np.array(list(range(n) if running is None else running), dtype=np.int32)
    out = np.zeros(4, dtype=np.int32)
    P = ctypes.c_void_p
    rc = B.lib().it_batch_form(P(ctypes.addressof(chs)), P(offs.ctypes.data), P(tr.ctypes.data), n,
                               B._exec(ex, host=False), P(run.ctypes.data), len(run), P(out.ctypes.data))
    assert rc == B.IT_OK
    return tuple(int(v) for v in out)


def cell(nx, ny, nz, **over):
    ch = W.chamber(nx, ny, nz, 3e-4, nz * 3e-4, 50.0, uniform_n0=1e8)
    ch.update(over)
    return ch, W.no_tracks()


@pytest.mark.parametrize("nx,ny,rows", [(24, 24, 3), (1, 128, 2), (2, 64, 2), (64, 2, 2), (46, 44, 4), (512, 2, 2),
                                        (170, 3, 3), (1, 2, 0), (2, 3, 0), (24, 23, 0), (47, 47, 0)])
def test_rows_of_a_cross_section(nx, ny, rows):
    R, threads, _, z = batch_form([cell(nx, ny, 40)])
    assert R == rows
    if R:
        assert ny % R == 0 and threads % 64 == 0 and nx * (ny // R) <= threads <= 512 and z >= 4


@pytest.mark.parametrize("over,ex", [(dict(lateral_bc=1), None), (dict(space_charge=1), None), ({}, dict(kernel=2)),
                                     ({}, dict(kernel=1)), ({}, dict(z_chunk=16)), ({}, dict(steps_per_pass=3)),
                                     (dict(n_pulses=3, pulse_period_s=1e-12), None)])
def test_other_batches_take_other_passes(over, ex):
    assert batch_form([cell(24, 24, 40, **over)], ex=ex)[0] == 0
    assert batch_form([cell(24, 24, 40), cell(24, 24, 30, **over)], ex=ex)[0] == 0


def test_the_crowded_form_gives_way():
    """Many chambers take the form for many blocks per CU, few the other."""
    cells = [cell(24, 24, 140 + q % 5) for q in range(192)]
    assert batch_form(cells)[2] == 1 and batch_form(cells, range(20))[2] == 0
