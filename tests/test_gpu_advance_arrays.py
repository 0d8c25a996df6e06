"""it_advance and the caller's arrays: they are read by the first launch and
written by the last one only; overlapping, unaligned and workspace-held arrays;
a plane offset beyond 2^31 bytes; one launch, two and several; a run that a
non-finite density ends."""
import ctypes

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
    yield it
    torch.cuda.empty_cache()


EXECS = [dict(kernel=1), dict(steps_per_pass=3), dict(steps_per_pass=2)]
NX, NY, NZ = 66, 31, 24
NODES = (NZ + 1) * NY * NX


def chamber():
    return W.chamber(NX, NY, NZ, 3e-4, NZ * 2e-4, 20.0, dy=4e-4)


def raw_advance(gpu, ch, dt, pos, neg, steps, ex, ws, ws_bytes):
    """The C entry on device addresses."""
    import torch
    from paper_1610_06749_amd import binding as B
    rc = B.lib().it_advance(ctypes.byref(B._chamber(ch)), dt, steps, B._exec(ex), ctypes.c_void_p(pos),
                            ctypes.c_void_p(neg), ctypes.c_void_p(ws), ws_bytes, B._stream(None), None)
    assert rc == gpu.IT_OK
    torch.cuda.synchronize()


def fields(steps, orc):
    ch = chamber()
    p0, n0 = W.perturbed_field((NZ + 1, NY, NX), seed=3, scale=1e10)
    dt = orc.dt(ch)
    return ch, dt, p0, n0, [orc.advance(ch, dt, p0, n0, s) for s in steps]


def close(got, ref):
    assert np.linalg.norm(got - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("ex", EXECS, ids=["T1", "T3", "T2"])
def test_only_the_last_launch_writes_them(gpu, orc, ex):
    """The passes between the first and the last one stand in the workspace."""
    import torch
    T = ex.get("steps_per_pass", 1)
    ch, dt, p0, n0, ((ap, an), (bp, bn), (cp, cn)) = fields((T, 2 * T, 3 * T), orc)
    p, n = torch.tensor(p0, device="cuda"), torch.tensor(n0, device="cuda")
    size = gpu.it_workspace_size(ch, 0)
    ws = torch.full((size // 8 + 1,), float("nan"), dtype=torch.float64, device="cuda").view(torch.uint8)[:size]
    gpu.it_advance(ch, dt, p, n, 3 * T, exec=ex, ws=ws)
    stride = (NODES * 8 + 255) // 256 * 256

    def held(k):
        return ws[k * stride:k * stride + NODES * 8].view(torch.float64).view(NZ + 1, NY, NX).cpu().numpy()
    for got, ref in ((held(2), ap), (held(3), an), (held(0), bp), (held(1), bn), (p.cpu().numpy(), cp),
                     (n.cpu().numpy(), cn)):
        close(got, ref)


@pytest.mark.parametrize("ex", EXECS, ids=["T1", "T3", "T2"])
@pytest.mark.parametrize("steps", [1, 2, 3, 4, 6, 7, 8])
def test_any_number_of_launches(gpu, orc, ex, steps):
    """Electrode planes full of garbage on entry: zero by definition."""
    import torch
    ch, dt, p0, n0, ((rp, rn),) = fields((steps,), orc)
    p0[0], p0[-1], n0[0], n0[-1] = 1e30, float("nan"), float("inf"), -5.0
    p, n = torch.tensor(p0, device="cuda"), torch.tensor(n0, device="cuda")
    gpu.it_advance(ch, dt, p, n, steps, exec=ex)
    close(p.cpu().numpy(), rp)
    close(n.cpu().numpy(), rn)


@pytest.mark.parametrize("ex", EXECS, ids=["T1", "T3", "T2"])
@pytest.mark.parametrize("place", ["unaligned", "first pair", "second pair"])
@pytest.mark.parametrize("steps", [3, 6, 9])
def test_arrays_anywhere(gpu, orc, ex, place, steps):
    import torch
    ch, dt, p0, n0, ((rp, rn),) = fields((steps,), orc)
    if place == "unaligned" and ex.get("kernel") == 1:
        ex = dict(ex, tile_y=8)
    size = gpu.it_workspace_size(ch, 0)
    stride = (NODES * 8 + 255) // 256 * 256 // 8
    ws = torch.zeros(size // 8 + 1, dtype=torch.float64, device="cuda")
    own = torch.zeros(2 * NODES + 3, dtype=torch.float64, device="cuda")
    if place == "unaligned":
        p, n = own[1:1 + NODES], own[NODES + 2:2 * NODES + 2]
    else:  # where the library keeps its first or second field pair
        k = 0 if place == "first pair" else 2
        p, n = ws[k * stride:k * stride + NODES], ws[(k + 1) * stride:(k + 1) * stride + NODES]
    p.copy_(torch.tensor(p0.ravel()))
    n.copy_(torch.tensor(n0.ravel()))
    raw_advance(gpu, ch, dt, p.data_ptr(), n.data_ptr(), steps, ex, ws.data_ptr(), size)
    close(p.cpu().numpy().reshape(rp.shape), rp)
    close(n.cpu().numpy().reshape(rn.shape), rn)


def test_same_array_twice(gpu, orc):
    """Overlapping arrays: stepped as copies, the negative ions' come back last."""
    import torch
    ch = chamber()
    p0, _ = W.perturbed_field((NZ + 1, NY, NX), seed=3, scale=1e10)
    dt = orc.dt(ch)
    _, rn = orc.advance(ch, dt, p0, p0, 6)
    p = torch.tensor(p0, device="cuda")
    gpu.it_advance(ch, dt, p, p, 6, exec=dict(steps_per_pass=3))
    close(p.cpu().numpy(), rn)


@pytest.mark.parametrize("ex", EXECS[:2], ids=["T1", "T3"])
def test_plane_offset_beyond_2_31_bytes(gpu, ex):
    """The cathode plane of 1024 x 1024 x 257 planes: zeroed where it is, and
    nothing else (a uniform density stays uniform away from the electrodes)."""
    import torch
    nz = 257
    ch = W.chamber(1024, 1024, nz, 4e-4, nz * 4e-4, 100.0, uniform_n0=1e6)
    dt = gpu.it_dt(ch)
    p = torch.full((nz + 1, 1024, 1024), 1e6, dtype=torch.float64, device="cuda")
    n = p.clone()
    gpu.it_advance(ch, dt, p, n, 6, exec=ex)
    for a in (p, n):
        assert not a[0].any() and not a[nz].any()
        mid = a[7:nz - 6]
        assert float(mid.max() - mid.min()) <= 1e-12 * float(mid.max()) and 0.9e6 < float(mid.min()) < 1e6
        assert bool((a[1] < a[100]).all() or (a[nz - 1] < a[100]).all())


def test_a_run_that_a_non_finite_density_ends(gpu):
    """The densities of the step that ended it come back, not those of a later
    launch (a step per launch: the last recorded step itself)."""
    import torch
    ch = chamber()
    dt = gpu.it_dt(ch)
    p = torch.full((NZ + 1, NY, NX), 1e200, dtype=torch.float64, device="cuda")
    n = p.clone()
    gpu.it_advance(ch, dt, p, n, 5, exec=dict(kernel=1))
    q = torch.full((NZ + 1, NY, NX), 1e200, dtype=torch.float64, device="cuda")
    r = q.clone()
    gpu.it_advance(ch, dt, q, r, 1, exec=dict(kernel=1))
    assert torch.equal(p.isfinite(), q.isfinite()) and torch.equal(n.isfinite(), r.isfinite())
    assert not bool(p[1:-1].isfinite().any())
