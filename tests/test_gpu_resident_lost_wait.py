"""A wait between a team's workgroups that is given up (its limit set to zero
from the host, so every workgroup leaves by itself) ends the call with
DEVICE_ERROR: it is not continued by launches from an x that members may have
written.  The next solve with the usual limit has the launches' bits."""
import numpy as np
import pytest

import fvcases as fc
from tests.gpu_util import DevCase, say, to_dev
from tests.test_gpu_resident import fv  # noqa: F401

pytestmark = pytest.mark.gpu


def solvers(fv, dc):  # noqa: F811
    import torch

    z = torch.zeros_like
    for method in ("pipecg", "pipecg_literal", "cg"):
        yield method, lambda m=method: fv.solve(dc.A, dc.b, x=z(dc.b), tol=1e-10, method=m)
        yield "noalloc " + method, lambda m=method: fv.solve_noalloc(dc.A, dc.b, z(dc.b), tol=1e-10, method=m)
    yield "mixed", lambda: fv.solve_mixed_reliable(dc.A, dc.b, x=z(dc.b), tol=1e-10, update_every=16)
    b = torch.stack([dc.b, 2.0 * dc.b.flip(0)])
    yield "bicgstab", lambda: fv.solve_bicgstab_multi(dc.A, b, x=z(b), tol=1e-10)


def check(fv, monkeypatch, name, run):  # noqa: F811
    import torch

    say("lost wait", name)
    monkeypatch.setenv("FVPCG_RESIDENT", "0")
    want = run()[0].clone()
    monkeypatch.setenv("FVPCG_RESIDENT", "1")
    monkeypatch.setenv("FVPCG_RESIDENT_SPIN_MS", "0")
    with pytest.raises(fv.FVPCGError) as e:
        run()
    assert e.value.code == fv.DEVICE_ERROR and "wait between workgroups" in str(e.value)
    monkeypatch.delenv("FVPCG_RESIDENT_SPIN_MS")
    assert torch.equal(run()[0], want)


def test_lost_wait_is_an_error(fv, monkeypatch):  # noqa: F811
    dc = DevCase(fc.varcoef((40, 36, 30), seed=6), fp32_copy=True)
    for name, run in solvers(fv, dc):
        check(fv, monkeypatch, name, run)
    dc.close()


@pytest.mark.parametrize("method", ["pipecg", "cg"])
def test_lost_wait_streamed(fv, monkeypatch, method):  # noqa: F811
    import torch

    dc = DevCase(fc.varcoef((112, 110, 108), seed=6, permute=False))
    check(fv, monkeypatch, "streamed " + method,
          lambda: fv.solve(dc.A, dc.b, x=torch.zeros_like(dc.b), tol=1e-4, method=method))
    dc.close()


@pytest.mark.parametrize("method", ["pipecg", "cg"])
def test_lost_wait_in_a_batch(fv, monkeypatch, method):  # noqa: F811
    """The bound of a batch handle's waits (FVPCG_BATCH_BARRIER_TIMEOUT_MS at
    its creation) holds for teams in one launch too."""
    import torch

    bt = fc.concat([fc.varcoef(s, seed=1, permute=False) for s in ((20, 20, 20), (33, 20, 17))])

    def batch():
        return fv.Batch(bt.cell_off, bt.face_off, to_dev(bt.owner, torch.int32), to_dev(bt.neighbour, torch.int32),
                        to_dev(bt.diag), to_dev(bt.upper))

    say("lost wait batch", method)
    b = to_dev(bt.b)
    B = batch()
    want, st, code = fv.solve_batched(B, b, x=torch.zeros_like(b), tol=1e-9, method=method)
    assert code == 0
    monkeypatch.setenv("FVPCG_BATCH_BARRIER_TIMEOUT_MS", "0")
    B0 = batch()
    monkeypatch.delenv("FVPCG_BATCH_BARRIER_TIMEOUT_MS")
    with pytest.raises(fv.FVPCGError) as e:
        fv.solve_batched(B0, b, x=torch.zeros_like(b), tol=1e-9, method=method)
    assert e.value.code == fv.DEVICE_ERROR and "wait between workgroups" in str(e.value)
    x, again, code = fv.solve_batched(B, b, x=torch.zeros_like(b), tol=1e-9, method=method)
    assert code == 0 and torch.equal(x, want) and [s["iters"] for s in again] == [s["iters"] for s in st]
    B0.close()
    B.close()


def test_queueing_is_not_a_lost_wait(fv, monkeypatch):  # noqa: F811
    """Teams of 99, 99 and 81 members on 256 workgroups: 58 members of the third
    system wait for the other 23 until these have finished a larger system.
    At a limit (of each wait) far below the time of that solve the batch ends
    with the usual bits."""
    import torch

    say("queued batch, short limit")
    bt = fc.concat([fc.varcoef((e, e, e), seed=e + k, permute=False) for k, e in enumerate((74, 74, 69))])
    assert [-(-c // 4096) for c in np.diff(bt.cell_off)] == [99, 99, 81]
    got = []
    for limit in ("5000", "4"):
        monkeypatch.setenv("FVPCG_BATCH_BARRIER_TIMEOUT_MS", limit)
        B = fv.Batch(bt.cell_off, bt.face_off, to_dev(bt.owner, torch.int32), to_dev(bt.neighbour, torch.int32),
                     to_dev(bt.diag), to_dev(bt.upper))
        b = to_dev(bt.b)
        x, st, code = fv.solve_batched(B, b, x=torch.zeros_like(b), tol=0.0, maxit=1200, method="cg")
        assert code == fv.NOT_CONVERGED and [s["iters"] for s in st] == [1200] * 3
        assert st[0]["device_ms"] > 8.0  # the queued system began after at least half of it
        got.append(x)
        B.close()
    assert torch.equal(got[0], got[1])
