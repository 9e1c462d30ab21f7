"""Resident solves (the whole solve in one launch, rows held on chip) against
the launch-per-iteration path and the oracle, at the edges of their tiles:
one row, one workgroup on its own (up to 2,048 cells), teams of 5 to 256
workgroups with 1 to 8 rows per thread, full and ragged last tiles, rows of
4, 6 and 8 slots, int16 and int32 columns; pipelined CG (folded and literal)
and standard CG.

Resident solves form their sums in the launch-per-iteration kernels' order
from the same expressions, so the two paths agree bit for bit.  Against the
oracle the bar is the strict one of the other solver tests, 1e-10 at equal
count."""
import numpy as np
import pytest

import fvcases as fc
import oracle
from tests.gpu_util import DevCase, rel, say, to_dev

pytestmark = pytest.mark.gpu
TILE, MOST = 512, 1 << 20


@pytest.fixture(scope="module")
def fv():
    import torch

    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_1505_07630_amd as fv

    fv.lib()
    return fv


def solve(fv, monkeypatch, dc, resident, x0=None, **kw):
    import torch

    monkeypatch.setenv("FVPCG_RESIDENT", "1" if resident else "0")
    x = torch.zeros_like(dc.b) if x0 is None else x0.clone()
    try:
        return fv.solve(dc.A, dc.b, x=x, **kw)
    except fv.FVPCGError as e:  # tol = 0 on a system solved exactly breaks down, on either path
        assert e.code == fv.BREAKDOWN
        return x, dict.fromkeys(("iters", "b_norm", "r0_norm", "rel_res", "true_rel_res"), None) | {"status": e.code}


def stencil(nx, ny, offsets, seed):
    """A 2-D mesh whose rows couple to the given (i, j) offsets and back."""
    rng = np.random.default_rng(seed)
    i, j = np.meshgrid(np.arange(nx), np.arange(ny))
    pairs = []
    for di, dj in offsets:
        a, b = i + di, j + dj
        ok = (a >= 0) & (a < nx) & (b >= 0) & (b < ny)
        pairs.append(np.stack([(i + nx * j)[ok], (a + nx * b)[ok]], 1))
    e = np.unique(np.sort(np.concatenate(pairs), axis=1), axis=0)
    n = nx * ny
    up = -np.exp(rng.standard_normal(len(e)))
    diag = np.full(n, 0.05)
    np.add.at(diag, e[:, 0], -up)
    np.add.at(diag, e[:, 1], -up)
    return fc.Case("stencil", (nx, ny, 1), n, e[:, 0].astype(np.int32), e[:, 1].astype(np.int32), diag, up, up.copy(),
                   rng.uniform(-1, 1, n))


LINE, CROSS = [(1, 0)], [(1, 0), (0, 1)]
STAR = [(1, 0), (0, 1), (1, 1), (-1, 1)]  # 8 neighbours
CASES = {
    "row": (lambda: stencil(1, 1, LINE, 1), ()),
    "line-512": (lambda: stencil(TILE, 1, LINE, 2), ()),
    "cube-504": (lambda: fc.varcoef((9, 8, 7), seed=3), ()),
    "cube-520": (lambda: fc.varcoef((13, 8, 5), seed=3), ()),
    "one-2048": (lambda: fc.varcoef((16, 16, 8), seed=4), ()),
    "team-2049": (lambda: stencil(683, 3, CROSS, 5), ()),
    "star-2500": (lambda: stencil(50, 50, STAR, 6), ()),
    "star-132000": (lambda: stencil(440, 300, STAR, 7), ()),
    "star-int32": (lambda: stencil(440, 300, STAR, 7), ("col32",)),
    "cube-131072": (lambda: fc.varcoef((64, 64, 32), seed=8), ()),
    "cube-131100": (lambda: fc.varcoef((23, 57, 100), seed=8, permute=False), ()),
    "cube-400k": (lambda: fc.varcoef((80, 50, 101), seed=9, permute=False), ()),
    "cube-400k-int32": (lambda: fc.varcoef((80, 50, 101), seed=9, permute=False), ("col32",)),
    "cube-700k": (lambda: fc.varcoef((100, 70, 100), seed=10, permute=False), ()),
    "cube-1M": (lambda: fc.varcoef((128, 64, 128), seed=11, permute=False), ()),
}


FORMS = [("pipecg", "jacobi"), ("pipecg", "none"), ("pipecg_literal", "jacobi"), ("cg", "jacobi"), ("cg", "none")]


@pytest.mark.parametrize("name", list(CASES))
def test_resident_equals_launches(fv, monkeypatch, name):
    make, opts = CASES[name]
    say("resident", name)
    if "col32" in opts:
        monkeypatch.setenv("FVPCG_COL16", "0")
    case = make()
    assert case.n <= MOST
    dc = DevCase(case)
    x0 = to_dev(np.random.default_rng(1).uniform(-1, 1, case.n))
    for method, precond in FORMS:
        for kw in (dict(tol=0.0, maxit=40), dict(tol=1e-9, maxit=60, x0=x0)):
            say("resident", name, method, precond, kw.get("tol"))
            xa, sa = solve(fv, monkeypatch, dc, False, method=method, precond=precond, **kw)
            xb, sb = solve(fv, monkeypatch, dc, True, method=method, precond=precond, **kw)
            for k in ("iters", "status", "b_norm", "r0_norm", "rel_res", "true_rel_res"):
                assert sa[k] == sb[k], k
            assert np.array_equal(xa.cpu().numpy(), xb.cpu().numpy())
    # the oracle at equal count, 25 iterations (fewer if it converges)
    for method, run in (("pipecg", oracle.pipecg), ("cg", oracle.cg)):
        xb, sb = solve(fv, monkeypatch, dc, True, method=method, tol=0.0, maxit=25)
        if sb["status"] == 1:
            xo, _ = run(oracle.system(case), case.b, tol=0.0, maxit=sb["iters"])
            assert rel(xb.cpu().numpy(), xo) <= 1e-10
    dc.close()


@pytest.mark.parametrize("shape", [(8, 8, 8), (20, 18, 16)])
def test_resident_edges(fv, monkeypatch, shape):
    """b = 0, an exact start, no iterations, a NaN right-hand side."""
    import torch

    say("resident edges", shape)
    case = fc.varcoef(shape, seed=5)
    dc = DevCase(case)
    for method in ("pipecg", "pipecg_literal", "cg"):
        monkeypatch.setenv("FVPCG_RESIDENT", "1")
        kw = dict(method=method)
        x, st = fv.solve(dc.A, torch.zeros_like(dc.b), x=torch.ones_like(dc.b), **kw)
        assert st["status"] == 0 and st["iters"] == 0 and st["true_rel_res"] == 0.0
        assert torch.count_nonzero(x).item() == 0
        xs, _ = fv.solve(dc.A, dc.b, tol=1e-12, **kw)
        x, st = fv.solve(dc.A, dc.b, x=xs.clone(), tol=1e-8, **kw)
        assert st["status"] == 0 and st["iters"] == 0 and torch.equal(x, xs)
        x, st = fv.solve(dc.A, dc.b, x=xs.clone(), tol=1e-20, maxit=0, **kw)
        assert st["status"] == 1 and st["iters"] == 0 and torch.equal(x, xs)
        bad = dc.b.clone()
        bad[case.n // 2] = float("nan")
        for res in ("0", "1"):
            monkeypatch.setenv("FVPCG_RESIDENT", res)
            with pytest.raises(fv.FVPCGError) as e:
                fv.solve(dc.A, bad, **kw)
            assert e.value.code == fv.BREAKDOWN
    dc.close()


def test_resident_rendezvous_limit(fv, monkeypatch):
    """A team that is given no time to come together leaves x alone and the
    launch-per-iteration path solves: the same bits either way."""
    import torch

    say("resident rendezvous limit")
    case = fc.varcoef((40, 36, 30), seed=6)
    dc = DevCase(case)
    xa, sa = solve(fv, monkeypatch, dc, False, tol=1e-10)
    monkeypatch.setenv("FVPCG_RESIDENT_MEET_MS", "0")
    for _ in range(3):
        xb, sb = solve(fv, monkeypatch, dc, True, tol=1e-10)
        assert sa["iters"] == sb["iters"] and torch.equal(xa, xb)
    monkeypatch.delenv("FVPCG_RESIDENT_MEET_MS")
    xb, sb = solve(fv, monkeypatch, dc, True, tol=1e-10)
    assert sa["iters"] == sb["iters"] and torch.equal(xa, xb)
    dc.close()


def test_resident_threads_and_streams(fv, monkeypatch):
    """Solves from several threads, each on its own stream and matrix: one
    team at a time holds the GPU, the others solve by launches; every result
    is bitwise that of the solve alone."""
    import threading

    import torch

    monkeypatch.setenv("FVPCG_RESIDENT", "1")
    cases = [DevCase(fc.varcoef(s, seed=7)) for s in ((40, 36, 30), (33, 31, 29), (12, 11, 10), (64, 32, 32))]
    alone = [fv.solve(dc.A, dc.b, tol=1e-10)[0].clone() for dc in cases]
    torch.cuda.synchronize()
    got, errors = {}, []

    def work(i):
        try:
            st = torch.cuda.Stream()
            st.wait_stream(torch.cuda.default_stream())
            with torch.cuda.stream(st):
                for rep in range(4):
                    got[i, rep] = fv.solve(cases[i].A, cases[i].b, tol=1e-10)[0]
            st.synchronize()
        except Exception as e:  # noqa: BLE001
            errors.append(e)

    say("resident threads")
    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(cases))]
    for t in ts:
        t.start()
    for t in ts:
        t.join(60)
    assert not errors and len(got) == 4 * len(cases)
    torch.cuda.synchronize()
    for (i, _), x in got.items():
        assert torch.equal(x, alone[i])
    for dc in cases:
        dc.close()


# ------------------------------------------------------------------ beyond what the chip holds whole

STREAMED = {
    "cube-830k-int32": (lambda: fc.varcoef((94, 94, 94), seed=12, permute=False), "0"),
    "star-600k": (lambda: stencil(800, 750, STAR, 13), "1"),
    "line-1.05M": (lambda: stencil(1050001, 1, LINE, 14), "1"),
    "cube-2097152": (lambda: fc.varcoef((128, 128, 128), seed=15, permute=False), "1"),
    "cube-2.1M": (lambda: fc.varcoef((129, 128, 128), seed=16, permute=False), "1"),
    "cube-4.2M-int32": (lambda: fc.varcoef((161, 162, 162), seed=17, permute=False), "0"),
    "cube-4.2M": (lambda: fc.varcoef((161, 162, 162), seed=17, permute=False), "1"),
}


@pytest.mark.parametrize("name", list(STREAMED))
def test_streamed_equals_launches(fv, monkeypatch, name):
    """Systems whose matrix is streamed, their vectors partly on chip: bitwise
    the launches' results (odd and even counts, a warm start that converges, no
    preconditioner), also when the team is given no time to come together."""
    import torch

    make, col16 = STREAMED[name]
    monkeypatch.setenv("FVPCG_COL16", col16)
    case = make()
    dc = DevCase(case)
    x0 = to_dev(np.random.default_rng(1).uniform(-1, 1, case.n))
    for kw in (dict(tol=0.0, maxit=8), dict(tol=0.0, maxit=7, x0=x0, precond="none"), dict(tol=3e-2, maxit=400)):
        got = []
        for mode in ("launches", "resident", "no-time"):
            say("streamed", name, mode, kw.get("tol"), kw["maxit"])
            monkeypatch.setenv("FVPCG_RESIDENT_MEET_MS", "0" if mode == "no-time" else "20")
            got.append(solve(fv, monkeypatch, dc, mode != "launches", **kw))
        (xa, sa) = got[0]
        for xb, sb in got[1:]:
            for k in ("iters", "status", "b_norm", "r0_norm", "rel_res", "true_rel_res"):
                assert sa[k] == sb[k], k
            assert torch.equal(xa, xb)
    dc.close()


# ------------------------------------------------------------------ batches

BATCHES = {
    # members per launch: all side by side at 2, 4 and 8 (standard CG 1, 2, 4) tiles each, then queued teams
    "side-by-side": lambda: [fc.varcoef(s, seed=1, permute=False) for s in ((20, 20, 20), (33, 20, 17), (5, 1, 1))],
    "queued": lambda: [fc.varcoef((e, e + 1, e + 3), seed=e, permute=False) for e in (60, 48, 47, 40, 31, 16, 16, 9)]
    + [stencil(683, 3, CROSS, 5), stencil(1, 1, LINE, 1)],
    "wide-rows": lambda: [stencil(50, 50, STAR, 6), stencil(130, 110, STAR, 7)],
}


@pytest.mark.parametrize("name", list(BATCHES))
@pytest.mark.parametrize("col32", [False, True])
def test_resident_batch(fv, monkeypatch, name, col32):
    """Every system of a resident batch against the oracle at its iteration
    count (the strict bar), bitwise reproducible, and the same statuses and
    counts within 2 as the queue's; a team without time to come together
    leaves the batch to the queue."""
    import torch

    say("resident batch", name, col32)
    monkeypatch.setenv("FVPCG_TUNE", "0")
    monkeypatch.setenv("FVPCG_COL16", "0" if col32 else "1")
    cases = BATCHES[name]()
    bt = fc.concat(cases)
    B = fv.Batch(bt.cell_off, bt.face_off, to_dev(bt.owner, torch.int32), to_dev(bt.neighbour, torch.int32),
                 to_dev(bt.diag), to_dev(bt.upper))
    b = to_dev(bt.b)
    for method, run in (("pipecg", oracle.pipecg), ("cg", oracle.cg)):
        got = {}
        for mode in ("queue", "resident", "again", "no-time"):
            say("resident batch", name, method, mode)
            monkeypatch.setenv("FVPCG_RESIDENT", "0" if mode == "queue" else "1")
            monkeypatch.setenv("FVPCG_RESIDENT_MEET_MS", "0" if mode == "no-time" else "20")
            x, st, code = fv.solve_batched(B, b, x=torch.zeros_like(b), tol=1e-9, maxit=20000, method=method)
            assert code == 0 and all(s["status"] == 0 for s in st)
            got[mode] = x.cpu().numpy(), [s["iters"] for s in st]
        assert np.array_equal(got["resident"][0], got["again"][0])
        x, its = got["resident"]
        for s, case in enumerate(cases):
            xs = x[bt.cell_off[s]:bt.cell_off[s + 1]]
            assert abs(its[s] - got["queue"][1][s]) <= 2 and abs(its[s] - got["no-time"][1][s]) <= 2
            xo, _ = run(oracle.system(case), case.b, tol=0.0, maxit=its[s])
            assert rel(xs, xo) <= 1e-10, s
    B.close()


# ------------------------------------------------------------------ mixed precision

MIXED = {
    "cube-504": lambda: fc.varcoef((9, 8, 7), seed=3),
    "line-1030": lambda: stencil(1030, 1, LINE, 2),
    "star-132000": lambda: stencil(440, 300, STAR, 7),
    "cube-262144": lambda: fc.varcoef((64, 64, 64), seed=8, permute=False),
    "cube-300k": lambda: fc.varcoef((67, 61, 75), seed=8, permute=False),
    "cube-1.3M": lambda: fc.varcoef((110, 109, 111), seed=10, permute=False),
    "cube-2M": lambda: fc.varcoef((128, 128, 127), seed=11, permute=False),
}


@pytest.mark.parametrize("name", list(MIXED))
def test_resident_mixed_equals_launches(fv, monkeypatch, name):
    """The FP32 iterations between two FP64 updates in one launch: bitwise the
    launches' results (odd and even update periods, int32 columns too), also
    when the team is given no time to come together."""
    import torch

    case = MIXED[name]()
    for col16 in ("1", "0"):
        monkeypatch.setenv("FVPCG_COL16", col16)
        dc = DevCase(case, fp32_copy=True)
        for every, tol, maxit in ((16, 1e-9, 160), (7, 0.0, 21)):
            got = []
            for mode in ("launches", "resident", "no-time"):
                say("resident mixed", name, col16, every, mode)
                monkeypatch.setenv("FVPCG_RESIDENT", "0" if mode == "launches" else "1")
                monkeypatch.setenv("FVPCG_RESIDENT_MEET_MS", "0" if mode == "no-time" else "20")
                x, st = fv.solve_mixed_reliable(dc.A, dc.b, tol=tol, update_every=every, maxit=maxit)
                got.append((x, st))
            (xa, sa) = got[0]
            for xb, sb in got[1:]:
                for k in ("iters", "outer_iters", "status", "b_norm", "r0_norm", "rel_res"):
                    assert sa[k] == sb[k], k
                assert torch.equal(xa, xb)
        dc.close()
