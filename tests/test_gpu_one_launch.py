"""Which path a solve took (stats' one_launch): at every size of the tests that
compare the one-launch forms with the launches, where they have to run and
where they end; just past their limits; and switched off.  A handful of iterations is
enough to tell."""
import pytest

import fvcases as fc
from tests import test_gpu_resident as res, test_gpu_resident_bicg as bicg, test_gpu_resident_cg_stream as cgs
from tests.gpu_util import DevCase, say, to_dev
from tests.test_gpu_resident import LINE, STAR, fv, stencil  # noqa: F401

pytestmark = pytest.mark.gpu
METHODS = ("pipecg", "pipecg_literal", "cg")


def path(fv, dc, method, **kw):  # noqa: F811
    import torch

    say("path", method, kw)
    try:
        return fv.solve(dc.A, dc.b, x=torch.zeros_like(dc.b), tol=0.0, maxit=3, method=method, **kw)[1]["one_launch"]
    except fv.FVPCGError as e:  # solved exactly: tol = 0 breaks down, without stats
        assert e.code == fv.BREAKDOWN
        return None


SOLVES = {**{k: (m, "0" if "col32" in o else "1") for k, (m, o) in res.CASES.items()}, **res.STREAMED, **cgs.SHAPES,
          "line-8388608": (lambda: stencil(8388608, 1, LINE, 1), "1")}
CG_MOST, LITERAL_MOST = 4194304, 524288


@pytest.mark.parametrize("name", list(SOLVES))
def test_solve_path(fv, monkeypatch, name):  # noqa: F811
    make, col16 = SOLVES[name]
    monkeypatch.setenv("FVPCG_COL16", col16)
    case = make()
    dc = DevCase(case)
    for method in METHODS:
        most = {"pipecg": 1 << 23, "cg": CG_MOST, "pipecg_literal": LITERAL_MOST}[method]
        got = path(fv, dc, method)
        assert got == int(case.n <= most) or (got is None and case.n == 1), method
    monkeypatch.setenv("FVPCG_RESIDENT", "0")
    for method in METHODS:
        assert not path(fv, dc, method)
    dc.close()


WIDE = [(i, j) for i in range(-1, 2) for j in range(3) if (i, j) > (0, 0)]  # 12 to 16 neighbours


@pytest.mark.parametrize("name", ["line-8388609", "wide rows"])
def test_solve_path_past_the_limits(fv, name):  # noqa: F811
    dc = DevCase(stencil(8388609, 1, LINE, 1) if name != "wide rows" else stencil(60, 50, WIDE, 2))
    assert [path(fv, dc, m) for m in METHODS] == [0, 0, 0]
    dc.close()


def test_no_time_to_meet_takes_launches(fv, monkeypatch):  # noqa: F811
    """A rendezvous limit of zero is never met, whatever the team's size."""
    monkeypatch.setenv("FVPCG_RESIDENT_MEET_MS", "0")
    for shape, meets in (((17, 13, 20), 0), ((128, 64, 128), 0), ((128, 128, 128), 0), ((12, 11, 10), 1)):
        dc = DevCase(fc.varcoef(shape, seed=11, permute=False))  # the last: one workgroup, nobody to meet
        for method in ("pipecg", "cg"):
            assert path(fv, dc, method) == meets
        dc.close()


@pytest.mark.parametrize("shape", [(17, 13, 11), (128, 128, 120)])
def test_no_time_to_meet_other_solvers(fv, monkeypatch, shape):  # noqa: F811
    """Mixed precision, BiCGSTAB and batches go on by launches from where the
    team left: the bits of the launches."""
    import torch

    monkeypatch.setenv("FVPCG_TUNE", "0")
    case = fc.varcoef(shape, seed=11, permute=False)
    dc = DevCase(case, fp32_copy=True)
    b3 = torch.stack([dc.b, dc.b.flip(0), 3.0 * dc.b])
    bt = fc.concat([fc.varcoef(s, seed=1, permute=False) for s in ((20, 20, 20), (33, 20, 17))])
    B = fv.Batch(bt.cell_off, bt.face_off, to_dev(bt.owner, torch.int32), to_dev(bt.neighbour, torch.int32),
                 to_dev(bt.diag), to_dev(bt.upper))
    bb = to_dev(bt.b)
    runs = {
        "mixed": lambda: fv.solve_mixed_reliable(dc.A, dc.b, tol=0.0, update_every=7, maxit=35),
        "bicgstab": lambda: fv.solve_bicgstab_multi(dc.A, b3, x=torch.zeros_like(b3), tol=1e-10, maxit=20),
        "batch": lambda: fv.solve_batched(B, bb, x=torch.zeros_like(bb), tol=1e-9, maxit=300)[:2],
    }
    for name, run in runs.items():
        got = []
        for on, meet in (("0", "20"), ("1", "0"), ("1", "20")):
            say("no time", name, shape, on, meet)
            monkeypatch.setenv("FVPCG_RESIDENT", on)
            monkeypatch.setenv("FVPCG_RESIDENT_MEET_MS", meet)
            x, st = run()
            st = st if isinstance(st, list) else [st]
            assert all(s["one_launch"] == int((on, meet) == ("1", "20")) for s in st), (name, on, meet)
            got.append((x.clone(), [(s["iters"], s["r0_norm"], s["rel_res"]) for s in st]))
        assert torch.equal(got[0][0], got[1][0]) and got[0][1] == got[1][1], name
    B.close()
    dc.close()


def test_noalloc_path(fv):  # noqa: F811
    import torch

    for shape in ((12, 11, 10), (40, 36, 30), (128, 64, 128)):
        dc = DevCase(fc.varcoef(shape, seed=3, permute=False))
        for method in ("pipecg", "cg"):
            say("noalloc path", shape, method)
            _, st = fv.solve_noalloc(dc.A, dc.b, torch.zeros_like(dc.b), tol=0.0, maxit=3, method=method)
            assert st["one_launch"] == 1
        dc.close()


@pytest.mark.parametrize("name", list(bicg.SHAPES))
def test_bicgstab_path(fv, monkeypatch, name):  # noqa: F811
    import torch

    case = fc.momentum(bicg.SHAPES[name], permute=False)
    dc = DevCase(case, symmetric=False)
    for nr in (1, 2, 3, 4):
        b = torch.stack([dc.b] * nr)
        for on in (1, 0):
            say("bicgstab path", name, nr, on)
            monkeypatch.setenv("FVPCG_RESIDENT", str(on))
            _, st = fv.solve_bicgstab_multi(dc.A, b, x=torch.zeros_like(b), tol=1e-10, maxit=2)
            most = {1: 131072, 2: 1 << 21, 3: 1 << 21, 4: 0}[nr]
            assert [s["one_launch"] for s in st] == [int(on and case.n <= most)] * nr
    dc.close()


MIXED = {**res.MIXED, "cube-2097152": lambda: fc.varcoef((128, 128, 128), seed=11, permute=False),
         "past": lambda: fc.varcoef((129, 128, 128), seed=11, permute=False)}


@pytest.mark.parametrize("name", list(MIXED))
def test_mixed_path(fv, monkeypatch, name):  # noqa: F811
    case = MIXED[name]()
    for col16, most in (("1", 1 << 21), ("0", 1 << 20)):
        monkeypatch.setenv("FVPCG_COL16", col16)
        dc = DevCase(case, fp32_copy=True)
        for on in (1, 0):
            say("mixed path", name, col16, on)
            monkeypatch.setenv("FVPCG_RESIDENT", str(on))
            _, st = fv.solve_mixed_reliable(dc.A, dc.b, tol=0.0, update_every=7, maxit=14)
            assert st["one_launch"] == int(on and case.n <= most)
        dc.close()


def test_mixed_path_of_short_periods(fv):  # noqa: F811
    """Below three iterations between updates the launches are the faster."""
    dc = DevCase(fc.varcoef((32, 31, 30), seed=11), fp32_copy=True)
    for every, want in ((1, 0), (2, 0), (3, 1)):
        say("mixed path", every)
        _, st = fv.solve_mixed_reliable(dc.A, dc.b, tol=0.0, update_every=every, maxit=6)
        assert st["one_launch"] == want
    dc.close()


@pytest.mark.parametrize("name,count,edge,order,want", [
    ("second round nearly empty", 300, 13, "yes", 0), ("in order", 200, 15, "yes", 1),
    ("rounds filled", 510, 13, "yes", 1), ("in no order", 300, 20, "no", 0), ("in order, larger", 300, 20, "yes", 1),
    ("few systems", 100, 15, "no", 1)])
def test_batch_path_of_standard_cg(fv, monkeypatch, name, count, edge, order, want):  # noqa: F811
    """Standard CG of many small systems, or of systems whose cells are in no
    order, keeps to the queue where the queue fills the chip; pipelined CG runs
    in one launch."""
    import torch

    from tests.test_gpu_one_launch_order import shuffled

    monkeypatch.setenv("FVPCG_TUNE", "0")
    case = fc.varcoef((edge, edge, edge), seed=2, permute=False)
    bt = fc.concat([case if order == "yes" else shuffled(case)] * count)
    B = fv.Batch(bt.cell_off, bt.face_off, to_dev(bt.owner, torch.int32), to_dev(bt.neighbour, torch.int32),
                 to_dev(bt.diag), to_dev(bt.upper))
    b = to_dev(bt.b)
    for method, path in (("pipecg", 1), ("cg", want)):
        say("batch path", name, method)
        _, st, _ = fv.solve_batched(B, b, x=torch.zeros_like(b), tol=1e-9, maxit=3, method=method)
        assert all(s["one_launch"] == path for s in st)
    B.close()


def test_batch_path(fv, monkeypatch):  # noqa: F811
    import torch

    monkeypatch.setenv("FVPCG_TUNE", "0")
    small = [fc.varcoef((12, 12, 12), seed=k) for k in range(5)]  # 1,728 cells on average
    for name, cases, want in [(k, m(), 1) for k, m in res.BATCHES.items()] + [
            ("small", small, 0), ("2,048 on average", [stencil(2048, 1, LINE, 1), stencil(64, 32, STAR, 2)], 1)]:
        bt = fc.concat(cases)
        B = fv.Batch(bt.cell_off, bt.face_off, to_dev(bt.owner, torch.int32), to_dev(bt.neighbour, torch.int32),
                     to_dev(bt.diag), to_dev(bt.upper))
        b = to_dev(bt.b)
        for method in ("pipecg", "cg"):
            for on, teams in ((1, None), (0, None), (1, "0")):
                say("batch path", name, method, on, teams)
                monkeypatch.setenv("FVPCG_RESIDENT", str(on))
                monkeypatch.delenv("FVPCG_BATCH_TEAMS", raising=False)
                if teams is not None:
                    monkeypatch.setenv("FVPCG_BATCH_TEAMS", teams)
                _, st, _ = fv.solve_batched(B, b, x=torch.zeros_like(b), tol=1e-9, maxit=5, method=method)
                assert [s["one_launch"] for s in st] == [int(want and on and teams is None)] * len(cases)
        B.close()
