"""A batch handle's launch plans of standard and pipelined CG are both kept:
calls that alternate between the methods neither plan again nor wait for work
on other streams, and give each method's bits."""
import pytest

import fvcases as fc
from tests.gpu_util import say, to_dev
from tests.test_gpu_resident import fv  # noqa: F401

pytestmark = pytest.mark.gpu


def test_alternating_methods_do_not_wait_for_other_streams(fv):  # noqa: F811
    import torch

    bt = fc.concat([fc.varcoef(s, seed=1, permute=False) for s in ((20, 20, 20), (33, 20, 17), (24, 24, 24))])
    B = fv.Batch(bt.cell_off, bt.face_off, to_dev(bt.owner, torch.int32), to_dev(bt.neighbour, torch.int32),
                 to_dev(bt.diag), to_dev(bt.upper))
    b = to_dev(bt.b)

    def run(method):
        x = torch.empty_like(b).zero_()
        _, st, code = fv.solve_batched(B, b, x=x, tol=1e-9, method=method)
        assert code == 0 and all(s["one_launch"] for s in st)
        return x

    say("batch plans")
    want = {m: run(m) for m in ("cg", "pipecg")}
    keep = [torch.empty_like(b) for _ in range(4)]  # torch's allocator has blocks for the calls below
    del keep
    torch.cuda.synchronize()
    main, side, ended = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Event()
    with torch.cuda.stream(side):
        torch.cuda._sleep(int(2e9))  # one workgroup, about a second
        ended.record()
    with torch.cuda.stream(main):
        got = [(m, run(m)) for m in ("cg", "pipecg") * 2]
        main.synchronize()
        waited = ended.query()
    assert not waited
    torch.cuda.synchronize()
    for m, x in got:
        assert torch.equal(x, want[m])
    B.close()
