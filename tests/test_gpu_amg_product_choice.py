"""FVPCG_AMG_PRODUCT: the three product kernels of the setup (hash tables, column
tiles, heap merge) give one hierarchy, entry for entry, whose operators are the
oracle's; a name that is none of theirs is refused."""
import numpy as np
import pytest

import fvcases as fc
import oracle
from tests.gpu_util import DevCase, say
from tests.test_gpu_amg_products import hierarchy
from tests.test_gpu_resident import fv  # noqa: F401

pytestmark = pytest.mark.gpu


def test_unknown_product_is_refused(fv, monkeypatch):  # noqa: F811
    say("unknown product kernel")
    dc = DevCase(fc.varcoef((16, 15, 14), seed=2))
    for name in ("hashed", "merge64", "0"):
        monkeypatch.setenv("FVPCG_AMG_PRODUCT", name)
        with pytest.raises(fv.FVPCGError) as e:
            fv.AMG(dc.A, coarse_size=16)
        assert e.value.code == fv.INVALID_ARG and name in str(e.value)
    monkeypatch.delenv("FVPCG_AMG_PRODUCT")
    fv.AMG(dc.A, coarse_size=16).close()
    dc.close()


@pytest.mark.parametrize("theta", [0.0, 0.02])
def test_product_kernels_agree(fv, monkeypatch, theta):  # noqa: F811
    case = fc.varcoef((32, 30, 28), seed=2)
    dc = DevCase(case)
    got = {}
    for mode in ("merge", "hash", "tiled"):
        say("product kernels", theta, mode)
        monkeypatch.setenv("FVPCG_AMG_PRODUCT", mode)
        M = fv.AMG(dc.A, theta=theta, coarse_size=16)
        got[mode] = hierarchy(M)
        if mode == "hash":
            H = oracle.AMG(oracle.system(case), theta=theta, coarse_size=16)
            assert M.levels == H.levels >= 3
            for l in range(1, M.levels):
                for a, o in zip(M.export(l, "A")[:2], H.export(l, "A")[:2]):
                    assert np.array_equal(a, o)
                a, o = M.export(l, "A")[2], H.export(l, "A")[2]
                assert np.max(np.abs(a - o)) <= 1e-12 * np.max(np.abs(o))
        M.close()
    for mode in ("hash", "tiled"):
        assert len(got[mode]) == len(got["merge"])
        assert all(np.array_equal(a, b) for a, b in zip(got["merge"], got[mode]))
    dc.close()
