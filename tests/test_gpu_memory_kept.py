"""What the library keeps of freed device memory while a handle lives stays
within the bound that FVPCG_POOL_MB sets: the scratch of an AMG setup and the
closed hierarchy are the device's again."""
import pytest

import fvcases as fc
from tests.gpu_util import DevCase, say
from tests.test_gpu_resident import fv  # noqa: F401

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bound", [0, 64])
def test_kept_memory_is_bounded(fv, monkeypatch, bound):  # noqa: F811
    import gc

    import torch

    say("kept memory", bound)
    monkeypatch.setenv("FVPCG_POOL_MB", str(bound))
    gc.collect()
    dc = DevCase(fc.varcoef((64, 64, 64), seed=3, permute=False))
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    for _ in range(2):  # a setup's scratch and hierarchy: about 430 MiB
        M = fv.AMG(dc.A)
        M.close()
    torch.cuda.synchronize()
    kept = free - torch.cuda.mem_get_info()[0]
    say("kept MiB:", kept / 2**20)
    assert kept <= (bound + 8) << 20  # 8: the driver's own granularity
    dc.close()
