"""transpose_a = -1 with a reduced-precision A is refused; the message states the
rule and not a copy that the products no longer make."""
import pytest
import torch

import paper_1609_09154_amd as nmf
from tests.gpu_util import step

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [torch.bfloat16, torch.float8_e4m3fn])
def test_transpose_a_refused(dt):
    step("transpose_a with %s" % dt)
    A = torch.rand(64, 64, device="cuda").to(dt)
    W, H = torch.rand(64, 4, device="cuda"), torch.rand(4, 64, device="cuda")
    with pytest.raises(nmf.NMFError) as e:
        nmf.nmf_dense(A, W, H, iters=1, transpose_a=False)
    assert "takes transpose_a 0 only" in str(e.value) and "copy" not in str(e.value)
