"""The sizes at which a launch rule changes kernels, or at which a kernel's own tiling leaves remainders, each against
the CPU oracle (or, where the oracle would take too long, an fp64 computation on the device)."""
import math

import numpy as np
import pytest
import torch

import oracle
from conftest import assert_rel_l2, to_np
from paper_2506_05096_amd import binding as ab

pytestmark = pytest.mark.gpu
DEV = "cuda"


# score: 16 tokens per workgroup below 49152 tokens, 64 per wave from there on; slabs of 256 bytes, four in flight;
# a width that is no multiple of the 16-byte vector ends on single channels.  Bit-exact.
@pytest.mark.parametrize("n,c,stride,dtype", [
    (15, 128, 128, torch.bfloat16), (16, 256, 256, torch.bfloat16), (17, 384, 384, torch.bfloat16),      # 1 - 3 slabs
    (33, 512, 512, torch.bfloat16), (40, 640, 648, torch.bfloat16), (31, 1152, 1152, torch.bfloat16),    # 4, 5, 9 slabs
    (50, 515, 520, torch.bfloat16), (50, 1, 8, torch.bfloat16), (50, 130, 131, torch.bfloat16),          # ragged widths, element path
    (47, 63, 64, torch.float32), (48, 64, 64, torch.float32), (49, 321, 324, torch.float32), (20, 3, 4, torch.float32),
    (49151, 24, 24, torch.bfloat16), (49152, 24, 24, torch.bfloat16), (49153, 40, 40, torch.float32),
])
@pytest.mark.parametrize("mode", [ab.DELTA_L2, ab.DELTA_MEAN_ABS])
def test_score_sizes(n, c, stride, dtype, mode):
    g = torch.Generator().manual_seed(n + c)
    prev, cur = torch.randn(n, stride, generator=g).to(dtype), torch.randn(n, stride, generator=g).to(dtype)
    exp = oracle.score(to_np(cur)[:, :c], to_np(prev)[:, :c], mode)
    out = torch.full((n,), -1.0, device=DEV)
    ab.astraea_score(cur.to(DEV)[:, :c], prev.to(DEV)[:, :c], out, mode)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy().view(np.uint32), exp.view(np.uint32))
