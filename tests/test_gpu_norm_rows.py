"""Residual + RMSNorm at the row lengths where the kernel changes path: the
ends of the 4- and 8-column register builds, rows past them, remainders; and
in place.  x_out is one fp32 addition (exact); u is one bf16 rounding of a
value whose fp32 scale is good to a few 1e-7, so it lies within one bf16 step
(2^-8 relative) of the fp64 result."""
import numpy as np
import pytest

import paper_2605_28283_amd as pp

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [1028, 2048, 4096, 4100, 8192, 8196, 12292])
@pytest.mark.parametrize("alias", ["none", "x", "y"])
def test_norm_rows(d, alias):
    import torch
    pp.load()
    T = 3
    rng = np.random.default_rng(d)
    x = rng.standard_normal((T, d)).astype(np.float32) * 7
    y = rng.standard_normal((T, d)).astype(np.float32)
    xd, yd = torch.from_numpy(x).cuda(), torch.from_numpy(y).cuda()
    out = {"none": torch.full((T, d), float("nan"), device="cuda"), "x": xd, "y": yd}[alias]
    u = torch.zeros((T, d), dtype=torch.bfloat16, device="cuda")
    pp.prunepath_residual_rmsnorm(xd, yd, out, T, d, 1e-5, u.view(torch.int16))
    torch.cuda.synchronize()
    s = x + y
    np.testing.assert_array_equal(out.cpu().numpy(), s)
    s = s.astype(np.float64)
    ref = s / np.sqrt((s ** 2).mean(1, keepdims=True) + 1e-5)
    np.testing.assert_allclose(u.float().cpu().numpy(), ref, rtol=2.0 ** -8, atol=0)
