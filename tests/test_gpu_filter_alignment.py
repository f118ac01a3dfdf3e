"""The similarity filter reads 16 bytes of each latent at a time where length and addresses allow it: the same errors from every start address
and for lengths around a vector, a pass of 1024 threads and four of them."""
import numpy as np
import pytest
import torch

import oracle
import paper_2605_28657_amd as pa

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n", [1, 7, 8, 9, 4096, 8192, 8200, 32768, 32776, 100001])
@pytest.mark.parametrize("at", [(0, 0), (1, 1), (8, 3)])
def test_filter_at_any_address(dtype, n, at):
    g = torch.Generator("cuda:0").manual_seed(n)
    flat = [torch.randn(2 * n + 16, device="cuda:0", generator=g).to(dtype) for _ in range(2)]
    a, b = (f[o:o + 2 * n].view(2, 1, n) for f, o in zip(flat, at))
    mse, flag = pa.latent_similarity(a, b, 2.0)
    for c in range(2):
        ref = oracle.latent_mse(a[c].float().cpu().numpy(), b[c].float().cpu().numpy())
        # doubles in any order, then one rounding to fp32
        assert float(mse[c]) == pytest.approx(ref, rel=2.0 ** -23, abs=1e-30)
        assert bool(flag[c]) == bool(np.float32(float(mse[c])) < np.float32(2.0))


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("n", [4096, 4099, 65536])
def test_the_error_does_not_depend_on_the_address(dtype, n):
    """Squared differences 1, 2^-24 and some 2^-54, whose sum is halfway between two fp32 values: the small ones count or are lost with the order of
    the sums in double.  The same latents give the same fp32 error wherever they start."""
    d = torch.zeros(n, dtype=torch.float64)
    d[0], d[1], d[2:8] = 1.0, 2.0 ** -12, 2.0 ** -27
    seen = []
    for at in range(9):
        a, b = (torch.zeros(n + 16, device="cuda:0", dtype=dtype) for _ in range(2))
        a[at:at + n] = d.to(dtype).to("cuda:0")
        mse, _ = pa.latent_similarity(a[at:at + n].view(1, 1, n), b[at // 2:at // 2 + n].view(1, 1, n), 2.0)
        seen.append(float(mse[0]))
    assert len(set(seen)) == 1 and seen[0] == pytest.approx(1.0 / n, rel=2.0 ** -22), seen
