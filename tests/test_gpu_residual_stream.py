"""A unit before a resampling convolution hands on its activated operand alone: its sum is written only for the debug tap, and the
result is the same with and without it, in every kernel that may stand there."""
import numpy as np
import pytest
import torch

import demon_inputs as di
from gpu_util import make, to_device
from paper_2605_28657_amd import DemonVAEEncoder

pytestmark = pytest.mark.gpu


# widths: fused units of 64, 128 and 256 channels, two kernels at 512 (streamed) and 96 (LDS-staged); frames: launches of few tiles and of many
@pytest.mark.parametrize("width", [64, 96, 128, 256, 512])
@pytest.mark.parametrize("T", [9, 1200, 24000])
@pytest.mark.parametrize("dtype,kw", [("bf16", {}), ("bf16", dict(wide_operands=2)), ("bf16", dict(flags=1)), ("f32", {})])
def test_sum_before_a_resampling_conv(width, T, dtype, kw):
    if dtype == "f32":
        T = min(T, 1200)
    spec = di.DecoderSpec(64, (2, 2), (width, 32), (1, 3))
    vae, w, z = make(spec, dtype, T, max_extended_frames=T, **kw)
    zt = to_device(z, dtype)
    got = vae.decode(zt)
    dst = torch.full((2 * T * width,), float("nan"), device="cuda:0")
    vae.tap(2, dst)                                          # the last unit of the first block
    tapped = vae.decode(zt)
    vae.tap(-1)
    assert torch.equal(got, tapped) and got.abs().max() > 0
    assert torch.isfinite(dst).all() and dst.abs().max() > 0
    vae.close()
    if dtype == "bf16" and not kw.get("wide_operands"):
        enc = DemonVAEEncoder(di.DecoderSpec(64, (2, 2), (64, width), (1, 3)), di.make_encoder_weights(di.DecoderSpec(64, (2, 2), (64, width), (1, 3)), bf16=True),
                              dtype=dtype, max_frames=T, max_extended_frames=T, **kw)
        x = torch.from_numpy(di.make_waveform(2, 4 * T, 40)[None]).to("cuda:0")
        m, _ = enc.encode(x)
        enc.tap(1, torch.zeros(4 * T * width, device="cuda:0"))
        mt, _ = enc.encode(x)
        assert torch.equal(m, mt) and np.isfinite(m.cpu().numpy()).all()
        enc.close()
