"""The gather's tiles of 32 frames x 16 channels: remainders of both, several of both, one frame, windows that start inside the clip, the
operand formats, and skipped clips, through a stack of one transposed convolution against the oracle."""
import numpy as np
import pytest
import torch

import demon_inputs as di
import oracle
from gpu_util import assert_close, make, to_device

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("grid")]


@pytest.mark.parametrize("c0,width,dtype,kw", [(1, 8, "f32", {}), (17, 16, "f32", {}), (40, 32, "f32", {}), (16, 32, "bf16", {}), (48, 64, "bf16", {}),
                                               (64, 512, "bf16", {}), (64, 512, "bf16", dict(wide_operands=2))])
@pytest.mark.parametrize("T", [1, 31, 32, 33, 70])
def test_gather(c0, width, dtype, kw, T):
    spec = di.DecoderSpec(c0, (2,), (width,), ())
    vae, w, z = make(spec, dtype, T, n_clips=3, snake="uniform", max_extended_frames=12 * T + 100, **kw)
    zt = to_device(z, dtype)
    ref = np.stack([oracle.decode(spec, w, c) for c in z])
    got = vae.decode(zt)
    assert_close(got.cpu().numpy(), ref, dtype, str(spec))
    b = T // 3
    part = vae.decode_windowed(zt, window=T, halo=-1, frame_begin=b, frame_end=T)
    assert torch.equal(part[:, :, 2 * b:], got[:, :, 2 * b:])
    out = torch.full_like(got, 7.0)
    vae.decode_windowed_gated(zt, torch.tensor([0, 1, 0], dtype=torch.int32, device="cuda:0"), out, window=9, halo=-1)
    assert torch.equal(out[::2], got[::2]) and (out[1] == 7).all()
    vae.close()
