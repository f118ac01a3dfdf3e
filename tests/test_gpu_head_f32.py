"""The head of the fp32 path on few windows, where a thread has one sample of one output channel: rows around its 128-sample workgroups, one and
several chunks of 16 channels, against the oracle (sums of 7 x channels products in fp32) and, bit for bit, as part of a call of many
windows, which takes four samples a thread."""
import numpy as np
import pytest
import torch

import demon_inputs as di
import oracle
from paper_2605_28657_amd import DemonVAE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [16, 32, 64])
@pytest.mark.parametrize("T", [1, 63, 64, 65, 200])          # rows: 2 T
def test_head(width, T):
    spec = di.DecoderSpec(16, (2,), (width,), ())
    w = di.make_weights(spec, snake="uniform")
    z = di.make_latent(16, T, 3)
    vae = DemonVAE(spec, w, dtype="f32", max_frames=T)
    y = vae.decode(torch.from_numpy(z).to("cuda:0"))
    ref = oracle.decode(spec, w, z)
    assert np.abs(y[0].cpu().numpy() - ref).max() <= 1e-5
    vae.close()


def test_few_and_many_samples_a_thread():
    spec, T = di.DecoderSpec(16, (2,), (32,), ()), 270000     # 528 workgroups of 1024 samples
    w = di.make_weights(spec, snake="uniform")
    z = torch.from_numpy(di.make_latent(16, T, 4)).to("cuda:0")
    vae = DemonVAE(spec, w, dtype="f32", max_frames=T)
    y = vae.decode(z)
    b, n = 135000 - 33, 333
    part = vae.decode_windowed(z, window=n, halo=-1, frame_begin=b, frame_end=b + n)
    assert torch.equal(part[:, :, 2 * b:2 * (b + n)], y[:, :, 2 * b:2 * (b + n)])
    vae.close()
