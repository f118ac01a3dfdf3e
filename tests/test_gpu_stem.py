"""The encoder's stem: the fp32 MFMA kernel (whole groups of 64 channels, at most 16 taps x channels) at the sizes where it can go
wrong -- remainders of its K steps, of its rows and of a wave's 16 rows, several groups of channels -- and the kernel beside it, through
stacks of a stem and one strided convolution against the oracle.  fp32: at most 16 products and a bias, then the strided conv; both
types at the bars of the encode."""
import numpy as np
import pytest
import torch

import demon_inputs as di
import oracle
from paper_2605_28657_amd import DemonVAEEncoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("width", [64, 128, 192, 96])       # 96: a row per thread
@pytest.mark.parametrize("ch,k", [(1, 1), (2, 7), (1, 15), (3, 5), (5, 3), (2, 9)])      # 9 x 2: more than 16 values
@pytest.mark.parametrize("T", [3, 256, 257, 777])           # rows: 2 T; 512 a workgroup
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_stem(width, ch, k, T, dtype):
    spec = di.DecoderSpec(64, (2,), (width,), (), head_kernel=k, out_channels=ch)
    w = di.make_encoder_weights(spec, bf16=dtype == "bf16", snake="uniform")
    x = di.make_waveform(ch, 2 * T, 40)[None]
    enc = DemonVAEEncoder(spec, w, dtype=dtype, max_frames=T, max_extended_frames=6 * T + 200)
    xt = torch.from_numpy(x).to("cuda:0")
    m, _ = enc.encode(xt)
    ref = oracle.encode_moments(spec, w, x)
    got = m.cpu().numpy()
    scale = max(1.0, float(np.abs(ref).max()))
    assert np.linalg.norm(got - ref) <= (1e-5 if dtype == "f32" else 1e-2) * np.linalg.norm(ref)
    assert np.abs(got - ref).max() <= (1e-5 if dtype == "f32" else 2e-2) * scale
    n = min(T, 61)                                           # rows off the tile's grid
    mw, _ = enc.encode_windowed(xt, window=n, halo=-1, frame_begin=T - n, frame_end=T)
    assert torch.equal(mw[:, :, T - n:], m[:, :, T - n:])
    # a value that is not finite stays within the rows that read it
    bad = xt.clone()
    bad[0, 0, 0] = float("inf")
    mb, _ = enc.encode(bad)
    far = min(T, 2 + (k + 1) // 2)
    assert torch.equal(mb[:, :, far:], m[:, :, far:])
    enc.close()
