"""The encoder's last convolution with its K in eight parts, summed by the sampling step: one stage of a part and several, both operand
formats, one and two row panels, columns around every tile, against the oracle at the bars of the encode.  The parts and their order
are the layer's, so a row has the same bits on every tile, in every window and through the debug tap, which takes the rounded sums.  Stacks of a
stem and two strided convolutions; of the last case the partial sums do not fit the buffer, and it goes in one piece."""
import numpy as np
import pytest
import torch

import demon_inputs as di
import oracle
from paper_2605_28657_amd import DemonVAEEncoder

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("latent,strides,widths", [(64, (2, 2), (1024, 64)), (64, (8, 2), (256, 64)), (128, (8, 2), (512, 64)),
                                                   (128, (10, 2), (1024, 64)), (64, (10, 2), (1024, 64)), (128, (8, 2), (256, 64))])
@pytest.mark.parametrize("T", [1, 33, 97, 1100])
def test_parts(latent, strides, widths, T):
    spec = di.DecoderSpec(latent, strides, widths, ())
    w = di.make_encoder_weights(spec, bf16=True, snake="uniform")
    x = di.make_waveform(2, spec.total_stride * T, 40)[None]
    eps = torch.from_numpy(di.make_noise(latent, T, 70)[None]).to("cuda:0")
    enc = DemonVAEEncoder(spec, w, dtype="bf16", max_frames=T, max_extended_frames=6 * T + 400)
    xt = torch.from_numpy(x).to("cuda:0")
    m, z = enc.encode(xt, eps=eps)
    ref = oracle.encode_moments(spec, w, x)
    got = m.cpu().numpy()
    assert np.linalg.norm(got - ref) <= 1e-2 * np.linalg.norm(ref)
    assert np.abs(got - ref).max() <= 2e-2 * max(1.0, float(np.abs(ref).max()))
    mean, logvar = m[0].double().split(latent)
    want = mean + torch.exp(0.5 * logvar) * eps[0].double()
    assert (z[0].double() - want).abs().max() <= 2.0 ** -8 * want.abs().max()            # bf16 rounding of z
    n = min(T, 61)                                           # rows off the tile's grid
    mw, _ = enc.encode_windowed(xt, window=n, halo=-1, frame_begin=T - n, frame_end=T)
    assert torch.equal(mw[:, :, T - n:], m[:, :, T - n:])
    dst = torch.full((2 * latent * T,), float("nan"), device="cuda:0")
    enc.tap(1, dst)
    mt, zt = enc.encode(xt, eps=eps)
    torch.cuda.synchronize()
    enc.tap(-1)
    assert torch.equal(mt, m) and torch.equal(zt, z)
    assert torch.equal(dst.reshape(T, 2 * latent).t(), m[0])
    enc.close()
    large = DemonVAEEncoder(spec, w, dtype="bf16", max_frames=T, small_tile_wgs=-1)      # 128 x 128 tiles
    ml, _ = large.encode(xt)
    assert torch.equal(ml, m)
    large.close()


def test_parts_keep_to_finite_rows():
    """A value that is not finite stays within the rows that read it."""
    spec, T = di.DecoderSpec(64, (2, 2), (1024, 64), ()), 40
    w = di.make_encoder_weights(spec, bf16=True, snake="uniform")
    xt = torch.from_numpy(di.make_waveform(2, 4 * T, 40)[None]).to("cuda:0")
    enc = DemonVAEEncoder(spec, w, dtype="bf16", max_frames=T)
    m, _ = enc.encode(xt)
    bad = xt.clone()
    bad[0, 0, 0] = float("inf")
    mb, _ = enc.encode(bad)
    assert torch.equal(mb[:, :, 6:], m[:, :, 6:])
    assert torch.isfinite(m).all()
    enc.close()
