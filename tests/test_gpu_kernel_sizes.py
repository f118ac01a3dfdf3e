"""Dilated convolutions of every kernel size on the streamed kernel (the taps are counted at run time for sizes other than 7):
sizes from one tap to the largest span, fewer blocks than the ring of requests holds, remainders of the ring, both operand formats,
calls from one column to the largest tile."""
import numpy as np
import pytest

import demon_inputs as di
import oracle
from gpu_util import assert_close, make, to_device
from paper_2605_28657_amd import DemonVAE

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("k,dils,width", [(1, (1, 5), 128), (3, (1, 9), 128), (3, (32,), 512), (5, (1, 3, 16), 512), (9, (1, 8), 128), (9, (2,), 640),
                                          (11, (1, 6), 512), (13, (5,), 256), (15, (4,), 384), (33, (2,), 128), (65, (1,), 128)])
@pytest.mark.parametrize("T", [1, 150, 2500])
def test_kernel_sizes(k, dils, width, T):
    spec = di.DecoderSpec(64, (2,), (width,), dils, res_kernel=k)
    kw = dict(flags=1, max_extended_frames=2 * T + 200)                 # no fused units
    vae, w, z = make(spec, "bf16", T, **kw)
    large = DemonVAE(spec, w, dtype="bf16", max_frames=T, small_tile_wgs=-1, **kw)
    zt = to_device(z, "bf16")
    full = vae.decode(zt).cpu().numpy()
    assert np.array_equal(large.decode(zt).cpu().numpy(), full)
    n = min(T, 40)
    assert np.array_equal(vae.decode_windowed(zt, window=n, halo=-1, frame_begin=T - n, frame_end=T).cpu().numpy()[:, :, -2 * n:], full[:, :, -2 * n:])
    ref = oracle.decode_windowed(spec, w, z[0], window=n, halo=max(oracle.receptive_field(spec)), frame_begin=0, frame_end=n)
    assert_close(full[0][:, :2 * n], ref[:, :2 * n], "bf16", f"kernel size {k}")
    vae.close(); large.close()


@pytest.mark.parametrize("width", [64, 128, 256, 512])
@pytest.mark.parametrize("T", [301, 45001])                             # launches of few tiles, and of those that fill the chip
def test_taps_of_zeros_change_no_bit(width, T):
    """Seven taps, and the same seven between two of zeros, which run on other kernels (staged weights, taps counted at run time): a zero
    product leaves a sum as it is, so that the results are the same bits if all kernels add in the same order."""
    seven, nine = (di.DecoderSpec(64, (2,), (width,), (1, 3, 6), res_kernel=k) for k in (7, 9))
    vae, w, z = make(seven, "bf16", T, max_extended_frames=T)
    w9 = np.zeros(di.n_weights(nine), np.float32)
    padded = di.split_weights(nine, w9)
    for name, v in di.split_weights(seven, w).items():
        (padded[name][..., 1:8] if name.endswith("c1.weight") else padded[name])[...] = v
    other = DemonVAE(nine, w9, dtype="bf16", max_frames=T, max_extended_frames=T)
    zt = to_device(z, "bf16")
    got = vae.decode(zt).cpu().numpy()
    assert np.abs(got).max() > 0 and np.array_equal(got, other.decode(zt).cpu().numpy())
    vae.close(); other.close()
