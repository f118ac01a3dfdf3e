"""The fp32 convolutions: every tile the launch can choose, channel counts that do not tile, and taps that span more rows
than the activation tile holds.  The tile depends on the size of the call only, and every tile adds in the same order."""
import numpy as np
import pytest

import demon_inputs as di
import oracle
import paper_2605_28657_amd as pa
from gpu_util import assert_close, make, to_device

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("grid")]


@pytest.mark.parametrize("spec,T,window", [
    (di.DecoderSpec(16, (2,), (256,), (1, 3)), 1, 1),                 # one frame
    (di.DecoderSpec(48, (2,), (144,), (1, 9)), 65, 16),               # half a 32-channel chunk, a ragged row tile
    (di.DecoderSpec(64, (4, 2), (256, 32), (1, 3)), 900, 301),        # 128 x 128 and 32 x 128 tiles in the full decode
    (di.DecoderSpec(12, (4, 2), (24, 10), (1, 3)), 20, 7),            # no whole tiles: the plain kernel
    (di.DecoderSpec(16, (2,), (16,), (120,)), 150, 40),               # taps spanning 720 rows: the plain kernel on tile-packed weights
])
def test_f32_tiles(spec, T, window):
    halo = max(oracle.receptive_field(spec))
    vae, w, z = make(spec, "f32", T, snake="uniform", max_extended_frames=(T + 2 * halo) * (T // window + 2))
    zt = to_device(z, "f32")
    full = vae.decode(zt).cpu().numpy()
    assert_close(full, oracle.decode(spec, w, z), "f32", str(spec))
    assert np.array_equal(vae.decode_windowed(zt, window=window, halo=-1).cpu().numpy(), full)
    vae.close()


@pytest.mark.parametrize("spec,T,window", [
    (di.DecoderSpec(16, (2,), (64,), (1, 9)), 1, 1),                  # one frame: two columns of one tile
    (di.DecoderSpec(16, (2, 2), (64, 32), (1, 3, 9)), 37, 9),         # short windows, ragged column tiles
    (di.DecoderSpec(16, (4, 2), (96, 32), (9,)), 4000, 1200),         # two column tiles a wave, 96 rows in tiles of 32
    (di.DecoderSpec(16, (4, 2), (32, 64), (1, 9)), 6000, 2500),       # three
])
def test_f32_units_in_one_kernel(spec, T, window):
    """A residual unit in one kernel adds in the order of its two convolutions on their own."""
    halo = max(oracle.receptive_field(spec))
    ext = (T + 2 * halo) * (T // window + 2)
    one, w, z = make(spec, "f32", T, snake="uniform", max_extended_frames=ext)
    two = pa.DemonVAE(spec, w, dtype="f32", max_frames=T, max_extended_frames=ext, flags=pa.DEMON_VAE_FLAG_NO_FUSED)
    zt = to_device(z, "f32")
    full = one.decode(zt).cpu().numpy()
    assert np.array_equal(full, two.decode(zt).cpu().numpy())
    assert np.array_equal(full, one.decode_windowed(zt, window=window, halo=-1).cpu().numpy())
    if T < 100:
        assert_close(full, oracle.decode(spec, w, z), "f32", str(spec))
    one.close()
    two.close()


@pytest.mark.parametrize("width,T", [(128, 100), (128, 210), (192, 700), (256, 210), (256, 310), (256, 520)])
def test_f32_column_tiles(width, T):
    """Launches that take 1, 2, 3, 4 and 6 column tiles a wave, against the oracle on their last rows and first."""
    spec = di.DecoderSpec(16, (10,), (width,), (1, 9))
    vae, w, z = make(spec, "f32", T, snake="uniform", max_extended_frames=2 * T)
    zt = to_device(z, "f32")
    full = vae.decode(zt).cpu().numpy()
    halo, n = max(oracle.receptive_field(spec)), 6
    for begin in (0, T - n):
        lo, hi = max(0, begin - halo), min(T, begin + n + halo)
        ref = oracle.decode(spec, w, z[:, :, lo:hi])
        assert_close(full[:, :, begin * 10:(begin + n) * 10], ref[:, :, (begin - lo) * 10:(begin - lo + n) * 10], "f32", f"{width} {T} {begin}")
    vae.close()
