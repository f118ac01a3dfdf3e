"""The fp32 convolutions: every tile the launch can choose, channel counts that do not tile, and taps that span more rows
than the activation tile holds.  The tile depends on the size of the call only, and every tile adds in the same order."""
import numpy as np
import pytest

import demon_inputs as di
import oracle
from gpu_util import assert_close, make, to_device

pytestmark = pytest.mark.gpu


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
