"""The head inside the last unit's kernel at its two tiles (128 and 256 columns, of which the head's k - 1 rows of context come off), on both
sides of the rule between them and at lengths that end inside a tile: the bits of the head kernel, for every kernel size and dilation
of the unit."""
import pytest
import torch

import demon_inputs as di
import paper_2605_28657_amd as pa
from gpu_util import make, to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T", [1, 61, 140000, 150001, 300007])          # 2 T rows; up to 2304 tiles of 122 columns, more
@pytest.mark.parametrize("k,oc,dils", [(7, 2, (1, 3, 9)), (1, 1, (3,)), (5, 3, (9, 1))])
def test_head_tiles(T, k, oc, dils):
    spec = di.DecoderSpec(64, (2,), (64,), dils, head_kernel=k, out_channels=oc)
    vae, w, z = make(spec, "bf16", T, max_extended_frames=T + 200)
    other = pa.DemonVAE(spec, w, dtype="bf16", max_frames=T, max_extended_frames=T + 200, flags=pa.DEMON_VAE_FLAG_NO_HEAD_FUSION)
    zt = to_device(z, "bf16")
    got = vae.decode(zt)
    assert torch.equal(got, other.decode(zt)) and got.abs().max() > 0
    n = T - T // 3
    args = dict(window=n, halo=-1, frame_begin=T - n, frame_end=T)
    out = torch.full_like(got, 7.0)
    assert torch.equal(vae.decode_windowed(zt, out=out, **args)[:, :, 2 * (T - n):], got[:, :, 2 * (T - n):])
    assert (out[:, :, :2 * (T - n)] == 7).all()
    vae.close(); other.close()
