"""The bf16 convolutions that stream their weights: every tile the launch can choose (the choice follows the size of the call
only), remainders of columns at every tile, both operand formats, one- and two-plane operands, taps unrolled and counted at
run time.  Every tile adds in the same order, so a handle restricted to the largest tile gives the same bits."""
import numpy as np
import pytest
import torch

import demon_inputs as di
import oracle
from gpu_util import assert_close, make, to_device
import paper_2605_28657_amd as pa
from paper_2605_28657_amd import DemonVAE, DemonVAEEncoder

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("grid")]


@pytest.mark.parametrize("spec,T,kw", [
    (di.DecoderSpec(64, (2,), (512,), (1, 3, 9)), 1, {}),                            # one frame: two columns
    (di.DecoderSpec(64, (2,), (512,), (1, 3, 9)), 257, {}),                          # 32-row tiles, half operands
    (di.DecoderSpec(64, (2, 2), (512, 256), (3, 9)), 501, dict(flags=1)),            # 64 x 64 / 80 / 96, unfused 256 channels
    (di.DecoderSpec(64, (2, 2), (512, 128), (1, 9)), 3001, dict(flags=1)),           # up to the 128 x 128 tile in one call
    (di.DecoderSpec(64, (2, 2), (512, 128), (9,)), 129, dict(wide_operands=2)),      # hi + lo operand planes
    (di.DecoderSpec(64, (2, 2), (512, 128), (1, 3), res_kernel=5), 130, dict(flags=1)),      # five taps
])
def test_stream_tiles(spec, T, kw):
    vae, w, z = make(spec, "bf16", T, max_extended_frames=T, **kw)
    large = DemonVAE(spec, w, dtype="bf16", max_frames=T, max_extended_frames=T, small_tile_wgs=-1, **kw)
    zt = to_device(z, "bf16")
    full = vae.decode(zt).cpu().numpy()
    assert np.array_equal(large.decode(zt).cpu().numpy(), full)
    n = min(T, 300)
    halo = max(oracle.receptive_field(spec))
    ref = oracle.decode_windowed(spec, w, z[0], window=n, halo=halo, frame_begin=0, frame_end=n)
    assert_close(full[0][:, :n * spec.total_stride], ref[:, :n * spec.total_stride], "bf16", str(spec))
    vae.close(); large.close()


@pytest.mark.parametrize("widths,T", [((512, 256), 97), ((512, 256), 1601), ((512, 256), 9001),      # 64 x 64; 128 x 64; more than 1024 tiles
                                      ((256, 128), 16401), ((256, 64), 3001)])                          # 256 merged channels; one chunk
def test_strided_tiles(widths, T):
    """The encoder's strided convolutions at their tiles: the same bits as on the 128 x 128 tile."""
    spec = di.DecoderSpec(64, (4, 4 if widths[1] > 64 else 2), widths, (1,))
    w = di.make_encoder_weights(spec, bf16=True)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(T)
    wave = (torch.randn(1, spec.out_channels, T * spec.total_stride, generator=g, device="cuda:0") * 0.25).clamp_(-1.0, 1.0)
    got = []
    for wgs in (0, -1):
        enc = DemonVAEEncoder(spec, w, dtype="bf16", max_frames=T, max_extended_frames=T, small_tile_wgs=wgs)
        got.append(enc.encode_windowed(wave, window=T)[0])
        enc.close()
    assert got[0].abs().max() > 0 and torch.equal(got[0], got[1])


@pytest.mark.parametrize("T,dils", [
    (1, (1, 3, 9)), (17, (1, 3, 9)),         # less than a tile, a remainder
    (4090, (9,)), (4099, (1, 9)),            # 32 columns at 256 tiles; 64 columns
    (8197, (1, 9)), (10241, (1, 9)),         # 80 and 96 columns
    (12299, (1, 3, 9)), (16385, (1, 9)),     # 128 columns, more than 256 tiles
])
def test_unit_256_stream_tiles(T, dils):
    """The 256-channel unit at every tile a launch can take: the same bits as the LDS-staged kernel, also window by window."""
    spec = di.DecoderSpec(64, (2,), (256,), dils)
    vae, w, z = make(spec, "bf16", T, max_extended_frames=2 * T + 64)
    staged = DemonVAE(spec, w, dtype="bf16", max_frames=T, max_extended_frames=2 * T + 64, small_tile_wgs=-1)
    zt = to_device(z, "bf16")
    full = vae.decode(zt).cpu().numpy()
    assert np.array_equal(staged.decode(zt).cpu().numpy(), full)
    assert np.array_equal(vae.decode_windowed(zt, window=max(1, T // 3), halo=-1).cpu().numpy(), full)
    n = min(T, 300)
    ref = oracle.decode_windowed(spec, w, z[0], window=n, halo=max(oracle.receptive_field(spec)), frame_begin=0, frame_end=n)
    assert_close(full[0][:, :n * spec.total_stride], ref[:, :n * spec.total_stride], "bf16", str(spec))
    vae.close(); staged.close()


@pytest.mark.parametrize("c,T,window", [
    (512, 32700, 16101),                     # the dilated convolutions' 256 x 128 tile
    (256, 4200, 37), (256, 13000, 6001),     # many ragged windows, two long ones: more tiles than the narrow kernel takes
    (128, 9000, 119), (128, 45000, 20001),   # 64 columns a workgroup; 256
    (64, 3001, 64), (64, 150001, 60000), (64, 530000, 300000),      # 128 columns (with the head in the short window); 256
])
def test_units_of_large_calls_window_by_window(c, T, window, grid):
    """The residual units' kernels for launches that fill the chip, on windows whose ends fall inside a tile: the same bits as the whole clip,
    and as a window short enough for the kernel of few tiles."""
    spec = di.DecoderSpec(64, (2,), (c,), (1, 3, 9))
    halo = max(oracle.receptive_field(spec))
    vae, w, z = make(spec, "bf16", T, max_extended_frames=T + (T // window + 1) * 2 * halo)
    zt = to_device(z, "bf16")
    full = vae.decode_windowed(zt, window=T, halo=-1)
    assert torch.equal(vae.decode_windowed(zt, window=window, halo=-1), full)
    assert vae.last_grid()[0] == (-(-T // window) if grid == "callers" else 2 if c == 512 else 1)
    out = vae.decode_windowed(zt, window=15, halo=-1, frame_begin=T // 2, frame_end=T // 2 + 15)
    S = spec.total_stride
    assert torch.equal(out[:, :, T // 2 * S:(T // 2 + 15) * S], full[:, :, T // 2 * S:(T // 2 + 15) * S])
    ref = oracle.decode_windowed(spec, w, z[0], window=60, halo=halo, frame_begin=T - 60, frame_end=T)
    assert_close(full[0].cpu().numpy()[:, (T - 60) * S:], ref[:, -60 * S:], "bf16", f"{c} channels")
    vae.close()


def test_two_planes_give_the_same_bits_at_every_size_of_call():
    """Two operand planes: a clip whose 1x1 and transposed convolutions take the largest tile, and windows of it that take the
    smallest; a value may not depend on which."""
    spec, T = di.DecoderSpec(64, (2, 2), (512, 512), (9,)), 4300
    vae, w, z = make(spec, "bf16", T, max_extended_frames=T + 200, wide_operands=2)
    zt = to_device(z, "bf16")
    full = vae.decode(zt)
    S = spec.total_stride
    for begin, n in ((0, 7), (2000, 61), (3900, 400)):
        out = vae.decode_windowed(zt, window=n, halo=-1, frame_begin=begin, frame_end=begin + n)
        assert torch.equal(out[:, :, begin * S:(begin + n) * S], full[:, :, begin * S:(begin + n) * S]), (begin, n)
    vae.close()


def test_tall_tile_on_bf16_operands():
    """A 256-channel unit on its two-kernel path in more than 512 tiles of 256 x 128: bf16 operands on the tall tile at every span, on
    windows whose ends fall inside a tile, against a window short enough for a small tile and the oracle."""
    spec, T = di.DecoderSpec(64, (2,), (256,), (1, 3, 9)), 33100
    vae, w, z = make(spec, "bf16", T, max_extended_frames=2 * T, flags=pa.DEMON_VAE_FLAG_NO_FUSED)
    zt = to_device(z, "bf16")
    full = vae.decode(zt)
    assert torch.equal(vae.decode_windowed(zt, window=16901, halo=-1), full)
    for begin in (0, 20011, T - 15):
        out = vae.decode_windowed(zt, window=15, halo=-1, frame_begin=begin, frame_end=begin + 15)
        assert torch.equal(out[:, :, 2 * begin:2 * begin + 30], full[:, :, 2 * begin:2 * begin + 30])
    ref = oracle.decode_windowed(spec, w, z[0], window=60, halo=max(oracle.receptive_field(spec)), frame_begin=T - 60, frame_end=T)
    assert_close(full[0].cpu().numpy()[:, -120:], ref[:, -120:], "bf16", "256 channels, unfused")
    vae.close()
