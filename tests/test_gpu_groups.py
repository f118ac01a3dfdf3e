"""Calls of many frames run as two groups of windows on two streams (bf16 path): the same bits as on one stream, for stacks whose
widest level is first, last or in between (the second group's region of a buffer starts at another row at every level), for
several clips, two operand planes and LDS-staged tiles, for the gated decode (one group) and replayed from a graph; on the windows that calls
compute and on the caller's, with a halo of the receptive field and a shorter one."""
import numpy as np
import pytest
import torch

import demon_inputs as di
import paper_2605_28657_amd as pa
from gpu_util import make, to_device

pytestmark = [pytest.mark.gpu, pytest.mark.usefixtures("grid")]


@pytest.mark.parametrize("spec,T,window,clips,kw", [
    (di.DecoderSpec(64, (4, 2), (128, 64)), 700, 90, 1, {}),                    # widest at the output
    (di.DecoderSpec(64, (2, 2), (512, 64), (1, 3)), 430, 429, 1, {}),           # widest in between; a second window of one frame
    (di.DecoderSpec(256, (2,), (64,), (1, 9)), 400, 150, 2, {}),                # widest at the latent
    (di.DecoderSpec(64, (2, 2), (512, 128), (1,)), 161, 40, 3, dict(wide_operands=2)),      # the caller's windows: the cut inside a clip
    (di.DecoderSpec(64, (4, 2), (128, 64)), 310, 64, 3, {}),                    # so here
    (di.DecoderSpec(32, (4, 2), (96, 32)), 240, 37, 1, {}),                     # LDS-staged tiles
    (di.DecoderSpec(64, (4, 2), (96, 64), (1, 3)), 230, 60, 1, {}),             # LDS-staged tiles, the head inside the last unit
    (di.DecoderSpec(64, (8, 6, 4, 4), (512, 256, 128, 64)), 690, 64, 1, {}),    # one clip, cut in two
    (di.DecoderSpec(32, (8, 6, 4, 4), (512, 256, 96, 32)), 1010, 90, 1, {}),     # so, LDS-staged tiles
])
def test_two_groups_equal_one_stream(spec, T, window, clips, kw, grid):
    vae, w, z = make(spec, "bf16", T, n_clips=clips, max_extended_frames=8 * T * clips, **kw)
    one = pa.DemonVAE(spec, w, dtype="bf16", max_frames=T, max_clips=clips, max_extended_frames=8 * T * clips,
                      flags=pa.DEMON_VAE_FLAG_ONE_STREAM, **kw)
    zt = to_device(z, "bf16")
    def grid_of(v, halo, groups):
        """The call ran in so many groups, on the grid this test is about."""
        n, _, g = v.last_grid()
        if grid == "callers" or halo != -1:
            assert n == clips * -(-T // window)
        elif v is vae:
            assert n == (2 if cut else clips)
        assert g == (groups if n > 1 else 1)
    cut = spec.total_stride > 100                # one clip of little work stays one window, which is one group
    ref = one.decode_windowed(zt, window=window, halo=-1)
    grid_of(one, -1, 1)
    for _ in range(3):
        assert torch.equal(vae.decode_windowed(zt, window=window, halo=-1), ref)
        grid_of(vae, -1, 2)
    assert torch.equal(vae.decode(zt), ref)
    # less than the receptive field: the rows depend on the windows, which are the caller's
    short = max(vae.receptive_field()) - 1
    other = one.decode_windowed(zt, window=window, halo=short)
    assert not torch.equal(other, ref)
    assert torch.equal(vae.decode_windowed(zt, window=window, halo=short), other)
    grid_of(vae, short, 2)
    # gated: the skipped clips keep what the buffer holds, the others are decoded as above
    skip = torch.tensor([1, 0, 1][:clips], dtype=torch.int32, device="cuda:0")
    out = torch.full_like(ref, 7.0)
    vae.decode_windowed_gated(zt, skip, out, window=window, halo=-1)
    assert vae.last_grid()[2] == 1
    for c in range(clips):
        assert torch.equal(out[c], torch.full_like(ref[c], 7.0) if skip[c] else ref[c])
    # recorded: the fork and the join are part of the graph
    out.zero_()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        vae.decode_windowed(zt, out=out, window=window, halo=-1)
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        assert torch.equal(vae.decode_windowed(zt, window=window, halo=-1), ref)         # eager work between the replays
    vae.close(); one.close()


@pytest.mark.parametrize("spec,T,clips", [(di.DecoderSpec(64, (4, 2), (128, 64)), 250, 2), (di.DecoderSpec(64, (8, 6, 4, 4), (512, 256, 128, 64)), 690, 1),
                                          (di.DecoderSpec(64, (32,), (64,)), 250, 2)])          # the last convolution's K in parts
@pytest.mark.parametrize("short", [0, 1])
def test_encode_in_two_groups_equals_one_stream(spec, T, clips, short):
    w = di.make_encoder_weights(spec, bf16=True)
    x = torch.from_numpy(np.stack([di.make_waveform(2, T * spec.total_stride, 40 + c) for c in range(clips)])).to("cuda:0")
    got = []
    for flags in (0, pa.DEMON_VAE_FLAG_ONE_STREAM):
        enc = pa.DemonVAEEncoder(spec, w, dtype="bf16", max_frames=T, max_clips=clips, max_extended_frames=3 * T * clips, flags=flags)
        halo = max(enc.receptive_field()) - short
        got.append(enc.encode_windowed(x, window=60, halo=halo))
        torch.cuda.synchronize()
        assert enc.last_grid()[2] == (1 if flags else 2)
        enc.close()
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
