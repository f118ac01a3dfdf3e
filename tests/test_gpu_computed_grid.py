"""A call computes each clip's span in as few windows as it can where the grid does not change a row.  The debug tap makes it compute the
caller's own windows, and so does a test aid that leaves streams and kernels as they are: the same bits, over window lengths from one frame to more than the clip, halos of the receptive field and more,
spans inside the clip and at its edges, one and several clips, sizes on both sides of the cut into two windows, every entry point.  With
less than the receptive field the windows are the caller's with and without the tap."""
import numpy as np
import pytest
import torch

import demon_inputs as di
import oracle
from gpu_util import TOL, errors, make, to_device
from paper_2605_28657_amd import DemonError, DemonVAEEncoder, DEMON_ERR_WORKSPACE

pytestmark = pytest.mark.gpu

STACKS = {"narrow": di.DecoderSpec(64, (4, 2), (128, 64)), "wide": di.DecoderSpec(64, (2, 2), (512, 256), (1, 3)),
          "staged": di.DecoderSpec(32, (4, 2), (96, 32), (1, 3)),
          # enough work for the cut: 0.63 and, with LDS-staged convolutions, 0.43 GFLOP a frame
          "deep": di.DecoderSpec(64, (8, 6, 4, 4), (512, 256, 128, 64)), "deep staged": di.DecoderSpec(32, (8, 6, 4, 4), (512, 256, 96, 32)), "full": di.FULL}
# clips, frames, begin, end, window
SPANS = [(1, 130, 0, 130, 1), (1, 130, 0, 130, 37), (1, 130, 5, 117, 16), (3, 90, 11, 90, 64), (2, 75, 0, 75, 500), (1, 700, 0, 700, 64), (1, 700, 0, 700, 700),
         (1, 900, 3, 881, 130), (3, 300, 0, 299, 50), (4, 200, 0, 200, 9)]


ALL = [(stack, *s) for stack in ("narrow", "wide", "staged") for s in SPANS]
LONG = [(stack, *s) for stack in ("deep", "deep staged") for s in SPANS if s[3] - s[2] > 250] + [("deep staged", 3, 340, 3, 339, 50), ("deep staged", 1, 1020, 0, 1017, 130)]


def held(spec, clips, T, fb, fe, window):
    """Extended frames of the caller's grid with the largest halo asked for."""
    return clips * max(T, -(-(fe - fb) // window) * (min(window, fe - fb) + 2 * (max(oracle.receptive_field(spec)) + 8)))


def both(handle, decode):
    """(the caller's windows, what a call computes)"""
    scratch = torch.zeros(1, device="cuda:0")
    handle.tap(0, scratch)
    ref = decode()
    handle.tap(-1)
    handle.callers_grid(True)
    assert torch.equal(decode(), ref)
    handle.callers_grid(False)
    return ref, decode()


@pytest.mark.parametrize("dtype,kw,stack,clips,T,fb,fe,window",
                         [(dt, kw, *c) for dt, kw in (("bf16", {}), ("bf16", dict(wide_operands=2)), ("f32", {})) for c in ALL + (LONG if dt == "bf16" else [])])
def test_decode(stack, clips, T, fb, fe, window, dtype, kw):
    spec = STACKS[stack]
    vae, _, z = make(spec, dtype, T, n_clips=clips, max_extended_frames=held(spec, clips, T, fb, fe, window), **kw)
    zt = to_device(z, dtype)
    rf = max(vae.receptive_field())
    S = spec.total_stride
    whole = vae.decode(zt)
    for halo in (-1, rf, rf + 7, rf - 1, 0):
        def run(decode=vae.decode_windowed, dt=torch.float32):
            out = torch.full((clips, spec.out_channels, T * S), 7.0, device="cuda:0")
            return decode(zt, out=out, window=window, halo=halo, frame_begin=fb, frame_end=fe)
        ref, got = both(vae, run)
        assert torch.equal(got, ref), f"halo {halo}"
        assert (got[:, :, :fb * S] == 7).all() and (got[:, :, fe * S:] == 7).all()
        if halo == -1 or halo >= rf or (fb == 0 and fe == T and window >= T):
            assert torch.equal(got[:, :, fb * S:fe * S], whole[:, :, fb * S:fe * S])
        elif window < fe - fb:
            assert not torch.equal(got[:, :, fb * S:fe * S], whole[:, :, fb * S:fe * S])
    args = dict(window=window, halo=-1, frame_begin=fb, frame_end=fe)
    pcm = both(vae, lambda: vae.decode_windowed_pcm16(zt, **args)[:, fb * S:fe * S].clone())
    assert torch.equal(*pcm)
    skip = torch.tensor([0, 1, 0, 1][:clips], dtype=torch.int32, device="cuda:0")
    gated = both(vae, lambda: vae.decode_windowed_gated(zt, skip, torch.full((clips, spec.out_channels, T * S), 7.0, device="cuda:0"), **args))
    assert torch.equal(*gated)
    try:
        static = both(vae, lambda: vae.decode_windowed_static(zt, out=torch.zeros((clips, spec.out_channels, T * S), device="cuda:0"), **args).clone())
    except DemonError as e:
        assert e.status == DEMON_ERR_WORKSPACE
    else:
        assert torch.equal(*static)
    vae.close()


@pytest.mark.parametrize("dtype,stack,clips,T,fb,fe,window", [("bf16", *c) for c in ALL + LONG] + [("f32", *c) for c in ALL])
def test_encode(stack, clips, T, fb, fe, window, dtype):
    spec = STACKS[stack]
    w = di.make_encoder_weights(spec, bf16=dtype == "bf16")
    enc = DemonVAEEncoder(spec, w, dtype=dtype, max_frames=T, max_clips=clips, max_extended_frames=held(spec, clips, T, fb, fe, window))
    x = torch.from_numpy(np.stack([di.make_waveform(spec.out_channels, T * spec.total_stride, 40 + c) for c in range(clips)])).to("cuda:0")
    rf = max(enc.receptive_field())
    whole, _ = enc.encode(x)
    for halo in (-1, rf + 3, rf - 1):
        ref, got = both(enc, lambda: enc.encode_windowed(x, window=window, halo=halo, frame_begin=fb, frame_end=fe)[0][:, :, fb:fe].clone())
        assert torch.equal(got, ref), f"halo {halo}"
        if halo != rf - 1:
            assert torch.equal(got, whole[:, :, fb:fe])
    enc.close()


@pytest.mark.parametrize("stack,encode,clips,T,windows", [
    ("full", False, 1, 419, 1), ("full", False, 1, 420, 2),                                                          # frames of one clip
    ("deep", False, 1, 682, 1), ("deep", False, 1, 683, 2), ("deep", True, 1, 681, 1), ("deep", True, 1, 682, 2),    # 430 GFLOP of a call
    ("deep", False, 3, 299, 3), ("deep", False, 3, 300, 6), ("deep", True, 3, 419, 3), ("deep", True, 3, 420, 6),    # frames of several
    ("deep", False, 5, 150, 5), ("deep", True, 7, 200, 7), ("deep", False, 2, 500, 2), ("deep", True, 4, 500, 4),
    ("deep staged", False, 1, 1003, 1), ("deep staged", False, 1, 1004, 2), ("deep staged", True, 1, 1002, 1), ("deep staged", True, 1, 1003, 2),
    ("deep staged", False, 3, 334, 3), ("deep staged", False, 3, 335, 6), ("deep staged", True, 3, 720, 3),
    ("narrow", False, 1, 2000, 1), ("narrow", False, 3, 700, 3), ("narrow", True, 1, 700, 1)])
def test_calls_that_cut_their_clips(stack, encode, clips, T, windows):
    """Every clip in two windows only where that is the faster side: the joins of many short clips cost more than equal groups give, and two groups
    are twice the launches, which little work does not cover."""
    spec = STACKS[stack]
    if encode:
        vae = DemonVAEEncoder(spec, di.make_encoder_weights(spec, bf16=True), dtype="bf16", max_frames=T, max_clips=clips)
        x = torch.zeros((clips, spec.out_channels, T * spec.total_stride), device="cuda:0")
        vae.encode(x)
    else:
        vae, _, z = make(spec, "bf16", T, n_clips=clips)
        vae.decode(to_device(z, "bf16"))
    rf = max(vae.receptive_field())
    frames = clips * T + (windows - clips) * 2 * rf
    assert vae.last_grid() == (windows, frames, 2 if windows > 1 else 1)
    vae.close()


@pytest.mark.parametrize("clips,T", [(1, 700), (3, 350)])
def test_gated_calls_cut_no_clip(clips, T):
    """A gated call runs as one group of windows, for which nothing is cut.  16 grids can be recorded whether or not calls on them are gated, and
    a gated call on a recorded grid takes that one where no entry of the window tables is left."""
    spec = STACKS["deep"]
    vae, _, z = make(spec, "bf16", T, n_clips=clips, max_extended_frames=3 * T * clips)
    zt = to_device(z, "bf16")
    S = spec.total_stride
    ref = vae.decode_windowed(zt, window=64)
    assert vae.last_grid()[0] == 2 * clips
    skip = torch.tensor([0, 1, 0][:clips], dtype=torch.int32, device="cuda:0")
    def gated(fe):
        out = torch.full_like(ref, 7.0)
        vae.decode_windowed_gated(zt, skip, out, window=64, frame_end=fe)
        for c in range(clips):
            assert (out[c] == 7).all() if skip[c] else torch.equal(out[c, :, :fe * S], ref[c, :, :fe * S])
    gated(T)
    assert vae.last_grid() == (clips, clips * T, 1)
    vae.close()
    # 16 recorded grids: no entry is left
    vae, _, _ = make(spec, "bf16", T, n_clips=clips, max_extended_frames=3 * T * clips)
    graphs, out = [], torch.zeros_like(ref)
    for i in range(16):
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            vae.decode_windowed(zt, out=out, window=64, frame_end=T - i)
        graphs.append(torch.cuda.CUDAGraph())
        with torch.cuda.graph(graphs[-1]):
            vae.decode_windowed_gated(zt, skip, out, window=64, frame_end=T - i)
    for i in (0, 15, 15):
        gated(T - i)
        assert vae.last_grid()[0] == 2 * clips
        out.zero_()
        graphs[2 * i].replay()
        torch.cuda.synchronize()
        assert torch.equal(out[:, :, :(T - i) * S], ref[:, :, :(T - i) * S])
        out.fill_(7.0)
        graphs[2 * i + 1].replay()
        torch.cuda.synchronize()
        for c in range(clips):
            assert (out[c] == 7).all() if skip[c] else torch.equal(out[c, :, :(T - i) * S], ref[c, :, :(T - i) * S])
    with pytest.raises(DemonError) as e:
        vae.decode_windowed_gated(zt, skip, out, window=65)
    assert e.value.status == DEMON_ERR_WORKSPACE
    vae.close()


def test_the_limits_are_those_of_the_callers_grid():
    spec, T = STACKS["deep"], 700
    rf = max(oracle.receptive_field(spec))
    tight, _, z = make(spec, "bf16", T, max_extended_frames=T)
    zt = to_device(z, "bf16")
    full = tight.decode(zt)                                  # one window: a cut one would need 2 rf frames more than are held
    with pytest.raises(DemonError) as e:
        tight.decode_windowed(zt, window=100, halo=-1)       # 6 joins of 2 rf frames
    assert e.value.status == DEMON_ERR_WORKSPACE
    roomy, w, _ = make(spec, "bf16", T, max_extended_frames=T + 2 * rf)
    assert tight.last_grid()[0] == 1
    assert torch.equal(roomy.decode(zt), full)               # cut in two
    assert roomy.last_grid()[0] == 2
    S = spec.total_stride
    ref = oracle.decode_windowed(spec, w, z[0], window=6, halo=rf, frame_begin=347, frame_end=353)       # around the cut
    ma, rl = errors(full[0, :, 347 * S:353 * S].cpu().numpy(), ref)
    assert ma <= TOL["bf16"][0] and rl <= TOL["bf16"][1]
    tight.close(); roomy.close()


def test_replay_with_and_without_the_tap():
    """A recorded grid keeps its table: the caller's windows and the computed ones are two entries."""
    spec, T = STACKS["deep"], 700
    vae, _, z = make(spec, "bf16", T, max_extended_frames=4 * T)
    zt = to_device(z, "bf16")
    out = torch.zeros((1, 2, T * spec.total_stride), device="cuda:0")
    ref = vae.decode(zt)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        vae.decode_windowed(zt, out=out, window=50, halo=-1)
    assert vae.last_grid()[0] == 2
    for _ in range(3):
        out.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        a, b = both(vae, lambda: vae.decode_windowed(zt, window=50, halo=-1))
        assert torch.equal(a, ref) and torch.equal(b, ref)
    vae.close()
