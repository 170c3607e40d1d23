"""GPU parity of dc_run_stack (whole per-frame path) against the oracle: match results,
reuse masks and propagated rectangles bit-exact; every tensor within 1e-4 (fp32) or
2e-2 (bf16) of the oracle, relative to the tensor's largest magnitude."""
import ctypes
import threading

import numpy as np
import pytest
import torch

from paper_1712_01670_amd import binding, synth

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def _rel_err(got, want):
    scale = max(float(np.abs(want).max()), 1e-30)
    return float(np.abs(got - want).max()) / scale


def _elem_err(got, want):
    """Element-wise variant: |g - o| / max(|o|, 1e-3 * max|o|), the floor keeps values near zero from deciding."""
    scale = max(float(np.abs(want).max()), 1e-30)
    return float((np.abs(got - want) / np.maximum(np.abs(want), 1e-3 * scale)).max())


def _run_both(oracle, layers, videos, block, radius, bf16, in_place=False, device_plan=None, exact_masks=False, **kw):
    exact_masks = exact_masks or bool(kw.get("cache_pool_add"))
    if kw.get("torus"):      # torus frames are planned on the GPU
        device_plan = True
    """Every frame of every stream against the oracle, with the frame planned on the host and (unless in-place frames
    are asked for, which only the host plans) once more with the frame planned on the GPU."""
    modes = [False] if in_place else ([False, True] if device_plan is None else [bool(device_plan)])
    if exact_masks:          # exact reuse maps exist on the GPU only
        modes = [True]
    first = None
    for dp in modes:
        res = _run_one(oracle, layers, videos, block, radius, bf16, in_place=in_place, device_plan=dp, exact_masks=exact_masks, **kw)
        if first is None:
            first = res
        else:
            assert res[1] == first[1]
    return first


def _run_one(oracle, layers, videos, block, radius, bf16, expiry=0, seed=1, bias_scale=0.05,
             residual_scale=1.0, check_tensors=None, resets=(), diamond=False, k_skip=1, in_place=False,
             extend_borders=False, device_plan=False, exact_masks=False, cache_pool_add=False, no_reuse=None, torus=False):
    """videos: uint8 [n_streams][T][H][W][C].  Compares every frame of every stream."""
    n, T, H, W, C = videos.shape
    ws, bs = synth.he_weights(layers, seed, bias_scale=bias_scale, residual_scale=residual_scale, input_shape=(H, W, C))
    tol = 2e-2 if bf16 else 1e-4
    dt = binding.DC_BF16 if bf16 else binding.DC_F32
    runner = binding.StackRunner(layers, ws, bs, n, H, W, C, block=block, radius=radius, dtype=dt, expiry=expiry,
                                 want_regions=True, k_skip=k_skip, in_place=in_place, extend_borders=extend_borders,
                                 match_method=binding.DC_MATCH_DIAMOND if diamond else binding.DC_MATCH_EXHAUSTIVE,
                                 device_plan=device_plan, exact_masks=exact_masks, cache_pool_add=cache_pool_add, no_reuse=no_reuse,
                                 torus=torus, want_origins=torus)
    streams = [oracle.Stream(layers, ws, bs, H, W, C, block=block, radius=radius, bf16=bf16, expiry=expiry,
                             diamond=diamond, k_skip=k_skip, extend_borders=extend_borders, exact_masks=exact_masks,
                             cache_pool_add=cache_pool_add, no_reuse=no_reuse)
               for _ in range(n)]
    dev_video = torch.from_numpy(np.ascontiguousarray(videos.transpose(1, 0, 2, 3, 4))).to(DEV)
    worst = worst_elem = 0.0
    reuse = []
    runner.in_place_frames = []
    shapes = runner.shapes
    for t in range(T):
        print(f"[stack] frame {t}/{T} n={n} {H}x{W} bf16={bf16} planned on the {'GPU' if device_plan else 'host'}"
              f"{', exact reuse maps' if exact_masks else ''}", flush=True)
        if t in resets:
            runner.reset()
            for s in streams:
                s.reset()
        tensors = runner.step(dev_video[t])
        torch.cuda.synchronize()
        runner.in_place_frames.append(bool(runner.last_in_place))
        got = [x.float().cpu().numpy() for x in runner.logical_tensors(tensors)]
        blocks = needed = 0
        for s in range(n):
            want = streams[s].step(videos[s, t])
            assert bool(runner.last_full) == bool(want["full"])
            if not want["full"]:
                m = want["match"]
                assert np.array_equal(runner.mv[s].cpu().numpy(), m["mv"])
                assert np.array_equal(runner.best_ssd[s].cpu().numpy().view(np.uint32), m["best_ssd"])
                assert runner.gmv[s].cpu().numpy().tolist() == m["gmv"].tolist()
                assert int(runner.n_pass[s]) == m["n_pass"]
                assert np.array_equal(runner.mask[s].cpu().numpy(), m["mask"])
                regs = runner.regions(s)
                for ti in range(len(layers) + 1):
                    if exact_masks:              # no rectangle lists in this mode; the maps are checked by the counters below
                        assert len(regs[ti]["rects"]) == 0
                        continue
                    assert regs[ti]["rects"].tolist() == want["rects"][ti].tolist(), (t, s, ti)
                    assert list(regs[ti]["dxy"]) == want["dxy"][ti].tolist()
                reuse.append(float(m["mask"].mean()))
                blocks += int(m["mask"].sum())
                for li, L in enumerate(layers):
                    if L["type"] == synth.CONV:
                        ho, wo, _ = shapes[li + 1]
                        reused = (int(want["masks"][li + 1].sum()) if exact_masks else
                                  int(sum(int(r[2]) * int(r[3]) for r in want["rects"][li + 1])))
                        if no_reuse is not None and no_reuse[li]:
                            reused = 0
                        kh, kw = synth.conv_geometry(L)[:2]
                        needed += (ho * wo - reused) * kh * kw * runner.layers[li]["cin"] * L["cout"]
            for ti in (check_tensors or range(len(layers) + 1)):
                g = got[ti][s]
                if ti == 0:          # tensor 0 may carry zero padding channels
                    assert not g[..., C:].any()
                    g = g[..., :C]
                e = _rel_err(g, want["tensors"][ti])
                worst = max(worst, e)
                worst_elem = max(worst_elem, _elem_err(g, want["tensors"][ti]))
                assert e <= tol, (t, s, ti, e)
        if not runner.last_full:     # the library's work counters against the oracle's masks and rectangles
            st = runner.read_stats()
            assert st.n_reusable_blocks == blocks and st.n_overflow_streams == 0
            assert st.macs_needed == needed and st.macs_issued >= st.macs_needed
    print(f"[stack] worst error relative to the tensor's largest magnitude {worst:.3e} (bound {tol:g}); element-wise "
          f"with floor 1e-3 of that magnitude {worst_elem:.3e}; mean block reuse {np.mean(reuse) if reuse else 0:.3f}", flush=True)
    return runner, reuse


@pytest.mark.parametrize("bf16", [False, True])
def test_tiny_config(oracle, bf16):
    f1, f2 = synth.tiny_pair(0)
    video = np.stack([f1, f2, f2, f1])[None]
    runner, reuse = _run_both(oracle, synth.tiny_net(), video, 8, 8, bf16)
    assert abs(reuse[0] - 45 / 64) < 1e-9
    assert reuse[1] == 1.0


def test_tiny_exact_shift_equals_full_forward_on_gpu(oracle):
    # the invariant of the oracle also holds for the HIP path: with an exact shift by a multiple of
    # the total stride the cached frame reproduces the full forward (copies are bit copies; recomputed
    # pixels go through the same kernel)
    layers = synth.tiny_net()
    f1, f2 = synth.shifted_pair(10, 64, 64, (4, -2))
    ws, bs = synth.he_weights(layers, 1, bias_scale=0.05)
    r = binding.StackRunner(layers, ws, bs, 1, 64, 64, 3, block=8, radius=8)
    d1, d2 = torch.from_numpy(f1[None]).to(DEV), torch.from_numpy(f2[None]).to(DEV)
    r.step(d1)
    cached = [t.clone() for t in r.step(d2)]
    torch.cuda.synchronize()
    assert r.read_stats().n_reusable_blocks >= 40
    r.reset()
    full = r.step(d2)
    for a, b in zip(cached, full):
        assert torch.equal(a, b)


def test_vgg16_224_first_frames(oracle):
    video = synth.panning_video(2000, n_frames=3)[None]
    _run_both(oracle, synth.vgg16(), video, 16, 16, False, bias_scale=0.0)


@pytest.mark.parametrize("k_skip", [1, 2])
def test_diamond_search_in_the_whole_path(oracle, k_skip):
    # the paper's matcher (diamond search, k-skip) feeding the same region logic and cached convolutions
    f1, f2 = synth.tiny_pair(0)
    runner, reuse = _run_both(oracle, synth.tiny_net(), np.stack([f1, f2, f2, f1])[None], 8, 8, False,
                              diamond=True, k_skip=k_skip)
    assert reuse[1] == 1.0
    v = np.stack([synth.panning_video(5100 + s, n_frames=4, H=96, W=96, fg=((24, 24),), margin=32) for s in range(2)])
    runner, reuse = _run_both(oracle, synth.vgg16(), v, 16, 16, False, bias_scale=0.0, diamond=True, k_skip=k_skip,
                              check_tensors=(0, 1, 2, 5, 10, 17))
    assert max(reuse) > 0.3


def test_exhaustive_search_with_k_skip_in_the_whole_path(oracle):
    f1, f2 = synth.tiny_pair(0)
    _run_both(oracle, synth.tiny_net(), np.stack([f1, f2, f2, f1])[None], 8, 8, False, k_skip=2)


@pytest.mark.parametrize("bf16", [False, True])
def test_alexnet_style_stack_small(oracle, bf16):
    """Every layer type of Table 2 in one stack: 11x11 stride-4 first layer, LRN, pooling, fully-connected, softmax
    (a narrow AlexNet at its 227x227 input size; the paper's 10-pixel blocks)."""
    layers = synth.alexnet(n_classes=40, width=0.25)
    video = np.stack([synth.panning_video(300 + s, n_frames=3, H=227, W=227) for s in range(2)])
    runner, reuse = _run_both(oracle, layers, video, 10, 8, bf16)
    assert len(reuse) == 4 and min(reuse) > 0.2


def test_alexnet_full_width_fp32(oracle):
    """The AlexNet-style stack at its real widths (96-256-384-384-256 channels, 4096-wide fully-connected layers),
    227x227, the paper's 10-pixel blocks: every tensor of a full and a cached frame against the oracle."""
    layers = synth.alexnet()
    video = synth.panning_video(310, n_frames=2, H=227, W=227)[None]
    _run_both(oracle, layers, video, 10, 8, False, bias_scale=0.02)


@pytest.mark.parametrize("bf16", [False, True])
def test_dave_orig_stack(oracle, bf16):
    """The steering network: a 66x200 frame (not square), 5x5 stride-2 convolutions without padding, channel counts
    (24, 36, 48) that are not whole 16-byte vectors in bf16, four fully-connected layers."""
    layers = synth.dave_orig()
    video = np.stack([synth.panning_video(800 + s, n_frames=3, H=66, W=200, fg=((16, 24),)) for s in range(2)])
    runner, reuse = _run_both(oracle, layers, video, 10, 8, bf16, bias_scale=0.02)
    assert runner.shapes[5] == (1, 18, 64) and runner.shapes[-1] == (1, 1, 1)


def test_googlenet_full_width_bf16(oracle):
    """The GoogLeNet-style stack at its real widths, 224x224, bf16: a full and a cached frame."""
    layers = synth.resolve_global_pooling(synth.googlenet(), 224, 224, 3)
    video = synth.panning_video(410, n_frames=2, H=224, W=224)[None]
    _run_both(oracle, layers, video, 16, 8, True, bias_scale=0.02)


def test_googlenet_style_stack_small(oracle):
    """Inception modules: four branches of different depth joined by a concat; global average pooling at the end."""
    layers = synth.resolve_global_pooling(synth.googlenet(n_classes=24, width=0.25), 224, 224, 3)
    assert sum(L["type"] == synth.CONV for L in layers) == 57
    video = np.stack([synth.panning_video(400 + s, n_frames=3, H=224, W=224) for s in range(1)])
    _run_both(oracle, layers, video, 16, 8, True)


def _static_then_moving(seed, H, W, n_static, n_moving):
    """A camera that stands still (only a small object moves), then pans, then stands still again."""
    still = synth.panning_video(seed, n_frames=n_static, H=H, W=W, fg=((24, 24),), pan_speeds=(0,))
    moving = synth.panning_video(seed, n_frames=n_static + n_moving, H=H, W=W, fg=((24, 24),), pan_speeds=(2,),
                                 redraw_every=100)[n_static:]
    return np.concatenate([still, moving, still[::-1]])


@pytest.mark.parametrize("bf16", [False, True])
def test_in_place_frames_of_a_static_camera(oracle, bf16):
    """No stream moves: the conv outputs are updated in the previous frame's buffers and nothing is copied; the
    values are the oracle's (which knows nothing of buffers)."""
    layers = synth.vgg16()[:7]
    video = np.stack([synth.panning_video(500 + s, n_frames=4, H=96, W=96, fg=((24, 24),), pan_speeds=(0,)) for s in range(2)])
    runner, reuse = _run_both(oracle, layers, video, 16, 8, bf16, in_place=True)
    assert runner.in_place_frames == [False, True, True, True]
    assert runner.stats.copy_bytes == 0 and runner.stats.macs_needed < runner.stats.macs_full
    assert min(reuse) > 0.5


def test_border_case_of_a_static_camera(oracle):
    """extend_borders: windows may reach into the zero padding when the stream did not move; regions and tensors
    follow the oracle with the same option, and more pixels are reused than with the printed rule."""
    layers = synth.vgg16()[:10]
    video = np.stack([_static_then_moving(700 + s, 96, 96, 3, 2) for s in range(2)])
    needed = {}
    for ext in (False, True):
        runner, _ = _run_both(oracle, layers, video, 16, 8, True, in_place=True, extend_borders=ext)
        needed[ext] = runner.stats.macs_needed          # last frame: static again
        assert runner.in_place_frames[-1]
    assert needed[True] < needed[False]


def test_in_place_and_copied_frames_mix(oracle):
    """Static and moving stretches in one video: in-place frames where every stream's motion is zero, shifted copies
    elsewhere, parity on every frame; and bit-identical tensors with the option off."""
    layers = synth.resnet50_trunk()[:14]
    video = np.stack([_static_then_moving(600 + s, 96, 96, 3, 3) for s in range(2)])
    runner, _ = _run_both(oracle, layers, video, 16, 8, True, residual_scale=0.5, in_place=True)
    flags = runner.in_place_frames
    assert flags[1] and flags[2] and not any(flags[3:6]) and flags[-1], flags
    ws, bs = synth.he_weights(layers, 1, bias_scale=0.05, residual_scale=0.5, input_shape=(96, 96, 3))
    dev_video = torch.from_numpy(np.ascontiguousarray(video.transpose(1, 0, 2, 3, 4))).to(DEV)
    runs = [binding.StackRunner(layers, ws, bs, 2, 96, 96, 3, block=16, radius=8, dtype=binding.DC_BF16, in_place=ip)
            for ip in (False, True)]
    for t in range(video.shape[1]):
        outs = []
        for r in runs:
            tensors = r.step(dev_video[t])
            torch.cuda.synchronize()
            outs.append([x.clone() for x in tensors])
        for a, b in zip(*outs):
            assert torch.equal(a, b), t


def test_vgg16_two_streams_bf16_small(oracle):
    # batch mode: per-stream caches, per-stream motion, one launch per layer
    v = np.stack([synth.panning_video(5000 + s, n_frames=3, H=96, W=96, fg=((24, 24),), margin=32) for s in range(2)])
    _run_both(oracle, synth.vgg16(), v, 16, 16, True, bias_scale=0.0)


def test_expiry_and_reset(oracle):
    f1, f2 = synth.tiny_pair(3)
    video = np.stack([f1, f2, f2, f1, f1, f2])[None]
    _run_both(oracle, synth.tiny_net(), video, 8, 8, False, expiry=3, resets=(4,))


def test_resnet_stage_small(oracle):
    layers = synth.resnet50_trunk()[:23]     # stem, pool, stage 1 (3 blocks), first block of stage 2
    v = synth.panning_video(3000, n_frames=3, H=96, W=96, fg=((24, 24),), margin=32)[None]
    _run_both(oracle, layers, v, 16, 16, True, bias_scale=0.0, residual_scale=0.5)
    _run_both(oracle, layers, v, 16, 16, False, bias_scale=0.0, residual_scale=0.5)


@pytest.mark.parametrize("bf16", [False, True])
def test_darknet_with_leaky_relu_small(oracle, bf16):
    """The published Darknet activation (leaky ReLU, slope 0.1) through every conv kernel family: first layer, 3x3,
    1x1, and the register-weight kernel's fallback."""
    layers = synth.darknet19(leaky=True)[:12]
    video = np.stack([synth.panning_video(900 + s, n_frames=3, H=96, W=96, fg=((24, 24),)) for s in range(2)])
    _run_both(oracle, layers, video, 16, 8, bf16)


def test_darknet_head_small(oracle):
    layers = synth.darknet19()[:12]
    v = synth.reuse_sweep_video(4001, 0.75, n_frames=3, H=128, W=128, cut_at=2)[None]
    _run_both(oracle, layers, v, 16, 16, True, bias_scale=0.0, resets=(2,))


# ---- full-size configurations -------------------------------------------------------------------

def _sampled_conv_check(oracle, layers, ws, bs, tensors, li, stream, bf16, n_samples, rng, tol):
    """Recompute sampled output pixels of conv layer li from the GPU's own input tensor with the oracle's
    direct loop (valid for pixels that were computed, i.e. on a full frame)."""
    L = layers[li]
    x = tensors[L["in0"]][stream].float().cpu().numpy()
    y = tensors[li + 1][stream].float().cpu().numpy()
    w = oracle.round_bf16(ws[li]) if bf16 else ws[li]
    if w.shape[-1] < x.shape[-1]:     # input channels padded by the runner
        wp = np.zeros(w.shape[:3] + (x.shape[-1],), np.float32)
        wp[..., :w.shape[-1]] = w
        w = wp
    k, s, p = L["k"], L["s"], L["p"]
    Ho, Wo, _ = y.shape
    scale = float(np.abs(y).max()) + 1e-30
    for _ in range(n_samples):
        oy, ox = int(rng.integers(0, Ho)), int(rng.integers(0, Wo))
        # window of the input around the sampled pixel, zero padded
        win = np.zeros((k, k, x.shape[-1]), np.float32)
        for ky in range(k):
            for kx in range(k):
                iy, ix = oy * s - p + ky, ox * s - p + kx
                if 0 <= iy < x.shape[0] and 0 <= ix < x.shape[1]:
                    win[ky, kx] = x[iy, ix]
        want = oracle.conv_cached(win, w, bs[li], k, 1, 0, L["relu"], bf16=bf16)[0, 0]
        assert np.abs(y[oy, ox] - want).max() / scale <= tol, (li, oy, ox)


def test_resnet50_trunk_224_bf16_full_size(oracle):
    """configs[2] at full size: two frames through the GPU path; frame 0 against the oracle's whole stack
    (full compute), frame 1 (cached) for rectangles bit-exact and features within tolerance."""
    layers = synth.resnet50_trunk()
    video = synth.panning_video(2000, n_frames=2)[None]
    _run_both(oracle, layers, video, 16, 16, True, bias_scale=0.0, residual_scale=0.5)


def test_darknet19_416_bf16_cached_frame_and_scene_cut(oracle):
    """configs[3] at full size (416x416, 19 conv layers, bf16, moving noise rectangles at half reuse): the last two
    frames of the first scene and the first two of the second, with the cache dropped at the cut as the config
    says.  Every tensor of the full frames and of the cached frames (reused pixels are the oracle's shifted cache,
    the others its convolution), match results, masks and rectangles against the oracle's stream."""
    layers = synth.darknet19()
    video = synth.reuse_sweep_video(4002, 0.5, n_frames=60)[28:32][None]
    runner, reuse = _run_both(oracle, layers, video, 16, 16, True, bias_scale=0.0, resets=(2,))
    assert len(reuse) == 2 and all(0.45 < r < 0.6 for r in reuse)


@pytest.mark.parametrize("device_plan,exact,torus", [(False, False, False), (True, False, False), (True, True, False),
                                                     (True, True, True)])
def test_throughput_mode_64_streams_bf16_sampled(oracle, device_plan, exact, torus):
    """configs[4] launch configuration: 64 streams in one batch, VGG-16-style, bf16, planned on the host, on the GPU, on
    the GPU with exact reuse maps, and the same with the conv outputs on a torus (what bench.py times).  Three streams
    are followed by the oracle over four time steps (everything compared); the others are checked for bit-exact match
    results on the cached steps."""
    layers = synth.vgg16()
    n, T = 64, 4 if torus else 3
    videos = np.stack([synth.panning_video(5000 + s, n_frames=T) for s in range(n)])
    ws, bs = synth.he_weights(layers, 1)
    r = binding.StackRunner(layers, ws, bs, n, 224, 224, 3, block=16, radius=16, dtype=binding.DC_BF16, want_regions=True,
                            device_plan=device_plan, exact_masks=exact, torus=torus, want_origins=torus)
    followed = [0, 31, 63]
    refs = {s: oracle.Stream(layers, ws, bs, 224, 224, 3, block=16, radius=16, bf16=True, exact_masks=exact) for s in followed}
    dv = torch.from_numpy(np.ascontiguousarray(videos.transpose(1, 0, 2, 3, 4))).to(DEV)
    for t in range(T):
        print(f"[batch64] step {t}", flush=True)
        tensors = r.step(dv[t])
        torch.cuda.synchronize()
        if torus:       # only the followed streams are rolled back to their logical layout
            moved = r.origins.copy()
            tensors = [x if not moved[followed, ti].any() else
                       {s: torch.roll(x[s], shifts=(-int(moved[s, ti, 1]), -int(moved[s, ti, 0])), dims=(0, 1)) for s in followed}
                       for ti, x in enumerate(tensors)]
        for s in followed:
            want = refs[s].step(videos[s, t])
            for ti in range(1, len(layers) + 1):
                g = tensors[ti][s].float().cpu().numpy()
                assert _rel_err(g, want["tensors"][ti]) <= 2e-2, (t, s, ti)
            if t > 0 and not exact:
                regs = r.regions(s)
                for ti in range(len(layers) + 1):
                    assert regs[ti]["rects"].tolist() == want["rects"][ti].tolist()
        if t > 0:
            if exact:       # the maps themselves: the multiply-adds the library counted are those of the oracle's maps
                assert r.read_stats().n_overflow_streams == 0
            masks = r.mask.cpu().numpy()
            gmv = r.gmv.cpu().numpy()
            for s in range(0, n, 7):
                m = oracle.match_blocks(videos[s, t], videos[s, t - 1], 16, 16, synth.max_block_ssd(16))
                assert np.array_equal(masks[s], m["mask"]) and gmv[s].tolist() == m["gmv"].tolist()


@pytest.mark.parametrize("bf16", [False, True])
def test_exact_reuse_maps_tiny_and_vgg(oracle, bf16):
    """dc_match_options.exact_masks: the conv layers reuse the pixels of the exact maps; tensors and work counters
    against the oracle's stream in the same mode."""
    f1, f2 = synth.tiny_pair(0)
    runner, reuse = _run_both(oracle, synth.tiny_net(), np.stack([f1, f2, f2, f1])[None], 8, 8, bf16, exact_masks=True)
    assert abs(reuse[0] - 45 / 64) < 1e-9
    v = np.stack([synth.panning_video(5000 + s, n_frames=3, H=96, W=96, fg=((24, 24),), margin=32) for s in range(2)])
    _run_both(oracle, synth.vgg16(), v, 16, 16, bf16, bias_scale=0.0, exact_masks=True)


def test_exact_reuse_maps_other_stacks(oracle):
    v = synth.panning_video(3000, n_frames=3, H=96, W=96, fg=((24, 24),), margin=32)[None]
    _run_both(oracle, synth.resnet50_trunk()[:23], v, 16, 16, True, bias_scale=0.0, residual_scale=0.5, exact_masks=True)
    v = synth.reuse_sweep_video(4001, 0.75, n_frames=3, H=128, W=128, cut_at=2)[None]
    _run_both(oracle, synth.darknet19()[:12], v, 16, 16, True, bias_scale=0.0, resets=(2,), exact_masks=True)
    layers = synth.alexnet(n_classes=40, width=0.25)
    video = np.stack([synth.panning_video(300 + s, n_frames=3, H=227, W=227) for s in range(2)])
    _run_both(oracle, layers, video, 10, 8, False, exact_masks=True)
    video = np.stack([_static_then_moving(700 + s, 96, 96, 3, 2) for s in range(2)])
    _run_both(oracle, synth.vgg16()[:10], video, 16, 8, True, extend_borders=True, exact_masks=True)


def test_exact_reuse_maps_vgg16_224_save_more(oracle):
    """configs[1] with exact maps: parity on the first frames, and fewer multiply-adds needed than with rectangles."""
    video = synth.panning_video(2000, n_frames=3)[None]
    exact, _ = _run_both(oracle, synth.vgg16(), video, 16, 16, False, bias_scale=0.0, exact_masks=True)
    rect, _ = _run_both(oracle, synth.vgg16(), video, 16, 16, False, bias_scale=0.0, device_plan=True)
    assert exact.read_stats().macs_needed < rect.read_stats().macs_needed


def _pool_add_stack(c=8):
    conv = lambda cin, cout, i, relu=1: dict(type=synth.CONV, k=3, s=1, p=1, cin=cin, cout=cout, relu=relu, in0=i, in1=-1)
    return [conv(3, c, 0), dict(type=synth.MAXPOOL, k=2, s=2, p=0, cin=c, cout=c, relu=0, in0=1, in1=-1),
            conv(c, c, 2), conv(c, c, 3, 0), dict(type=synth.ADD, k=1, s=1, p=0, cin=c, cout=c, relu=1, in0=4, in1=2),
            dict(type=synth.MAXPOOL, k=3, s=2, p=1, cin=c, cout=c, relu=0, in0=5, in1=-1), conv(c, c, 6)]


@pytest.mark.parametrize("bf16", [False, True])
def test_cached_pool_and_add_layers(oracle, bf16):
    """dc_match_options.cache_pool_add: max-pooling and add outputs come from the cache where their maps are set
    (Section 5).  The case is one where the option changes the result, so a library that ignored it would fail."""
    layers = _pool_add_stack()
    f1, f2 = synth.tiny_pair(0)                   # a noisy frame moved by (3, -2): not a multiple of the strides
    video = np.stack([f1, f2, f2, f1])[None]
    H, W, C = f1.shape
    ws, bs = synth.he_weights(layers, 1, bias_scale=0.05, input_shape=(H, W, C))
    on = oracle.Stream(layers, ws, bs, H, W, C, block=8, radius=8, bf16=bf16, exact_masks=True, cache_pool_add=True)
    off = oracle.Stream(layers, ws, bs, H, W, C, block=8, radius=8, bf16=bf16, exact_masks=True)
    a = [on.step(f) for f in (f1, f2)][1]["tensors"][2]
    b = [off.step(f) for f in (f1, f2)][1]["tensors"][2]
    assert _rel_err(a, b) > 0.05
    _run_both(oracle, layers, video, 8, 8, bf16, cache_pool_add=True)
    # several streams, a scene cut and a forced full frame in between
    video = np.stack([synth.reuse_sweep_video(4100 + s, 0.75, n_frames=5, H=96, W=96, cut_at=3) for s in range(3)])
    _run_both(oracle, layers, video, 8, 8, bf16, cache_pool_add=True, resets=(2,))


def test_cached_pool_and_add_in_the_model_stacks(oracle):
    v = np.stack([synth.panning_video(5000 + s, n_frames=3, H=96, W=96, fg=((24, 24),), margin=32) for s in range(2)])
    _run_both(oracle, synth.vgg16(), v, 16, 16, True, bias_scale=0.0, cache_pool_add=True)
    v = synth.panning_video(3000, n_frames=3, H=96, W=96, fg=((24, 24),), margin=32)[None]
    _run_both(oracle, synth.resnet50_trunk()[:23], v, 16, 16, True, bias_scale=0.0, residual_scale=0.5, cache_pool_add=True)
    v = synth.reuse_sweep_video(4001, 0.75, n_frames=3, H=128, W=128)[None]
    _run_both(oracle, synth.darknet19()[:12], v, 16, 16, False, bias_scale=0.0, cache_pool_add=True)


def test_cache_pool_add_needs_exact_maps_and_previous_outputs(oracle):
    layers = _pool_add_stack()
    f1, f2 = synth.tiny_pair(0)
    H, W, C = f1.shape
    ws, bs = synth.he_weights(layers, 1, input_shape=(H, W, C))
    r = binding.StackRunner(layers, ws, bs, 1, H, W, C, block=8, radius=8, dtype=binding.DC_F32, device_plan=True,
                            exact_masks=True, cache_pool_add=True)
    r.match_options.exact_masks = 0
    with pytest.raises(binding.DcError) as e:
        r.step(torch.from_numpy(f1[None]).to(DEV))
    assert e.value.status == -4
    torch.cuda.synchronize()


@pytest.mark.parametrize("exact", [False, True])
def test_conv_layers_that_do_not_use_the_cache(oracle, exact):
    """dc_match_options.no_reuse: flagged conv layers are computed in full, the others reuse; planned on the host and on
    the GPU, rectangles and exact maps."""
    layers = synth.tiny_net()
    f1, f2 = synth.tiny_pair(0)
    video = np.stack([f1, f2, f2, f1])[None]
    for flags in ([0, 1, 0], [1, 0, 1], [1, 1, 1]):
        _run_both(oracle, layers, video, 8, 8, False, exact_masks=exact, no_reuse=np.array(flags, np.uint8))
    # the break-even policy on a model stack: layers with few multiply-adds per output are not cached
    v = np.stack([synth.panning_video(5000 + s, n_frames=3, H=96, W=96, fg=((24, 24),), margin=32) for s in range(2)])
    layers = synth.vgg16()
    flags = synth.no_reuse_flags(layers, 600)
    assert flags.tolist()[:5] == [1, 1, 0, 1, 0] and flags.sum() == 3
    _run_both(oracle, layers, v, 16, 16, True, bias_scale=0.0, exact_masks=exact, no_reuse=flags)
    layers = synth.resnet50_trunk()[:23]
    v = synth.panning_video(3000, n_frames=3, H=96, W=96, fg=((24, 24),), margin=32)[None]
    _run_both(oracle, layers, v, 16, 16, True, bias_scale=0.0, residual_scale=0.5, exact_masks=exact,
              no_reuse=synth.no_reuse_flags(layers, 600))


@pytest.mark.parametrize("bf16", [False, True])
def test_stack_with_kernels_that_are_not_square_or_dilated(oracle, bf16):
    """1 x 7 / 7 x 1 pairs, dilated 3 x 3 and 5 x 3 kernels (dc_layer.k2 / p2 / dil) through the whole path: regions,
    exact maps, copies and the general conv kernels, planned on the host and on the GPU."""
    layers = synth.factorised_net(16)
    video = np.stack([synth.panning_video(900 + s, n_frames=3, H=96, W=96, fg=((24, 24),), margin=32) for s in range(2)])
    runner, reuse = _run_both(oracle, layers, video, 8, 8, bf16)
    assert max(reuse) > 0.3
    _run_both(oracle, layers, video, 8, 8, bf16, exact_masks=True)
    f1, f2 = synth.tiny_pair(0)
    _run_both(oracle, layers, np.stack([f1, f2, f2])[None], 8, 8, bf16, extend_borders=True)


def _torus_stack(c=64):
    """first layer on a padded pixel vector, 3x3 layers with whole 64-byte rows, 2x2 poolings: what the torus mode takes"""
    return synth.small_vgg(c)


@pytest.mark.parametrize("exact", [False, True])
@pytest.mark.parametrize("bf16", [False, True])
def test_conv_outputs_on_a_torus(oracle, bf16, exact):
    """dc_match_options.torus: nothing is copied, every conv output is one buffer whose origin moves with the frames; the
    tensors, read from their origins, are those of the oracle's stream (and of the copying path)."""
    layers = _torus_stack()
    # a pan that crosses the seams several times, streams that move differently, a scene cut, an expiry in between
    video = np.stack([synth.panning_video(7000 + s, n_frames=7, H=96, W=96, fg=((24, 24),), margin=32) for s in range(3)])
    runner, reuse = _run_one(oracle, layers, video, 16, 16, bf16, device_plan=True, exact_masks=exact, torus=True, resets=(4,),
                             expiry=3, bias_scale=0.0)
    assert max(reuse) > 0.3 and runner.torus
    # the tiny pair: motion (-3, +2), then a frame that does not move, then back
    f1, f2 = synth.tiny_pair(0)
    _run_one(oracle, _torus_stack(64), np.stack([f1, f2, f2, f1, f2])[None], 8, 8, bf16, device_plan=True, exact_masks=exact, torus=True)


def test_torus_vgg16_two_streams(oracle):
    v = np.stack([synth.panning_video(5000 + s, n_frames=4, H=96, W=96, fg=((24, 24),), margin=32) for s in range(2)])
    runner, _ = _run_one(oracle, synth.vgg16(), v, 16, 16, True, device_plan=True, exact_masks=True, torus=True, bias_scale=0.0)
    assert runner.origins.any()          # some origin moved
    assert runner.read_stats().copy_bytes == 0


def test_torus_tensors_read_without_a_wait(oracle):
    """dc_torus_read with the device address of the frame's origins (origins_dev_out): the logical tensors without any
    host wait, equal to those rolled on the host from origins_out; full frames (no origins) included."""
    layers = synth.small_vgg()
    video = np.stack([synth.panning_video(7600 + s, n_frames=6, H=96, W=96, fg=((24, 24),), margin=32) for s in range(3)])
    ws, bs = synth.he_weights(layers, 1, bias_scale=0.05)
    r = binding.StackRunner(layers, ws, bs, 3, 96, 96, 3, block=16, radius=16, dtype=binding.DC_BF16, device_plan=True,
                            exact_masks=True, cache_pool_add=True, torus=True, want_origins=True, expiry=4)
    dv = torch.from_numpy(np.ascontiguousarray(video.transpose(1, 0, 2, 3, 4))).to(DEV)
    moved = False
    for t in range(6):
        tensors = r.step(dv[t])
        got = [r.read_tensor(ti, tensors) for ti in range(len(layers) + 1)]      # queued behind the frame, nothing waited for
        torch.cuda.synchronize()
        want = r.logical_tensors(tensors)
        moved = moved or bool(r.origins.any())
        for ti in range(len(layers) + 1):
            assert torch.equal(got[ti], want[ti]), (t, ti)
    assert moved
    # odd channel counts and element sizes take the narrower vectors
    x = torch.randn((2, 5, 7, 3), device=DEV)
    org = torch.tensor([[3, 1], [6, 4]], dtype=torch.int32, device=DEV)
    out = torch.empty_like(x)
    L = binding.lib()
    import ctypes as C
    assert L.dc_torus_read(C.c_void_p(x.data_ptr()), C.c_void_p(out.data_ptr()), C.c_void_p(org.data_ptr()), 2, 2, 5, 7, 3,
                           binding.DC_F32, None) == 0
    torch.cuda.synchronize()
    for s in range(2):
        assert torch.equal(out[s], torch.roll(x[s], shifts=(-int(org[s, 1]), -int(org[s, 0])), dims=(0, 1)))
    assert L.dc_torus_read(C.c_void_p(x.data_ptr()), C.c_void_p(x.data_ptr()), None, 2, 2, 5, 7, 3, binding.DC_F32, None) == -1


@pytest.mark.parametrize("bf16", [False, True])
def test_poolings_on_the_torus_too(oracle, bf16):
    """torus with cache_pool_add: the poolings' outputs are cache values on a torus of their own, a pooled pixel whose map
    bit is set is not touched; the oracle's stream with max-pooling through the cache gives the logical tensors."""
    video = np.stack([synth.panning_video(7100 + s, n_frames=7, H=96, W=96, fg=((24, 24),), margin=32) for s in range(3)])
    runner, reuse = _run_one(oracle, _torus_stack(), video, 16, 16, bf16, device_plan=True, exact_masks=True, cache_pool_add=True,
                             torus=True, resets=(4,), expiry=3)
    assert max(reuse) > 0.3 and runner.origins[:, 3].any()       # tensor 3 is the first pooling's output
    v = np.stack([synth.panning_video(5000 + s, n_frames=4, H=96, W=96, fg=((24, 24),), margin=32) for s in range(2)])
    _run_one(oracle, synth.vgg16(), v, 16, 16, bf16, device_plan=True, exact_masks=True, cache_pool_add=True, torus=True, bias_scale=0.0)
    if bf16:     # enough units for the register-weight kernel in the second layer, whose output the first pooling reads
        v32 = np.stack([synth.panning_video(7700 + s, n_frames=4, H=96, W=96, fg=((24, 24),), margin=32) for s in range(32)])
        runner, _ = _run_one(oracle, synth.small_vgg(), v32, 16, 16, True, device_plan=True, exact_masks=True, cache_pool_add=True,
                             torus=True, resets=(2,))
        assert runner.layer_stats()["kernel_id"][1] == 130


def test_torus_with_the_border_case_and_layers_outside_the_cache(oracle):
    layers = _torus_stack()
    video = np.stack([_static_then_moving(700 + s, 96, 96, 3, 2) for s in range(2)])
    _run_one(oracle, layers, video, 16, 8, True, extend_borders=True, device_plan=True, exact_masks=True, torus=True)
    flags = np.zeros(len(layers), np.uint8)
    flags[1] = flags[4] = 1
    v = np.stack([synth.panning_video(7200 + s, n_frames=5, H=96, W=96, fg=((24, 24),), margin=32) for s in range(2)])
    _run_one(oracle, layers, v, 16, 16, False, device_plan=True, exact_masks=False, torus=True, no_reuse=flags)


@pytest.mark.parametrize("bf16,leaky", [(True, False), (False, True)])
def test_torus_darknet_with_1x1_layers(oracle, bf16, leaky):
    """The Darknet-19-style stack on a torus: 3x3 layers, 1x1 bottlenecks (the 1x1 kernel reads and writes through
    origins), 2x2 poolings, maps with ragged units (13 x 13 at the end), ReLU or leaky ReLU."""
    video = np.stack([synth.panning_video(7500 + s, n_frames=5, H=208, W=208, fg=((48, 48),), margin=32) for s in range(2)])
    runner, reuse = _run_one(oracle, synth.darknet19(leaky=leaky)[:17], video, 16, 8, bf16, device_plan=True, exact_masks=True,
                             torus=True, resets=(3,), bias_scale=0.02)
    assert max(reuse) > 0.3 and runner.origins.any() and runner.shapes[-1][0] == 13


def test_torus_on_a_frame_whose_maps_do_not_fit_the_lds(oracle):
    """640 x 480: the reuse bitmaps of the stack (more than 128 KB) are built in the workspace; the origins come from the
    same planning kernel.  One full and two cached frames of one stream."""
    video = synth.panning_video(7400, n_frames=3, H=480, W=640, fg=((96, 96),), margin=64)[None]
    runner, reuse = _run_one(oracle, synth.small_vgg(), video, 16, 16, True, device_plan=True, exact_masks=True, torus=True,
                             bias_scale=0.0)
    assert max(reuse) > 0.5 and runner.origins.any()


def test_torus_with_more_streams_than_the_origin_tables_hold(oracle):
    """Beyond 2048 streams the persistent kernels do not keep the origins in LDS: the first layer loads them from memory
    and the 64-channel layers take the tiled GEMM kernel.  2100 small streams (three videos, repeated); six are compared."""
    layers = synth.small_vgg()
    n, T, H, W = 2100, 3, 32, 32
    base = np.stack([synth.panning_video(7300 + s, n_frames=T, H=H, W=W, fg=((8, 8),), margin=16) for s in range(3)])
    videos = base[np.arange(n) % 3]
    ws, bs = synth.he_weights(layers, 1, bias_scale=0.05)
    r = binding.StackRunner(layers, ws, bs, n, H, W, 3, block=16, radius=8, dtype=binding.DC_BF16, device_plan=True,
                            exact_masks=True, torus=True, want_origins=True)
    followed = [0, 1, 2, 1037, 2098, 2099]
    refs = {s: oracle.Stream(layers, ws, bs, H, W, 3, block=16, radius=8, bf16=True, exact_masks=True) for s in followed}
    dv = torch.from_numpy(np.ascontiguousarray(videos.transpose(1, 0, 2, 3, 4))).to(DEV)
    reused = 0
    for t in range(T):
        print(f"[many streams] step {t}", flush=True)
        tensors = r.step(dv[t])
        torch.cuda.synchronize()
        org = r.origins.copy()
        for s in followed:
            want = refs[s].step(videos[s, t])
            for ti in range(1, len(layers) + 1):
                g = torch.roll(tensors[ti][s], shifts=(-int(org[s, ti, 1]), -int(org[s, ti, 0])), dims=(0, 1)).float().cpu().numpy()
                assert _rel_err(g, want["tensors"][ti]) <= 2e-2, (t, s, ti)
        if t > 0:
            reused += int(r.read_stats().n_reusable_blocks)
    assert reused > 0


def test_torus_is_refused_for_stacks_it_cannot_take(oracle):
    layers = synth.resnet50_trunk()[:10]         # 1x1 and strided layers, adds
    H = W = 64
    ws, bs = synth.he_weights(layers, 1, input_shape=(H, W, 3))
    r = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=8, dtype=binding.DC_BF16, device_plan=True, torus=True)
    with pytest.raises(binding.DcError) as e:
        r.step(torch.zeros((1, H, W, 3), dtype=torch.uint8, device=DEV))
    assert e.value.status == -4
    torch.cuda.synchronize()


def test_border_case_planned_on_the_gpu(oracle):
    """extend_borders with the frame planned on the GPU (copy path: in-place frames are the host's)."""
    layers = synth.vgg16()[:10]
    video = np.stack([_static_then_moving(700 + s, 96, 96, 3, 2) for s in range(2)])
    _run_both(oracle, layers, video, 16, 8, True, extend_borders=True, device_plan=True)


@pytest.mark.parametrize("n_streams,bf16", [(1, False), (3, True)])
def test_frames_planned_on_the_gpu_without_any_wait(oracle, n_streams, bf16):
    """Frames planned on the GPU, two in flight: the host never waits for the frame that it has just issued (no regions are asked
    for), expiry and a scene cut included; every tensor of every frame is cloned on the caller's stream, before the step that
    is given its buffer again, and compared with the oracle at the end, and the work counters of the last frame are read once
    everything is done."""
    layers = synth.vgg16()[:10]
    T, H, W = 9, 96, 96
    videos = np.stack([synth.panning_video(6100 + s, n_frames=T, H=H, W=W, fg=((24, 24),), margin=32) for s in range(n_streams)])
    ws, bs = synth.he_weights(layers, 1, bias_scale=0.05)
    dt = binding.DC_BF16 if bf16 else binding.DC_F32
    r = binding.StackRunner(layers, ws, bs, n_streams, H, W, 3, block=16, radius=8, dtype=dt, expiry=4, device_plan=True)
    refs = [oracle.Stream(layers, ws, bs, H, W, 3, block=16, radius=8, bf16=bf16, expiry=4) for _ in range(n_streams)]
    dv = torch.from_numpy(np.ascontiguousarray(videos.transpose(1, 0, 2, 3, 4))).to(DEV)
    torch.cuda.synchronize()
    kept, cloned = [], []
    for t in range(T):
        if t == 6:
            r.reset()
        if t >= 2:
            cloned[t - 2].synchronize()          # this step's first stage may overwrite that frame's tensors at once
        kept.append([x.clone() for x in r.step(dv[t])])
        cloned.append(torch.cuda.Event())
        cloned[t].record()
    torch.cuda.synchronize()
    tol = 2e-2 if bf16 else 1e-4
    last_blocks = 0
    for t in range(T):
        for s in range(n_streams):
            if t == 6:
                refs[s].reset()
            want = refs[s].step(videos[s, t])
            for ti in range(1, len(layers) + 1):
                assert _rel_err(kept[t][ti][s].float().cpu().numpy(), want["tensors"][ti]) <= tol, (t, s, ti)
            if t == T - 1:
                assert not want["full"]
                last_blocks += int(want["match"]["mask"].sum())
    assert r.read_stats().n_reusable_blocks == last_blocks


@pytest.mark.parametrize("net,size,bf16", [("vgg16", 96, False), ("resnet", 64, True)])
def test_overlap_modes_give_identical_tensors(net, size, bf16):
    """Two frames in flight, matching on a second stream only, and everything on the caller's stream run the
    same kernels with the same plans: every tensor of every frame must be bit-identical, also when the frames
    are issued back to back without any synchronisation in between (Section 7.6: asynchronous stages)."""
    H = W = size
    if net == "vgg16":
        layers = synth.vgg16()
        ws, bs = synth.he_weights(layers, 3, bias_scale=0.05)
    else:
        layers = synth.resnet50_trunk()[:24]       # stem, pool, the first two bottleneck blocks
        ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, residual_scale=0.5)
    T = 14
    video = torch.from_numpy(synth.panning_video(77, n_frames=T, H=H, W=W, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    dt = binding.DC_BF16 if bf16 else binding.DC_F32
    results = {}
    for mode, kw in (("pipeline", dict(overlap=True, pipeline=True)), ("overlap", dict(overlap=True, pipeline=False)),
                     ("plain", dict(overlap=False))):
        print(f"[overlap modes] {net} {mode}", flush=True)
        runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=16, dtype=dt, expiry=5, **kw)
        kept = []
        for stop in (3, 8, T):                        # the tensors are read when a run of frames has drained
            runner.reset()
            for t in range(stop):
                tensors = runner.step(frames[t])      # no synchronisation between the frames of a run
            torch.cuda.synchronize()
            kept.append([x.clone() for x in tensors])
        results[mode] = kept
        del runner
    for mode in ("overlap", "plain"):
        for f, (a, b) in enumerate(zip(results["pipeline"], results[mode])):
            for i, (x, y) in enumerate(zip(a, b)):
                assert torch.equal(x, y), (net, mode, f, i)


def test_pipelined_frames_with_irregular_buffer_alternation():
    """The writer of a tensor that crosses from one stage to the next waits for the readers of the frame that last used its
    buffer, and a tensor that turns out to have the same buffer in consecutive frames is kept inside one stage; a caller that
    alternates the buffers irregularly must still get the same tensors.  The runner's choice of the set for the tensors that are not conv outputs is overridden
    frame by frame with a pattern that holds every transition; frames are issued without synchronisation."""
    H = W = 96
    layers = synth.vgg16()
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05)
    T = 14
    video = torch.from_numpy(synth.panning_video(78, n_frames=T, H=H, W=W, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    pattern = [0, 1, 0, 0, 1, 1, 1, 0, 1, 0, 0, 0, 1, 0]
    finals = {}
    for mode, kw in (("pipeline", dict(overlap=True, pipeline=True)), ("plain", dict(overlap=False))):
        print(f"[irregular alternation] {mode}", flush=True)
        runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=16, dtype=binding.DC_F32, expiry=6, **kw)
        kept = []
        for stop in (5, 9, T):
            runner.reset()
            for t in range(stop):
                if mode == "pipeline":
                    runner.cur_other = pattern[t]
                tensors = runner.step(frames[t])
            torch.cuda.synchronize()
            kept.append([x.clone() for x in tensors])
        finals[mode] = kept
        del runner
    for f, (a, b) in enumerate(zip(finals["pipeline"], finals["plain"])):
        for i, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x, y), (f, i)


def test_pageable_host_workspace_gives_the_same_tensors():
    """The frame's plans reach the device through a kernel that reads the pinned staging buffer, or through an
    asynchronous copy when the host workspace is pageable memory: same tensors either way."""
    H = W = 64
    layers = synth.vgg16()[:7]
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05)
    T = 6
    video = torch.from_numpy(synth.panning_video(79, n_frames=T, H=H, W=W, fg=((16, 16), (8, 24)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    outs = {}
    for pinned in (True, False):
        print(f"[host workspace] pinned={pinned}", flush=True)
        runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=16, dtype=binding.DC_F32)
        if not pinned:
            runner.ws_host = torch.empty(runner.ws_host.numel(), dtype=torch.uint8)
        kept = []
        for t in range(T):
            tensors = runner.step(frames[t])
            torch.cuda.synchronize()
            kept.append([x.clone() for x in tensors])
        assert runner.stats.n_reusable_blocks > 0
        outs[pinned] = kept
        del runner
    for a, b in zip(outs[True], outs[False]):
        for x, y in zip(a, b):
            assert torch.equal(x, y)


def test_lookahead_matching_gives_the_same_tensors():
    """Section 7.6: the matching of the next frame started one step early (dc_prefetch_match) must change
    nothing but the time at which it runs: same tensors and the same masks as without it, across cache expiry,
    a scene cut, and a look-ahead that names a frame other than the one that follows (it must be ignored)."""
    H = W = 96
    layers = synth.vgg16()[:10]
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05)
    T = 12
    video = torch.from_numpy(synth.panning_video(80, n_frames=T, H=H, W=W, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    order = list(range(T)) + [3, 4, 5]              # a jump back: a scene cut handled by reset()
    results = {}
    for look in (False, True):
        print(f"[lookahead] {look}", flush=True)
        runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=16, dtype=binding.DC_F32, expiry=5)
        kept = []
        for j, t in enumerate(order):
            if j == T:
                runner.reset()
            nxt = None
            if look and j + 1 < len(order):
                nxt = frames[order[j + 1]]
                if j == 6:
                    nxt = frames[0]                 # wrong guess: the next call must match again itself
            tensors = runner.step(frames[t], next_frames=nxt)
            torch.cuda.synchronize()
            kept.append(([x.clone() for x in tensors], runner.stats.n_reusable_blocks, runner.stats.full))
        results[look] = kept
        del runner
    assert any(not full and reusable > 0 for _, reusable, full in results[True])
    for j, ((a, ra, fa), (b, rb, fb)) in enumerate(zip(results[False], results[True])):
        assert (ra, fa) == (rb, fb), j
        for i, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x, y), (j, i)


def test_lookahead_matching_without_synchronisation():
    """The same with two frames in flight and no synchronisation between the steps."""
    H = W = 96
    layers = synth.vgg16()
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05)
    T = 14
    video = torch.from_numpy(synth.panning_video(81, n_frames=T, H=H, W=W, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    finals = {}
    for look in (False, True):
        runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=16, dtype=binding.DC_F32, expiry=6)
        kept = []
        for stop in (4, 9, T):
            runner.reset()
            for t in range(stop):
                tensors = runner.step(frames[t], next_frames=frames[t + 1] if (look and t + 1 < stop) else None)
            torch.cuda.synchronize()
            kept.append([x.clone() for x in tensors])
        finals[look] = kept
        del runner
    for a, b in zip(finals[False], finals[True]):
        for x, y in zip(a, b):
            assert torch.equal(x, y)


@pytest.mark.parametrize("net,size", [("tiny", 64), ("vgg", 96), ("vgg", 320)])
def test_lookahead_planned_on_the_gpu_is_dropped_by_a_full_frame(net, size):
    """Look-ahead matches of frames planned on the GPU, taken, guessed wrong and dropped by a full frame that comes in between
    (the next cached frame writes the same match buffers and must come after the dropped match): stacks of one stage, which
    match on the caller's stream, and of several, no synchronisation between the steps of a run.  Same masks, motion and
    tensors as without look-ahead (fp32; a split K may be grouped differently: K <= 4608 products, sqrt(K) 2^-24 a layer)."""
    H = W = size
    layers = synth.tiny_net() if net == "tiny" else synth.vgg16()[:17]
    block = 8 if net == "tiny" else 16
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(H, W, 3))
    T = 10
    video = torch.from_numpy(synth.panning_video(86, n_frames=T, H=H, W=W, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    finals = {}
    for look in (False, True):
        print(f"[lookahead, GPU plan] {net} {size} {look}", flush=True)
        runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=block, radius=block, dtype=binding.DC_F32, device_plan=True,
                                     exact_masks=True)
        kept = []
        for stop in (2, 3, 4, 6, T, T, T):
            runner.reset()
            for t in range(stop):
                nxt = frames[t + 1] if look and t + 1 < T else None
                if look and t == 4:
                    nxt = frames[0]                                  # a wrong guess
                force = t in (3, 7)                                  # a full frame drops the match of the step before it
                tensors = runner.step(frames[t], force_full=force, next_frames=nxt)
            runner.reset()                                           # the last match was for a frame that never comes
            runner.step(frames[0])
            tensors = runner.step(frames[1])
            torch.cuda.synchronize()
            kept.append([x.clone() for x in tensors[1:]] + [runner.mask.clone(), runner.gmv.clone(), runner.mv.clone()])
        finals[look] = kept
        del runner
    for f, (a, b) in enumerate(zip(finals[True], finals[False])):
        assert all(torch.equal(x, y) for x, y in zip(a[-3:], b[-3:])), f
        assert int(a[-3].sum()) > 0
        for i, (x, y) in enumerate(zip(a[:-3], b[:-3])):
            assert _max_rel(x, y) <= 3e-4, (f, i)


def _max_rel(a, b):
    a, b = a.float(), b.float()
    return float((a - b).abs().max() / b.abs().max().clamp_min(1e-30))


@pytest.mark.parametrize("net,plan", [("vgg", dict(torus=True)), ("googlenet", {}), ("resnet", dict(cache_pool_add=True))])
def test_long_pipelined_runs_stay_with_the_plain_path(net, plan):
    """Pipelined frames planned on the GPU over a run long enough for the stages to be cut anew from measured times, launched
    or replayed as measured and replayed throughout: the tensors of the last frame of runs that end at different places are
    those of the plain path (one stream, no handle), which takes neither.  fp32; the lists' lengths are known to the launches
    with different delays, so partial sums of a split K may be added in another grouping: K <= 4608 products, relative
    error of a sum up to sqrt(K) 2^-24 per layer, over at most 60 layers below 3e-4."""
    H = W = 96
    if net == "vgg":
        layers = synth.small_vgg()
    elif net == "googlenet":
        layers = synth.resolve_global_pooling(synth.googlenet(n_classes=40, width=0.25), H, W, 3)
    else:
        layers = synth.resnet50_trunk()[:44]
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, residual_scale=0.5, input_shape=(H, W, 3))
    T = 12
    video = torch.from_numpy(synth.panning_video(83, n_frames=T, H=H, W=W, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    finals = {}
    for mode, kw in (("pipeline", dict(overlap=True, pipeline=True)), ("replayed", dict(overlap=True, pipeline=True)), ("plain", dict(overlap=False))):
        print(f"[long run] {net} {mode}", flush=True)
        runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=16, dtype=binding.DC_F32, expiry=6,
                                     device_plan=True, exact_masks=True, want_origins=False, **plan, **kw)
        if mode == "replayed":
            runner.set_replay(1)
        kept = []
        for stop in (5, 61, 90, 11):
            runner.reset()
            for t in range(stop):
                if t % T == 0:
                    runner.reset()
                tensors = runner.step(frames[t % T])
            last = [runner.read_tensor(i, tensors) if (not runner.torus or runner.layers[i - 1]["type"] == synth.CONV) else tensors[i]
                    for i in range(1, len(layers) + 1)]
            torch.cuda.synchronize()
            kept.append([x.clone() for x in last] + [runner.mask.clone(), runner.gmv.clone()])
        finals[mode] = kept
        if mode == "replayed":
            c = runner.overlap_counters()
            assert c.failed == 0 and c.replayed > c.frames // 3, [(n, getattr(c, n)) for n, _ in c._fields_]
        del runner
    for mode in ("pipeline", "replayed"):
        for f, (a, b) in enumerate(zip(finals[mode], finals["plain"])):
            assert torch.equal(a[-1], b[-1]) and torch.equal(a[-2], b[-2]), (mode, f)
            for i, (x, y) in enumerate(zip(a[:-2], b[:-2])):
                assert _max_rel(x, y) <= 3e-4, (mode, f, i)


def _replay_run(layers, ws, bs, frames, block, bf16, mode, order, before=None, **kw):
    """A runner whose frames are replayed from graphs always (1), never (0) or that has no handle (None), over `order`
    (frame index, or None: drop the cache); clones of the last frame's tensors, the mask and the motion after every None."""
    H, W = frames[0].shape[1:3]
    runner = binding.StackRunner(layers, ws, bs, frames[0].shape[0], H, W, 3, block=block, radius=block,
                                 dtype=binding.DC_BF16 if bf16 else binding.DC_F32, device_plan=True, exact_masks=True,
                                 overlap=mode is not None, **kw)
    if mode is not None:
        runner.set_replay(mode)
    kept, tensors = [], None
    on_torus = [runner.torus and (L["type"] == synth.CONV or (runner.cache_pool_add and L["type"] == synth.MAXPOOL)) for L in runner.layers]
    for j, t in enumerate(order):
        if before is not None:
            before(j, runner)
        if t is not None:
            tensors = runner.step(frames[t])
            continue
        last = [runner.read_tensor(i, tensors) if on_torus[i - 1] else tensors[i] for i in range(1, len(layers) + 1)]
        torch.cuda.synchronize()
        kept.append([x.clone() for x in last] + [runner.mask.clone(), runner.gmv.clone()])
        runner.reset()
    counters = runner.overlap_counters() if mode is not None else None
    return kept, counters, list(runner._kid)


@pytest.mark.parametrize("net,size,kw", [("vgg16", 224, dict(torus=True)), ("vgg16", 96, {}), ("darknet19", 96, dict(torus=True)),
                                         ("darknet19", 224, {})])
def test_replayed_frames_are_the_launched_ones(net, size, kw):
    """Frames replayed from recorded graphs, frames launched kernel by kernel and frames without a handle: every tensor bit
    for bit, several replays of every graph, full frames and cached ones, other work of the program and synchronisations in
    between.  (The launch shapes are fixed: units per workgroup and no split of K.)"""
    _check_replays(net, size, kw, 4)


@pytest.mark.parametrize("net,size,kw", [("darknet19", 96, dict(torus=True)), ("darknet19", 224, {})])
def test_replayed_frames_with_1x1_layers_that_split_k(net, size, kw):
    """The same with two units per workgroup: no tile of the 1x1 layers, which choose their kernel by the size of their maps."""
    kernels = {binding.conv_kernel_name(k) for k in _check_replays(net, size, kw, 2) if k >= 0}
    assert any(k.startswith("conv_pw_split_kernel") for k in kernels), kernels


def _check_replays(net, size, kw, units):
    print(f"[replay] {net} {size} {kw} {units}", flush=True)
    layers = synth.resolve_global_pooling(synth.vgg16()[:18] if net == "vgg16" else synth.darknet19()[:19], size, size, 3)
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(size, size, 3))
    T = 10
    video = torch.from_numpy(synth.panning_video(87, n_frames=T, H=size, W=size, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    order = (list(range(T)) + [None]) * 4 + [0, 1, 2, None, 0, None] + (list(range(T)) + list(range(T - 1, -1, -1)) + [None]) * 2
    binding.dc_conv_tuning(0, units, 1, 0)
    try:
        runs = {mode: _replay_run(layers, ws, bs, frames, 16, False, mode, order, **kw) for mode in (1, 0, None)}
    finally:
        binding.dc_conv_tuning()
    c = runs[1][1]
    steps = sum(t is not None for t in order)
    assert c.frames == steps and c.failed == 0 and c.recorded >= 4 and c.replayed >= steps // 3, [(n, getattr(c, n)) for n, _ in c._fields_]
    assert runs[0][1].replayed == runs[0][1].recorded == 0
    if size == 224:
        assert c.stages > 1
    assert int(runs[0][0][0][-2].sum()) > 0
    for other in (0, None):
        for f, (a, b) in enumerate(zip(runs[1][0], runs[other][0])):
            for i, (x, y) in enumerate(zip(a, b)):
                assert torch.equal(x, y), (other, f, i)
    return runs[0][2]


def test_replayed_frames_follow_a_change_of_the_launch_shapes():
    """dc_conv_tuning holds for replayed frames too: a graph recorded before the change is not replayed after it (the kernels
    of the layers are reported as they are launched), and the one recorded before is replayed again afterwards."""
    layers = synth.vgg16()[:10]
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(96, 96, 3))
    video = torch.from_numpy(synth.panning_video(88, n_frames=8, H=96, W=96, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(8)]
    torch.cuda.synchronize()
    ids, seen = {}, []

    def before(j, runner):
        if j % 40 == 0:
            binding.dc_conv_tuning(*((1, 4, 1, 0) if j // 40 % 2 == 0 else (2, 4, 1, 0)))
        if j % 40 == 39:
            seen.append(runner.overlap_counters().replayed)
            ids[j // 40] = list(runner._kid)
    order = list(range(8)) * 20
    try:
        _replay_run(layers, ws, bs, frames, 16, True, 1, order, before=before)
    finally:
        binding.dc_conv_tuning()
    names = [[binding.conv_kernel_name(v) for v in ids[k] if v >= 0] for k in range(4)]
    print("[replay tuning]", names[0][-1], names[1][-1], seen, flush=True)
    assert names[0] != names[1] and names[0] == names[2] and names[1] == names[3]
    assert all(b > a for a, b in zip([0] + seen, seen))


def test_recordings_are_dropped_and_evicted():
    """A recording whose lists have become much longer is given up and made anew, and the seventeenth recording of a stack
    drives the least recently used one out: same tensors as without replay all the while."""
    layers = synth.vgg16()[:10]
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(96, 96, 3))
    rng = np.random.default_rng(9)
    still = rng.integers(0, 256, (1, 96, 96, 3), np.uint8)
    noise = [rng.integers(0, 256, (1, 96, 96, 3), np.uint8) for _ in range(4)]
    part = [still.copy() for _ in range(4)]
    for k, p in enumerate(part):
        p[0, 8 * k:8 * k + 24, 30:60] = noise[k][0, :24, :30]            # a moving object over a still picture
    frames = [torch.from_numpy(v).to(DEV) for v in part + noise]
    torch.cuda.synchronize()
    order = [j % 4 for j in range(60)] + [None] + [4 + j % 4 for j in range(90)] + [j % 4 for j in range(20)] + [None] + \
            [j % 4 for j in range(7 * 16)] + [None]
    results = {}
    copies = [[torch.from_numpy(b).to(DEV) if b is not None else None for b in bs] for _ in range(7)]     # the same values elsewhere: other keys
    torch.cuda.synchronize()
    tail = len(order) - 7 * 16 - 1

    def before(j, runner):
        if j >= tail and (j - tail) % 16 == 0 and order[j] is not None:
            runner._bp = (ctypes.c_void_p * len(layers))(*[None if b is None else b.data_ptr() for b in copies[(j - tail) // 16]])
    for mode in (1, 0):
        binding.dc_conv_tuning(0, 4, 1, 0)
        try:
            results[mode] = _replay_run(layers, ws, bs, frames, 16, False, mode, order, before=before)
        finally:
            binding.dc_conv_tuning()
    c = results[1][1]
    print("[dropped, evicted]", [(n, getattr(c, n)) for n, _ in c._fields_], flush=True)
    assert c.failed == 0 and c.dropped >= 1 and c.evicted >= 1 and c.replayed > 20
    for f, (a, b) in enumerate(zip(results[1][0], results[0][0])):
        for i, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x, y), (f, i)


def test_a_recording_is_dropped_for_one_layer_alone():
    """Two layers that are always computed in full hold most of the units; the lists of the others grow from a few units to
    everything.  Their launches are not kept for that reason (in the sum over the layers it is less than a quarter)."""
    layers = synth.vgg16()[:10]
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(96, 96, 3))
    rng = np.random.default_rng(10)
    still = rng.integers(0, 256, (1, 96, 96, 3), np.uint8)
    part = [still.copy() for _ in range(4)]
    for k, p in enumerate(part):
        p[0, 8 * k:8 * k + 8, 30:40] = rng.integers(0, 256, (8, 10, 3), np.uint8)
    frames = [torch.from_numpy(v).to(DEV) for v in part + [rng.integers(0, 256, (1, 96, 96, 3), np.uint8) for _ in range(4)]]
    torch.cuda.synchronize()
    order = [j % 4 for j in range(60)] + [4 + j % 4 for j in range(90)] + [None]
    flags = np.array([1, 1] + [0] * (len(layers) - 2), np.uint8)
    binding.dc_conv_tuning(0, 4, 1, 0)
    try:
        results = {mode: _replay_run(layers, ws, bs, frames, 16, False, mode, order, no_reuse=flags) for mode in (1, 0)}
    finally:
        binding.dc_conv_tuning()
    c = results[1][1]
    print("[dropped for one layer]", [(n, getattr(c, n)) for n, _ in c._fields_], flush=True)
    assert c.failed == 0 and c.dropped >= 1 and c.recorded > c.dropped
    for x, y in zip(results[1][0][0], results[0][0][0]):
        assert torch.equal(x, y)


def test_frames_of_more_blocks_than_the_gpu_plans_run_as_host_planned():
    """A frame of more than 64 blocks per row is planned on the host whatever device_plan says: same tensors bit for bit as
    without the option, and the same pipeline: no stage of layers on the stream of the matching, which the host waits for."""
    H, W, T = 96, 16 * 66, 9
    layers = synth.vgg16()
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(H, W, 3))
    video = torch.from_numpy(synth.panning_video(89, n_frames=T, H=H, W=W, fg=((24, 24), (32, 160)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    results = {}
    for dp in (False, True):
        print(f"[66 blocks] device_plan={dp}", flush=True)
        runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=8, dtype=binding.DC_F32, expiry=6, device_plan=dp,
                                     exact_masks=dp)
        kept = []
        for t in range(T):
            tensors = runner.step(frames[t])
            if t in (2, T - 1):
                torch.cuda.synchronize()
                assert runner.stats.n_reusable_blocks > 0
                kept.append([x.clone() for x in tensors[1:]] + [runner.mask.clone()])
        results[dp] = kept, runner.overlap_counters().stages
        del runner
    assert results[True][1] == results[False][1] <= 3, (results[True][1], results[False][1])
    for a, b in zip(results[True][0], results[False][0]):
        for i, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x, y), i


def test_short_stacks_are_cut_into_few_stages():
    """A stage costs the host about 30 us per frame: a stack of under 150 us on the GPU is not cut into four (it was, and
    ran slower than without stages), a longer one is."""
    stages = {}
    for net, H, W in (("dave", 66, 200), ("resnet50", 224, 224)):
        layers = synth.resolve_global_pooling(synth.dave_orig() if net == "dave" else synth.resnet50_trunk(), H, W, 3)
        ws, bs = synth.he_weights(layers, 3, residual_scale=0.5, input_shape=(H, W, 3))
        video = torch.from_numpy(synth.panning_video(90, n_frames=8, H=H, W=W, fg=((16, 16),))).to(DEV)
        frames = [video[t:t + 1].contiguous() for t in range(8)]
        torch.cuda.synchronize()
        runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=16, dtype=binding.DC_F32, device_plan=True, exact_masks=True)
        for t in range(48):
            if t % 8 == 0:
                runner.reset()
            runner.step(frames[t % 8])
        torch.cuda.synchronize()
        stages[net] = runner.overlap_counters().stages
        del runner
    print("[stages]", stages, flush=True)
    assert stages["dave"] <= 3 and stages["resnet50"] == 4


@pytest.mark.parametrize("net,size,streams", [("vgg16", 224, 1), ("vgg16", 160, 3), ("darknet19", 224, 2)])
def test_stages_across_tensors_with_a_single_buffer(net, size, streams):
    """Convolutions and poolings on the torus: every tensor is one buffer, and a stage starts with the only reader of what the
    stage before it wrote; the next frame's writer waits for that reader.  Several stages, no synchronisation between the frames
    of a run: every tensor bit for bit that of the path without a handle (fixed launch shapes)."""
    print(f"[tight stages] {net} {size} x{streams}", flush=True)
    layers = synth.vgg16()[:18] if net == "vgg16" else synth.darknet19()[:17]
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(size, size, 3))
    T = 10
    videos = [synth.panning_video(91 + s, n_frames=T, H=size, W=size, fg=((24, 24), (16, 32))) for s in range(streams)]
    frames = [torch.from_numpy(np.stack([v[t] for v in videos])).to(DEV) for t in range(T)]
    torch.cuda.synchronize()
    order = (list(range(T)) + [None]) * 3 + [0, 1, 2, 3, None] + (list(range(T)) + list(range(T - 1, -1, -1)) + [None]) * 2
    binding.dc_conv_tuning(0, 4, 1, 0)
    try:
        runs = {mode: _replay_run(layers, ws, bs, frames, 16, False, mode, order, torus=True, cache_pool_add=True) for mode in (1, None)}
    finally:
        binding.dc_conv_tuning()
    c = runs[1][1]
    assert c.stages > 1 and c.replayed == c.recorded == 0, [(n, getattr(c, n)) for n, _ in c._fields_]
    assert int(runs[1][0][0][-2].sum()) > 0
    for f, (a, b) in enumerate(zip(runs[1][0], runs[None][0])):
        for i, (x, y) in enumerate(zip(a, b)):
            assert torch.equal(x, y), (f, i)


def test_the_callers_own_work_shortens_the_last_stage():
    """The last stage shares the caller's stream with what the caller queues there behind every frame: with much of it (16
    passes over 64 MiB) the last stage is cut shorter than without, and the tensors are the same bit for bit."""
    layers = synth.vgg16()
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(224, 224, 3))
    video = torch.from_numpy(synth.panning_video(94, n_frames=8, H=224, W=224, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(8)]
    work = torch.zeros(64 << 20, dtype=torch.uint8, device=DEV)
    torch.cuda.synchronize()
    results = {}
    binding.dc_conv_tuning(0, 4, 1, 0)
    try:
        for passes in (0, 16):
            runner = binding.StackRunner(layers, ws, bs, 1, 224, 224, 3, block=16, radius=16, dtype=binding.DC_F32, device_plan=True,
                                         exact_masks=True, torus=True)
            for t in range(48):
                if t % 8 == 0:
                    runner.reset()
                tensors = runner.step(frames[t % 8])
                for _ in range(passes if t < 47 else 0):
                    work.add_(1)
            last = [runner.read_tensor(i + 1, tensors) for i, L in enumerate(layers) if L["type"] == synth.CONV]
            torch.cuda.synchronize()
            results[passes] = runner.overlap_counters(), [x.clone() for x in last] + [tensors[-1].clone(), runner.mask.clone()]
            del runner
    finally:
        binding.dc_conv_tuning()
    print("[last stage]", {k: (v[0].stages, v[0].last_layers) for k, v in results.items()}, flush=True)
    assert results[16][0].last_layers < results[0][0].last_layers
    for i, (x, y) in enumerate(zip(results[0][1], results[16][1])):
        assert torch.equal(x, y), i


def test_one_long_wait_in_the_callers_work_does_not_decide_the_cut():
    """Of the four frames that are timed after a cut one has 10 ms of the caller's work behind it, the others none: the layers are
    cut anew from the times of their stages as without it."""
    layers = synth.resolve_global_pooling(synth.dave_orig(), 66, 200, 3)
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(66, 200, 3))
    video = torch.from_numpy(np.stack([synth.panning_video(94 + s, n_frames=8, H=66, W=200, fg=((24, 24), (16, 32))) for s in range(16)], 1)).to(DEV)
    frames = [video[t].contiguous() for t in range(8)]
    torch.cuda.synchronize()
    cuts = {}
    for wait in (False, True, False):
        runner = binding.StackRunner(layers, ws, bs, 16, 66, 200, 3, block=16, radius=16, dtype=binding.DC_BF16, device_plan=True, exact_masks=True)
        for t in range(40):
            if t % 8 == 0:
                runner.reset()
            runner.step(frames[t % 8])
            if t == 0 or (wait and t == 1):                # (behind the first, full frame: the timed ones still run at the next call)
                torch.cuda._sleep(24_000_000)
        torch.cuda.synchronize()
        c = runner.overlap_counters()
        print(f"[one wait] {wait}: {c.recuts} recuts, {c.stages} stages, {c.last_layers} layers in the last", flush=True)
        cuts.setdefault(wait, []).append(c.recuts)
        del runner
    assert cuts[True][0] >= 1 or 0 in cuts[False], cuts     # (the first cut could be as good as it gets on another host)


def test_one_handle_for_two_stacks_and_two_caller_streams():
    """A handle that is handed from one stack to another and called on changing streams orders every frame behind the
    earlier ones: same tensors as with a handle of their own.  (Stages of different stacks use the same streams, and the
    last stage runs on the caller's.)"""
    H = W = 96
    stacks = [synth.small_vgg(), synth.vgg16()[:10]]
    T = 10
    video = torch.from_numpy(synth.panning_video(84, n_frames=T, H=H, W=W, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    torch.cuda.synchronize()

    def make():
        return [binding.StackRunner(L, *synth.he_weights(L, 3, bias_scale=0.05), 1, H, W, 3, block=16, radius=16,
                                    dtype=binding.DC_F32, expiry=6) for L in stacks]
    want = []
    for r in make():
        for t in range(T):
            tensors = r.step(frames[t])
        torch.cuda.synchronize()
        want.append([x.clone() for x in tensors])
    runners = make()
    own = runners[1].overlap
    runners[1].overlap = runners[0].overlap
    try:
        for t in range(T):
            for k, r in enumerate(runners):
                with torch.cuda.stream(streams[(t // 3 + k) % 2]):
                    tensors = r.step(frames[t])
                if t == T - 1:
                    torch.cuda.synchronize()
                    for i, (x, y) in enumerate(zip(tensors, want[k])):
                        assert torch.equal(x, y), (k, i)
    finally:
        torch.cuda.synchronize()
        runners[1].overlap = own


def test_two_threads_with_a_stack_each():
    """Handles of two threads share the stage streams of the GPU, and both threads record graphs while the other one issues
    frames: same tensors as one after the other.  (A recording takes nothing but its own stack's launches.)"""
    H = W = 96
    T = 12
    layers = synth.resnet50_trunk()[:44]
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, residual_scale=0.5)
    video = torch.from_numpy(synth.panning_video(85, n_frames=T, H=H, W=W, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [[video[t:t + 1].contiguous() for t in range(T)], [video[T - 1 - t:T - t].contiguous() for t in range(T)]]
    torch.cuda.synchronize()
    results, errors = {}, []

    def work(key, mine):
        try:
            torch.cuda.set_device(0)
            with torch.cuda.stream(torch.cuda.Stream()):
                runner = binding.StackRunner(layers, ws, bs, 1, H, W, 3, block=16, radius=16, dtype=binding.DC_F32, expiry=6,
                                             device_plan=True, exact_masks=True)
                runner.set_replay(1)
                for t in range(10 * T):
                    if t % T == 0:
                        runner.reset()
                    tensors = runner.step(mine[t % T])
                torch.cuda.current_stream().synchronize()
                c = runner.overlap_counters()
                assert c.failed == 0 and c.recorded >= 4 and c.replayed > 10, [(n, getattr(c, n)) for n, _ in c._fields_]
                results[key] = [x.clone() for x in tensors[1:]] + [runner.mask.clone(), runner.gmv.clone()]
                torch.cuda.current_stream().synchronize()
        except Exception as e:                       # noqa: BLE001 (reported by the main thread)
            errors.append(e)
    for k in range(2):
        print(f"[threads] alone {k}", flush=True)
        work(("alone", k), frames[k])
    print("[threads] together", flush=True)
    threads = [threading.Thread(target=work, args=(("together", k), frames[k])) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not errors, errors
    for k in range(2):
        a, b = results["alone", k], results["together", k]
        assert torch.equal(a[-1], b[-1]) and torch.equal(a[-2], b[-2]), k
        for i, (x, y) in enumerate(zip(a[:-2], b[:-2])):
            assert _max_rel(x, y) <= 3e-4, (k, i)    # (partial sums of a split K: see the test of long runs)


# Counters of earlier frames tune the launches of a frame planned on the GPU, and they are there or not as it happens.  Some rules
# that follow them change the order of sums (a split K, the channel chunk); these layers keep to one order over the lengths here.
_HINTED = {"3x3": [(64, 3, 1, 1), (32, 3, 1, 1), (64, 3, 1, 1)],      # [(cout, k, s, p)]
           "1x1": [(64, 3, 1, 1), (256, 1, 1, 0), (128, 1, 1, 0), (512, 1, 1, 0), (64, 1, 1, 0)]}


@pytest.mark.parametrize("bf16", [False, True])
@pytest.mark.parametrize("name", list(_HINTED))
def test_outputs_do_not_depend_on_the_counters_of_earlier_frames(name, bf16):
    """The first clip of a runner has no counters for its first reused frame, the second clip has those of the first: the same bits."""
    n, H, W, T = 1, 64, 64, 4
    layers, cin = [], 3
    for cout, k, s, p in _HINTED[name]:
        layers.append(dict(type=synth.CONV, k=k, s=s, p=p, cin=cin, cout=cout, relu=1, in0=len(layers), in1=-1))
        cin = cout
    ws, bs = synth.he_weights(layers, 5, bias_scale=0.05, input_shape=(H, W, 3))
    rng = np.random.default_rng(3)
    back = synth._box_blur5(rng.integers(0, 256, (H, W, 3)).astype(np.uint8))
    video = np.stack([back] * T)
    for t in range(T):                                # a still picture with one moving square of noise
        video[t, 4:16, 4 + 2 * t:16 + 2 * t] = rng.integers(0, 256, (12, 12, 3))
    video = torch.from_numpy(video[:, None]).to(DEV)
    runner = binding.StackRunner(layers, ws, bs, n, H, W, 3, block=8, radius=8, dtype=binding.DC_BF16 if bf16 else binding.DC_F32,
                                 expiry=T, device_plan=True, exact_masks=True)
    clips = []
    for clip in range(3):
        frames = []
        for t in range(T):
            print(f"[counters] {name} bf16={bf16} clip {clip} frame {t}", flush=True)
            tensors = runner.step(video[t])
            torch.cuda.synchronize()
            assert runner.last_full == (t == 0)
            if t:
                assert float(runner.mask.float().mean()) >= 0.6      # the list is a fraction of the map
            frames.append([x.clone() for x in tensors])
        clips.append(frames)
    for clip in clips[1:]:
        for t in range(T):
            for i in range(len(layers) + 1):
                assert torch.equal(clip[t][i], clips[0][t][i]), (name, t, i)


@pytest.mark.parametrize("cout,kernel", [(32, "conv_pw_split_kernel<1, 2, 4>"), (40, "conv_pw_split_kernel<2, 2, 4>"),
                                         (128, "conv_pw_split_kernel<2, 2, 4>"), (136, "conv_pw_kernel<float, 2>")])
def test_kernel_of_a_1x1_layer_follows_the_size_of_its_map(cout, kernel):
    """256 units: at most 256 tiles of one unit x 32 channels, at most 512 of two, or the ring, in full frames and in quiet ones."""
    print(f"[1x1 rule] cout={cout}", flush=True)
    layers = [dict(type=synth.CONV, k=1, s=1, p=0, cin=3, cout=cout, relu=1, in0=0, in1=-1)]
    ws, bs = synth.he_weights(layers, 5, bias_scale=0.05, input_shape=(64, 64, 3))
    frame = torch.from_numpy(np.random.default_rng(1).integers(0, 256, (1, 64, 64, 3)).astype(np.uint8)).to(DEV)
    for dtype, want in ((binding.DC_F32, kernel), (binding.DC_BF16, "conv_pw_kernel<__hip_bfloat16, 2>")):
        runner = binding.StackRunner(layers, ws, bs, 1, 64, 64, 3, block=8, radius=8, dtype=dtype, expiry=4, device_plan=True, exact_masks=True)
        for t in range(4):
            runner.step(frame)
            torch.cuda.synchronize()
            assert runner.last_full == (t == 0)
            assert binding.conv_kernel_name(runner.layer_stats()["kernel_id"][0]) == want, t


@pytest.mark.parametrize("units,width", [(8, -1), (7, 2)])
def test_torus_through_the_kernel_with_weights_in_registers(oracle, units, width):
    """Tensors on a torus, lists built on the GPU, through the bf16 kernel whose weights go straight to registers."""
    video = np.stack([synth.panning_video(7100 + s, n_frames=5, H=96, W=96, fg=((24, 24),), margin=32) for s in range(3)])
    layers = [dict(type=synth.CONV, k=3, s=1, p=1, cin=3, cout=64, relu=1, in0=0, in1=-1),
              dict(type=synth.CONV, k=3, s=1, p=1, cin=64, cout=256, relu=1, in0=1, in1=-1),
              dict(type=synth.CONV, k=3, s=1, p=1, cin=256, cout=128, relu=1, in0=2, in1=-1),
              dict(type=synth.CONV, k=3, s=1, p=1, cin=128, cout=256, relu=1, in0=3, in1=-1)]
    binding.dc_conv_tuning(5, units, width)
    try:
        runner, reuse = _run_one(oracle, layers, video, 16, 16, True, device_plan=True, exact_masks=True, torus=True, resets=(3,),
                                 bias_scale=0.02)
        names = [binding.conv_kernel_name(k) for k in runner.layer_stats()["kernel_id"][1:]]
    finally:
        binding.dc_conv_tuning()
    assert names == [f"conv_deep_kernel<{2 if width == 2 or c == 128 else 4}, {units}>" for c in (256, 128, 256)] and max(reuse) > 0.3


# Stems of bf16 stacks, whose input patch goes through LDS with four channels a pixel: 7x7 and the three widths of 11x11, frames
# of three and four channels, more units than a launch has workgroups (the walk over the list) and fewer, ragged maps.
@pytest.mark.parametrize("k,s,p,cout,C,n,H,W,kid", [
    (7, 2, 3, 64, 3, 3, 224, 224, 0), (7, 2, 3, 128, 4, 1, 61, 83, 0), (7, 2, 0, 64, 3, 2, 64, 48, 0),
    (11, 4, 0, 96, 3, 4, 227, 227, 3), (11, 4, 2, 192, 4, 1, 70, 99, 3), (11, 4, 2, 64, 3, 2, 64, 80, 2), (11, 4, 5, 32, 3, 3, 96, 64, 1)])
def test_stems_with_four_channels_a_pixel(oracle, k, s, p, cout, C, n, H, W, kid):
    video = np.stack([synth.panning_video(7300 + i, n_frames=3, H=H, W=W, fg=((24, 24),), margin=32) for i in range(n)])
    if C == 4:
        video = np.concatenate([video, video[..., :1] ^ 85], axis=-1)
    layers = [dict(type=synth.CONV, k=k, s=s, p=p, cin=C, cout=cout, relu=1, in0=0, in1=-1)]
    binding.dc_conv_tuning(-1, 4, -1, -1)           # (few units: a 7x7 layer would take the other kernel)
    try:
        runner, reuse = _run_one(oracle, layers, video, 16, 8, True, device_plan=True, exact_masks=True, bias_scale=0.1)
        kernel_id = runner.layer_stats()["kernel_id"][0]
    finally:
        binding.dc_conv_tuning()
    assert max(reuse) > 0.2
    assert binding.conv_kernel_name(kernel_id) == \
        ("conv_stem4_kernel<7, 2, 4, 1, 4>" if k == 7 else f"conv_stem4_kernel<11, 4, 2, {kid}, 1>")


@pytest.mark.parametrize("k,s,p,cout,C,n,H,W", [
    (7, 2, 3, 64, 3, 8, 224, 224), (7, 2, 3, 128, 4, 5, 301, 203), (7, 2, 0, 64, 1, 2, 64, 48),
    (11, 4, 0, 96, 3, 6, 227, 227), (11, 4, 2, 192, 4, 3, 170, 199), (11, 4, 2, 64, 3, 8, 224, 224), (11, 4, 5, 32, 2, 9, 196, 264)])
def test_both_stem_kernels_give_the_same_bits(k, s, p, cout, C, n, H, W):
    """Frames through the kernel with the patch in LDS and through the other, and the layer alone over all eight channels of a
    pixel: the same sums in the same order, so the same bits.  Channel 0 has an infinite weight, channel 1 nothing but
    zeros of both signs and a bias of -0."""
    layers = [dict(type=synth.CONV, k=k, s=s, p=p, cin=C, cout=cout, relu=0, in0=0, in1=-1)]
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.1)
    w = np.array(ws[0], np.float32).reshape(cout, k, k, C)
    b = np.array(bs[0], np.float32)
    w[0, 1, 2, 0] = np.inf
    w[1], b[1] = np.where(np.arange(k * k * C).reshape(k, k, C) % 2, -0.0, 0.0), -0.0
    video = np.stack([synth.panning_video(7700 + i, n_frames=3, H=H, W=W, fg=((24, 24),), margin=32) for i in range(n)])
    video = np.concatenate([video, video[..., :1] ^ 85], axis=-1)[..., :C]
    dev = torch.from_numpy(np.ascontiguousarray(video.transpose(1, 0, 2, 3, 4))).to(DEV)
    runs = {}
    for units in (1, 4):
        binding.dc_conv_tuning(-1, units, -1, -1)
        try:
            runner = binding.StackRunner(layers, [w.reshape(ws[0].shape)], [b], n, H, W, C, block=16, radius=8, dtype=binding.DC_BF16,
                                         device_plan=True, exact_masks=True)
            frames = []
            for t in range(3):
                print(f"[stems] k={k} cout={cout} C={C} n={n} {H}x{W} units={units} frame {t}", flush=True)
                got = runner.step(dev[t])
                torch.cuda.synchronize()
                frames.append((got[0].clone(), got[1].clone()))
            name = binding.conv_kernel_name(runner.layer_stats()["kernel_id"][0])
        finally:
            binding.dc_conv_tuning()
        assert name.startswith("conv_stem4_kernel" if units == 4 else f"conv_stem{11 if k == 11 else ''}_kernel"), name
        runs[units] = frames
    for t in range(3):
        assert torch.equal(runs[1][t][1].view(torch.int16), runs[4][t][1].view(torch.int16)), t
    wide = np.zeros((cout, k, k, 8), np.float32)
    wide[..., :C] = w
    alone = binding.dc_cached_conv_layer(dict(layers[0], cin=8), runs[4][0][0], torch.from_numpy(wide).bfloat16().to(DEV), torch.from_numpy(b).to(DEV))
    assert torch.equal(alone.view(torch.int16), runs[4][0][1].view(torch.int16))


def test_stem_kernel_follows_the_number_of_units():
    """7x7 in bf16: the kernel with the patch in LDS from about 6000 units of 64 channels on, on lists from 3000."""
    few, many = "conv_stem_kernel<__hip_bfloat16, 2>", "conv_stem4_kernel<7, 2, 4, 1, 4>"
    for n, cout, full, cached in ((2, 64, few, few), (7, 64, few, many), (8, 64, many, many), (4, 128, many, many)):
        layers = [dict(type=synth.CONV, k=7, s=2, p=3, cin=3, cout=cout, relu=1, in0=0, in1=-1)]
        ws, bs = synth.he_weights(layers, 3)
        runner = binding.StackRunner(layers, ws, bs, n, 224, 224, 3, dtype=binding.DC_BF16, device_plan=True, exact_masks=True, no_reuse=[1])
        for want in (full, cached):         # (a layer outside the cache: its list names every unit)
            runner.step(torch.zeros((n, 224, 224, 3), dtype=torch.uint8, device=DEV))
            torch.cuda.synchronize()
            assert binding.conv_kernel_name(runner.layer_stats()["kernel_id"][0]) == want, (n, cout)


@pytest.mark.parametrize("bf16,n,units", [(True, 1, -1), (True, 3, -1), (False, 12, -1), (True, 1, 8), (True, 3, 8), (False, 3, 8)])
def test_sums_written_by_the_convolution_before_them(bf16, n, units):
    """A residual block's sum is written by the 1x1 convolution before it; with a profile attached it is a launch of its own.
    The same bits, in full frames and in cached ones (units without work, units with some reusable pixels, layers outside the
    cache); the 64 x 64 tile and the 128 x 128 one, which so few units would not choose."""
    try:
        binding.dc_conv_tuning(-1, units, -1, -1)
        _check_sums(bf16, n, f"conv_pw_add_kernel<{'__hip_bfloat16' if bf16 else 'float'}, {4 if units == 8 else 2}>")
    finally:
        binding.dc_conv_tuning()


def _check_sums(bf16, n, kernel):
    layers = synth.resnet50_trunk()[:24]
    H = W = 96
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, residual_scale=0.5, input_shape=(H, W, 3))
    video = np.stack([synth.panning_video(7400 + s, n_frames=4, H=H, W=W, fg=((24, 24),), margin=32) for s in range(n)])
    dev = torch.from_numpy(np.ascontiguousarray(video.transpose(1, 0, 2, 3, 4))).to(DEV)
    flags = np.zeros(len(layers), np.uint8)
    flags[4] = 1
    for no_reuse in (None, flags):
        runs = []
        for profile in (False, True):
            runner = binding.StackRunner(layers, ws, bs, n, H, W, 3, block=16, radius=16, device_plan=True, exact_masks=True, overlap=False,
                                         dtype=binding.DC_BF16 if bf16 else binding.DC_F32, no_reuse=no_reuse)
            runner.enable_profile(profile)
            frames = []
            for t in range(4):
                print(f"[sums] {kernel} n={n} profile={profile} frame {t}", flush=True)
                got = runner.step(dev[t])
                torch.cuda.synchronize()
                names = {binding.conv_kernel_name(k) for k in runner.layer_stats()["kernel_id"] if k >= 0}
                sums = {v for v in names if v.startswith("conv_pw_add_kernel")}
                assert sums == (set() if profile else {kernel}), (t, names)
                frames.append([x.clone() for x in got])
            runs.append((frames,))
        for t in range(4):
            for i, (a, b) in enumerate(zip(runs[0][0][t], runs[1][0][t])):
                assert torch.equal(a, b), (t, i)


@pytest.mark.parametrize("torus", [False, True])
@pytest.mark.parametrize("H,W", [(52, 52), (56, 40)])
def test_whole_map_kernel_in_cached_frames(oracle, H, W, torus):
    """Maps of 13x13 and 14x10 in frames planned on the GPU, some of whose pixels come from the cache, through the kernel that
    takes whole maps: reusable pixels keep their values (oracle), on a torus as well."""
    video = np.stack([synth.panning_video(7500 + s, n_frames=5, H=H, W=W, fg=((12, 12),), margin=32) for s in range(3)])
    layers = synth._chain([("c", 64, 3, 1, 1), ("p", 2, 2, 0), ("c", 64, 3, 1, 1), ("p", 2, 2, 0), ("c", 128, 3, 1, 1), ("c", 64, 3, 1, 1)], 3)
    convs = [i for i, L in enumerate(layers) if L["type"] == synth.CONV][-2:]
    binding.dc_conv_tuning(6, 4, -1, -1)
    try:
        runner, reuse = _run_one(oracle, layers, video, 4, 8, True, device_plan=True, exact_masks=True, torus=torus, resets=(2,), bias_scale=0.02)
        stats = runner.layer_stats()
    finally:
        binding.dc_conv_tuning()
    upw = (((H // 4) * (W // 4) + 15) // 16 + 3) // 4
    assert [binding.conv_kernel_name(stats["kernel_id"][i]) for i in convs] == [f"conv_map_kernel<{upw}, 4>", f"conv_map_kernel<{upw}, 2>"]
    assert runner.read_stats() and runner.layer_stats()["reused_px"][convs[0]] > 0


@pytest.mark.parametrize("device_plan", [True, False])
@pytest.mark.parametrize("bf16,n,units", [(True, 1, -1), (True, 6, -1), (False, 40, -1), (True, 1, 8), (True, 3, 8), (False, 3, 4), (False, 3, 8)])
def test_pointwise_layers_of_one_tensor_in_one_launch(bf16, n, units, device_plan):
    """The three 1x1 convolutions of an inception module that read the module's input go out as one launch; with a profile
    attached they are three.  The same bits in full frames and in cached ones, with the stem outside the cache or not; the
    64 x 64 tile and the 128 x 128 one, which so few units would not choose.  (In fp32 maps as small as these split K instead, and
    such layers go out alone.)"""
    try:
        binding.dc_conv_tuning(-1, units, -1, -1)
        _check_pointwise(bf16, n, units, device_plan)
    finally:
        binding.dc_conv_tuning()


def _check_pointwise(bf16, n, units, device_plan):
    layers = synth.googlenet(width=0.5)[:23]
    H = W = 64
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, input_shape=(H, W, 3))
    video = np.stack([synth.panning_video(7600 + s, n_frames=4, H=H, W=W, fg=((24, 24),), margin=32) for s in range(n)])
    dev = torch.from_numpy(np.ascontiguousarray(video.transpose(1, 0, 2, 3, 4))).to(DEV)
    together = [i for i, L in enumerate(layers) if L["type"] == synth.CONV and L["k"] == 1 and sum(o["type"] == synth.CONV and o["k"] == 1 and o["in0"] == L["in0"] for o in layers) == 3]
    assert len(together) == 6
    flags = np.zeros(len(layers), np.uint8)
    flags[together[1]] = 1
    for no_reuse in (None, flags):
        runs = []
        for profile in (False, True):
            runner = binding.StackRunner(layers, ws, bs, n, H, W, 3, block=16, radius=16, device_plan=device_plan, exact_masks=device_plan, overlap=False,
                                         dtype=binding.DC_BF16 if bf16 else binding.DC_F32, no_reuse=no_reuse)
            runner.enable_profile(profile)
            frames = []
            for t in range(4):
                print(f"[pointwise] bf16={bf16} n={n} units={units} device_plan={device_plan} profile={profile} frame {t}", flush=True)
                got = runner.step(dev[t])
                torch.cuda.synchronize()
                names = [binding.conv_kernel_name(k) if k >= 0 else "" for k in runner.layer_stats()["kernel_id"]]
                many = f"conv_pw_many_kernel<{'__hip_bfloat16' if bf16 else 'float'}, {4 if units == 8 else 2}>"
                if profile or (not bf16 and units < 0):
                    assert not any("conv_pw_many_kernel" in v for v in names), (t, names)
                else:
                    assert all(names[i] == many for i in together), (t, names)
                frames.append([x.clone() for x in got])
            runs.append((frames,))
        for t in range(4):
            for i, (a, b) in enumerate(zip(runs[0][0][t], runs[1][0][t])):
                assert torch.equal(a, b), (t, i)


def _c11(cin, cout, in0, relu=1, k=1):
    return dict(type=synth.CONV, k=k, s=1, p=k // 2, cin=cin, cout=cout, relu=relu, in0=in0, in1=-1)


def _full_frame(layers, share, profile, n=3, H=40, W=36):
    """One full frame through a runner whose tensor t lies in tensor share[t]'s buffer; the last tensor and the kernels."""
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, residual_scale=0.5, input_shape=(H, W, 3))
    video = np.stack([synth.panning_video(7800 + s, n_frames=1, H=H, W=W, fg=((16, 16),)) for s in range(n)])
    runner = binding.StackRunner(layers, ws, bs, n, H, W, 3, block=8, radius=8, dtype=binding.DC_BF16, device_plan=True, exact_masks=True, overlap=False)
    runner.enable_profile(profile)
    for t, v in share.items():
        assert runner.bufs[0][t].shape == runner.bufs[0][v].shape
        for tables in runner._tp:
            for table in tables:
                table[t] = table[v]
    runner.step(torch.from_numpy(video[:, 0].copy()).to(DEV), force_full=True)
    torch.cuda.synchronize()
    return runner.bufs[0][len(layers)].clone(), [binding.conv_kernel_name(k) if k >= 0 else "" for k in runner.layer_stats()["kernel_id"]]


MANY = "conv_pw_many_kernel<__hip_bfloat16, 2>"
ALONE = "conv_pw_kernel<__hip_bfloat16, 2>"


@pytest.mark.parametrize("share,kernels", [
    ({}, (MANY, MANY, MANY)),                      # three layers of one tensor
    ({4: 2}, (MANY, ALONE, MANY)),                 # the second writes over what the 3x3 layer before it reads: it waits for its turn,
                                                   # and the third, launched with the first, is not launched again with it
    ({5: 2}, (MANY, MANY, ALONE)),                 # the same for the third
    ({4: 2, 5: 3}, (ALONE, MANY, MANY)),           # neither may move up to the first, but the third to the second
])
def test_layers_of_one_tensor_whose_buffers_are_shared(share, kernels):
    """1x1 layers that read one tensor are launched with the first of them only where nothing between them reads or writes
    their outputs' memory.  (With a profile attached every layer is a launch of its own.)"""
    layers = [dict(_c11(3, 64, 0), k=3, p=1), _c11(64, 64, 1), _c11(64, 64, 2, k=3), _c11(64, 64, 1), _c11(64, 64, 1)]
    layers += [synth._concat([64, 64, 64, 64], [2, 3, 4, 5]) if not share else synth._concat([64, 64], [4, 5])]
    got, names = _full_frame(layers, share, False)
    want, apart = _full_frame(layers, {}, True)
    assert (names[1], names[3], names[4]) == kernels and {apart[i] for i in (1, 3, 4)} == {ALONE}
    assert torch.equal(got, want)


@pytest.mark.parametrize("share,fused", [({}, True), ({4: 1}, True),       # the sum may replace its other summand
                                         ({4: 2}, False),                  # the convolution's input
                                         ({4: 3}, False)])                 # the convolution's output
def test_sums_whose_buffers_are_shared(share, fused):
    """A sum is written by the convolution before it only where that convolution does not read the sum's memory."""
    layers = [dict(_c11(3, 64, 0), k=3, p=1), _c11(64, 64, 1), _c11(64, 64, 2, relu=0), synth._add(64, 3, 1, True), _c11(64, 32, 4)]
    got, names = _full_frame(layers, share, False)
    want, apart = _full_frame(layers, {}, True)
    assert names[2] == ("conv_pw_add_kernel<__hip_bfloat16, 2>" if fused else ALONE) and apart[2] == ALONE
    assert torch.equal(got, want)


@pytest.mark.parametrize("net,bf16,units", [("resnet50", True, 4), ("resnet50", True, 8), ("resnet50", False, 8),
                                            ("googlenet", True, 4), ("googlenet", True, 8), ("googlenet", False, 8)])
def test_layers_launched_together_under_several_stages(net, bf16, units):
    """Sums written by the convolution before them and 1x1 layers of one tensor in one launch, in frames that are cut into stages,
    launched and replayed, with the tiles of both sizes: every tensor bit for bit that of the same layers launched one by one
    (a profile attached, no stages).  The launch shapes are fixed."""
    layers = synth.resolve_global_pooling(synth.resnet50_trunk() if net == "resnet50" else synth.googlenet(), 224, 224, 3)
    ws, bs = synth.he_weights(layers, 3, bias_scale=0.05, residual_scale=0.5, input_shape=(224, 224, 3))
    T = 5
    video = torch.from_numpy(synth.panning_video(95, n_frames=T, H=224, W=224, fg=((24, 24), (16, 32)))).to(DEV)
    frames = [video[t:t + 1].contiguous() for t in range(T)]
    torch.cuda.synchronize()
    order = (list(range(T)) + [None]) * 12
    binding.dc_conv_tuning(0, units, 1, 0)
    try:
        runs = {}
        for mode in (0, 1, None):
            print(f"[together] {net} bf16={bf16} units={units} mode={mode}", flush=True)
            runs[mode] = _replay_run(layers, ws, bs, frames, 16, bf16, mode, order,
                                     before=lambda j, r: r.enable_profile(True) if mode is None and j == 0 else None)
    finally:
        binding.dc_conv_tuning()
    names = {mode: {binding.conv_kernel_name(k) for k in runs[mode][2] if k >= 0} for mode in runs}
    together = f"conv_pw_{'add' if net == 'resnet50' else 'many'}_kernel<{'__hip_bfloat16' if bf16 else 'float'}, {units // 2}>"
    assert together in names[0] and together in names[1] and together not in names[None], names
    assert runs[0][1].stages > 1 and runs[1][1].stages > 1 and runs[1][1].replayed > 0 and runs[0][1].replayed == 0
    assert int(runs[0][0][0][-2].sum()) > 0
    for mode in (0, 1):
        for f, (a, b) in enumerate(zip(runs[mode][0], runs[None][0])):
            for i, (x, y) in enumerate(zip(a, b)):
                assert torch.equal(x, y), (mode, f, i)
