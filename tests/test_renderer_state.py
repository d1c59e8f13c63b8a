"""What a Renderer keeps between frames: it works in every mode a caller may
be in, and holds no more than it needs."""
import numpy as np
import pytest

from paper_2604_12626_amd import synth

from parity import to_dev

F32 = np.float32


@pytest.fixture
def dev():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    return torch.device("cuda:0")


def _scene(dev):
    import torch
    W, H = 80, 64
    g = to_dev(synth.gaussians_cube(2000, np.random.default_rng(3), sh_degree=1), dev)
    cam = torch.from_numpy(synth.identity_camera(90.0, 90.0, W / 2, H / 2)[None].astype(F32)).to(dev)
    return W, H, g, cam


@pytest.mark.gpu
@pytest.mark.parametrize("mode", ["inference", "default_device"])
def test_render_in_a_callers_mode_and_after_it(dev, mode):
    """The second frame of the same sizes is the first that makes the host
    flag: made in inference mode or under a default device it has to serve the
    frames outside too."""
    import torch
    from paper_2604_12626_amd import render
    W, H, g, cam = _scene(dev)
    r = render.Renderer(W, H, capacity=1 << 16, device=dev)
    want = r.render([g], cam).rgb.clone()
    with (torch.inference_mode() if mode == "inference" else torch.device(dev)):
        inside = r.render([g], cam).rgb.clone()
    after = r.render([g], cam).rgb.clone()
    assert torch.equal(inside, want) and torch.equal(after, want)
    leaf = g["means"].clone().requires_grad_(True)  # and training on the same renderer
    rgb, _, _ = render.rasterize(leaf, g["log_scales"], g["quats"], g["opacity"], g["sh"], cam, r)
    rgb.sum().backward()
    assert torch.equal(rgb.detach(), want) and float(leaf.grad.abs().max()) > 0


@pytest.mark.gpu
@pytest.mark.parametrize("how", ["deepcopy", "pickle"])
def test_renderer_copies_after_frames(dev, how):
    """A renderer that has drawn frames copies and pickles as a fresh one
    does; the copy draws into buffers of its own."""
    import copy
    import pickle
    import torch
    from paper_2604_12626_amd import render
    W, H, g, cam = _scene(dev)
    r = render.Renderer(W, H, capacity=1 << 16, device=dev)
    for _ in range(3):
        f = r.render([g], cam)
    want = f.rgb.clone()
    c = copy.deepcopy(r) if how == "deepcopy" else pickle.loads(pickle.dumps(r))
    for _ in range(3):
        f2 = c.render([g], cam)
        assert torch.equal(f2.rgb, want)
    assert f2.rgb.data_ptr() != f.rgb.data_ptr()
    f2.rgb.zero_()
    assert torch.equal(f.rgb, want)


@pytest.mark.gpu
@pytest.mark.parametrize("frames", [1, 2, 3])
def test_checked_render_under_capture_is_refused_and_leaves_the_gpu_usable(dev, frames):
    """render() checks for an overflow, which needs the GPU's answer: under
    capture it is refused, the capture ends, and eager frames go on."""
    import torch
    from paper_2604_12626_amd import render
    W, H, g, cam = _scene(dev)
    r = render.Renderer(W, H, capacity=1 << 16, device=dev)
    for _ in range(frames):
        want = r.render([g], cam).rgb.clone()
    torch.cuda.synchronize()
    with pytest.raises(RuntimeError, match="capturing"):
        with torch.cuda.graph(torch.cuda.CUDAGraph()):
            r.render([g], cam)
    torch.cuda.synchronize()
    for _ in range(3):
        assert torch.equal(r.render([g], cam).rgb, want)


@pytest.mark.parametrize("grow", ["sizes", "capacity"])
def test_grown_buffers_free_the_old_ones_one_by_one(grow):
    """While a frame of larger sizes is shaped, each buffer that grows is freed
    when its successor is there: a renderer of a frame that its caller has
    dropped never holds the old set and the new one together."""
    import weakref
    from paper_2604_12626_amd import render
    r = render.Renderer(64, 48, capacity=1 << 12, device="cpu")
    r.alloc_frame(1000, 1)
    old = {k: weakref.ref(t.untyped_storage()) for k, t in r._bufs.items()}
    seen = []
    cut = r._buf

    def buf(name, *a, **kw):
        t = cut(name, *a, **kw)
        if r._bufs[name].untyped_storage() is not old[name]():
            seen.append((name, old[name]() is None))
        return t

    r._buf = buf
    if grow == "sizes":
        r.alloc_frame(5000, 3)
    else:
        r.capacity = 1 << 14
        r.alloc_frame(1000, 1)
    assert len(seen) >= 3 and all(freed for _, freed in seen), seen


def test_retry_after_an_overflow_drops_the_small_frame_first():
    """render() lets go of the frame that overflowed before it allocates the
    larger one."""
    import torch
    import weakref
    from paper_2604_12626_amd import render
    r = render.Renderer(64, 48, capacity=1 << 12, device="cpu")
    refs, alive, calls = [], [], []
    alloc = r.alloc_frame

    def alloc_frame(*a):
        alive.extend(x() is not None for x in refs)
        f = alloc(*a)
        refs.append(weakref.ref(f))
        return f

    def forward(segs, cams, view_segs, f, check, ahead):
        calls.append(r.capacity)
        f.num.fill_(100_000)
        return len(calls) == 1

    r.alloc_frame, r._forward = alloc_frame, forward
    seg = {"means": torch.zeros(10, 3), "sh_degree": 0, "opacity": torch.zeros(10), "sh": torch.zeros(10, 1, 3),
           "log_scales": torch.zeros(10, 3), "quats": torch.zeros(10, 4)}
    f = r.render([seg], torch.zeros(1, 16))
    assert len(calls) == 2 and calls[1] >= 100_000 and f.keys.shape[0] == calls[1]
    assert alive == [False]
