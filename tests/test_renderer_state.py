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
