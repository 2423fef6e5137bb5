"""Edges of the kernels' tiles, dispatch rules and buffers, against the float64 oracle."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import neus2_oracle as o
from paper_2212_05231_amd import binding as nb
from paper_2212_05231_amd import workloads as wl

pytestmark = pytest.mark.gpu

GRAD_TOL = 1e-4


@pytest.fixture(scope="module", autouse=True)
def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    nb.lib()


def cuda(a):
    return torch.as_tensor(np.ascontiguousarray(a)).cuda()


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def guarded(shape):
    """A zeroed tensor and the 64 floats behind it, which hold -0.0: even an added zero changes their bits."""
    count = int(np.prod(shape))
    flat = torch.full((count + 64,), -0.0, device="cuda")
    flat[:count] = 0.0
    return flat[:count].view(shape), flat[count:]


@pytest.mark.parametrize("n", [1, 31, 33, 1000])
@pytest.mark.parametrize("given", [True, False])
def test_color_backward_gradients_and_nothing_behind_them(n, given):
    rng = np.random.default_rng(n)
    cfg = wl.make_config(2)
    cfg.samples_per_ray = 1
    c = nb.make_config(cfg)
    W = [rng.normal(size=(cfg.color_dims[i + 1], cfg.color_dims[i])).astype(np.float32) * 0.3 for i in range(3)]
    pos = rng.uniform(size=(n, 3)).astype(np.float32)
    nrm, y = rng.normal(size=(n, 3)).astype(np.float32), rng.normal(size=(n, 16)).astype(np.float32)
    dirs = rng.normal(size=(n, 3))
    dirs = (dirs / np.linalg.norm(dirs, axis=1, keepdims=True)).astype(np.float32)
    d_rgb = rng.normal(size=(n, 3)).astype(np.float32)
    Wg, args = [cuda(w) for w in W], (cuda(pos), cuda(nrm), cuda(dirs), cuda(y))
    rgb = torch.empty(n, 3, device="cuda")
    kept = torch.zeros(2, n, 2, dtype=torch.int32, device="cuda")
    nb.color_fwd(c, *args, Wg, n, rgb, masks=kept)
    dW, behind = zip(*[guarded(w.shape) for w in W])
    d_normal = torch.zeros(n, 3, device="cuda")
    nb.color_bwd(c, *args, Wg, rgb, cuda(d_rgb), None, n, list(dW), torch.empty(n, 16, device="cuda"), d_normal,
                 masks=kept if given else None)
    torch.cuda.synchronize()
    rgb_r, acts, masks = o.color_forward(W, o.color_input(pos, nrm.astype(np.float64), dirs, y.astype(np.float64), 1))
    want = o.mlp_backward(W, acts, masks, d_rgb * rgb_r * (1 - rgb_r))[0]
    for got, ref, guard in zip(dW, want, behind):
        assert rel(got.cpu().numpy(), ref) <= GRAD_TOL
        assert bool(torch.signbit(guard).all())
