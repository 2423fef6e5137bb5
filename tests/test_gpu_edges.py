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


@pytest.mark.parametrize("n", [(7 << 12) - 1, 7 << 12, 40001, (1 << 16) - 1, 1 << 16])
@pytest.mark.parametrize("table_bits,dtype", [(15, "f16"), (19, "f32")])
def test_scatter_on_both_sides_of_the_list_and_record_sizes(n, table_bits, dtype):
    """Atomic kernel, lists of wide records and lists of packed records, with the position gradient.  Wide records and
    atomics keep binary32 values: at most ten roundings of 2^-24 each, 6e-7; packed ones 4e-6 rms."""
    rng = np.random.default_rng(n + table_bits)
    cfg = wl.make_config(2)
    cfg.log2_table_size, cfg.res = table_bits, wl.level_resolutions(16, 16, 512)
    cfg.dense, cfg.table_dtype = wl.dense_flags(cfg.res, cfg.table_size), dtype
    c, L, T = nb.make_config(cfg), cfg.n_levels, cfg.table_size
    tab = rng.uniform(-1.0, 1.0, size=(L, T, 2)).astype(np.float16 if dtype == "f16" else np.float32)
    pos = wl.make_rays(n // 64 + 1, 64, n)["pos"][:n]
    q, d_enc = (rng.normal(size=(n, 2 * L)).astype(np.float32) for _ in range(2))
    d_normal = (rng.normal(size=(n, 3)) * 1e-2).astype(np.float32)
    to_lm = lambda a: cuda(a.reshape(n, L, 2).transpose(1, 0, 2))
    want = o.table_gradient(cfg, pos, q, d_enc, d_normal)
    size = nb.workspace_bytes(c, n)
    assert (size == 0) == (n < 7 << 12)
    found = []
    for with_lists in ([True, False] if size else [False]):
        ws = torch.zeros(size // 4, dtype=torch.int32, device="cuda") if with_lists else None
        got, d_pos = torch.zeros(L, T, 2, device="cuda"), torch.zeros(n, 3, device="cuda")
        nb.hash_scatter_bwd(c, cuda(pos), cuda(tab), to_lm(q), to_lm(d_enc), cuda(d_normal), n, got, d_pos=d_pos, workspace=ws)
        torch.cuda.synchronize()
        error = rel(got.cpu().numpy(), want)
        print(n, table_bits, with_lists, error, flush=True)
        assert error <= (1e-5 if with_lists and n >= 1 << 16 else 1e-6)
        found.append(d_pos.cpu().numpy())
    assert all(rel(f, found[0]) <= 1e-5 for f in found)


@pytest.mark.parametrize("n,hidden,table,active,levels", [(1, 2, "f16", 16, 16), (31, 1, "f32", 16, 16), (33, 2, "f32", 5, 16),
                                                         (4097, 2, "f16", 16, 16), (1000, 1, "f16", 8, 8)])
def test_sdf_values_equal_the_forward_calls(n, hidden, table, active, levels):
    """The value-only path does the same arithmetic: the same bits as the encoding and the forward kernel; nothing behind
    the n values is written."""
    import dataclasses
    rng = np.random.default_rng(n + hidden)
    cfg = wl.make_config(2 if levels == 16 else 1)
    cfg = dataclasses.replace(cfg, table_dtype=table, active_levels=active, sdf_dims=[2 * levels] + [64] * hidden + [16])
    assert cfg.n_levels == levels
    c = nb.make_config(cfg)
    pos = cuda(rng.uniform(size=(n, 3)).astype(np.float32))
    tables = cuda(rng.normal(size=(levels, cfg.table_size, 2)).astype(np.float32) * 0.1)
    if table == "f16":
        tables = tables.half()
    H = [cuda((rng.normal(size=(o_, i)) * (2.0 / i) ** 0.5).astype(np.float32)) for i, o_ in zip(cfg.sdf_dims, cfg.sdf_dims[1:])]
    enc, jac, q = torch.empty(levels * n * 2, device="cuda"), torch.empty(levels * n * 6, device="cuda"), torch.empty(levels * n * 2, device="cuda")
    y, normal = torch.empty(n, 16, device="cuda"), torch.empty(n, 3, device="cuda")
    nb.hash_encode(c, pos, tables, enc, jac)
    nb.sdf_fwd_grad(c, enc, jac, H, n, y, q, normal)
    sdf, behind = guarded((n,))
    scratch = torch.full((levels * n * 2,), float("nan"), device="cuda")
    nb.sdf_values(c, pos, tables, H, n, scratch, sdf)
    assert torch.equal(sdf, y[:, 0]) and float(y[:, 0].abs().max()) > 0
    assert torch.equal(scratch[: 2 * n * active], enc[: 2 * n * active])
    assert torch.all(torch.signbit(behind)) and torch.all(behind == 0)
