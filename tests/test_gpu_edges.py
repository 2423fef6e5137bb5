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


@pytest.mark.parametrize("capacity", [1 << 16, 70000])
@pytest.mark.parametrize("n", [7 << 12, (1 << 16) - 1])
def test_lists_for_every_batch_a_workspace_was_made_for(n, capacity):
    """A workspace made for more points: a smaller batch goes through the lists too (the cursors in its header count their
    records), with both gradients as without a workspace."""
    rng = np.random.default_rng(n)
    cfg = wl.make_config(2)
    c, L, T = nb.make_config(cfg), cfg.n_levels, cfg.table_size
    tab = cuda(wl.make_params(cfg, 3)["tables"])
    pos = cuda(wl.make_rays(n // 64 + 1, 64, n)["pos"][:n])
    q, d_enc = (cuda(rng.normal(size=(L, n, 2)).astype(np.float32)) for _ in range(2))
    d_normal = cuda((rng.normal(size=(n, 3)) * 1e-2).astype(np.float32))
    found = []
    for ws in (torch.zeros(nb.workspace_bytes(c, capacity) // 4, dtype=torch.int32, device="cuda"), None):
        got, d_pos = torch.zeros(L, T, 2, device="cuda"), torch.zeros(n, 3, device="cuda")
        nb.hash_scatter_bwd(c, pos, tab, q, d_enc, d_normal, n, got, d_pos=d_pos, workspace=ws)
        found.append((got.cpu(), d_pos.cpu()))
        assert ws is None or bool(ws.any())
    for a, b in zip(*found):
        assert rel(a, b) <= 1e-6                       # ten roundings of binary32 on either side


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


@pytest.mark.parametrize("n,hidden,levels,active", [(1, 2, 16, 16), (31, 1, 16, 3), (33, 2, 8, 8), (257 * 32 + 7, 2, 16, 15), (4096 * 32 + 1, 1, 8, 5)])
def test_sdf_forward_over_tiles_and_levels(n, hidden, levels, active):
    """Tiles that are not full, workgroups with one wavefront at work and with a second round; an inactive level's arrays
    may hold anything.  Sums of at most 64 products in binary32: 1e-5 of the norm is the oracle tests' bound."""
    import dataclasses
    rng = np.random.default_rng(n + levels)
    cfg = wl.make_config(2 if levels == 16 else 1)
    cfg = dataclasses.replace(cfg, active_levels=active, sdf_dims=[2 * levels] + [64] * hidden + [16])
    c = nb.make_config(cfg)
    H = [cuda((rng.normal(size=(o_, i)) * (2.0 / i) ** 0.5).astype(np.float32)) for i, o_ in zip(cfg.sdf_dims, cfg.sdf_dims[1:])]
    gen = torch.Generator(device="cuda").manual_seed(n)
    enc, jac = torch.randn(levels, n, 2, device="cuda", generator=gen), torch.randn(levels, 3, n, 2, device="cuda", generator=gen)
    enc[active:], jac[active:] = float("nan"), float("nan")
    (y, behind_y), (q, behind_q), (normal, behind_n) = guarded((n, 16)), guarded((levels, n, 2)), guarded((n, 3))
    masks = torch.zeros(2, n, 2, dtype=torch.int32, device="cuda")
    nb.sdf_fwd_grad(c, enc, jac, H, n, y, q, normal, masks=masks)
    x = torch.zeros(n, 2 * levels, dtype=torch.float64, device="cuda")
    x[:, : 2 * active] = enc[:active].permute(1, 0, 2).reshape(n, -1).double()
    x.requires_grad_()
    z, on = x, []
    for h in H[:-1]:
        z = torch.relu(z @ h.double().T)
        on.append(z > 0)
    ref = z @ H[-1].double().T
    g, = torch.autograd.grad(ref[:, 0].sum(), x)
    # a pre-activation within rounding of zero may fall the other way: such points are left out of the gradient's comparison
    count = sum(int(m.sum()) for m in on)
    bits = sum(int(((masks[:hidden] >> b) & 1).sum()) for b in range(32))
    assert abs(bits - count) <= 1 + count // 10 ** 5
    agree = torch.ones(n, dtype=torch.bool, device="cuda")
    for layer, m in enumerate(on):
        word_bits = torch.stack([(masks[layer] >> b) & 1 for b in range(32)]).sum(0).sum(1)
        agree &= word_bits == m.sum(1)
    assert int((~agree).sum()) <= 1 + n // 10 ** 4
    qq = q.permute(1, 0, 2).reshape(n, -1)
    J = jac[:active].permute(2, 0, 1, 3).reshape(n, active, 2, 3).double()
    nrm = (g[:, : 2 * active].reshape(n, active, 2, 1) * J).sum((1, 2))
    assert rel(y.cpu(), ref.detach().cpu()) <= 1e-5
    assert rel(qq[agree][:, : 2 * active].cpu(), g[agree][:, : 2 * active].cpu()) <= 1e-5
    assert rel(normal[agree].cpu(), nrm[agree].cpu()) <= 1e-5
    for behind in (behind_y, behind_q, behind_n):
        assert torch.all(torch.signbit(behind)) and torch.all(behind == 0)


@pytest.mark.parametrize("levels,hidden,active", [(16, 2, a) for a in (0, 1, 4, 5, 8, 9, 11, 12, 13)] + [(8, 2, 1), (8, 1, 4), (8, 2, 5), (16, 1, 8)])
def test_networks_with_fewer_active_levels(levels, hidden, active):
    """Each group of four levels has a variant of the network kernels: the same bits as with all levels active and zeros in
    the others, whose arrays may hold anything here."""
    import dataclasses
    n = 32 * 9 + 5
    cfg = wl.make_config(2 if levels == 16 else 1)
    cfg = dataclasses.replace(cfg, sdf_dims=[2 * levels] + [64] * hidden + [16])
    gen = torch.Generator(device="cuda").manual_seed(active)
    randn = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)
    H = [randn(o_, i) * (2.0 / i) ** 0.5 for i, o_ in zip(cfg.sdf_dims, cfg.sdf_dims[1:])]
    enc, jac, d_y, d_normal = randn(levels, n, 2), randn(levels, 3, n, 2), randn(n, 16), randn(n, 3)
    found = []
    for count, fill in ((active, float("nan")), (levels, 0.0)):
        c = nb.make_config(dataclasses.replace(cfg, active_levels=count))
        enc[active:], jac[active:] = fill, fill
        y, q, normal, d_enc, d_pos = (torch.zeros(*s, device="cuda") for s in ((n, 16), (levels, n, 2), (n, 3), (levels, n, 2), (n, 3)))
        masks, dH = torch.zeros(2, n, 2, dtype=torch.int32, device="cuda"), [torch.zeros_like(h) for h in H]
        nb.sdf_fwd_grad(c, enc, jac, H, n, y, q, normal, masks=masks)
        nb.sdf_mlp_bwd(c, enc, jac, H, d_y, d_normal, n, dH, d_enc, d_pos=d_pos, masks=masks)
        found.append(([y, q, normal, masks, d_enc, d_pos], dH))
    for a, b in zip(found[0][0], found[1][0]):
        assert torch.equal(a, b)
    for a, b in zip(found[0][1], found[1][1]):
        assert float((a - b).abs().max()) <= 1e-5 * float(b.abs().max())    # ten workgroups' sums in any order


@pytest.mark.parametrize("levels,hidden", [(16, 2), (8, 1)])
def test_networks_from_2_26_points_on(levels, hidden):
    """Where a lane's byte offsets need 64 bits: the same bits per point, forward and backward, as the same points give in a
    small batch; the backward call goes by the masks it is given (here the forward call's with some bits cleared)."""
    import dataclasses
    n, m = (1 << 26) + 5, 3000
    if torch.cuda.mem_get_info()[0] < 1.2 * 4 * n * (levels * 12 + 45):
        pytest.skip("not enough free device memory")
    cfg = wl.make_config(2 if levels == 16 else 1)
    cfg = dataclasses.replace(cfg, sdf_dims=[2 * levels] + [64] * hidden + [16])
    c, gen = nb.make_config(cfg), torch.Generator(device="cuda").manual_seed(levels)
    randn = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)
    H = [randn(o_, i) * (2.0 / i) ** 0.5 for i, o_ in zip(cfg.sdf_dims, cfg.sdf_dims[1:])]
    chosen = torch.cat([torch.arange(1000), torch.arange(n // 2, n // 2 + 1000), torch.arange(n - 1000, n)]).cuda()

    def call(enc, jac, d_y, d_normal, points, cleared):
        count = enc.shape[1]
        empty = lambda *shape: torch.empty(*shape, device="cuda")
        y, q, normal, d_enc = empty(count, 16), empty(levels, count, 2), empty(count, 3), empty(levels, count, 2)
        masks, dH = torch.empty(2, count, 2, dtype=torch.int32, device="cuda"), [torch.zeros_like(h) for h in H]
        nb.sdf_fwd_grad(c, enc, jac, H, count, y, q, normal, masks=masks)
        kept = [masks[:hidden, points].clone()]
        masks[:hidden, points] &= cleared
        nb.sdf_mlp_bwd(c, enc, jac, H, d_y, d_normal, count, dH, d_enc, masks=masks)
        return kept + [y[points], normal[points], q[:, points], d_enc[:, points]], dH

    small = [randn(m, 16), randn(m, 3)]
    cleared = torch.randint(-2 ** 31, 2 ** 31, (hidden, m, 2), device="cuda", generator=gen, dtype=torch.int64).to(torch.int32)
    enc, jac = randn(levels, n, 2), randn(levels, 3, n, 2)
    d_y, d_normal = torch.zeros(n, 16, device="cuda"), torch.zeros(n, 3, device="cuda")
    d_y[chosen], d_normal[chosen] = small[0], small[1]
    got, dH = call(enc, jac, d_y, d_normal, chosen, cleared)
    few = (enc[:, chosen].contiguous(), jac[:, :, chosen].contiguous())
    del enc, jac, d_y, d_normal
    want, dH_few = call(*few, *small, torch.arange(m, device="cuda"), cleared)
    torch.cuda.empty_cache()
    for a, b in zip(got, want):
        assert torch.equal(a, b) and bool(a.any())
    for a, b in zip(dH, dH_few):
        assert rel(a.cpu(), b.cpu()) <= 1e-5                     # the same terms in another order


@pytest.mark.parametrize("n", [1, 31, 33, 1000])
@pytest.mark.parametrize("given", [True, False])
def test_color_backward_adjoints_and_nothing_behind_them(n, given):
    """The adjoints of every input of the colour network, d_normal added to, d_sdf passed on; tiles that are not full."""
    rng = np.random.default_rng(n + 7)
    cfg = wl.make_config(2)
    cfg.samples_per_ray = 1
    c = nb.make_config(cfg)
    W = [rng.normal(size=(cfg.color_dims[i + 1], cfg.color_dims[i])).astype(np.float32) * 0.3 for i in range(3)]
    pos = rng.uniform(size=(n, 3)).astype(np.float32)
    nrm, y, dn0 = (rng.normal(size=(n, k)).astype(np.float32) for k in (3, 16, 3))
    dirs = rng.normal(size=(n, 3))
    dirs = (dirs / np.linalg.norm(dirs, axis=1, keepdims=True)).astype(np.float32)
    d_rgb, d_sdf = rng.normal(size=(n, 3)).astype(np.float32), rng.normal(size=n).astype(np.float32)
    Wg, args = [cuda(w) for w in W], (cuda(pos), cuda(nrm), cuda(dirs), cuda(y))
    rgb, kept = torch.empty(n, 3, device="cuda"), torch.zeros(2, n, 2, dtype=torch.int32, device="cuda")
    nb.color_fwd(c, *args, Wg, n, rgb, masks=kept)
    rgb_r, acts, masks = o.color_forward(W, o.color_input(pos, nrm.astype(np.float64), dirs, y.astype(np.float64), 1))
    d_in = o.mlp_backward(W, acts, masks, d_rgb * rgb_r * (1 - rgb_r))[1]
    want_dy = d_in[:, 22:38].copy()
    want_dy[:, 0] += d_sdf
    (d_y, behind_y), (d_normal, behind_n), (d_pos, behind_p) = guarded((n, 16)), guarded((n, 3)), guarded((n, 3))
    d_normal += cuda(dn0)
    nb.color_bwd(c, *args, Wg, rgb, cuda(d_rgb), cuda(d_sdf), n, [torch.zeros_like(w) for w in Wg], d_y, d_normal, d_pos,
                 masks=kept if given else None)
    for got, want in ((d_y, want_dy), (d_normal, dn0 + d_in[:, 3:6]), (d_pos, d_in[:, 0:3])):
        assert rel(got.cpu().numpy(), want) <= GRAD_TOL
    for behind in (behind_y, behind_n, behind_p):
        assert torch.all(torch.signbit(behind)) and torch.all(behind == 0)


@pytest.mark.parametrize("n,levels,hidden", [(1, 16, 2), (31, 8, 2), (33, 16, 1), (257 * 32 + 7, 16, 2)])
def test_sdf_backward_with_and_without_masks_and_nothing_behind(n, levels, hidden):
    """Both kernels of the SDF backward call on tiles that are not full, with the position gradient added to: two terms per
    factor on one side, three on the other, 1e-4 of the norm apart at most."""
    import dataclasses
    cfg = wl.make_config(2 if levels == 16 else 1)
    c = nb.make_config(dataclasses.replace(cfg, sdf_dims=[2 * levels] + [64] * hidden + [16]))
    gen = torch.Generator(device="cuda").manual_seed(n)
    randn = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)
    H = [randn(o_, i) * (2.0 / i) ** 0.5 for i, o_ in zip([2 * levels] + [64] * hidden, [64] * hidden + [16])]
    enc, jac, d_y, d_normal = randn(levels, n, 2), randn(levels, 3, n, 2), randn(n, 16), randn(n, 3)
    masks = torch.zeros(2, n, 2, dtype=torch.int32, device="cuda")
    nb.sdf_fwd_grad(c, enc, jac, H, n, torch.empty(n, 16, device="cuda"), torch.empty_like(enc), torch.empty(n, 3, device="cuda"), masks=masks)
    found, start = [], randn(n, 3)
    for kept in (masks, None):
        (d_enc, behind_e), (d_pos, behind_p) = guarded((levels, n, 2)), guarded((n, 3))
        d_pos += start
        dH, behind = zip(*[guarded(h.shape) for h in H])
        nb.sdf_mlp_bwd(c, enc, jac, H, d_y, d_normal, n, list(dH), d_enc, d_pos=d_pos, masks=kept)
        for guard in (behind_e, behind_p, *behind):
            assert torch.all(torch.signbit(guard)) and torch.all(guard == 0)
        found.append([d_enc, d_pos, *dH])
    for a, b in zip(*found):
        assert rel(a.cpu(), b.cpu()) <= GRAD_TOL and bool(a.any())


@pytest.mark.parametrize("n_rays", [509, 1023])
def test_step_position_gradient_through_wide_records(n_rays):
    """A whole step below 2^16 points that wants the position gradient: its encode kernel clears the lists' header and leaves
    the second derivatives behind 20-byte records.  Against the step without a workspace on all points and against the
    oracle on a sample of rays (adjoints scale with 1/rays)."""
    w = wl.make_workload(2, n_rays=n_rays)
    cfg, params, batch = w["cfg"], w["params"], w["batch"]
    params["tables"] = (params["tables"].astype(np.float64) * 2000.0).astype(params["tables"].dtype)
    n, spr = batch["pos"].shape[0], cfg.samples_per_ray
    assert 7 << 12 <= n < 1 << 16
    found = []
    for use_ws in (True, False):
        step = nb.Step(cfg, params, n, want_pos_grad=True, use_workspace=use_ws)
        step.set_batch(batch)
        step.zero_grads()
        step.train_step()
        found.append((step.d_pos.cpu().numpy(), step.d_tables.cpu().numpy()))
        assert not use_ws or bool(step.workspace[64:64 + 32 * 256].any())           # the cursors of the lists
    assert rel(found[0][0], found[1][0]) <= 1e-5 and rel(found[0][1], found[1][1]) <= 1e-5
    pick = np.sort(np.random.default_rng(n_rays).choice(n_rays, size=40, replace=False))
    points = (pick[:, None] * spr + np.arange(spr)[None, :]).reshape(-1)
    sub = {"pos": batch["pos"][points], "dirs": batch["dirs"][pick], "target": batch["target"][pick]}
    ref = o.train_step(cfg, params, sub, want_pos_grad=True)
    assert rel(found[0][0][points], ref["dpos"] * (len(pick) / n_rays)) <= GRAD_TOL


def test_concentrated_batch_overflows_the_lists_of_wide_records():
    """40 000 samples inside a cube of side 2e-3: their rows crowd into a few ranges of every hashed level, and the surplus of
    those lists goes through global atomics.  A slot's sum of m values of either sign in binary32 is off by about
    2^-24 sqrt(m) of itself, m at most 160 000 here: 2.4e-5."""
    rng = np.random.default_rng(6)
    cfg = wl.make_config(2)
    c, L, T, n = nb.make_config(cfg), cfg.n_levels, cfg.table_size, 40000
    pos = (0.37 + 2e-3 * rng.uniform(size=(n, 3))).astype(np.float32)
    q, d_enc = (rng.normal(size=(n, 2 * L)).astype(np.float32) for _ in range(2))
    d_normal = (rng.normal(size=(n, 3)) * 1e-2).astype(np.float32)
    to_lm = lambda a: cuda(a.reshape(n, L, 2).transpose(1, 0, 2))
    ws = torch.zeros(nb.workspace_bytes(c, n) // 4, dtype=torch.int32, device="cuda")
    got = torch.zeros(L, T, 2, device="cuda")
    nb.hash_scatter_bwd(c, cuda(pos), cuda(wl.make_params(cfg, 3)["tables"]), to_lm(q), to_lm(d_enc), cuda(d_normal), n, got, workspace=ws)
    capacity = ((4 * n // (T >> 13)) * 3 // 2 + 1023) // 64 * 64
    assert int(ws[64:64 + 32 * 256].max()) > capacity
    assert rel(got.cpu().numpy(), o.table_gradient(cfg, pos, q, d_enc, d_normal)) <= 2.4e-5


@pytest.mark.parametrize("n,size_y,size_w", [(1, 1.0, 1.0), (31, 1e-20, 1.0), (33, 1e10, 1e-9), (257 * 128 + 5, 1.0, 1.0), (1000, 0.0, 1.0)])
def test_colour_forward_without_masks(n, size_y, size_w):
    """A forward pass that is not asked for masks, features and matrices of any size (one of zeros among them).  At most 64
    products, each within 2^-22 of its size, random signs: 1e-6 of the norm, as the masked pass."""
    rng = np.random.default_rng(n)
    cfg = wl.make_config(2)
    cfg.samples_per_ray = 1
    W = [rng.normal(size=(cfg.color_dims[i + 1], cfg.color_dims[i])).astype(np.float32) * 0.3 for i in range(3)]
    W[0] = (W[0] * size_w).astype(np.float32)
    W[2] = (W[2] / max(size_y * size_w, 1.0)).astype(np.float32)
    if size_y == 0.0:
        W[1][:] = 0.0
    pos, nrm = rng.uniform(size=(n, 3)).astype(np.float32), rng.normal(size=(n, 3)).astype(np.float32)
    y = (rng.normal(size=(n, 16)) * size_y).astype(np.float32)
    dirs = rng.normal(size=(n, 3))
    dirs = (dirs / np.linalg.norm(dirs, axis=1, keepdims=True)).astype(np.float32)
    rgb, behind = guarded((n, 3))
    nb.color_fwd(nb.make_config(cfg), cuda(pos), cuda(nrm), cuda(dirs), cuda(y), [cuda(w) for w in W], n, rgb)
    want, _, _ = o.color_forward(W, o.color_input(pos, nrm.astype(np.float64), dirs, y.astype(np.float64), 1))
    got = rgb.cpu().numpy()
    assert rel(got, want) <= 1e-6
    assert np.ptp(want) > 1e-3 if size_y else np.all(got == 0.5)
    assert torch.all(torch.signbit(behind)) and torch.all(behind == 0)


def runs_of_one_cell(n, res, rng):
    """Positions in runs of 1 to 40 neighbours that share a cell of a grid of `res` cells, as marched samples do."""
    lengths = rng.integers(1, 41, size=n)
    cell = np.repeat(rng.integers(0, res, size=(n, 3)), lengths, axis=0)[:n]
    return ((cell + rng.uniform(0.05, 0.95, size=(n, 3))) / res).astype(np.float32)


@pytest.mark.parametrize("n,log2_t,res,broken", [(65536, 15, [16, 30], False),      # in place: one range, and three point lists
                                                 (65537, 14, [16, 22], True),         # in place: one and two ranges
                                                 (70001, 19, [33, 70, 300], False),   # point lists, a hashed level of 64 ranges
                                                 (66000, 13, [16, 64], False),        # a hashed level of one range: cells may share slots
                                                 (524288 + 77, 21, [40, 900], False)])  # 256 ranges: 1024 points a binning workgroup
def test_scatter_add_of_runs_in_one_cell(n, log2_t, res, broken):
    """Runs of samples in one cell are summed before they reach the table; lists against 64-bit sums of the corner values.
    Sums in doubles, one rounding to binary32 on a dense level (1e-6), 2^-18 of a record's largest value on a hashed one with lists (1e-5).
    A non-finite adjoint reaches its own cell's entries and no others."""
    import dataclasses
    rng = np.random.default_rng(n)
    dense = wl.dense_flags(res, 1 << log2_t)
    levels = len(res)
    cfg = dataclasses.replace(wl.make_config(2), log2_table_size=log2_t, res=res + [4] * (16 - levels), dense=dense + [1] * (16 - levels),
                              active_levels=levels)
    c = nb.make_config(cfg)
    pos = runs_of_one_cell(n, res[0], rng)
    gen = torch.Generator(device="cuda").manual_seed(n)
    q, d_enc = (torch.randn(16, n, 2, device="cuda", generator=gen) for _ in range(2))
    d_normal = torch.randn(n, 3, device="cuda", generator=gen) * 0.05
    if broken:
        d_enc[0, 1000, 1], d_enc[1, 2000, 0] = float("nan"), float("inf")
    tables = torch.zeros(16, 1 << log2_t, 2, device="cuda", dtype=torch.float16)
    d_tables, behind = guarded((16, 1 << log2_t, 2))
    ws = torch.zeros(nb.workspace_bytes(c, n) // 4, dtype=torch.int32, device="cuda")
    nb.hash_scatter_bwd(c, cuda(pos), tables, q, d_enc, d_normal, n, d_tables, workspace=ws)
    assert bool(ws.any())
    q, d_enc, d_normal = (t.cpu().numpy().astype(np.float64) for t in (q, d_enc, d_normal))
    for level in range(levels):
        p = o.grid_coords(pos, res[level])
        cell = np.minimum(np.floor(p), res[level] - 1)
        w = p - cell
        want = np.zeros((1 << log2_t, 2))
        for k in range(8):
            f = [w[:, a] if (k >> a) & 1 else 1 - w[:, a] for a in range(3)]
            s = [res[level] if (k >> a) & 1 else -res[level] for a in range(3)]
            slope = s[0] * f[1] * f[2] * d_normal[:, 0] + f[0] * s[1] * f[2] * d_normal[:, 1] + f[0] * f[1] * s[2] * d_normal[:, 2]
            value = (f[0] * f[1] * f[2])[:, None] * d_enc[level] + q[level] * slope[:, None]
            corner = np.stack([cell[:, a] + ((k >> a) & 1) for a in range(3)], axis=1)
            slot = o.vertex_index(corner, res[level], dense[level], 1 << log2_t)
            for x in range(2):
                want[:, x] += np.bincount(slot, weights=value[:, x], minlength=1 << log2_t)
        got = d_tables[level].cpu().numpy().astype(np.float64)
        finite = np.isfinite(want)
        assert np.array_equal(finite, np.isfinite(got)) and int((~finite).sum()) == (8 if broken else 0)
        tol = 1e-6 if dense[level] or (1 << log2_t) <= 8192 else 1e-5
        assert rel(got[finite], want[finite]) <= tol, level
    assert torch.all(torch.signbit(behind)) and torch.all(behind == 0)


@pytest.mark.parametrize("n,log2_t", [(131072, 16), (131073, 16), (262144, 15), (262145, 15), (80001, 14)])
def test_scatter_add_over_few_ranges(n, log2_t):
    """Both orders of the binning workgroups, on either side of the number of records where one follows the other: several
    hashed levels of two to eight ranges that the groups share out unevenly, point lists and in-place levels beside them."""
    test_scatter_add_of_runs_in_one_cell(n, log2_t, [12, 24 if log2_t < 16 else 36, 50, 64, 90, 120, 200], False)


def colour_inputs(n, rng):
    cfg = wl.make_config(2)
    cfg.samples_per_ray = 1
    W = [rng.normal(size=(cfg.color_dims[i + 1], cfg.color_dims[i])).astype(np.float32) * 0.3 for i in range(3)]
    pos, nrm = rng.uniform(size=(n, 3)).astype(np.float32), rng.normal(size=(n, 3)).astype(np.float32)
    y = rng.normal(size=(n, 16)).astype(np.float32)
    dirs = rng.normal(size=(n, 3))
    return nb.make_config(cfg), W, pos, nrm, (dirs / np.linalg.norm(dirs, axis=1, keepdims=True)).astype(np.float32), y


def without_neuron_scales(rng, mats, low=-30, high=30):
    """The same network with each hidden neuron scaled by a power of two: row of one matrix up, column of the next down."""
    scaled = [m.copy() for m in mats]
    for l in range(len(mats) - 1):
        scale = np.ldexp(np.float32(1), rng.integers(low, high + 1, size=mats[l].shape[0])).astype(np.float32)
        scaled[l] *= scale[:, None]
        scaled[l + 1] /= scale[None, :]
    return scaled


@pytest.mark.parametrize("n", [33, 4099])
def test_colour_calls_without_masks_decide_the_gates_alike(n):
    """Points whose input makes one pre-activation of the first layer cancel to its rounding errors.  The forward call
    without masks is the masked one to the last bit, and the backward call without masks takes the gates that the masked
    forward call wrote: one gate the other way is a term of 0.3 / 8 of a point's adjoint and more, the two backward kernels
    differ by 2e-5."""
    rng = np.random.default_rng(n)
    c, W, pos, nrm, dirs, y = colour_inputs(n, rng)
    neuron = rng.integers(0, 64, size=n)
    cin = o.color_input(pos, nrm.astype(np.float64), dirs, y.astype(np.float64), 1)
    weights = W[0].astype(np.float64)[neuron]
    last = weights[:, 37]
    ok = np.abs(last) > 0.03
    y[ok, 15] -= (np.sum(weights * cin, axis=1)[ok] / last[ok]).astype(np.float32)
    cin = o.color_input(pos, nrm.astype(np.float64), dirs, y.astype(np.float64), 1)
    z, size = np.sum(weights * cin, axis=1), np.sum(np.abs(weights * cin), axis=1)
    assert np.mean(np.abs(z) < 2.0 ** -22 * size) > 0.5
    args, Wg = (cuda(pos), cuda(nrm), cuda(dirs), cuda(y)), [cuda(w) for w in W]
    kept = torch.zeros(2, n, 2, dtype=torch.int32, device="cuda")
    rgb, plain = torch.empty(n, 3, device="cuda"), torch.empty(n, 3, device="cuda")
    nb.color_fwd(c, *args, Wg, n, rgb, masks=kept)
    nb.color_fwd(c, *args, Wg, n, plain)
    assert torch.equal(rgb, plain)
    d_rgb = cuda(rng.choice([-1.0, 1.0], size=(n, 3)).astype(np.float32))
    got = []
    for masks in (kept, None):
        d_y, d_normal, d_pos = torch.empty(n, 16, device="cuda"), torch.zeros(n, 3, device="cuda"), torch.empty(n, 3, device="cuda")
        nb.color_bwd(c, *args, Wg, rgb, d_rgb, None, n, [torch.zeros_like(w) for w in Wg], d_y, d_normal, d_pos, masks=masks)
        got.append(torch.cat([d_y, d_normal, d_pos], dim=1).double())
    norm = got[0].norm(dim=1)
    off = (got[1] - got[0]).norm(dim=1) / norm.clamp_min(1e-3 * float(norm.mean()))
    assert float(off.max()) <= 5e-3


@pytest.mark.parametrize("masks", [False, True])
def test_colour_forward_whatever_the_scale_of_a_neuron(masks):
    """Factors of two between a neuron's weights and those that read it change no bit: every element keeps 24 bits of its
    own, whatever its neighbours in the vector or the matrix are."""
    n, rng = 1031, np.random.default_rng(7)
    c, W, pos, nrm, dirs, y = colour_inputs(n, rng)
    got = []
    for mats in (W, without_neuron_scales(rng, W)):
        got.append(torch.empty(n, 3, device="cuda"))
        kept = torch.zeros(2, n, 2, dtype=torch.int32, device="cuda") if masks else None
        nb.color_fwd(c, cuda(pos), cuda(nrm), cuda(dirs), cuda(y), [cuda(w) for w in mats], n, got[-1], masks=kept)
    assert torch.equal(*got)


@pytest.mark.parametrize("levels,hidden,masks,row0", [(16, 2, False, -24), (16, 2, True, -24), (16, 1, False, 30), (8, 2, False, -24), (8, 1, False, -40)])
def test_sdf_forward_whatever_the_scale_of_a_neuron(levels, hidden, masks, row0):
    """As for the colours: hidden neurons scaled by powers of two change no bit of the values, dd/de and the normals, and
    neither does the size of the SDF's row beside the fifteen feature rows (undone afterwards, exactly)."""
    import dataclasses
    n, rng = 1031, np.random.default_rng(levels + hidden)
    cfg = wl.make_config(2 if levels == 16 else 1)
    cfg = dataclasses.replace(cfg, sdf_dims=[2 * levels] + [64] * hidden + [16])
    c = nb.make_config(cfg)
    H = [(rng.normal(size=(o_, i)) * (2.0 / i) ** 0.5).astype(np.float32) for i, o_ in zip(cfg.sdf_dims, cfg.sdf_dims[1:])]
    other = without_neuron_scales(rng, H)
    other[-1][0] = np.ldexp(other[-1][0], row0)
    pos, enc, jac = (cuda(rng.normal(size=k).astype(np.float32)) for k in ((n, 3), (levels, n, 2), (levels, 3, n, 2)))
    pos.sigmoid_()
    tables = cuda(rng.normal(size=(levels, cfg.table_size, 2)).astype(np.float32) * 0.1)
    if cfg.table_dtype == "f16":
        tables = tables.half()
    found = []
    for mats, back in ((H, 0), (other, -row0)):
        y, q, normal, sdf = (torch.empty(*k, device="cuda") for k in ((n, 16), (levels, n, 2), (n, 3), (n,)))
        kept = torch.zeros(2, n, 2, dtype=torch.int32, device="cuda") if masks else None
        Hg = [cuda(m) for m in mats]
        nb.sdf_fwd_grad(c, enc, jac, Hg, n, y, q, normal, masks=kept)
        nb.sdf_values(c, pos, tables, Hg, n, torch.empty(levels * n * 2, device="cuda"), sdf)
        found.append([y[:, 0] * 2.0 ** back, y[:, 1:], q * 2.0 ** back, normal * 2.0 ** back, sdf * 2.0 ** back])
    for a, b in zip(*found):
        assert torch.equal(a, b) and bool(a.any()) and bool(torch.isfinite(a).all())


@pytest.mark.parametrize("levels,hidden", [(16, 2), (8, 1)])
def test_sdf_forward_is_the_same_with_and_without_masks(levels, hidden):
    """Whether the masks are wanted changes no bit of the results."""
    import dataclasses
    n = 257 * 32 + 7
    cfg = wl.make_config(2 if levels == 16 else 1)
    cfg = dataclasses.replace(cfg, sdf_dims=[2 * levels] + [64] * hidden + [16])
    gen = torch.Generator(device="cuda").manual_seed(levels)
    randn = lambda *shape: torch.randn(*shape, device="cuda", generator=gen)
    H = [randn(o_, i) * (2.0 / i) ** 0.5 for i, o_ in zip(cfg.sdf_dims, cfg.sdf_dims[1:])]
    enc, jac = randn(levels, n, 2), randn(levels, 3, n, 2)
    found = []
    for kept in (None, torch.zeros(2, n, 2, dtype=torch.int32, device="cuda")):
        found.append([torch.empty(*k, device="cuda") for k in ((n, 16), (levels, n, 2), (n, 3))])
        nb.sdf_fwd_grad(nb.make_config(cfg), enc, jac, H, n, *found[-1], masks=kept)
    assert all(torch.equal(a, b) for a, b in zip(*found))
