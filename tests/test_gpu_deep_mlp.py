"""The deeper SDF network (neus2_sdf_deep_fwd_grad / neus2_sdf_deep_bwd: a run of layers per launch and
direction, up to eight hidden layers, the depths of the paper's Fig. 7) against the
float64 oracle: (d,g), dd/de and the normal at forward tolerance; every weight gradient, first
order plus the second-order term of Theorem 1, and dL/de at gradient tolerance.  At the depths the
fused kernels hold as well the two paths are also compared with each other."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

from oracle import neus2_oracle as o
from paper_2212_05231_amd import binding as nb, workloads as wl

pytestmark = pytest.mark.gpu

FWD_TOL, GRAD_TOL = 1e-5, 1e-4


def rel(a, b):
    a, b = np.asarray(a, dtype=np.float64), np.asarray(b, dtype=np.float64)
    return float(np.linalg.norm(a - b) / np.linalg.norm(b))


def cuda(x, dtype=torch.float32):
    return torch.as_tensor(np.ascontiguousarray(x)).to("cuda", dtype)


def level_major(e, L):
    n = e.shape[0]
    return cuda(e.reshape(n, L, 2).transpose(1, 0, 2))


def jac_level_major(J, L):
    n = J.shape[0]
    return cuda(J.reshape(n, L, 2, 3).reshape(n, L, 3, 2).transpose(1, 2, 0, 3))     # six values as three pairs per level


def from_level_major(t, n):
    return t.cpu().numpy().transpose(1, 0, 2).reshape(n, -1)


def make_net(rng, enc_dim, hidden):
    dims = [enc_dim] + [64] * hidden + [16]
    return [(rng.normal(size=(dims[i + 1], dims[i])) * (2.0 / dims[i]) ** 0.5).astype(np.float32) for i in range(hidden + 1)]


def oracle_gradients(H64, e, J, d_y, d_normal):
    """Theorem 1 with i = 0, every depth: dH_l = delta_l a_{l-1}^T + S_l^T t_{l-1}^T."""
    K = len(H64)
    y, acts, masks = o.mlp_forward(H64, e)
    S, q = o.mlp_input_gradient(H64, masks, 0)
    dH, d_e, _ = o.mlp_backward(H64, acts, masks, d_y)
    t = np.einsum("nka,na->nk", J, d_normal)
    for l in range(K):
        if l < K - 1:
            dH[l] += S[l].T @ t
            t = masks[l] * (t @ H64[l].T)
        else:
            dH[l][0] += t.sum(axis=0)
    return y, q, dH, d_e


@pytest.mark.parametrize("enc_dim,hidden,n", [(32, 1, 3000 + 5), (32, 2, 2048), (32, 4, 5000 + 17), (32, 8, 4096 + 1), (16, 4, 1000 + 3)])
def test_layer_by_layer_network_against_the_oracle(enc_dim, hidden, n):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(100 + hidden + enc_dim)
    L = enc_dim // 2
    H = make_net(rng, enc_dim, hidden)
    e = rng.normal(size=(n, enc_dim)).astype(np.float32)
    J = (rng.normal(size=(n, enc_dim, 3)) * 0.3).astype(np.float32)
    d_y = (rng.normal(size=(n, 16)) / n).astype(np.float32)
    d_normal = (rng.normal(size=(n, 3)) / n).astype(np.float32)
    Hg = [cuda(h) for h in H]
    enc, jac = level_major(e, L), jac_level_major(J, L)
    ws = torch.empty(nb.sdf_deep_workspace_bytes(len(H), n), dtype=torch.uint8, device="cuda")
    y = torch.empty(n, 16, device="cuda")
    q = torch.full((L, n, 2), 7.0, device="cuda")
    normal = torch.empty(n, 3, device="cuda")
    nb.sdf_deep_fwd_grad(enc_dim, enc, jac, Hg, n, y, q, normal, ws)
    dH = [torch.full_like(h, 0.5) for h in Hg]                     # ADDED into: start from a known value
    d_enc = torch.full((L, n, 2), 7.0, device="cuda")
    ws.fill_(0xFF)                                                 # the backward call needs nothing from the forward call
    nb.sdf_deep_bwd(enc_dim, enc, jac, Hg, cuda(d_y), cuda(d_normal), n, dH, d_enc, ws)
    torch.cuda.synchronize()

    H64 = [h.astype(np.float64) for h in H]
    yr, qr, dHr, der = oracle_gradients(H64, e.astype(np.float64), J.astype(np.float64), d_y.astype(np.float64),
                                        d_normal.astype(np.float64))
    errs = {"y": rel(y.cpu().numpy(), yr), "q": rel(from_level_major(q, n), qr),
            "normal": rel(normal.cpu().numpy(), np.einsum("nk,nka->na", qr, J.astype(np.float64)))}
    for k, v in errs.items():
        assert v <= FWD_TOL, (k, v, errs)
    g = {f"dH{l}": rel(dH[l].cpu().numpy().astype(np.float64) - 0.5, dHr[l]) for l in range(len(H))}
    g["d_enc"] = rel(from_level_major(d_enc, n), der)
    print(f"enc_dim {enc_dim}, {hidden} hidden layers, n {n}:", {k: f"{v:.1e}" for k, v in {**errs, **g}.items()})
    for k, v in g.items():
        assert v <= GRAD_TOL, (k, v, g)


@pytest.mark.parametrize("hidden", [1, 2])
def test_layer_by_layer_and_fused_kernels_agree(hidden):
    """At one and two hidden layers both paths exist: same outputs at the tolerances each is held to."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(7 + hidden)
    n, enc_dim, L = 6000 + 11, 32, 16
    cfg = wl.make_config(2)
    cfg.sdf_dims = [32] + [64] * hidden + [16]
    c = nb.make_config(cfg)
    H = [cuda(h) for h in make_net(rng, enc_dim, hidden)]
    e = rng.normal(size=(n, enc_dim)).astype(np.float32)
    J = (rng.normal(size=(n, enc_dim, 3)) * 0.3).astype(np.float32)
    enc, jac = level_major(e, L), jac_level_major(J, L)
    d_y = cuda(rng.normal(size=(n, 16)) / n)
    d_normal = cuda(rng.normal(size=(n, 3)) / n)
    out = {}
    for path in ("fused", "layers"):
        y, q, normal = torch.empty(n, 16, device="cuda"), torch.empty(L, n, 2, device="cuda"), torch.empty(n, 3, device="cuda")
        dH, d_enc = [torch.zeros_like(h) for h in H], torch.empty(L, n, 2, device="cuda")
        if path == "fused":
            nb.sdf_fwd_grad(c, enc, jac, H, n, y, q, normal)
            nb.sdf_mlp_bwd(c, enc, jac, H, d_y, d_normal, n, dH, d_enc)
        else:
            ws = torch.empty(nb.sdf_deep_workspace_bytes(len(H), n), dtype=torch.uint8, device="cuda")
            nb.sdf_deep_fwd_grad(enc_dim, enc, jac, H, n, y, q, normal, ws)
            nb.sdf_deep_bwd(enc_dim, enc, jac, H, d_y, d_normal, n, dH, d_enc, ws)
        torch.cuda.synchronize()
        out[path] = [t.cpu().numpy() for t in (y, q, normal, d_enc, *dH)]
    for k, (a, b) in enumerate(zip(out["layers"], out["fused"])):
        assert rel(a, b) <= (2 * FWD_TOL if k < 3 else 2 * GRAD_TOL), (k, rel(a, b))


def test_layer_by_layer_calls_reject_what_they_do_not_support():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    assert nb.sdf_deep_workspace_bytes(1, 100) == -1 and nb.sdf_deep_workspace_bytes(10, 100) == -1
    n = 64
    H = [torch.zeros(64, 32, device="cuda"), torch.zeros(16, 64, device="cuda")]
    buf = torch.zeros(16 * n * 6, device="cuda")
    small = torch.zeros(16, dtype=torch.uint8, device="cuda")
    with pytest.raises(RuntimeError):
        nb.sdf_deep_fwd_grad(32, buf, buf, H, n, buf, buf, buf, small)            # workspace too small
    with pytest.raises(RuntimeError):
        nb.sdf_deep_fwd_grad(24, buf, buf, H, n, buf, buf, buf, buf)              # input width


@pytest.mark.parametrize("enc_dim,hidden,n", [(32, 5, 31), (16, 6, 33), (32, 7, 64), (16, 1, 1)])
def test_runs_of_layers_at_their_edges(enc_dim, hidden, n):
    """Six matrices fill a run, seven make two; an even number of matrices leaves no single layer for the last gradient
    launch; tiles of 32 points that are not full, just begun and exactly full."""
    test_layer_by_layer_network_against_the_oracle(enc_dim, hidden, n)


@pytest.mark.parametrize("n_mats,enc_dim,n", [(2, 32, 1), (3, 16, 33), (7, 32, 64), (9, 32, 95)])
def test_workspace_holds_what_is_used_and_no_more(n_mats, enc_dim, n):
    """Two vectors of 32 floats per lane and layer (the encoding serves as the first one's), one per order handed on, a mask
    word per lane and hidden layer; nothing behind the size asked for is written."""
    lanes = (n + 31) // 32 * 64
    size = nb.sdf_deep_workspace_bytes(n_mats, n)
    assert size == 4 * lanes * (32 * (2 * n_mats + 1) + n_mats - 1)
    rng = np.random.default_rng(n)
    L, H = enc_dim // 2, [cuda(h) for h in make_net(rng, enc_dim, n_mats - 1)]
    held = torch.full((size + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
    enc, jac, d_y, d_normal = (torch.randn(*s, device="cuda") for s in ((L, n, 2), (L, 3, n, 2), (n, 16), (n, 3)))
    y, q, normal, d_enc = (torch.zeros(*s, device="cuda") for s in ((n, 16), (L, n, 2), (n, 3), (L, n, 2)))
    nb.sdf_deep_fwd_grad(enc_dim, enc, jac, H, n, y, q, normal, held[:size])
    nb.sdf_deep_bwd(enc_dim, enc, jac, H, d_y, d_normal, n, [torch.zeros_like(h) for h in H], d_enc, held[:size])
    assert bool((held[size:] == 0x5A).all()) and bool((held[:size] != 0x5A).any())


@pytest.mark.parametrize("enc_dim,hidden", [(32, 1), (32, 5), (32, 6), (32, 7), (32, 8), (16, 8)])
def test_forward_whatever_the_scale_of_a_neuron(enc_dim, hidden):
    """Hidden neurons scaled by powers of two (a row up, the column that reads it down) and another size of the SDF's row
    beside the feature rows change no bit of the values, dd/de and the normals (the row's size undone exactly): every element
    keeps 24 bits of its own, in one run of layers and in two."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    rng = np.random.default_rng(enc_dim + hidden)
    n, L = 32 * 16 + 5, enc_dim // 2
    H = make_net(rng, enc_dim, hidden)
    other = [h.copy() for h in H]
    for l in range(hidden):
        scale = np.ldexp(np.float32(1), rng.integers(-30, 31, size=64)).astype(np.float32)
        other[l] *= scale[:, None]
        other[l + 1] /= scale[None, :]
    other[-1][0] = np.ldexp(other[-1][0], -24)
    enc, jac = cuda(rng.normal(size=(L, n, 2))), cuda(rng.normal(size=(L, 3, n, 2)) * 0.3)
    ws = torch.empty(nb.sdf_deep_workspace_bytes(len(H), n), dtype=torch.uint8, device="cuda")
    found = []
    for mats, back in ((H, 0), (other, 24)):
        y, q, normal = torch.empty(n, 16, device="cuda"), torch.empty(L, n, 2, device="cuda"), torch.empty(n, 3, device="cuda")
        nb.sdf_deep_fwd_grad(enc_dim, enc, jac, [cuda(m) for m in mats], n, y, q, normal, ws)
        found.append([y[:, 0] * 2.0 ** back, y[:, 1:], q * 2.0 ** back, normal * 2.0 ** back])
    for a, b in zip(*found):
        assert torch.equal(a, b) and bool(a.any()) and bool(torch.isfinite(a).all())
