"""Filter and embedding kernels at the edges of their dispatch: input widths,
folded and unfolded LayerNorm gains, and unit, workgroup and run remainders."""
import numpy as np
import pytest
import torch

from paper_2402_09633_amd import inputs as I
from tests.gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    from paper_2402_09633_amd import gnn
    return gnn


def set_gains(views, prefix, kind, rng):
    """Gains with signs (folded), or so uneven that they are not folded."""
    for k in (".0.g", ".1.g"):
        g = views[prefix + k]
        g *= rng.choice([-1.0, 1.0], g.size).astype(np.float32)
        if kind == "uneven":
            g[3] = 1e-4
        if kind == "zero":
            g[5] = 0.0


@pytest.mark.parametrize("kind", ["signs", "uneven", "zero"])
@pytest.mark.parametrize("H", [64, 128])
@pytest.mark.parametrize("F", [1, 3, 5, 16])
def test_filter_widths_and_gains(G, oracle_mod, F, H, kind):
    rng = np.random.default_rng(F * H)
    n, e = 700, 4133
    x = rng.normal(size=(n, F)).astype(np.float32)
    ei = rng.integers(0, n, size=(2, e)).astype(np.int32)
    w = I.make_filter_weights(F, H, 11, affine_noise=0.3)
    set_gains(I.filter_blob_views(w, F, H), "filter", kind, rng)
    f = G.gnn_filter_create(w, G.make_filter_dims(F, H))
    try:
        sc = torch.empty(e, device="cuda")
        out = torch.empty(2 * e, dtype=torch.int32, device="cuda")
        k = G.gnn_filter_apply(f, dev(x), dev(ei), n, e, 0.5, sc, out)
        s = sc.cpu().numpy()
    finally:
        G.gnn_filter_destroy(f)
    ref, _ = oracle_mod.filter_edges(w, x, ei, H, 0.5)
    np.testing.assert_allclose(s, ref, rtol=0, atol=2e-6)  # the bound of the parity tests
    np.testing.assert_array_equal(out.cpu().numpy()[:2 * k].reshape(2, k),
                                  ei[:, s > np.float32(0.5)])


@pytest.mark.parametrize("e", [1, 31, 32, 33, 511, 513, 32 * 256, 32 * 256 + 1, 32 * 2048 + 1,
                               600_001])
def test_filter_compaction_remainders(G, e):
    """Kept edges of every run length equal a compaction of the same scores,
    scores given or not, from none kept to all."""
    rng = np.random.default_rng(e)
    n = 300
    x, ei = dev(rng.normal(size=(n, 3)).astype(np.float32)), rng.integers(0, n, (2, e))
    ei = dev(ei.astype(np.int32))
    f = G.gnn_filter_create(I.make_filter_weights(3, 64, 5, 0.2), G.make_filter_dims(3, 64))
    try:
        sc = torch.empty(e, device="cuda")
        out = torch.empty(2 * e, dtype=torch.int32, device="cuda")
        G.gnn_filter_apply(f, x, ei, n, e, 0.5, sc, out)
        for thr in (-1.0, float(sc.median()), 2.0):
            want = ei[:, sc > thr]
            for scores in (sc.clone(), None):
                out.fill_(-7)
                k = G.gnn_filter_apply(f, x, ei, n, e, thr, scores, out)
                assert k == want.shape[1]
                assert torch.equal(out[:2 * k].view(2, k), want)
                assert bool((out[2 * k:] == -7).all())
    finally:
        G.gnn_filter_destroy(f)


@pytest.mark.parametrize("kind", ["signs", "uneven", "zero"])
@pytest.mark.parametrize("F,H,D,n", [(3, 128, 8, 70_001), (3, 64, 8, 33), (1, 64, 1, 31),
                                     (4, 128, 16, 32), (16, 64, 7, 8193), (3, 128, 12, 1)])
def test_embedding_widths_and_gains(G, oracle_mod, F, H, D, n, kind):
    rng = np.random.default_rng(n)
    x = rng.normal(size=(n, F)).astype(np.float32)
    w = I.make_embed_weights(F, H, D, 13, affine_noise=0.3)
    set_gains(I.embed_blob_views(w, F, H, D), "embed", kind, rng)
    m = G.Embedder(w, G.make_embed_dims(F, H, D))
    try:
        z = m(dev(x)).cpu().numpy()
        # rows that do not start on a 16-byte boundary
        buf = torch.full((n * D + 3,), 9.0, device="cuda")
        z2 = buf[1:1 + n * D].view(n, D)
        m(dev(x), z2)
        assert np.array_equal(z2.cpu().numpy(), z)
        assert buf[0] == 9.0 and bool((buf[1 + n * D:] == 9.0).all())
    finally:
        m.close()
    ref = oracle_mod.embed(w, x, H, D)
    # sums of H fp32 terms of O(1): a few 2^-24 sqrt(H) |z|, far below 1e-5
    np.testing.assert_allclose(z, ref, rtol=0, atol=1e-5 * max(1.0, np.abs(ref).max()))


def embed_exact(w, x, F, H, D):
    """z, and per output the sum of its terms' magnitudes, in 64 bits."""
    p = {k: torch.as_tensor(v.astype(np.float64)) for k, v in I.embed_blob_views(w, F, H, D).items()}
    a = torch.as_tensor(x.astype(np.float64))
    for k in ("embed.0", "embed.1"):
        y = a @ p[k + ".W"].T + p[k + ".b"]
        y = torch.nn.functional.layer_norm(y, (H,), p[k + ".g"], p[k + ".beta"], 1e-5)
        a = torch.relu(y)
    W, b = p["embed.2.W"], p["embed.2.b"]
    return (a @ W.T + b).numpy(), (a @ W.abs().T + b.abs()).numpy()


@pytest.mark.parametrize("kind", ["rows", "tiny_rows", "huge_gain", "huge_rows", "one_large_entry",
                                  "tiny_layer", "huge_hidden"])
@pytest.mark.parametrize("H", [64, 128])
def test_embedding_output_rows_of_any_size(G, H, kind):
    """Every output keeps fp32's precision whatever the sizes of its row, of
    the other rows and of the gains that are folded into it."""
    F, D, n = 3, 8, 4001
    rng = np.random.default_rng(H)
    x = rng.normal(size=(n, F)).astype(np.float32)
    w = I.make_embed_weights(F, H, D, 13, affine_noise=0.3)
    v = I.embed_blob_views(w, F, H, D)
    W, b = v["embed.2.W"], v["embed.2.b"]
    b *= 1e-3
    if kind == "rows":
        s = 2.0 ** -np.array([0, 4, 12, 16, 20, 24, 28, 32])
        W *= s[:, None]
        b *= s
    elif kind == "tiny_rows":
        s = 2.0 ** -np.array([0, 45, 60, 80, 100, 0, 1, 2])
        W *= s[:, None]
        b *= s
    elif kind == "huge_gain":  # |g| W past 2^56
        v["embed.1.g"][:] *= 1e20
        v["embed.1.beta"][:] *= 1e20
    elif kind == "huge_rows":
        W[1] *= 1e25
        W[3] *= 2.0 ** 110
    elif kind == "one_large_entry":  # ... of a feature that is never active
        v["embed.1.beta"][7] = -40.0 * abs(v["embed.1.g"][7])
        W[:, 7] *= 2.0 ** np.array([0, 8, 14, 18, 22, 26, 30, 34])
    elif kind == "tiny_layer":
        W *= 2.0 ** -70
        b *= 2.0 ** -70
    elif kind == "huge_hidden":  # layer 1 times the first gains leaves its records' scale
        v["embed.0.g"][:] *= 1000.0
        v["embed.1.W"][:] *= 2.0 ** 57
        v["embed.1.b"][:] = 0.0
    m = G.Embedder(w, G.make_embed_dims(F, H, D))
    try:
        z = m(dev(x)).cpu().numpy().astype(np.float64)
    finally:
        m.close()
    ref, mag = embed_exact(w, x, F, H, D)
    # the hidden outputs' own error (about 1e-6 of the largest, under the
    # parity bound 1e-5) times the terms' magnitudes; the largest terms also
    # cover points where few features are active
    scale = np.maximum(mag, mag.max(axis=0, keepdims=True) * 1e-1)
    err = np.abs(z - ref) / scale
    assert np.isfinite(z).all()
    assert err.max() <= 1e-5, err.max(axis=0)
