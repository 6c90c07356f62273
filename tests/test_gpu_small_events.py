"""Small events: the launch rules that spread a partial round over the CUs."""
import numpy as np
import pytest
import torch

from gpu_util import assert_logits_close, dev

pytestmark = pytest.mark.gpu

DTYPES = [("fp32", 0), ("bf16", 0), ("bf16", 8)]


@pytest.mark.parametrize("dtype,flags", DTYPES)
@pytest.mark.parametrize("hidden", [64, 128])
def test_spread_and_packed_launches_agree(oracle_mod, dtype, flags, hidden):
    """One event at a time (spread) and a queue of several instances (packed)
    give the same bits around one unit, one unit per CU and the last spread
    size, and the smallest ones match the oracle."""
    from paper_2402_09633_amd import gnn as G
    from paper_2402_09633_amd import inputs as I

    n_cu = torch.cuda.get_device_properties(0).multi_processor_count
    w = I.make_weights(3, hidden, 1, 5, affine_noise=0.1)
    m = G.Model(w, G.make_dims(3, hidden, 2, dtype=G.GNN_BF16 if dtype == "bf16" else G.GNN_FP32,
                               flags=flags))
    s = G.Server(m, 3)
    sizes = [(1, 1), (31, 33), (33, 31), (32 * n_cu - 1, 32 * n_cu + 1),
             (32 * n_cu + 1, 32 * n_cu), (128 * n_cu, 64), (128 * n_cu + 1, 32 * n_cu * 8 + 1)]
    try:
        for k, (n, e) in enumerate(sizes):
            g = I.uniform_graph(n, e, seed=60 + k)
            x, ei = dev(g.x), dev(g.edge_index)
            direct = m(x, ei)
            queued = torch.full((e,), -1.0, device="cuda")
            torch.cuda.synchronize()
            s.wait(s.submit(x, ei, queued))
            assert torch.equal(direct, queued), (n, e)
            if n < 100:
                ref = oracle_mod.forward(w, g.x, g.edge_index, hidden, 2)
                if dtype == "fp32":
                    z = m(x, ei, logits=True).cpu().numpy()
                    assert_logits_close(z, ref["logits"], what=f"{n} nodes, {e} edges")
                else:  # the bf16 bound of every parity test
                    got = direct.cpu().numpy().astype(np.float64)
                    ref_s = 1.0 / (1.0 + np.exp(-np.asarray(ref["logits"], np.float64)))
                    assert np.abs(got - ref_s).max() <= 2e-2, (n, e)
    finally:
        s.close()
        m.close()


def test_calls_in_flight_are_seen():
    """A call finds the GPU shared exactly while another inference, of its own
    model or of another one, is in flight on another stream (spread over the
    CUs, the launches of 10k-hit events of four threads hold back one another's:
    4050 -> 5710 us for four calls each)."""
    from paper_2402_09633_amd import gnn as G
    from paper_2402_09633_amd import inputs as I

    w = I.make_weights(3, 128, 1, 5, affine_noise=0.1)
    a, b = (G.Model(w, G.make_dims(3, 128, 8)) for _ in range(2))
    g, big = I.uniform_graph(2_000, 8_000, seed=1), I.uniform_graph(200_000, 700_000, seed=2)
    x, ei, bx, bei = dev(g.x), dev(g.edge_index), dev(big.x), dev(big.edge_index)
    out, bout = torch.empty(8_000, device="cuda"), torch.empty(700_000, device="cuda")
    s0, s1 = torch.cuda.Stream(), torch.cuda.Stream()
    try:
        a(bx, bei, out=bout, stream=s0)  # (allocates the workspace)
        a(x, ei, out=out, stream=s1)
        torch.cuda.synchronize()
        ref = out.clone()
        torch.cuda.synchronize()
        out.zero_()
        torch.cuda.synchronize()
        for m in (a, b):
            assert not G.gnn_debug_shared(m.handle, s0)
            assert not G.gnn_debug_shared(m.handle, s1)
        for _ in range(4):
            a(bx, bei, out=bout, stream=s0)  # some 15 ms of work
        assert G.gnn_debug_shared(a.handle, s1)  # another stream, the same model
        assert G.gnn_debug_shared(b.handle, s1)  # ... and another one
        assert not G.gnn_debug_shared(a.handle, s0)  # ordered after it: not beside it
        a(x, ei, out=out, stream=s1)
        torch.cuda.synchronize()
        assert torch.equal(out, ref)
        assert not G.gnn_debug_shared(a.handle, s0) and not G.gnn_debug_shared(b.handle, s1)
        b(bx, bei, out=bout, stream=s0)
        b.close()  # waits; a destroyed handle is no longer looked at
        assert not G.gnn_debug_shared(a.handle, s1)
    finally:
        a.close()
        b.close()


def test_capture_beside_running_calls():
    """Looking for other calls breaks no capture, this thread's or another's:
    a call is captured while one of another model runs, and one is issued by
    another thread while the capture is open."""
    import threading

    from paper_2402_09633_amd import gnn as G
    from paper_2402_09633_amd import inputs as I

    w = I.make_weights(3, 128, 1, 5, affine_noise=0.1)
    a, b = (G.Model(w, G.make_dims(3, 128, 2)) for _ in range(2))
    g, big = I.uniform_graph(2_000, 8_000, seed=1), I.uniform_graph(40_000, 150_000, seed=2)
    x, ei, bx, bei = dev(g.x), dev(g.edge_index), dev(big.x), dev(big.edge_index)
    out, bout = torch.zeros(8_000, device="cuda"), torch.zeros(150_000, device="cuda")
    side, cap, other = (torch.cuda.Stream() for _ in range(3))
    try:
        ref, bref = a(x, ei).clone(), b(bx, bei).clone()
        b(x, ei, out=torch.empty(8_000, device="cuda"), stream=other)  # a second workspace of b's
        G.gnn_infer_noalloc(a.handle, x, ei, 2_000, 8_000, out)  # (looks up its scratch)
        torch.cuda.synchronize()
        out.zero_()
        out2 = torch.zeros(8_000, device="cuda")
        torch.cuda.synchronize()
        b(bx, bei, out=bout, stream=side)  # in flight while the capture looks
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=cap, capture_error_mode="thread_local"):
            G.gnn_infer_noalloc(a.handle, x, ei, 2_000, 8_000, out, cap)
            t = threading.Thread(target=lambda: b(x, ei, out=out2, stream=other))
            t.start()
            t.join()
        torch.cuda.synchronize()
        assert torch.equal(bout, bref) and torch.equal(out2, ref)
        for _ in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, ref)
    finally:
        a.close()
        b.close()
