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
