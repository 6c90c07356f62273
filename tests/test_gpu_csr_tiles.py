"""CSR builds at the edges of the sort's tile sizes equal the oracle's."""
import numpy as np
import pytest

from paper_2402_09633_amd import inputs as I
from tests.test_gpu_csr import check

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def G():
    from paper_2402_09633_amd import gnn
    return gnn


@pytest.fixture(scope="module")
def handle(G):
    h = G.gnn_create(I.make_weights(3, 64, 1, 0), G.make_dims(3, 64, 2))
    yield h
    G.gnn_destroy(h)


@pytest.mark.parametrize("e", [2047, 2048, 2049, 8193, (1 << 17) - 1, 1 << 17, (1 << 17) + 1,
                               (1 << 19), (1 << 19) + 1])
@pytest.mark.parametrize("n", [3, 1 << 10, (1 << 10) + 1, 1 << 21])
def test_tile_edges(G, handle, oracle_mod, e, n):
    rng = np.random.default_rng(e + n)
    ei = rng.integers(0, n, (2, e)).astype(np.int32)
    ei[0].sort()  # source order, as events arrive; the destinations are not
    check(G, handle, oracle_mod, ei, n)
