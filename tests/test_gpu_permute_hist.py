"""The permutation of batches of more than 4096 tokens: over the block histograms in one launch up to 32768 counters, by scan and
scatter beyond, at the edge between the two, with one counter column per thread and with many.  Integers bit for bit."""
import pytest

from test_gpu_parity import _runner, check_routing, make

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,T,k", [(64, 16128, 2), (64, 16129, 2), (1, 8193, 1), (8, 116481, 2), (7, 131073, 1), (37, 4127, 2)])
def test_permutation_parity(n, T, k):
    inp = make("permute", 32, (32,) * n, T, "bf16", k, seed=31)
    r = _runner(inp)
    r.route()
    check_routing(inp, r.routing_host())
