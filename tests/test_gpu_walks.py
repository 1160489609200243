"""The bit walks, which MUSTAFAR_ROUTE_WALKS still takes, over what the default route's
tests cover with the matrix-core kernel: every group size and head size, ring windows of
ragged batches, per-channel caches and a peaked softmax. The same cases and
bounds as those tests, on the other kernel."""
import pytest

import paper_2505_22913_amd as mf
from tests import test_gpu_channel, test_gpu_parity, test_gpu_sink, test_gpu_window
from tests.gpu_common import announce

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def walks():
    mf.mustafar_attn_set_route(mf.ROUTE_WALKS)
    announce("route: walks")
    yield
    mf.mustafar_attn_set_route(mf.ROUTE_DEFAULT)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("sK,sV", [(0.5, 0.7), (0.0, 0.9), (1.0, 0.3)])
def test_one_head(d, sK, sV):
    test_gpu_parity._attn_case(B=2, Hkv=2, G=1, Ns=517, Nd=32, d=d, sK=sK, sV=sV, splits=0, seed=d)
    test_gpu_parity._attn_case(B=1, Hkv=2, G=1, Ns=65, Nd=0, d=d, sK=sK, sV=sV, splits=1, seed=d + 1)
    test_gpu_parity._attn_case(B=1, Hkv=2, G=1, Ns=1000, Nd=5, d=d, sK=sK, sV=sV, splits=3, seed=d + 2)


@pytest.mark.parametrize("W,G,sk,sv", [(32, 1, 0.5, 0.7), (8, 2, 0.7, 0.7), (5, 4, 0.5, 0.5), (16, 8, 0.7, 0.5)])
def test_ragged_ring_windows(W, G, sk, sv):
    test_gpu_window.test_window_lifecycle_ragged(W, G, sk, sv)


@pytest.mark.parametrize("G,d", [(1, 128), (4, 64), (2, 256), (8, 128)])
def test_per_channel_values(G, d):
    test_gpu_channel.test_attention_over_grouped_values(G, d)
    test_gpu_channel.test_attention_over_grouped_values_clustered(G, d)


@pytest.mark.parametrize("G", [1, 4])
@pytest.mark.parametrize("late", [False, True])
def test_sink_softmax(G, late):
    test_gpu_sink.test_sink_softmax_long_context(G, 32768, late, 26.0)
