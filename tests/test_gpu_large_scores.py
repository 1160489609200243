"""Decode attention on scores so large that an ulp of the scaled maximum exceeds 1:
finite fp16 queries and keys whose products are multiples of 2^20, so that every
kernel's fp32 dot products (below 2^24 of that unit) are exact in any order, and the
softmax is 1 at the largest score (shared where it is tied) and 0 elsewhere. Tied
maxima meet inside a segment, across segments and in the window. Against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2505_22913_amd as mf
from tests.gpu_common import ATTN_TOL, announce, attn_error, to_dev

pytestmark = pytest.mark.gpu


def _inputs(B, H, G, n, d, seed):
    rng = np.random.default_rng(seed)
    K = (1024 * rng.integers(-7, 8, (B, H, n, d))).astype(np.float16)
    q = (1024 * rng.choice([-2, -1, 1, 2], (B, H * G, d))).astype(np.float16)
    V = rng.standard_normal((B, H, n, d)).astype(np.float16)
    return q, K, V


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("G", [1, 4])
@pytest.mark.parametrize("sK,scale", [(0.5, 1.0), (0.0, 0.25), (0.7, 0.0)])
def test_sparse(d, G, sK, scale):
    B, H, n, W = 1, 4, 300, 32
    q, K, V = _inputs(B, H, G, n, d, seed=d + G)
    K[:, :, 250] = K[:, :, 17]                # ties across segments, and with the window
    K[:, :, n - 2] = K[:, :, 17]
    nc = n - W
    Kp, Vp = np.ascontiguousarray(K[:, :, :nc]), np.ascontiguousarray(V[:, :, :nc])
    KL, VL = np.ascontiguousarray(K[:, :, nc:]), np.ascontiguousarray(V[:, :, nc:])
    Kc, Vc = mf.CompressedCache(B, H, d, sK, nc), mf.CompressedCache(B, H, d, 0.5, nc)
    mf.mustafar_prune_compress(Kc, to_dev(Kp))
    mf.mustafar_prune_compress(Vc, to_dev(Vp))
    ref = oracle.sparse_decode_attention(q, oracle.compress(Kp, sK), oracle.compress(Vp, 0.5), KL, VL, scale)
    for splits in (0, 1, 3):
        announce(f"large scores sparse d={d} G={G} sK={sK} scale={scale} splits={splits}")
        out = mf.mustafar_sparse_decode_attn(to_dev(q), Kc, Vc, to_dev(KL), to_dev(VL), scale=scale, n_splits=splits)
        err = attn_error(out.cpu().numpy(), ref)
        assert err <= ATTN_TOL, (splits, err)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("G", [1, 4])
@pytest.mark.parametrize("scale", [1.0, 0.0])
def test_dense(d, G, scale):
    B, H, n = 1, 4, 300
    q, K, V = _inputs(B, H, G, n, d, seed=d + G + 1)
    K[:, :, 250] = K[:, :, 17]
    ref = oracle.decode_attention(q, K, V, scale=scale)
    for splits in (0, 1, 3):
        announce(f"large scores dense d={d} G={G} scale={scale} splits={splits}")
        out = mf.mustafar_dense_decode_attn(to_dev(q), to_dev(K), to_dev(V), scale=scale, n_splits=splits)
        err = attn_error(out.cpu().numpy(), ref)
        assert err <= ATTN_TOL, (splits, err)
