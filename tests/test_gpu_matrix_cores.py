"""The matrix-core attention kernel at the edges of its blocks and staging.

A block is 64 / (d / 64) tokens in groups of 16; a key tile is staged in 16-byte
pieces of 8 values and a block's values in chunks of 512, both bounded by the
sparsity, which also picks the kernel's instance. The cases put the token count
on either side of a group, a block and a segment, and the sparsity at all kept,
each staging bound, a few values per token and none. Tolerance: the fp16 rounding
of p (2^-11 relative) and of the output (2^-11 of max|o|), both below the 2e-3 of
the other attention tests.
"""
import numpy as np
import pytest

import oracle
import paper_2505_22913_amd as mf
from paper_2505_22913_amd import synth
from tests.gpu_common import ATTN_TOL, announce, attn_error, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("sK,sV", [(0.0, 0.0), (0.0, 0.9), (0.35, 0.5), (0.7, 0.3), (0.7, 0.7), (0.97, 1.0), (1.0, 0.5)])
def test_blocks_and_staging_bounds(d, sK, sV):
    import torch
    B, H = 1, 2
    for n, G, splits in ((1, 1, 0), (15, 8, 0), (17, 4, 1), (32, 2, 1), (63, 1, 1), (65, 4, 1), (129, 1, 1), (200, 8, 2)):
        announce(f"matrix cores d={d} s=({sK},{sV}) n={n} G={G} splits={splits}")
        K, V = synth.make_kv(B, H, n, d, seed=n + d)
        q = synth.make_q(B, H * G, d, seed=n)
        Kc, Vc = mf.CompressedCache(B, H, d, sK, n), mf.CompressedCache(B, H, d, sV, n)
        mf.mustafar_prune_compress(Kc, to_dev(K))
        mf.mustafar_prune_compress(Vc, to_dev(V))
        out = mf.mustafar_sparse_decode_attn(to_dev(q), Kc, Vc, n_splits=splits)
        torch.cuda.synchronize()
        ref = oracle.sparse_decode_attention(q, oracle.compress(K, sK), oracle.compress(V, sV),
                                             np.zeros((B, H, 0, d), np.float16), np.zeros((B, H, 0, d), np.float16))
        err = attn_error(out.cpu().numpy(), ref)
        assert err <= ATTN_TOL, (n, G, err)


@pytest.mark.parametrize("d", [64, 128, 256])
def test_full_tiles_beside_empty_ones(d):
    # All kept channels of a token in one tile (the other tiles empty): the widest
    # key tile and offsets that advance by whole tiles.
    import torch
    n, G = 70, 4
    K, V = synth.make_kv(1, 1, n, d, seed=3)
    for j in range(n):
        lo = 64 * (j % (d // 64))
        K[0, 0, j, lo:lo + 64] += np.float16(100) * np.sign(K[0, 0, j, lo:lo + 64])
        V[0, 0, j, lo:lo + 64] += np.float16(100) * np.sign(V[0, 0, j, lo:lo + 64])
    K *= np.float16(0.01)
    q = synth.make_q(1, G, d, seed=5)
    s = max(0.1, 1 - 64 / d)
    Kc, Vc = mf.CompressedCache(1, 1, d, s, n), mf.CompressedCache(1, 1, d, s, n)
    mf.mustafar_prune_compress(Kc, to_dev(K))
    mf.mustafar_prune_compress(Vc, to_dev(V))
    announce(f"matrix cores full tiles d={d}")
    out = mf.mustafar_sparse_decode_attn(to_dev(q), Kc, Vc)
    torch.cuda.synchronize()
    ref = oracle.sparse_decode_attention(q, oracle.compress(K, s), oracle.compress(V, s),
                                         np.zeros((1, 1, 0, d), np.float16), np.zeros((1, 1, 0, d), np.float16))
    assert attn_error(out.cpu().numpy(), ref) <= ATTN_TOL


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_dense_blocks(d, G):
    # The dense kernel's blocks are 32 tokens in two groups of 16; rows past a
    # segment's end repeat its last token. Probabilities in two fp16 parts.
    import torch
    B, H = 2, 2
    for n, splits in ((1, 0), (15, 1), (17, 0), (32, 1), (33, 0), (64, 0), (65, 2), (127, 1), (300, 3), (1000, 0)):
        announce(f"dense blocks d={d} G={G} n={n} splits={splits}")
        K, V = synth.make_kv(B, H, n, d, seed=n + d)
        q = synth.make_q(B, H * G, d, seed=n)
        out = mf.mustafar_dense_decode_attn(to_dev(q), to_dev(K), to_dev(V), n_splits=splits)
        torch.cuda.synchronize()
        err = attn_error(out.cpu().numpy(), oracle.decode_attention(q, K, V))
        assert err <= ATTN_TOL, (n, err)


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("at", [64, 66, 69])
def test_dense_infinite_values(d, at):
    # A value that overflowed to infinity gives an infinite output in its channel (at
    # the token with the largest probability, beside it, and at the last row, which
    # the lanes past the end repeat) and leaves the other channels as they are. In the
    # second segment: the merge weighs the first one's output with zero where it pads.
    import torch
    n, G = 70, 4
    K, V = synth.make_kv(1, 1, n, d, seed=at + d)
    q = synth.make_q(1, G, d, seed=5)
    K[0, 0, 64] = q[0, 0]                    # head 0's largest probability
    ref = oracle.decode_attention(q, K, V)
    V[0, 0, at, 3], V[0, 0, at, d - 1] = np.inf, -np.inf
    announce(f"dense infinite value d={d} at={at}")
    out = mf.mustafar_dense_decode_attn(to_dev(q), to_dev(K), to_dev(V), n_splits=2)
    torch.cuda.synchronize()
    out = out.cpu().numpy()
    assert (out[..., 3] == np.inf).all() and (out[..., d - 1] == -np.inf).all()
    rest = np.r_[0:3, 4:d - 1]
    assert np.abs(out[..., rest] - np.asarray(ref)[..., rest]).max() <= ATTN_TOL * np.abs(ref).max()
