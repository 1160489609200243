"""Bulk compression at the edges of its chunks, which are 2, 4, 8 or 16 waves of 32
tokens (64 at d = 64) by head size, streams and tokens: one token either side of every
chunk width, in one call and in two (the second starts at the first's length), with 2:4
selection, and for bitmaps that another kernel selected (per-channel pruning). Bit for
bit against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2505_22913_amd as mf
from paper_2505_22913_amd import synth
from tests.gpu_common import all_pairs, announce, compare_format, read_cache, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("B,H", [(1, 2), (3, 7)])
def test_chunk_edges_bit_exact(d, B, H):
    for n in (127, 129, 255, 257, 511, 513, 1025):
        announce(f"chunks d={d} B={B} H={H} n={n}")
        K, _ = synth.make_kv(B, H, n, d, seed=n)
        want = oracle.compress(K, 0.6)
        Kc = mf.CompressedCache(B, H, d, 0.6, n)
        mf.mustafar_prune_compress(Kc, to_dev(K))
        compare_format(read_cache(Kc), want, n, all_pairs(B, H))
        m = n // 3
        Kc.desc.n_tokens = 0
        mf.mustafar_prune_compress(Kc, to_dev(np.ascontiguousarray(K[:, :, :m])))
        mf.mustafar_prune_compress(Kc, to_dev(np.ascontiguousarray(K[:, :, m:])))
        compare_format(read_cache(Kc), want, n, all_pairs(B, H))


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("B,H", [(73, 7), (32, 16)])
def test_chunk_edges_either_side_of_many_streams(d, B, H):
    # 511 streams take the wide chunks, 512 the narrow ones.
    for n in (63, 130):
        announce(f"chunks d={d} B={B} H={H} n={n}")
        K, _ = synth.make_kv(B, H, n, d, seed=n)
        Kc = mf.CompressedCache(B, H, d, 0.6, n)
        mf.mustafar_prune_compress(Kc, to_dev(K))
        compare_format(read_cache(Kc), oracle.compress(K, 0.6), n, all_pairs(B, H))


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("B,H", [(1, 2), (3, 7)])
def test_selected_bitmaps_at_chunk_edges(d, B, H):
    # 2:4 pruning, selected in the compression itself.
    for n in (129, 255, 513, 1025):
        announce(f"chunks 2:4 d={d} B={B} H={H} n={n}")
        K, _ = synth.make_kv(B, H, n, d, seed=n + 1)
        Kc = mf.CompressedCache(B, H, d, 0.5, n)
        mf.mustafar_prune_compress_ex(Kc, to_dev(K), mode=mf.PRUNE_2_4)
        got = read_cache(Kc)
        grp = np.abs(K.astype(np.float32)).reshape(B, H, n, d // 4, 4)
        order = np.argsort(-grp, axis=-1, kind="stable")       # ties to the lower channel
        keep = np.zeros(grp.shape, bool)
        np.put_along_axis(keep, order[..., :2], True, axis=-1)
        bits = keep.reshape(B, H, n, d // 64, 64)
        want = np.packbits(bits, axis=-1, bitorder="little").view(np.uint64)[..., 0]
        assert np.array_equal(got["bitmaps"][:, :, :n], want)
        # every tile keeps 32 values: tile i of a stream starts at 32 i
        offs = np.arange(n * (d // 64), dtype=np.uint32).reshape(n, -1) * 32
        assert (got["offsets"][:, :, :n] == offs).all() and (got["stream_len"] == n * d // 2).all()
        vals = K.view(np.uint16).reshape(B, H, -1)[bits.reshape(B, H, -1)].reshape(B, H, -1)
        assert np.array_equal(got["values"][:, :, :n * d // 2], vals)


@pytest.mark.parametrize("d,B,H,n", [(128, 1, 4, 96), (128, 1, 4, 128), (128, 1, 4, 160), (128, 2, 16, 2048), (128, 2, 16, 2080),
                                     (128, 1, 8, 16352), (128, 1, 8, 16416), (128, 16, 32, 64), (128, 16, 32, 96),
                                     (64, 1, 4, 224), (64, 1, 4, 288), (64, 2, 16, 4128), (64, 1, 16, 16416), (64, 16, 32, 160),
                                     (256, 1, 4, 96), (256, 1, 4, 160), (256, 16, 32, 96)])
def test_per_channel_at_chunk_edges(d, B, H, n):
    # A group of 32 tokens either side of a chunk of 2, 4, 8 and 16 waves; then in two calls.
    announce(f"chunks per channel d={d} B={B} H={H} n={n}")
    V, _ = synth.make_kv(B, H, n, d, seed=n + 2)
    want = oracle.compress_grouped(V, 0.7, threads=4)
    c = mf.CompressedCache(B, H, d, 0.7, n, grouped=True)
    mf.mustafar_prune_compress(c, to_dev(V))
    compare_format(read_cache(c), want, n, all_pairs(B, H))
    c.desc.n_tokens = 0
    m = n // 64 * 32
    mf.mustafar_prune_compress(c, to_dev(np.ascontiguousarray(V[:, :, :m])))
    mf.mustafar_prune_compress(c, to_dev(np.ascontiguousarray(V[:, :, m:])))
    compare_format(read_cache(c), want, n, all_pairs(B, H))
