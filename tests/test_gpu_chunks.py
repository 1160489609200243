"""Bulk compression at the edges of its chunks, which are 2, 4, 8 or 16 waves of 32
tokens (64 at d = 64) by head size and stream count: one token either side of every
chunk width, in one call and in two (the second starts at the first's length), for
selected bitmaps too. Bit for bit against the oracle."""
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
    # 2:4 pruning: the packing runs on bitmaps that another kernel selected.
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
