"""Output-aware and 2:4 selection in the bulk compression, where it can go wrong:
ties of every key in a token and over a group's edge, zero weights, scores that
differ only in their low 16 bits, subnormal and largest magnitudes, a token count
that leaves waves of a chunk empty, kept counts per head, appended calls. Bit for bit
against the oracle."""
import numpy as np
import pytest

import oracle
import paper_2505_22913_amd as mf
from tests.gpu_common import all_pairs, announce, compare_format, read_cache, to_dev

pytestmark = pytest.mark.gpu


def _inputs(rng, B, H, n, d):
    x = rng.standard_normal((B, H, n, d), dtype=np.float32).astype(np.float16)
    w = rng.random((B, H, n, d), dtype=np.float32) * 40
    x[..., 0::7, :] = np.float16(1)                       # scores decided by the weights alone
    w[..., 0::7, :] = np.float32(3)
    w[..., 0::7, ::5] += np.float32(2 ** -21) * rng.integers(0, 8, w[..., 0::7, ::5].shape)
    w[..., 1::11, :] = 0                                  # all scores equal (zero)
    x[..., 2::9, :] = rng.choice(np.array([0.0, -0.0, 6e-8, -6e-8, 65504, -65504], np.float16), x[..., 2::9, :].shape)
    return x, w


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("B,H,s", [(1, 2, 0.7), (2, 9, 0.5), (1, 1, 0.97)])
def test_scored_selection_bit_exact(d, B, H, s):
    import torch
    for n in (1, 33, 257, 700):
        announce(f"scored d={d} B={B} H={H} s={s} n={n}")
        rng = np.random.default_rng(n + d)
        x, w = _inputs(rng, B, H, n, d)
        want = oracle.compress_variant(x, "output_aware", k=oracle.keep_count(d, s), weights=w)
        Kc = mf.CompressedCache(B, H, d, s, n)
        m = n // 2 if n > 40 else n
        for lo, hi in ((0, m), (m, n)):
            if hi > lo:
                mf.mustafar_prune_compress_ex(Kc, to_dev(np.ascontiguousarray(x[:, :, lo:hi])), mode=mf.PRUNE_OUTPUT_AWARE,
                                              weights=torch.from_numpy(np.ascontiguousarray(w[:, :, lo:hi])).cuda())
        compare_format(read_cache(Kc), want, n, all_pairs(B, H))


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("skip", [1, 2, 3])
def test_scored_weights_at_any_float(d, skip):
    # The weights need 4-byte alignment only.
    import torch
    B, H, n, s = 1, 2, 77, 0.7
    announce(f"scored weights {4 * skip} bytes into a buffer, d={d}")
    x, w = _inputs(np.random.default_rng(d + skip), B, H, n, d)
    buf = torch.zeros(w.size + 4, dtype=torch.float32, device="cuda")
    wd = buf[skip:skip + w.size].view(w.shape)
    wd.copy_(torch.from_numpy(w))
    assert wd.data_ptr() % 16 == 4 * skip
    Kc = mf.CompressedCache(B, H, d, s, n)
    mf.mustafar_prune_compress_ex(Kc, to_dev(x), mode=mf.PRUNE_OUTPUT_AWARE, weights=wd)
    want = oracle.compress_variant(x, "output_aware", k=oracle.keep_count(d, s), weights=w)
    compare_format(read_cache(Kc), want, n, all_pairs(B, H))


@pytest.mark.parametrize("d", [64, 128, 256])
def test_negative_zero_weights(d):
    # A weight of -0.0 is a zero: bulk and append agree with the oracle.
    import torch
    B, H, n, s = 1, 2, 40, 0.7
    announce(f"scored, weights of -0.0, d={d}")
    x, w = _inputs(np.random.default_rng(d + 9), B, H, n, d)
    w[..., 3::4] = np.float32(-0.0)
    w[:, :, 5] = np.float32(-0.0)
    w[:, :, 6, : d // 2] = np.float32(-0.0)
    wd = torch.from_numpy(w).cuda()
    want = oracle.compress_variant(x, "output_aware", k=oracle.keep_count(d, s), weights=w)
    Kc, Ka = mf.CompressedCache(B, H, d, s, n), mf.CompressedCache(B, H, d, s, n)
    mf.mustafar_prune_compress_ex(Kc, to_dev(x), mode=mf.PRUNE_OUTPUT_AWARE, weights=wd)
    for i in range(n):
        mf.mustafar_append_ex(Ka, to_dev(np.ascontiguousarray(x[:, :, i])), mode=mf.PRUNE_OUTPUT_AWARE,
                              weights=wd[:, :, i].contiguous())
    compare_format(read_cache(Kc), want, n, all_pairs(B, H))
    compare_format(read_cache(Ka), want, n, all_pairs(B, H))


@pytest.mark.parametrize("d", [64, 128, 256])
def test_scored_counts_per_head(d):
    import torch
    B, H, n = 2, 4, 130
    announce(f"scored per head d={d}")
    rng = np.random.default_rng(d)
    x, w = _inputs(rng, B, H, n, d)
    hk = [d // 2, d // 4, 1, 0]
    Kc = mf.CompressedCache(B, H, d, 0.5, n)
    mf.mustafar_prune_compress_ex(Kc, to_dev(x), mode=mf.PRUNE_OUTPUT_AWARE, head_keep=hk,
                                  weights=torch.from_numpy(w).cuda())
    compare_format(read_cache(Kc), oracle.compress_variant(x, "output_aware", head_keep=hk, weights=w), n, all_pairs(B, H))


@pytest.mark.parametrize("d", [64, 128, 256])
@pytest.mark.parametrize("B,H", [(1, 2), (2, 9)])
def test_two_four_ties_bit_exact(d, B, H):
    for n in (1, 65, 300, 700):
        announce(f"2:4 d={d} B={B} H={H} n={n}")
        x, _ = _inputs(np.random.default_rng(n), B, H, n, d)
        Kc = mf.CompressedCache(B, H, d, 0.5, n)
        mf.mustafar_prune_compress_ex(Kc, to_dev(x), mode=mf.PRUNE_2_4)
        compare_format(read_cache(Kc), oracle.compress_variant(x, "2:4"), n, all_pairs(B, H))


@pytest.mark.parametrize("mode", ["output_aware", "2:4"])
@pytest.mark.parametrize("d,n", [(128, 8225), (64, 16449)])
def test_long_streams_take_wide_chunks(d, n, mode):
    # 16 streams of 4096 waves of tokens and more: 8 waves a chunk (the other tests: 4).
    import torch
    B, H = 1, 16
    announce(f"{mode} selection in wide chunks d={d} n={n}")
    x, w = _inputs(np.random.default_rng(d), B, H, n, d)
    Kc = mf.CompressedCache(B, H, d, 0.5, n)
    if mode == "2:4":
        mf.mustafar_prune_compress_ex(Kc, to_dev(x), mode=mf.PRUNE_2_4)
        want = oracle.compress_variant(x, "2:4")
    else:
        mf.mustafar_prune_compress_ex(Kc, to_dev(x), mode=mf.PRUNE_OUTPUT_AWARE, weights=torch.from_numpy(w).cuda())
        want = oracle.compress_variant(x, "output_aware", k=d // 2, weights=w)
    compare_format(read_cache(Kc), want, n, all_pairs(B, H))
