"""The bulk compressor's bounded look-back wait, forced to give up from the host.

mustafar_prune_compress_bounded with max_polls = 0 lets no chunk but the first
of a stream read its predecessors' totals, so every stream of more than one
chunk gives up; every kernel still finishes. Checked: the call reports the
give-up in the workspace's status word, the streams are poisoned
(stream_len = MUSTAFAR_STREAM_POISONED), later compressions and appends write
nothing to them, and the decode attention treats their compressed part as
empty (the output equals the oracle's attention over the window alone), while
a healthy cache in the same calls stays bit-exact against the oracle. A
one-chunk compression under the same bound gives up nowhere.
"""
import numpy as np
import pytest

import oracle
import paper_2505_22913_amd as mf
from paper_2505_22913_amd import synth
from tests.gpu_common import ATTN_TOL, all_pairs, announce, attn_error, compare_format, read_cache, to_dev

pytestmark = pytest.mark.gpu


def test_give_up_poisons_the_stream_and_later_calls_skip_it():
    import torch
    announce("look-back give-up forced from the host")
    B, H, d, N, n_more, Nd = 1, 4, 128, 5000, 64, 32
    K, V = synth.make_kv(B, H, N + n_more + 1, d, seed=91)
    KL, VL = synth.make_tail(B, H, Nd, d, seed=91)
    q = synth.make_q(B, H, d, seed=91)
    Kc = mf.CompressedCache(B, H, d, 0.5, N + n_more + 1)
    Vc = mf.CompressedCache(B, H, d, 0.7, N + n_more + 1)
    ws = torch.empty(mf.mustafar_compress_workspace_bytes(B, H, N), dtype=torch.uint8, device="cuda")
    mf.mustafar_prune_compress_bounded(Kc, to_dev(np.ascontiguousarray(K[:, :, :N])), 0, ws=ws)
    assert mf.compress_status(ws) != 0
    lens = read_cache(Kc)["stream_len"]
    assert (lens == mf.STREAM_POISONED).all(), lens
    # the value cache, compressed with the default bound through the same workspace
    mf.mustafar_prune_compress(Vc, to_dev(np.ascontiguousarray(V[:, :, :N])), ws=ws)
    assert mf.compress_status(ws) == 0

    # later calls: a bulk compression and an append write nothing to the poisoned streams
    mf.mustafar_prune_compress(Kc, to_dev(np.ascontiguousarray(K[:, :, N:N + n_more])), ws=ws)
    mf.mustafar_prune_compress(Vc, to_dev(np.ascontiguousarray(V[:, :, N:N + n_more])), ws=ws)
    n = N + n_more
    mf.mustafar_append_kv(Kc, Vc, to_dev(np.ascontiguousarray(K[:, :, n])),
                          to_dev(np.ascontiguousarray(V[:, :, n])))
    n += 1
    got_k, got_v = read_cache(Kc), read_cache(Vc)
    assert (got_k["stream_len"] == mf.STREAM_POISONED).all()
    compare_format(got_v, oracle.compress(np.ascontiguousarray(V[:, :, :n]), 0.7), n, all_pairs(B, H))

    # attention: the poisoned key streams contribute nothing, the window does
    out = mf.mustafar_sparse_decode_attn(to_dev(q), Kc, Vc, to_dev(KL), to_dev(VL))
    empty = np.zeros((B, H, 0, d), np.float16)
    ref = oracle.decode_attention(q, empty, empty, KL, VL)
    err = attn_error(out.cpu().numpy(), ref)
    announce(f"look-back give-up: window-only attention error {err:.2e}")
    assert err <= ATTN_TOL
    # with no window either, every part of the softmax is empty: the output is 0
    out0 = mf.mustafar_sparse_decode_attn(to_dev(q), Kc, Vc, None, None)
    assert not out0.cpu().numpy().any()


@pytest.mark.parametrize("d", [64, 128])
def test_one_chunk_needs_no_look_back(d):
    import torch
    announce(f"look-back bound 0 on one chunk d={d}")
    B, H, N = 2, 3, 64
    K, _ = synth.make_kv(B, H, N, d, seed=92)
    Kc = mf.CompressedCache(B, H, d, 0.5, N)
    ws = torch.empty(mf.mustafar_compress_workspace_bytes(B, H, N), dtype=torch.uint8, device="cuda")
    mf.mustafar_prune_compress_bounded(Kc, to_dev(K), 0, ws=ws)
    assert mf.compress_status(ws) == 0
    compare_format(read_cache(Kc), oracle.compress(K, 0.5), N, all_pairs(B, H))


@pytest.mark.parametrize("d,B,H,n,chunk", [
    (128, 1, 4, 129, 128), (128, 2, 16, 2048, 256), (128, 1, 8, 16384, 512), (128, 16, 32, 65, 64),
    (64, 1, 4, 257, 256), (64, 2, 16, 4096, 512), (64, 1, 16, 16384, 1024), (64, 16, 32, 129, 128),
    (256, 1, 4, 129, 128), (256, 16, 32, 65, 64)])
@pytest.mark.parametrize("grouped", [False, True])
def test_give_up_at_every_chunk_width(d, B, H, n, chunk, grouped):
    # 2, 4, 8 and 16 waves a chunk: with bound 0 a stream's first chunk alone is written
    # and every stream is poisoned; refilled with the default bound it is whole.
    import torch
    n = (n + 31) // 32 * 32 if grouped else n
    announce(f"look-back bound 0 d={d} {B}x{H} streams n={n} grouped={grouped}")
    X, _ = synth.make_kv(B, H, n, d, seed=93)
    x = to_dev(X)
    c = mf.CompressedCache(B, H, d, 0.5, n, grouped=grouped)
    ws = torch.empty(mf.mustafar_compress_workspace_bytes(B, H, n), dtype=torch.uint8, device="cuda")
    mf.mustafar_prune_compress_bounded(c, x, 0, ws=ws)
    assert mf.compress_status(ws) != 0
    got = read_cache(c)
    want = oracle.compress_grouped(X, 0.5) if grouped else oracle.compress(X, 0.5, threads=4)
    assert (got["stream_len"] == mf.STREAM_POISONED).all()
    assert np.array_equal(got["offsets"][:, :, :chunk], want["offsets"][:, :, :chunk])
    assert not got["offsets"][:, :, chunk:].any()
    for b, h in ((0, 0), (B - 1, H - 1)):
        end = int(want["offsets"][b, h, chunk, 0])
        assert np.array_equal(got["values"][b, h, :end], want["values"][b, h, :end])
        assert not got["values"][b, h, end:].any()
    c.desc.n_tokens = 0
    mf.mustafar_prune_compress(c, x, ws=ws)
    assert mf.compress_status(ws) == 0
    compare_format(read_cache(c), want, n, all_pairs(B, H))
