"""Window prefill of many entries at once: with a workspace for all of them, with
the smallest allowed one (fewer entries a launch), and entry by entry through one-
entry windows, every cache, ring and state must come out the same. Lengths from 0
over either side of the window and of a chunk."""
import numpy as np
import pytest

import paper_2505_22913_amd as mf
from paper_2505_22913_amd import synth
from tests.gpu_common import announce, read_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("grouped", [False, True])
@pytest.mark.parametrize("d,H", [(64, 3), (128, 2), (256, 1)])
def test_entries_together_and_alone(d, H, grouped):
    import torch
    W = 64 if grouped else 32
    lens = [700, 0, 1, W, W + 1, 31, 33, 545, 64, 289, 577, 96, 700, 2, 513, 512, 65, 320, 33]
    B, n_max = len(lens), 700
    K, V = synth.make_kv_torch(B, H, n_max, d, 7)

    def caches(B):
        return (mf.CompressedCache(B, H, d, 0.6, n_max), mf.CompressedCache(B, H, d, 0.7, n_max, grouped=grouped),
                mf.DenseWindow(B, H, d, W))

    one = [caches(1) for _ in lens]
    for b, n in enumerate(lens):
        announce(f"prefill alone d={d} grouped={grouped} entry {b} n={n}")
        Kc, Vc, win = one[b]
        mf.mustafar_window_prefill(win, Kc, Vc, K[b:b + 1], V[b:b + 1], [n])
    for ws in (None, torch.empty(mf.mustafar_compress_workspace_bytes(1, H, n_max), dtype=torch.uint8, device="cuda")):
        announce(f"prefill together d={d} grouped={grouped} ws={'default' if ws is None else 'smallest'}")
        Kc, Vc, win = caches(B)
        mf.mustafar_window_prefill(win, Kc, Vc, K, V, lens, ws=ws)
        assert Kc.n_tokens == max(c[0].n_tokens for c in one) and win.max_len == max(c[2].max_len for c in one)
        for b, n in enumerate(lens):
            for got, want in ((Kc, one[b][0]), (Vc, one[b][1])):
                g, w = read_cache(got), read_cache(want)
                for f in ("bitmaps", "offsets"):
                    assert np.array_equal(g[f][b, :, :n_max], w[f][0, :, :n_max]), (f, b)
                if n > W:
                    assert np.array_equal(g["stream_len"][b], w["stream_len"][0])
                assert np.array_equal(g["values"][b], w["values"][0]), b
            for f in ("len", "head", "n_comp", "k", "v"):
                assert torch.equal(getattr(win, f)[b], getattr(one[b][2], f)[0]), (f, b)
