"""Window steps on either side of the stream count up to which one workgroup takes a
whole batch entry: every entry's caches, ring and counters against the same entry
stepped alone in a window of fewer streams, with entries that sit steps out."""
import numpy as np
import pytest

import paper_2505_22913_amd as mf
from paper_2505_22913_amd import synth
from tests.gpu_common import announce, read_cache

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("d,H", [(64, 1), (128, 8), (128, 9), (256, 3), (64, 20)])
def test_streams_of_an_entry_step_alike(d, H, weighted):
    import torch
    B, W, n, steps = 3, 32, 40, 45
    lens = [40, 5, 33]
    K, V = synth.make_kv_torch(B, H, n + steps, d, 3)
    g = torch.Generator(device="cuda")
    g.manual_seed(1)
    q = torch.randn((steps, B, H, d), generator=g, device="cuda").half()

    def run(hs):
        ks, vs = K[:, hs].contiguous(), V[:, hs].contiguous()
        h = ks.shape[1]
        Kc, Vc = mf.CompressedCache(B, h, d, 0.6, n + steps), mf.CompressedCache(B, h, d, 0.7, n + steps)
        win = mf.DenseWindow(B, h, d, W)
        kacc = torch.zeros((B, h, W, d), device="cuda")
        mf.mustafar_window_prefill(win, Kc, Vc, ks[:, :, :n].contiguous(), vs[:, :, :n].contiguous(), lens)
        for i in range(steps):
            act = torch.tensor([1, int(i % 3 != 0), int(i < 30)], dtype=torch.int32, device="cuda")
            kn, vn = ks[:, :, n + i].contiguous(), vs[:, :, n + i].contiguous()
            if weighted:
                mf.mustafar_window_step_weighted(win, Kc, Vc, kn, vn, kacc, active=act)
                mf.mustafar_window_key_weights(q[i][:, hs].contiguous(), win, kacc, active=act)
            else:
                mf.mustafar_window_step(win, Kc, Vc, kn, vn, active=act)
        return read_cache(Kc), read_cache(Vc), win, kacc

    announce(f"steps d={d} H={H} weighted={weighted}")
    whole = run(slice(0, H))
    assert whole[2].n_comp.tolist() == [8 + 45, max(0, 5 + 30 - W), 1 + 30]
    for h in range(H):
        alone = run(slice(h, h + 1))
        for c in range(2):
            for f in ("bitmaps", "offsets", "values"):
                assert np.array_equal(whole[c][f][:, h], alone[c][f][:, 0]), (f, h)
            assert np.array_equal(whole[c]["stream_len"][:, h], alone[c]["stream_len"][:, 0])
        for f in ("len", "head", "n_comp"):
            assert torch.equal(getattr(whole[2], f), getattr(alone[2], f))
        assert torch.equal(whole[2].k[:, h], alone[2].k[:, 0]) and torch.equal(whole[2].v[:, h], alone[2].v[:, 0])
        assert torch.equal(whole[3][:, h], alone[3][:, 0])
