"""Lookahead weights of 32 queries at the edges of the kernel's runs: one query,
either side of a round of 32 positions and of the longest run (256), a last round
that the sequence ends in, head counts that are no power of two, every head size.
The weights are fp32 sums in a stated order, so they match the oracle bit for bit."""
import numpy as np
import pytest

import oracle
import paper_2505_22913_amd as mf
from tests.gpu_common import announce, to_dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,B,Hkv,G", [(64, 2, 3, 1), (128, 1, 2, 3), (128, 1, 1, 8), (256, 1, 2, 4)])
def test_lookahead_runs_bit_exact(d, B, Hkv, G):
    import torch
    for n in (1, 31, 32, 33, 63, 64, 65, 255, 257, 600):
        announce(f"lookahead runs d={d} n={n} G={G}")
        rng = np.random.default_rng(n + d)
        q = rng.standard_normal((B, Hkv * G, n, d), dtype=np.float32).astype(np.float16)
        got = mf.mustafar_query_lookahead(to_dev(q), Hkv)
        torch.cuda.synchronize()
        assert np.array_equal(got.cpu().numpy(), oracle.query_lookahead(q, Hkv, 32)), n


@pytest.mark.parametrize("d", [64, 128])
def test_long_runs_match_ordered_sums(d):
    # Enough streams that the runs are 256 positions long; the reference adds the
    # positions one after the other in fp32.
    import torch
    B, Hkv, n = 16, 16, 2100 if d == 128 else 4200
    q = torch.randn((B, Hkv, n, d), device="cuda").half()
    announce(f"lookahead long runs d={d}")
    got = mf.mustafar_query_lookahead(q, Hkv)
    a = torch.nn.functional.pad(q.abs().float(), (0, 0, 0, 31))
    want = torch.zeros((B, Hkv, n, d), device="cuda")
    for u in range(32):
        want += a[:, :, u:u + n]
    assert torch.equal(got, want)
