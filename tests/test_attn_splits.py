"""The split of a sparse call that leaves it to the library (mustafar_sparse_attn_splits,
host only): of the whole-block splits that a default-sized workspace holds it is the
cheapest by the rule's own cost (rounds of resident waves times a wave's blocks and its
start; the window calls over several batch entries allow for shorter ones), it is kept when passed back,
and shrinks to what a smaller workspace holds. d = 128, where the resident waves are
11 a CU with both caches at 70% and 8 with 50% keys (LDS and registers)."""
import ctypes
from fractions import Fraction

import pytest

import paper_2505_22913_amd as mf
from tests.test_abi_host import _fake_cache, lib  # noqa: F401  (fixture)


def _taken(lib, Kc, Vc, Hq, ws, window=1):
    return lib.mustafar_sparse_attn_splits(ctypes.byref(Kc), ctypes.byref(Vc), Hq, window, ws)


@pytest.mark.parametrize("sK,sV,waves", [(0.7, 0.7, 11), (0.5, 0.7, 8)])
@pytest.mark.parametrize("window", [0, 1])
@pytest.mark.parametrize("B,H,G", [(1, 32, 1), (16, 32, 1), (8, 32, 1), (4, 8, 4), (1, 8, 8), (3, 5, 2), (1, 1, 8)])
def test_default_split_by_cost(lib, B, H, G, window, sK, sV, waves):  # noqa: F811
    slots, Hq = 256 * waves, H * G
    for n in (1, 64, 65, 700, 1500, 2500, 4096, 6000, 9001, 16384, 32768, 131072):
        Kc, Vc = _fake_cache(B, H, 128, sK, n)[0], _fake_cache(B, H, 128, sV, n)[0]
        Kc.n_tokens = Vc.n_tokens = n
        ws = lib.mustafar_attn_workspace_bytes(B, Hq, H, 128, n, 0)
        most = max(lib.mustafar_attn_default_splits(B, Hq, H, n, k) for k in (mf.ATTN_SPARSE, mf.ATTN_DENSE))
        blocks = -(-n // 64)

        def cost(segs):
            k, streams, per = -(-blocks // segs), B * H, segs + 1
            r = Fraction(streams * per, slots)
            full = 1 if r <= Fraction(17, 16) else r.numerator // r.denominator
            part = r - full if r - full > Fraction(1, 16) else 0
            if not window or B == 1:
                return (full + (part > 0)) * (k + 1)
            half = Fraction(1, 2)
            few = max(1, Fraction(streams * (6 * segs + 10), 10 * slots))
            met = 1 if streams < 64 or r <= Fraction(17, 16) or per % 4 else Fraction(11, 8) if per % 8 else Fraction(7, 4)
            over = half + k * min(1, part * 3 / 2) if part else 0
            return full * (k + half) + over + met * few * (k + half) / 4

        got = _taken(lib, Kc, Vc, Hq, ws, window)
        assert 1 <= got <= most and got == -(-blocks // -(-blocks // got))
        for k in (1, 2, 3, 4, 5, 6, 7, 8, 10, 12, 14, 16, 20, 24, 32):
            segs = -(-blocks // k)
            if segs <= most:
                assert float(cost(got)) <= float(cost(segs)) * (1 + 1e-12), (n, got, segs)
        # a workspace of the sparse kind's default only: no more than it holds
        counted = lib.mustafar_attn_default_splits(B, Hq, H, n, mf.ATTN_SPARSE)
        small = lib.mustafar_attn_workspace_bytes(B, Hq, H, 128, n, counted)
        assert lib.mustafar_attn_workspace_bytes(B, Hq, H, 128, n, _taken(lib, Kc, Vc, Hq, small)) <= small
        assert _taken(lib, Kc, Vc, Hq, small - 1) == mf.EWORKSPACE


def test_rejected_and_empty(lib):  # noqa: F811
    Kc, Vc = _fake_cache(1, 8, 128, 0.7, 100)[0], _fake_cache(1, 8, 128, 0.7, 100)[0]
    assert _taken(lib, Kc, Vc, 8, 1 << 20) == 0
    Kc.n_tokens = 100
    assert _taken(lib, Kc, Vc, 8, 1 << 20) == mf.EINVAL        # token counts differ
    Vc.n_tokens = 100
    assert _taken(lib, Kc, Vc, 9, 1 << 20) == mf.EINVAL
    assert _taken(lib, Kc, Vc, 24, 1 << 20) == mf.EUNSUPPORTED
    try:
        lib.mustafar_attn_set_route(mf.ROUTE_WALKS)            # the walks take their default count
        assert _taken(lib, Kc, Vc, 8, 1 << 20) == lib.mustafar_attn_default_splits(1, 8, 8, 100, mf.ATTN_SPARSE)
    finally:
        lib.mustafar_attn_set_route(mf.ROUTE_DEFAULT)
