"""How attention calls are cut up: row blocks, key ranges, workspaces (host code of the library, no GPU)."""
import ctypes as C

import pytest

from paper_2406_17276_amd import api
from tests import _util as U

SYNC, SCRATCH = 4096, 8 << 20


def _bytes(B, Hkv, g, n, D, plan):
    """Workspace of a plan: sync words, 256 bytes to spare, and O in bf16 and (reference, sum) for each padded row and range."""
    rows, splits, _ = plan
    blocks = B * Hkv * -(-g * n // rows)
    return SYNC + 256 + (blocks * rows * splits * (2 * D + 8) if splits > 1 else 0)


@pytest.mark.parametrize("B,Hkv,g,n,D,L,kv8,fewest", [
    (1, 8, 4, 50, 128, 32768, False, 16), (1, 8, 4, 50, 128, 131072, True, 28), (1, 2, 4, 50, 64, 32768, False, 24),
    (1, 8, 8, 60, 128, 131072, False, 16), (1, 1, 2, 60, 128, 56997, False, 24), (1, 8, 1, 64, 64, 16384, False, 22),
    (1, 8, 1, 64, 64, 65536, True, 28), (25, 4, 2, 60, 128, 8192, True, 5), (3, 8, 8, 60, 128, 8192, False, 5),
    (3, 2, 1, 17, 128, 2720, True, 11), (5, 8, 1, 17, 64, 4732, True, 11), (25, 4, 1, 50, 64, 1000, True, 5),
])
def test_long_prefixes_go_in_as_many_ranges_as_pay(B, Hkv, g, n, D, L, kv8, fewest):
    """Shapes measured to take up to 2.4 times as long with eight ranges (twelve in 64-row blocks of 64), or with as many as
    fill the compute units once."""
    assert U.attention_plan(B, Hkv * g, Hkv, D, n, L, kv8=kv8)[1] >= fewest


@pytest.mark.parametrize("Hkv,D,L,n,kv8,ranges", [
    (8, 128, 190, 120, True, 5), (8, 128, 30, 65, True, 3), (8, 128, 100, 65, True, 4), (64, 128, 120, 100, True, 4),
    (32, 64, 120, 100, False, 4), (33, 64, 120, 100, False, 1), (8, 128, 120, 100, False, 4), (16, 128, 120, 100, False, 1), (65, 64, 120, 100, True, 1),
])
def test_few_tiles_go_in_a_range_each(Hkv, D, L, n, kv8, ranges):
    """Up to a fourth slower in one range, but for many heads."""
    assert U.attention_plan(1, Hkv, Hkv, D, n, L, kv8=kv8)[1] == ranges


@pytest.mark.parametrize("B,Hkv,g,n,L,kv8,rows", [
    (25, 40, 16, 50, 149, True, 128), (32, 8, 16, 64, 384, True, 128), (32, 8, 16, 64, 385, True, 256), (32, 8, 8, 60, 320, True, 256), (16, 8, 8, 60, 4096, True, 256),
    (20, 8, 8, 60, 700, True, 128), (20, 8, 8, 60, 1300, True, 256), (25, 8, 8, 60, 700, True, 256), (16, 8, 8, 60, 700, True, 256),
    (25, 40, 16, 50, 149, False, 256), (16, 8, 8, 60, 4096, False, 256),
])
def test_few_tiles_of_an_8_bit_cache_stay_with_128_rows(B, Hkv, g, n, L, kv8, rows):
    """Up to a third slower in 256-row blocks, which widen each tile two tiles ahead; and where half a round of the compute units
    is enough in 128-row blocks."""
    assert U.attention_plan(B, Hkv * g, Hkv, 128, n, L, kv8=kv8)[0] == rows


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("Hkv,g", [(1, 1), (8, 1), (32, 1), (8, 4), (8, 8), (2, 8)])
def test_ranges_follow_the_workspace(Hkv, g, D):
    """More room, more ranges; the size the library asks for is enough, the full size gives the best plan, and the library's own
    array serves every call that it can hold with the fewest ranges."""
    for B in (1, 3, 12, 40):
        for n in (1, 50, 60, 128):
            for L in (0, 100, 1000, 4096, 10000, 40000, 131072):
                p = U.attention_params(B, Hkv * g, Hkv, D, n, L)
                need, full = api.attn_workspace_bytes(p), int(api.lib().ot_attn_workspace_bytes_full(C.byref(p)))
                least_of = []
                for kv8 in (False, True):
                    plan = lambda room: U.attention_plan(B, Hkv * g, Hkv, D, n, L, kv8=kv8, room=room)
                    size = lambda room: _bytes(B, Hkv, g, n, D, plan(room))
                    least, best = plan(0), plan(1 << 50)
                    least_of.append(size(0))
                    assert least[0] == best[0] and 1 <= least[1] <= best[1] <= 32
                    last = least[1]
                    for room in (size(0), need, (need + full) // 2, full - 1, full):
                        if room < size(0):
                            continue
                        got = plan(room)
                        assert size(room) <= room and (least[1] <= got[1] <= best[1])
                        if room >= need:
                            assert got[1] >= last
                            last = got[1]
                    assert plan(full) == best
                assert need <= full and (need <= SCRATCH) == (max(least_of) <= SCRATCH)
