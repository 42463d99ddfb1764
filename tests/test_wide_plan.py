"""The prompt-sized product's division of K among splits and K-groups (host)."""
import ctypes

import pytest

H = pytest.importorskip("paper_2411_17525_amd.higgs")


def k_range(inp, kps, split, groups, q):
    out = [ctypes.c_int() for _ in range(3)]
    H.lib().higgs_internal_wide_range(inp, kps, split, groups, q, *map(ctypes.byref, out))
    return tuple(v.value for v in out)


@pytest.mark.parametrize("groups", [1, 2, 4])
@pytest.mark.parametrize("step", [64, 128])
def test_k_groups_cover_k_and_stay_inside(groups, step):
    """Every 64 weights of K belong to one K-group of one split, group 0 has the
    most, groups of 128 and more start at even stages, and the stage that a group
    requests first lies inside the row also where the group has none."""
    empty = 0
    for inp in list(range(512, 3000, step)) + [5120, 14336, 14336 + step, 1 << 20]:
        for kps in (256, 512, 768, 1280, 4096, (inp + 255) // 256 * 256):
            splits = -(-inp // kps)
            if splits > 60:
                continue
            covered = []
            for split in range(splits):
                turns = set()
                for q in range(groups):
                    first, stages, t = k_range(inp, kps, split, groups, q)
                    turns.add(t)
                    assert 0 <= first <= inp - 64 and first % 64 == 0
                    assert 0 <= stages <= t
                    assert q > 0 or stages == t or (groups > 1 and (stages, t) == (1, 2))
                    if stages > 0:
                        assert first % 128 == 0
                        assert step == 64 or stages % 2 == 0
                    else:
                        empty += 1
                    covered += range(first, first + 64 * stages, 64)
                assert len(turns) == 1
            assert covered == list(range(0, inp, 64))
    assert (empty > 0) == (groups > 1)
