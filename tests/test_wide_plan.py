"""The prompt-sized product's plans and its division of K among splits and
K-groups (host)."""
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


def plan(p, n, batch, out, inp, g):
    f = H.lib().higgs_internal_wide_plan
    f.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 3 + [ctypes.c_void_p]
    splits = ctypes.c_int64()
    return f(batch, out, inp, p, n, g, ctypes.byref(splits)), splits.value


@pytest.mark.parametrize("p,n", [(2, 64), (2, 256), (2, 1024), (1, 16), (1, 256)])
def test_gpu_cases_reach_every_plan(p, n):
    """The sizes of the GPU tests take every kernel instance of the code width,
    with and without a K-split."""
    pytest.importorskip("torch")
    from test_gpu_prompt import CASES
    got = set()
    for case in CASES:
        if case[:2] == (p, n):
            shape, splits = plan(*case)
            assert shape >= 0, case
            got.add(("g64" if case[5] == 64 else "", shape, splits > 1))
    want = {("", 0), ("", 2)}
    if n != 1024:
        want |= {("", 1)}
    if p == 1:
        want |= {("g64", 1), ("g64", 2), ("g64", 3)}
    if (p, n) == (1, 256):
        want |= {("", 3)}
    assert {k[:2] for k in got} == want
    missing = {(*k, split) for k in want for split in (False, True)} - got
    assert not missing, missing


def test_gpu_groups_mix_splits():
    """Among the groups of the GPU tests: layers of one block shape with
    different and with equal K-splits, split and unsplit layers."""
    pytest.importorskip("torch")
    from test_gpu_prompt import GROUPS
    mixed = same = some = 0
    for p, n, g, batch, inp, outs in GROUPS:
        plans = [plan(p, n, batch, out, inp, g) for out in outs]
        assert all(s >= 0 for s, _ in plans)
        by_shape = {s: {k for t, k in plans if t == s} for s, _ in plans}
        mixed += any(len(v) > 1 for v in by_shape.values())
        same += len(set(plans)) == 1
        some += {k > 1 for _, k in plans} == {False, True}
    assert mixed and same and some


def test_plan_starts_where_the_rule_says():
    for (p, n, g, inp), first in {(2, 256, 1024, 4096): 65, (1, 16, 64, 4096): 17,
                                  (1, 16, 64, 6208): 49, (1, 256, 64, 4096): 9,
                                  (1, 256, 64, 6208): 33, (1, 256, 128, 4096): 33,
                                  (1, 256, 128, 8192): 33, (1, 16, 128, 4096): 65}.items():
        assert plan(p, n, first - 1, 512, inp, g)[0] == -1
        assert plan(p, n, first, 512, inp, g)[0] >= 0


def test_plans_split_long_rows_and_keep_the_fixed_scratch_calls():
    """Rows too long for the fixed scratch are split all the same; calls whose
    64-column product fits in the scratch still fit."""
    need64 = H.lib()["_ZN5higgs23qgemm64_workspace_bytesElllii"]
    need64.argtypes = [ctypes.c_int64] * 3 + [ctypes.c_int] * 2
    need64.restype = ctypes.c_int64
    scratch = 32 << 20
    for batch, out, inp in ((127, 128, 131072), (129, 128, 131072), (300, 128, 65536),
                            (250, 128, 65536), (2048, 512, 8192), (65, 1, 1 << 20)):
        shape, splits = plan(2, 256, batch, out, inp, 1024)
        tiles = -(-out // 128) * -(-batch // 128)
        assert shape == 2 and tiles * splits >= 64, (batch, out, inp, splits)
    kept = 0
    for p, n, bits in ((2, 64, 6), (2, 256, 8), (2, 1024, 10), (1, 16, 8), (1, 256, 16)):
        for batch in (65, 100, 128, 250, 500, 1000, 1900, 2040):
            for out in (1, 128, 1000, 4096, 14336):
                for inp in (1024, 4096, 8192, 14336, 32768, 65536, 130048, 131072, 262144):
                    if need64(batch, out, inp, 1024, bits) <= scratch:
                        kept += 1
                        assert H.qmatmul_workspace_bytes(batch, out, inp, p, n, 1024) <= scratch
    assert kept > 500


def test_workspace_of_a_larger_batch_is_taken():
    """A program may keep the workspace of its largest batch: where the
    64-column product's need for a batch is no larger, the call takes it, though
    a smaller batch's plan may have more splits."""
    def c_fn(name, types):
        f = H.lib()[name]
        f.argtypes, f.restype = types, ctypes.c_int64
        return f
    i64, i32 = ctypes.c_int64, ctypes.c_int
    need64 = c_fn("_ZN5higgs23qgemm64_workspace_bytesElllii", [i64] * 3 + [i32] * 2)
    least = c_fn("_ZN5higgs27qgemm_least_workspace_bytesElllii" + "i", [i64] * 3 + [i32] * 3)
    group = c_fn("_ZN5higgs33qgemm_group_least_workspace_bytesEilPKlliii",
                 [i32, i64, ctypes.c_void_p, i64, i32, i32, i32])
    batches = (9, 17, 33, 64, 65, 80, 129, 160, 257, 300, 600, 2048)
    larger_plan = 0
    for p, n, bits, g in ((2, 64, 6, 1024), (2, 256, 8, 1024), (2, 1024, 10, 128),
                          (1, 16, 8, 64), (1, 256, 16, 64), (1, 256, 16, 128)):
        for out, inp in ((4096, 4096), (14336, 4096), (4096, 14336), (1024, 1024), (500, 8192)):
            for i, small in enumerate(batches):
                own = H.qmatmul_workspace_bytes(small, out, inp, p, n, g)
                assert least(small, out, inp, p, n, g) <= own
                for large in batches[i + 1:]:
                    kept = H.qmatmul_workspace_bytes(large, out, inp, p, n, g)
                    larger_plan += own > kept
                    if need64(small, out, inp, g, bits) <= need64(large, out, inp, g, bits):
                        assert least(small, out, inp, p, n, g) <= kept
                        outs = (i64 * 2)(out, out)
                        assert group(2, small, outs, inp, p, n, g) <= \
                            H.qmatmul_fused_multi_workspace_bytes(large, (out, out), inp, p, n, g)
    assert larger_plan > 50
