"""Host-only checks of the C-ABI library: it loads, exports every symbol the header
declares, and its argument validation answers before anything touches a GPU."""
import ctypes
import os
import re

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def R():
    from paper_2508_09072_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        from paper_2508_09072_amd import build
        build.build()
    binding.load()
    return binding


def entry_points_with_dims(R):
    """The calls that take dimensions, with what follows them (tensors on the CPU, which none of them takes)."""
    import torch
    i32, bf16 = torch.zeros(1, dtype=torch.int32), torch.zeros(1, dtype=torch.bfloat16)
    attn = (bf16, bf16, bf16, bf16, bf16, i32, i32, i32)
    return [(R.reader_tree_attn, attn + (bf16, None, 1, None)), (R.reader_tree_attn_noalloc, attn + (bf16, None, 1)),
            (R.reader_accept_path, (i32,) * 6), (R.reader_kv_compact, (bf16, bf16, i32, i32, bf16, bf16, i32, i32)),
            (R.reader_verify_step, attn + (i32, i32, bf16, None, i32, i32, i32, 1, None)),
            (R.reader_kv_compact_layers, (i32, i32, bf16, bf16, i32, i32))]


def test_only_dimensions_are_taken_as_dimensions(R):
    class Other(ctypes.Structure):
        _fields_ = R.ReaderDims._fields_

    class Mine(R.ReaderDims):
        pass
    size = ctypes.sizeof(R.ReaderDims)
    for call, rest in entry_points_with_dims(R):
        for no in (bytes(size), bytearray(2 * size), np.zeros(size, dtype=np.uint8), Other(), None, 7, R.ReaderDims):
            with pytest.raises(TypeError):
                call(no, *rest)
        for yes in (R.make_dims(1, 1, 1, 1, 64, 1, 1, 1), Mine(1, 1, 1, 1, 64)):
            with pytest.raises(ValueError, match="GPU"):
                call(yes, *rest)


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "reader.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(reader_[a-z_]+)\s*\(", text)))


def test_every_declared_symbol_is_exported(R):
    names = declared_symbols()
    assert set(names) == set(R.EXPORTS)
    lib = ctypes.CDLL(R.LIB_PATH)
    for n in names:
        assert getattr(lib, n) is not None


def test_dims_struct_matches_header(R):
    text = open(os.path.join(ROOT, "include", "reader.h")).read()
    body = re.search(r"typedef struct reader_dims \{(.*?)\} reader_dims;", text, flags=re.S).group(1)
    body = re.sub(r"/\*.*?\*/", "", body, flags=re.S)
    fields = re.findall(r"(int32_t|int64_t|float)\s+(\w+);", body)
    ctype = {"int32_t": ctypes.c_int32, "int64_t": ctypes.c_int64, "float": ctypes.c_float}
    assert [(n, ctype[t]) for t, n in fields] == list(R.ReaderDims._fields_)


def test_version_and_strerror(R):
    assert "gfx950" in R.version()
    assert R.strerror(0) == "ok" and "workspace" in R.strerror(R.READER_EWORKSPACE)


def test_validate_tree(R):
    good = np.asarray([[-1, 0, 0, 2], [-1, 0, 1, 2]], dtype=np.int32)
    assert R.reader_validate_tree(good) == R.READER_OK
    for bad in ([[0, 0, 1]], [[-1, -1, 0]], [[-1, 1, 0]], [[-1, 0, 2]], [[-1, 0, 0], [-1, 0, 7]]):
        assert R.reader_validate_tree(np.asarray(bad, dtype=np.int32)) == R.READER_EINVAL


def test_workspace_bytes_is_pure_and_monotone(R):
    d = R.make_dims(16, 32, 32, 8, 128, 260, 7, 3000)
    a, b = R.reader_workspace_bytes(d, 4096), R.reader_workspace_bytes(d, 4096)
    assert a == b and a % 256 == 0 and a > 0
    assert R.reader_workspace_bytes(R.make_dims(16, 32, 32, 8, 100, 260, 7, 3000), 4096) == 0   # bad D
    assert R.reader_workspace_bytes(d, 64) <= a


def test_a_workspace_for_the_largest_step_serves_every_smaller_one(R):
    rng = np.random.default_rng(20)
    for _ in range(3000):
        Hkv, G, D = int(rng.choice((1, 2, 4, 8, 16))), int(rng.choice((1, 2, 4, 8, 16))), int(rng.choice((64, 128)))
        T, B, L = int(rng.integers(1, 129)), int(2 ** rng.uniform(0, 7.5)), int(2 ** rng.uniform(0, 15))
        most = R.reader_workspace_bytes(R.make_dims(B, T, G * Hkv, Hkv, D, 2048, 1, 4096), L)
        small_b, small_l = int(rng.integers(1, B + 1)), int(rng.integers(0, L + 1))
        d = R.make_dims(small_b, T, G * Hkv, Hkv, D, 2048, 1, 4096)
        assert R.reader_workspace_bytes(d, small_l) <= most, (B, T, G, Hkv, D, L, small_b, small_l)
        # ... and the records of the kernel that is taken fit the workspace of the call itself, behind its header
        check_records_fit(R, d, small_l)


def check_records_fit(R, d, bound):
    plan = R.reader_attn_plan(d, bound)
    header = -(-(256 * 4 + 256 * 8 * 4 + d.B * d.Hkv * 8) // 256) * 256
    short = plan["kernel_id"] == 4
    records = plan["key_ranges"] * plan["row_chunks"] * (1 if short else 2)
    if short and plan["key_ranges"] == d.B * d.Hkv:
        records = 0                                     # (a short problem's pair that is not cut leaves none)
    need = records * plan["rows_per_workgroup"] * (d.D // 2 + 2) * 4
    have = R.reader_workspace_bytes(d, bound) - header
    assert need <= have, (plan, need, have, d.B, d.T, d.Hq, d.Hkv, d.D, bound)
    return plan


def test_records_fit_the_calls_own_workspace_on_every_route(R):
    # three and five chunks of 128 rows and their neighbours, where the plan and the size of the records follow
    # different rules, and the lengths around which a pair is cut
    rng = np.random.default_rng(21)
    met = set()
    for _ in range(20000):
        D, Hkv, G = int(rng.choice((64, 128))), int(rng.choice((1, 2, 4, 8))), int(rng.choice((1, 3, 4, 5, 8, 16)))
        rows = int(rng.choice((100, 128, 129, 250, 256, 257, 300, 384, 385, 512, 513, 600, 640, 641, 800, 1000)))
        T, B, L = min(128, -(-rows // G)), int(2 ** rng.uniform(0, 7)), int(2 ** rng.uniform(4, 17))
        plan = check_records_fit(R, R.make_dims(B, T, G * Hkv, Hkv, D, 1 << 14, 1, 1 << 20), L)
        met.add((D, plan["kernel_id"], plan["row_chunks"]))
    assert {(D, k, c) for D in (64, 128) for k in (1, 4) for c in (1, 2, 3, 4, 5)} <= met
    assert {(128, 3, 2), (128, 3, 3), (64, 2, 2), (64, 2, 4)} <= met


@pytest.mark.parametrize("D", [64, 128])
def test_one_workgroup_per_compute_unit_and_no_smaller_workspace_is_taken(R, D):
    # the cut, and with it the bits of the result, follows from the sizes alone: not from how much workspace a call brings
    one, lib, rng = ctypes.c_void_p(256), R.load(), np.random.default_rng(22)     # (pointers never dereferenced: the size is checked first)
    for _ in range(300):
        Hkv, G, T = int(rng.choice((1, 2, 4, 8))), int(rng.choice((1, 4, 8, 16))), int(rng.integers(1, 129))
        d = R.make_dims(int(2 ** rng.uniform(0, 8)), T, G * Hkv, Hkv, D, 1 << 11, 1, 1 << 18)
        L = int(2 ** rng.uniform(5, 14))
        plan = R.reader_attn_plan(d, L)
        assert plan["kernel_id"] == 4 or plan["key_ranges"] * plan["row_chunks"] <= 256, plan
        less = R.reader_workspace_bytes(d, L) - 1
        assert lib.reader_tree_attn(ctypes.byref(d), *[one] * 9, None, L, one, less, None, None) == R.READER_EWORKSPACE
        assert lib.reader_verify_step(ctypes.byref(d), *[one] * 11, None, one, one, one, L, one, less, None, None) == R.READER_EWORKSPACE


@pytest.mark.parametrize("B,T,Hq,Hkv,D,bound,short", [
    (16, 16, 32, 8, 128, 1200, True), (16, 16, 32, 8, 128, 1400, False), (16, 16, 32, 8, 128, 2400, False),   # two shares: 10 tiles, 12, 20
    (8, 16, 32, 8, 128, 3500, True), (8, 16, 32, 8, 128, 3700, False), (32, 64, 8, 2, 128, 2400, False),       # four: 14, 15; two: 20
    (8, 64, 32, 8, 64, 5000, True), (8, 64, 32, 8, 64, 5300, False),                       # head dimension 64, four: 20, 21
    (13, 64, 32, 8, 64, 1900, True), (13, 64, 32, 8, 64, 2100, False),                     # two: 16, 17
    (1, 64, 32, 8, 128, 16000, True), (1, 16, 8, 8, 64, 32000, True),                      # one sequence: all shares are alike
    (32, 16, 32, 8, 128, 1200, True), (24, 16, 32, 8, 64, 1400, True)])                    # pairs that are not cut
def test_long_shares_of_several_sequences_are_left_to_the_ring_kernels(R, B, T, Hq, Hkv, D, bound, short):
    # every share is as long as the bound makes it: one sequence of 2400 positions among 15 of 64 took 29 us, 23 in the
    # ring kernels, which cut what there is evenly
    plan = R.reader_attn_plan(R.make_dims(B, T, Hq, Hkv, D, 2048, 1, 4096), bound)
    assert (plan["kernel_id"] == 4) == short, plan


@pytest.mark.parametrize("T,D,B,bound,rows", [
    (72, 128, 2, 32768, 256), (72, 128, 16, 32768, 256), (80, 128, 64, 8192, 256),        # five chunks, long pairs
    (72, 128, 64, 3000, 128), (72, 128, 8, 8192, 128), (72, 64, 16, 32768, 128),          # shorter ones; head dimension 64
    (40, 128, 16, 32768, 256), (33, 128, 8, 32768, 256), (40, 128, 2, 32768, 128), (40, 64, 16, 32768, 128),   # three chunks, the last
    (41, 128, 16, 32768, 128), (48, 128, 64, 8192, 128)])                                 # ... 256 rows up to a quarter full, and more
def test_three_and_five_chunks_of_128_rows_are_for_shorter_pairs(R, T, D, B, bound, rows):
    # eight query rows per node; 16 sequences of 8 to 32 K positions: 1021 us in 128-row workgroups, 938 in 256-row ones
    plan = R.reader_attn_plan(R.make_dims(B, T, 64, 8, D, 2100, 1, 200000), bound)
    assert plan["rows_per_workgroup"] == rows, plan


@pytest.mark.parametrize("T,D,B,bound,rows", [
    (72, 128, 1, 22000, 128), (72, 128, 1, 23000, 256), (80, 128, 2, 16400, 128), (80, 128, 3, 13300, 128),   # five chunks
    (41, 128, 1, 31000, 128), (41, 128, 1, 32768, 256), (48, 128, 2, 32768, 128), (48, 128, 4, 32768, 128),   # three, more than 320 rows
    (40, 128, 1, 32768, 128), (72, 64, 1, 32768, 128), (48, 64, 1, 32768, 128)])
def test_one_long_sequence_crosses_over_sooner(R, T, D, B, bound, rows):
    dims = R.make_dims(B, T, 64, 8, D, 2100, 1, 200000)
    assert R.reader_attn_plan(dims, bound)["rows_per_workgroup"] == rows
    check_records_fit(R, dims, bound)


def whole_pairs(lens, T, Hkv, ranges, front, cost):
    """The (sequence, kv head) pairs that no start of a range falls into, by the cut that the ring kernels make: a pair is
    `front` positions, its tiles, and the rest of `cost` positions behind them; all positions are shared out evenly."""
    tiles = [-(-n // 64) + -(-T // 64) for n in lens]
    pairs = [(b, h) for b in range(len(lens)) for h in range(Hkv)]
    begin = np.concatenate(([0], np.cumsum([tiles[b] + cost for b, _ in pairs])))
    starts = np.arange(1, ranges) * begin[-1] // ranges
    at = np.searchsorted(begin, starts, side="right") - 1
    tile = starts - begin[at] - front                        # the first tile at or behind the start of the range
    n = np.asarray([tiles[b] for b, _ in pairs])
    return {pairs[i] for i in range(len(pairs))} - {pairs[i] for i, t in zip(at, tile) if 0 < t < n[i]}


def test_the_model_of_the_cut():
    # one pair of ten tiles over two ranges is cut in its middle; as long as there are as many ranges as equal pairs none is
    assert whole_pairs([600], 16, 1, 2, 1, 3) == set()
    assert whole_pairs([600], 16, 8, 8, 1, 3) == {(0, h) for h in range(8)}
    assert whole_pairs([18000, 1500, 1500], 72, 8, 48, 1, 3) - whole_pairs([18000, 1500, 1500], 72, 8, 80, 4, 8)


def test_odd_row_chunks_change_over_early_only_where_no_pair_is_newly_cut(R):
    # a cut pair's result is rounded once more.  Below the lines that were drawn by speed alone 256-row workgroups may run
    # only where they leave every pair whole that 128-row workgroups would, whatever the lengths below the bound.
    rng = np.random.default_rng(22)
    shapes = [(72, 8, [18000, 1500, 1500]), (72, 4, [18000] + [1500] * 5), (72, 2, [18000] + [600] * 11), (48, 8, [32768, 3000, 3000])]
    shapes += [(T, Hkv, [n]) for T in (41, 48, 65, 80) for Hkv in (1, 2, 4, 8, 9, 10, 16, 17, 25) for n in (20000, 23000, 32768, 65536)]
    for _ in range(400):
        B, Hkv = int(rng.integers(1, 26)), int(rng.choice((1, 2, 4, 8, 16, 25)))
        longest = int(2 ** rng.uniform(13, 17))
        lens = [longest] + [int(longest * 2 ** -rng.uniform(0, 7)) for _ in range(B - 1)]
        shapes.append((int(rng.choice((41, 44, 48, 65, 72, 80))), Hkv, lens))
    early = 0
    for T, Hkv, lens in shapes:
        M, bound, B = 8 * T, max(lens), len(lens)
        chunks, tiles = -(-M // 128), -(-bound // 64) + -(-T // 64)
        if B * Hkv * tiles * tiles > (2500000 if chunks == 5 else 1 << 62):
            continue                                           # (beyond the lines by speed)
        dims = R.make_dims(B, T, 8 * Hkv, Hkv, 128, 1 << 13, 1, 1 << 20)
        plan = R.reader_attn_plan(dims, bound)
        if plan["kernel_id"] == 4 or plan["rows_per_workgroup"] == 128:
            continue
        early += 1
        R.reader_tuning_override(R.TUNE_ATTN_ROWS, 128)
        try:
            narrow = R.reader_attn_plan(dims, bound)
        finally:
            R.reader_tuning_override(R.TUNE_ATTN_ROWS, -1)
        assert narrow["kernel_id"] == 1 and plan["kernel_id"] == 3
        below = [lens] + [[max(0, n * k // 64 - 5) for n in lens] for k in range(64)] + [[k] * B for k in range(0, 1400, 31)]
        for actual in below:
            new = whole_pairs(actual, T, Hkv, plan["key_ranges"], 4, 8)
            assert whole_pairs(actual, T, Hkv, narrow["key_ranges"], 1, 3) <= new, (T, Hkv, actual[:4])
    assert early >= 20


def test_attention_plan_follows_the_query_rows_and_the_overrides(R):
    # few query rows per kv head: 128-row workgroups with copying wavefronts; many rows on a long context: 256-row
    # workgroups, four wavefronts at head dimension 128 and eight at 64; the override names either
    small = R.reader_attn_plan(R.make_dims(16, 32, 32, 8, 128, 260, 7, 3000), 4096)
    assert small["kernel_id"] == 1 and small["rows_per_workgroup"] == 128 and small["row_chunks"] == 1
    assert 1 <= small["key_ranges"] <= 256
    big = R.reader_attn_plan(R.make_dims(64, 64, 64, 8, 128, 520, 7, 30000), 8192)
    assert big["kernel_id"] == 3 and big["rows_per_workgroup"] == 256 and big["row_chunks"] == 2
    assert big["kernel"] == "tree_attn_wide_kernel<128>"
    big64 = R.reader_attn_plan(R.make_dims(64, 64, 64, 8, 64, 520, 7, 30000), 8192)
    assert big64["kernel_id"] == 2
    try:
        R.reader_tuning_override(R.TUNE_ATTN_WIDE, 0)
        assert R.reader_attn_plan(R.make_dims(64, 64, 64, 8, 128, 520, 7, 30000), 8192)["kernel_id"] == 2
        R.reader_tuning_override(R.TUNE_ATTN_ROWS, 128)
        forced = R.reader_attn_plan(R.make_dims(64, 64, 64, 8, 128, 520, 7, 30000), 8192)
        assert forced["kernel_id"] == 1 and forced["row_chunks"] == 4
    finally:
        R.reader_tuning_override(R.TUNE_ATTN_WIDE, -1)
        R.reader_tuning_override(R.TUNE_ATTN_ROWS, -1)
    for D in (64, 128):                    # the name is the one a kernel trace shows
        short = R.reader_attn_plan(R.make_dims(1, 64, 32, 8, D, 260, 7, 300), 4096)
        assert short["kernel"] == "tree_attn_short_kernel<%d>" % D and short["rows_per_workgroup"] == 128
    scalar = R.reader_attn_plan(R.make_dims(2, 8, 8, 2, 64, 10, 4, 20, variant=1), 100)
    assert scalar["kernel_id"] == 0
    with pytest.raises(RuntimeError):
        R.reader_attn_plan(R.make_dims(2, 8, 8, 2, 96, 10, 4, 20), 100)


@pytest.mark.parametrize("change,code", [
    (dict(T=0), -1), (dict(T=129), -2), (dict(D=96), -2), (dict(Hkv=3), -1), (dict(page_size=32), -2),
    (dict(max_path=0), -1), (dict(max_path=33), -1), (dict(Hq=64, Hkv=2), -2), (dict(B=-1), -1),
])
def test_bad_dims_are_refused_on_the_host(R, change, code):
    base = dict(B=2, T=32, Hq=32, Hkv=8, D=128, max_pages_per_seq=16, max_path=7, num_pages=40)
    base.update(change)
    page_size = base.pop("page_size", 16)
    d = R.make_dims(**base, page_size=page_size)
    lib = R.load()
    null = [None] * 10
    assert lib.reader_tree_attn(ctypes.byref(d), *null, 0, None, 0, None, None) == code
    assert lib.reader_accept_path(ctypes.byref(d), *[None] * 8) == code
    assert lib.reader_kv_compact(ctypes.byref(d), *[None] * 10) == code
    assert lib.reader_verify_step(ctypes.byref(d), *[None] * 15, 0, None, 0, None, None) == code


def test_null_pointers_and_workspace_are_refused(R):
    d = R.make_dims(2, 32, 32, 8, 128, 16, 7, 40)
    lib = R.load()
    one = ctypes.c_void_p(256)            # never dereferenced: the checks fail first
    assert lib.reader_tree_attn(ctypes.byref(d), *[None] * 10, 128, None, 0, None, None) == R.READER_EINVAL
    assert lib.reader_tree_attn(ctypes.byref(d), *[one] * 9, None, 128, None, 0, None, None) == R.READER_EWORKSPACE
    assert lib.reader_tree_attn(ctypes.byref(d), *[one] * 9, None, 128, one, 16, None, None) == R.READER_EWORKSPACE
    assert lib.reader_tree_attn(ctypes.byref(d), *[one] * 9, None, 10**6, one, 1 << 40, None, None) == R.READER_EINVAL
    assert lib.reader_accept_path(ctypes.byref(d), one, one, None, one, one, one, None, None) == R.READER_EINVAL
    assert lib.reader_kv_compact(ctypes.byref(d), *[one] * 7, None, None, None) == R.READER_EINVAL
    assert lib.reader_tree_attn(None, *[one] * 9, None, 128, one, 1 << 40, None, None) == R.READER_EINVAL
    # B = 0 is a valid empty problem: nothing is enqueued
    d0 = R.make_dims(0, 32, 32, 8, 128, 16, 7, 40)
    assert lib.reader_tree_attn(ctypes.byref(d0), *[None] * 10, 0, None, 0, None, None) == R.READER_OK
    assert lib.reader_accept_path(ctypes.byref(d0), *[None] * 8) == R.READER_OK
    assert lib.reader_kv_compact(ctypes.byref(d0), *[None] * 10) == R.READER_OK
    assert lib.reader_verify_step(ctypes.byref(d0), *[None] * 15, 0, None, 0, None, None) == R.READER_OK
    # the fused step checks what the three calls check
    assert lib.reader_verify_step(ctypes.byref(d), *[None] * 15, 128, None, 0, None, None) == R.READER_EINVAL
    assert lib.reader_verify_step(ctypes.byref(d), *[one] * 8, None, one, one, None, one, one, one, 128, one, 1 << 40,
                                  None, None) == R.READER_EINVAL            # draft tokens missing
    assert lib.reader_verify_step(ctypes.byref(d), *[one] * 11, None, one, one, one, 128, one, 16, None, None) \
        == R.READER_EWORKSPACE


def test_binding_refuses_cpu_tensors(R):
    import torch
    d = R.make_dims(1, 4, 4, 4, 64, 4, 3, 8)
    t = torch.zeros(4, dtype=torch.int32)
    with pytest.raises(ValueError):
        R.reader_accept_path(d, t, t, t, t, t, t)


def test_rearrange_arguments_are_checked_on_the_host(R):
    lib = R.load()
    one = ctypes.c_void_p(256)
    assert R.reader_kv_rearrange_scratch_bytes(16, 4224) >= (16 * 4224 + 64) * 4
    assert R.reader_kv_rearrange_scratch_bytes(16, 4224) % 256 == 0
    assert lib.reader_kv_rearrange(1, 2, 8, 0, 128, one, one, one, one, one, 1 << 20, None) == R.READER_EINVAL
    assert lib.reader_kv_rearrange(1, 2, 8, 2, 96, one, one, one, one, one, 1 << 20, None) == R.READER_EUNSUPPORTED
    assert lib.reader_kv_rearrange(1, 2, 8, 2, 128, None, one, one, one, one, 1 << 20, None) == R.READER_EINVAL
    assert lib.reader_kv_rearrange(1, 2, 8, 2, 128, one, one, one, one, None, 0, None) == R.READER_EWORKSPACE
    assert lib.reader_kv_rearrange(1, 2, 8, 2, 128, one, one, one, one, one, 16, None) == R.READER_EWORKSPACE
    assert lib.reader_kv_rearrange(1, 0, 8, 2, 128, None, None, None, None, None, 0, None) == R.READER_OK   # empty batch
    # more workgroups than one launch holds: layers x samples x (kv heads + 1) must stay below 2^31
    assert lib.reader_kv_rearrange(40000, 8192, 8, 8, 128, one, one, one, one, one, 1 << 20, None) == R.READER_EUNSUPPORTED



def test_target_token_arguments_are_checked_on_the_host(R):
    lib = R.load()
    one = ctypes.c_void_p(256)
    assert lib.reader_target_argmax(-1, 10, one, one, None) == R.READER_EINVAL
    assert lib.reader_target_argmax(4, 0, one, one, None) == R.READER_EINVAL
    assert lib.reader_target_argmax(4, 10, None, one, None) == R.READER_EINVAL
    assert lib.reader_target_argmax(0, 10, None, None, None) == R.READER_OK
    s = lib.reader_target_sample
    assert s(-1, 4, 10, one, one, one, 1.0, one, None) == R.READER_EINVAL
    assert s(2, 0, 10, one, one, one, 1.0, one, None) == R.READER_EINVAL
    assert s(2, 129, 10, one, one, one, 1.0, one, None) == R.READER_EINVAL          # more nodes than a tree may have
    assert s(2, 4, 0, one, one, one, 1.0, one, None) == R.READER_EINVAL
    assert s(2, 4, (1 << 22) + 1, one, one, one, 1.0, one, None) == R.READER_EINVAL  # vocabulary beyond the limit
    for bad in (0.0, -1.0, 1e-9, 1e9, float("inf"), float("nan")):
        assert s(2, 4, 10, one, one, one, bad, one, None) == R.READER_EINVAL
    assert s(2, 4, 10, None, one, one, 1.0, one, None) == R.READER_EINVAL
    assert s(2, 4, 10, one, one, None, 1.0, one, None) == R.READER_EINVAL
    assert s(0, 4, 10, None, None, None, 1.0, None, None) == R.READER_OK             # empty batch


def test_layered_compaction_arguments_are_checked_on_the_host(R):
    lib = R.load()
    one = ctypes.c_void_p(256)
    dims = R.make_dims(2, 16, 8, 2, 128, 8, 8, 40)
    f = lib.reader_kv_compact_layers
    assert f(ctypes.byref(dims), -1, one, one, one, one, one, one, None, None) == R.READER_EINVAL
    assert f(ctypes.byref(dims), 70000, one, one, one, one, one, one, None, None) == R.READER_EINVAL
    assert f(ctypes.byref(dims), 2, None, one, one, one, one, one, None, None) == R.READER_EINVAL
    assert f(ctypes.byref(dims), 2, one, one, None, one, one, one, None, None) == R.READER_EINVAL
    empty = R.make_dims(0, 16, 8, 2, 128, 8, 8, 40)
    assert f(ctypes.byref(empty), 2, None, None, None, None, None, None, None, None) == R.READER_OK


@pytest.mark.parametrize("B,T,Hq,Hkv,D,bound,shares", [
    (1, 64, 32, 8, 128, 4160, 16),      # sixteen pairs' chunks: all compute units
    (8, 32, 8, 8, 128, 444, 4),
    (5, 83, 2, 2, 128, 3020, 24),
    (3, 25, 32, 8, 128, 2556, 10),
    (1, 16, 8, 8, 64, 568, 10),         # sqrt(12 tiles)
])
def test_a_short_problem_has_as_many_shares_as_the_rule_says(R, B, T, Hq, Hkv, D, bound, shares):
    # none are given up for the sake of one launch: longer shares are rounded worse
    plan = R.reader_attn_plan(R.make_dims(B, T, Hq, Hkv, D, 300, 4 if T > 3 else 1, 5000), bound)
    assert plan["kernel_id"] == 4
    assert plan["key_ranges"] == B * Hkv * shares


@pytest.mark.parametrize("B,T,Hq,Hkv,D,bound,one", [
    (1, 64, 32, 8, 128, 4160, False),   # two pairs' chunks of sixteen shares fill every XCD: no place for the keeper
    (3, 25, 32, 8, 128, 2556, True),    # three of ten shares and a keeper
    (1, 16, 8, 8, 64, 568, True),
    (128, 12, 8, 8, 128, 52, True), (129, 12, 8, 8, 128, 52, False),     # whole pairs: as many marks as there are, and more
    (64, 64, 64, 8, 128, 8192, False),  # ring kernels
    (0, 64, 64, 8, 128, 8192, False),   # nothing to do
])
def test_when_the_fused_step_is_one_launch(R, B, T, Hq, Hkv, D, bound, one):
    dims = R.make_dims(B, T, Hq, Hkv, D, 600, 4, 50000)
    assert R.reader_step_is_one_launch(dims, bound) is one
    R.reader_tuning_override(R.TUNE_JOIN, 0)
    try:
        assert R.reader_step_is_one_launch(dims, bound) is False
    finally:
        R.reader_tuning_override(R.TUNE_JOIN, -1)
    with pytest.raises(RuntimeError):
        R.reader_step_is_one_launch(R.make_dims(2, 8, 8, 2, 96, 10, 4, 20), 100)
    with pytest.raises(RuntimeError):
        R.reader_step_is_one_launch(dims, -1)


@pytest.mark.parametrize("D,most", [(64, 63), (128, 31)])
def test_forced_shares_are_one_launch_as_long_as_an_xcd_holds_them_and_the_keeper(R, D, most):
    dims = R.make_dims(1, 8, 2, 2, D, 300, 4, 5000)
    for n, one in ((most, True), (most + 1, False)):
        R.reader_tuning_override(R.TUNE_ATTN_SHORT, n)
        try:
            assert R.reader_step_is_one_launch(dims, 4096) is one
        finally:
            R.reader_tuning_override(R.TUNE_ATTN_SHORT, -1)


@pytest.mark.parametrize("B,T,Hq,Hkv,D,longest,fused,kernel,whole_step,workgroups", [
    (1, 16, 8, 8, 64, 512, True, "verify_short_join_kernel<64>", True, 8 * 10 + 1),
    (1, 16, 8, 8, 64, 512, False, "tree_attn_short_kernel<64>", False, 8 * 10),
    (1, 64, 32, 8, 128, 4096, True, "tree_attn_short_kernel<128>", False, 8 * 2 * 16),
    (129, 12, 8, 8, 128, 40, True, "verify_short_kernel<128>", False, 129 * 8),
    (64, 64, 64, 8, 128, 8192, True, "tree_attn_wide_kernel<128>", False, 256),
])
def test_the_bench_line_names_the_launch_that_it_times(R, B, T, Hq, Hkv, D, longest, fused, kernel, whole_step, workgroups):
    import types

    import bench
    w = types.SimpleNamespace(B=B, T=T, Hq=Hq, Hkv=Hkv, D=D, max_pages=600, max_path=6, num_pages=50000, seq_lens=np.array([longest]))
    got = bench.timed_kernel(R, w, fused)
    assert (got["kernel"], got["whole_step"], got["workgroups"]) == (kernel, whole_step, workgroups)
