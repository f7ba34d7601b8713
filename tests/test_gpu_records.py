"""Partial records of cut pairs: bf16 outputs of any size, each channel as exact as it would be alone."""
import numpy as np
import pytest

from paper_2508_09072_amd import workloads as W
from helpers import assert_close
from test_gpu_parity import R, bf16_to_np, run_attn, tune  # noqa: F401

pytestmark = pytest.mark.gpu


def route(R, tune, kernel):
    """Overrides that send a problem of two kv heads through one of the kernels that leave records."""
    if kernel == "short":
        tune(R.TUNE_ATTN_SHORT, 5)
    else:
        tune(R.TUNE_ATTN_SHORT, 0)
        tune(R.TUNE_ATTN_RANGES, 9)
        tune(R.TUNE_ATTN_ROWS, 128 if kernel == "rows128" else 256)
        tune(R.TUNE_ATTN_WIDE, 1 if kernel == "waves4" else 0)


def scale_heads(w):
    """Values of the four kv heads times these units, and one infinite value in the second head."""
    unit = np.asarray([2.0 ** -90, 2.0 ** 70, 0.0, 2.0 ** -11])
    for name in ("v_cache", "v_tree"):
        a = W.bf16_bits_to_f32(getattr(w, name)).astype(np.float64)
        a *= unit[None, :, None, None] if name == "v_cache" else unit[None, None, :, None]
        canary = np.isnan(a)
        bits = W.to_bf16_bits(a.astype(np.float32))
        bits[canary] = getattr(w, name)[canary]
        setattr(w, name, bits)
    w.v_cache[int(w.page_table[0, 3]), 1, 5, 7] = 0x7F80
    return unit


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kernel", ["short", "rows128", "waves8", "waves4"])
def test_outputs_of_any_size_survive_the_records(R, oracle_mod, kernel, D, tune):
    # one kv head with values around 2^-90, one around 2^70 and one infinite value among them, one with zeros, one with
    # values of 2^-10 and less after averaging: the errors scale with them
    route(R, tune, kernel)
    w = W.make_custom("units_%s" % kernel, B=2, Hq=8, Hkv=4, D=D, T=33, seq_lens=[700, 333], tree="trie", depth=6, seed=530)
    unit = scale_heads(w)
    ref, ref_lse = oracle_mod.tree_attn(w.q, w.k_tree, w.v_tree, w.k_cache, w.v_cache, w.page_table, w.seq_lens, w.parents)
    out, lse = run_attn(R, w)
    G = w.Hq // w.Hkv
    assert np.isinf(ref[0, :, G:2 * G, 7]).all() and np.array_equal(out[0, :, G:2 * G, 7], ref[0, :, G:2 * G, 7])
    out[0, :, G:2 * G, 7] = ref[0, :, G:2 * G, 7] = 0
    assert np.isfinite(out).all()
    for h in range(w.Hkv):
        got, want = out[:, :, h * G:(h + 1) * G].astype(np.float64), ref[:, :, h * G:(h + 1) * G]
        assert (np.abs(got - want) <= 2e-2 * unit[h] + 2e-2 * np.abs(want)).all(), (kernel, h)
    assert np.abs(lse - ref_lse).max() <= 2e-2


@pytest.mark.parametrize("rows,T", [(128, 16), (128, 80), (256, 80)])
def test_a_cut_pair_is_as_exact_as_its_records(R, oracle_mod, rows, T, tune):
    # bf16 weights and the final rounding leave 2.3e-3, 1.7e-3 of it the rounding; a record is rounded once more, which makes
    # sqrt(2.3^2 + 1.7^2) = 2.86e-3 of it, a ratio of 1.24.  30000 roundings and more scatter by half a percent; the parts' own largest
    # weights, which are exactly 1, move the ratio by up to three percent
    tune(R.TUNE_ATTN_SHORT, 0)
    tune(R.TUNE_ATTN_ROWS, rows)
    w = W.make_custom("exact_%d_%d" % (rows, T), B=8, Hq=16, Hkv=8, D=64, T=T, seq_lens=[1200] * 8, tree="trie", depth=5, seed=531)
    ref, _ = oracle_mod.tree_attn(w.q, w.k_tree, w.v_tree, w.k_cache, w.v_cache, w.page_table, w.seq_lens, w.parents)
    err = []
    for ranges in (64, 200):                     # as many as there are pairs, all alike: none is cut
        tune(R.TUNE_ATTN_RANGES, ranges)
        out, _ = run_attn(R, w)
        err.append(np.linalg.norm(out - ref) / np.linalg.norm(ref))
    print("whole %.4e, cut %.4e" % tuple(err), flush=True)
    assert err[1] <= 1.24 * 1.04 * err[0]


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kernel", ["short", "rows128", "waves8", "waves4"])
def test_channels_of_any_size_survive_the_records(R, oracle_mod, kernel, D, tune):
    # channel c of every value row is 2^-(c mod 32) of what it was: each channel has the error that it would have alone.  Weights,
    # records and results are rounded to bf16, 2^-9 at most each; the parts' sums have random signs, so that none of the three is more
    # of the result than that
    route(R, tune, kernel)
    w = W.make_custom("channels_%s" % kernel, B=2, Hq=8, Hkv=4, D=D, T=33, seq_lens=[700, 333], tree="trie", depth=6, seed=533)
    for name in ("v_cache", "v_tree"):
        a = W.bf16_bits_to_f32(getattr(w, name)).astype(np.float64)
        canary = np.isnan(a)
        bits = W.to_bf16_bits((a * 2.0 ** -(np.arange(D) % 32)).astype(np.float32))
        bits[canary] = getattr(w, name)[canary]
        setattr(w, name, bits)
    ref, _ = oracle_mod.tree_attn(w.q, w.k_tree, w.v_tree, w.k_cache, w.v_cache, w.page_table, w.seq_lens, w.parents)
    out, _ = run_attn(R, w)
    err = np.linalg.norm((out - ref).reshape(-1, D), axis=0) / np.linalg.norm(ref.reshape(-1, D), axis=0)
    print("worst channel %d of %d: %.2e" % (int(err.argmax()), D, err.max()), flush=True)
    assert err.max() <= 3 * 2.0 ** -9


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("T,G,splits", [(5, 1, 7), (6, 1, 16), (33, 2, 5), (67, 2, 11)])
def test_what_the_workspace_held_before_does_not_show(R, D, T, G, splits, tune):
    # rows past the last one share a merging wavefront with real ones, and nobody writes their part of a record
    import torch
    tune(R.TUNE_ATTN_SHORT, splits)
    w = W.make_custom("held_T%d" % T, B=6, Hq=4 * G, Hkv=4, D=D, T=T, seq_lens=[1500, 1100, 1900, 1717, 2000, 1250],
                      tree="trie", depth=5, seed=534)
    results = []
    for fill in (0x00, 0xFF, 0x80):
        dw = R.to_device(w)
        dw.workspace.fill_(fill)
        R.reader_tree_attn(dw.dims, dw.q, dw.k_tree, dw.v_tree, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents,
                           dw.out, dw.lse, dw.max_seq_len, dw.workspace, dw.status)
        torch.cuda.synchronize()
        results.append((dw.out.clone(), dw.lse.clone()))
    for out, lse in results[1:]:
        assert torch.equal(out.view(torch.uint8), results[0][0].view(torch.uint8))
        assert torch.equal(lse.view(torch.uint8), results[0][1].view(torch.uint8))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("kernel", ["short", "rows128", "waves8", "waves4"])
@pytest.mark.parametrize("nan", [0x7FC0, 0xFFC0])
def test_an_undefined_key_leaves_both_results_undefined(R, oracle_mod, kernel, D, nan, tune):
    # NaN of either sign in one key of the second kv head: every row of that head attends to it and is NaN, its log-sum-exp too
    route(R, tune, kernel)
    w = W.make_custom("undefined_%s" % kernel, B=2, Hq=4, Hkv=2, D=D, T=33, seq_lens=[700, 333], tree="trie", depth=6, seed=535)
    clean, clean_lse = oracle_mod.tree_attn(w.q, w.k_tree, w.v_tree, w.k_cache, w.v_cache, w.page_table, w.seq_lens, w.parents)
    w.k_cache[int(w.page_table[0, 3]), 1, 5] = nan
    out, lse = run_attn(R, w)
    assert np.isnan(out[0, :, 2:]).all()
    assert np.isnan(lse[0, 2:]).all()
    assert_close(out[0, :, :2], clean[0, :, :2], what=kernel)
    assert_close(out[1], clean[1], what=kernel)
    assert_close(lse[0, :2], clean_lse[0, :2], what=kernel)
    assert_close(lse[1], clean_lse[1], what=kernel)


@pytest.mark.parametrize("D", [64, 128])
def test_a_pair_left_whole_beside_cut_ones_is_rounded_once(R, D, tune):
    # the short sequence's pairs fit one share: the bits of a launch that cuts nothing
    import torch
    w = W.make_custom("left_whole", B=2, Hq=12, Hkv=12, D=D, T=60, seq_lens=[1100, 64], tree="trie", depth=6, seed=536)
    bound, outs = 1100, []
    for splits in (-1, 1):
        tune(R.TUNE_ATTN_SHORT, splits)
        dw = R.to_device(w)
        plan = R.reader_attn_plan(dw.dims, bound)
        assert plan["kernel_id"] == 4 and (plan["key_ranges"] > 24) == (splits < 0)
        R.reader_tree_attn(dw.dims, dw.q, dw.k_tree, dw.v_tree, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents,
                           dw.out, dw.lse, bound, dw.workspace, dw.status)
        torch.cuda.synchronize()
        outs.append((dw.out[1:].clone(), dw.lse[1:].clone()))
    for a, b in zip(*outs):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("splits", [3, 7, 17])
def test_outputs_of_any_size_survive_the_records_of_a_step_in_one_launch(R, D, splits, tune):
    # bit for bit those of the separate calls, with a pair's shares on one XCD and on several, also where nobody waits
    import torch
    w = W.make_custom("units_step", B=2, Hq=8, Hkv=4, D=D, T=30, seq_lens=[1500, 1333], tree="trie", depth=6, seed=537)
    scale_heads(w)
    tune(R.TUNE_ATTN_SHORT, splits)
    bound, want = 1500, None
    for join, spread in ((0, 0), (-1, 0), (-1, 1), (1, 0), (1, 1)):
        tune(R.TUNE_JOIN, join)
        tune(R.TUNE_JOIN_SPREAD, spread)
        dw = R.to_device(w)
        assert R.reader_step_is_one_launch(dw.dims, bound) is (join != 0)
        dw.workspace.fill_(255)
        if join == 0:
            R.reader_tree_attn(dw.dims, dw.q, dw.k_tree, dw.v_tree, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents,
                               dw.out, dw.lse, bound, dw.workspace, dw.status)
        else:
            R.reader_verify_step(dw.dims, dw.q, dw.k_tree, dw.v_tree, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents,
                                 dw.draft_tokens, dw.target_tokens, dw.out, dw.lse, dw.accept_len, dw.path, dw.bonus, bound,
                                 dw.workspace, dw.status)
        torch.cuda.synchronize()
        got = [t.clone().view(torch.uint8) for t in (dw.out, dw.lse)]
        want = want or got
        assert all(torch.equal(a, b) for a, b in zip(got, want)), (join, spread)
