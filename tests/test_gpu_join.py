"""Launches for short problems that merge, accept and append by themselves, their workgroups waiting for one another:
the same bits as with launches of their own, and also where nobody waits (a bound of nothing on every wait: whoever finds
somebody missing leaves, and the last to arrive does what is left)."""
import numpy as np
import pytest

from paper_2508_09072_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    from paper_2508_09072_amd import binding
    binding.load()
    return binding


@pytest.fixture
def tune(R):
    touched = []

    def set_(which, value):
        touched.append(which)
        R.reader_tuning_override(which, value)
    yield set_
    for which in touched:
        R.reader_tuning_override(which, -1)


def put_tree_in_cache(w):
    """The tree rows written behind each sequence, node n at position L + n, as a model's forward pass leaves them."""
    for b in range(w.B):
        for n in range(w.T):
            pos = int(w.seq_lens[b]) + n
            page = w.page_table[b, pos // 16]
            w.k_cache[page, :, pos % 16] = w.k_tree[b, n]
            w.v_cache[page, :, pos % 16] = w.v_tree[b, n]


NAMES = ("out", "lse", "accept_len", "path", "bonus", "seq_lens", "k_cache", "v_cache", "status")


@pytest.mark.parametrize("B,Hkv,G,D,T,lens,splits", [
    (1, 8, 1, 64, 16, [512], 9), (1, 8, 1, 128, 16, [512], 5),         # one wavefront's records, four wavefronts'
    (3, 2, 4, 64, 45, [700, 0, 130], 4), (3, 2, 4, 128, 45, [700, 0, 130], 12),   # two row chunks, empty shares
    (5, 3, 1, 128, 7, [64, 1, 300, 65, 0], 1), (40, 4, 1, 64, 20, list(range(3, 203, 5)), 1),   # pairs that are not cut
    (2, 1, 16, 128, 128, [900, 333], 7), (1, 2, 1, 64, 128, [4000], 64),   # sixteen row chunks; as many shares as may be
    (1, 1, 1, 64, 1, [0], 1), (1, 1, 1, 128, 1, [0], 4),               # a root alone; more shares than tiles
    (64, 8, 2, 64, 12, [40] * 64, 1), (128, 8, 1, 128, 12, [40] * 128, 1), (129, 8, 1, 64, 3, [40] * 129, 1), (9, 3, 1, 128, 12, [240] * 9, 5),   # more workgroups than run at once, as many as there are marks, and more; no multiple of the XCDs
    (4, 1, 1, 64, 60, [2400, 64, 64, 64], None), (2, 16, 1, 128, 60, [1100, 64], None),   # the planner's choice: pairs that stay whole among cut ones
])
@pytest.mark.parametrize("in_cache", [False, True])
def test_launches_that_wait_inside_give_the_same_bits(R, B, Hkv, G, D, T, lens, splits, in_cache, tune):
    import torch
    w = W.make_custom("join_T%d_D%d" % (T, D), B=B, Hq=Hkv * G, Hkv=Hkv, D=D, T=T, seq_lens=lens, tree="trie" if T > 1 else "chain",
                      depth=min(12, max(1, T - 1)), p_match=0.9, max_path=T, seed=700 + T + B)
    if in_cache:
        put_tree_in_cache(w)
    dims = R.make_dims(w.B, w.T, w.Hq, w.Hkv, w.D, w.max_pages, w.max_path, w.num_pages)
    if splits is not None:
        tune(R.TUNE_ATTN_SHORT, splits)
    results, bound = {}, max(lens)
    for join in (0, -1, 1):
        tune(R.TUNE_JOIN, join)
        for what in ("attn", "step"):
            dw = R.to_device(w)
            assert R.reader_attn_plan(dims, bound)["kernel_id"] == 4
            kt, vt = (None, None) if in_cache else (dw.k_tree, dw.v_tree)
            dw.out.fill_(float("nan"))
            dw.lse.fill_(float("nan"))
            dw.workspace.fill_(255)
            args = (dims, dw.q, kt, vt, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents)
            for again in range(3 if what == "attn" else 1):
                if what == "attn":
                    R.reader_tree_attn(*args, dw.out, dw.lse, bound, dw.workspace, dw.status)
                else:
                    R.reader_verify_step(*args, dw.draft_tokens, dw.target_tokens, dw.out, dw.lse, dw.accept_len, dw.path, dw.bonus,
                                         bound, dw.workspace, dw.status)
            torch.cuda.synchronize()
            results[join, what] = {n: getattr(dw, n).clone() for n in NAMES}
            assert not torch.isnan(dw.out).any() and not torch.isnan(dw.lse).any()
    for join in (-1, 1):
        for what in ("attn", "step"):
            for name in NAMES if what == "step" else ("out", "lse", "k_cache", "v_cache", "seq_lens", "status"):
                a, b = results[join, what][name], results[0, what][name]
                assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), (join, what, name)
    assert int(results[0, "step"]["status"].item()) == 0
    assert int((results[0, "step"]["seq_lens"] - torch.from_numpy(w.seq_lens).cuda()).min()) >= 1


@pytest.mark.parametrize("join", [-1, 1])
@pytest.mark.parametrize("fault", ["page", "end", "tree", "length", "cut path"])
@pytest.mark.parametrize("in_cache", [False, True])
@pytest.mark.parametrize("splits", [1, 3])
def test_what_is_refused_stays_refused(R, join, fault, in_cache, splits, tune):
    # a sequence that cannot be appended to is left as it was, with the bits of the separate launches, and the others go on
    import torch
    w = W.make_custom("join_%s" % fault, B=3, Hq=4, Hkv=2, D=64, T=40, seq_lens=[70, 0, 31], tree="chain", p_match=1.0,
                      max_path=40, seed=720)
    if fault == "cut path":
        w.max_path = 7
    if in_cache:
        put_tree_in_cache(w)
    if fault == "page":
        w.page_table[0, 70 // 16 + 1] = w.num_pages + 5
    elif fault == "end" and not in_cache:              # (the tree rows would not fit the table either: refused on the host)
        w.page_table = np.ascontiguousarray(w.page_table[:, :5])
    elif fault == "tree":
        w.parents[1, 9] = 30
    elif fault == "length":
        w.seq_lens[2] = -4
    tune(R.TUNE_ATTN_SHORT, splits)
    dims = R.make_dims(w.B, w.T, w.Hq, w.Hkv, w.D, w.page_table.shape[1], w.max_path, w.num_pages)
    got = []
    for mode in (0, join):
        tune(R.TUNE_JOIN, mode)
        dw = R.to_device(w)
        kt, vt = (None, None) if in_cache else (dw.k_tree, dw.v_tree)
        R.reader_verify_step(dims, dw.q, kt, vt, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents, dw.draft_tokens,
                             dw.target_tokens, dw.out, dw.lse, dw.accept_len, dw.path, dw.bonus, 70, dw.workspace, dw.status)
        torch.cuda.synchronize()
        got.append({n: getattr(dw, n).clone() for n in NAMES})
    for name in NAMES:
        assert torch.equal(got[0][name].view(torch.uint8), got[1][name].view(torch.uint8)), name
