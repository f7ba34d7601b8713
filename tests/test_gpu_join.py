"""Launches for short problems that merge, accept and append by themselves, their workgroups waiting for one another:
the same bits as with launches of their own, also where nobody waits (a bound of nothing on every wait: whoever finds
somebody missing leaves, and the last to arrive does what is left) and where a pair's shares run on different XCDs, whose
caches do not see each other (each merge variant then reads the records past them)."""
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


@pytest.mark.parametrize("B,Hkv,G,D,T,lens,splits,one", [
    (1, 8, 1, 64, 16, [512], 9, True), (1, 8, 1, 128, 16, [512], 5, True),         # more and less than eight records: two sizes of batches
    (3, 2, 4, 64, 45, [700, 0, 130], 4, True), (3, 2, 4, 128, 45, [700, 0, 130], 12, True),   # two row chunks, empty shares
    (5, 3, 1, 128, 7, [64, 1, 300, 65, 0], 1, True), (40, 4, 1, 64, 20, list(range(3, 203, 5)), 1, True),   # pairs that are not cut
    (2, 1, 16, 128, 128, [900, 333], 7, True), (1, 2, 1, 64, 128, [4000], 63, True),   # sixteen row chunks; as many shares as an XCD holds beside a keeper
    (1, 1, 4, 64, 40, [1500], 17, True), (1, 2, 1, 64, 60, [3000], 33, True), (1, 3, 2, 128, 40, [2100], 31, True),   # more than 16 records, more than one trip's 32
    (1, 2, 1, 64, 128, [4000], 64, False), (1, 8, 4, 128, 64, [1100], 16, False),   # no place for the keeper: launches of their own
    (1, 1, 1, 64, 1, [0], 1, True), (1, 1, 1, 128, 1, [0], 4, True),               # a root alone; more shares than tiles
    (64, 8, 2, 64, 12, [40] * 64, 1, True), (128, 8, 1, 128, 12, [40] * 128, 1, True), (129, 8, 1, 64, 3, [40] * 129, 1, False),   # more workgroups than run at once, as many as there are marks, and more
    (9, 3, 1, 128, 12, [240] * 9, 5, True),                            # no multiple of the XCDs
    (4, 1, 1, 64, 60, [2400, 64, 64, 64], None, True), (2, 12, 1, 128, 60, [1100, 64], None, True),   # the planner's choice: pairs that stay whole among cut ones
    (2, 16, 1, 128, 60, [1100, 64], None, False),
])
@pytest.mark.parametrize("in_cache", [False, True])
def test_launches_that_wait_inside_give_the_same_bits(R, B, Hkv, G, D, T, lens, splits, one, in_cache, tune):
    import torch
    w = W.make_custom("join_T%d_D%d" % (T, D), B=B, Hq=Hkv * G, Hkv=Hkv, D=D, T=T, seq_lens=lens, tree="trie" if T > 1 else "chain",
                      depth=min(12, max(1, T - 1)), p_match=0.9, max_path=T, seed=700 + T + B)
    if in_cache:
        put_tree_in_cache(w)
    dims = R.make_dims(w.B, w.T, w.Hq, w.Hkv, w.D, w.max_pages, w.max_path, w.num_pages)
    if splits is not None:
        tune(R.TUNE_ATTN_SHORT, splits)
    results, bound = {}, max(lens)
    for join, spread in ((0, 0), (-1, 0), (1, 0), (-1, 1), (1, 1)):
        tune(R.TUNE_JOIN, join)
        tune(R.TUNE_JOIN_SPREAD, spread)
        assert R.reader_step_is_one_launch(dims, bound) is (one and join != 0)
        for what in ("attn", "step") if spread == 0 else ("step",):
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
            results[join, spread, what] = {n: getattr(dw, n).clone() for n in NAMES}
            assert not torch.isnan(dw.out).any() and not torch.isnan(dw.lse).any()
    for (join, spread, what), got in results.items():
        for name in NAMES if what == "step" else ("out", "lse", "k_cache", "v_cache", "seq_lens", "status"):
            assert torch.equal(got[name].view(torch.uint8), results[0, 0, what][name].view(torch.uint8)), (join, spread, what, name)
    assert int(results[0, 0, "step"]["status"].item()) == 0
    assert int((results[0, 0, "step"]["seq_lens"] - torch.from_numpy(w.seq_lens).cuda()).min()) >= 1


def test_a_workspace_serves_one_step_after_the_other(R, tune):
    # joined steps of other sizes, launches of their own and ring kernels leave their marks, records and flags in the same
    # header, never cleared: none of it counts as an arrival of a later launch
    import torch
    kinds = [dict(B=3, Hq=8, Hkv=2, D=64, T=45, lens=[700, 20, 130], short=4, one=True), dict(B=40, Hq=4, Hkv=4, D=64, T=20, lens=list(range(3, 203, 5)), short=1, one=True),
             dict(B=3, Hq=8, Hkv=2, D=128, T=45, lens=[700, 20, 130], short=12, one=True), dict(B=5, Hq=64, Hkv=4, D=128, T=33, lens=[900] * 5, short=0, one=False),
             dict(B=1, Hq=2, Hkv=2, D=64, T=60, lens=[3000], short=33, one=True), dict(B=5, Hq=3, Hkv=3, D=128, T=7, lens=[64, 1, 300, 65, 8], short=1, one=True)]
    work = [W.make_custom("chain_%d" % i, B=k["B"], Hq=k["Hq"], Hkv=k["Hkv"], D=k["D"], T=k["T"], seq_lens=k["lens"], tree="trie", depth=5,
                          p_match=0.9, seed=740 + i) for i, k in enumerate(kinds)]
    results = []
    for join in (0, -1):
        tune(R.TUNE_JOIN, join)
        shared = torch.full((64 << 20,), 255, dtype=torch.uint8, device="cuda")
        devs, got = [R.to_device(w) for w in work], []
        for turn in range(3):
            for k, dw in zip(kinds, devs):
                tune(R.TUNE_ATTN_SHORT, k["short"])
                tune(R.TUNE_JOIN_SPREAD, turn & 1)         # (and what one XCD has written and read another may do next)
                assert R.reader_workspace_bytes(dw.dims, dw.max_seq_len) <= shared.numel()
                assert R.reader_step_is_one_launch(dw.dims, dw.max_seq_len) is (k["one"] and join != 0)
                lens = dw.seq_lens.clone()
                R.reader_verify_step(dw.dims, dw.q, dw.k_tree, dw.v_tree, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents,
                                     dw.draft_tokens, dw.target_tokens, dw.out, dw.lse, dw.accept_len, dw.path, dw.bonus, dw.max_seq_len,
                                     shared, dw.status)
                torch.cuda.synchronize()
                got.append({n: getattr(dw, n).clone() for n in NAMES})
                assert int((dw.seq_lens - lens).min()) >= 1
                dw.seq_lens.copy_(lens)                # (the next turn's step of this kind starts where this one did)
        results.append(got)
    for i, (a, b) in enumerate(zip(*results)):
        for name in NAMES:
            assert torch.equal(a[name].view(torch.uint8), b[name].view(torch.uint8)), (i, name)


@pytest.mark.parametrize("join", [-1, 1])
@pytest.mark.parametrize("fault", ["page", "end", "tree", "length", "cut path"])
@pytest.mark.parametrize("in_cache", [False, True])
@pytest.mark.parametrize("splits", [1, 3])
def test_what_is_refused_stays_refused(R, join, fault, in_cache, splits, tune):
    # a sequence that cannot be appended to is left as it was, with the bits of the separate launches, and the others go on: the
    # chains of 40 nodes match all the way, a bad link at node 9 ends the path in front of it
    import torch
    w = W.make_custom("join_%s" % fault, B=3, Hq=4, Hkv=2, D=64, T=40, seq_lens=[70, 0, 31], tree="chain", p_match=1.0,
                      max_path=40, seed=720)
    if fault == "cut path":
        w.max_path = 7
    if in_cache:
        put_tree_in_cache(w)
    if fault == "page":
        w.page_table[0, 70 // 16 + 1] = w.num_pages + 5
    elif fault == "end":
        w.page_table = np.ascontiguousarray(w.page_table[:, :5])
    elif fault == "tree":
        w.parents[1, 9] = 30
    elif fault == "length":
        w.seq_lens[2] = -4
    tune(R.TUNE_ATTN_SHORT, splits)
    dims = R.make_dims(w.B, w.T, w.Hq, w.Hkv, w.D, w.page_table.shape[1], w.max_path, w.num_pages)
    got = []
    status, more = {"page": (R.STATUS_BAD_PAGE, [0, 40, 40]), "end": (R.STATUS_BAD_PATH, [0, 40, 40]), "tree": (R.STATUS_BAD_TREE, [40, 9, 40]),
                    "length": (R.STATUS_BAD_PATH, [40, 40, 0]), "cut path": (R.STATUS_BAD_PATH, [7, 7, 7])}[fault]
    for mode in (0, join):
        tune(R.TUNE_JOIN, mode)
        assert R.reader_step_is_one_launch(dims, 70) is (mode != 0)
        dw = R.to_device(w)
        kt, vt = (None, None) if in_cache else (dw.k_tree, dw.v_tree)
        if fault == "end" and in_cache:                # (the tree rows would not fit the table either: refused on the host)
            with pytest.raises(R.ReaderError):
                R.reader_verify_step(dims, dw.q, kt, vt, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents, dw.draft_tokens,
                                     dw.target_tokens, dw.out, dw.lse, dw.accept_len, dw.path, dw.bonus, 70, dw.workspace, dw.status)
            continue
        R.reader_verify_step(dims, dw.q, kt, vt, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents, dw.draft_tokens,
                             dw.target_tokens, dw.out, dw.lse, dw.accept_len, dw.path, dw.bonus, 70, dw.workspace, dw.status)
        torch.cuda.synchronize()
        got.append({n: getattr(dw, n).clone() for n in NAMES})
        assert int(dw.status.item()) == status
        assert (dw.seq_lens.cpu().numpy() - w.seq_lens).tolist() == more
    for name in NAMES if got else ():
        assert torch.equal(got[0][name].view(torch.uint8), got[1][name].view(torch.uint8)), name


@pytest.mark.parametrize("B,Hkv,G,D,T,lens,splits", [
    (1, 2, 4, 128, 65, [700], 5), (3, 2, 2, 64, 128, [700, 0, 130], 4),            # two nodes per lane; shares without tiles
    (2, 1, 1, 128, 1, [0, 300], 3), (2, 1, 1, 64, 1, [300, 0], 3),                 # a root alone
    (33, 8, 1, 128, 12, [200] * 33, 2), (40, 8, 1, 64, 3, [150] * 40, 1),          # cut and whole pairs of more workgroups than run at once
    (3, 2, 4, 128, 65, [700, 0, 130], 0), (5, 1, 16, 64, 45, [900, 64, 0, 1, 65], 0),   # the ring kernels: two and six chunks of 128 rows
    (1, 1, 1, 128, 1, [0], 0), (300, 2, 1, 64, 5, [40] * 300, 0),                  # ranges without tiles; more sequences than workgroups
    (256, 2, 1, 64, 5, [40] * 256, 0), (257, 2, 1, 128, 5, [40] * 257, 0)])          # as many, and one more
@pytest.mark.parametrize("in_cache", [False, True])
def test_a_path_chosen_by_the_attention_launch_is_the_one_of_separate_calls(R, B, Hkv, G, D, T, lens, splits, in_cache, tune):
    # every result and the cache bit for bit, as a call and as replays of a captured graph
    import torch
    w = W.make_custom("rides_T%d_D%d" % (T, D), B=B, Hq=Hkv * G, Hkv=Hkv, D=D, T=T, seq_lens=lens, tree="trie" if T > 1 else "chain",
                      depth=min(9, max(1, T - 1)), p_match=0.9, max_path=T, seed=760 + T + B)
    if in_cache:
        put_tree_in_cache(w)
    bound = max(lens)
    tune(R.TUNE_ATTN_SHORT, splits)
    tune(R.TUNE_JOIN, 0)
    assert splits > 0 or R.reader_attn_plan(R.make_dims(w.B, w.T, w.Hq, w.Hkv, w.D, w.max_pages, w.max_path, w.num_pages), bound)["rows_per_workgroup"] == 128

    def step(dw):
        kt, vt = (None, None) if in_cache else (dw.k_tree, dw.v_tree)
        R.reader_verify_step(dw.dims, dw.q, kt, vt, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents, dw.draft_tokens,
                             dw.target_tokens, dw.out, dw.lse, dw.accept_len, dw.path, dw.bonus, bound, dw.workspace, dw.status)

    dw = R.to_device(w)
    kt, vt = (None, None) if in_cache else (dw.k_tree, dw.v_tree)
    R.reader_tree_attn(dw.dims, dw.q, kt, vt, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents, dw.out, dw.lse, bound,
                       dw.workspace, dw.status)
    R.reader_accept_path(dw.dims, dw.draft_tokens, dw.target_tokens, dw.parents, dw.accept_len, dw.path, dw.bonus, dw.status)
    if in_cache:
        R.reader_kv_compact_layers(dw.dims, dw.path, dw.accept_len, dw.k_cache.unsqueeze(0), dw.v_cache.unsqueeze(0), dw.page_table,
                                   dw.seq_lens, dw.status)
    else:
        R.reader_kv_compact(dw.dims, kt, vt, dw.path, dw.accept_len, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.status)
    torch.cuda.synchronize()
    want = {n: getattr(dw, n).clone() for n in NAMES}
    dw = R.to_device(w)
    first = {n: getattr(dw, n).clone() for n in NAMES}
    graph = None
    for turn in range(4):
        for name in NAMES:
            getattr(dw, name).copy_(first[name])
        if turn == 1:
            torch.cuda.synchronize()
            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph):
                step(dw)
        graph.replay() if graph else step(dw)
        torch.cuda.synchronize()
        for name in NAMES:
            assert torch.equal(getattr(dw, name).view(torch.uint8), want[name].view(torch.uint8)), (turn, name)


@pytest.mark.parametrize("B,Hkv,G,D,T,lens,splits", [
    (256, 1, 4, 128, 24, [70] * 256, 0), (257, 1, 4, 128, 24, [70] * 257, 0),      # ring kernel: as many sequences as workgroups, one more
    (5, 2, 4, 128, 32, [900, 64, 0, 1, 65], 0), (5, 2, 4, 128, 33, [900, 64, 0, 1, 65], 0),    # one full chunk of rows, two
    (16, 8, 1, 64, 40, [200] * 16, 2), (16, 8, 1, 64, 41, [200] * 16, 2),          # short problems, cut pairs: 640 sets of eight rows to merge, 768
    (16, 8, 1, 128, 40, [200] * 16, 2), (16, 8, 1, 128, 41, [200] * 16, 2)])
@pytest.mark.parametrize("in_cache", [False, True])
def test_on_both_sides_of_the_rules_for_who_accepts(R, B, Hkv, G, D, T, lens, splits, in_cache, tune):
    test_a_path_chosen_by_the_attention_launch_is_the_one_of_separate_calls(R, B, Hkv, G, D, T, lens, splits, in_cache, tune)
