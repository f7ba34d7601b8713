"""What the binding refuses before anything is launched, and what it takes for a number."""
import numpy as np
import pytest

from paper_2508_09072_amd import workloads as W

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def R():
    import torch
    assert torch.cuda.is_available(), "these tests need the GPU"
    from paper_2508_09072_amd import binding
    binding.load()
    return binding


def attn_args(dw):
    return [dw.dims, dw.q, dw.k_tree, dw.v_tree, dw.k_cache, dw.v_cache, dw.page_table, dw.seq_lens, dw.parents, dw.out,
            dw.lse, dw.max_seq_len, dw.workspace, dw.status]


@pytest.mark.parametrize("at", [1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 13])
def test_attention_refuses_tensors_of_another_place_layout_or_type(R, at):
    import torch
    dw = R.to_device(W.make_config(0))
    good = attn_args(dw)
    t = good[at]
    wide = torch.zeros(t.shape + (2,), dtype=t.dtype, device="cuda")
    other = torch.float16 if t.dtype == torch.bfloat16 else torch.int64
    dw.out.fill_(7)
    for bad, error in ((t.cpu(), ValueError), (wide[..., 0], ValueError), (t.to(other), ValueError), (t.cpu().float().numpy(), TypeError)):
        if t.numel() == 1 and bad.shape == t.shape and getattr(bad, "is_cuda", False) and bad.dtype == t.dtype:
            continue                                        # (one value is contiguous whatever its stride)
        with pytest.raises(error):
            R.reader_tree_attn(*(good[:at] + [bad] + good[at + 1:]))
    if at not in (2, 3, 10, 13):                            # (the tree rows, the log-sum-exp and the status word may be left out)
        with pytest.raises(ValueError):
            R.reader_tree_attn(*(good[:at] + [None] + good[at + 1:]))
    torch.cuda.synchronize()
    assert bool((dw.out == 7).all())


def test_shapes_that_do_not_fit_each_other_are_refused(R):
    import torch
    bf, i32 = dict(dtype=torch.bfloat16, device="cuda"), dict(dtype=torch.int32, device="cuda")
    k = torch.zeros((2, 3, 32, 4, 64), **bf)
    valid, new_len = torch.ones((3, 32), dtype=torch.uint8, device="cuda"), torch.zeros(3, **i32)
    scratch = torch.zeros(R.reader_kv_rearrange_scratch_bytes(3, 32), dtype=torch.uint8, device="cuda")
    for bad in ((k, k[:1], valid, new_len), (k, k, valid[:2], new_len), (k, k, valid, new_len[:2])):
        with pytest.raises(AssertionError):
            R.reader_kv_rearrange(*bad, scratch)
    with pytest.raises(ValueError):                         # not five dimensions
        R.reader_kv_rearrange(k[0], k[0], valid, new_len, scratch)
    logits, par = torch.zeros((2, 4, 100), **bf), torch.zeros((2, 4), **i32)
    uni = torch.zeros((2, 4), dtype=torch.float32, device="cuda")
    for bad in ((logits, par[:1], uni, 0.7, par), (logits, par, uni[:1], 0.7, par), (logits, par, uni, 0.7, par[:1])):
        with pytest.raises(AssertionError):
            R.reader_target_sample(*bad)
    with pytest.raises(ValueError):                         # not three dimensions
        R.reader_target_sample(logits[0], par, uni, 0.7, par)
    with pytest.raises(AssertionError):
        R.reader_target_argmax(logits, par[:1])
    dims = R.make_dims(2, 4, 4, 4, 64, 2, 2, 3)
    cache, ones = torch.zeros((2, 3, 4, 16, 64), **bf), torch.zeros(2, **i32)
    for kc, vc in ((cache, cache[:1]), (cache[0], cache[0])):
        with pytest.raises(AssertionError):
            R.reader_kv_compact_layers(dims, par[:, :2].contiguous(), ones, kc, vc, par[:, :2].contiguous(), ones)


def test_a_temperature_is_whatever_float_takes(R):
    import torch
    rng = np.random.Generator(np.random.PCG64(3))
    logits = torch.from_numpy(rng.standard_normal((1, 8, 5000), dtype=np.float32)).cuda().to(torch.bfloat16)
    parents = torch.full((1, 8), -1, dtype=torch.int32, device="cuda")
    uniforms = torch.from_numpy(rng.random((1, 8), dtype=np.float32)).cuda()
    got = []
    for temperature in (0.75, "0.75", np.float32(0.75), torch.tensor(0.75)):
        out = torch.full((1, 8), -1, dtype=torch.int32, device="cuda")
        R.reader_target_sample(logits, parents, uniforms, temperature, out)
        got.append(out.cpu())
    assert all(torch.equal(g, got[0]) for g in got) and int(got[0].min()) >= 0
    for no in (None, "warm", [0.7]):
        with pytest.raises((TypeError, ValueError)):
            R.reader_target_sample(logits, parents, uniforms, no, parents)
