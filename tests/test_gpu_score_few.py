"""The score kernel of launches of few tokens (16 tokens a workgroup, rows gathered, nothing pipelined): parity with the oracle as in
test_gpu_parity.py, at the edges of its workgroups and of the rule that chooses it."""
import re

import numpy as np
import pytest

from paper_2506_18879_amd import synth

from test_gpu_parity import assert_rows, gpu, oracle_out  # noqa: F401  (gpu: fixture)
from test_gpu_score_stream import _check

pytestmark = pytest.mark.gpu


def _make(name, Hq, lens, Mk, dtype="bf16"):
    w = synth.make_workload(name, B=len(lens), Hq=Hq, Hkv=8, seqlens=lens, Mk=Mk, Mv=16, dtype=dtype, seed=Mk + Hq + sum(lens))
    # queries at, before (negative distances) and past the end
    w.q_pos = np.array([(max(1, x) - 1, x // 3, x + 777)[i % 3] for i, x in enumerate(lens)], np.int32)
    return w


@pytest.mark.parametrize("Mk,G,dtype", [(16, 1, "bf16"), (16, 4, "bf16"), (32, 2, "bf16"), (32, 4, "bf16"), (32, 8, "bf16"), (16, 8, "f32"), (32, 4, "f32")])
@pytest.mark.parametrize("lens", [[1], [17, 15, 16], [0, 33, 0, 100, 31, 0], [64, 1, 63, 65, 2, 129, 5, 48]])
def test_edges_of_workgroups(gpu, oracle, Mk, G, dtype, lens):  # noqa: F811
    w = _make(f"few_m{Mk}_g{G}_{dtype}_{len(lens)}", 8 * G, lens, Mk, dtype)
    op = gpu.DecodeAttention(w, max_position=1024)
    assert (op.plan.score_kernel, op.plan.score_split_len) == (0, 16)
    op.close()
    _check(gpu, oracle, w, max_position=1024)


@pytest.mark.parametrize("Mk,lens,kernel", [(32, [2734], 0), (32, [2735], 1), (16, [5468], 0), (16, [5469], 1), (16, [4000] + [1] * 8, 1)])
def test_either_side_of_the_rule(gpu, oracle, Mk, lens, kernel):  # noqa: F811
    # by tokens x heads x codebooks, and by the workgroups that one long sequence gives the short ones beside it
    w = _make(f"rule_m{Mk}_{len(lens)}_{lens[-1]}", 32, lens, Mk)
    op = gpu.DecodeAttention(w, max_position=8192)
    assert op.plan.score_kernel == kernel
    op.close()
    _check(gpu, oracle, w, max_position=8192)


@pytest.mark.parametrize("Mk,G,tokens,kernel", [(32, 4, 1392, "k_score_few"), (32, 4, 1393, "k_score"), (32, 8, 3600, "k_score_few"), (32, 8, 3601, "k_score"),
                                                (32, 2, 3700, "k_score_few"), (16, 8, 3700, "k_score_few")])
def test_fp32_rows_with_many_heads(gpu, oracle, Mk, G, tokens, kernel):  # noqa: F811
    # 696 and 704, 1800 and 1808 workgroups of 16 tokens: tiles of four tokens a wavefront in both kernels
    import torch
    from torch.profiler import ProfilerActivity, profile
    w = _make(f"wide_m{Mk}_g{G}_{tokens}", 8 * G, [tokens], Mk, "f32")
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w, max_position=4096)
    assert (op.plan.score_kernel, op.plan.score_split_len) == (0, 16)
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        op(dw)
        torch.cuda.synchronize()
    op.close()
    assert {m.group(1) for e in trace.events() for m in [re.search(r"(k_score\w*)<", e.name)] if m} == {kernel}
    _check(gpu, oracle, w, max_position=4096)


@pytest.mark.parametrize("Mk", [16, 32])
def test_explicit_positions_and_storage_that_is_not_aligned(gpu, oracle, Mk):  # noqa: F811
    import torch
    w = _make(f"odd_m{Mk}", 32, [300, 77], Mk)
    rng = np.random.default_rng(Mk)
    for key_pos in (None, rng.integers(0, 5000, w.total_tokens).astype(np.int32)):
        w.key_pos = key_pos
        dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w, max_position=8192)
        for name in ("q", "key_codebooks"):                    # two bytes past a 16-byte boundary
            t = getattr(dw, name)
            room = torch.empty(t.numel() + 1, dtype=t.dtype, device="cuda")
            room[1:] = t.view(-1)
            setattr(dw, name, room[1:])
        out = op(dw)
        torch.cuda.synchronize()
        assert_rows(out.cpu().numpy(), oracle_out(oracle, w), w.name)
        op.close()


@pytest.mark.parametrize("Mk,tokens", [(16, 900), (16, 7000), (32, 900), (32, 7000)])
def test_which_copy_of_registered_key_codebooks_is_read(gpu, Mk, tokens):  # noqa: F811
    # few tokens: the caller's; slices: the packed one.  Each result is the same with the other copy cleared.
    import torch
    import paper_2506_18879_amd as cv
    w = _make(f"copies_m{Mk}_{tokens}", 32, [tokens], Mk)
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w, max_position=8192)
    assert op.plan.score_kernel == (tokens > 5000)
    want = op(dw).clone()
    packed = torch.empty(cv.commvq_packed_key_codebook_bytes(op.handle), dtype=torch.uint8, device="cuda")
    cv.commvq_pack_key_codebooks(op.handle, dw.key_codebooks, packed, op.stream_ptr())
    (dw.key_codebooks if op.plan.score_kernel else packed).zero_()
    assert torch.equal(op(dw), want)
    op.close()


@pytest.mark.parametrize("Mk,dtype", [(16, "bf16"), (32, "bf16"), (16, "f32"), (32, "f32")])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_infinities_and_nan_stay_where_they_are(gpu, Mk, dtype, bad):  # noqa: F811
    # in an element of one query head: that head's logits; in one codeword of one KV head: those of the tokens that have it. All others keep their bits.
    import torch
    w = _make(f"bad_m{Mk}_{dtype}", 32, [200, 33], Mk, dtype)
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w, max_position=1024)
    assert (op.plan.score_kernel, op.plan.score_split_len) == (0, 16)
    clean, out = op.scores(dw).clone(), op(dw).clone()
    lens, code = np.diff(w.cu_seqlens), int(w.key_codes[0])    # first codebook of KV head 0: a codeword that a token has
    heads = lambda x: [x[32 * c:32 * (c + n)].view(32, n) for c, n in zip(w.cu_seqlens[:-1], lens)]
    tokens = [np.asarray(w.key_codes[8 * Mk * c:8 * Mk * (c + n)]).reshape(8, n, Mk)[0, :, 0] == code for c, n in zip(w.cu_seqlens[:-1], lens)]

    dw.q.view(2, 32, 128)[1, 5, 77] = bad
    s, got = op.scores(dw), op(dw)
    for b, (x, y) in enumerate(zip(heads(s), heads(clean))):
        for h in range(32):
            assert not x[h].isfinite().any() if (b, h) == (1, 5) else torch.equal(x[h], y[h])
    hit = torch.zeros((2, 32), dtype=torch.bool, device="cuda")
    hit[1, 5] = True
    assert torch.equal(got.view(2, 32, 128)[~hit], out.view(2, 32, 128)[~hit])

    dw = gpu.DeviceWorkload(w)
    dw.key_codebooks.view(8, Mk, 256, 128)[0, 0, code, 33] = bad
    s, got = op.scores(dw), op(dw)
    assert tokens[0].any() and not tokens[0].all()
    for x, y, t in zip(heads(s), heads(clean), tokens):
        t = torch.from_numpy(t).cuda()
        assert not x[:4, t].isfinite().any() and torch.equal(x[:4, ~t], y[:4, ~t]) and torch.equal(x[4:], y[4:])
    assert torch.equal(got.view(2, 32, 128)[:, 4:], out.view(2, 32, 128)[:, 4:])
    op.close()


@pytest.mark.parametrize("G", [4, 8])
def test_sequences_that_share_a_workgroup_of_the_slices(gpu, oracle, G):  # noqa: F811
    # 16 codebooks and more tokens than the rule leaves to this kernel: the segments of several sequences in k_score_stream
    lens = [512, 1, 513, 511, 1024, 700, 0, 3, 512, 1537, 1200]
    w = _make(f"share_g{G}", 8 * G, lens, 16)
    op = gpu.DecodeAttention(w, max_position=4096)
    assert op.plan.score_kernel == 1
    op.close()
    _check(gpu, oracle, w, max_position=4096)
