"""The slice-streaming score kernel where a workgroup's passes (512-token segments) belong to several sequences, and every
number of passes a workgroup can have: parity with the oracle as in test_gpu_parity.py."""
import dataclasses
import re

import numpy as np
import pytest

from paper_2506_18879_amd import synth

from test_gpu_parity import TOL_SCORE, assert_rows, gpu, oracle_out, oracle_out_paired  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu


def _check(gpu, oracle, w, **kw):
    import torch
    print(f"case {w.name} lens={np.diff(w.cu_seqlens)[:12]}", flush=True)
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w, **kw)
    s, out = op.scores(dw), op(dw)
    torch.cuda.synchronize()
    keep, got = np.diff(w.cu_seqlens) > 0, out.cpu().numpy()
    assert (got[~keep] == 0).all()                             # softmax over nothing
    full = dataclasses.replace(w, q=w.q[keep], q_pos=w.q_pos[keep], cu_seqlens=w.cu_seqlens[np.r_[True, keep]])
    ref, ref_scores, _ = (oracle_out_paired if w.key_format == "paired" else oracle_out)(oracle, full, return_intermediates=True)
    assert np.abs(s.cpu().numpy().astype(np.float64) - ref_scores).max() <= TOL_SCORE
    assert_rows(got[keep], ref, w.name)
    op.close()


def launched(op, dw, kernel):
    """The template arguments (whole numbers) of the one kernel of that name that a call launches."""
    import torch
    from torch.profiler import ProfilerActivity, profile
    with profile(activities=[ProfilerActivity.CUDA]) as trace:
        op(dw)
        torch.cuda.synchronize()
    names = {m.group(1) for e in trace.events() for m in [re.search(kernel + r"<([\d, ]+)>", e.name)] if m}
    assert len(names) == 1, [e.name for e in trace.events()]
    return tuple(int(x) for x in names.pop().split(","))


@pytest.mark.parametrize("Mk,G", [(16, 4), (16, 8), (32, 2), (32, 8)])
@pytest.mark.parametrize("lens", [[512, 1, 513, 511, 1024, 700, 3, 512, 1537], [40, 2000, 512, 0, 1023, 9],
                                  [0, 2700, 0, 0, 1513, 1300, 0]])
def test_sequences_that_share_a_workgroup(gpu, oracle, Mk, G, lens):  # noqa: F811
    # boundaries between sequences at even and odd passes, queries at, before (negative distances) and past the end, an empty
    # sequence between two others, at the beginning and at the end
    w = synth.make_workload(f"share_m{Mk}_g{G}_{len(lens)}", B=len(lens), Hq=8 * G, Hkv=8, seqlens=lens, Mk=Mk, Mv=16,
                            dtype="bf16", seed=Mk + G + len(lens))
    w.q_pos = np.array([(max(1, x) - 1, x // 3, x + 777)[i % 3] for i, x in enumerate(lens)], np.int32)
    op = gpu.DecodeAttention(w, max_position=4096)
    assert op.plan.score_kernel == 1
    op.close()
    _check(gpu, oracle, w, max_position=4096)


@pytest.mark.parametrize("Mk", [16, 32])
def test_more_sequences_than_one_round_of_the_segment_lookup(gpu, oracle, Mk):  # noqa: F811
    lens = [(37 * i) % 601 + 1 for i in range(150)]
    _check(gpu, oracle, synth.make_workload(f"many_m{Mk}", B=150, Hq=4, Hkv=1, seqlens=lens, Mk=Mk, Mv=16, dtype="bf16", seed=Mk))


@pytest.mark.parametrize("Mk", [16, 32])
@pytest.mark.parametrize("heads,L", [(4, 20000), (4, 13000), (8, 20000), (8, 9000), (1, 33000)])
def test_numbers_of_passes(gpu, oracle, Mk, heads, L):  # noqa: F811
    # one KV head at long lengths: two or three passes a workgroup, 4 to 16 slice groups
    _check(gpu, oracle, synth.make_workload(f"passes_m{Mk}_g{heads}_{L}", B=1, Hq=heads, Hkv=1, seqlens=[L], Mk=Mk, Mv=16,
                                            dtype="bf16", seed=L + Mk))


# (M_k, query heads per KV head, KV heads, sequences, longest, passes, slice groups): every kernel that a plan can name, in batches whose workgroups go
# through several slices.  Up to 4 heads: logits in halves, or rows exchanged in pairs of passes.
HALVES, EXCHANGE, WIDE = 1, 0, 2


@pytest.mark.parametrize("Mk,G,Hkv,B,longest,passes,groups,form", [
    (16, 4, 8, 42, 700, 2, 1, EXCHANGE), (16, 2, 16, 42, 700, 4, 1, EXCHANGE), (16, 2, 16, 22, 255, 6, 4, EXCHANGE), (16, 2, 16, 30, 255, 8, 4, EXCHANGE),
    (16, 4, 16, 1, 14477, 2, 1, HALVES), (16, 2, 2, 18, 11000, 3, 1, HALVES), (16, 2, 8, 66, 900, 4, 1, HALVES), (16, 2, 16, 50, 600, 5, 1, HALVES),
    (16, 2, 16, 26, 800, 6, 2, HALVES), (16, 2, 16, 66, 700, 7, 1, HALVES), (16, 4, 16, 66, 900, 8, 1, HALVES),
    (16, 8, 8, 42, 600, 2, 1, WIDE), (16, 8, 8, 66, 514, 3, 1, WIDE), (16, 8, 16, 42, 600, 4, 1, WIDE), (16, 8, 16, 50, 600, 5, 1, WIDE),
    (16, 8, 16, 66, 514, 6, 1, WIDE), (16, 8, 16, 26, 300, 7, 4, WIDE), (16, 8, 16, 66, 900, 8, 1, WIDE),
    (32, 2, 2, 42, 514, 2, 4, HALVES), (32, 4, 8, 18, 3000, 3, 1, HALVES), (32, 4, 16, 42, 600, 4, 1, HALVES), (32, 2, 16, 50, 600, 5, 1, HALVES),
    (32, 4, 16, 66, 514, 6, 1, HALVES), (32, 1, 16, 66, 700, 7, 1, HALVES), (32, 4, 16, 66, 900, 8, 1, HALVES),
    (32, 8, 4, 26, 300, 2, 4, WIDE), (32, 8, 4, 26, 514, 3, 4, WIDE), (32, 8, 16, 26, 1300, 4, 1, WIDE), (32, 8, 16, 50, 600, 5, 1, WIDE),
    (32, 8, 16, 66, 514, 6, 1, WIDE), (32, 8, 16, 26, 300, 7, 4, WIDE), (32, 8, 16, 66, 900, 8, 1, WIDE)])
def test_every_number_of_passes(gpu, oracle, Mk, G, Hkv, B, longest, passes, groups, form):  # noqa: F811
    # an empty sequence at the beginning and at the end, queries at, before (negative distances) and past the ends
    lens = [longest] if B == 1 else [0] + [longest - 97 * i % (longest // 2) for i in range(B - 2)] + [0]
    w = synth.make_workload(f"np{passes}_m{Mk}_g{G}_{B}", B=B, Hq=G * Hkv, Hkv=Hkv, seqlens=lens, Mk=Mk, Mv=16, dtype="bf16", seed=B + longest)
    w.q_pos = np.array([(max(1, x) - 1, x // 3, x + 777)[i % 3] for i, x in enumerate(lens)], np.int32)
    most = longest + 1024
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w, max_position=most)
    assert op.plan.score_slice_groups == groups
    assert launched(op, dw, "k_score_stream") == (Mk, form, passes)
    op.close()
    _check(gpu, oracle, w, max_position=most)


def test_partial_logits_of_every_number_of_groups(gpu, oracle):  # noqa: F811
    # sums of 2, 4, 8 and 16 groups' partial logits, for lengths around the 256 tokens of a round and the 1024 of a workgroup, empty sequences
    seen = set()
    for i, (Hkv, Mk, lens) in enumerate([(1, 32, [255]), (2, 32, [256, 0, 257]), (1, 16, [1023, 1024, 1025]), (2, 16, [700, 0, 1, 1300]), (8, 32, [5121, 511]),
                                         (2, 16, [7000, 1, 6143]), (2, 32, [20001]), (8, 16, [9000]), (8, 16, [7000] * 3), (8, 32, [32768]), (4, 16, [9001] * 5), (8, 16, [1025, 256, 255] * 7)]):
        w = synth.make_workload(f"parts_{i}", B=len(lens), Hq=4 * Hkv, Hkv=Hkv, seqlens=lens, Mk=Mk, Mv=16, dtype="bf16", seed=600 + i)
        op = gpu.DecodeAttention(w)
        if op.plan.score_kernel == 1:
            seen.add(op.plan.score_slice_groups)
        op.close()
        _check(gpu, oracle, w)
    assert {2, 4, 8, 16} <= seen, seen


def test_query_that_is_not_16_byte_aligned(gpu, oracle):  # noqa: F811
    import torch
    w = synth.make_workload("odd_q", B=2, Hq=8, Hkv=2, seqlens=[900, 1300], Mk=16, Mv=16, dtype="bf16", seed=3)
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w)
    room = torch.empty(dw.q.numel() + 1, dtype=dw.q.dtype, device="cuda")
    room[1:] = dw.q.view(-1)
    dw.q = room[1:]
    out = op(dw)
    torch.cuda.synchronize()
    assert_rows(out.cpu().numpy(), oracle_out(oracle, w), w.name)
    op.close()


@pytest.mark.parametrize("max_position", [64, 100, 127, 128, 129])
@pytest.mark.parametrize("form", ["m16", "m32", "paired", "gathered"])
def test_keys_after_the_query_up_to_the_largest_distance(gpu, oracle, form, max_position):  # noqa: F811
    """A negative distance is 64 H + lo with lo >= 0, so |H| reaches max_position / 64 rounded up."""
    L = max_position + 1
    if form == "paired":
        w = synth.make_pair_workload(f"far_{form}", B=2, Hq=8, Hkv=2, seqlens=[L, L], R=11, Mv=16, seed=L)
    else:
        w = synth.make_workload(f"far_{form}", B=2, Hq=8, Hkv=2, seqlens=[L, L], Mk=32 if form == "m32" else 16, Mv=16,
                                dtype="f32" if form == "gathered" else "bf16", seed=L)
    w.q_pos = np.array([0, L - 1], np.int32)
    _check(gpu, oracle, w, max_position=max_position)
