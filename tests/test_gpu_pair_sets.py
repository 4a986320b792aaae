"""Paired keys at the numbers of levels where the score kernel's sets of four levels begin and end, with contexts around its passes and
tiles and of several sequences: logits and outputs against the oracle as in test_gpu_parity.py."""
import numpy as np
import pytest

from paper_2506_18879_amd import synth

from test_gpu_parity import TOL_SCORE, assert_rows, gpu  # noqa: F401  (gpu: fixture)
from test_gpu_score_stream import launched

pytestmark = pytest.mark.gpu


def check(gpu, oracle, R, G, Hkv, lens, cut=None, form=None):  # noqa: F811
    import torch
    w = synth.make_pair_workload(f"sets_R{R}_{len(lens)}", B=len(lens), Hq=Hkv * G, Hkv=Hkv, seqlens=lens, R=R, Mv=16, seed=40 + R + len(lens))
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w)
    op.workspace.fill_(0xFF)
    s = op.scores(dw)
    out = op(dw)
    torch.cuda.synchronize()
    if cut:                                                # (passes of 512 tokens, groups of slices)
        _, launched_form, passes = launched(op, dw, "k_score_pair")
        assert (passes, op.plan.score_slice_groups) == cut and form in (None, launched_form)
    keep = [i for i, n in enumerate(lens) if n > 0]        # (the oracle rejects empty sequences; their rows are zeros)
    kc = oracle.paired_as_indexed(w.key_codes, w.key_levels, w.cu_seqlens, w.Hkv)
    cu = np.concatenate([[0], np.cumsum([lens[i] for i in keep])]).astype(np.int32)
    ref, ref_scores, _ = oracle.decode_attn(w.as_f64("q")[keep], kc, w.val_codes, oracle.tied_table_as_codebooks(w.as_f64("key_codebooks"), K=w.K),
                                            w.as_f64("val_codebooks"), cu, w.q_pos[keep], rope_base=w.rope_base, n_threads=16, return_intermediates=True)
    assert np.abs(s.cpu().numpy().astype(np.float64) - ref_scores).max() <= TOL_SCORE
    got = out.cpu().numpy()
    assert_rows(got[keep], ref, w.name)
    assert not np.delete(got, keep, axis=0).any()
    op.close()


@pytest.mark.parametrize("R,G,lens", [(1, 4, [700]), (4, 8, [513, 1]), (5, 4, [511, 0, 64, 63]), (12, 4, [1024, 2049]), (12, 8, [4095]), (13, 4, [300, 65]),
                                      (15, 2, [600]), (16, 4, [4100, 7]), (17, 8, [900, 130]), (20, 4, [1537]), (21, 8, [2500, 511, 0, 1024]),
                                      (21, 4, [97] * 9), (11, 4, [700, 40, 2100, 0, 333, 512, 1])])
def test_levels_around_sets(gpu, oracle, R, G, lens):  # noqa: F811
    check(gpu, oracle, R, G, 2, lens)


# Launches that are cut into three passes of 512 tokens per workgroup: whole and partly filled last ones.
@pytest.mark.parametrize("R,G,Hkv,lens,groups", [(12, 4, 8, [513, 512, 511, 514, 513], 8), (21, 4, 8, [4500], 8), (14, 4, 8, [1537] * 5, 4),
                                                 (21, 8, 8, [1536, 1537, 1535, 1600, 1537], 4), (21, 4, 16, [8400], 2), (11, 2, 16, [17500], 1)])
def test_three_passes(gpu, oracle, R, G, Hkv, lens, groups):  # noqa: F811
    check(gpu, oracle, R, G, Hkv, lens, (3, groups))


# Workgroups that go through several slices, and every number of passes, for one and two groups of four heads and each number of sets.
@pytest.mark.parametrize("R,G,Hkv,lens,cut", [
    (11, 4, 8, [14000], (2, 2)), (11, 4, 8, [30000], (2, 1)), (12, 4, 8, [40000], (3, 1)), (11, 4, 8, [70001], (8, 1)),
    (14, 4, 8, [20000], (2, 1)), (14, 4, 8, [45000], (4, 1)), (14, 4, 8, [90001], (6, 1)),
    (21, 4, 8, [15000], (2, 2)), (21, 4, 8, [40001], (6, 2)), (21, 4, 8, [70000], (6, 1)), (21, 4, 8, [2500, 100, 511, 0, 1037] * 17, (6, 1)),
    (11, 8, 8, [20000], (2, 1)), (11, 8, 8, [62001], (4, 1)), (11, 8, 8, [100000], (8, 1)),
    (14, 8, 8, [12000], (2, 2)), (14, 8, 8, [40000], (4, 1)), (14, 8, 8, [90001], (6, 1)),
    (21, 8, 8, [17000], (2, 1)), (21, 8, 8, [40000], (4, 1)), (21, 8, 8, [90000], (6, 1))])
def test_several_slices(gpu, oracle, R, G, Hkv, lens, cut):  # noqa: F811
    check(gpu, oracle, R, G, Hkv, lens, cut)


# Batches of up to 4 heads that exchange rows in pairs of passes: two passes, short sequences with every even number, an empty
# sequence at the beginning and at the end.
@pytest.mark.parametrize("R,G,Hkv,B,longest,cut", [
    (11, 1, 8, 50, 511, (2, 1)), (11, 4, 8, 26, 1300, (2, 1)), (11, 4, 16, 66, 255, (4, 1)), (11, 2, 8, 26, 300, (4, 4)),
    (14, 4, 16, 26, 300, (2, 1)), (14, 2, 16, 66, 255, (4, 1)), (21, 4, 16, 26, 300, (2, 1)), (21, 4, 16, 66, 255, (4, 1)), (21, 1, 4, 26, 300, (4, 8)),
    (11, 2, 16, 74, 255, (8, 1)), (14, 2, 16, 18, 255, (6, 4)), (21, 2, 16, 18, 255, (6, 4))])
def test_rows_exchanged_in_pairs_of_passes(gpu, oracle, R, G, Hkv, B, longest, cut):  # noqa: F811
    check(gpu, oracle, R, G, Hkv, [0] + [longest - 97 * i % (longest // 2) for i in range(B - 2)] + [0], cut, form=0)
