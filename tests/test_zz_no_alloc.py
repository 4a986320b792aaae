"""commvq_decode_attn_static (the entry point that allocates nothing: its workspace is a static device array
inside the library) against commvq_decode_attn with a caller's workspace: same kernels, so the outputs must be
bit-identical, on two calls in a row of which the second is smaller, so that whatever the first left in the shared
array cannot leak into the second."""
import numpy as np
import pytest

from paper_2506_18879_amd import synth

pytestmark = pytest.mark.gpu


def _both(cv, device, w, torch):
    dw = device.DeviceWorkload(w)
    op = device.DecodeAttention(w)
    ref = op(dw).clone()                                            # existing entry point, caller's workspace
    torch.cuda.synchronize()
    out = torch.full_like(ref, float("nan"))
    cv.commvq_decode_attn_static(op.handle, dw.q, dw.key_codes, dw.val_codes, dw.key_codebooks, dw.val_codebooks,
                                 dw.positions, out, op.stream_ptr())
    torch.cuda.synchronize()
    return op, dw, ref, out


def test_static_scratch_entry_point_matches_workspace_entry_point(oracle):
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2506_18879_amd as cv
    from paper_2506_18879_amd import device
    assert cv.commvq_static_scratch_bytes() == 48 << 20
    # first call: the 8B-shaped 1-bit layer at 40000 tokens (several score tiles and value splits, ragged tail)
    big = synth.config(3, max_len=40000)
    op, dw, ref, out = _both(cv, device, big, torch)
    assert cv.commvq_workspace_bytes(op.handle, big.B, big.total_tokens, big.max_seqlen) <= cv.commvq_static_scratch_bytes()
    assert torch.equal(out, ref)
    want = oracle.decode_attn(big.as_f64("q"), big.key_codes, big.val_codes, big.as_f64("key_codebooks"),
                              big.as_f64("val_codebooks"), big.cu_seqlens, big.q_pos, rope_base=big.rope_base,
                              unit_mask=np.eye(1, 8, 3, dtype=bool), n_threads=1)
    got = out.cpu().numpy().astype(np.float64)
    err = np.abs(got[0, 12:16] - want[0, 12:16]).max(axis=-1) / np.abs(want[0, 12:16]).max(axis=-1)
    assert err.max() <= 2e-5
    op.close()
    # second call, smaller and of another shape (ragged batch, 2-bit values, one empty sequence): fewer score tiles,
    # fewer value splits and a different carve-up of the same array
    small = synth.make_workload("static_small", B=3, Hq=16, Hkv=4, seqlens=[1500, 0, 333], Mk=32, Mv=32, dtype="bf16", seed=321)
    op2, dw2, ref2, out2 = _both(cv, device, small, torch)
    assert torch.equal(out2, ref2)
    # again, straight after, on the same handle: the array is reused as it was left
    out3 = torch.full_like(ref2, float("nan"))
    cv.commvq_decode_attn_static(op2.handle, dw2.q, dw2.key_codes, dw2.val_codes, dw2.key_codebooks, dw2.val_codebooks,
                                 dw2.positions, out3, op2.stream_ptr())
    torch.cuda.synchronize()
    assert torch.equal(out3, ref2)
    # a batch shape beyond the array is refused before anything is launched
    too_big = cv.binding.make_positions(1, dw2.cu_seqlens, dw2.q_pos, None, 4_000_000, 4_000_000)
    op_big = device.DecodeAttention(small, max_position=1 << 23)
    with pytest.raises(cv.CommVQError) as e:
        cv.commvq_decode_attn_static(op_big.handle, dw2.q, dw2.key_codes, dw2.val_codes, dw2.key_codebooks,
                                     dw2.val_codebooks, too_big, out3, op_big.stream_ptr())
    assert e.value.status == 4
    op_big.close()
    op2.close()


@pytest.mark.parametrize("B,L,Hq,Mk,Mv", [(8, 3000, 32, 16, 16), (1, 24000, 64, 16, 16), (2, 24000, 32, 32, 32)])
def test_tiles_cut_along_the_slices_fit_the_static_scratch(oracle, B, L, Hq, Mk, Mv):
    """Partial logits, packed codebook and bins share memory: the static array holds these shapes, and the outputs do not depend on
    what the workspace held or on where the packed codebook lies."""
    import torch
    import paper_2506_18879_amd as cv
    from paper_2506_18879_amd import device
    lens = [L if i == 0 else max(1, L // 5 - 61 * i) if B == 2 else L - 7 * i for i in range(B)]
    w = synth.make_workload(f"cut_b{B}", B=B, Hq=Hq, Hkv=8, seqlens=lens, Mk=Mk, Mv=Mv, dtype="bf16", seed=B + L)
    op, dw, ref, out = _both(cv, device, w, torch)
    print(f"case B={B} L={L} groups={op.plan.score_slice_groups} workspace={op.workspace_bytes}", flush=True)
    assert op.plan.score_slice_groups > 1 and op.workspace_bytes <= cv.commvq_static_scratch_bytes()
    assert torch.equal(out, ref)
    op.workspace.fill_(0xFF)                                       # NaN wherever it is read as a float
    assert torch.equal(op(dw), ref)
    op.workspace.fill_(0xFF)
    assert torch.equal(op.staged(dw), ref)
    op.pack_key_codebooks(dw)
    op.pack_value_codebooks(dw)
    op.workspace.fill_(0xFF)
    assert torch.equal(op(dw), ref)
    want = oracle.decode_attn(w.as_f64("q"), w.key_codes, w.val_codes, w.as_f64("key_codebooks"), w.as_f64("val_codebooks"),
                              w.cu_seqlens, w.q_pos, rope_base=w.rope_base, unit_mask=np.eye(1, 8 * B, 3, dtype=bool).reshape(B, 8),
                              n_threads=16)
    G = Hq // 8
    got, want = ref.cpu().numpy().astype(np.float64)[0, 3 * G:4 * G], want[0, 3 * G:4 * G]
    assert (np.abs(got - want).max(axis=-1) / np.abs(want).max(axis=-1)).max() <= 2e-5
    op.close()
