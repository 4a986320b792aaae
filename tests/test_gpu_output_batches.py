"""Batches in the output stage.  Binary values: k_out_mfma with one and several value splits, batches that do not fill the last group of
sequences, all widths of the code, the value codebook packed ahead and re-laid by the call.  Indexed values: the same batches through k_values.
Parity with the oracle as in test_gpu_parity.py and test_gpu_binary_values.py."""
import pytest

from paper_2506_18879_amd import synth

from test_gpu_binary_values import TOL_REGRESS, errors
from test_gpu_binary_values import oracle_out as oracle_binary
from test_gpu_parity import assert_rows, gpu, oracle_out  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu


def lengths(B, longest):
    lens = [(53 * i) % 97 + 1 for i in range(B)]
    lens[B // 2] = longest
    return lens


@pytest.mark.parametrize("B,G,Hkv,Mv", [(15, 4, 8, 32), (17, 4, 8, 32), (33, 4, 8, 32), (61, 4, 8, 32), (31, 8, 8, 32), (65, 1, 16, 16)])
def test_indexed_values_of_batches(gpu, oracle, B, G, Hkv, Mv):  # noqa: F811
    import torch
    w = synth.make_workload(f"out_b{B}_g{G}", B=B, Hq=G * Hkv, Hkv=Hkv, seqlens=lengths(B, 1500), Mk=16, Mv=Mv, dtype="bf16", seed=B + G)
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w)
    out = op(dw)
    torch.cuda.synchronize()
    assert_rows(out.cpu().numpy(), oracle_out(oracle, w), w.name)
    op.close()


# 16 / G sequences share a workgroup: the last group has one of 4, 2 of 4, one of 2, 1 of 16, 2 of 8 and all of its sequences.  A range of one
# workgroup of the value stage has at most 2^16 tokens, so that 66000 leave two splits however large the batch is.
@pytest.mark.parametrize("B,G,Hkv,Nc,longest,splits", [(5, 4, 8, 1024, 6000, 6), (130, 4, 8, 2048, 300, 1), (130, 4, 8, 4096, 1500, 1), (65, 8, 8, 4096, 1500, 1),
                                                       (65, 1, 32, 4096, 3000, 1), (130, 2, 8, 2048, 66000, 2), (64, 4, 8, 1024, 66000, 2), (15, 8, 2, 2048, 4000, 4)])
def test_binary_values_of_batches(gpu, oracle, B, G, Hkv, Nc, longest, splits):  # noqa: F811
    import torch
    import paper_2506_18879_amd as cv
    w = synth.make_workload(f"vbits_b{B}_g{G}", B=B, Hq=G * Hkv, Hkv=Hkv, seqlens=lengths(B, longest), Mk=16, Mv=16, dtype="bf16", seed=B + G)
    w = synth.with_binary_values(w, Nc)
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w)
    assert op.plan.value_splits == splits
    op.workspace.fill_(0xFF)
    relaid = op(dw).clone()
    op.pack_value_codebooks(dw)
    packed = op(dw).clone()
    cv.commvq_forget_packed_value_codebooks(op.handle, dw.val_codebooks)
    forgotten = op(dw).clone()
    torch.cuda.synchronize()
    op.close()
    assert torch.equal(relaid, packed) and torch.equal(relaid, forgotten)
    row, element = errors(relaid.cpu().numpy(), oracle_binary(oracle, w))
    assert row <= TOL_REGRESS and element <= 1e3 * TOL_REGRESS, (row, element)
