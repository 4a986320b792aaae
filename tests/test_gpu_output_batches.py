"""The batched output stage where a workgroup takes one, two or four chunks of codebook rows, with one and several value splits
and batches that do not fill the last group of sequences: parity with the oracle as in test_gpu_parity.py."""
import numpy as np
import pytest

from paper_2506_18879_amd import synth

from test_gpu_parity import assert_rows, gpu, oracle_out  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu


# chunks per workgroup: 1 (17 sequences), 2 (33), 4 (61; 31 with 8 heads); 15 leaves two value splits, 65 of one head five groups
@pytest.mark.parametrize("B,G,Hkv,Mv", [(15, 4, 8, 32), (17, 4, 8, 32), (33, 4, 8, 32), (61, 4, 8, 32), (31, 8, 8, 32), (65, 1, 16, 16)])
def test_chunks_of_a_workgroup(gpu, oracle, B, G, Hkv, Mv):  # noqa: F811
    import torch
    lens = [(53 * i) % 97 + 1 for i in range(B)]
    lens[B // 2] = 1500
    w = synth.make_workload(f"out_b{B}_g{G}", B=B, Hq=G * Hkv, Hkv=Hkv, seqlens=lens, Mk=16, Mv=Mv, dtype="bf16", seed=B + G)
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w)
    out = op(dw)
    torch.cuda.synchronize()
    assert_rows(out.cpu().numpy(), oracle_out(oracle, w), w.name)
    op.close()
