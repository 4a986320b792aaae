"""k_values at the sizes where its shape changes or can go wrong: edges of token ranges and of rounds of 512 and 1024 threads, whole
sequences side by side (two or four, the last group not full, empty ones among them), column parts, every group size, both codebook types and
a codebook that is only element-aligned; parity with the oracle as in test_gpu_parity.py, and the stage-by-stage calls give the same bits."""
import numpy as np
import pytest

from paper_2506_18879_amd import synth

from test_gpu_parity import assert_rows, gpu, oracle_out  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu


def _many(B, longest):
    return [0 if i % 11 == 5 else longest if i == B // 2 else (97 * i) % longest + 1 for i in range(B)]


@pytest.mark.parametrize("G,Hkv,Mv,dtype,lens", [
    (4, 8, 16, "bf16", [1]), (4, 8, 32, "bf16", [1023, 1025]), (8, 8, 16, "bf16", [4097, 511, 513]), (4, 8, 16, "bf16", [9000]),
    (2, 2, 32, "bf16", [2049]), (1, 1, 16, "bf16", [1537, 2]), (1, 1, 32, "f32", [4096]), (4, 2, 16, "f32", [3000, 64]), (8, 1, 16, "f32", [1025]),
    (2, 8, 32, "f32", [700, 5]), (4, 8, 16, "bf16", _many(9, 5000)), (8, 8, 32, "bf16", _many(9, 2000)),
    (4, 8, 32, "bf16", _many(33, 1100)), (4, 8, 16, "bf16", _many(33, 600)), (8, 8, 32, "bf16", _many(17, 700))])
def test_values_shapes(gpu, oracle, G, Hkv, Mv, dtype, lens):  # noqa: F811
    import torch
    w = synth.make_workload(f"val_g{G}_{len(lens)}", B=len(lens), Hq=G * Hkv, Hkv=Hkv, seqlens=lens, Mk=16, Mv=Mv, dtype=dtype, seed=G + len(lens))
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w)
    op.workspace.fill_(0xFF)
    out = op(dw).clone()
    op.workspace.fill_(0xFF)
    assert torch.equal(op.staged(dw), out)
    flat = dw.val_codebooks.reshape(-1)
    room = torch.zeros(flat.numel() + 1, dtype=flat.dtype, device="cuda")
    room[1:] = flat
    dw.val_codebooks = room[1:].view(dw.val_codebooks.shape)
    assert torch.equal(op(dw), out)
    torch.cuda.synchronize()
    keep = [i for i, n in enumerate(lens) if n > 0]        # (the oracle rejects empty sequences; their rows are zeros)
    got = out.cpu().numpy()
    ref = oracle.decode_attn(w.as_f64("q")[keep], w.key_codes, w.val_codes, w.as_f64("key_codebooks"), w.as_f64("val_codebooks"),
                             np.concatenate([[0], np.cumsum([lens[i] for i in keep])]).astype(np.int32), w.q_pos[keep],
                             rope_base=w.rope_base, n_threads=8)
    assert_rows(got[keep], ref, w.name)
    assert not np.delete(got, keep, axis=0).any()
    op.close()


@pytest.mark.parametrize("scale", [0.0, 1.0, 3.0])
def test_values_of_flat_and_peaked_softmax(gpu, oracle, scale):  # noqa: F811
    # hot codewords and weights from equal to a single token: the fixed-point unit follows the exp-sum of the range
    w = synth.make_workload("val_peak", B=2, Hq=32, Hkv=8, seqlens=[3000, 700], Mk=16, Mv=16, dtype="f32", seed=5, code_dist="zipf")
    w.q[...] = w.q * scale
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w)
    got = op(dw).cpu().numpy()
    assert_rows(got, oracle_out(oracle, w), w.name)
    op.close()
