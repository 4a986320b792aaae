"""Binary values: sums of the bins over the context splits in k_out, at the numbers of splits where a wavefront takes another
split or another round, with 16 wavefronts a workgroup (launches of up to 256) and with four, against the fp64 oracle.

Same bar as the other binary-value tests, 2e-5 of a row's largest element: fp32 sums of at most 64 splits and 4096 rows.
"""
import numpy as np
import pytest

from paper_2506_18879_amd import device, synth

from test_gpu_binary_values import errors, gpu, make, oracle_out, run_gpu  # noqa: F401  (gpu: a fixture)
from test_gpu_score_stream import _check, launched

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Hq,Hkv,lens,Nc,dtype", [
    (4, 1, [16 * 1024], 1024, "bf16"), (4, 1, [16 * 1024 + 1], 1024, "bf16"), (4, 1, [33000], 1024, "f32"),  # 16, 17, 33 splits
    (4, 1, [40000, 5000], 1024, "bf16"), (4, 1, [5000, 33000, 1], 1024, "f32"),  # fewer splits than the longest sequence
    (1, 1, [33000], 1024, "bf16"), (2, 1, [33000, 2000], 1024, "bf16"), (1, 1, [20000], 1024, "f32"), (2, 1, [20000], 1024, "f32"),
    (8, 1, [33000], 1024, "bf16"), (8, 1, [33000], 1024, "f32"),
    (16, 16, [5000], 1024, "bf16"), (17, 17, [5000], 1024, "bf16"),               # 256 and 272 workgroups, one head each
    (34, 17, [5000], 1024, "f32"), (64, 16, [9000], 2048, "bf16"), (64, 8, [9000], 4096, "bf16"), (64, 8, [5000], 4096, "f32"),
])
def test_output_over_many_splits(gpu, oracle, Hq, Hkv, lens, Nc, dtype):  # noqa: F811
    w = make(len(lens), Hq, Hkv, lens, Nc, dtype=dtype, seed=sum(lens) + Hq)
    print(f"case Hq={Hq} Hkv={Hkv} lens={lens} Nc={Nc} {dtype}", flush=True)
    got = run_gpu(gpu, w)
    row, _ = errors(got, oracle_out(oracle, w))
    assert np.isfinite(got).all() and row <= 2e-5, row


@pytest.mark.parametrize("Hq,Hkv,Mv,lens,ahead", [
    (32, 8, 16, [300, 0, 40] * 7, 1), (64, 8, 16, [700] * 9, 1),                  # up to 4 rows: one a thread
    (32, 8, 32, [1000, 0], 4), (32, 8, 16, [3500], 4), (32, 8, 16, [4097], 16),  # 8, 16 and 20
    (4, 1, 16, [16384, 1, 0, 5000], 16), (4, 1, 16, [16385], 16), (4, 1, 32, [40000], 16)])  # 64 and more: the rest in a loop
def test_rows_asked_for_ahead_of_the_length(gpu, oracle, Hq, Hkv, Mv, lens, ahead):  # noqa: F811
    # indexed values: range and codebook group of a workgroup each have a row per head
    w = synth.make_workload(f"ahead_{Hq}_{len(lens)}", B=len(lens), Hq=Hq, Hkv=Hkv, seqlens=lens, Mk=16, Mv=Mv, dtype="bf16", seed=Hq + sum(lens))
    dw, op = device.DeviceWorkload(w), device.DecodeAttention(w)
    assert launched(op, dw, "k_out_final") == (ahead,)
    op.close()
    _check(device, oracle, w)
