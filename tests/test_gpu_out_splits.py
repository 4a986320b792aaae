"""Binary values: sums of the bins over the context splits in k_out, at the numbers of splits where a wavefront takes another
split or another round, with 16 wavefronts a workgroup (launches of up to 256) and with four, against the fp64 oracle.

Same bar as the other binary-value tests, 2e-5 of a row's largest element: fp32 sums of at most 64 splits and 4096 rows.
"""
import numpy as np
import pytest

from test_gpu_binary_values import errors, gpu, make, oracle_out, run_gpu  # noqa: F401  (gpu: a fixture)

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
