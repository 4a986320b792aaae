"""The statistics that the value stages gather from the score tiles, by 64 lanes and up to four tiles a lane at once: one fp32 head has
tiles of 16 tokens, so that contexts of a few thousand tokens have 63 to 325 of them.  Peaked weights: the maximum lies anywhere."""
import numpy as np
import pytest

from paper_2506_18879_amd import synth

from test_gpu_binary_values import check, make
from test_gpu_parity import assert_rows, gpu, oracle_out  # noqa: F401  (gpu: fixture)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("L", [1008, 1024, 1040, 2049, 4096, 4097, 5200])
@pytest.mark.parametrize("binary", [False, True])
def test_tiles_of_a_context(gpu, oracle, L, binary):  # noqa: F811
    if binary:
        w = make(1, 1, 1, [L], 1024, dtype="f32", seed=L)
    else:
        w = synth.make_workload("tiles", B=1, Hq=1, Hkv=1, seqlens=[L], Mk=16, Mv=16, dtype="f32", seed=L)
    w.q[...] = w.q * 2.0
    if binary:
        check(gpu, oracle, w)
        return
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w)
    got = op(dw).cpu().numpy()
    assert_rows(got, oracle_out(oracle, w), w.name)
    op.close()
