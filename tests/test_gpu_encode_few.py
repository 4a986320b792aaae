"""Index-form vectors, few at a time: the parts of up to five tokens in one operand, costs summed in another order, near ties taken again.
The codes are those of a call of hundreds: bit for bit, also where rows tie, nearly tie, overflow or are not numbers."""
import numpy as np
import pytest

from paper_2506_18879_amd import synth
from test_gpu_encode import encode_on_gpu, gpu  # noqa: F401
from test_gpu_encode_many import _inputs

pytestmark = pytest.mark.gpu


# 2 heads: up to 640 tokens in workgroups of five; 700 go to workgroups of 16
@pytest.mark.parametrize("kind", ["gaussian", "equal rows", "close rows", "small", "large", "overflow", "not finite"])
def test_codes_of_few_vectors(gpu, kind):  # noqa: F811
    w = synth.make_workload("enc_few", B=1, Hq=2, Hkv=2, seqlens=[8], Mk=32, Mv=16, dtype="bf16", seed=5)
    keys, cb = _inputs(kind, 700, w, np.random.default_rng(5))
    w.key_codebooks = cb.reshape(w.key_codebooks.shape)
    want = encode_on_gpu(gpu, w, keys, L_cap=700)
    for n in (1, 4, 5, 6, 11, 640):
        assert np.array_equal(encode_on_gpu(gpu, w, np.ascontiguousarray(keys[:n]), L_cap=n + 1), want[:, :n]), n
