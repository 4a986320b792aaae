"""Index-form vectors, few at a time: the parts of up to five tokens in one operand, costs summed in another order, near ties taken again.
The codes are those of a call of hundreds: bit for bit, also where rows tie, nearly tie, overflow or are not numbers."""
import numpy as np
import pytest

from paper_2506_18879_amd import synth
from test_gpu_encode import encode_on_gpu, gpu  # noqa: F401
from test_gpu_encode_many import _inputs

pytestmark = pytest.mark.gpu


# 2 heads: up to 640 tokens in workgroups of five; 700 go to workgroups of 16
@pytest.mark.parametrize("kind", ["gaussian", "equal rows", "close rows", "zero levels", "small", "large", "overflow", "not finite"])
def test_codes_of_few_vectors(gpu, kind):  # noqa: F811
    w = synth.make_workload("enc_few", B=1, Hq=2, Hkv=2, seqlens=[8], Mk=32, Mv=16, dtype="bf16", seed=5)
    keys, cb = _inputs(kind, 700, w, np.random.default_rng(5))
    w.key_codebooks = cb.reshape(w.key_codebooks.shape)
    want = encode_on_gpu(gpu, w, keys, L_cap=700)
    for n in (1, 4, 5, 6, 11, 640):
        assert np.array_equal(encode_on_gpu(gpu, w, np.ascontiguousarray(keys[:n]), L_cap=n + 1), want[:, :n]), n


# Constant vectors and rows that are permutations of one row: every row of a level is as near as every other, and which one has the
# least cost depends on the roundings of the sums alone.  The first two levels' rows are constant, so that what they leave fills all
# three parts.  The vectors are 2^10 times longer than the rows: the costs are off by their product and not by the rows' own norms.  At
# 2^-40 and 2^-62 the square of that product is below what fp32 holds.
@pytest.mark.parametrize("scale", [0, -40, -62])
def test_ties_of_long_vectors_and_small_rows(gpu, scale):  # noqa: F811
    w = synth.make_workload("enc_ties", B=1, Hq=2, Hkv=2, seqlens=[8], Mk=16, Mv=16, dtype="bf16", seed=6)
    rng = np.random.default_rng(6)
    cb = rng.permuted(np.repeat(rng.standard_normal((2, 16, 1, 128)), 256, axis=2), axis=-1)
    cb[:, 0], cb[:, 1] = 1.3828125, 1.171875 * 2.0 ** -7
    keys = np.repeat(rng.uniform(1.0, 2.0, (700, 2, 1)), 128, axis=-1)
    keys = synth.f32_to_bf16_bits((keys * 2.0 ** (10 + scale)).astype(np.float32))
    w.key_codebooks = synth.f32_to_bf16_bits((cb * 2.0 ** scale).astype(np.float32)).reshape(w.key_codebooks.shape)
    want = encode_on_gpu(gpu, w, keys, L_cap=700)
    for n in (3, 640):
        differ = int((encode_on_gpu(gpu, w, np.ascontiguousarray(keys[:n]), L_cap=n + 1) != want[:, :n]).any(axis=-1).sum())
        assert differ == 0, n
