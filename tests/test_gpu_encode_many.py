"""Index-form vectors in one call of thousands: costs screened with two parts of the residual, near ties taken again from all
three.  The codes are those of calls of a few hundred, which take every cost from all three parts: bit for bit, also where
rows tie, nearly tie, overflow or are not numbers."""
import numpy as np
import pytest

from paper_2506_18879_amd import synth
from test_gpu_encode import encode_on_gpu, gpu  # noqa: F401

pytestmark = pytest.mark.gpu


def _inputs(kind, n, w, rng):
    cb = w.as_f64("key_codebooks").astype(np.float32)                     # [heads][levels][256][128]
    keys = rng.standard_normal((n, w.Hkv, 128)).astype(np.float32)
    with np.errstate(over="ignore"):
        if kind == "equal rows":                                          # in another tile, and next to each other
            cb[:, :, 128:] = cb[:, :, :128]
            cb[:, :, 1::4] = cb[:, :, 0::4]
        elif kind == "close rows":                                        # one element differs in its last bit or two
            bits = synth.f32_to_bf16_bits(cb)
            bits[:, :, 1::4] = bits[:, :, 0::4]
            bits[:, :, 1::4, 5] ^= 1
            bits[:, :, 128:] = bits[:, :, :128]
            bits[:, :, 128:, 77] ^= 2
            cb = synth.bf16_bits_to_f32(bits)
        elif kind == "small":
            cb, keys = cb * 2.0 ** -62, keys * 2.0 ** -62
        elif kind == "large":
            cb, keys = cb * 2.0 ** 50, keys * 2.0 ** 50
        elif kind == "overflow":
            cb, keys = cb * 2.0 ** 40, keys * 2.0 ** np.float32(rng.integers(60, 100, (n, 1, 1)))
        elif kind == "not finite":
            keys[rng.integers(0, n, 40), 0, rng.integers(0, 128, 40)] = np.nan
            keys[rng.integers(0, n, 40), 1, rng.integers(0, 128, 40)] = np.inf
            cb[0, 3, rng.integers(0, 256, 9), 4] = np.nan
            cb[1, 2, rng.integers(0, 256, 9), 4] = -np.inf
    return synth.f32_to_bf16_bits(keys.astype(np.float32)), synth.f32_to_bf16_bits(cb.astype(np.float32))


# 2 heads: more than 8192 tokens in one launch of 128 a workgroup; 8: a full round of 4096, and a last workgroup of 97 tokens
@pytest.mark.parametrize("n,heads,kind", [(8193, 2, "gaussian"), (6300, 8, "gaussian"), (2145, 8, "gaussian"), (8500, 2, "equal rows"), (8500, 2, "close rows"),
                                          (8500, 2, "small"), (8500, 2, "large"), (8500, 2, "overflow"), (8500, 2, "not finite")])
def test_codes_do_not_depend_on_the_size_of_the_call(gpu, n, heads, kind):  # noqa: F811
    w = synth.make_workload("enc_many", B=1, Hq=heads, Hkv=heads, seqlens=[8], Mk=16, Mv=16, dtype="bf16", seed=n)
    keys, cb = _inputs(kind, n, w, np.random.default_rng(n))
    w.key_codebooks = cb.reshape(w.key_codebooks.shape)
    got = encode_on_gpu(gpu, w, keys, L_cap=n)
    some = np.unique(np.r_[0:512, n - 512:n, np.random.default_rng(1).integers(0, n, 500)])[:1500]
    few = 512 if heads == 8 else 500
    want = np.concatenate([encode_on_gpu(gpu, w, np.ascontiguousarray(keys[some[i:i + few]]), L_cap=few + 1) for i in range(0, len(some), few)], axis=1)
    assert np.array_equal(got[:, some], want)
