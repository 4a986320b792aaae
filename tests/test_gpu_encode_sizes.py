"""The encoders at the sizes where their launch changes: tokens per workgroup, as many as one workgroup per compute unit
holds, and full rounds followed by a rest."""
import numpy as np
import pytest

from paper_2506_18879_amd import synth
from test_gpu_encode import _keys, encode_on_gpu, gpu, judge  # noqa: F401

pytestmark = pytest.mark.gpu


# 8 heads: up to 512 tokens 16 per workgroup, 1024: 32, 2048: 64, 4096: 128; a rest of one token after a full round
@pytest.mark.parametrize("n,heads", [(1, 2), (15, 2), (17, 2), (63, 1), (64, 1), (512, 8), (513, 8), (1025, 8), (2049, 8), (4097, 8), (129, 3)])
def test_encode_rows_sizes(gpu, oracle, n, heads):  # noqa: F811
    w = synth.make_workload("enc_rows", B=1, Hq=heads, Hkv=heads, seqlens=[8], Mk=16, Mv=16, dtype="bf16", seed=n)
    keys, kf = _keys(np.random.default_rng(n), n, w)
    got = encode_on_gpu(gpu, w, keys, L_cap=n + 3)
    pick = np.unique(np.r_[0:min(n, 20), max(0, n - 20):n, np.random.default_rng(1).integers(0, n, 40)])
    same = [judge(oracle, kf[pick, g], w.as_f64("key_codebooks")[g], got[g, pick], False) for g in (0, heads - 1)]
    assert np.concatenate(same).mean() >= 0.99


# 8 heads: up to 64 tokens a workgroup each, 1024: 32 per workgroup, 2048: 64, 4096: 128; a rest of one token after a full round
@pytest.mark.parametrize("n,heads,R", [(1, 2, 11), (65, 8, 21), (257, 2, 2), (1025, 8, 3), (2049, 8, 3), (4097, 8, 3), (700, 3, 11)])
def test_encode_pairs_sizes(gpu, oracle, n, heads, R):  # noqa: F811
    w = synth.make_pair_workload("enc_pairs", B=1, Hq=heads, Hkv=heads, seqlens=[8], R=R, Mv=16, seed=n)
    keys, kf = _keys(np.random.default_rng(n), n, w)
    got = encode_on_gpu(gpu, w, keys, L_cap=n + 3)
    pick = np.unique(np.r_[0:min(n, 20), max(0, n - 20):n, np.random.default_rng(1).integers(0, n, 40)])
    same = []
    for g in (0, heads - 1):
        codes = np.stack(oracle.unpack_key_pairs(np.ascontiguousarray(got[g, pick]), R), axis=-1)
        same.append(judge(oracle, kf[pick, g], w.as_f64("key_codebooks")[g], codes, True))
    assert np.concatenate(same).mean() >= 0.98


def _tied_vectors(seed, n):
    """One level of one head whose costs tie in fp32 although they differ: sub-space 1 adds the same 1 - 2 * 4096 to every
    a, so that the sum of the two halves of a cost is rounded to 2^-10, while sub-space 0 holds small multiples of 2^-6.  All
    products and sums of them are exact in fp32, in any order; U rounds once, V + cross not at all."""
    rng = np.random.default_rng(seed)
    cb = np.zeros((1, 1, 64, 128), np.float32)
    cb[0, 0, :, 0:2] = rng.integers(-3, 4, (64, 2)) / 64.0
    cb[0, 0, :, 2] = 1.0
    keys = np.zeros((n, 1, 128), np.float32)
    keys[:, 0, 0:2] = rng.integers(-16, 17, (n, 2)) / 16.0
    keys[:, 0, 2] = 4096.0
    return cb, keys


# one workgroup per token, and 32, 64 and 128 tokens per workgroup
@pytest.mark.parametrize("n", [1, 200, 512, 5000, 16000, 33000])
def test_paired_ties_go_to_the_lowest_index_at_every_size(gpu, oracle, n):  # noqa: F811
    """Costs (||C[a]||^2 - 2 res.C[a]) + ((||C[b]||^2 - 2 res.(i C[b])) + cross), summed in fp32; the lowest a * 64 + b of equals."""
    cb, few = _tied_vectors(3, 500)
    keys = few[np.arange(n) % 500]
    w = synth.make_pair_workload("ties", B=1, Hq=1, Hkv=1, seqlens=[8], R=1, Mv=16, seed=1)
    w.key_codebooks = synth.f32_to_bf16_bits(cb).reshape(w.key_codebooks.shape)
    got = encode_on_gpu(gpu, w, synth.f32_to_bf16_bits(keys), L_cap=n)
    codes = np.stack(oracle.unpack_key_pairs(np.ascontiguousarray(got[0]), 1), axis=-1).reshape(n, 2).astype(np.int64)
    c = (cb[0, 0, :, 0::2] + 1j * cb[0, 0, :, 1::2]).astype(np.complex128)
    k = (few[:, 0, 0::2] + 1j * few[:, 0, 1::2]).astype(np.complex128)
    norm = (np.abs(c) ** 2).sum(1)
    U = (norm - 2 * (k @ c.conj().T).real).astype(np.float32)
    V = (norm - 2 * (k @ (1j * c).conj().T).real).astype(np.float32)
    X = (2 * (c @ (1j * c).conj().T).real).astype(np.float32)
    cost = U[:, :, None] + (V[:, None, :] + X)
    want = cost.reshape(len(k), -1).argmin(1)                  # the first of equals
    assert ((cost.reshape(len(k), -1) == cost.reshape(len(k), -1).min(1, keepdims=True)).sum(1) > 1).mean() > 0.5
    assert np.array_equal(codes[:, 0] * 64 + codes[:, 1], want[np.arange(n) % 500])


@pytest.mark.parametrize("form,n", [("f32", 3), ("bf16", 3), ("bf16", 700), ("paired", 3), ("paired", 1100), ("paired", 4200)])
def test_vectors_that_are_not_finite_leave_their_neighbours_alone(gpu, form, n):  # noqa: F811
    """NaN and infinite vectors get some record (every kernel keeps its row index in range); the others' do not change."""
    if form == "paired":
        w = synth.make_pair_workload("enc_nan", B=1, Hq=2, Hkv=2, seqlens=[8], R=3, Mv=16, seed=5)
    else:
        w = synth.make_workload("enc_nan", B=1, Hq=2, Hkv=2, seqlens=[8], Mk=16, Mv=16, dtype=form, seed=5)
    keys, _ = _keys(np.random.default_rng(n), n, w)
    bad = keys.copy()
    bad[1, 0], bad[n - 1, 1] = (np.nan, np.inf) if form == "f32" else (0x7fc0, 0x7f80)
    a, b = encode_on_gpu(gpu, w, keys, L_cap=n), encode_on_gpu(gpu, w, bad, L_cap=n)
    same = np.ones((2, n), bool)
    same[0, 1] = same[1, n - 1] = False
    assert np.array_equal(a[same], b[same])
