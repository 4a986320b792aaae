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
