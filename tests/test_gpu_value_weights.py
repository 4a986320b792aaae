"""The softmax weights of indexed values, fixed-point numbers in k_values, against 64 bits: the value stage and the product with the codebook
from the logits that the score stage left, where a workgroup's range of tokens is longer than a value split of the plan."""
import math

import numpy as np
import pytest

from paper_2506_18879_amd import synth

from test_gpu_parity import gpu  # noqa: F401  (fixture)

pytestmark = pytest.mark.gpu


def make(keys, G, Hkv, Mv, dtype, lens):
    """Codebooks of mean zero: in the mean of many values the weights' rounding averages out as the values do, so that it is seen at any length."""
    kw = dict(B=len(lens), Hq=G * Hkv, Hkv=Hkv, seqlens=lens, Mv=Mv, seed=G + len(lens))
    w = synth.make_pair_workload("weights", R=11, **kw) if keys == "paired" else synth.make_workload("weights", Mk=16, dtype=dtype, **kw)
    cb = w.as_f64("val_codebooks")
    cb = (cb - cb.mean(axis=2, keepdims=True)).astype(np.float32)
    w.val_codebooks = synth.f32_to_bf16_bits(cb) if dtype == "bf16" else cb
    return w


def exact_output(w, logits, vlen):
    """Output rows from the logits in 64 bits, and the relative error (2-norm, random signs) that weights rounded to 2^-30 of the exp-sum of
    value splits of vlen tokens would give: half a unit per token at most, uniform, on values whose coordinates have unit variance."""
    import torch
    cb = torch.from_numpy(w.as_f64("val_codebooks")).cuda()                # [Hkv][M][K][d]
    G = w.Hq // w.Hkv
    out = torch.zeros((w.B, w.Hq, w.d), dtype=torch.float64, device="cuda")
    noise = 0.0
    for b in range(w.B):
        c0, L = int(w.cu_seqlens[b]), int(w.cu_seqlens[b + 1] - w.cu_seqlens[b])
        codes = torch.from_numpy(w.val_codes[c0 * w.Hkv * w.Mv:(c0 + L) * w.Hkv * w.Mv].astype(np.int64)).cuda().view(w.Hkv, L, w.Mv)
        s = logits[c0 * w.Hq:(c0 + L) * w.Hq].view(w.Hq, L).double()
        p = torch.exp(s - s.max(dim=1, keepdim=True).values)
        for h in range(w.Hq):
            rows = (torch.arange(w.Mv, device="cuda") * w.K + codes[h // G]).view(-1)
            bins = torch.zeros(w.Mv * w.K, dtype=torch.float64, device="cuda").index_add_(0, rows, p[h].repeat_interleave(w.Mv))
            out[b, h] = bins @ cb[h // G].reshape(w.Mv * w.K, w.d) / p[h].sum()
        for part in p.split(vlen, dim=1):
            noise += float(((part.sum(dim=1) / p.sum(dim=1) * 2.0 ** -30) ** 2).sum()) * part.shape[1] / 12 * w.d
    return out, math.sqrt(noise / float((out ** 2).sum()))


# 4 and 8 codebooks a workgroup, 4 and 8 heads, one head, fp32 codebooks, column parts; ranges of 4 to 32 value splits, not whole ones among them
SHAPES = [("indexed", 4, 8, 32, "bf16", [32768]), ("indexed", 4, 8, 32, "bf16", [30001]), ("indexed", 8, 8, 32, "bf16", [32768, 20011]),
          ("indexed", 1, 32, 32, "f32", [12000]), ("indexed", 4, 32, 16, "bf16", [9999, 16384]), ("indexed", 4, 33, 32, "bf16", [16500]),
          ("indexed", 8, 16, 16, "f32", [17000]), ("paired", 8, 1, 16, "bf16", [33000, 31000]), ("free", 4, 8, 16, "bf16", [65536]),
          ("indexed", 2, 8, 32, "bf16", [40000]), ("indexed", 4, 24, 32, "bf16", [9000, 7000, 9000]), ("indexed", 4, 64, 32, "bf16", [65536])]


@pytest.mark.parametrize("keys,G,Hkv,Mv,dtype,lens", SHAPES)
def test_weights_are_as_fine_as_value_splits_make_them(gpu, keys, G, Hkv, Mv, dtype, lens):  # noqa: F811
    import torch
    w = make(keys, G, Hkv, Mv, dtype, lens)
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w, position_free=keys == "free")
    logits, out = op.scores(dw), op(dw).clone()
    assert torch.equal(op.staged(dw), out)
    ref, coarse = exact_output(w, logits, op.plan.value_split_len)
    err = float((out.double() - ref).norm() / ref.norm())
    # Besides the weights' unit: logit - max and its product with log2 e are rounded (2^-24 of the exponent each, up to 8 where the weights matter:
    # 2e-7 in all, of random sign over the tokens), sums of up to a few dozen partial rows and the exp-sums (2^-24 each: 2e-7).  Sums over the
    # rows of a codebook in fp32: nearly equal bins, 1 / K each, times M rows' coordinates of variance 1 / M are partial sums of K^-1/2, rounded
    # to 2^-24 of that, of which the output keeps what the weights' differences leave; two such roundings are allowed.
    sums = 2.0 * 2.0 ** -24 / math.sqrt(w.K) / float((ref ** 2).mean().sqrt())
    bound = math.hypot(coarse, 3e-7, sums)
    print(f"  error {err:.2e}, bound {bound:.2e} (splits of {op.plan.value_split_len}: {coarse:.2e})", flush=True)
    assert err <= bound
    op.close()


# Codebooks of any magnitude: a power of two comes through unchanged.  (Bins are whole numbers of up to 2^32, of which a product with them as they
# are would overflow from 2^96 on.)
@pytest.mark.parametrize("exponent", [-100, 100])
@pytest.mark.parametrize("G,Hkv,Mv,dtype,lens", [(4, 8, 16, "bf16", [3000]), (4, 8, 32, "bf16", [9000]), (8, 8, 32, "bf16", [3000, 5]),
                                                 (4, 8, 32, "bf16", [300] * 40), (1, 1, 16, "f32", [4000]), (8, 2, 16, "f32", [2000])])
def test_codebooks_of_any_magnitude(gpu, G, Hkv, Mv, dtype, lens, exponent):  # noqa: F811
    import torch
    w = make("indexed", G, Hkv, Mv, dtype, lens)
    dw, op = gpu.DeviceWorkload(w), gpu.DecodeAttention(w)
    plain = op(dw).clone()
    dw.val_codebooks = (dw.val_codebooks.float() * 2.0 ** exponent).to(dw.val_codebooks.dtype)
    assert torch.equal(op(dw), plain * 2.0 ** exponent)
    op.close()
