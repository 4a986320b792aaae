"""The work that a user of this library has it do, as cases that can be measured.

One pass of a case is one step of a serving or learning program through the public entry points: decode attention of
one layer over a compressed cache, the encoding of new keys and values for cache append, one iteration of the codebook
learner.  A case is a dict of plain values:

  what      "decode", "encode" or "learn"
  decode    q_heads, kv_heads      the layer's shape (head_dim 128 and 256 codewords throughout)
            batch, shortest, longest, spread   context lengths: even on [shortest, longest], one of them the longest
                                               (spread: the seed of the lengths)
            keys    "indexed" with m_key codebooks, or "paired" with key_levels levels
            values  "indexed" with m_val codebooks, or "binary" with value_bits bits per token
            storage "bf16" or "f32" (queries and codebooks), codes "uniform" or "zipf", position_free
  encode    tokens new tokens of a layer with kv_heads heads: their keys (keys, m_key / key_levels) and values (m_val)
  learn     points calibration vectors of `group` sub-spaces that share one code, `centres` centres per index

A program keeps its handle, workspace, output buffer, packed codebooks and encoder tables from call to call, so they
belong to prepare(); the inputs are drawn on the GPU from the seed alone, with the distributions of the package's
synthetic workloads (block parameters N(0, M^-1/2), queries N(0, 1), uniform or Zipf(1.1) codes, code bits of density 1/2).
"""
import math
import random

import torch

import paper_2506_18879_amd as cv

HEAD_DIM, WORDS, PAIR_WORDS = 128, 256, 64
ROPE_BASE, MAX_POSITION = 500000.0, 131072
TEMPERATURE = 2.0


def _decode(name=None, **kw):
    case = {"what": "decode", "q_heads": 32, "kv_heads": 8, "batch": 1, "shortest": 1, "longest": 1, "spread": 0,
            "keys": "indexed", "m_key": 0, "key_levels": 0, "values": "indexed", "m_val": 0, "value_bits": 0,
            "storage": "bf16", "codes": "uniform", "position_free": False}
    case.update(kw)
    return case if name is None else dict(case, name=name)


def _encode(name=None, **kw):
    case = {"what": "encode", "kv_heads": 8, "tokens": 1, "keys": "indexed", "m_key": 0, "key_levels": 0, "m_val": 16}
    case.update(kw)
    return case if name is None else dict(case, name=name)


def _learn(name=None, **kw):
    case = {"what": "learn", "group": 64, "centres": 64, "points": 1}
    case.update(kw)
    return case if name is None else dict(case, name=name)


def listed():
    return [
        # a single fp32 head over a short context: the first benchmark configuration, all latency and launches
        _decode("one_head_f32_4k", q_heads=1, kv_heads=1, shortest=4096, longest=4096, m_key=32, m_val=32, storage="f32"),
        # the beginning of a chat on the 8B-shaped layer, 2 bits per scalar: a context of odd length that cannot fill the chip
        _decode("chat_8b_2bit_1k", shortest=1237, longest=1237, m_key=32, m_val=32),
        # the same layer at an ordinary long prompt (second benchmark configuration)
        _decode("long_8b_2bit_32k", shortest=32768, longest=32768, m_key=32, m_val=32),
        # the headline workload: one sequence at 128K, 1 bit, skewed code usage (third benchmark configuration)
        _decode("longest_8b_1bit_128k", shortest=131072, longest=131072, m_key=16, m_val=16, codes="zipf"),
        # serving, few long sequences of ragged length (fourth benchmark configuration)
        _decode("ragged_8b_2bit_8x64k", batch=8, shortest=8192, longest=65536, spread=5, m_key=32, m_val=32),
        # serving, many short sequences: continuous batching of chats
        _decode("chats_8b_2bit_64x1k", batch=64, shortest=512, longest=1024, spread=6, m_key=32, m_val=32),
        # the 70B-shaped layer, four sequences at 128K, 2-bit keys and 1-bit values (fifth benchmark configuration)
        _decode("largest_70b_4x128k", q_heads=64, batch=4, shortest=131072, longest=131072, m_key=32, m_val=16),
        # the paper's own 1-bit setting at 128K: paired keys and binary values
        _decode("paper_8b_1bit_128k", shortest=131072, longest=131072, keys="paired", key_levels=11, values="binary",
                value_bits=1024),
        # keys quantized after RoPE: scores from the scalar look-up table
        _decode("position_free_8b_1bit_128k", shortest=131072, longest=131072, m_key=16, m_val=16, codes="zipf",
                position_free=True),
        # cache append of one decode step of eight sequences: paired keys, indexed values
        _encode("append_8b_8_tokens", tokens=8, keys="paired", key_levels=11, m_val=16),
        # cache fill after a prompt: paired keys and indexed values at 2 bits
        _encode("prompt_8b_4000_tokens", tokens=4000, keys="paired", key_levels=21, m_val=32),
        # offline: one iteration of the learner of the tied pair table
        _learn("learn_8k_vectors", points=8192),
    ]


def _between(rng, lo, hi):
    """A whole number on [lo, hi], even over its logarithm, odd about every other time."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case of the ranges that the listed ones stand for."""
    kind = rng.choice(("one_head", "single", "single", "single", "batch", "batch", "chats", "paper", "paper",
                       "position_free", "append", "prompt", "learn"))
    if kind == "one_head":
        n = _between(rng, 300, 4096)
        return _decode(q_heads=1, kv_heads=1, shortest=n, longest=n, m_key=rng.choice((16, 32)), m_val=rng.choice((16, 32)),
                       storage="f32")
    if kind == "append":
        keys = rng.choice(({"keys": "paired", "key_levels": rng.choice((11, 21))}, {"keys": "indexed", "m_key": rng.choice((16, 32))}))
        return _encode(tokens=_between(rng, 1, 63), m_val=rng.choice((16, 32)), **keys)
    if kind == "prompt":
        keys = rng.choice(({"keys": "paired", "key_levels": rng.choice((11, 21))}, {"keys": "indexed", "m_key": rng.choice((16, 32))}))
        most = 2800 if keys["keys"] == "indexed" else 4000  # (256 dot products a level instead of 128)
        return _encode(tokens=_between(rng, 64, most), m_val=rng.choice((16, 32)), **keys)
    if kind == "learn":
        return _learn(points=_between(rng, 1000, 8192))
    layer = {"q_heads": rng.choice((32, 32, 64)), "codes": rng.choice(("uniform", "zipf"))}
    layer.update(rng.choice(({"m_key": 16, "m_val": 16}, {"m_key": 32, "m_val": 32}, {"m_key": 32, "m_val": 16})))
    if kind == "single":
        n = _between(rng, 200, MAX_POSITION)
        return _decode(shortest=n, longest=n, **layer)
    if kind == "batch":
        batch = _between(rng, 2, 16)
        n = _between(rng, 4096, min(MAX_POSITION, 524288 // batch))
        return _decode(batch=batch, shortest=max(1, n // 8), longest=n, spread=rng.randrange(1 << 20), **layer)
    if kind == "chats":
        batch = _between(rng, 17, 64)
        n = _between(rng, 256, 4096)
        return _decode(batch=batch, shortest=n // 2, longest=n, spread=rng.randrange(1 << 20), **layer)
    if kind == "position_free":
        batch = rng.choice((1, 1, 2, 4))
        n = _between(rng, 1000, MAX_POSITION // batch)
        return _decode(batch=batch, shortest=max(1, n // 2), longest=n, spread=rng.randrange(1 << 20), position_free=True, **layer)
    batch = rng.choice((1, 1, 3, 8))
    n = _between(rng, 2000, MAX_POSITION // batch)
    levels, bits = rng.choice(((11, 1024), (21, 2048)))
    return _decode(batch=batch, shortest=max(1, n // 2), longest=n, spread=rng.randrange(1 << 20), keys="paired", key_levels=levels,
                   values="binary", value_bits=bits)


def _lengths(case):
    r = random.Random(case["spread"])
    lens = [r.randint(case["shortest"], case["longest"]) for _ in range(case["batch"])]
    lens[r.randrange(len(lens))] = case["longest"]
    return lens


def _pair_record(levels):
    return (12 * levels + 7) // 8


class _Handle:
    """A library handle that goes with the state that uses it."""

    def __init__(self, case):
        paired = case["keys"] == "paired"
        binary = case.get("values") == "binary"
        kind = cv.COMMVQ_F32 if case.get("storage") == "f32" else cv.COMMVQ_BF16
        self.ptr = cv.commvq_create(cv.Config(
            case.get("q_heads", 4 * case["kv_heads"]), case["kv_heads"], HEAD_DIM, 16 if paired else case["m_key"],
            16 if binary else case["m_val"], WORDS, kind, kind, ROPE_BASE, 0.0, MAX_POSITION,
            cv.COMMVQ_KEYS_PAIRED if paired else cv.COMMVQ_KEYS_INDEXED, case["key_levels"] if paired else 0,
            1 if case.get("position_free") else 0, cv.COMMVQ_VALUES_BINARY if binary else cv.COMMVQ_VALUES_INDEXED,
            case["value_bits"] if binary else 0))

    def __del__(self):
        cv.commvq_destroy(self.ptr)


def _normal(gen, shape, std=1.0, bf16=True):
    x = torch.randn(shape, generator=gen, device="cuda")
    x.mul_(std)
    return x.to(torch.bfloat16) if bf16 else x


def _codes(gen, lens, heads, m, dist):
    """[sequence][heads][tokens][m] index bytes, one sequence after the other."""
    if dist == "uniform":
        return torch.randint(0, WORDS, (sum(lens) * heads * m,), generator=gen, device="cuda", dtype=torch.uint8)
    cdf = torch.cumsum(torch.arange(1, WORDS + 1, device="cuda", dtype=torch.float64) ** -1.1, 0)
    cdf = (cdf / cdf[-1]).to(torch.float32)
    words = torch.rand((heads, m, WORDS), generator=gen, device="cuda").argsort(-1).to(torch.uint8)  # rank -> codeword
    base = (torch.arange(heads * m, device="cuda") * WORDS).view(heads, 1, m)
    parts = []
    for n in lens:
        rank = torch.searchsorted(cdf, torch.rand((heads, n, m), generator=gen, device="cuda")).clamp_(max=WORDS - 1)
        parts.append(words.view(-1)[rank + base].view(-1))
    return torch.cat(parts)


def _pair_table(gen, case):
    levels = case["key_levels"]
    return _normal(gen, (case["kv_heads"], levels, PAIR_WORDS, HEAD_DIM), (2 * levels) ** -0.5)


def _pair_codes(gen, tokens, levels):
    """Records of uniform 6-bit pairs: every one of the 12 * levels bits is even, the unused ones are zero."""
    rec = torch.randint(0, 256, (tokens, _pair_record(levels)), generator=gen, device="cuda", dtype=torch.uint8)
    if 12 * levels % 8:
        rec[:, -1] &= (1 << 12 * levels % 8) - 1
    return rec.view(-1)


def _prepare_decode(case, gen):
    lens = _lengths(case)
    hkv, bf16 = case["kv_heads"], case["storage"] == "bf16"
    s = {"run": _run_decode, "handle": _Handle(case), "total": sum(lens), "max": max(lens)}
    h = s["handle"].ptr
    s["q"] = _normal(gen, (case["batch"], case["q_heads"], HEAD_DIM), 1.0, bf16)
    if case["keys"] == "paired":
        s["key_cb"] = _pair_table(gen, case)
        s["key_codes"] = _pair_codes(gen, s["total"] * hkv, case["key_levels"])
    else:
        s["key_cb"] = _normal(gen, (hkv, case["m_key"], WORDS, HEAD_DIM), case["m_key"] ** -0.5, bf16)
        s["key_codes"] = _codes(gen, lens, hkv, case["m_key"], case["codes"])
    if case["values"] == "binary":
        bits = case["value_bits"]
        s["val_cb"] = _normal(gen, (bits, hkv * HEAD_DIM), (0.5 * bits) ** -0.5, bf16)
        s["val_codes"] = torch.randint(0, 256, (s["total"] * bits // 8,), generator=gen, device="cuda", dtype=torch.uint8)
    else:
        s["val_cb"] = _normal(gen, (hkv, case["m_val"], WORDS, HEAD_DIM), case["m_val"] ** -0.5, bf16)
        s["val_codes"] = _codes(gen, lens, hkv, case["m_val"], case["codes"])
    ends = [0]
    for n in lens:
        ends.append(ends[-1] + n)
    s["cu"] = torch.tensor(ends, dtype=torch.int32, device="cuda")
    s["q_pos"] = torch.tensor([n - 1 for n in lens], dtype=torch.int32, device="cuda")
    s["positions"] = cv.make_positions(case["batch"], s["cu"], s["q_pos"], None, s["total"], s["max"])
    s["workspace"] = torch.empty(cv.commvq_workspace_bytes(h, case["batch"], s["total"], s["max"]), dtype=torch.uint8, device="cuda")
    s["out"] = torch.empty((case["batch"], case["q_heads"], HEAD_DIM), device="cuda")
    if bf16:  # the codebooks are a layer's constants: laid out once
        stream = torch.cuda.current_stream().cuda_stream
        s["packed_keys"] = torch.empty(cv.commvq_packed_key_codebook_bytes(h), dtype=torch.uint8, device="cuda")
        cv.commvq_pack_key_codebooks(h, s["key_cb"], s["packed_keys"], stream)
        s["packed_values"] = torch.empty(cv.commvq_packed_value_codebook_bytes(h), dtype=torch.uint8, device="cuda")
        cv.commvq_pack_value_codebooks(h, s["val_cb"], s["packed_values"], stream)
    return s


def _run_decode(s):
    cv.commvq_decode_attn(s["handle"].ptr, s["q"], s["key_codes"], s["val_codes"], s["key_cb"], s["val_cb"], s["positions"],
                          s["out"], s["workspace"], s["workspace"].numel(), torch.cuda.current_stream().cuda_stream)
    return s["out"]


def _prepare_encode(case, gen):
    hkv, n = case["kv_heads"], case["tokens"]
    s = {"run": _run_encode, "handle": _Handle(case), "tokens": n}
    h = s["handle"].ptr
    s["keys"] = _normal(gen, (n, hkv, HEAD_DIM))
    s["values"] = _normal(gen, (n, hkv, HEAD_DIM))
    if case["keys"] == "paired":
        s["key_cb"], rec = _pair_table(gen, case), _pair_record(case["key_levels"])
    else:
        s["key_cb"], rec = _normal(gen, (hkv, case["m_key"], WORDS, HEAD_DIM), case["m_key"] ** -0.5), case["m_key"]
    s["val_cb"] = _normal(gen, (hkv, case["m_val"], WORDS, HEAD_DIM), case["m_val"] ** -0.5)
    s["key_tables"] = torch.empty(cv.commvq_encoder_table_bytes(h), dtype=torch.uint8, device="cuda")
    s["val_tables"] = torch.empty(cv.commvq_value_encoder_table_bytes(h), dtype=torch.uint8, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    cv.commvq_encoder_prepare(h, s["key_cb"], s["key_tables"], stream)
    cv.commvq_value_encoder_prepare(h, s["val_cb"], s["val_tables"], stream)
    s["key_codes"] = torch.zeros((hkv, n, rec), dtype=torch.uint8, device="cuda")
    s["val_codes"] = torch.zeros((hkv, n, case["m_val"]), dtype=torch.uint8, device="cuda")
    return s


def _run_encode(s):
    n, stream = s["tokens"], torch.cuda.current_stream().cuda_stream
    for encode, new, book, tables, codes in ((cv.commvq_encode_keys, "keys", "key_cb", "key_tables", "key_codes"),
                                             (cv.commvq_encode_values, "values", "val_cb", "val_tables", "val_codes")):
        rec = s[codes].shape[-1]
        encode(s["handle"].ptr, s[new], n, s[book], s[tables], s[codes], rec, n * rec, stream)
    return {"key_codes": s["key_codes"], "val_codes": s["val_codes"]}


def _prepare_learn(case, gen):
    g, n, c = case["group"], case["points"], case["centres"]
    s = {"run": _run_learn, "shape": (g, n, c)}
    s["data"] = _normal(gen, (n, g, 2), 1.0, False)
    s["start"] = _normal(gen, (g, c, 2), 0.5, False)
    s["phi"] = torch.empty_like(s["start"])
    s["workspace"] = torch.empty(cv.commvq_em_shared_workspace_bytes(g, n, c), dtype=torch.uint8, device="cuda")
    return s


def _run_learn(s):
    # the iteration works in place: it starts from the same table each time, so that a pass is the same work each time
    s["phi"].copy_(s["start"])
    cv.commvq_em_step_shared(s["data"], *s["shape"], TEMPERATURE, s["phi"], s["workspace"], s["workspace"].numel(),
                             torch.cuda.current_stream().cuda_stream)
    return s["phi"]


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    return {"decode": _prepare_decode, "encode": _prepare_encode, "learn": _prepare_learn}[case["what"]](case, gen)


def run(state):
    return state["run"](state)


def work(case):
    """Bytes: every input read once, every output written once.  Operations: those of the formulation that the library
    documents (gather-sum, rotation and query product; code bins and one codebook product; distances by dot products)."""
    d = HEAD_DIM
    if case["what"] == "learn":
        g, n, c = case["group"], case["points"], case["centres"]
        return {"bytes": 8 * g * n + 2 * 8 * g * c, "flops": n * (8 * c * g + 33 * c * c)}
    hkv = case["kv_heads"]
    paired = case["keys"] == "paired"
    key_rec = _pair_record(case["key_levels"]) if paired else case["m_key"]
    if case["what"] == "encode":
        n, levels, m_val = case["tokens"], case["key_levels"], case["m_val"]
        key_rows = levels * PAIR_WORDS if paired else case["m_key"] * WORDS
        key_ops = levels * (4 * d * PAIR_WORDS + 2 * PAIR_WORDS ** 2 + 2 * d) if paired else case["m_key"] * (2 * d * WORDS + 2 * WORDS + d)
        return {"bytes": n * hkv * (2 * 2 * d + key_rec + m_val) + 2 * d * hkv * (key_rows + m_val * WORDS),
                "flops": n * hkv * (key_ops + m_val * (2 * d * WORDS + 2 * WORDS + d))}
    size = 2 if case["storage"] == "bf16" else 4
    tokens, hq, batch = sum(_lengths(case)), case["q_heads"], case["batch"]
    adds = 2 * case["key_levels"] if paired else case["m_key"]
    key_rows = case["key_levels"] * PAIR_WORDS if paired else case["m_key"] * WORDS
    if case["position_free"]:
        flops = 2 * batch * hq * key_rows * d + tokens * hq * adds
    else:
        flops = tokens * hkv * d * (adds + 3) + 2 * tokens * hq * d
    nbytes = tokens * hkv * key_rec + 2 * 4 * (batch + 1) + batch * hq * d * (size + 4) + size * d * hkv * key_rows
    if case["values"] == "binary":
        bits = case["value_bits"]
        flops += 2 * hq * bits * tokens + 2 * batch * hq * bits * d
        nbytes += tokens * bits // 8 + size * d * hkv * bits
    else:
        flops += tokens * hq * case["m_val"] + 2 * batch * hq * case["m_val"] * WORDS * d
        nbytes += tokens * hkv * case["m_val"] + size * d * hkv * case["m_val"] * WORDS
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """All results are sums of 32-bit arithmetic; codes are bytes, of which a near tie of two distances may turn a few."""
    if case["what"] == "encode":
        return {"differ": 5e-4}
    return {"rel": 1e-5 if case["what"] == "decode" else 2e-5}
