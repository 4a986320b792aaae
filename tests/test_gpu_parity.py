"""GPU parity: libcommvq (through its C ABI) against the fp64 CPU oracle, element by element.

Contract: per (sequence, head) row, max |out - ref| / max |ref| <= 2e-3 on the attention output; logits from the
score stage within 2e-5 absolute (fp32 accumulation of ~4k terms of order 1).  Beside the contract every case also
has to stay within a regression bar ten times the error observed when the kernels were written (2e-6 per row):
2e-5 per row, and 2e-2 element by element relative to max(|ref|, 1e-3 max|ref|) (outputs are sign-mixed and pass
through zero, so a pure element-wise relative error is not defined).
"""
import numpy as np
import pytest

from paper_2506_18879_amd import synth

pytestmark = pytest.mark.gpu

TOL_OUT = 2e-3        # the contract
TOL_REGRESS = 2e-5    # ten times the observed row error
TOL_ELEM = 2e-2       # element-wise, with the floor below
ELEM_FLOOR = 1e-3
TOL_SCORE = 2e-5


@pytest.fixture(scope="module")
def gpu():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2506_18879_amd as cv
    cv.load_library()
    from paper_2506_18879_amd import device
    return device


def oracle_out(oracle, w, **kw):
    return oracle.decode_attn(w.as_f64("q"), w.key_codes, w.val_codes, w.as_f64("key_codebooks"),
                              w.as_f64("val_codebooks"), w.cu_seqlens, w.q_pos, key_pos=w.key_pos,
                              rope_base=w.rope_base, n_threads=16, **kw)


def row_err(got, ref):
    got = np.asarray(got, np.float64)
    return np.abs(got - ref).max(axis=-1) / np.abs(ref).max(axis=-1)


def elem_err(got, ref):
    got = np.asarray(got, np.float64)
    floor = ELEM_FLOOR * np.abs(ref).max(axis=-1, keepdims=True)
    return np.abs(got - ref) / np.maximum(np.abs(ref), floor)


def assert_rows(got, ref, what="", regress=TOL_REGRESS):
    """The contract and the regression bars on a set of output rows; returns the largest row error."""
    assert np.isfinite(np.asarray(got)).all(), what
    e, el = float(row_err(got, ref).max()), float(elem_err(got, ref).max())
    assert e <= TOL_OUT, (what, "contract", e)
    assert e <= regress, (what, "regression bar", e)
    assert el <= 1e3 * regress, (what, "element-wise regression bar", el)
    return e


def run_gpu(gpu, w, staged=False, **kw):
    import torch
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w, **kw)
    out = op.staged(dw) if staged else op(dw)
    torch.cuda.synchronize()
    res = out.cpu().numpy()
    op.close()
    return res


def check(gpu, oracle, w, regress=TOL_REGRESS, **kw):
    print(f"case {w.name} B={w.B} Hq={w.Hq} Hkv={w.Hkv} Mk={w.Mk} Mv={w.Mv} lens={np.diff(w.cu_seqlens)[:8]}", flush=True)
    got = run_gpu(gpu, w, **kw)
    ref = oracle_out(oracle, w)
    err = assert_rows(got, ref, w.name, regress)
    print(f"  max row error {err:.3e}, element-wise (floor {ELEM_FLOOR:g}) {elem_err(got, ref).max():.3e}", flush=True)
    return got, ref


# ---------------------------------------------------------------- the score stage on its own
@pytest.mark.parametrize("idx,L", [(1, 777), (2, 1500), (2, 6001), (3, 1100), (3, 7000), (5, 900), (5, 2100)])
def test_scores_match_oracle_logits(gpu, oracle, idx, L):
    import torch
    w = synth.config(idx, max_len=L)
    print(f"scores case config {idx} L={L}", flush=True)
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w)
    s = op.scores(dw)
    torch.cuda.synchronize()
    got = s.cpu().numpy().astype(np.float64)
    op.close()
    _, ref, _ = oracle_out(oracle, w, return_intermediates=True)
    assert np.abs(got - ref).max() <= TOL_SCORE, np.abs(got - ref).max()


# ---------------------------------------------------------------- the five configurations, reduced lengths
@pytest.mark.parametrize("idx,L", [(1, 4096), (2, 3000), (3, 5001), (3, 7001), (4, 4099), (5, 2500)])
def test_configs_reduced(gpu, oracle, idx, L):
    # several score/value splits and a ragged tail (lengths are not multiples of 64)
    check(gpu, oracle, synth.config(idx, max_len=L))


@pytest.mark.parametrize("L", [3000, 7000])                 # rows gathered; slices
def test_staged_entry_points_equal_fused_call(gpu, L):
    w = synth.config(3, max_len=L)
    a = run_gpu(gpu, w)
    b = run_gpu(gpu, w, staged=True)
    # same kernels, same order; the bins are integer, so even the atomics are order-independent
    assert np.array_equal(a, b)


@pytest.mark.parametrize("idx", [3, 2, 6, 7])
def test_prepacked_key_codebooks_give_identical_bits(gpu, idx):
    import torch
    w = synth.config(idx, max_len=7000)     # index form with 16 / 32 codebooks, paired format with one / two level blocks
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w)
    assert op.plan.score_kernel == 1        # (the kernels that read the packed copy)
    a = op(dw).clone()
    op.pack_key_codebooks(dw)
    b = op(dw).clone()
    import paper_2506_18879_amd as cv
    cv.commvq_forget_packed_key_codebooks(op.handle, dw.key_codebooks)
    c = op(dw).clone()
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(a, c)
    # fp32 codebooks go through the other score kernel: packing is refused, nothing is registered
    w32 = synth.config(1, max_len=600)
    op32 = gpu.DecodeAttention(w32)
    with pytest.raises(cv.CommVQError) as e:
        cv.commvq_packed_key_codebook_bytes(op32.handle)
    assert e.value.status == 2
    op.close()
    op32.close()


# ---------------------------------------------------------------- edge cases
@pytest.mark.parametrize("L", [1, 2, 63, 64, 65, 255, 256, 257, 1023, 1024, 1025])
def test_lengths_around_tile_boundaries(gpu, oracle, L):
    w = synth.make_workload(f"edge_L{L}", B=1, Hq=8, Hkv=2, seqlens=[L], Mk=16, Mv=32, dtype="bf16", seed=100 + L)
    check(gpu, oracle, w)


@pytest.mark.parametrize("G,Hkv", [(1, 3), (2, 2), (4, 1), (8, 1)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_group_sizes_and_dtypes(gpu, oracle, G, Hkv, dtype):
    w = synth.make_workload(f"g{G}_{dtype}", B=2, Hq=G * Hkv, Hkv=Hkv, seqlens=[700, 333], Mk=32, Mv=16, dtype=dtype,
                            seed=7 * G + Hkv)
    check(gpu, oracle, w)


@pytest.mark.parametrize("G,Hkv", [(1, 2), (2, 1), (4, 2), (8, 2)])
def test_two_bit_values_with_every_group_size(gpu, oracle, G, Hkv):
    # M_v = 32: with 8 heads the bins of a KV head exceed a compute unit's LDS and are split over two workgroups
    w = synth.make_workload(f"v32_g{G}", B=2, Hq=G * Hkv, Hkv=Hkv, seqlens=[1300, 2300], Mk=16, Mv=32, dtype="bf16",
                            seed=57 * G + Hkv)
    print(f"case {w.name}", flush=True)
    check(gpu, oracle, w)


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_every_combination_of_group_size_and_code_widths(gpu, oracle, dtype):
    # every instantiation the library dispatches to: G x M_k x M_v (x codebook type), at a length with a ragged tail
    worst = 0.0
    for G in (1, 2, 4, 8):
        for Mk in (16, 32):
            for Mv in (16, 32):
                w = synth.make_workload(f"all_g{G}_k{Mk}_v{Mv}_{dtype}", B=2, Hq=G, Hkv=1, seqlens=[333, 1090], Mk=Mk, Mv=Mv,
                                        dtype=dtype, seed=1000 * G + 10 * Mk + Mv)
                print(f"case {w.name}", flush=True)
                worst = max(worst, assert_rows(run_gpu(gpu, w), oracle_out(oracle, w), w.name))
    print(f"  worst row error {worst:.3e}", flush=True)


@pytest.mark.parametrize("G,Hkv", [(1, 2), (2, 2), (8, 1)])
@pytest.mark.parametrize("L", [900, 2600, 5000])
def test_one_bit_keys_group_sizes_and_tile_lengths(gpu, oracle, G, Hkv, L):
    # M_k = 16 with every group size, at lengths that select 1024-, 2048- and 4096-token score tiles
    w = synth.make_workload(f"m16_g{G}_L{L}", B=1, Hq=G * Hkv, Hkv=Hkv, seqlens=[L], Mk=16, Mv=16, dtype="bf16",
                            seed=31 * G + L)
    check(gpu, oracle, w)


@pytest.mark.parametrize("Mk,G,lens", [(16, 4, [3000]), (32, 4, [8192]), (32, 8, [5000, 700]), (16, 1, [4097, 1, 2049]), (32, 2, [1500])])
def test_short_contexts_cut_along_the_codebook_slices(gpu, oracle, Mk, G, lens):
    # contexts too short to fill the chip with whole score tiles: several workgroups per tile, each with a group of
    # the codebook slices, partial logits added by k_score_combine (which also writes the 1024-token statistics)
    import torch
    w = synth.make_workload(f"groups_m{Mk}_g{G}", B=len(lens), Hq=2 * G, Hkv=2, seqlens=lens, Mk=Mk, Mv=16, dtype="bf16",
                            seed=4000 + Mk + G + lens[0])
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w)
    assert op.plan.score_kernel == 1 and op.plan.score_slice_groups > 1, (op.plan.score_split_len, op.plan.score_slice_groups)
    print(f"case {w.name}: tiles of {op.plan.score_split_len} tokens, {op.plan.score_slice_groups} slice groups", flush=True)
    s = op.scores(dw)
    out = op(dw)
    torch.cuda.synchronize()
    ref, ref_scores, _ = oracle_out(oracle, w, return_intermediates=True)
    assert np.abs(s.cpu().numpy().astype(np.float64) - ref_scores).max() <= TOL_SCORE
    assert_rows(out.cpu().numpy(), ref, w.name)
    op.close()


def test_slice_groups_on_the_8b_layer_at_16k(gpu, oracle):
    # the 8B-shaped layer at a 16K context, 2-bit keys: 4096-token tiles in 8 slice groups of two slices each
    import torch
    w = synth.make_workload("groups_8b_16k", B=1, Hq=32, Hkv=8, seqlens=[16384], Mk=32, Mv=32, dtype="bf16", seed=616)
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w)
    assert (op.plan.score_split_len, op.plan.score_slice_groups) == (4096, 8)
    out = op(dw)
    torch.cuda.synchronize()
    assert_rows(out.cpu().numpy(), oracle_out(oracle, w), w.name)
    op.close()


def _random_shape(case):
    """One seeded shape within the documented limits: group size, code widths, storage, key format, batch and lengths."""
    rng = np.random.Generator(np.random.PCG64(9100 + case))
    G = int(rng.choice([1, 2, 4, 8]))
    Hkv = int(rng.integers(1, 4))
    kind = ["short", "mixed", "many", "long"][case % 4]
    if kind == "short":
        lens = rng.integers(1, 700, size=int(rng.integers(1, 7)))
    elif kind == "mixed":
        lens = rng.integers(1, 6000, size=int(rng.integers(2, 6)))
    elif kind == "many":     # a serving batch: many short sequences
        lens = rng.integers(1, 300, size=int(rng.integers(20, 40)))
    else:
        lens = rng.integers(5000, 14000, size=int(rng.integers(1, 3)))
    lens = [int(x) for x in lens]
    if max(lens) < 1:
        lens[0] = 1
    return G, Hkv, lens, rng


@pytest.mark.parametrize("case", range(16))
def test_random_shapes_index_form(gpu, oracle, case):
    G, Hkv, lens, rng = _random_shape(case)
    Mk, Mv = int(rng.choice([16, 32])), int(rng.choice([16, 32]))
    dtype = "f32" if case % 5 == 4 else "bf16"
    w = synth.make_workload(f"rnd{case}", B=len(lens), Hq=G * Hkv, Hkv=Hkv, seqlens=lens, Mk=Mk, Mv=Mv, dtype=dtype,
                            seed=9200 + case, code_dist="zipf" if case % 3 == 0 else "uniform")
    check(gpu, oracle, w)


@pytest.mark.parametrize("case", range(8))
def test_random_shapes_paired_keys(gpu, oracle, case):
    G, Hkv, lens, rng = _random_shape(case + 100)
    R = int(rng.integers(1, 22))
    w = synth.make_pair_workload(f"rndp{case}", B=len(lens), Hq=G * Hkv, Hkv=Hkv, seqlens=lens, R=R, Mv=int(rng.choice([16, 32])),
                                 seed=9300 + case)
    print(f"case {w.name} R={R} G={G} Hkv={Hkv} lens={lens[:8]}", flush=True)
    got = run_gpu(gpu, w)
    assert_rows(got, oracle_out_paired(oracle, w), w.name)


@pytest.mark.parametrize("Mk", [16, 32])
@pytest.mark.parametrize("qpos", [0, 1234, 70000])
def test_contiguous_keys_with_query_inside_or_far_beyond_the_context(gpu, oracle, Mk, qpos):
    # implicit key positions 0..L-1 with the query at the start, in the middle (distances of both
    # signs inside one tile) and far past the end (large coarse phase index)
    w = synth.make_workload(f"qpos{qpos}_m{Mk}", B=2, Hq=8, Hkv=2, seqlens=[2500, 1300], Mk=Mk, Mv=16, dtype="bf16",
                            seed=17 + qpos + Mk)
    w.q_pos = np.array([qpos, qpos // 2], np.int32)
    check(gpu, oracle, w, max_position=80000)


@pytest.mark.parametrize("Mk,Mv", [(16, 16), (32, 32)])
def test_million_token_context_at_the_position_limit(gpu, oracle, Mk, Mv):
    # one sequence of 2^20 + 77 tokens with the query at the largest supported position (2^24 - 1): 257 score
    # tiles, the maximum of 256 value splits, coarse phase rows up to the end of the table
    L = (1 << 20) + 77
    w = synth.make_workload(f"long_m{Mk}", B=1, Hq=4, Hkv=1, seqlens=[L], Mk=Mk, Mv=Mv, dtype="bf16", seed=2020 + Mk)
    w.q_pos = np.array([(1 << 24) - 1], np.int32)
    check(gpu, oracle, w, max_position=1 << 24)


def test_batch_with_empty_sequences(gpu, oracle):
    # a sequence without context tokens (softmax over nothing) gets zero rows; its neighbours are unaffected
    lens = [0, 300, 0, 0, 1077, 0]
    w = synth.make_workload("empties", B=6, Hq=8, Hkv=2, seqlens=lens, Mk=16, Mv=32, dtype="bf16", seed=99)
    got = run_gpu(gpu, w)
    keep = [b for b, L in enumerate(lens) if L > 0]
    ref = oracle.decode_attn(w.as_f64("q")[keep], w.key_codes, w.val_codes, w.as_f64("key_codebooks"), w.as_f64("val_codebooks"),
                             np.concatenate([[0], np.cumsum([lens[b] for b in keep])]).astype(np.int32), w.q_pos[keep],
                             rope_base=w.rope_base, n_threads=4)
    assert np.isfinite(got).all()
    assert_rows(got[keep], ref, "empties")
    for b, L in enumerate(lens):
        if L == 0:
            assert not got[b].any()


def test_ragged_batch_with_length_one_sequence(gpu, oracle):
    w = synth.make_workload("ragged", B=5, Hq=8, Hkv=2, seqlens=[1, 2100, 64, 1, 517], Mk=32, Mv=32, dtype="bf16", seed=5)
    got, ref = check(gpu, oracle, w)
    # L = 1: the output is the decoded value of the only token
    assert row_err(got[0], ref[0]).max() <= 1e-6


def test_explicit_positions_and_negative_distances(gpu, oracle):
    rng = np.random.default_rng(3)
    w = synth.make_workload("pos", B=2, Hq=8, Hkv=2, seqlens=[900, 450], Mk=16, Mv=16, dtype="bf16", seed=11)
    w.key_pos = rng.integers(0, 131072, w.total_tokens).astype(np.int32)
    w.q_pos = np.array([131071, 40000], np.int32)  # second sequence sees keys on both sides of the query
    check(gpu, oracle, w, max_position=131072)


def test_shift_invariance_on_gpu(gpu):
    # scores depend on t - p only (Eq. attention): shifting every position leaves the output unchanged
    w = synth.make_workload("shift", B=1, Hq=4, Hkv=1, seqlens=[1200], Mk=16, Mv=16, dtype="bf16", seed=12)
    w.key_pos = np.arange(1200, dtype=np.int32)
    a = run_gpu(gpu, w, max_position=70000)
    w.key_pos = w.key_pos + 60000
    w.q_pos = w.q_pos + 60000
    b = run_gpu(gpu, w, max_position=70000)
    assert np.abs(a - b).max() <= 1e-6 * np.abs(a).max()


def test_equal_positions_scalar_lut_case(gpu, oracle):
    # the paper's hypothetical "R_i independent of i": RoPE cancels
    w = synth.make_workload("nope", B=1, Hq=4, Hkv=1, seqlens=[800], Mk=32, Mv=32, dtype="bf16", seed=13)
    w.key_pos = np.full(800, 4242, np.int32)
    w.q_pos = np.array([4242], np.int32)
    check(gpu, oracle, w)


def test_zero_query_histogram_closed_form(gpu):
    # q = 0 => uniform weights => out = hist C_V / L (Eq. optimized_v)
    w = synth.make_workload("q0", B=1, Hq=4, Hkv=1, seqlens=[1500], Mk=16, Mv=16, dtype="bf16", seed=14)
    w.q[...] = 0
    got = run_gpu(gpu, w)
    vc = w.seq_codes("val", 0)[0]
    cb = w.as_f64("val_codebooks")[0]
    want = sum(np.bincount(vc[:, m], minlength=256) @ cb[m] for m in range(16)) / 1500
    for h in range(4):
        assert np.abs(got[0, h] - want).max() <= 1e-5 * np.abs(want).max()


def test_peaked_softmax_large_logits(gpu, oracle):
    # logits of order 1e2: max-subtraction must hold on the GPU too
    w = synth.make_workload("peak", B=1, Hq=4, Hkv=1, seqlens=[2000], Mk=16, Mv=16, dtype="f32", seed=15)
    w.q *= 25.0
    check(gpu, oracle, w)


def test_run_to_run_spread(gpu):
    w = synth.config(3, max_len=4000)
    a, b, c = run_gpu(gpu, w), run_gpu(gpu, w), run_gpu(gpu, w)
    # fixed-point bins and fixed-order reductions: bit-reproducible
    assert np.array_equal(a, b) and np.array_equal(a, c)


# ---------------------------------------------------------------- keys in the paper's own paired format
def oracle_out_paired(oracle, w, **kw):
    """The oracle sees the same packed records and the same tied table, as index form with 2R tied codebooks."""
    kc = oracle.paired_as_indexed(w.key_codes, w.key_levels, w.cu_seqlens, w.Hkv)
    kcb = oracle.tied_table_as_codebooks(w.as_f64("key_codebooks"), K=w.K)
    return oracle.decode_attn(w.as_f64("q"), kc, w.val_codes, kcb, w.as_f64("val_codebooks"), w.cu_seqlens, w.q_pos,
                              rope_base=w.rope_base, n_threads=16, **kw)


@pytest.mark.parametrize("R", [11, 21, 3, 16, 17])
@pytest.mark.parametrize("G,Hkv", [(4, 2), (1, 2), (8, 1), (2, 1)])
def test_paired_keys_match_oracle(gpu, oracle, R, G, Hkv):
    w = synth.make_pair_workload(f"pair_R{R}_g{G}", B=2, Hq=G * Hkv, Hkv=Hkv, seqlens=[1500, 333], R=R, Mv=16,
                                 seed=1000 + 10 * R + G)
    print(f"case {w.name}", flush=True)
    err = assert_rows(run_gpu(gpu, w), oracle_out_paired(oracle, w), w.name)
    print(f"  max row error {err:.3e}", flush=True)


@pytest.mark.parametrize("R,L", [(11, 1), (11, 255), (11, 257), (21, 1025), (11, 5000), (21, 4097)])
def test_paired_keys_lengths_and_logits(gpu, oracle, R, L):
    import torch
    w = synth.make_pair_workload(f"pair_R{R}_L{L}", B=1, Hq=8, Hkv=2, seqlens=[L], R=R, Mv=32, seed=77 + L)
    print(f"case {w.name}", flush=True)
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w)
    s = op.scores(dw)
    out = op(dw)
    torch.cuda.synchronize()
    ref, ref_scores, _ = oracle_out_paired(oracle, w, return_intermediates=True)
    assert np.abs(s.cpu().numpy().astype(np.float64) - ref_scores).max() <= TOL_SCORE
    assert_rows(out.cpu().numpy(), ref, w.name)
    # packing the tied table ahead of time changes nothing
    op.pack_key_codebooks(dw)
    out2 = op(dw).clone()
    torch.cuda.synchronize()
    assert torch.equal(out, out2)
    op.close()


def test_paired_keys_query_inside_context_and_rejections(gpu, oracle):
    import paper_2506_18879_amd as cv
    w = synth.make_pair_workload("pair_qpos", B=2, Hq=8, Hkv=2, seqlens=[2100, 900], R=11, Mv=16, seed=5)
    w.q_pos = np.array([700, 60000], np.int32)
    got = run_gpu(gpu, w, max_position=70000)
    assert_rows(got, oracle_out_paired(oracle, w), w.name)
    # explicit key positions are not supported with paired keys; neither are fp32 tables or R > 21
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w, max_position=70000)
    import torch
    kp = torch.zeros(w.total_tokens, dtype=torch.int32, device="cuda")
    bad = cv.binding.make_positions(2, dw.cu_seqlens, dw.q_pos, kp, w.total_tokens, w.max_seqlen)
    with pytest.raises(cv.CommVQError) as e:
        cv.commvq_decode_attn(op.handle, dw.q, dw.key_codes, dw.val_codes, dw.key_codebooks, dw.val_codebooks, bad,
                              op.out, op.workspace, op.workspace_bytes)
    assert e.value.status == 2
    op.close()
    cfg = cv.Config(8, 2, 128, 16, 16, 256, cv.COMMVQ_BF16, cv.COMMVQ_BF16, 500000.0, 0.0, 4096, cv.COMMVQ_KEYS_PAIRED, 22)
    assert cv.commvq_validate_config(cfg) == 2
    cfg = cv.Config(8, 2, 128, 16, 16, 256, cv.COMMVQ_F32, cv.COMMVQ_F32, 500000.0, 0.0, 4096, cv.COMMVQ_KEYS_PAIRED, 11)
    assert cv.commvq_validate_config(cfg) == 2
    cfg = cv.Config(8, 2, 128, 16, 16, 256, cv.COMMVQ_BF16, cv.COMMVQ_BF16, 500000.0, 0.0, 4096, cv.COMMVQ_KEYS_PAIRED, 21)
    assert cv.commvq_validate_config(cfg) == 0


@pytest.mark.parametrize("idx,units", [(6, 2), (7, 1)])
def test_paired_keys_full_size_sampled_units(gpu, oracle, idx, units):
    """The 128K paired-format workloads at full size (the launch shapes bench.py --config 6 / 7 times); the
    oracle computes `units` sampled (sequence, KV head) units."""
    w = synth.config(idx)
    print(f"full-size case {w.name} T={w.total_tokens}", flush=True)
    got = run_gpu(gpu, w)
    assert np.isfinite(got).all()
    rng = np.random.default_rng(idx)
    mask = np.zeros(w.B * w.Hkv, bool)
    mask[rng.choice(w.B * w.Hkv, size=units, replace=False)] = True
    ref = oracle_out_paired(oracle, w, unit_mask=mask.reshape(w.B, w.Hkv))
    G = w.Hq // w.Hkv
    worst = 0.0
    for u in np.flatnonzero(mask):
        b, g = divmod(int(u), w.Hkv)
        worst = max(worst, assert_rows(got[b, g * G:(g + 1) * G], ref[b, g * G:(g + 1) * G], f"{w.name} unit {u}"))
    print(f"  worst row error over {units} units: {worst:.3e}", flush=True)


# ---------------------------------------------------------------- position-free keys (scalar look-up table)
def oracle_out_position_free(oracle, w, **kw):
    """No rotation at all == every key at the query's position (the rotations cancel in the dot product)."""
    kp = np.concatenate([np.full(int(n), int(p), np.int32) for n, p in zip(np.diff(w.cu_seqlens), w.q_pos)])
    return oracle.decode_attn(w.as_f64("q"), w.key_codes, w.val_codes, w.as_f64("key_codebooks"),
                              w.as_f64("val_codebooks"), w.cu_seqlens, w.q_pos, key_pos=kp, rope_base=w.rope_base,
                              n_threads=16, **kw)


@pytest.mark.parametrize("G,Hkv", [(1, 2), (2, 1), (4, 2), (8, 1)])
@pytest.mark.parametrize("Mk,dtype", [(16, "bf16"), (32, "bf16"), (32, "f32"), (16, "f32")])
def test_position_free_scalar_lut(gpu, oracle, G, Hkv, Mk, dtype):
    import torch
    w = synth.make_workload(f"lut_g{G}_m{Mk}_{dtype}", B=2, Hq=G * Hkv, Hkv=Hkv, seqlens=[2300, 517], Mk=Mk, Mv=16,
                            dtype=dtype, seed=50 + 3 * G + Mk)
    print(f"case {w.name}", flush=True)
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w, position_free=True)
    s = op.scores(dw)
    out = op(dw)
    torch.cuda.synchronize()
    ref, ref_scores, _ = oracle_out_position_free(oracle, w, return_intermediates=True)
    assert np.abs(s.cpu().numpy().astype(np.float64) - ref_scores).max() <= TOL_SCORE
    assert_rows(out.cpu().numpy(), ref, w.name)
    op.close()


@pytest.mark.parametrize("L", [1, 1023, 1025, 4097, 9000])
def test_position_free_lengths(gpu, oracle, L):
    w = synth.make_workload(f"lut_L{L}", B=1, Hq=8, Hkv=2, seqlens=[L], Mk=16, Mv=32, dtype="bf16", seed=600 + L)
    got = run_gpu(gpu, w, position_free=True)
    assert_rows(got, oracle_out_position_free(oracle, w), w.name)


# ---------------------------------------------------------------- HIP graph capture of the whole call
@pytest.mark.parametrize("idx", [3, 6])
def test_decode_attn_replays_from_a_hip_graph(gpu, idx):
    """commvq_decode_attn allocates nothing and clears memory with kernels only, so a caller may capture it.
    Every replay (with eager work and synchronisations in between, and with new queries) must give the
    eager result bit for bit."""
    import torch
    w = synth.config(idx, max_len=6000)
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w)
    eager0 = op(dw).clone()                       # also the warm-up that sets kernel attributes
    side = torch.cuda.Stream()
    graph = torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        op(dw)
        torch.cuda.synchronize()
        with torch.cuda.graph(graph, stream=side):
            op(dw)
    torch.cuda.synchronize()
    q0 = dw.q.clone()
    for rep in range(3):
        if rep:                                   # new query contents in the captured buffer
            dw.q.copy_((q0.float() * (1.0 + 0.25 * rep)).to(q0.dtype))
        op.out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        replayed = op.out.clone()
        eager = op(dw).clone()                    # eager work between replays
        torch.cuda.synchronize()
        assert torch.equal(replayed, eager), rep
        if rep == 0:
            assert torch.equal(replayed, eager0)
    op.close()


# ---------------------------------------------------------------- stage timing
def test_stage_events_are_sampled_and_leave_the_result_alone(gpu):
    import torch
    import paper_2506_18879_amd as cv
    w = synth.config(3, max_len=3000)
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w)
    plain = op(dw).clone()
    cv.commvq_profile_enable(op.handle, 3)      # calls 1, 4 and 7 of the next seven are bracketed with events
    for _ in range(7):
        out = op(dw)
    torch.cuda.synchronize()
    ms, n = cv.commvq_profile_read(op.handle)
    assert n == 3 and len(ms) == 3 and all(0.0 < t < 50.0 for t in ms), (ms, n)
    assert torch.equal(out, plain)
    cv.commvq_profile_enable(op.handle, 0)
    op(dw)
    torch.cuda.synchronize()
    assert cv.commvq_profile_read(op.handle)[1] == 0
    op.close()


# ---------------------------------------------------------------- argument checking through the C ABI
def test_error_statuses(gpu):
    import torch
    import paper_2506_18879_amd as cv
    w = synth.make_workload("err", B=1, Hq=4, Hkv=1, seqlens=[100], Mk=16, Mv=16, dtype="bf16", seed=16)
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w)
    args = (dw.q, dw.key_codes, dw.val_codes, dw.key_codebooks, dw.val_codebooks)

    def status(fn):
        with pytest.raises(cv.CommVQError) as e:
            fn()
        return e.value.status

    assert status(lambda: cv.commvq_decode_attn(op.handle, None, *args[1:], dw.positions, op.out, op.workspace,
                                                op.workspace_bytes)) == 1
    assert status(lambda: cv.commvq_decode_attn(op.handle, *args, dw.positions, op.out, op.workspace,
                                                op.workspace_bytes - 1)) == 4
    assert status(lambda: cv.commvq_decode_attn(op.handle, *args, dw.positions, op.out,
                                                op.workspace.data_ptr() + 16, op.workspace_bytes)) == 4
    assert status(lambda: cv.commvq_decode_attn(op.handle, dw.q, dw.key_codes.data_ptr() + 1, *args[2:], dw.positions,
                                                op.out, op.workspace, op.workspace_bytes)) == 3
    bad = cv.binding.make_positions(1, dw.cu_seqlens, dw.q_pos, None, 0, 100)
    assert status(lambda: cv.commvq_decode_attn(op.handle, *args, bad, op.out, op.workspace, op.workspace_bytes)) == 3
    bad = cv.binding.make_positions(1, None, dw.q_pos, None, 100, 100)
    assert status(lambda: cv.commvq_decode_attn(op.handle, *args, bad, op.out, op.workspace, op.workspace_bytes)) == 1
    # and the handle still works afterwards
    op(dw)
    torch.cuda.synchronize()
    assert torch.isfinite(op.out).all()
    op.close()


# ---------------------------------------------------------------- full benchmark sizes, sampled units
@pytest.mark.parametrize("idx,units", [(2, 8), (3, 2), (4, 3), (5, 2)])
def test_full_size_sampled_units(gpu, oracle, idx, units):
    """The configurations at their full sizes (the launch shapes bench.py times); the oracle
    computes `units` sampled (sequence, KV head) units, i.e. all G heads of each."""
    w = synth.config(idx)
    print(f"full-size case {w.name} T={w.total_tokens}", flush=True)
    got = run_gpu(gpu, w)
    assert np.isfinite(got).all()
    rng = np.random.default_rng(idx)
    mask = np.zeros(w.B * w.Hkv, bool)
    mask[rng.choice(w.B * w.Hkv, size=units, replace=False)] = True
    ref = oracle_out(oracle, w, unit_mask=mask.reshape(w.B, w.Hkv))
    G = w.Hq // w.Hkv
    worst = 0.0
    for u in np.flatnonzero(mask):
        b, g = divmod(int(u), w.Hkv)
        worst = max(worst, assert_rows(got[b, g * G:(g + 1) * G], ref[b, g * G:(g + 1) * G], f"{w.name} unit {u}"))
    print(f"  worst row error over {units} units: {worst:.3e}", flush=True)


@pytest.mark.parametrize("path", ["sliced", "row_gather", "paired", "position_free"])
def test_rope_base_and_softmax_scale_from_the_configuration(gpu, oracle, path):
    # theta_j = base^(-2j/d) with a base other than the workloads' 500000, and a logit scale other than 1/sqrt(d):
    # both are fields of the configuration and reach every score path through the handle's phase tables / scale
    import torch
    base, scale = 10000.0, 0.05
    kw = dict(B=2, Hq=8, Hkv=2, seqlens=[2100, 700], Mv=16, seed=8800, rope_base=base)
    if path == "paired":
        w = synth.make_pair_workload("cfg_paired", R=11, **kw)
    else:
        w = synth.make_workload(f"cfg_{path}", Mk=16, dtype="f32" if path == "row_gather" else "bf16", **kw)
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w, softmax_scale=scale, position_free=path == "position_free")
    got = op(dw)
    torch.cuda.synchronize()
    ref_fn = {"paired": oracle_out_paired, "position_free": oracle_out_position_free}.get(path, oracle_out)
    assert_rows(got.cpu().numpy(), ref_fn(oracle, w, scale=scale), w.name)
    op.close()


@pytest.mark.parametrize("path", ["sliced", "row_gather", "paired", "position_free"])
def test_query_type_independent_of_the_codebook_type(gpu, oracle, path):
    # q_dtype and codebook_dtype are separate fields: fp32 queries on bf16 codebooks (and bf16 queries on fp32 ones).
    # The query values stay those of the workload (widened or already representable), so the oracle result is the same.
    import torch
    kw = dict(B=2, Hq=8, Hkv=2, seqlens=[1900, 640], Mv=16, seed=8900)
    if path == "paired":
        w = synth.make_pair_workload("qt_paired", R=11, **kw)
    else:
        w = synth.make_workload(f"qt_{path}", Mk=32, dtype="f32" if path == "row_gather" else "bf16", **kw)
    dw = gpu.DeviceWorkload(w)
    if w.dtype == "bf16":
        dw.q = dw.q.float().contiguous()                       # exact widening
        q_dtype = "f32"
    else:
        w.q = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(w.q))  # representable in bf16, before either side sees it
        dw.q = gpu.to_device(synth.f32_to_bf16_bits(w.q), bf16=True)
        q_dtype = "bf16"
    op = gpu.DecodeAttention(w, q_dtype=q_dtype, position_free=path == "position_free")
    got = op(dw)
    torch.cuda.synchronize()
    ref_fn = {"paired": oracle_out_paired, "position_free": oracle_out_position_free}.get(path, oracle_out)
    assert_rows(got.cpu().numpy(), ref_fn(oracle, w), w.name)
    op.close()


def test_two_handles_on_two_streams_do_not_disturb_each_other(gpu):
    # independent handles, workspaces and streams: calls that overlap on the GPU give the bits of calls run alone
    import torch
    wa = synth.config(3, max_len=20000)
    wb = synth.make_pair_workload("conc_paired", B=2, Hq=8, Hkv=2, seqlens=[3000, 1200], R=21, Mv=32, seed=77)
    dwa, dwb = gpu.DeviceWorkload(wa), gpu.DeviceWorkload(wb)
    opa, opb = gpu.DecodeAttention(wa), gpu.DecodeAttention(wb)
    ref_a, ref_b = opa(dwa).clone(), opb(dwb).clone()
    torch.cuda.synchronize()
    sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
    outs_a = [torch.empty_like(ref_a) for _ in range(8)]
    outs_b = [torch.empty_like(ref_b) for _ in range(8)]
    for k in range(8):
        with torch.cuda.stream(sa):
            opa(dwa, out=outs_a[k])
        with torch.cuda.stream(sb):
            opb(dwb, out=outs_b[k])
    torch.cuda.synchronize()
    for k in range(8):
        assert torch.equal(outs_a[k], ref_a) and torch.equal(outs_b[k], ref_b), k
    opa.close()
    opb.close()


@pytest.mark.parametrize("G,Hkv,Mv,lens", [(4, 2, 16, [900, 40, 2100, 0, 333]), (8, 1, 32, [1500, 700]), (1, 2, 32, [300] * 17),
                                           (2, 2, 16, [64, 1, 5000, 129, 77, 2048, 3, 999, 12])])
def test_batched_output_stage_on_the_matrix_cores(gpu, oracle, G, Hkv, Mv, lens):
    # batches of indexed values: bins x value codebook on the matrix cores inside k_values.  It reads the codebook as it is: packing and
    # forgetting are accepted and change nothing.  (What they do for binary values: test_gpu_output_batches.py)
    import torch
    import paper_2506_18879_amd as cv
    assert len(lens) * G >= 16
    w = synth.make_workload(f"outmfma_g{G}_v{Mv}", B=len(lens), Hq=G * Hkv, Hkv=Hkv, seqlens=lens, Mk=16, Mv=Mv, dtype="bf16",
                            seed=6100 + G + Mv)
    dw = gpu.DeviceWorkload(w)
    op = gpu.DecodeAttention(w)
    a = op(dw).clone()
    op.pack_value_codebooks(dw)
    b = op(dw).clone()
    cv.commvq_forget_packed_value_codebooks(op.handle, dw.val_codebooks)
    c = op(dw).clone()
    torch.cuda.synchronize()
    assert torch.equal(a, b) and torch.equal(a, c)
    keep = [i for i, n in enumerate(lens) if n > 0]       # (the oracle rejects empty sequences; their rows are zeros)
    got = a.cpu().numpy()
    ref = oracle.decode_attn(w.as_f64("q")[keep], w.key_codes, w.val_codes, w.as_f64("key_codebooks"), w.as_f64("val_codebooks"),
                             np.concatenate([[0], np.cumsum([lens[i] for i in keep])]).astype(np.int32), w.q_pos[keep],
                             rope_base=w.rope_base, n_threads=8)
    assert_rows(got[keep], ref, w.name)
    for i, n in enumerate(lens):
        if n == 0:
            assert not got[i].any()
    op.close()
