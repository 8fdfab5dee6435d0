"""GPU parity: the HIP path, called through the C ABI, against the CPU oracle on the same seeded
inputs.  Staged (row statistics, column scores, selection) and end to end."""
import zlib

import numpy as np
import pytest
import torch

import inputs
import oracle
import paper_2508_17892_amd as il
from parity import (ABS_TOL, REL_TOL, check_index_structure, index_set_report, index_set_report_max_avg, score_errors,
                    to_device)

pytestmark = pytest.mark.gpu


def _announce(msg):
    print(f"[case] {msg}", flush=True)


SHAPES = [
    # name, L, Lq, Hq, Hkv, dtype, channel_scale
    ("bf16_ragged_small", 1000, 8, 8, 2, "bf16", False),       # 32 rows/group: mostly padded rows, ragged tail
    ("bf16_multi_tile", 5000, 64, 8, 2, "bf16", True),         # 256 rows/group: 4-wave workgroups
    ("bf16_two_query_blocks", 3333, 160, 8, 1, "bf16", True),  # 1280 rows/group: 8-wave workgroups, 3 query blocks
    ("f32_small", 777, 32, 8, 2, "f32", False),
    ("f32_two_query_blocks", 2100, 48, 8, 2, "f32", True),     # 192 rows/group: 2 query blocks of 128
    ("bf16_single_token", 1, 4, 4, 2, "bf16", False),
    ("bf16_exact_tiles", 4096, 32, 32, 8, "bf16", False),
    # head counts of the other models the paper evaluates (Section 4): GQA groups of 7 and of 8
    ("qwen2_5_7b_heads", 3000, 64, 28, 4, "bf16", True),       # 448 rows/group: one 8-wave query block, 64 rows padded
    ("qwen3_32b_heads", 2500, 40, 64, 8, "bf16", True),        # 320 rows/group: a block of 256 and one of 128
]


@pytest.mark.parametrize("name,L,Lq,Hq,Hkv,dtype,cs", SHAPES, ids=[s[0] for s in SHAPES])
def test_staged_scoring(name, L, Lq, Hq, Hkv, dtype, cs):
    _announce(f"staged_scoring {name} L={L} Lq={Lq} Hq={Hq} Hkv={Hkv} {dtype}")
    inp = inputs.custom(L=L, Lq=Lq, Hq=Hq, Hkv=Hkv, d=128, dtype=dtype, n_spans=2 if L > 200 else 0,
                        span_len=(8, 24), channel_scale=cs, seed=zlib.crc32(name.encode()) % 1000)
    q, k = to_device(inp.q), to_device(inp.k)
    want_score, want_max, want_sum = oracle.scores(inp.q, inp.k)

    # exact form: the reference is the row maximum itself
    row_max, row_sumexp = il.ilre_row_stats(q, k, flags=il.ILRE_FLAG_EXACT_ROW_MAX)
    torch.cuda.synchronize()
    gm, gz = row_max.cpu().numpy().astype(np.float64), row_sumexp.cpu().numpy().astype(np.float64)
    np.testing.assert_allclose(gm, want_max, rtol=0, atol=1e-4)
    np.testing.assert_allclose(gz, want_sum, rtol=2e-4)
    # default form: a reference at or below the maximum, same log-sum-exp
    row_max, row_sumexp = il.ilre_row_stats(q, k)
    torch.cuda.synchronize()
    gm, gz = row_max.cpu().numpy().astype(np.float64), row_sumexp.cpu().numpy().astype(np.float64)
    assert (gm <= want_max + 1e-4).all() and np.isfinite(gz).all() and (gz >= 1.0 - 1e-5).all()
    np.testing.assert_allclose(gm + np.log(gz), want_max + np.log(want_sum), rtol=0, atol=2e-4)

    got = il.ilre_col_scores(q, k, row_max, row_sumexp)
    torch.cuda.synchronize()
    bad, worst = score_errors(got.cpu().numpy(), want_score)
    assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"
    assert abs(float(got.double().sum()) - Hq * Lq) < 1e-3 * Hq * Lq

    # column scores from the oracle's own row statistics (stage isolation)
    got2 = il.ilre_col_scores(q, k, torch.from_numpy(want_max.astype(np.float32)).cuda(),
                              torch.from_numpy(want_sum.astype(np.float32)).cuda())
    bad, worst = score_errors(got2.cpu().numpy(), want_score)
    assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"

    # Eq. 5 as printed: max over heads and queries
    want_mx, _, _ = oracle.scores(inp.q, inp.k, mode=oracle.MODE_MAX)
    got_mx = il.ilre_col_scores(q, k, row_max, row_sumexp, score_mode=il.ILRE_SCORE_MAX)
    bad, worst = score_errors(got_mx.cpu().numpy(), want_mx)
    assert bad == 0, f"max mode: {bad} scores out of tolerance, worst {worst:.2f}x"


@pytest.mark.parametrize("Lq,Hq,Hkv,L", [(1, 2, 2, 64), (1, 2, 2, 40001), (17, 28, 4, 9000), (32, 4, 1, 64 * 515), (32, 8, 2, 65), (43, 3, 1, 9000),
                                         (150, 14, 2, 9000), (170, 16, 2, 3001), (90, 21, 3, 12000),
                                         (257, 1, 1, 65), (64, 5, 1, 3000), (96, 32, 8, 9000), (48, 24, 3, 20001), (385, 1, 1, 200)],
                         ids=["1_row", "1_row_many_splits", "119_rows", "128_rows", "128_rows_ragged", "129_rows", "1050_rows", "1360_rows", "630_rows",
                              "257_rows", "320_rows", "384_rows", "384_rows_ragged", "385_rows"])
def test_scoring_narrow_query_block(Lq, Hq, Hkv, L):
    """Up to 128 query rows a kv head go one 32-row block a wavefront, more go two: both sides of the line, tiles of 64
    tokens, one and several of them a split.  257 to 384 rows are a block of 256 and one of 128 in one launch; more blocks a kv
    head than divide the places on an XCD.  Tolerance as everywhere: what fp32 sums of bf16 products allow."""
    _announce(f"narrow query block Lq={Lq} Hq={Hq} Hkv={Hkv} L={L}")
    inp = inputs.custom(L=L, Lq=Lq, Hq=Hq, Hkv=Hkv, d=128, dtype="bf16", n_spans=2 if L > 200 else 0, span_len=(8, 24),
                        channel_scale=True, seed=Lq + L)
    q, k = to_device(inp.q), to_device(inp.k)
    for gpu_mode, mode in ((il.ILRE_SCORE_SUM, oracle.MODE_SUM), (il.ILRE_SCORE_MAX, oracle.MODE_MAX)):
        want, _, _ = oracle.scores(inp.q, inp.k, mode=mode)
        _, got = il.ilre_recall(q, k, 16, (3,), score_mode=gpu_mode)
        torch.cuda.synchronize()
        bad, worst = score_errors(got.cpu().numpy(), want)
        assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"


@pytest.mark.parametrize("L,Lq,Hq,Hkv,dtype", [(300, 1, 8, 8, "bf16"), (9000, 17, 28, 4, "bf16"), (700, 40, 16, 4, "bf16"), (9000, 87, 16, 4, "bf16"),
                                               (5000, 131, 12, 4, "bf16"), (40000, 65, 28, 4, "bf16"), (300, 1, 8, 8, "f32"), (2000, 43, 12, 4, "f32"),
                                               (2000, 16, 16, 4, "f32"), (2000, 13, 20, 4, "f32")],
                         ids=["1_row", "119_rows", "160_rows", "348_rows", "393_rows", "455_rows_64_splits", "f32_1_row", "f32_129_rows",
                              "f32_64_rows", "f32_65_rows"])
def test_query_rows_however_they_lie(L, Lq, Hq, Hkv, dtype):
    """Query rows reach the kernels' registers by two ways, one for heads that follow each other without a gap; fp32 rows up to 64 a kv head
    are read without LDS in between.  Blocks of 128, 256, 256 + 128 and 512
    rows, the last of them partly filled, one row and many splits: the same bits from rows with gaps between them,
    with gaps between the heads and with the heads side by side, and the oracle's scores."""
    _announce(f"query rows L={L} Lq={Lq} {Hq}/{Hkv} {dtype}")
    inp = inputs.custom(L=L, Lq=Lq, Hq=Hq, Hkv=Hkv, d=128, dtype=dtype, n_spans=1, span_len=(8, 24), channel_scale=True, seed=Lq)
    q, k = to_device(inp.q), to_device(inp.k)
    wide = torch.zeros(Hq, Lq + 3, 136, dtype=q.dtype, device="cuda")
    token_major = torch.zeros(Lq, Hq, 128, dtype=q.dtype, device="cuda").permute(1, 0, 2)
    layouts = [wide[:, :Lq, :128], wide.new_zeros(Hq, Lq + 1, 128)[:, 1:], token_major]
    for x in layouts:
        x.copy_(q)
    for gpu_mode, mode in ((il.ILRE_SCORE_SUM, oracle.MODE_SUM), (il.ILRE_SCORE_MAX, oracle.MODE_MAX)):
        idx, scores = il.ilre_recall(q, k, 64, (3, 7), score_mode=gpu_mode)
        want, _, _ = oracle.scores(inp.q, inp.k, mode=mode)
        torch.cuda.synchronize()
        bad, worst = score_errors(scores.cpu().numpy(), want)
        assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"
        for x in layouts:
            other = il.ilre_recall(x, k, 64, (3, 7), score_mode=gpu_mode)
            torch.cuda.synchronize()
            assert torch.equal(idx, other[0]) and torch.equal(scores, other[1]), x.stride()


def test_unequal_query_blocks_want_a_workspace_for_them():
    """A block of 256 rows and one of 128 leave two partial score vectors a kv head.  A workspace that has room for one serves as
    well: one padded block is taken then."""
    L, Lq, Hq, Hkv = 9000, 96, 32, 8
    _announce("unequal query blocks, small workspace")
    inp = inputs.custom(L=L, Lq=Lq, Hq=Hq, Hkv=Hkv, d=128, dtype="bf16", n_spans=2, span_len=(8, 24), channel_scale=True, seed=3)
    q, k = to_device(inp.q), to_device(inp.k)
    full = il.alloc_workspace(L, Lq, Hq, Hkv, 128, 2, il.ILRE_BF16)
    small = torch.empty(full.numel() - Hkv * L * 4, dtype=torch.uint8, device="cuda")
    got = []
    for ws in (full, small):
        idx, scores = il.ilre_recall(q, k, 500, (3, 7), workspace=ws)
        ref, total = il.ilre_row_stats(q, k, workspace=ws)
        staged = il.ilre_col_scores(q, k, ref, total, workspace=ws)
        torch.cuda.synchronize()
        scores = scores.cpu().numpy()
        assert idx.cpu().numpy().tolist() == oracle.allocate(scores, (3, 7), 500).tolist()
        np.testing.assert_allclose(staged.cpu().numpy(), scores, rtol=4e-6, atol=0)
        got.append(scores)
    np.testing.assert_allclose(got[0], got[1], rtol=4e-6, atol=0)
    with pytest.raises(il.IlreError):
        il.ilre_recall(q, k, 500, (3, 7), workspace=small[: small.numel() // 2 // 256 * 256])


@pytest.mark.parametrize("L,Lq,Hq,Hkv", [(33001, 300, 32, 32), (60001, 2080, 16, 2)], ids=["blocks_of_256_and_128", "65_blocks_of_256"])
def test_blocks_of_unequal_size_and_rounds_with_ranges_by_the_xcds_speed(L, Lq, Hq, Hkv):
    """The second pass's token ranges follow the XCDs' speed where a split is 64 tiles and more, in launches of unequal query blocks (8 splits
    of 65 tiles of 64 tokens) and of several rounds (12 of 79) as well: the same bits with the first pass's table, without one, and in the whole path,
    and what 64 bits give."""
    _announce(f"ranges by the XCDs' speed L={L} Lq={Lq} {Hq}/{Hkv}")
    g = torch.Generator(device="cuda")
    g.manual_seed(12)
    q = torch.randn(Hq, Lq, 128, device="cuda", generator=g).to(torch.bfloat16)
    k = torch.randn(Hkv, L, 128, device="cuda", generator=g).to(torch.bfloat16)
    ws = il.alloc_workspace(L, Lq, Hq, Hkv, 128, 2, il.ILRE_BF16)
    rmax, rsum = il.ilre_row_stats(q, k, workspace=ws)
    with_table = il.ilre_col_scores(q, k, rmax, rsum, workspace=ws).clone()
    without = il.ilre_col_scores(q, k, rmax, rsum, workspace=torch.zeros_like(ws))
    _, whole = il.ilre_recall(q, k, 64, (3, 7), workspace=ws)
    want = torch.zeros(L, dtype=torch.float64, device="cuda")
    for h in range(Hq):
        kk = k[h // (Hq // Hkv)].double().t().contiguous()
        for part in q[h].double().split(256):
            want += torch.softmax(part @ kk / 128 ** 0.5, dim=1).sum(0)
    torch.cuda.synchronize()
    assert torch.equal(with_table, without) and torch.equal(with_table, whole)
    bad, worst = score_errors(whole.cpu().numpy(), want.cpu().numpy())
    assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"


@pytest.mark.parametrize("L,Lq,Hq,Hkv,dtype", [(3001, 540, 32, 1, "bf16"), (1500, 2080, 16, 2, "bf16"), (1300, 260, 32, 1, "f32"), (2100, 32, 24, 6, "f32")],
                         ids=["34_blocks_of_512", "65_blocks_of_256", "65_blocks_of_128", "fp32_33_splits"])
def test_query_blocks_that_outnumber_an_xcds_places(L, Lq, Hq, Hkv, dtype):
    """Many query blocks a kv head run in several rounds of workgroups, with more splits, and fp32 states of few tiles take more splits than the
    second pass merges where that is less work for each; a workspace that only has room for the fewer splits' partial statistics serves as well.  Tolerances as everywhere, and between the two what another order of sums gives."""
    _announce(f"many query blocks L={L} Lq={Lq} {Hq}/{Hkv} {dtype}")
    inp = inputs.custom(L=L, Lq=Lq, Hq=Hq, Hkv=Hkv, d=128, dtype=dtype, n_spans=2, span_len=(8, 24), channel_scale=True, seed=L)
    q, k = to_device(inp.q), to_device(inp.k)
    full = il.alloc_workspace(L, Lq, Hq, Hkv, 128, 2, il.ILRE_BF16 if dtype == "bf16" else il.ILRE_F32)
    small = torch.empty(full.numel() - 8 * Hq * Lq, dtype=torch.uint8, device="cuda")
    want, _, _ = oracle.scores(inp.q, inp.k)
    got = []
    for ws in (full, small):
        idx, scores = il.ilre_recall(q, k, 300, (3, 7), workspace=ws)
        ref, total = il.ilre_row_stats(q, k, workspace=ws)
        staged = il.ilre_col_scores(q, k, ref, total, workspace=ws)
        torch.cuda.synchronize()
        scores = scores.cpu().numpy()
        bad, worst = score_errors(scores, want)
        assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"
        assert idx.cpu().numpy().tolist() == oracle.allocate(scores, (3, 7), 300).tolist()
        np.testing.assert_allclose(staged.cpu().numpy(), scores, rtol=4e-6, atol=0)
        got.append(scores)
    np.testing.assert_allclose(got[0], got[1], rtol=4e-6, atol=0)


@pytest.mark.parametrize("dtype,Lq,G,Hkv", [("bf16", 20, 2, 4), ("bf16", 50, 4, 4), ("bf16", 64, 8, 2), ("bf16", 96, 4, 4), ("f32", 33, 2, 4), ("f32", 80, 2, 4)],
                         ids=["pair_of_threads_a_row", "4_waves", "8_waves", "blocks_of_256_and_128", "f32", "f32_two_query_blocks"])
def test_second_pass_merges_the_partial_statistics(dtype, Lq, G, Hkv):
    """In the whole path the second scoring pass merges the splits' partial row statistics itself, up to 32 splits (64 where all
    workgroups have as many rows, bf16), in the order the merge kernel of the staged call uses: the scores are the same bits either way.  Numbers of splits
    around the 16 sums and the line (bf16: one a tile up to 64; fp32: one for two tiles of 32 tokens, or fewer of more tiles where that keeps
    every compute unit as busy: 17 to 32 of 66 to 128 tiles with two blocks of rows); one row of a head far above the others in one split, so
    that its partial has another reference."""
    tile = 128 if dtype == "bf16" and Lq * G == 512 else 64
    g = torch.Generator(device="cuda")
    g.manual_seed(5)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    q = torch.randn(Hkv * G, Lq, 128, device="cuda", generator=g).to(dt)
    for n in (1, 2, 15, 16, 17, 24, 31, 32, 33, 48, 63, 64, 65, 100):
        L = tile * n - (n % 3)
        _announce(f"partials merged in pass 2: {dtype} Lq={Lq} G={G} Hkv={Hkv} L={L}")
        k = torch.randn(Hkv, L, 128, device="cuda", generator=g).to(dt)
        k[:, L // 2] = 12 * q[::G, 0]
        for mode in (il.ILRE_SCORE_SUM, il.ILRE_SCORE_MAX):
            rmax, rsum = il.ilre_row_stats(q, k)
            staged = il.ilre_col_scores(q, k, rmax, rsum, score_mode=mode)
            _, whole = il.ilre_recall(q, k, 16, (3,), score_mode=mode)
            torch.cuda.synchronize()
            assert torch.isfinite(whole).all()
            assert torch.equal(staged, whole), n


@pytest.mark.parametrize("seed", range(3))
def test_scoring_randomised_shapes(seed):
    """Random shapes around the kernels' block sizes (32-row query blocks, 64/128-token tiles, 4- and 8-wave
    workgroups, several token splits), both element types, sum and max reduction, whole path."""
    _announce(f"randomised scoring shapes, seed {seed}")
    rng = np.random.default_rng(7000 + seed)
    for case in range(6):
        Hkv = int(rng.choice([1, 2, 3]))
        G = int(rng.choice([1, 2, 4, 5]))
        Lq = int(rng.choice([1, 7, 31, 33, 64, 100, 130]))
        L = int(rng.choice([1, 31, 64, 127, 129, 1000, 4097, 12000])) + int(rng.integers(0, 3))
        dtype = "bf16" if rng.random() < 0.7 else "f32"
        inp = inputs.custom(L=L, Lq=Lq, Hq=Hkv * G, Hkv=Hkv, d=128, dtype=dtype, n_spans=1 if L > 300 else 0,
                            span_len=(8, 24), channel_scale=bool(rng.integers(2)), seed=100 * seed + case)
        q, k = to_device(inp.q), to_device(inp.k)
        mode = oracle.MODE_MAX if case % 3 == 2 else oracle.MODE_SUM
        want, _, _ = oracle.scores(inp.q, inp.k, mode=mode)
        _, got = il.ilre_recall(q, k, 16, (3,), score_mode=il.ILRE_SCORE_MAX if mode == oracle.MODE_MAX else il.ILRE_SCORE_SUM)
        torch.cuda.synchronize()
        bad, worst = score_errors(got.cpu().numpy(), want)
        assert bad == 0, (seed, case, L, Lq, Hkv, G, dtype, mode, bad, worst)


SELECT_CASES = [
    # name, L, kernels, budget, kind
    ("random_small", 3000, (3, 7, 15), 256, "random"),
    ("random_multi_chunk", 50000, (1, 3, 7, 15, 31), 4096, "random"),
    ("plateaus", 20000, (3, 7, 15, 31), 1024, "few_values"),
    ("all_equal", 10000, (3, 7, 15), 100, "equal"),
    ("budget_exceeds_L", 300, (3, 7), 1000, "random"),
    ("L_smaller_than_kernel", 9, (31, 15), 4, "random"),
    ("budget_not_divisible", 7000, (3, 7, 15), 256, "random"),
    ("budget_below_kernel_count", 500, (1, 3, 5, 7), 3, "random"),
    ("single_token", 1, (3,), 1, "random"),
    ("wide_kernel", 30000, (2047, 1, 255), 600, "random"),
    ("needle_like", 100000, (1, 3, 7, 15, 31), 4096, "needles"),
    ("dense_background_ties", 200000, (3, 7, 15, 31), 4096, "narrow"),
    ("max_budget", 40000, (3, 31), 8192, "random"),
    ("twelve_kernels_two_groups", 30000, (1, 3, 5, 7, 9, 11, 13, 15, 31, 63, 127, 3), 3000, "needles"),
    ("all_equal_large", 300000, (3, 7, 15, 31), 4096, "equal"),
    ("two_values_heavy_ties", 150000, (1, 7), 5000, "two_values"),
    # a later list whose best tokens are all taken: the walk has to go past its first stretch of ranks
    ("repeated_kernel_sizes", 60000, (7, 7, 7, 7), 2000, "random"),
    ("small_after_large", 80000, (63, 3, 1), 3000, "needles"),
    # long contexts: the pruning pre-pass (fine-chunk maxima) decides which chunks are visited
    ("pruned_needles", 5000000, (1, 3, 7, 15, 31), 4096, "needles"),
    ("pruned_dense_background", 4500001, (3, 31), 1000, "narrow"),
    ("pruned_wide_kernel", 5000000, (511, 3), 500, "needles"),
    ("pruned_all_equal", 4200000, (3, 7), 64, "equal"),
]


def _scores_for(kind, L, rng):
    if kind == "random":
        return rng.random(L).astype(np.float32)
    if kind == "few_values":
        return (rng.integers(1, 9, size=L) / 16.0).astype(np.float32)
    if kind == "two_values":
        return np.where(rng.random(L) < 0.01, 0.5, 0.25).astype(np.float32)
    if kind == "equal":
        return np.full(L, 0.125, dtype=np.float32)
    if kind == "narrow":   # a dense background inside one binade, as real scores are
        return (0.0078125 * (1.0 + 0.5 * rng.random(L))).astype(np.float32)
    s = (0.008 * (1.0 + 0.3 * rng.standard_normal(L))).clip(1e-4).astype(np.float32)
    for start in rng.integers(0, L - 300, size=20):
        n = int(rng.integers(64, 256))
        s[start:start + n] = (rng.random(n) * 8).astype(np.float32)
    return s


@pytest.mark.parametrize("name,L,kernels,budget,kind", SELECT_CASES, ids=[c[0] for c in SELECT_CASES])
def test_select_exact_on_given_scores(name, L, kernels, budget, kind):
    _announce(f"select {name} L={L} kernels={kernels} budget={budget}")
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    s = _scores_for(kind, L, rng)
    want = oracle.allocate(s, kernels, budget)
    got = il.ilre_select(torch.from_numpy(s).cuda(), budget, kernels)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    check_index_structure(got, L, budget)
    assert got.tolist() == want.tolist()


SINK_CASES = [
    # name, L, sink, kernels, budget, kind
    ("paper_sink_needles", 100000, 4, (1, 3, 7, 15, 31), 4096, "needles"),
    ("sink_scores_dominate", 20000, 5, (3, 7, 15), 1000, "random"),
    ("sink_is_everything", 37, 37, (3,), 16, "random"),
    ("sink_leaves_one_token", 38, 37, (3, 7), 16, "random"),
    ("sink_and_budget_exceed_L", 300, 4, (3, 7), 1000, "random"),
    ("sink_all_equal", 10000, 3, (3, 7, 15), 100, "equal"),
    ("sink_pruned_long_context", 4500001, 4, (1, 3, 7, 15, 31), 4096, "needles"),
]


@pytest.mark.parametrize("name,L,sink,kernels,budget,kind", SINK_CASES, ids=[c[0] for c in SINK_CASES])
def test_select_with_a_sink_part(name, L, sink, kernels, budget, kind):
    """Window-max form with the sink part of Algorithm 1: the first `sink` tokens always kept and invisible to
    the pooling (their scores are set far above everything else, so any leak would show), the budget counting
    the others; bit-exact with the oracle."""
    _announce(f"select with sink {name} L={L} sink={sink} kernels={kernels} budget={budget}")
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    s = _scores_for(kind, L, rng) if L > 300 else rng.random(L).astype(np.float32)
    s[:sink] = 1000.0
    want = oracle.allocate(s, kernels, budget, sink=sink)
    got = il.ilre_select(torch.from_numpy(s).cuda(), budget, kernels, sink=sink)
    torch.cuda.synchronize()
    got = got.cpu().numpy()
    assert got.shape == (sink + min(budget, L - sink),) and got.dtype == np.int32
    assert got.tolist() == want.tolist()


def test_recall_with_a_sink_part():
    """Whole path with a sink part: same scores as without (Eq. 4 runs over all L positions), selection equal to
    the staged call and to the oracle's Algorithm 1 on the GPU's own scores."""
    _announce("end_to_end with sink 4 (ragged bf16)")
    inp = inputs.custom(L=9001, Lq=40, Hq=16, Hkv=4, d=128, dtype="bf16", n_spans=3, span_len=(16, 40),
                        channel_scale=True, seed=78)
    q, k = to_device(inp.q), to_device(inp.k)
    kernels, budget, sink = (1, 3, 7, 15, 31), 512, 4
    idx, scores = il.ilre_recall(q, k, budget, kernels, sink=sink)
    _, plain_scores = il.ilre_recall(q, k, budget, kernels)
    staged = il.ilre_select(scores, budget, kernels, sink=sink)
    torch.cuda.synchronize()
    assert torch.equal(scores, plain_scores) and torch.equal(idx, staged)
    assert idx.cpu().numpy().tolist() == oracle.allocate(scores.cpu().numpy(), kernels, budget, sink=sink).tolist()
    want_scores, _, _ = oracle.scores(inp.q, inp.k)
    bad, worst = score_errors(scores.cpu().numpy(), want_scores)
    assert bad == 0, worst


PAPER_MAX, PAPER_AVG = (2, 4, 8), tuple(range(1, 17))     # the paper's default pooling set (Section 3.2)

MAX_AVG_CASES = [
    # name, L, sink, max kernels, avg kernels, budget, kind of scores
    ("paper_default_needles", 100000, 4, PAPER_MAX, PAPER_AVG, 4096, "needles"),
    ("paper_default_ragged", 50001, 4, PAPER_MAX, PAPER_AVG, 1024, "random"),
    ("snapkv_special_case", 30000, 0, (1,), (7,), 1000, "random"),
    ("plain_topk", 20000, 0, (1,), (1,), 512, "random"),
    ("one_max_avg", 40000, 4, (4,), (5,), 2048, "needles"),
    ("odd_max_kernels", 33333, 3, (3, 5, 6, 7), (1, 2, 3, 4, 9), 3000, "random"),
    ("candidates_exhausted", 3000, 2, (8, 8, 4), (1, 2, 3), 2500, "random"),
    ("budget_exceeds_L", 700, 4, (2, 4), (1, 3), 5000, "random"),
    ("budget_below_combination_count", 5000, 4, PAPER_MAX, PAPER_AVG, 5, "random"),
    ("all_equal", 60000, 4, PAPER_MAX, (1, 2, 5, 16), 4096, "equal"),
    ("plateaus", 70000, 0, (2, 8), (1, 4, 16), 4096, "few_values"),
    ("two_values_heavy_ties", 150000, 4, (2, 4), (1, 2), 6000, "two_values"),
    ("dense_background", 200000, 4, PAPER_MAX, PAPER_AVG, 4096, "narrow"),
    ("signed_with_zeros", 25000, 1, (2, 3), (1, 2, 6), 800, "signed"),
    ("wide_kernels", 90000, 0, (1024, 256), (1024, 33), 8192, "needles"),
    ("L_below_max_kernel", 5, 0, (8, 2), (1, 3), 4, "random"),
    ("sink_is_everything", 37, 37, (2,), (3,), 16, "random"),
    ("sink_leaves_one_token", 38, 37, (1, 2), (3,), 16, "random"),
    ("max_budget", 50000, 4, PAPER_MAX, PAPER_AVG, 8192, "random"),
    ("one_million_paper_default", 1 << 20, 4, PAPER_MAX, PAPER_AVG, 4096, "needles"),
]


@pytest.mark.parametrize("name,L,sink,mk,ak,budget,kind", MAX_AVG_CASES, ids=[c[0] for c in MAX_AVG_CASES])
def test_select_max_avg_exact_on_given_scores(name, L, sink, mk, ak, budget, kind):
    """Algorithm 1 as printed (strided max pooling, average pooling, K_m cap, sink part): bit-exact with
    the oracle on the same float32 scores, the unused tail of the output marked -1."""
    _announce(f"select_max_avg {name} L={L} sink={sink} max={mk} avg={ak} budget={budget}")
    rng = np.random.default_rng(zlib.crc32(name.encode()))
    if kind == "signed":
        s = rng.standard_normal(L).astype(np.float32)
        s[rng.random(L) < 0.3] = 0.0
        s[rng.random(L) < 0.1] = -0.0
    else:
        s = _scores_for(kind, L, rng) if L > 300 else rng.random(L).astype(np.float32)
    want = oracle.allocate_max_avg(s, mk, ak, budget, sink=sink)
    got, count = il.ilre_select_max_avg(torch.from_numpy(s).cuda(), budget, mk, ak, sink)
    torch.cuda.synchronize()
    got, count = got.cpu().numpy(), int(count.item())
    assert got.shape == (sink + min(budget, L - sink),) and got.dtype == np.int32
    assert count == len(want)
    assert got[:count].tolist() == want.tolist()
    assert (got[count:] == -1).all()


def test_select_max_avg_reuses_a_workspace():
    """Two calls in a row on one workspace, the second smaller: nothing of the first leaks into it."""
    _announce("select_max_avg workspace reuse")
    rng = np.random.default_rng(11)
    big, small = _scores_for("needles", 80000, rng), rng.random(9000).astype(np.float32)
    ws = il.alloc_workspace_max_avg(80000, 1, 1, 1, 128, 4, PAPER_MAX, len(PAPER_AVG), il.ILRE_F32)
    for s, budget in ((big, 4096), (small, 700), (big, 4096)):
        want = oracle.allocate_max_avg(s, PAPER_MAX, PAPER_AVG, budget, sink=4)
        got, count = il.ilre_select_max_avg(torch.from_numpy(s).cuda(), budget, PAPER_MAX, PAPER_AVG, 4, workspace=ws)
        torch.cuda.synchronize()
        assert got.cpu().numpy()[:int(count.item())].tolist() == want.tolist()


def _end_to_end(inp, kernels, budget):
    wl = inp.workload
    q, k = to_device(inp.q), to_device(inp.k)
    idx, scores = il.ilre_recall(q, k, budget, kernels)
    torch.cuda.synchronize()
    idx, scores = idx.cpu().numpy(), scores.cpu().numpy()
    want_scores, _, _ = oracle.scores(inp.q, inp.k)
    bad, worst = score_errors(scores, want_scores)
    assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"
    check_index_structure(idx, wl.L, budget)
    # the selection is Algorithm 1 run on the scores the GPU itself produced: bit-exact, no tolerance
    assert idx.tolist() == oracle.allocate(scores, kernels, budget).tolist()
    rep = index_set_report(idx, want_scores, kernels, budget)
    assert not rep["unexcused"], rep
    return idx, scores, rep


@pytest.mark.parametrize("L,Lq,Hq,Hkv,spread", [(1, 1, 1, 1, 0), (31, 3, 2, 1, 0), (33, 33, 4, 1, 2), (64, 16, 8, 1, 0), (65, 129, 2, 2, 0), (1000, 8, 8, 2, 3),
                                                (4097, 5, 28, 4, 0), (2100, 40, 16, 2, 1)])
def test_fp32_states_keep_their_precision(L, Lq, Hq, Hkv, spread):
    """fp32 states against 64 bits, at the edges of the kernels' tiles (32 tokens, 128 rows) and with channels of very different
    scale.  A logit sees 8 additions at its own size, 40 at 2^-8 of it and a few more, each rounded to 2^-24, and products that
    are 2^-24 short at most: within 16 * 2^-24 of the sum of its products' magnitudes.  A row's logarithm of a sum moves by no more
    than the worst of its logits, the sum's own rounding (2^-24 for each of its levels: 64 tokens a lane at most, in four sums, and 65 splits, in 16; 80 is more than
    all of them) and the exponentials' (2^-22 with the scaling).  A score's terms move by their logits, their rows' logarithms and the
    exponent's roundings (2^-22 of its size with the row's offset); their sum is 16 a lane, 8 of a tile and up to 16 blocks, fewer than 40
    levels.  Exponentials below the smallest normal number may be 0."""
    _announce(f"fp32 precision L={L} Lq={Lq} {Hq}/{Hkv} spread {spread}")
    rng = np.random.default_rng(L + Lq)
    channel = np.exp(spread * rng.standard_normal(128))
    q = (rng.standard_normal((Hq, Lq, 128)) * channel).astype(np.float32)
    k = (rng.standard_normal((Hkv, L, 128)) / channel * np.exp(0.3 * spread * rng.standard_normal((Hkv, L, 1)))).astype(np.float32)
    qd, kd = torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda()
    row_max, row_sum = il.ilre_row_stats(qd, kd)
    got_sum, got_top = (il.ilre_col_scores(qd, kd, row_max, row_sum, score_mode=mode) for mode in (il.ILRE_SCORE_SUM, il.ILRE_SCORE_MAX))
    torch.cuda.synchronize()
    got = row_max.cpu().numpy().astype(np.float64) + np.log(row_sum.cpu().numpy().astype(np.float64))
    group = Hq // Hkv
    scale = 1.0 / np.sqrt(128.0)
    want_sum, off_sum, want_top, off_top = (np.zeros(L) for _ in range(4))
    for h in range(Hq):
        kk = k[h // group].astype(np.float64)
        s = (q[h].astype(np.float64) @ kk.T) * scale
        size = (np.abs(q[h]).astype(np.float64) @ np.abs(kk).T) * scale
        top = s.max(axis=1)
        want = top + np.log(np.exp(s - top[:, None]).sum(axis=1))
        bound = 16 * 2.0 ** -24 * size.max(axis=1) + 2.0 ** -22 * (1 + np.abs(s).max(axis=1)) + 80 * 2.0 ** -24
        assert (np.abs(got[h * Lq:(h + 1) * Lq] - want) <= bound).all(), (h, np.abs(got[h * Lq:(h + 1) * Lq] - want).max(), bound.min())
        prob = np.exp(s - want[:, None])
        off = prob * np.expm1(16 * 2.0 ** -24 * size + bound[:, None] + 2.0 ** -22 * (1 + np.abs(s) + np.abs(want[:, None])))
        want_sum, off_sum = want_sum + prob.sum(axis=0), off_sum + off.sum(axis=0)
        want_top, off_top = np.maximum(want_top, prob.max(axis=0)), np.maximum(off_top, off.max(axis=0))
    assert (np.abs(got_sum.cpu().numpy() - want_sum) <= off_sum + 40 * 2.0 ** -24 * want_sum + 1e-37).all()
    assert (np.abs(got_top.cpu().numpy() - want_top) <= off_top + 1e-37).all()


@pytest.mark.parametrize("channels", [1, 2, 3, 4])
@pytest.mark.parametrize("kind", ["normal", "worst"])
def test_fp32_products_keep_their_precision(kind, channels):
    """Single logits (one token, exact row maxima) of fp32 states with few channels at work, where rounding does not average out.
    Each channel's large product is added with a rounding of 2^-24 but the first, the other parts with one more, what is left
    out of a product is 2^-24 at most, and the maximum leaves the library with one multiplication by ln 2: channels + 2 of
    them, with 2^-6 on top for the rounding of the small parts.  `worst`: significands that leave the most out where the parts are cut off
    instead of rounded (2^-22 of a product)."""
    _announce(f"fp32 products, {channels} channels {kind}")
    rng = np.random.default_rng(channels)
    Hkv, Lq, ln2 = 64, 256, np.float32(np.log(2.0))
    assert np.float32(ln2 * np.float32(1.4426950408889634)) == 1  # the scale that makes logits of base 2 the products themselves
    q, k = np.zeros((Hkv, Lq, 128), np.float32), np.zeros((Hkv, 1, 128), np.float32)
    for x in (q, k):
        some = rng.standard_normal(x.shape[:2] + (channels,))
        x[..., rng.choice(128, channels, replace=False) if x is q else np.flatnonzero(q[0, 0])] = some if kind == "normal" else 1.0078 + 1e-5 * some
    row_max, _ = il.ilre_row_stats(torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), scale=float(ln2), flags=il.ILRE_FLAG_EXACT_ROW_MAX)
    torch.cuda.synchronize()
    got = row_max.cpu().numpy().astype(np.float64).reshape(Hkv, Lq) / np.float64(ln2)
    products = q.astype(np.float64) * k.astype(np.float64)
    off = np.abs(got - products.sum(-1)) / np.abs(products).sum(-1)
    assert off.max() <= (channels + 2) * 2.0 ** -24 * (1 + 2.0 ** -6), off.max() * 2.0 ** 24


@pytest.mark.parametrize("small", [1e-25, 1e-32, 3e-35, 2.0 ** -126, 2.0 ** -132])
@pytest.mark.parametrize("which", ["keys", "queries"])
def test_fp32_states_of_any_magnitude(small, which):
    """Small states with partners as large as brings their products back to one: the products' errors are those of usual states (16 *
    2^-24 of the sum of their magnitudes, as above; the two multiplications behind it 2 * 2^-24), and the parts of a number below
    2^-126 are multiples of 2^-147."""
    _announce(f"fp32 states, {which} of {small}")
    rng = np.random.default_rng(7)
    large = min(1.0 / small, 2.0 ** 120)
    q, k = rng.standard_normal((8, 16, 128)), rng.standard_normal((8, 1, 128))
    q, k = (q * large, k * small) if which == "keys" else (q * small, k * large)
    q, k, ln2 = q.astype(np.float32), k.astype(np.float32), np.float32(np.log(2.0))
    row_max, _ = il.ilre_row_stats(torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), scale=float(ln2), flags=il.ILRE_FLAG_EXACT_ROW_MAX)
    torch.cuda.synchronize()
    got = row_max.cpu().numpy().astype(np.float64).reshape(8, 16) / np.float64(ln2)
    products = q.astype(np.float64) * k.astype(np.float64)
    bound = 18 * 2.0 ** -24 * np.abs(products).sum(-1) + 2.0 ** -148 * np.abs(q if which == "keys" else k).astype(np.float64).sum(-1)
    off = np.abs(got - products.sum(-1))
    assert (off <= bound).all(), (off / bound).max()


def test_fp32_states_near_the_largest_float():
    """The largest floats would round to an infinite bf16; products that are finite stay so."""
    _announce("fp32 states near the largest float")
    top = np.finfo(np.float32).max
    k = np.zeros((1, 3, 128), np.float32)
    k[0, 0, 0], k[0, 1, 0], k[0, 2, 0] = top, -top, np.float32(3.3961e38)
    q = np.zeros((1, 2, 128), np.float32)
    q[0, 0, 0], q[0, 1, 0] = 1.0, -0.3
    row_max, row_sum = il.ilre_row_stats(torch.from_numpy(q).cuda(), torch.from_numpy(k).cuda(), scale=1e-37)
    torch.cuda.synchronize()
    got = row_max.cpu().numpy().astype(np.float64) + np.log(row_sum.cpu().numpy().astype(np.float64))
    s = np.float64(np.float32(1e-37)) * (q[0].astype(np.float64) @ k[0].astype(np.float64).T)
    np.testing.assert_allclose(got, np.log(np.exp(s).sum(axis=1)), rtol=1e-6)


def test_end_to_end_cfg1():
    _announce("end_to_end cfg1")
    inp = inputs.config(1)
    idx, scores, rep = _end_to_end(inp, inp.workload.pool_kernels, inp.workload.budget)
    mask = inp.needle_mask
    assert mask[idx].sum() >= 0.95 * mask.sum()


def test_end_to_end_cfg2():
    _announce("end_to_end cfg2")
    inp = inputs.config(2)
    idx, scores, rep = _end_to_end(inp, inp.workload.pool_kernels, inp.workload.budget)
    mask = inp.needle_mask
    assert mask[idx].sum() >= 0.95 * mask.sum()


def test_end_to_end_ragged_bf16():
    _announce("end_to_end ragged bf16")
    inp = inputs.custom(L=9001, Lq=40, Hq=16, Hkv=4, d=128, dtype="bf16", n_spans=3, span_len=(16, 40),
                        channel_scale=True, seed=77)
    _end_to_end(inp, (1, 3, 7, 15, 31), 512)


def _end_to_end_max_avg(inp, mk, ak, budget, sink):
    """Whole path with Algorithm 1 as printed: scores within tolerance of the oracle's, bit-identical to
    the window-max entry point's (same scoring kernels), indices equal to the staged call on those scores,
    and equal to the oracle's set up to tokens at a combination's threshold."""
    q, k = to_device(inp.q), to_device(inp.k)
    idx, count, scores = il.ilre_recall_max_avg(q, k, budget, mk, ak, sink)
    _, ref_scores = il.ilre_recall(q, k, min(budget, 64), (3,))
    staged_idx, staged_count = il.ilre_select_max_avg(scores, budget, mk, ak, sink)
    torch.cuda.synchronize()
    assert torch.equal(scores, ref_scores)
    assert torch.equal(idx, staged_idx) and int(count.item()) == int(staged_count.item())
    n = int(count.item())
    idx, scores = idx.cpu().numpy(), scores.cpu().numpy()
    want_scores, _, _ = oracle.scores(inp.q, inp.k)
    bad, worst = score_errors(scores, want_scores)
    assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"
    assert (idx[:sink] == np.arange(sink)).all() and (np.diff(idx[:n].astype(np.int64)) > 0).all()
    assert (idx[n:] == -1).all() and idx[:n].max() < inp.workload.L
    # Algorithm 1 as printed on the scores the GPU itself produced: bit-exact, no tolerance
    assert idx[:n].tolist() == oracle.allocate_max_avg(scores, mk, ak, budget, sink=sink).tolist()
    rep = index_set_report_max_avg(idx[:n], want_scores, mk, ak, budget, sink)
    assert not rep["unexcused"], rep
    return idx[:n], rep


def test_end_to_end_max_avg_cfg1():
    _announce("end_to_end max/avg cfg1 (paper default pooling set, sink 4)")
    inp = inputs.config(1)
    idx, rep = _end_to_end_max_avg(inp, PAPER_MAX, PAPER_AVG, inp.workload.budget, 4)
    mask = inp.needle_mask
    assert mask[idx].sum() >= 0.95 * mask.sum()


def test_end_to_end_max_avg_cfg2():
    _announce("end_to_end max/avg cfg2 (paper default pooling set, sink 4)")
    inp = inputs.config(2)
    idx, rep = _end_to_end_max_avg(inp, PAPER_MAX, PAPER_AVG, inp.workload.budget, 4)
    mask = inp.needle_mask
    assert mask[idx].sum() >= 0.95 * mask.sum()


def test_end_to_end_max_avg_ragged_bf16():
    _announce("end_to_end max/avg ragged bf16")
    inp = inputs.custom(L=9001, Lq=40, Hq=16, Hkv=4, d=128, dtype="bf16", n_spans=3, span_len=(16, 40),
                        channel_scale=True, seed=77)
    _end_to_end_max_avg(inp, (4,), (5,), 512, 0)          # the paper's One-Max-Avg ablation setting
    _end_to_end_max_avg(inp, PAPER_MAX, tuple(range(1, 10)), 1000, 4)   # Less-Avg-Kernels


def test_gather_ids_is_the_compressed_prompt():
    """Last line of Algorithm 1, C[I]: by definition the input IDs at the returned indices."""
    _announce("gather ids")
    rng = np.random.default_rng(17)
    # a normal selection, and one whose candidates run out (21 tokens, cells of 8: 16 reachable, budget 20)
    for L, budget, mk, ak, sink, short in ((50000, 3000, (2, 4, 8), (1, 2, 3), 4, False), (21, 20, (8,), (1,), 0, True)):
        ids = rng.integers(0, 128256, size=L).astype(np.int32)
        s = _scores_for("needles", L, rng) if L > 300 else rng.random(L).astype(np.float32)
        idx, count = il.ilre_select_max_avg(torch.from_numpy(s).cuda(), budget, mk, ak, sink)
        got = il.ilre_gather_ids(torch.from_numpy(ids).cuda(), idx)
        torch.cuda.synchronize()
        idx_h, n = idx.cpu().numpy(), int(count.item())
        assert (n < idx_h.size) == short and (idx_h[n:] == -1).all()
        want = np.where(idx_h >= 0, ids[np.clip(idx_h, 0, L - 1)], -1)
        assert got.cpu().numpy().tolist() == want.tolist()


def test_token_major_strides():
    _announce("token-major strided K and strided Q")
    inp = inputs.custom(L=2500, Lq=16, Hq=8, Hkv=2, d=128, dtype="bf16", n_spans=1, span_len=(16, 16), seed=5)
    q, k = to_device(inp.q), to_device(inp.k)
    k_tm = k.permute(1, 0, 2).contiguous().permute(1, 0, 2)          # storage [L, Hkv, d]
    q_pad = torch.zeros(8, 16, 256, dtype=q.dtype, device="cuda")[:, :, :128]
    q_pad.copy_(q)
    a_idx, a_sc = il.ilre_recall(q, k, 128, (3, 7))
    b_idx, b_sc = il.ilre_recall(q_pad, k_tm, 128, (3, 7))
    torch.cuda.synchronize()
    assert torch.equal(a_idx, b_idx) and torch.equal(a_sc, b_sc)


def test_bitwise_reproducible():
    _announce("run-to-run determinism")
    inp = inputs.custom(L=20000, Lq=64, Hq=8, Hkv=2, d=128, dtype="bf16", n_spans=4, span_len=(16, 64), seed=6)
    q, k = to_device(inp.q), to_device(inp.k)
    first = il.ilre_recall(q, k, 1024, (1, 3, 7, 15, 31))
    for _ in range(3):
        again = il.ilre_recall(q, k, 1024, (1, 3, 7, 15, 31))
        torch.cuda.synchronize()
        assert torch.equal(first[0], again[0]) and torch.equal(first[1], again[1])


def test_column_scores_do_not_depend_on_how_the_tokens_are_cut():
    """Long contexts: the second scoring pass sizes each workgroup's token range by how fast its XCD ran the first
    pass (a table the first pass leaves in the workspace).  The scores must be the same bits with that table, without
    it (a workspace nothing was left in), with a workspace full of noise, and inside the whole path."""
    _announce("second pass: token ranges from the XCDs' speed vs even ranges")
    L, Lq, Hq, Hkv = 1100000, 64, 8, 2   # 253 token ranges of 68 tiles (64 tokens each) per kv head
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    q = torch.randn(Hq, Lq, 128, device="cuda", generator=g).to(torch.bfloat16)
    k = torch.randn(Hkv, L, 128, device="cuda", generator=g).to(torch.bfloat16)
    nbytes = il.ilre_workspace_bytes(L, Lq, Hq, Hkv, 128, 5, il.ILRE_BF16)
    ws = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    rmax, rsum = il.ilre_row_stats(q, k, workspace=ws)
    with_table = il.ilre_col_scores(q, k, rmax, rsum, workspace=ws).clone()
    clean = torch.zeros(nbytes, dtype=torch.uint8, device="cuda")
    without = il.ilre_col_scores(q, k, rmax, rsum, workspace=clean).clone()
    noise = torch.randint(0, 256, (nbytes,), dtype=torch.uint8, device="cuda", generator=g)
    noisy = il.ilre_col_scores(q, k, rmax, rsum, workspace=noise).clone()
    idx, whole = il.ilre_recall(q, k, 2048, (1, 3, 7, 15, 31), workspace=ws)
    # a stand-alone selection uses the workspace from its base and may write over what the first pass left there
    il.ilre_row_stats(q, k, workspace=ws)
    il.ilre_select(whole, 2048, (1, 3, 7, 15, 31), workspace=ws)
    after_select = il.ilre_col_scores(q, k, rmax, rsum, workspace=ws).clone()
    torch.cuda.synchronize()
    assert torch.equal(with_table, without)
    assert torch.equal(with_table, noisy)
    assert torch.equal(with_table, whole)
    assert torch.equal(with_table, after_select)
    total = float(with_table.double().sum())
    assert abs(total - Hq * Lq) < 1e-3 * Hq * Lq  # every softmax row sums to one (Section 3.2, Eq. 4)


def test_custom_scale():
    _announce("custom softmax scale")
    inp = inputs.custom(L=1500, Lq=8, Hq=4, Hkv=2, d=128, dtype="bf16", seed=8)
    q, k = to_device(inp.q), to_device(inp.k)
    want, _, _ = oracle.scores(inp.q, inp.k, scale=0.05)
    _, got = il.ilre_recall(q, k, 64, (3,), scale=0.05)
    torch.cuda.synchronize()
    bad, worst = score_errors(got.cpu().numpy(), want)
    assert bad == 0, worst


@pytest.mark.parametrize("dtype,Lq", [("f32", 16), ("bf16", 64), ("bf16", 256)])
def test_extreme_logits_take_the_safe_row_statistics_path(dtype, Lq):
    """A key far above everything else, in contexts of one tile a split, which follow the running maximum throughout (splits that freeze
    their references have a test of their own)."""
    _announce(f"extreme logits {dtype} Lq={Lq}")
    L, Hq, Hkv = 6000, 4, 2
    inp = inputs.custom(L=L, Lq=Lq, Hq=Hq, Hkv=Hkv, d=128, dtype=dtype, seed=31)
    qf = inputs.as_float(inp.q).copy()
    kf = inputs.as_float(inp.k).copy()
    kf[0, 4500, :] = 12.0 * qf[0, 0, :]          # logit of row (0,0) ~ 12*128/sqrt(128) = 136 nats = 196 base-2 units
    kf[1, 5100, :] = -14.0 * qf[3, 1, :]
    if dtype == "bf16":
        q_in, k_in = inputs.f32_to_bf16_bits(qf), inputs.f32_to_bf16_bits(kf)
    else:
        q_in, k_in = qf, kf
    want_score, want_max, want_sum = oracle.scores(q_in, k_in)
    assert want_max.max() > 100.0
    q, k = to_device(q_in), to_device(k_in)
    row_max, row_sumexp = il.ilre_row_stats(q, k)
    scores = il.ilre_col_scores(q, k, row_max, row_sumexp)
    torch.cuda.synchronize()
    gm, gz = row_max.cpu().numpy().astype(np.float64), row_sumexp.cpu().numpy().astype(np.float64)
    assert np.isfinite(gm).all() and np.isfinite(gz).all()
    np.testing.assert_allclose(gm + np.log(gz), want_max + np.log(want_sum), rtol=2e-5, atol=2e-4)
    bad, worst = score_errors(scores.cpu().numpy(), want_score)
    assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"


@pytest.mark.parametrize("Lq,tile,tiles", [(40, 64, 4), (256, 64, 4), (330, 64, 8), (512, 128, 4)],
                         ids=["128_rows_idle_waves", "256_rows", "256_and_128_rows_idle_wave", "512_rows"])
def test_a_split_is_walked_again_where_a_frozen_reference_does_not_hold(Lq, tile, tiles):
    """The first pass freezes every row's reference after two tiles of a split.  64 kv heads leave 8 splits of 4 tiles (blocks of 256 and
    128 rows: 4 of 8, blocks of 512: 4 of 4); the large key lies in the fourth tile of the second split, of every other head against the
    first row and of the others against the last.  22 nats: the reference stays below the maximum, which shows that the tile is one
    of the frozen ones.  79 nats (a finite sum beyond the limit) and 158 nats (an infinite one): the split is walked again and the reference is
    the maximum itself.  Tolerances as everywhere."""
    H, L = 64, 2045
    rng = np.random.default_rng(Lq)
    qf = rng.standard_normal((H, Lq, 128), dtype=np.float32)
    base = rng.standard_normal((H, L, 128), dtype=np.float32)
    at = (tiles + 3) * tile + 10
    row = np.where(np.arange(H) % 2 == 0, 0, Lq - 1)
    qf[np.arange(H), row] *= (np.sqrt(128.0) / np.linalg.norm(qf[np.arange(H), row], axis=1))[:, None].astype(np.float32)
    loud = np.arange(H) * Lq + row  # of the statistics, head by head
    for factor in (2.0, 7.0, 14.0):
        _announce(f"frozen references Lq={Lq} factor={factor}")
        kf = base.copy()
        kf[:, at] = factor * qf[np.arange(H), row]
        q_in, k_in = inputs.f32_to_bf16_bits(qf), inputs.f32_to_bf16_bits(kf)
        want_score, want_max, want_sum = oracle.scores(q_in, k_in)
        q, k = to_device(q_in), to_device(k_in)
        row_max, row_sumexp = il.ilre_row_stats(q, k)
        staged = il.ilre_col_scores(q, k, row_max, row_sumexp)
        _, whole = il.ilre_recall(q, k, 64, (3, 7))
        torch.cuda.synchronize()
        gm, gz = row_max.cpu().numpy().astype(np.float64).ravel(), row_sumexp.cpu().numpy().astype(np.float64).ravel()
        want_max, want_sum = np.asarray(want_max).ravel(), np.asarray(want_sum).ravel()
        assert np.isfinite(gm).all() and np.isfinite(gz).all()
        np.testing.assert_allclose(gm + np.log(gz), want_max + np.log(want_sum), rtol=2e-5, atol=2e-4)
        if factor == 2.0:
            assert (gm[loud] < want_max[loud] - 5).all()
        else:
            np.testing.assert_allclose(gm[loud], want_max[loud], rtol=2e-5)
        for got in (staged, whole):
            bad, worst = score_errors(got.cpu().numpy(), want_score)
            assert bad == 0, f"{bad} scores out of tolerance, worst {worst:.2f}x"
        assert torch.equal(staged, whole)


def test_recall_replays_from_a_captured_graph():
    """The library neither allocates nor synchronises, so a whole recall step can be captured into a HIP
    graph; every replay, with eager work and synchronisations in between, gives the eager result."""
    _announce("graph capture and replay")
    inp = inputs.custom(L=30000, Lq=64, Hq=8, Hkv=2, d=128, dtype="bf16", n_spans=4, span_len=(16, 64), seed=12)
    q, k = to_device(inp.q), to_device(inp.k)
    kernels, budget, mk, ak = (1, 3, 7, 15, 31), 1024, (2, 4, 8), tuple(range(1, 17))
    ws = il.alloc_workspace(30000, 64, 8, 2, 128, len(kernels), il.ILRE_BF16)
    ws2 = il.alloc_workspace_max_avg(30000, 64, 8, 2, 128, 4, mk, len(ak), il.ILRE_BF16)
    eager_idx, eager_sc = il.ilre_recall(q, k, budget, kernels, workspace=ws)
    eager_pidx, eager_cnt, _ = il.ilre_recall_max_avg(q, k, budget, mk, ak, 4, workspace=ws2)
    torch.cuda.synchronize()
    eager_idx, eager_sc, eager_pidx = eager_idx.clone(), eager_sc.clone(), eager_pidx.clone()
    out_idx, out_sc = torch.empty_like(eager_idx), torch.empty_like(eager_sc)
    out_pidx, out_cnt, out_psc = torch.empty_like(eager_pidx), torch.empty_like(eager_cnt), torch.empty_like(eager_sc)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side):
        il.ilre_recall(q, k, budget, kernels, workspace=ws, out_idx=out_idx, out_scores=out_sc)       # warm-up on the capture stream
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            il.ilre_recall(q, k, budget, kernels, workspace=ws, out_idx=out_idx, out_scores=out_sc)
            il.ilre_recall_max_avg(q, k, budget, mk, ak, 4, workspace=ws2, out_idx=out_pidx, out_count=out_cnt,
                                   out_scores=out_psc)
    torch.cuda.current_stream().wait_stream(side)
    for rep in range(3):
        out_idx.fill_(-7)
        out_sc.zero_()
        out_pidx.fill_(-7)
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out_idx, eager_idx) and torch.equal(out_sc, eager_sc), f"replay {rep}"
        assert torch.equal(out_pidx, eager_pidx) and int(out_cnt.item()) == int(eager_cnt.item()), f"replay {rep}"
        # eager work between the replays
        again, _ = il.ilre_recall(q, k, budget, kernels, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(again, eager_idx)


@pytest.mark.parametrize("seed", range(6))
def test_select_randomised_against_oracle(seed):
    """Many small random problems per seed, both forms of Algorithm 1: sizes around the chunk, bin and list
    boundaries of the kernels, score distributions with and without ties, all bit-exact with the oracle."""
    _announce(f"randomised selection, seed {seed}")
    rng = np.random.default_rng(9000 + seed)
    kinds = ("random", "few_values", "two_values", "equal", "narrow", "needles")
    for case in range(40):
        L = int(rng.choice([1, 2, 63, 64, 65, 255, 256, 257, 511, 513, 1000, 2047, 2049, 4097, 9999, 20000]))
        L = max(1, L + int(rng.integers(-3, 4)))
        kind = kinds[int(rng.integers(len(kinds)))]
        s = _scores_for(kind, L, rng) if L > 400 or kind != "needles" else rng.random(L).astype(np.float32)
        budget = int(rng.choice([1, 2, 7, 64, 255, 1000, 4096, 8192]))
        if min(budget, L) > 8192:
            budget = 8192
        dev = torch.from_numpy(s).cuda()
        if case % 2 == 0:
            n = int(rng.integers(1, 7))
            kernels = tuple(int(2 * rng.integers(0, 40) + 1) for _ in range(n))
            sink = int(rng.integers(0, min(L, 6) + 1)) if case % 4 == 0 else 0
            want = oracle.allocate(s, kernels, budget, sink=sink)
            got = il.ilre_select(dev, budget, kernels, sink=sink)
            torch.cuda.synchronize()
            assert got.cpu().numpy().tolist() == want.tolist(), (seed, case, L, kind, budget, kernels, sink)
        else:
            mk = tuple(int(rng.integers(1, 20)) for _ in range(int(rng.integers(1, 4))))
            ak = tuple(int(rng.integers(1, 24)) for _ in range(int(rng.integers(1, 5))))
            sink = int(rng.integers(0, min(L, 6) + 1))
            want = oracle.allocate_max_avg(s, mk, ak, budget, sink=sink)
            got, count = il.ilre_select_max_avg(dev, budget, mk, ak, sink)
            torch.cuda.synchronize()
            n_got = int(count.item())
            got = got.cpu().numpy()
            assert got[:n_got].tolist() == want.tolist() and (got[n_got:] == -1).all(), (seed, case, L, kind, budget, mk, ak, sink)


# the walk's set of allocated tokens is a bitmap in LDS up to so many tokens and a table of 32-token words beyond
BITMAP_TOKENS = 136 * 256 * 32
WALK_CASES = [
    # L, sink, budget, window sizes (stride-1 form), max / average sizes (printed form)
    (BITMAP_TOKENS - 1, 0, 8192, (1, 63, 3), (1,), (1, 3)),      # the bitmap one token short of full; 8 rounds a list
    (BITMAP_TOKENS, 0, 4096, (1, 3, 7), (2, 5), (1, 2)),         # exactly full
    (BITMAP_TOKENS + 4, 4, 4096, (2047, 1), (32, 33), (1, 4)),   # the body exactly full; intervals and cells over many words
    (BITMAP_TOKENS + 1, 0, 8192, (1, 1, 31), (1, 64), (2, 1)),   # one token more: the table
    (1179648, 0, 4096, (1, 3, 7), (2, 5), (1, 2)),
    # the table with intervals of more and fewer than 512 tokens, shares that end inside them, many and few of them
    (1200001, 3, 8192, (2047, 513, 511, 35), (1024, 600), (1, 2)),
    (1200000, 0, 700, (2047, 65, 2047), (513, 512), (3,)),
    (1300000, 1, 8191, (2047,), (1000, 33, 1), (1,)),
    (1300033, 0, 4096, tuple(range(1, 1023, 64)), (64, 700), (1, 3)),
    (8192, 0, 8191, (65, 129, 1), (3, 7), (1, 2, 5)),            # nearly every token kept: shares end inside intervals
    (8224, 1, 1, (1,), (8,), (16,)),
]


@pytest.mark.parametrize("L,sink,budget,windows,mk,ak", WALK_CASES, ids=[f"L{c[0]}_B{c[2]}" for c in WALK_CASES])
def test_walk_over_bitmap_and_word_table(L, sink, budget, windows, mk, ak):
    """Both forms of the walk at the edges of its set representations, bit-exact with the oracle.  The last tokens are among
    the best ones, so that the bitmap's last chunk is read off."""
    _announce(f"walk L={L} sink={sink} budget={budget}")
    rng = np.random.default_rng(L + budget)
    s = _scores_for("needles", L, rng)
    s[-3:] = (9.0, 8.5, 9.5)
    if L >= 1300000:  # a background whose best tokens lie side by side: short intervals among long ones
        s[L // 2:L // 2 + 6000] = (20 + rng.random(6000)).astype(np.float32)
    dev = torch.from_numpy(s).cuda()
    got = il.ilre_select(dev, budget, windows, sink=sink)
    got_p, count = il.ilre_select_max_avg(dev, budget, mk, ak, sink)
    torch.cuda.synchronize()
    assert got.cpu().numpy().tolist() == oracle.allocate(s, windows, budget, sink=sink).tolist()
    n = int(count.item())
    got_p = got_p.cpu().numpy()
    assert got_p[:n].tolist() == oracle.allocate_max_avg(s, mk, ak, budget, sink=sink).tolist() and (got_p[n:] == -1).all()


def _crowd_between(L, rng):
    """A crowd in one of the ranking's bins, a few values so far above it that they stretch the bins, and the rest so far
    below it that it would lie beyond the last bin: keys that are not ranked have no bin."""
    s = (1e-6 * rng.random(L)).astype(np.float32)
    at = rng.permutation(L)[:820]
    s[at[:20]] = 1e6 * (1.0 + rng.random(20))
    s[at[20:]] = 1.0 + 1e-4 * rng.random(800)
    bits = np.sort(s.view(np.uint32))[::-1].astype(np.int64)  # positive floats rank as their bits do
    shift = max(0, int(bits[0] - bits[819]).bit_length() - 11)
    assert bits[20] - bits[819] < 1 << shift and bits[0] - bits[820] >> shift >= 2048
    return s


BRIEF_CASES = [
    # L, sink, budget, windows, kind: selections that one workgroup does (up to 16384 tokens, 2048 kept, windows of up to 65), at the edges
    # of what its threads take and of the rule
    (1, 0, 1, (1,), "random"), (2, 2, 1, (3,), "random"), (70, 0, 70, (65, 1), "random"), (1023, 1, 300, (3, 7, 15), "needles"), (1025, 0, 64, (65,), "equal"),
    (4096, 0, 2048, (31, 3, 1), "few_values"), (4097, 0, 1025, (7,), "needles"), (8192, 0, 2048, (65, 63, 1), "random"), (8193, 4, 2047, (3, 7, 15, 31), "narrow"),
    (16384, 0, 2048, (1, 3, 7, 15, 31), "needles"), (16384, 1, 2048, (65,), "two_values"), (16385, 0, 2048, (65,), "random"), (16380, 4, 2049, (3,), "random"),
    (9000, 0, 500, (67, 3), "random"), (5000, 0, 2000, (5, 5, 5), "equal"), (12000, 3, 900, (3, 33), "outliers"), (16000, 0, 1500, (1, 3), "denormal"),
    (6000, 2, 700, (9, 31), "signed"), (6000, 2, 2048, (9, 65), "half_zero"), (16384, 0, 2048, (3, 31), "one_far"), (7000, 0, 40, tuple(range(1, 65, 2)) * 2, "flat"),
    (9000, 0, 600, (3, 7), "crowd_between"), (3000, 1, 600, (1,), "crowd_between"),
]


@pytest.mark.parametrize("L,sink,budget,windows,kind", BRIEF_CASES, ids=[f"L{c[0]}_B{c[2]}_{c[4]}" for c in BRIEF_CASES])
def test_short_selections_in_one_launch(L, sink, budget, windows, kind):
    _announce(f"short selection L={L} sink={sink} budget={budget} {kind}")
    rng = np.random.default_rng(L + budget)
    if kind == "one_far":
        s = (1.0 + 0.01 * rng.random(L)).astype(np.float32)
        s[L // 3] = 1e30
    elif kind == "crowd_between":
        s = _crowd_between(L, rng)
    elif kind in ("random", "few_values", "two_values", "equal", "narrow", "needles"):
        s = _scores_for(kind, L, rng)
    else:
        s = _any_scores(kind, L, rng)
    got = il.ilre_select(torch.from_numpy(s).cuda(), budget, windows, sink=sink)
    torch.cuda.synchronize()
    assert got.cpu().numpy().tolist() == oracle.allocate(s, windows, budget, sink=sink).tolist()


@pytest.mark.parametrize("mode", [il.ILRE_SCORE_SUM, il.ILRE_SCORE_MAX], ids=["sum", "max"])
@pytest.mark.parametrize("L,Lq,Hq,Hkv,sink", [(5, 1, 2, 2, 0), (1000, 8, 8, 2, 3), (4096, 16, 32, 8, 0), (4097, 8, 32, 8, 1), (8192, 16, 16, 4, 0), (8193, 8, 8, 2, 0), (3000, 200, 64, 8, 2)])
def test_short_recalls_add_up_their_partial_scores(L, Lq, Hq, Hkv, sink, mode):
    """The whole path up to 8192 tokens: one workgroup adds up the partial score vectors (or, of many, a kernel before it): the
    same scores as from the staged call, and the oracle's indices for them."""
    _announce(f"short recall L={L} Lq={Lq} {Hq}/{Hkv} sink={sink}")
    inp = inputs.custom(L=L, Lq=Lq, Hq=Hq, Hkv=Hkv, d=128, dtype="bf16", n_spans=2 if L > 200 else 0, span_len=(8, 24), channel_scale=True, seed=L)
    q, k = to_device(inp.q), to_device(inp.k)
    budget = max(1, L // 5)
    idx, scores = il.ilre_recall(q, k, budget, (3, 7, 15), score_mode=mode, sink=sink)
    row_max, row_sum = il.ilre_row_stats(q, k)
    staged = il.ilre_col_scores(q, k, row_max, row_sum, score_mode=mode)
    torch.cuda.synchronize()
    scores = scores.cpu().numpy()
    np.testing.assert_allclose(scores, staged.cpu().numpy(), rtol=1e-6, atol=0)  # (the row offsets are merged elsewhere: an ulp of the exponent)
    assert idx.cpu().numpy().tolist() == oracle.allocate(scores, (3, 7, 15), budget, sink=sink).tolist()


SHORT_CASES = [
    # L, sink, budget, max sizes, average sizes, kind: combinations ranked by a workgroup each (up to 16384 cells, cells of up to 8 tokens,
    # windows of up to 64) or by one for each 4096 or 8192 cells, at the edges of what a thread, a workgroup and the rule take
    (4096, 0, 700, (1,), (1, 2, 3), "random"), (4097, 0, 700, (1,), (4, 5), "needles"), (8192, 0, 64, (1,), (16, 63, 64), "random"),
    (8193, 1, 64, (1, 2), (2, 64, 65), "random"), (16384, 0, 3000, (1,), (7,), "narrow"), (16385, 0, 3000, (1,), (7,), "narrow"),
    (16386, 1, 8192, (1,), (1,), "equal"), (13, 0, 5, (3, 5, 7), (1, 64), "random"), (4, 4, 3, (2,), (2,), "random"), (3, 0, 2, (8, 2), (3,), "random"),
    (8000, 0, 999, (1,), (3,), "needles"), (8000, 0, 1000, (1,), (3,), "needles"),       # the best of each four counted, all counted
    (9000, 0, 8192, (6, 7, 8), (1, 6), "few_values"), (9000, 0, 500, (9, 8), (1, 6), "random"), (12000, 3, 8191, (1,), (5, 9), "half_zero"),
    (16000, 0, 300, (2, 4), (1, 9), "signed"), (16000, 0, 4000, (1,), (2, 8), "outliers"), (9000, 0, 900, (2,), (1, 3), "denormal"),
    (3 * 4096, 0, 4096, (1,), (2,), "one_far"), (16380, 0, 8192, (1, 2), (8,), "one_far"),  # crowded bins
    (20000, 0, 500, (1,), (1, 16), "needles"), (20481, 0, 60, (1,), (64,), "logarithms"), (40000, 0, 100, (1,), (3,), "equal"),  # in parts
    (40000, 2, 1500, (1, 8), (4, 5), "two_values"), (40000, 0, 8192, (2,), (4,), "one_far"), (64 * 4096, 0, 64, (1,), (5,), "random"),
    (64 * 4096 + 1, 0, 64, (1,), (5,), "random"), (70000, 0, 4096, (2,), (1, 2, 3, 4), "narrow"), (300001, 0, 64, (2, 4, 8), (1, 2, 3, 4, 5, 6), "flat"),
    (100003, 0, 4000, (8,), (1, 2, 3, 17, 33), "needles"), (60000, 0, 2000, (3,), (15,), "mostly_equal"),
    (4000, 0, 600, (1,), (1,), "crowd_between"), (13000, 0, 600, (1,), (1, 2), "crowd_between"), (40000, 0, 600, (1,), (1,), "crowd_between"),
]


@pytest.mark.parametrize("L,sink,budget,mk,ak,kind", SHORT_CASES, ids=[f"L{c[0]}_B{c[2]}_{c[5]}" for c in SHORT_CASES])
def test_few_windows_are_ranked_by_a_workgroup(L, sink, budget, mk, ak, kind):
    _announce(f"few windows L={L} sink={sink} budget={budget} max={mk} avg={ak} {kind}")
    rng = np.random.default_rng(L + budget)
    if kind == "one_far":          # a range that leaves nearly everything in a few bins
        s = (1.0 + 0.01 * rng.random(L)).astype(np.float32)
        s[L // 3] = 1e30
    elif kind == "crowd_between":
        s = _crowd_between(L, rng)
    elif kind == "mostly_equal":   # parts that hand on all they have
        s = np.full(L, 0.5, dtype=np.float32)
        s[rng.integers(0, L, 300)] = 0.75
    elif kind in ("random", "few_values", "two_values", "equal", "narrow", "needles"):
        s = _scores_for(kind, L, rng)
    else:
        s = _any_scores(kind, L, rng)
    want = oracle.allocate_max_avg(s, mk, ak, budget, sink=sink)
    got, count = il.ilre_select_max_avg(torch.from_numpy(s).cuda(), budget, mk, ak, sink)
    torch.cuda.synchronize()
    n = int(count.item())
    got = got.cpu().numpy()
    assert got[:n].tolist() == want.tolist() and (got[n:] == -1).all()


ALL16 = tuple(range(1, 17))
RELAY_CASES = [
    # L, sink, budget, max sizes, average sizes, kind: combinations that take turns (shares of at most 96 cells, four of them or more)
    (9000, 4, 1000, (2, 4, 8), ALL16, "needles"), (9001, 0, 30, (2, 4, 8), ALL16, "random"),  # .. fewer tokens than combinations
    (40000, 0, 64 * 96, (1,), tuple(range(1, 65)), "needles"),    # 64 of them, lists of more cells than are fetched ahead (1024)
    (40001, 1, 64 * 96, (1,), (5,) * 64, "random"),               # .. all alike: every list's front is taken
    (40000, 0, 64 * 96 + 1, (1,), (5,) * 64, "random"),           # .. one token more: not by turns
    (40000, 2, 8192, (32, 8, 4, 2), ALL16, "equal"), (30000, 0, 5000, (16, 32), (3, 4), "narrow"),
    (700, 0, 700, (2, 4, 8), ALL16, "few_values"), (20, 3, 17, (32, 1, 16), (1, 2, 9), "random"),  # lists that run out, empty ones
    (9000, 0, 4 * 95 + 1, (1,), (1, 2, 3, 4), "random"), (9000, 0, 300, (8,), (1, 2, 3), "random"),
    (131072, 0, 4096, (2, 4, 8), ALL16, "random"), (131073, 0, 900, (2, 4, 8), ALL16, "random"),  # 16 chunks of the set, one more
    (262144, 0, 900, (2, 4, 8), ALL16, "random"), (262145, 0, 4096, (2, 4, 8), ALL16, "random"),  # 32, one more
    (1200000, 4, 4096, (2, 4, 8), ALL16, "needles"), (1200001, 0, 3000, (1,), (7,) * 33, "two_values"),  # the word table
]


@pytest.mark.parametrize("L,sink,budget,mk,ak,kind", RELAY_CASES, ids=[f"L{c[0]}_B{c[2]}_{c[5]}" for c in RELAY_CASES])
def test_walk_by_turns(L, sink, budget, mk, ak, kind):
    _announce(f"turns L={L} sink={sink} budget={budget} max={mk} avg={len(ak)} {kind}")
    s = _scores_for(kind, L, np.random.default_rng(L + budget))
    want = oracle.allocate_max_avg(s, mk, ak, budget, sink=sink)
    dev = torch.from_numpy(s).cuda()
    for _ in range(3):
        got, count = il.ilre_select_max_avg(dev, budget, mk, ak, sink)
        torch.cuda.synchronize()
        n = int(count.item())
        got = got.cpu().numpy()
        assert got[:n].tolist() == want.tolist() and (got[n:] == -1).all()


AVERAGE_CASES = [
    # L, budget, max sizes, average sizes, kind: chunks of 128 / 256 windows and their remainders, the straight-line code for
    # sizes 1..16 and the loop for others (over 16, repeated), shares that want little, much or all of the cells
    (256, 20, (2,), (1, 16), "random"), (258, 20, (2,), (2, 15), "random"), (2047, 40, (8,), (3, 16, 7), "needles"),
    (2056, 250, (8, 1), (1, 2), "random"), (4096, 60, (2, 16), (16,), "random"), (5000, 1200, (3,), (1, 5), "random"),
    (5000, 1240, (1,), (16, 1), "random"), (20000, 100, (2, 4), (17, 1), "needles"), (20000, 100, (2, 4), (5, 5, 3), "needles"),
    (70000, 300, (1,), (64, 1, 2), "needles"), (70000, 8000, (4, 2), tuple(range(1, 17)), "random"), (30000, 200, (2,), (1, 2, 3), "equal"),
    (30000, 200, (2,), (17, 18), "equal"), (9000, 100, (1, 2), (3, 7), "tiny"), (9000, 100, (1, 2), (3, 7, 16), "negative"),
    (9000, 100, (2, 3), (1, 6), "huge_range"),
    # .. of more windows, or larger ones, than a workgroup or a few rank on their own
    (16385, 8000, (1,), (1, 16), "random"), (16511, 8000, (1,), (2, 15), "needles"), (33000, 7000, (2, 1), (3, 16, 7), "random"),
    (20001, 8192, (1,), (16,), "few_values"), (4096, 60, (2, 16), (1, 7, 16), "random"), (9216, 300, (9,), (2, 16), "random"),
    (33001, 8000, (1,), (3, 7, 16), "negative"), (33001, 8192, (1, 2), (1, 6), "huge_range"), (33001, 8000, (1,), (3, 7), "tiny"),
    # .. max kernels with unequal numbers of workgroups: as many as have their place among the first ends, one more, the most, two groups
    # of average kernels, one cell and none
    (300000, 3000, tuple(range(1, 9)), (3, 5), "needles"), (300000, 3000, (9, 1, 64, 2, 33, 5, 1, 16, 128), (2, 16), "needles"),
    (70000, 2000, tuple(range(1, 65)), (3,), "random"), (200000, 4000, (1, 24, 2), tuple(range(1, 22)), "needles"),
    (1000, 100, (9, 1000, 1024, 2), (1, 3), "random"),
]


@pytest.mark.parametrize("L,budget,mk,ak,kind", AVERAGE_CASES, ids=[f"L{c[0]}_{c[4]}_{len(c[3])}x{c[3][0]}" for c in AVERAGE_CASES])
def test_averages_at_the_edges_of_their_chunks_and_bins(L, budget, mk, ak, kind):
    _announce(f"averages L={L} budget={budget} max={mk} avg={ak} {kind}")
    rng = np.random.default_rng(L + len(ak))
    if kind == "tiny":            # quotients whose remainders underflow, denormals among them
        s = (rng.random(L) * 2.0 ** -120).astype(np.float32)
        s[::7] = np.float32(2.0 ** -140)
    elif kind == "negative":
        s = (-1.0 - rng.random(L)).astype(np.float32)
    elif kind == "huge_range":    # far more than the bins span on either side
        s = np.exp2(rng.uniform(-100, 100, size=L)).astype(np.float32)
    else:
        s = _scores_for(kind, L, rng)
    want = oracle.allocate_max_avg(s, mk, ak, budget, sink=0)
    got, count = il.ilre_select_max_avg(torch.from_numpy(s).cuda(), budget, mk, ak, 0)
    torch.cuda.synchronize()
    n = int(count.item())
    got = got.cpu().numpy()
    assert got[:n].tolist() == want.tolist() and (got[n:] == -1).all()


@pytest.mark.parametrize("ak", [tuple(range(1, 10)), (5,), (2, 7, 16), tuple(range(1, 17))], ids=["1_to_9", "5_alone", "2_7_16", "1_to_16"])
@pytest.mark.parametrize("top", [3e37, 3.2e38, -3e37], ids=["9_cells_finite", "2_cells_infinite", "negative"])
def test_averages_of_scores_near_the_largest_float(top, ak):
    """Finite scores whose window sums pass the largest float: of sizes up to 16 a window sum is formed whether the size was
    asked for or not, and a sum of +inf must not count for one that was not.  Both ways of counting (a share of a small and
    of a large part of the cells), a span inside and one at the end of the body."""
    _announce(f"averages near the largest float: {top} {ak}")
    rng = np.random.default_rng(7)
    L = 9001
    s = rng.random(L).astype(np.float32)
    s[3000:3040] = np.float32(top) * (0.9 + 0.1 * rng.random(40)).astype(np.float32)
    s[-20:] = np.float32(top)
    for mk in ((2, 4), (1,), (3,)):
        for budget in (100, 5000):
            with np.errstate(over="ignore"):
                want = oracle.allocate_max_avg(s, mk, ak, budget, sink=1)
            got, count = il.ilre_select_max_avg(torch.from_numpy(s).cuda(), budget, mk, ak, 1)
            torch.cuda.synchronize()
            n = int(count.item())
            got = got.cpu().numpy()
            assert got[:n].tolist() == want.tolist() and (got[n:] == -1).all(), (mk, budget)


RANK_CASES = [
    # L, budget, copies of a value, kind: lists of one element up to the 4096 that the counting sort takes and one more, bins
    # of up to 256 equal elements (ranked inside the bin) and one more (the network), ranges of one value and of all
    (1, 1, 1, "random"), (64, 64, 1, "random"), (1025, 1025, 1, "random"), (4096, 4096, 1, "random"), (4097, 4097, 1, "random"),
    (4096, 4000, 127, "copies"), (4096, 4000, 128, "copies"), (4096, 4000, 129, "copies"), (4096, 4096, 4096, "copies"),
    (4096, 4000, 255, "copies"), (4096, 4096, 256, "copies"), (4096, 4000, 257, "copies"), (3000, 2900, 257, "copies"),
    (4000, 4000, 1, "two_ends"), (128, 128, 128, "copies"), (4096, 4096, 2, "signs"), (9000, 2000, 3, "signs"),
]


@pytest.mark.parametrize("L,budget,copies,kind", RANK_CASES, ids=[f"L{c[0]}_B{c[1]}_{c[2]}x_{c[3]}" for c in RANK_CASES])
def test_rank_order_of_a_combinations_list(L, budget, copies, kind):
    """One cell a token, no averaging: the list is ranked scores, bit-exact with the oracle.  A second combination takes
    what the first one's rank order left, so an exchange inside a list shows in what is allocated."""
    _announce(f"rank order L={L} budget={budget} copies={copies} {kind}")
    rng = np.random.default_rng(L + budget + copies)
    s = np.repeat((1 + rng.permutation((L + copies - 1) // copies)).astype(np.float32), copies)[:L]
    if kind == "two_ends":        # two bins hold everything
        s = np.where(rng.random(L) < 0.5, 1e30, 1e-30).astype(np.float32) * (1 + 0.01 * rng.random(L)).astype(np.float32)
    elif kind == "signs":
        s *= np.where(rng.random(L) < 0.5, -1, 1).astype(np.float32)
    elif kind == "random":
        s = rng.random(L).astype(np.float32)
    s = s[rng.permutation(L)]
    for mk, ak in (((1,), (1,)), ((1,), (1, 2, 3)), ((2, 1), (1, 3))):
        for b in sorted({budget, max(1, budget // 2), max(1, budget // 7)}):
            want = oracle.allocate_max_avg(s, mk, ak, b, sink=0)
            got, count = il.ilre_select_max_avg(torch.from_numpy(s).cuda(), b, mk, ak, 0)
            torch.cuda.synchronize()
            n = int(count.item())
            got = got.cpu().numpy()
            assert got[:n].tolist() == want.tolist() and (got[n:] == -1).all(), (mk, ak, b)


SEED_CASES = [
    # L, budget, sink, kind: where the K-th best lies among the histogram's bins -- inside the fine ones, in the coarse ones
    # on either side, all in one bin (the boundary list is then radix-selected), below everything that is counted
    (1, 1, 0, "random"), (255, 255, 0, "random"), (3000, 2999, 1, "random"), (9000, 8192, 0, "needles"), (20000, 60, 3, "negative"),
    (300001, 3000, 0, "sign_mixed"), (300001, 500, 0, "flat"), (262144, 4096, 0, "one_bin"), (262145, 2000, 2, "huge_range"),
    (262145, 8192, 0, "mostly_zero"), (4200001, 900, 1, "flat"), (4200001, 900, 0, "clustered"), (4200000, 64, 0, "negative"),
]


@pytest.mark.parametrize("L,budget,sink,kind", SEED_CASES, ids=[f"L{c[0]}_B{c[1]}_{c[3]}" for c in SEED_CASES])
def test_seeds_of_any_distribution(L, budget, sink, kind):
    _announce(f"seeds L={L} budget={budget} sink={sink} {kind}")
    rng = np.random.default_rng(L + budget)
    if kind == "negative":
        s = (-1.0 - rng.random(L)).astype(np.float32)
    elif kind == "sign_mixed":
        s = rng.standard_normal(L).astype(np.float32)
    elif kind == "flat":
        s = (1.0 + 1e-6 * rng.standard_normal(L)).astype(np.float32)
    elif kind == "one_bin":       # a sample never sees the two ends: the bulk, and the cut in it, are one coarse bin
        s = np.where(np.arange(L) % 1024 == 0, np.where(np.arange(L) % 2048 == 0, 1e30, 1e-30), 1.5 + 0.4 * rng.random(L)).astype(np.float32)
    elif kind == "huge_range":
        s = np.exp2(rng.uniform(-140, 120, size=L)).astype(np.float32) * np.where(rng.random(L) < 0.5, -1, 1).astype(np.float32)
    elif kind == "mostly_zero":
        s = np.where(rng.random(L) < 0.01, rng.random(L), 0.0).astype(np.float32)
    elif kind == "clustered":     # many seeds in few chunks: their maxima are far below the cut
        s = (0.01 + 0.001 * rng.random(L)).astype(np.float32)
        s[1000:9000] = 4 + 4 * rng.random(8000)
    else:
        s = _scores_for(kind, L, rng) if L > 300 else rng.random(L).astype(np.float32)
    got = il.ilre_select(torch.from_numpy(s).cuda(), budget, (1, 3, 7), sink=sink)
    torch.cuda.synchronize()
    assert got.cpu().numpy().tolist() == oracle.allocate(s, (1, 3, 7), budget, sink=sink).tolist()


@pytest.mark.parametrize("L,scale,qfactor,sink", [(70000, 0.0, 0.0, 0), (70000, 0.0, 1e-3, 1), (140001, 40.0, 1.0, 0), (9000, 40.0, 1.0, 2), (63, 0.0, 1.0, 0)],
                         ids=["all_equal", "flat", "spiky", "spiky_short", "one_wavefront"])
def test_recall_where_the_mean_says_little(L, scale, qfactor, sink):
    """In the whole path the bins follow the scores' mean: scores all equal to it, nearly so, and nearly all far below it
    (a few keys take everything); the selection is the oracle's on the GPU's own scores, and on the selection alone."""
    _announce(f"recall L={L} scale={scale} q*{qfactor}")
    inp = inputs.custom(L=L, Lq=16, Hq=8, Hkv=2, d=128, dtype="f32", n_spans=2 if L > 200 else 0, span_len=(8, 24), channel_scale=True, seed=5)
    q, k = to_device(inp.q) * qfactor, to_device(inp.k)
    budget = min(3000, L // 2)
    for mode in (il.ILRE_SCORE_SUM, il.ILRE_SCORE_MAX):
        idx, scores = il.ilre_recall(q, k, budget, (3, 7), score_mode=mode, sink=sink, scale=scale)
        alone = il.ilre_select(scores, budget, (3, 7), sink=sink)
        torch.cuda.synchronize()
        want = oracle.allocate(scores.cpu().numpy(), (3, 7), budget, sink=sink).tolist()
        assert idx.cpu().numpy().tolist() == want and alone.cpu().numpy().tolist() == want


def _device_us(call, rounds=5, reps=4):
    """Time of one call in a row of them, the best of a few rounds."""
    call()
    best = float("inf")
    for _ in range(rounds):
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        begin.record()
        for _ in range(reps):
            call()
        end.record()
        end.synchronize()
        best = min(best, begin.elapsed_time(end) * 1000 / reps)
    return best


def _raised(L, seed, every=0, first=0.0):
    """A dense background, every so many tokens three times as high, the first token on its own."""
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    s = torch.randn(L, device="cuda", generator=g).mul_(0.0024).add_(0.008).clamp_(min=1e-4)
    if every:
        s[::every] *= 3
    if first:
        s[0] = first
    return s


@pytest.mark.parametrize("L,budget,every,first", [(1 << 20, 4096, 1024, 0.0), (1 << 17, 4096, 1024, 0.0), (16 << 20, 256, 0, 1e20)],
                         ids=["chunk_starts_1M", "chunk_starts_128K", "sink_16M"])
def test_time_of_a_selection_does_not_follow_the_places_of_its_scores(L, budget, every, first):
    """The histogram's bins are placed by a sample.  High scores on a regular grid, or at the very front, are as quickly
    sorted out as the same scores in random places (when the sample fell in with the grid: 10 times as long on 1M tokens).
    Three times as long is far from what two runs differ by."""
    _announce(f"time of a selection, L={L} every {every} first {first}")
    s = _raised(L, 3, every, first)
    g = torch.Generator(device="cuda")
    g.manual_seed(4)
    mixed = s[torch.randperm(L, device="cuda", generator=g)].contiguous()
    ws = il.alloc_workspace(L, 1, 1, 1, 128, 3, il.ILRE_F32)
    out = il.ilre_select(s, budget, (1, 3, 7), workspace=ws)
    torch.cuda.synchronize()
    if L <= 1 << 20:
        assert out.cpu().numpy().tolist() == oracle.allocate(s.cpu().numpy(), (1, 3, 7), 4096).tolist()
    as_it_is = _device_us(lambda: il.ilre_select(s, budget, (1, 3, 7), workspace=ws))
    at_random = _device_us(lambda: il.ilre_select(mixed, budget, (1, 3, 7), workspace=ws))
    print(f"{as_it_is:.1f} us, in random places {at_random:.1f} us", flush=True)
    assert as_it_is < 3 * at_random + 10


@pytest.mark.parametrize("L,kind", [(1 << 17, "equal"), (1 << 17, "mostly_zero"), (100001, "two_values")])
def test_time_of_a_selection_among_equal_scores(L, kind):
    """Where more scores are equal than are wanted, one workgroup sorts them out by their places.  That takes about four
    times as long as scores that differ (a pass and an addition per key for each digit they share: 23 times)."""
    _announce(f"time of a selection among equal scores, L={L} {kind}")
    rng = np.random.default_rng(5)
    s = {"equal": np.full(L, 0.25), "mostly_zero": np.where(rng.random(L) < 0.01, rng.random(L), 0.0),
         "two_values": np.where(rng.random(L) < 0.02, 0.5, 0.25)}[kind].astype(np.float32)
    dev, ws = torch.from_numpy(s).cuda(), il.alloc_workspace(L, 1, 1, 1, 128, 3, il.ILRE_F32)
    got = il.ilre_select(dev, 4096, (1, 3, 7), workspace=ws)
    torch.cuda.synchronize()
    assert got.cpu().numpy().tolist() == oracle.allocate(s, (1, 3, 7), 4096).tolist()
    other = torch.from_numpy(rng.random(L).astype(np.float32)).cuda()
    equal = _device_us(lambda: il.ilre_select(dev, 4096, (1, 3, 7), workspace=ws))
    differ = _device_us(lambda: il.ilre_select(other, 4096, (1, 3, 7), workspace=ws))
    print(f"{equal:.1f} us, scores that differ {differ:.1f} us", flush=True)
    assert equal < 10 * differ


@pytest.mark.parametrize("mode,factor", [(il.ILRE_SCORE_SUM, 0.05), (il.ILRE_SCORE_MAX, 5e-4)], ids=["sum", "max"])
def test_time_of_a_recall_of_a_flat_attention(mode, factor):
    """Query states that hardly tell the keys apart: scores that differ by a thousandth and less, within a hundredth of their mean.
    The bins there are fine enough to find the cut, where one bin held most of the scores before, and the indices are the
    oracle's on the GPU's own scores."""
    _announce(f"time of a recall of a flat attention, mode {mode}")
    L, Lq, Hq, Hkv = 131072, 64, 32, 8
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    q = torch.randn(Hq, Lq, 128, device="cuda", generator=g)
    k = torch.randn(Hkv, L, 128, device="cuda", generator=g).bfloat16()
    flat, other = (factor * q).bfloat16(), q.bfloat16()
    ws = il.alloc_workspace(L, Lq, Hq, Hkv, 128, 3, il.ILRE_BF16)
    idx, scores = il.ilre_recall(flat, k, 4096, (1, 3, 7), score_mode=mode, sink=4, workspace=ws)
    torch.cuda.synchronize()
    spread = float(scores.std() / scores.mean())
    assert 5e-5 < spread < 3e-3 and abs(float(scores.mean()) * L / (Hq * Lq if mode == il.ILRE_SCORE_SUM else 1) - 1) < 0.015
    assert idx.cpu().numpy().tolist() == oracle.allocate(scores.cpu().numpy(), (1, 3, 7), 4096, sink=4).tolist()
    t_flat = _device_us(lambda: il.ilre_recall(flat, k, 4096, (1, 3, 7), score_mode=mode, sink=4, workspace=ws))
    t_other = _device_us(lambda: il.ilre_recall(other, k, 4096, (1, 3, 7), score_mode=mode, sink=4, workspace=ws))
    print(f"{t_flat:.1f} us, other states {t_other:.1f} us", flush=True)
    assert t_flat < 1.35 * t_other


def _any_scores(kind, L, rng):
    if kind == "signed":
        return rng.standard_normal(L).astype(np.float32)
    if kind == "logarithms":
        return np.log(0.008 * (1 + 0.3 * rng.standard_normal(L)).clip(0.01)).astype(np.float32)
    if kind == "half_zero":
        return np.where(rng.random(L) < 0.5, rng.random(L), 0.0).astype(np.float32)
    if kind == "flat":
        return (0.008 * (1 + 1e-3 * rng.standard_normal(L))).astype(np.float32)
    if kind == "outliers":        # a few dozen of either sign, the sums in between within a thousandth
        s = (1 + 1e-3 * rng.random(L)).astype(np.float32)
        s[rng.integers(0, L, 30)] = 1e30
        s[rng.integers(0, L, 30)] = -1e30
        return s
    if kind == "denormal":
        return (rng.integers(-3, 4, size=L) * 2.0 ** -149).astype(np.float32)
    if kind == "chunk_starts":
        s = (0.008 * (1 + 0.3 * rng.standard_normal(L))).clip(1e-4).astype(np.float32)
        s[::1024] *= 3
        return s
    return (0.008 * (1 + 0.3 * rng.standard_normal(L))).clip(1e-4).astype(np.float32)


@pytest.mark.parametrize("kind", ["signed", "logarithms", "half_zero", "flat", "outliers", "denormal"])
def test_averages_of_any_sign_and_scale(kind):
    """The bins of the averages start at a sampled sum of any sign: both ways of counting, a body of few cells (all of the
    sample is one of them) and of many, the straight-line sizes and others; bit-exact with the oracle."""
    for L, budget, mk, ak in ((60, 20, (4, 64), (1, 3)), (9001, 100, (2, 8), tuple(range(1, 17))), (9001, 6000, (1, 3), (2, 16)),
                              (70001, 2000, (2,), (5, 17, 33)), (262144, 4096, (2, 4, 8), (1, 2, 7, 16))):
        _announce(f"averages of any sign and scale: {kind} L={L} budget={budget} max={mk} avg={ak}")
        s = _any_scores(kind, L, np.random.default_rng(L + budget))
        want = oracle.allocate_max_avg(s, mk, ak, budget, sink=1)
        got, count = il.ilre_select_max_avg(torch.from_numpy(s).cuda(), budget, mk, ak, 1)
        torch.cuda.synchronize()
        n = int(count.item())
        got = got.cpu().numpy()
        assert got[:n].tolist() == want.tolist() and (got[n:] == -1).all(), (L, budget, mk, ak)


@pytest.mark.parametrize("kind,sink", [("chunk_starts", 0), ("flat", 4), ("logarithms", 4), ("half_zero", 0), ("half_zero", 4)])
def test_time_of_a_printed_selection_does_not_follow_its_scores(kind, sink):
    """A sample of each combination's own sums places its bins: scores that are raised on a grid, hardly differ, are negative
    or half of them zero take about as long as others (two to eleven times with bins of one width upward from the
    scores' median)."""
    _announce(f"time of a printed selection: {kind} sink {sink}")
    L, mk, ak = 1 << 20, (2, 4, 8), tuple(range(1, 17))
    rng = np.random.default_rng(2)
    ws = il.alloc_workspace_max_avg(L, 1, 1, 1, 128, sink, mk, len(ak), il.ILRE_F32)
    us = []
    for k in (kind, "dense"):
        dev = torch.from_numpy(_any_scores(k, L, rng)).cuda()
        us.append(_device_us(lambda: il.ilre_select_max_avg(dev, 4096, mk, ak, sink, workspace=ws)))
    print(f"{us[0]:.1f} us, other scores {us[1]:.1f} us", flush=True)
    assert us[0] < 1.7 * us[1]


@pytest.mark.parametrize("n_nan", [1, 500, 5000])
def test_scores_that_are_not_numbers_leave_a_valid_index_list(n_nan):
    """Scores are finite by contract.  What a NaN among them does to the ranking is open, but the indices stay valid ones:
    ascending, unique, as many as asked for."""
    _announce(f"{n_nan} scores of NaN")
    rng = np.random.default_rng(n_nan)
    s = rng.random(9000).astype(np.float32)
    s[rng.permutation(9000)[:n_nan]] = np.nan
    dev = torch.from_numpy(s).cuda()
    for mk, ak, budget in (((1,), (1,), 8000), ((2, 4), (1, 2, 3), 600), ((1, 2), (5, 17), 6000)):
        got, count = il.ilre_select_max_avg(dev, budget, mk, ak, 0)
        torch.cuda.synchronize()
        n = int(count.item())
        got = got.cpu().numpy()
        assert 0 < n <= budget and (np.diff(got[:n]) > 0).all() and got[0] >= 0 and got[n - 1] < 9000 and (got[n:] == -1).all()
    got = il.ilre_select(dev, 600, (3, 7)).cpu().numpy()
    assert (np.diff(got) > 0).all() and got[0] >= 0 and got[-1] < 9000


@pytest.mark.parametrize("L,mk", [(9000, (9, 15)), (9001, (3,)), (9001, (3, 5, 7)), (9002, (6, 2)), (9001, (16, 17, 1)), (40000, (63, 64)), (70001, (65, 2)), (70000, (1024, 1023)), (1000, (1024, 8)), (1025, (1024,))],
                         ids=lambda x: str(x).replace(" ", ""))
def test_large_cells_and_long_windows(L, mk):
    """Cells of other than 1, 2, 4 and 8 tokens (3 with windows of up to 16), or windows of more than 64 cells, are pooled by a
    kernel of their own: sizes around its 1, 4, 16 and 64 lanes a cell, bodies that end inside a cell or are shorter than one, windows around the eight cells that are
    read together; bit-exact with the oracle."""
    for ak in ((1, 16), (7, 8, 9), (64, 65), (1024, 3), (5, 5, 1000)):
        for budget in (50, min(3000, L - 1)):
            _announce(f"large cells and long windows L={L} max={mk} avg={ak} budget={budget}")
            s = _any_scores("signed" if ak[0] == 7 else "dense", L, np.random.default_rng(L + budget))
            want = oracle.allocate_max_avg(s, mk, ak, budget, sink=1)
            got, count = il.ilre_select_max_avg(torch.from_numpy(s).cuda(), budget, mk, ak, 1)
            torch.cuda.synchronize()
            n = int(count.item())
            got = got.cpu().numpy()
            assert got[:n].tolist() == want.tolist() and (got[n:] == -1).all(), (ak, budget)


@pytest.mark.parametrize("mk,ak,most", [((64,), tuple(range(1, 17)), 2.5), ((1024,), (5,), 2.5), ((2,), (1024,), 5.0), ((1024,), (1024,), 5.0)],
                         ids=["cells_of_64", "cells_of_1024", "windows_of_1024", "both"])
def test_time_of_a_printed_selection_with_large_sizes(mk, ak, most):
    """Against cells of 8 tokens and windows of up to 16 of them.  (A lane that reads a cell's tokens one after the other,
    each cell for every window that reaches over it, and adds a window's cells one by one: 7 to 50 times as long.)"""
    _announce(f"time of a printed selection: max {mk} avg {ak}")
    L = 1 << 20
    dev = torch.from_numpy(_any_scores("dense", L, np.random.default_rng(2))).cuda()
    us = []
    for m, a in ((mk, ak), ((8,), tuple(range(1, 17)))):
        ws = il.alloc_workspace_max_avg(L, 1, 1, 1, 128, 0, m, len(a), il.ILRE_F32)
        us.append(_device_us(lambda: il.ilre_select_max_avg(dev, 4096, m, a, 0, workspace=ws)))
    print(f"{us[0]:.1f} us, ordinary sizes {us[1]:.1f} us", flush=True)
    assert us[0] < most * us[1]


def test_time_of_long_contexts_with_few_or_huge_takings():
    """3M tokens, where the walk's set is the table.  Windows of 2047 tokens take about twice as long as small ones (six times
    when a lane marked an interval by itself), the best 64 of the printed form about as long as those of the window form
    (twice when every chunk of windows reserved its places)."""
    _announce("time of long contexts with few or huge takings")
    L = 3 << 20
    dev = torch.from_numpy(_scores_for("needles", L, np.random.default_rng(9))).cuda()
    ws = il.alloc_workspace(L, 1, 1, 1, 128, 1, il.ILRE_F32)
    ws_p = il.alloc_workspace_max_avg(L, 1, 1, 1, 128, 0, (1,), 1, il.ILRE_F32)
    huge = _device_us(lambda: il.ilre_select(dev, 4096, (2047,), workspace=ws))
    small = _device_us(lambda: il.ilre_select(dev, 4096, (31,), workspace=ws))
    few = _device_us(lambda: il.ilre_select_max_avg(dev, 64, (1,), (7,), 0, workspace=ws_p))
    few_window = _device_us(lambda: il.ilre_select(dev, 64, (7,), workspace=ws))
    print(f"{huge:.1f} us, small windows {small:.1f} us; {few:.1f} us, window form {few_window:.1f} us", flush=True)
    assert huge < 3.5 * small and few < 1.75 * few_window
