"""GPU parity of marl_prefill_attn and marl_kv_write_prompt against the float64 reference,
through the C ABI.

Tolerance.  The kernel rounds the softmax weights to bf16 before the value product (unit
roundoff 2^-8: bf16 keeps 8 significant bits) and, for bf16 output, rounds the result once more
(another 2^-8, relative).  Unlike a decode query over hundreds of tokens, an early prompt row
averages only a few values, so its output is O(max |V|) and the errors do not average out: the
bound is the worst case, stated relative to the softmax-weighted mean of |V| of the row, which
the reference computes:
    |delta| <= 1e-3 + 2^-8 * sum_j p_j |V_j|      (2^-7 for bf16 output).
Rows over many tokens stay far inside it (their errors average out as in the decode tests)."""
import numpy as np
import pytest
import torch

from oracle import reference as R
from paper_2602_09578_amd import binding as B
from paper_2602_09578_amd import inputs as I

pytestmark = pytest.mark.gpu


def reference(inp):
    qb, kb, vb = I.bf16_bits(inp.q), I.bf16_bits(inp.k_pages), I.bf16_bits(inp.v_pages)
    args = (inp.prefix_block_table.cpu().numpy(), inp.q_start.cpu().numpy(), inp.q_pos0.cpu().numpy(),
            inp.scale, inp.Hq, inp.Hkv)
    return R.prefill_attn(qb, kb, vb, *args), R.prefill_attn(qb, kb, vb & 0x7fff, *args)


def run_gpu(inp_cpu, out_dtype, expect_flags=0):
    dev = inp_cpu.to("cuda")
    shape, ws, out = B.prepare_prefill(dev, out_dtype)
    out.fill_(float("nan"))
    B.run_prefill(dev, shape, ws, out)
    torch.cuda.synchronize()
    assert B.marl_attn_read_flags(ws) == expect_flags
    return out.float().cpu().numpy().astype(np.float64)


def check(inp_cpu, out_dtype=B.MARL_OUT_F32):
    want, want_abs = reference(inp_cpu)
    got = run_gpu(inp_cpu, out_dtype)
    covered = np.isfinite(want)
    assert np.isfinite(got[covered]).all()
    assert np.isnan(got[~covered]).all()          # rows no group covers are left alone
    rel = 2.0 ** -8 if out_dtype == B.MARL_OUT_F32 else 2.0 ** -7
    excess = np.abs(got - want)[covered] - (1e-3 + rel * want_abs[covered])
    assert excess.size == 0 or excess.max() <= 0, f"worst excess over the bound {excess.max()}"


@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (28, 4), (64, 8), (4, 4), (16, 1)])
@pytest.mark.parametrize("out_dtype", [B.MARL_OUT_F32, B.MARL_OUT_BF16])
def test_ragged_prompts_match_reference(Hq, Hkv, out_dtype):
    lens = [1, 5, 16, 17, 33, 100, 0, 257]
    check(I.build_prefill_inputs(Hq, Hkv, lens, [0] * len(lens), seed=Hq + Hkv), out_dtype)


@pytest.mark.parametrize("seed", range(12))
def test_random_shapes(seed):
    """Seeded random head counts, prompt lengths (zeros, page and row-block boundaries, a few
    hundred tokens) and context lengths in front of the chunk."""
    rng = np.random.default_rng(500 + seed)
    Hkv = int(rng.choice([1, 2, 4, 8]))
    Rq = int(rng.choice([1, 2, 4, 7, 8, 16]))
    n = int(rng.integers(1, 7))
    edge = np.array([0, 1, 15, 16, 17, 47, 48, 49, 191, 192, 193])
    lens = np.where(rng.random(n) < 0.4, rng.choice(edge, n), rng.integers(1, 420, n))
    pos0 = np.where(rng.random(n) < 0.5, 0, rng.integers(0, 300, n))
    print("case: prefill random shape", seed, Hkv * Rq, Hkv, lens.tolist(), pos0.tolist(), flush=True)
    out_dtype = B.MARL_OUT_F32 if seed % 2 == 0 else B.MARL_OUT_BF16
    check(I.build_prefill_inputs(Hkv * Rq, Hkv, lens.tolist(), pos0.tolist(), seed=seed), out_dtype)


def test_chunked_prefill_with_context():
    # chunks that start in the middle of a page, at a page boundary and deep into the prompt
    check(I.build_prefill_inputs(28, 4, [40, 7, 64, 1, 130], [5, 16, 96, 300, 257], seed=3))
    check(I.build_prefill_inputs(8, 2, [40, 7, 64, 1, 130], [5, 16, 96, 300, 257], seed=4), B.MARL_OUT_BF16)


@pytest.mark.parametrize("scale", [1.0, -0.7, 0.0])
def test_peaked_flat_and_sign_flipped_scores(scale):
    # scale 1 makes the scores ~N(0, 128): nearly one-hot rows whose running maximum keeps moving
    # (the accumulator rescale runs in most steps); a negative scale flips every score; scale 0
    # gives uniform weights (running means of the values)
    from dataclasses import replace
    inp = I.build_prefill_inputs(28, 4, [300, 77, 513], [0, 64, 5], seed=21)
    check(replace(inp, scale=scale))
    check(replace(inp, scale=scale), B.MARL_OUT_BF16)


@pytest.mark.parametrize("first,later", [(-3.0, -3.0), (-3.0, 3.0), (3.0, -3.0), (-0.8, -0.8)])
@pytest.mark.parametrize("chunks,context", [([3, 20, 200], [0, 31, 0]), ([40, 1], [300, 64])])
def test_scores_far_from_the_first_reference(first, later, chunks, context):
    """Keys that put every score at about -200 or -50 in base 2, or the first page at -200 and the others at +200, and the
    other way round; items that begin with a whole step and items that begin on the causal edge."""
    print("case: prefill scores far from 0", first, later, chunks, context, flush=True)
    inp = I.build_prefill_inputs(28, 4, chunks, context, seed=31)
    inp.q += 4
    inp.k_pages += later
    inp.k_pages[inp.prefix_block_table[:, 0].long()] += first - later
    check(inp)
    check(inp, B.MARL_OUT_BF16)


@pytest.mark.parametrize("share", [0.5, 0.8])
@pytest.mark.parametrize("Hq,Hkv,chunks,context", [(28, 4, [200, 330], [0, 300]), (4, 4, [700], [0]), (16, 1, [40], [900])])
def test_a_key_that_holds_much_of_a_row_costs_no_rounding(share, Hq, Hkv, chunks, context):
    """An attention sink: about `share` of every row's mass sits on the prompt's first key.  As the reference maximum its weight
    is exactly 1 in bf16; the other n keys hold 1 - share between them, their weights each rounded by at most 2^-8 of
    itself (2^-8 / sqrt(3) in the root mean square): together (1 - share) / sqrt(n) of that, times sqrt(e) for the spread of
    their weights, whose scores are N(0, 1).  Relative to a row that is share of one value, over rows of at least n = 64 keys:
    2^-8 / sqrt(3) * (1 - share) / share * sqrt(e / 64) = 4.6e-4 for half; a rounded weight of the sink itself would add about
    1.2e-3 whatever n is.  Scores lie about 1 for the sink, where neither their size nor their sign makes the rows move."""
    print("case: prefill sink", share, Hq, Hkv, chunks, context, flush=True)
    inp = I.build_prefill_inputs(Hq, Hkv, chunks, context, seed=17)
    inp.q.mul_(0.25).add_(1.0)                                  # |q|^2 = 136: scores against N(0, 1) keys are N(0, 1.06)
    sums = inp.q.float().sum(-1).mean().item() * inp.scale      # of a key of ones
    keys = np.array(chunks) + np.array(context) / 2
    for g, pages in enumerate(inp.prefix_block_table):
        used = pages[pages >= 0].long()
        inp.k_pages[used] += float((0.5 - np.log(keys[g] * share / (1 - share))) / sums)
        inp.k_pages[int(pages[0]), :, 0, :] = 1.0 / sums
    want, _ = reference(inp)
    got = run_gpu(inp, B.MARL_OUT_F32)
    pos = np.concatenate([np.arange(n) + p0 for n, p0 in zip(chunks, context)])
    rows = pos >= 64
    rel = np.sqrt(((got - want)[rows] ** 2).sum() / (want[rows] ** 2).sum())
    print("relative error", rel, flush=True)
    assert rel <= 2.0 ** -8 / 3 ** 0.5 * (1 - share) / share * np.sqrt(np.e / 64)


def test_many_small_groups_and_more_than_one_plan_round():
    rng = np.random.default_rng(0)
    lens = rng.integers(0, 12, size=1500).tolist()      # plan scans 1024 groups per round
    pos0 = rng.integers(0, 20, size=1500).tolist()
    check(I.build_prefill_inputs(8, 2, lens, pos0, seed=5))


def test_long_prompt_sampled_rows_against_the_decode_checker():
    # 3 prompts of 2048 / 1500 / 700 tokens, Qwen-7B head layout; the reference prefill would need
    # minutes, so sampled rows are checked one by one with the C decode checker
    inp = I.build_prefill_inputs(28, 4, [2048, 1500, 700], [0, 0, 512], seed=6)
    got = run_gpu(inp, B.MARL_OUT_F32)
    assert np.isfinite(got).all()
    qs, p0 = inp.q_start.numpy(), inp.q_pos0.numpy()
    rng = np.random.default_rng(1)
    picks = [(0, 0), (0, 2047), (0, 31), (0, 32), (1, 1499), (2, 0), (2, 699)] + \
            [(int(g), int(rng.integers(0, qs[g + 1] - qs[g]))) for g in rng.integers(0, 3, size=25)]
    rows = np.array([qs[g] + tau for g, tau in picks])
    gid = np.array([g for g, _ in picks])
    plens = np.array([p0[g] + tau + 1 for g, tau in picks], dtype=np.int32)
    n = len(picks)
    qb, kb, vb = I.bf16_bits(inp.q)[rows], I.bf16_bits(inp.k_pages), I.bf16_bits(inp.v_pages)
    common = (inp.prefix_block_table.numpy()[gid], np.zeros((n, 1), dtype=np.int32), plens,
              np.zeros(n, dtype=np.int32), np.arange(n, dtype=np.int32), inp.scale, 28, 4)
    want = R.decode_attn(qb, kb, vb, *common)
    want_abs = R.decode_attn(qb, kb, vb & 0x7fff, *common)
    excess = np.abs(got[rows] - want) - (1e-3 + 2.0 ** -8 * want_abs)
    assert excess.max() <= 0, f"worst excess over the bound {excess.max()}"


def test_reruns_are_bit_identical_and_page_placement_does_not_matter():
    a = I.build_prefill_inputs(28, 4, [300, 77], [0, 40], seed=7)
    out1, out2 = run_gpu(a, B.MARL_OUT_F32), run_gpu(a, B.MARL_OUT_F32)
    np.testing.assert_array_equal(out1, out2)
    # same logical contents on other physical pages
    perm = np.random.default_rng(2).permutation(a.num_pages)
    inv = np.argsort(perm)
    tab = a.prefix_block_table.numpy().copy()
    tab[tab >= 0] = perm[tab[tab >= 0]]
    from dataclasses import replace
    b = replace(a, k_pages=a.k_pages[torch.from_numpy(inv)], v_pages=a.v_pages[torch.from_numpy(inv)],
                prefix_block_table=torch.from_numpy(tab))
    np.testing.assert_array_equal(run_gpu(b, B.MARL_OUT_F32), out1)


def test_bad_contents_are_flagged_not_followed():
    from dataclasses import replace
    a = I.build_prefill_inputs(8, 2, [20, 30], [0, 0], seed=8, poison=False)
    # a table entry out of range: reads page 0 instead, flag 4
    tab = a.prefix_block_table.clone()
    tab[1, 0] = a.num_pages + 5
    got = run_gpu(replace(a, prefix_block_table=tab), B.MARL_OUT_F32, expect_flags=B.FLAG_BAD_PAGE)
    assert np.isfinite(got).all()
    # a chunk that does not fit its table row is cut short, flag 2
    pos0 = a.q_pos0.clone()
    pos0[1] = 16          # 30 tokens from position 16 need 46 positions, the row has 32
    got = run_gpu(replace(a, q_pos0=pos0), B.MARL_OUT_F32, expect_flags=B.FLAG_LEN_CLAMPED)
    assert np.isfinite(got[:36]).all() and np.isnan(got[36:]).all()
    # q_start beyond the q array drops the group, flag 1
    qs = a.q_start.clone()
    qs[2] = 60
    got = run_gpu(replace(a, q_start=qs), B.MARL_OUT_F32, expect_flags=B.FLAG_BAD_GROUP)
    assert np.isfinite(got[:20]).all() and np.isnan(got[20:]).all()


def test_prompt_scatter_is_bit_exact_and_feeds_attention():
    inp = I.build_prefill_inputs(28, 4, [37, 0, 16, 130], [0, 3, 16, 21], seed=9)
    dev = inp.to("cuda")
    shape, ws, out = B.prepare_prefill(dev, B.MARL_OUT_F32)
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.marl_kv_write_prompt(shape, dev.k_new, dev.v_new, dev.k_pages, dev.v_pages, dev.prefix_block_table,
                           dev.q_start, dev.q_pos0, flags)
    torch.cuda.synchronize()
    assert int(flags.item()) == 0
    kp, vp = R.kv_write_prompt(I.bf16_bits(inp.k_pages), I.bf16_bits(inp.v_pages), inp.prefix_block_table.numpy(),
                               inp.q_start.numpy(), inp.q_pos0.numpy(), I.bf16_bits(inp.k_new), I.bf16_bits(inp.v_new))
    # NaN poison compares by bit pattern
    np.testing.assert_array_equal(I.bf16_bits(dev.k_pages.cpu()), kp)
    np.testing.assert_array_equal(I.bf16_bits(dev.v_pages.cpu()), vp)
    B.run_prefill(dev, shape, ws, out)
    torch.cuda.synchronize()
    args = (inp.prefix_block_table.numpy(), inp.q_start.numpy(), inp.q_pos0.numpy(), inp.scale, 28, 4)
    want = R.prefill_attn(I.bf16_bits(inp.q), kp, vp, *args)
    want_abs = R.prefill_attn(I.bf16_bits(inp.q), kp, vp & 0x7fff, *args)
    excess = np.abs(out.cpu().numpy().astype(np.float64) - want) - (1e-3 + 2.0 ** -8 * want_abs)
    assert excess.max() <= 0


def scatter_equals_reference(inp, flag=0):
    dev = inp.to("cuda")
    shape, _, _ = B.prepare_prefill(dev, B.MARL_OUT_F32)
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.marl_kv_write_prompt(shape, dev.k_new, dev.v_new, dev.k_pages, dev.v_pages, dev.prefix_block_table, dev.q_start, dev.q_pos0, flags)
    torch.cuda.synchronize()
    assert int(flags.item()) == flag
    kp, vp = R.kv_write_prompt(I.bf16_bits(inp.k_pages), I.bf16_bits(inp.v_pages), inp.prefix_block_table.numpy(),
                               inp.q_start.numpy(), inp.q_pos0.numpy(), I.bf16_bits(inp.k_new), I.bf16_bits(inp.v_new))
    np.testing.assert_array_equal(I.bf16_bits(dev.k_pages.cpu()), kp)
    np.testing.assert_array_equal(I.bf16_bits(dev.v_pages.cpu()), vp)


@pytest.mark.parametrize("heads,chunk,ctx", [
    ((16, 1), [1], [0]), ((8, 2), [1, 2000, 3, 0, 17], [4000, 5, 15, 100, 31]), ((4, 4), [16, 16, 15, 17], [0, 8, 1, 15]),
    ((8, 2), [3000] + [1] * 40, [7] + [63] * 40), ((8, 2), [0, 0, 33], [16, 0, 8000]),
    # by places, up to and beyond what a wave sees at once, and the most groups that it is done for; and by rounds beyond
    ((16, 4), [2000] + [1] * 63, [3] + [900] * 63), ((16, 4), [1] * 64 + [2000], [900] * 64 + [15]),
    ((2, 2), [1] * 500 + [1500] + [2, 17, 0] * 174 + [18], [95] * 1024), ((2, 2), [1] * 500 + [1500] + [2, 17, 0] * 174 + [18] * 2, [95] * 1025),
    ((8, 8), [18, 2, 34, 1, 14, 3, 16], [15, 15, 31, 4000, 2, 14, 16]),
    # every column, and twice the mean of the chunks'
    ((4, 4), [700] * 30 + [1500], [300] * 31), ((4, 4), [200] * 60 + [1000], [900] * 60 + [0])])
def test_scatter_of_uneven_chunks(heads, chunk, ctx):
    """Chunks much longer than the mean, and such as touch few columns of a wide table, whole and in part, on each way a call can take."""
    print("case: scatter", heads, chunk[:5], ctx[:5], flush=True)
    scatter_equals_reference(I.build_prefill_inputs(*heads, chunk, ctx, seed=3))


@pytest.mark.parametrize("groups", [4, 40, 80])
def test_scatter_of_groups_that_share_rows(groups):
    """Entries of q_start in no order: every group that is consistent in itself has its pages written, the others are flagged."""
    from dataclasses import replace
    print("case: scatter, shared rows", groups, flush=True)
    inp = I.build_prefill_inputs(8, 1, [21] * groups, [979] * groups, seed=5, poison=False)
    ends = torch.zeros(groups + 1, dtype=torch.int32)
    ends[1:groups:2] = 21                                        # 0..21, back to 0, again: shared rows and reversed ones
    scatter_equals_reference(replace(inp, q_start=ends), B.FLAG_BAD_GROUP)


def test_scatter_flags_tokens_it_cannot_place():
    from dataclasses import replace
    inp = I.build_prefill_inputs(8, 2, [20, 30], [0, 0], seed=10, poison=False)
    dev = inp.to("cuda")
    shape, _, _ = B.prepare_prefill(dev, B.MARL_OUT_F32)
    tab = dev.prefix_block_table.clone()
    tab[0, 1] = -1
    before_k = dev.k_pages.clone()
    flags = torch.zeros(1, dtype=torch.int32, device="cuda")
    B.marl_kv_write_prompt(shape, dev.k_new, dev.v_new, dev.k_pages, dev.v_pages, tab, dev.q_start, dev.q_pos0, flags)
    torch.cuda.synchronize()
    assert int(flags.item()) == B.FLAG_BAD_PAGE
    # tokens 16..19 of group 0 were skipped: their former page is untouched
    pg = int(inp.prefix_block_table[0, 1])
    assert torch.equal(dev.k_pages[pg], before_k[pg])


def test_last_prompt_row_equals_the_decode_call_on_the_same_cache():
    # the decode entry point with an empty suffix over the same pages must agree with the last
    # prefill row up to the two kernels' rounding
    inp = I.build_prefill_inputs(28, 4, [513, 100], [0, 0], seed=11).to("cuda")
    shape, ws, out = B.prepare_prefill(inp, B.MARL_OUT_F32)
    B.run_prefill(inp, shape, ws, out)
    last = (inp.q_start[1:] - 1).long()
    dshape = B.make_shape(2, 2, 28, 4, inp.num_pages, int(inp.prefix_block_table.shape[1]), 1, B.MARL_OUT_F32)
    lay = B.marl_attn_plan_layout_for(dshape)
    dws = B.alloc_workspace(lay.total_bytes, "cuda")
    dout = torch.empty((2, 28, 128), device="cuda")
    B.marl_decode_attn(dshape, dws, inp.q[last].contiguous(), inp.k_pages, inp.v_pages, inp.prefix_block_table,
                       torch.full((2, 1), -1, dtype=torch.int32, device="cuda"),
                       torch.tensor([513, 100], dtype=torch.int32, device="cuda"),
                       torch.zeros(2, dtype=torch.int32, device="cuda"),
                       torch.arange(2, dtype=torch.int32, device="cuda"), inp.scale, dout)
    torch.cuda.synchronize()
    assert float((out[last] - dout).abs().max()) < 2e-3


def test_overlapping_groups_cannot_overrun_the_item_list():
    # three groups that all claim rows 0..299 of a 300-row q: the workspace is sized for groups
    # that share no rows, so the ones that do not fit are dropped and flagged
    from dataclasses import replace
    a = I.build_prefill_inputs(28, 4, [300, 0, 0], [0, 0, 0], seed=12, poison=False)
    tab = a.prefix_block_table[0:1].expand(3, -1).contiguous()
    qs = torch.tensor([0, 300, 0, 300], dtype=torch.int32)       # group 1 is inconsistent, group 2 overlaps group 0
    # q_start[1..2] = (300, 0): negative count -> flag 1; group 2 = rows 0..299 again
    got = run_gpu(replace(a, prefix_block_table=tab, q_start=qs), B.MARL_OUT_F32, expect_flags=B.FLAG_BAD_GROUP)
    want, want_abs = reference(a)
    assert (np.abs(got - want) <= 1e-3 + 2.0 ** -8 * want_abs).all()


def test_full_size_prompts_of_the_bench_workload_sampled_rows():
    """The prompts bench.py's prefill leg runs (256 prompts of the qwen7b workload, 329 k tokens),
    in the same launch configuration; sampled query rows are checked one by one with the C decode
    checker on a compact copy of the pages that row sees."""
    w = I.WORKLOADS["qwen7b"]
    lens = I.draw_lengths(w, np.random.default_rng(w.seed)).prefix_lens.tolist()
    inp = I.build_prefill_inputs(w.Hq, w.Hkv, lens, [0] * len(lens), device="cuda", seed=w.seed, poison=False)
    shape, ws, out = B.prepare_prefill(inp, B.MARL_OUT_BF16)
    B.run_prefill(inp, shape, ws, out)
    torch.cuda.synchronize()
    assert B.marl_attn_read_flags(ws) == 0
    assert bool(torch.isfinite(out.float()).all())
    qs = inp.q_start.cpu().numpy()
    rng = np.random.default_rng(4)
    longest, shortest = int(np.argmax(lens)), int(np.argmin(lens))
    picks = [(longest, lens[longest] - 1), (longest, 0), (shortest, lens[shortest] - 1), (0, 17), (255, lens[255] // 2)] + \
            [(int(g), int(rng.integers(0, lens[g]))) for g in rng.integers(0, len(lens), size=19)]
    worst = 0.0
    for g, tau in picks:
        npages = tau // 16 + 1
        pages = inp.prefix_block_table[g, :npages].long()
        kb, vb = I.bf16_bits(inp.k_pages[pages].cpu()), I.bf16_bits(inp.v_pages[pages].cpu())
        qb = I.bf16_bits(inp.q[qs[g] + tau:qs[g] + tau + 1].cpu())
        common = (np.arange(npages, dtype=np.int32)[None, :], np.zeros((1, 1), dtype=np.int32),
                  np.array([tau + 1], dtype=np.int32), np.zeros(1, dtype=np.int32), np.zeros(1, dtype=np.int32),
                  inp.scale, w.Hq, w.Hkv)
        want = R.decode_attn(qb, kb, vb, *common)[0]
        want_abs = R.decode_attn(qb, kb, vb & 0x7fff, *common)[0]
        got = out[qs[g] + tau].float().cpu().numpy().astype(np.float64)
        excess = np.abs(got - want) - (1e-3 + 2.0 ** -7 * want_abs)
        assert excess.max() <= 0, (g, tau, excess.max())
        worst = max(worst, float(np.abs(got - want).max()))
    print("prefill full size: worst |delta| over sampled rows", worst, flush=True)


@pytest.mark.parametrize("groups", [511, 512, 513, 700])
def test_lists_sorted_and_in_group_order(groups):
    """Row-block lists on both sides of the length up to which they are sorted; with two KV heads the
    longer ones give every workgroup items drawn from the counter.  One token per group behind
    contexts of different lengths: items of one step and of several, in any order."""
    print("case: prefill list", groups, flush=True)
    rng = np.random.default_rng(groups)
    pos0 = rng.choice([0, 1, 31, 32, 95, 127, 128, 129, 200], groups)
    check(I.build_prefill_inputs(6, 2, [1] * groups, pos0.tolist(), seed=groups), B.MARL_OUT_BF16)


@pytest.mark.parametrize("R", [1, 3, 5, 7, 11, 13, 16])
def test_rows_per_token(R):
    """Every block boundary inside a token for group sizes that do not divide 16; both output types."""
    print("case: prefill rows per token", R, flush=True)
    inp = I.build_prefill_inputs(2 * R, 2, [193, 64, 97], [0, 33, 500], seed=R)
    check(inp)
    check(inp, B.MARL_OUT_BF16)


@pytest.mark.parametrize("Hq,Hkv,chunks,context", [(1, 1, [1300], [0]), (8, 1, [100], [3000]), (16, 1, [30], [9000]),
                                                   (14, 2, [200, 33, 1], [1500, 40, 511])])
def test_few_long_items_are_divided_along_their_keys(Hq, Hkv, chunks, context):
    """Blocks of up to 16 parts; the first and the last case mix divided and whole blocks.  The parts are added in their order whoever finishes last: runs agree bit
    for bit.  A workspace with room for the list alone gives the same results from whole blocks."""
    print("case: prefill parts", Hq, Hkv, chunks, context, flush=True)
    inp = I.build_prefill_inputs(Hq, Hkv, chunks, context, seed=Hq)
    check(inp)
    check(inp, B.MARL_OUT_BF16)
    dev = inp.to("cuda")
    shape, ws, out = B.prepare_prefill(dev, B.MARL_OUT_F32)
    first = B.run_prefill(dev, shape, ws, out).clone()
    for _ in range(3):
        assert torch.equal(B.run_prefill(dev, shape, ws, out.zero_()), first)
    entries = lambda: int(ws[256:512].view(torch.int32)[len(chunks)])   # of the list, behind the header
    divided = entries()
    whole = B.run_prefill(dev, shape, ws[:4096], out.zero_())   # 256 header + 256 starts + 8 bytes for each block
    assert divided > entries()
    want, want_abs = reference(inp)
    assert (np.abs(whole.cpu().numpy() - want) <= 1e-3 + 2.0 ** -8 * want_abs).all()


@pytest.mark.parametrize("Hq,Hkv,chunks,context", [(8, 8, [2] * 140 + [100] * 2, [100] * 140 + [2500] * 2),
                                                   (16, 16, [1] * 66 + [96] * 2, [100] * 66 + [2500] * 2),
                                                   (16, 8, [1] * 120 + [90] * 4, [300] * 120 + [3000] * 4)])
def test_divided_blocks_among_items_drawn_from_the_counter(Hq, Hkv, chunks, context):
    """A few long blocks in parts among many short ones: more items than two for every workgroup, so parts and
    whole blocks are drawn while others run."""
    print("case: prefill parts drawn", Hq, Hkv, len(chunks), flush=True)
    inp = I.build_prefill_inputs(Hq, Hkv, chunks, context, seed=Hkv)
    check(inp)
    dev = inp.to("cuda")
    shape, ws, out = B.prepare_prefill(dev, B.MARL_OUT_F32)
    first = B.run_prefill(dev, shape, ws, out).clone()
    for _ in range(3):
        assert torch.equal(B.run_prefill(dev, shape, ws, out.zero_()), first)
    starts = (len(chunks) + 1 + 63) // 64 * 256
    entries = lambda: int(ws[256:256 + starts].view(torch.int32)[len(chunks)])   # of the list, behind the header
    divided = entries()
    assert divided * Hkv > 2 * 2 * torch.cuda.get_device_properties(0).multi_processor_count   # two workgroups per CU
    B.run_prefill(dev, shape, ws[:256 + starts + 4096], out)   # room for the list alone
    assert divided > entries()


@pytest.mark.parametrize("Hkv,groups", [(1, 600), (1, 1100), (2, 1100), (2, 1700)])
def test_lists_in_group_order_end_with_a_long_group(Hkv, groups):
    """Lists too long to be sorted: up to two items per workgroup, and more, of which the last two per workgroup
    are drawn by whoever is done, with none, some and many items bound ahead before them.  Short items, then a
    prompt of several blocks."""
    print("case: prefill late items", Hkv, groups, flush=True)
    rng = np.random.default_rng(groups + Hkv)
    pos0 = rng.choice([0, 1, 31, 95, 127, 200], groups).tolist() + [40]
    inp = I.build_prefill_inputs(2 * Hkv, Hkv, [1] * groups + [300], pos0, seed=groups)
    check(inp, B.MARL_OUT_BF16)
    dev = inp.to("cuda")
    shape, ws, out = B.prepare_prefill(dev, B.MARL_OUT_F32)
    first = B.run_prefill(dev, shape, ws, out).clone()
    for _ in range(3):
        assert torch.equal(B.run_prefill(dev, shape, ws, out.zero_()), first)


@pytest.mark.parametrize("blocks", [15, 16, 17, 64, 65, 130, 520])
@pytest.mark.parametrize("before", [0, 3, 1030])
def test_groups_of_many_blocks_are_listed_whole(blocks, before):
    """A group's blocks are listed by one thread up to 16 and by a wave above that, 64 at a time; the long groups stand in
    the plan's first round or its second, alone or among short ones, in lists that are sorted and that are not.  12 tokens
    of 16 heads fill a block."""
    print("case: prefill group of", blocks, "blocks behind", before, "groups", flush=True)
    inp = I.build_prefill_inputs(16, 1, [1] * before + [12 * blocks, 5, 12 * blocks - 11], [9] * before + [0, 40, 7], seed=blocks)
    check(inp)


def _general(inp):
    """The same call with a table too wide for the one launch of small calls."""
    from dataclasses import replace
    tab = inp.prefix_block_table
    wide = torch.full((tab.shape[0], 61), -1, dtype=torch.int32)
    wide[:, :tab.shape[1]] = tab
    return replace(inp, prefix_block_table=wide)


@pytest.mark.parametrize("Hq,Hkv,chunks,context", [
    (28, 4, [45], [0]), (1, 1, [1], [959]), (16, 1, [960], [0]), (16, 16, [31], [0]), (16, 16, [1] * 20 + [11], [0] * 21),
    (8, 8, [1] * 30 + [100, 0, 400], [5] * 33), (12, 4, [0, 3, 0, 0, 64, 65, 129], [0, 0, 8, 950, 17, 600, 1]), (4, 4, [1] * 64 + [200] * 3 + [1] * 60, [7] * 127),
    (2, 1, [1] * 255 + [97], [3] * 256), (2, 1, [1] * 600 + [200], [3] * 601), (64, 8, [100] * 12, [860] * 12),
    (16, 8, [2] * 60 + [40], [446] * 60 + [1]), (16, 8, [2] * 60 + [40], [447] * 60 + [1]), (4, 4, [5] * 766, [11] * 766), (4, 4, [5] * 767, [11] * 767)])
def test_small_calls_in_one_launch_equal_the_planned_ones(Hq, Hkv, chunks, context):
    """Bit for bit, at the edges of the rule (960 keys in a table row, one item fewer than there are workgroups at once; 448 keys, six
    items per workgroup), with empty groups, groups in the second and third round of 256, and blocks of one and several per group."""
    print("case: small prefill", Hq, Hkv, len(chunks), chunks[:3], context[:3], flush=True)
    inp = I.build_prefill_inputs(Hq, Hkv, chunks, context, seed=len(chunks))
    assert inp.prefix_block_table.shape[1] <= 60
    for out_dtype in (B.MARL_OUT_F32, B.MARL_OUT_BF16):
        np.testing.assert_array_equal(run_gpu(inp, out_dtype), run_gpu(_general(inp), out_dtype))
    check(inp)


@pytest.mark.parametrize("what", ["page", "page past the tokens", "long", "rows", "order", "overlap"])
def test_small_calls_flag_what_planned_ones_flag(what):
    from dataclasses import replace
    a = I.build_prefill_inputs(28, 4, [100, 40, 0, 77], [0, 16, 3, 5], seed=5, poison=False, extra_cols=13)
    tab, qs, pos0 = a.prefix_block_table.clamp(min=0), a.q_start.clone(), a.q_pos0.clone()   # (320 positions a row)
    if what == "page": tab[3, 5] = a.num_pages
    if what == "page past the tokens": tab[1, 4] = -7           # (56 tokens: four pages)
    if what == "long": pos0[0] = 290
    if what == "rows": qs[4] = 250
    if what == "order": qs[1] = 150
    if what == "overlap": qs = torch.tensor([0, 217, 0, 217, 0], dtype=torch.int32)
    flag = {"page": B.FLAG_BAD_PAGE, "page past the tokens": 0, "long": B.FLAG_LEN_CLAMPED}.get(what, B.FLAG_BAD_GROUP)
    bad = replace(a, prefix_block_table=tab, q_start=qs, q_pos0=pos0)
    got = run_gpu(bad, B.MARL_OUT_F32, flag)
    if what == "long":                                          # (a wider table would hold the tokens)
        assert np.isfinite(got[:30]).all() and np.isnan(got[30:100]).all()
    else:
        np.testing.assert_array_equal(got, run_gpu(_general(bad), B.MARL_OUT_F32, flag))


def test_small_calls_flag_groups_past_the_room_for_blocks():
    """Groups that all claim all rows: the room for blocks is used up by the first ones, and a group of a later round of 256 whose
    tokens do not fit its table row is flagged for that as well."""
    from dataclasses import replace
    print("case: small prefill, flags of late groups", flush=True)
    NG = 400
    a = I.build_prefill_inputs(8, 1, [1] * NG, [7] * NG, seed=2, poison=False)
    qs = torch.zeros(NG + 1, dtype=torch.int32)
    qs[1::2] = NG                                               # 0..400, 400..0 (flagged), 0..400 ...
    pos0 = a.q_pos0.clone().zero_()
    tab = torch.zeros(NG, 38, dtype=torch.int32)                # (608 positions, all of them on page 0)
    bad = replace(a, q_start=qs, q_pos0=pos0, prefix_block_table=tab)
    late = replace(bad, q_pos0=pos0.clone().index_fill_(0, torch.tensor([398]), 1000))
    for inp, flags in ((bad, B.FLAG_BAD_GROUP), (late, B.FLAG_BAD_GROUP | B.FLAG_LEN_CLAMPED)):
        run_gpu(inp, B.MARL_OUT_F32, flags)
        run_gpu(_general(inp), B.MARL_OUT_F32, flags)
