"""The one-launch kernel that serves small decode calls: against the float64 oracle and against the general
kernels (which calls that name their chunk sizes take), at the edges of its rule and of its parts."""
import numpy as np
import pytest
import torch

from paper_2602_09578_amd import binding as B
from tests.gpu_common import ATTN_TOL, gpu_attn, oracle_attn
from tests.test_gpu_attn import custom_inputs
from tests.test_gpu_plan import compare

pytestmark = pytest.mark.gpu


def used_kernels(inp, call):
    """Stages of one call that ran: the small kernel counts as the prefix stage and has no plan stage."""
    B.marl_profile_begin(1)
    B.run_attn(inp, call)
    torch.cuda.synchronize()
    ms, n, _ = B.marl_profile_end()
    assert n == 1
    return {k for k in ("plan", "prefix", "suffix", "merge") if ms[k] > 0}


# (prefix lengths, own lengths, group of each sequence, Hq, Hkv, kernels): one part, several parts, parts without a
# token, tokens on and around page and step boundaries, sequences without a group, the largest size that the
# kernel takes and one token row more
RAGGED = ([0, 1, 16, 17, 31, 33, 300], [0, 5, 16, 31, 32, 33, 0, 64, 65, 1, 100, 0], [0, 1, 2, 3, 4, 5, 6, 6, 5, 2, 1, 5])
SMALL, PARTS, GENERAL = {"prefix"}, {"prefix", "merge"}, None   # (the general kernels: whichever there are, after a plan kernel)
CASES = [
    ("ragged, one row per head", *RAGGED, 4, 4, SMALL),
    ("ragged, sixteen rows", *RAGGED, 16, 1, SMALL),
    ("one token", [0], [1], [0], 7, 1, SMALL),
    ("no tokens of their own", [40, 70], [0, 0, 0], [0, 1, 1], 28, 4, SMALL),
    ("1008 tokens", [500], [496, 3], [0, 0], 8, 2, SMALL),
    ("1024 tokens", [512], [512, 3, 0], [0, 0, 0], 8, 2, PARTS),
    ("parts without a step", [0, 6000], [1, 0, 40, 129], [0, 0, 1, 1], 12, 4, PARTS),
    ("512 sequences", [30] * 64, [3 + s % 30 for s in range(512)], [(s * 7) % 64 for s in range(512)], 2, 1, SMALL),
    ("513 sequences", [30] * 64, [3 + s % 30 for s in range(512)] + [200], [(s * 7) % 64 for s in range(513)], 2, 1, GENERAL),
    ("one sequence, parts of eight heads", [100], [2300], [0], 16, 8, PARTS),
    ("seven sequences, parts", [17, 900], [1000, 1, 700, 33, 0, 1200, 64], [0, 1, 0, 1, 1, 0, 0], 8, 4, PARTS),
    ("seventeen sequences, three heads", [50, 70], [3 * s for s in range(17)], [s % 2 for s in range(17)], 6, 3, SMALL),
    ("nine sequences, five heads, parts", [600], [500 - s for s in range(9)], [0] * 9, 5, 5, PARTS),
    ("last rows of tokens", [16] * 2, [3 * 2 ** 19 // 64 - 16] + [9 + s for s in range(63)], [s % 2 for s in range(64)], 1, 1, PARTS),
    ("beyond them", [32] * 2, [3 * 2 ** 19 // 64 - 16] + [9 + s for s in range(63)], [s % 2 for s in range(64)], 1, 1, GENERAL),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_small_calls(case):
    name, pl, sl, gos, Hq, Hkv, kernels = case
    print("case: small call:", name, flush=True)
    inp = custom_inputs(pl, sl, gos, Hq, Hkv, seed=len(name))
    want = oracle_attn(inp)
    got, call = gpu_attn(inp, B.MARL_OUT_F32)
    general, _ = gpu_attn(inp, B.MARL_OUT_F32, suffix_chunk_tokens=1024, prefix_chunk_tokens=256)
    # float32 output: the weights' rounding to bf16 only, which averages out over hundreds of tokens and is at most
    # 2^-9 of a value of up to 5 over a few (as the general kernels', which are held to the same)
    bound = ATTN_TOL + 2.0 ** -9 * np.abs(want).max()
    assert np.abs(got - want).max() <= bound and np.abs(general - want).max() <= bound
    again, _ = gpu_attn(inp, B.MARL_OUT_F32)
    assert np.array_equal(got, again)
    dev = inp.to("cuda")
    used = used_kernels(dev, B.prepare_attn(dev, B.MARL_OUT_F32))
    assert used == kernels if kernels else "plan" in used


@pytest.mark.parametrize("scale", [-0.11, 0.0, 1.0])
def test_scales_and_output_types(scale):
    print("case: small call, scale", scale, flush=True)
    for tokens in (90, 1500):
        inp = custom_inputs([tokens, 40], [33, 7, 129, 64], [0, 0, 1, 1], 28, 4, seed=21, scale=scale)
        want = oracle_attn(inp)
        f32, _ = gpu_attn(inp, B.MARL_OUT_F32)
        # (scale 1: nearly one-hot weights, outputs of up to about 4, each weight rounded by 2^-9 of itself)
        assert np.abs(f32 - want).max() <= (4 * 2.0 ** -8 if scale == 1.0 else ATTN_TOL)
        bf16, _ = gpu_attn(inp, B.MARL_OUT_BF16)
        assert np.all(np.abs(bf16 - f32) <= np.abs(f32) * 2.0 ** -8 + 1e-30)   # one rounding apart


def work_list(call, NG, NS):
    """The plan that a call has left in its workspace; items in order of their contents."""
    L, host = call.layout, call.workspace.cpu().numpy()
    i32 = lambda off, n: host[off:off + 4 * n].view(np.int32).copy()
    ctr = i32(L.counters_off, 64)
    return (ctr, i32(L.group_count_off, NG), i32(L.group_start_off, NG + 1), i32(L.group_seqs_off, NS), i32(L.seq_chunks_off, NS),
            sorted(map(tuple, i32(L.suffix_items_off, 4 * ctr[0]).reshape(-1, 4).tolist())),
            sorted(map(tuple, i32(L.prefix_items_off, 4 * ctr[1]).reshape(-1, 4).tolist())))


def test_work_list_and_flags_are_left_as_the_header_says():
    """The workspace of a small call holds the plan that marl_attn_plan builds, and the flags of bad contents."""
    print("case: small call, workspace", flush=True)
    rng = np.random.default_rng(8)
    gos = rng.permutation(np.repeat(np.arange(6), [1, 2, 3, 8, 0, 5]))
    inp = custom_inputs(rng.integers(0, 300, 6), rng.integers(0, 300, len(gos)), gos, 8, 2, seed=2, poison=False).to("cuda")
    call = B.prepare_attn(inp, B.MARL_OUT_F32)
    shape = call.shape
    compare(shape, inp.prefix_lens.cpu(), inp.suffix_lens.cpu(), gos.astype(np.int32), 8, 2)   # marl_attn_plan against its reference
    lists = lambda: work_list(call, 6, len(gos))
    call.workspace.fill_(0xAB)
    B.marl_attn_plan(shape, call.workspace, inp.prefix_lens, inp.suffix_lens, inp.group_of_seq)
    want = lists()
    call.workspace.fill_(0xAB)
    B.run_attn(inp, call)
    torch.cuda.synchronize()
    for w, g in zip(want, lists()):
        assert np.array_equal(w, g)
    # a bad page id counts where a token needs it, and only there
    good = call.out.clone()
    empty = int(np.setdiff1d(np.arange(6), gos)[0])
    inp.prefix_block_table[empty, :] = 10 ** 8
    inp.suffix_block_table[0, (int(inp.suffix_lens[0]) + 15) // 16:] = -7
    B.run_attn(inp, call)
    assert B.marl_attn_read_flags(call.workspace) == 0 and torch.equal(call.out, good)
    inp.suffix_block_table[3, (int(inp.suffix_lens[3]) - 1) // 16] = inp.num_pages
    B.run_attn(inp, call)
    assert B.marl_attn_read_flags(call.workspace) == B.FLAG_BAD_PAGE
    others = [s for s in range(len(gos)) if s != 3]
    assert torch.equal(call.out[others], good[others]) and torch.isfinite(call.out[3]).all()


@pytest.mark.parametrize("NS,NG", [(1, 1), (64, 65), (300, 257), (512, 512), (512, 40)])   # (members are in order in groups of at most 64)
@pytest.mark.parametrize("longest", [255, 512, 1100])
def test_work_list_of_whole_chunks(NS, NG, longest):
    """Sequences and groups of none, one and several whole chunks side by side in a wave, and waves without any; one or two of each
    per thread of the plan's workgroup."""
    print("case: small call, whole chunks", NS, NG, longest, flush=True)
    rng = np.random.default_rng(NS + longest)
    own, prefix = rng.integers(0, longest + 1, NS), rng.integers(0, longest + 1, NG)
    own[NS // 3: NS // 2] %= 256      # (chunks of 256 tokens and more)
    prefix[NG // 2:] %= 256
    gos = rng.integers(0, NG, NS)
    inp = custom_inputs(prefix, own, gos, 4, 1, seed=2, poison=False).to("cuda")
    call = B.prepare_attn(inp, B.MARL_OUT_F32)
    assert used_kernels(inp, call) in (SMALL, PARTS)
    compare(call.shape, prefix, own, gos.astype(np.int32), 4, 1)   # marl_attn_plan against its reference
    call.workspace.fill_(0xAB)
    B.marl_attn_plan(call.shape, call.workspace, inp.prefix_lens, inp.suffix_lens, inp.group_of_seq)
    want = work_list(call, NG, NS)
    call.workspace.fill_(0xAB)
    B.run_attn(inp, call)
    torch.cuda.synchronize()
    n = int(want[2][-1])
    for k, (w, g) in enumerate(zip(want, work_list(call, NG, NS))):
        assert np.array_equal(w[:n], g[:n]) if k == 3 else np.array_equal(w, g)


# (sequences, longest own row in pages, capacity of a row in pages): one row and a row or more for every eight lanes of the
# plan's workgroup, rows of less than one request and of several
@pytest.mark.parametrize("seqs,longest,capacity", [(1, 3, 40), (1, 2060, 4000), (2, 3, 3), (70, 2, 2), (40, 4, 4), (3, 65, 65), (32, 70, 90), (33, 17, 100), (130, 9, 200), (512, 3, 160)])
def test_bad_page_ids_in_tables_of_a_fixed_capacity(seqs, longest, capacity):
    """Entries outside the pool count up to a row's last addressed one, and not behind it (where there is nothing but them)."""
    print("case: small call, tables of a fixed capacity", seqs, longest, capacity, flush=True)
    rng = np.random.default_rng(seqs + longest)
    slens = rng.integers(1, 16 * longest + 1, seqs)
    slens[0] = 16 * longest
    groups = max(1, seqs // 5)
    inp = custom_inputs(rng.integers(0, 200, groups), slens, np.arange(seqs) % groups, 2, 1, seed=seqs, poison=False)
    want = oracle_attn(inp)
    inp = inp.to("cuda")
    def widen(table, pages):
        wide = torch.randint(0, 2, (table.shape[0], pages), dtype=torch.int32, device="cuda") * (2 ** 31 - 1) - (2 ** 30)
        wide[:, :table.shape[1]] = torch.where(table < 0, wide[:, :table.shape[1]], table)
        return wide
    inp.suffix_block_table, inp.prefix_block_table = widen(inp.suffix_block_table, capacity), widen(inp.prefix_block_table, 20)
    call = B.prepare_attn(inp, B.MARL_OUT_F32)
    used = used_kernels(inp, call)
    assert "plan" not in used
    assert B.marl_attn_read_flags(call.workspace) == 0
    good = call.out.clone()
    assert np.abs(good.cpu().numpy() - want).max() <= ATTN_TOL + 2.0 ** -9 * np.abs(want).max()
    lens = inp.suffix_lens.tolist()
    for s in sorted({0, seqs // 2, seqs - 1}):
        last = (lens[s] - 1) // 16
        for page in sorted({0, last // 2, last}):
            kept = int(inp.suffix_block_table[s, page])
            inp.suffix_block_table[s, page] = inp.num_pages + int(rng.integers(0, 3))
            B.run_attn(inp, call)
            assert B.marl_attn_read_flags(call.workspace) == B.FLAG_BAD_PAGE, (s, page)
            inp.suffix_block_table[s, page] = kept
    g = int(inp.group_of_seq[seqs - 1])
    last = (int(inp.prefix_lens[g]) - 1) // 16
    if last >= 0:
        inp.prefix_block_table[g, last] = -1
        B.run_attn(inp, call)
        assert B.marl_attn_read_flags(call.workspace) == B.FLAG_BAD_PAGE
