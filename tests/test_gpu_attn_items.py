"""The kernel that takes prefix and suffix items from one queue: against the float64 oracle where its queue, its
rule and what it leaves to the merge kernel change."""
import numpy as np
import pytest

from paper_2602_09578_amd import binding as B
from tests.gpu_common import ATTN_TOL, gpu_attn, oracle_attn
from tests.test_gpu_attn import custom_inputs
from tests.test_gpu_attn_small import used_kernels

pytestmark = pytest.mark.gpu
CTR_DRAWN = 2   # items that were drawn from the queue
CTR_FIRST = 8   # suffix items that the queue has before the prefix items


def counter(call, which):
    return int(call.workspace[:256].cpu().numpy().view(np.int32)[which])


def first_items(call):
    return counter(call, CTR_FIRST)


def check(inp, call_args, tol=ATTN_TOL):
    want = oracle_attn(inp)
    got, call = gpu_attn(inp, B.MARL_OUT_F32, **call_args)
    assert np.abs(got - want).max() <= tol + 2.0 ** -9 * np.abs(want).max()   # (2^-9: a weight's rounding, for rows of a few tokens)
    again, _ = gpu_attn(inp, B.MARL_OUT_F32, **call_args)
    assert np.array_equal(got, again)
    return call


@pytest.mark.parametrize("samples,Hq,Hkv", [(5, 28, 4), (24, 28, 4), (3, 16, 1)])
def test_kinds_of_items(samples, Hq, Hkv):
    """Long suffixes before the prefix items, beside sequences without a prefix, without tokens of their own, of one
    short item, of one long item and of several with a short tail; blocks of 128 and of 256 rows."""
    print("case: kinds of items", samples, flush=True)
    rng = np.random.default_rng(samples)
    plens = [0, 65, 97, 129]
    gos = rng.permutation(np.repeat(np.arange(4), samples))
    slens = rng.choice([0, 1, 127, 128, 129, 160, 161, 511, 512, 513, 600, 1100], size=len(gos))
    slens[:3] = [1100, 0, 640]
    inp = custom_inputs(plens, slens, gos, Hq, Hkv, seed=samples)
    call = check(inp, dict(suffix_chunk_tokens=512, prefix_chunk_tokens=96))
    assert "plan" in used_kernels(inp.to("cuda"), call)
    # the head of the list: items of at least 4 x 96 tokens (the longest prefix item), to 32 tokens
    tokens = np.concatenate([np.full(n // 512, 512) for n in slens] + [slens % 512])
    assert (tokens >= 4 * 96 + 31).sum() <= first_items(call) <= (tokens > 4 * 96 - 32).sum()
    call = check(inp, dict(suffix_chunk_tokens=64, prefix_chunk_tokens=32))   # no long item at all
    assert first_items(call) == 0


@pytest.mark.parametrize("seqs", [768, 769])
def test_pairs_at_the_rule(seqs):
    """6144 (sequence, KV head) pairs share a launch, more do not; a chunk named so that no call is a small one."""
    print("case: pairs at the rule", seqs, flush=True)
    rng = np.random.default_rng(4)
    gos = np.arange(seqs) % 40
    inp = custom_inputs(rng.integers(0, 90, 40), rng.integers(0, 200, seqs), gos, 8, 8, seed=4)
    call = check(inp, dict(suffix_chunk_tokens=8192))
    assert used_kernels(inp.to("cuda"), call) == ({"plan", "suffix", "merge"} if seqs * 8 <= 6144 else {"plan", "prefix", "suffix", "merge"})


@pytest.mark.parametrize("Hq,Hkv,scale", [(28, 4, None), (16, 1, -0.1), (4, 4, None)])
def test_short_items_behind_none_one_and_several_prefix_partials(Hq, Hkv, scale):
    """Items of one wave, of one step and of several, with and without a ragged end: their first prefix partial is requested
    before the last step is done, further ones after it."""
    print("case: short items", Hq, Hkv, scale, flush=True)
    plens = [0, 1, 64, 65, 200, 300]   # 0, 1, 1, 2, 4 and 5 chunks
    own = [1, 16, 17, 31, 32, 33, 48, 64, 65, 127, 128]
    gos = np.repeat(np.arange(6), len(own))
    inp = custom_inputs(plens, own * 6, gos, Hq, Hkv, seed=Hq, scale=scale)
    check(inp, dict(suffix_chunk_tokens=512, prefix_chunk_tokens=64))


@pytest.mark.parametrize("seqs,Hkv,drawn", [(30, 4, 0), (600, 4, 0), (600, 8, 1)])
def test_short_items_are_not_drawn(seqs, Hkv, drawn):
    """Two sequences of several chunks with a short tail among many of one short item: entries of a short
    queue, else taken by waves before it, and what the merge kernel finishes costs no draw.  (The last case draws for
    its prefix items.)"""
    print("case: short items and draws", seqs, Hkv, flush=True)
    rng = np.random.default_rng(seqs)
    slens = rng.integers(1, 129, seqs)
    slens[[3, seqs - 1]] = [2 * 160 + 40, 160 + 128]
    groups = seqs // 4 if drawn else 8
    inp = custom_inputs(rng.integers(1, 90, groups), slens, np.arange(seqs) % groups, 2 * Hkv, Hkv, seed=seqs)
    call = check(inp, dict(suffix_chunk_tokens=160, prefix_chunk_tokens=96))
    prefix = groups * Hkv
    assert counter(call, CTR_DRAWN) <= drawn * (prefix + 3 * Hkv)
    check(inp, dict(suffix_chunk_tokens=32, prefix_chunk_tokens=32))


@pytest.mark.parametrize("Hq,Hkv", [(6, 6), (14, 2)])
def test_partials_behind_the_first_ones(Hq, Hkv):
    """Rows and short items whose number of partials stands at and beside the numbers that are requested together (four
    partials of a row, eight maxima behind the first four, or behind a short item's first one); one head per KV head, where
    the merge kernel has more waves of short items than of rows."""
    print("case: many partials", Hq, Hkv, flush=True)
    plens = [0, 32, 96, 128, 160, 256, 288, 320, 384, 416, 544]   # up to 17 prefix partials
    own = [0, 5, 128, 129, 300, 512]                              # 0 to 4 partials of their own, or one short item
    gos = np.repeat(np.arange(len(plens)), len(own))
    inp = custom_inputs(plens, own * len(plens), gos, Hq, Hkv, seed=Hq)
    check(inp, dict(suffix_chunk_tokens=128, prefix_chunk_tokens=32))
    check(inp, dict(suffix_chunk_tokens=32, prefix_chunk_tokens=512))
