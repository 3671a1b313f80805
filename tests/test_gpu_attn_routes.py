"""What holds for every decode-attention call, on each of the ways a call can take: the one kernel of a small call,
prefix and suffix items from one queue, and a kernel each for prefix items, long suffix items and the rest.  Which way it
was is read from the stages that ran."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2602_09578_amd import binding as B
from tests.gpu_common import ATTN_TOL, gpu_attn, oracle_attn
from tests.test_gpu_attn import custom_inputs
from tests.test_gpu_attn_small import used_kernels

pytestmark = pytest.mark.gpu

NAMED = dict(suffix_chunk_tokens=160, prefix_chunk_tokens=96)
# name -> (sequences, groups, Hq, Hkv, chunk sizes, stages, rows of a block of prefix rows)
ROUTES = {
    "small": (24, 4, 28, 4, {}, {"prefix"}, 128),
    "small, parts": (24, 4, 8, 2, {}, {"prefix", "merge"}, 128),
    "items": (40, 4, 28, 4, NAMED, {"plan", "suffix", "merge"}, 128),
    "items, wide": (48, 2, 28, 4, NAMED, {"plan", "suffix", "merge"}, 256),
    "items, long list": (300, 20, 16, 8, NAMED, {"plan", "suffix", "merge"}, 128),   # (short items by waves, not from the queue)
    "separate": (800, 40, 16, 8, NAMED, {"plan", "prefix", "suffix", "merge"}, 128),
    "separate, wide": (800, 5, 16, 8, NAMED, {"plan", "prefix", "suffix", "merge"}, 256),
}
# of the first sequences: own tokens of one long item and of one short one, several chunks with a short tail and without, none
FIRST = [150, 40, 2 * 160 + 100, 160 + 150, 0]


def route_inputs(route, seed, poison=True):
    NS, NG, Hq, Hkv, chunks, stages, rows = ROUTES[route]
    rng = np.random.default_rng(seed)
    plens = rng.integers(1, 260, NG)
    plens[:2] = [1200 if route == "small, parts" else 250, 0]
    slens = np.where(rng.random(NS) < 0.5, rng.integers(0, 129, NS), rng.integers(100, 300, NS))
    gos = np.arange(NS) % NG
    slens[:5 * NG:NG] = FIRST   # (sequences of group 0)
    inp = custom_inputs(plens, slens, gos, Hq, Hkv, seed=seed, poison=poison)
    return inp, chunks


def check_route(route, inp_dev, call):
    used = used_kernels(inp_dev, call)
    assert used == ROUTES[route][5] and call.layout.rows_per_qblock == ROUTES[route][6], route


@pytest.mark.parametrize("route", ROUTES)
def test_oracle_reruns_and_page_permutations(route):
    print("case: routes, reruns", route, flush=True)
    a, chunks = route_inputs(route, seed=31)
    out, call = gpu_attn(a, B.MARL_OUT_F32, **chunks)
    want = oracle_attn(a)
    assert np.abs(out - want).max() <= ATTN_TOL + 2.0 ** -9 * np.abs(want).max()   # (2^-9: a weight's rounding, for rows of a few tokens)
    dev = a.to("cuda")
    check_route(route, dev, call)
    for _ in range(3):
        B.run_attn(dev, call)
        torch.cuda.synchronize()
        assert np.array_equal(call.out.cpu().numpy().astype(np.float64), out)
    perm = torch.from_numpy(np.random.default_rng(5).permutation(a.num_pages))
    inv = torch.empty_like(perm)
    inv[perm] = torch.arange(a.num_pages)
    table = lambda t: torch.where(t >= 0, inv[t.clamp(min=0).long()].int(), -1)
    b = dataclasses.replace(a, k_pages=a.k_pages[perm], v_pages=a.v_pages[perm], prefix_block_table=table(a.prefix_block_table),
                            suffix_block_table=table(a.suffix_block_table))
    assert np.array_equal(gpu_attn(b, B.MARL_OUT_F32, **chunks)[0], out)


@pytest.mark.parametrize("route", ROUTES)
def test_what_no_token_owns_does_not_matter(route):
    print("case: routes, poison", route, flush=True)
    a, chunks = route_inputs(route, seed=32, poison=True)
    b, _ = route_inputs(route, seed=32, poison=False)   # same draws, unused locations hold ordinary numbers
    oa, call = gpu_attn(a, B.MARL_OUT_F32, **chunks)
    check_route(route, a.to("cuda"), call)
    ob, _ = gpu_attn(b, B.MARL_OUT_F32, **chunks)
    assert np.isfinite(oa).all() and np.array_equal(oa, ob)


@pytest.mark.parametrize("route", ROUTES)
def test_bad_page_ids_are_flagged(route):
    """Of a prefix, of one long item, of one short item, of a chunk and of a short tail: the flag is raised, outputs stay
    finite, and sequences that do not need the entry are computed as if nothing had happened."""
    print("case: routes, bad page ids", route, flush=True)
    inp, chunks = route_inputs(route, seed=33, poison=False)
    NG = ROUTES[route][1]
    dev = inp.to("cuda")
    call = B.prepare_attn(dev, B.MARL_OUT_F32, **chunks)
    check_route(route, dev, call)
    assert B.marl_attn_read_flags(call.workspace) == 0
    good = call.out.clone()
    seqs = torch.arange(len(inp.suffix_lens), device="cuda")
    cases = [("prefix_block_table", 0, 2, dev.group_of_seq == 0), ("prefix_block_table", 0, int(inp.prefix_lens[0] - 1) // 16, dev.group_of_seq == 0),
             ("suffix_block_table", 0, 9, seqs == 0), ("suffix_block_table", NG, 1, seqs == NG),
             ("suffix_block_table", 2 * NG, 3, seqs == 2 * NG), ("suffix_block_table", 2 * NG, 26, seqs == 2 * NG)]
    for name, row, page, needs in cases:
        table = getattr(dev, name)
        kept = int(table[row, page])
        for bad in (inp.num_pages, -5, 10 ** 8):
            table[row, page] = bad
            B.run_attn(dev, call)
            assert B.marl_attn_read_flags(call.workspace) == B.FLAG_BAD_PAGE, (name, row, page, bad)
            assert torch.isfinite(call.out).all() and torch.equal(call.out[~needs], good[~needs]), (name, row, page, bad)
        table[row, page] = kept
    B.run_attn(dev, call)
    assert B.marl_attn_read_flags(call.workspace) == 0 and torch.equal(call.out, good)


@pytest.mark.parametrize("route", ROUTES)
def test_captured_calls_replay_bit_identical(route):
    """New queries and lengths between the replays, with the program's own work and synchronisations."""
    print("case: routes, graph", route, flush=True)
    inp, chunks = route_inputs(route, seed=34)
    dev = inp.to("cuda")
    call = B.prepare_attn(dev, B.MARL_OUT_BF16, **chunks)
    check_route(route, dev, call)   # (also the warm-up: one-time device queries)
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(graph, stream=side):
            B.run_attn(dev, call)
    torch.cuda.synchronize()
    gen = torch.Generator(device="cuda").manual_seed(3)
    for rep in range(4):
        dev.q.copy_(torch.randn(dev.q.shape, generator=gen, device="cuda").to(torch.bfloat16))
        if rep % 2 == 1:
            dev.suffix_lens.copy_(torch.clamp(dev.suffix_lens - 17, min=0))
        B.run_attn(dev, call)
        torch.cuda.synchronize()
        want = call.out.clone()
        call.out.zero_()
        _ = (dev.q.float() ** 2).sum().item()
        graph.replay()
        torch.cuda.synchronize()
        assert B.marl_attn_read_flags(call.workspace) == 0
        assert torch.equal(call.out.view(torch.int16), want.view(torch.int16)), rep


@pytest.mark.parametrize("suffix_chunk", [8192, 160, 64])
def test_separate_kernels_on_ragged_groups(suffix_chunk):
    """Groups of 8, 9, 16 and 17 row tiles, an odd tile count, second blocks of one row and of ten tiles (one query row per
    sequence), chunks of one step with a few tokens, and short items by the prefix kernel's waves."""
    print("case: routes, ragged", suffix_chunk, flush=True)
    rng = np.random.default_rng(suffix_chunk)
    sizes = [128, 129, 136, 144, 145, 257, 400]
    gos = rng.permutation(np.repeat(np.arange(len(sizes)), sizes))
    slens = rng.choice([0, 1, 16, 33, 64, 65, 127, 128, 129, 200, 330], size=len(gos))
    inp = custom_inputs([0, 71, 39, 33, 64, 1, 130], slens, gos, 8, 8, seed=7)
    want = oracle_attn(inp)
    for prefix_chunk in (32, 0):
        got, call = gpu_attn(inp, B.MARL_OUT_F32, suffix_chunk_tokens=suffix_chunk, prefix_chunk_tokens=prefix_chunk)
        assert np.abs(got - want).max() <= ATTN_TOL + 2.0 ** -9 * np.abs(want).max()
        used = used_kernels(inp.to("cuda"), call)
        assert used == {"plan", "prefix", "merge"} | ({"suffix"} if suffix_chunk > 128 else set()) and call.layout.rows_per_qblock == 256
