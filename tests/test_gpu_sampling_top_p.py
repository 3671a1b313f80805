"""GPU parity of marl_sample_tokens_top_p.  Two integers are decided by floating-point sums
(float32 on the GPU, float64 in the reference): which value is the nucleus threshold, and
which token passes the scaled uniform.  A drawn token is accepted when it is what the
reference draws for top_p and u moved by at most 4e-6 (relative) / 2e-6 (of the nucleus mass);
it must EQUAL the reference token whenever no nucleus boundary lies within 4e-6 of top_p and
no CDF step within 2e-6 of u.  The log-probability must match the reference's for that token
to 1e-3."""
import numpy as np
import pytest
import torch

from oracle import reference as ref
from paper_2602_09578_amd import binding as B
from paper_2602_09578_amd import inputs as I

pytestmark = pytest.mark.gpu
P_TOL, CDF_TOL = 4e-6, 2e-6


def run(logits: torch.Tensor, u: np.ndarray, T: float, top_p: float):
    d = logits.cuda()
    rows = d.shape[0]
    tok = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    out = torch.zeros(rows, dtype=torch.float32, device="cuda")
    B.marl_sample_tokens_top_p(d, torch.from_numpy(u.astype(np.float32)).cuda(), T, top_p, tok, out)
    torch.cuda.synchronize()
    return tok.cpu().numpy(), out.cpu().numpy().astype(np.float64)


def check(logits: torch.Tensor, u: np.ndarray, T: float, top_p: float, rows_to_check=None):
    tok, out = run(logits, u, T, top_p)
    u32 = u.astype(np.float32).astype(np.float64)
    tp = float(np.float32(top_p))
    exact = 0
    for r in (range(len(u)) if rows_to_check is None else rows_to_check):
        p, _ = ref.softmax_cdf(I.bf16_bits(logits[r:r + 1])[0], T)
        t = int(tok[r])
        assert 0 <= t < len(p) and p[t] > 0, (r, t)
        masks = [ref.nucleus(p, min(1.0, tp * f)) for f in (1 - P_TOL, 1.0, 1 + P_TOL)]
        ok = False
        for keep in masks:
            if not keep[t]:
                continue
            q = np.where(keep, p, 0.0)
            cdf, mass = np.cumsum(q), q.sum()
            lo = cdf[t] - q[t]
            ok |= lo - CDF_TOL * mass <= u32[r] * mass <= cdf[t] + CDF_TOL * mass
        assert ok, (r, t, top_p)
        decidable = all(np.array_equal(masks[0], m) for m in masks[1:])
        if decidable:
            q = np.where(masks[1], p, 0.0)
            cdf, mass = np.cumsum(q), q.sum()
            steps = cdf[masks[1]]
            if np.abs(steps - u32[r] * mass).min() > CDF_TOL * mass:
                want, _ = ref.sample_tokens_top_p(I.bf16_bits(logits[r:r + 1]), [u32[r]], T, tp)
                assert t == want[0], (r, t, want[0])
                exact += 1
        assert abs(out[r] - np.log(p[t])) <= 1e-3
    return exact


@pytest.mark.parametrize("rows,vocab,T,top_p", [
    (16, 4096, 1.0, 0.9), (12, 152064, 1.0, 0.95), (3, 152064, 0.6, 0.5), (100, 32000, 1.7, 0.8),
    (7, 4099, 1.0, 0.99), (5, 7, 1.0, 0.6), (2, 1, 1.0, 0.3), (9, 20481, 0.9, 0.1), (6, 8192, 1.0, 1.0),
    (6, 8193, 1.3, 1e-4),
    # rows longer than the register-resident variant holds (163840 logits): every pass re-reads memory
    (3, 200003, 1.0, 0.9), (2, 262144, 0.7, 0.97),
    # the two sides of that limit
    (2, 163840, 1.0, 0.8), (2, 163841, 1.0, 0.8)])
def test_tokens_match_the_reference(rows, vocab, T, top_p):
    print("case: top-p", rows, vocab, T, top_p, flush=True)
    lp = I.build_logprob_inputs(rows, vocab, 3.0, 31, temperature=T)
    rng = np.random.default_rng(rows * 11 + vocab)
    u = rng.random(rows)
    u[0] = 0.0
    if rows > 1:
        u[1] = np.nextafter(np.float32(1.0), np.float32(0.0))
    exact = check(lp.logits, u, T, top_p)
    # where the steps of the ranking's running mass and of the CDF are far apart compared with the
    # tolerances, nearly every draw is decidable (with top_p = 0.99 the boundary lies among tail
    # tokens of probability ~1e-5 and is rarely decidable)
    if 64 <= vocab <= 8192 and top_p <= 0.9:
        assert exact >= rows - 2
    if rows >= 100:   # a vocabulary of 32000: most draws are decided, and decided right
        assert exact >= 0.7 * rows, (exact, rows)


def test_flat_rows_ties_and_masks():
    print("case: top-p special", flush=True)
    V = 10000
    flat = torch.full((4, V), 0.5, dtype=torch.bfloat16)        # every token ties: the first ceil(top_p V) are kept
    u = np.array([0.00005, 0.25003, 0.5, 0.99996])
    tok, out = run(flat, u, 1.0, 0.3)
    assert np.abs(tok - np.floor(u.astype(np.float32).astype(np.float64) * 3000)).max() <= 1
    assert tok.max() < 3001 and np.abs(out + np.log(V)).max() <= 1e-3
    x = torch.zeros(3, 5000, dtype=torch.bfloat16); x[:, :100] = float("-inf"); x[:, 4000:] = float("-inf")
    x[2, :] = float("-inf")
    tok, out = run(x, np.array([0.0, 0.9999999, 0.5]), 1.0, 0.5)  # 3900 equal tokens, half of them kept
    assert tok[0] == 100 and abs(tok[1] - (100 + 1949)) <= 1 and tok[2] == -1 and np.isnan(out[2])
    # the same on a row that is re-read from memory for every pass
    V2 = 170000
    flat2 = torch.full((2, V2), -1.25, dtype=torch.bfloat16)
    u2 = np.array([0.25003, 0.99996])
    tok, out = run(flat2, u2, 1.0, 0.3)
    assert np.abs(tok - np.floor(u2.astype(np.float32).astype(np.float64) * 51000)).max() <= 1
    assert tok.max() < 51001 and np.abs(out + np.log(V2)).max() <= 1e-3
    # +0 and -0 are different bit patterns of the same probability: they tie, by index
    z = torch.zeros(2, 1000, dtype=torch.bfloat16); z[:, ::2] = -0.0
    tok, _ = run(z, np.array([0.5003, 0.99996]), 1.0, 0.25)
    assert list(tok) == [125, 249]
    # a peaked row: one token holds 99 %: any top_p up to that returns it whatever u is
    y = torch.zeros(2, 3000, dtype=torch.bfloat16); y[:, 1234] = 12.5
    tok, _ = run(y, np.array([0.0, 0.999]), 1.0, 0.9)
    assert list(tok) == [1234, 1234]


def test_nucleus_below_the_first_window_of_values():
    # logits spread over a wide range with top_p close to 1: the threshold value lies more than
    # 32768 bf16 values below the maximum (beyond the first histogram window)
    rng = np.random.default_rng(3)
    x = torch.from_numpy(rng.uniform(-0.9, 0.3, size=(6, 6000)).astype(np.float32)).to(torch.bfloat16)
    u = rng.random(6)
    assert check(x, u, 1.0, 0.98) >= 4
    assert check(x, u, 1.0, 0.999999) >= 0


def test_full_size_rows_rerun_identical_and_sampled_check():
    print("case: top-p full size", flush=True)
    w = I.WORKLOADS["qwen7b"]
    lp = I.build_logprob_inputs(w.num_seqs, w.vocab, w.logit_sigma, w.seed, device="cuda")
    u = np.random.default_rng(9).random(w.num_seqs)
    tok1, out1 = run(lp.logits, u, 1.0, 0.9)
    tok2, out2 = run(lp.logits, u, 1.0, 0.9)
    assert np.array_equal(tok1, tok2) and np.array_equal(out1, out2)
    sample = list(range(0, w.num_seqs, 128))
    sub = lp.logits[sample].cpu()
    tok_s, out_s = run(sub, u[sample], 1.0, 0.9)
    assert np.array_equal(tok_s, tok1[sample])                 # a row's result does not depend on the batch
    check(sub, u[sample], 1.0, 0.9)


def run_rows(logits, u, T, top_p):
    rows = logits.shape[0]
    tok, lp = torch.empty(rows, dtype=torch.int32, device="cuda"), torch.empty(rows, dtype=torch.float32, device="cuda")
    B.marl_sample_tokens_top_p(logits, torch.from_numpy(u.astype(np.float32)).cuda(), T, top_p, tok, lp)
    torch.cuda.synchronize()
    return tok.cpu().numpy(), lp.cpu().numpy()


def _route_rows(kind, V, rng):
    """Rows that send the threshold search down one of its routes."""
    x = (rng.standard_normal((3, V)) * 3).astype(np.float32)
    if kind == "negative":           # every logit negative: the list's cut has to be positive
        x = -np.abs(x) - 0.5
    elif kind == "shifted":          # all positive, within a few octaves
        x = x + 40.0
    elif kind == "one_wave":         # the likely tokens lie in every eighth group of 2048: one wave's list overflows
        x = x * 0.3
        pos = np.arange(V)
        x[:, (pos // 2048) % 8 == 2] += 9.0
    elif kind == "unsampled":        # the unlikely half of the mass lies where the estimate does not look
        x = np.full((3, V), -20.0, dtype=np.float32)
        pos = np.arange(V)
        x[:, (pos % 512) % 8 >= 4] = 4.0
        x[:, 7::1024] = 11.0
    elif kind == "near_zero":        # a flat row: the threshold value is a tiny number of either sign
        x = x * 0.05
    return torch.from_numpy(x).to(torch.bfloat16)


@pytest.mark.parametrize("kind", ["normal", "negative", "shifted", "one_wave", "unsampled", "near_zero"])
@pytest.mark.parametrize("V,T,top_p", [(2047, 1.0, 0.9), (2049, 0.7, 0.6), (20481, 1.0, 0.9), (65536, 1.3, 0.8), (152064, 1.0, 0.95)])
def test_threshold_search_routes(kind, V, T, top_p):
    """Short list (found, too long, cut not positive, threshold missed by the estimate) and the count of
    whole rows by windows of values give the same nucleus as the reference."""
    print("case: top-p routes", kind, V, T, top_p, flush=True)
    rng = np.random.default_rng(V + len(kind))
    check(_route_rows(kind, V, rng), np.array([0.0, rng.random(), 0.999999]), T, top_p)


@pytest.mark.parametrize("V", [327680, 327681])
def test_longest_row_with_a_list(V):
    print("case: top-p list limit", V, flush=True)
    rng = np.random.default_rng(V)
    check(_route_rows("normal", V, rng)[:2], np.array([0.3, 0.8]), 0.7, 0.9)


@pytest.mark.parametrize("top_p", [0.98, 0.983, 0.986])
def test_threshold_just_below_zero(top_p):
    """Logits and a temperature near 1e-19, one logit in 500 exactly +0 or -0, the threshold value
    negative: over the rows (equal shapes whose maxima lie 2^-72 apart) the estimated cut passes the value at
    which a window of 8192 values ends right below zero, so that the zeros are what lies above it."""
    print("case: top-p window below zero", top_p, flush=True)
    L, V, rows = 2.0 ** -63, 20481, 256
    rng = np.random.default_rng(17)
    x = np.empty((rows, V))
    for r in range(rows):
        x[r] = (0.25 + r % 128 / 512.0) - rng.random(V) * 1.7
        x[r, rng.random(V) < 0.002] = 0.0
        x[r, 5] = 0.25 + r % 128 / 512.0
    x[:, 1::2][x[:, 1::2] == 0.0] = -0.0
    check(torch.from_numpy(x * L).to(torch.bfloat16), rng.random(rows), 1.4426950408889634 * L / 4, top_p)


@pytest.mark.parametrize("V", [1, 513, 2048, 16384, 16385, 32768, 65536, 65537, 155648, 163841])
@pytest.mark.parametrize("sigma,T,top_p", [(2.0, 1.0, 0.95), (2.0, 1.3, 0.95), (3.0, 0.7, 0.8)])
def test_wide_nuclei_at_every_row_length(V, sigma, T, top_p):
    """A third of the row or most of it in the nucleus, its threshold just above zero or negative, at the row
    lengths where the sample's density and the number of lanes that share a group's list change."""
    print("case: top-p row lengths", V, sigma, T, top_p, flush=True)
    lp = I.build_logprob_inputs(4, V, sigma, V, temperature=T)
    check(lp.logits, np.array([0.0, 0.37, 0.71, 0.999999]), T, top_p)


@pytest.mark.parametrize("groups", [2, 3, 5, 6, 7, 10, 11, 12, 13, 17, 20])
def test_lists_of_every_number_of_groups(groups):
    """Groups per wave on both sides of the numbers at which other numbers of lanes share one, the last wave with a group less."""
    V = groups * 16384 - 2048 - 700
    print("case: top-p groups", groups, V, flush=True)
    lp = I.build_logprob_inputs(5, V, 3.0, groups, temperature=0.8)
    check(lp.logits, np.array([0.0, 0.2, 0.5, 0.8, 0.999999]), 0.8, 0.9)


@pytest.mark.parametrize("rows,V", [(256, 49153), (257, 49153), (256, 49152), (3, 152064), (3, 157697)])
@pytest.mark.parametrize("sigma,T,top_p", [(2.0, 1.0, 0.95), (3.0, 1.3, 0.95), (2.0, 1.3, 0.9), (2.0, 1.3, 0.95)])
def test_long_lists_of_rows_alone_on_a_cu(rows, V, sigma, T, top_p):
    """Both sides of the rule for rows that have a CU's LDS for their list; nuclei of a tenth of the row to most of it, which fit
    the longer list, or neither."""
    print("case: top-p alone", rows, V, sigma, T, top_p, flush=True)
    lp = I.build_logprob_inputs(rows, V, sigma, V + rows, temperature=T)
    check(lp.logits, np.random.default_rng(rows).random(rows), T, top_p)


@pytest.mark.parametrize("V", [28671, 28673, 28675, 32767, 49155, 100003])
@pytest.mark.parametrize("first", [0, 1, 7])
def test_rows_that_start_anywhere(V, first):
    """Rows at every distance from a 16-byte boundary, the first one in the middle of a buffer whose other elements must not be
    drawn or counted: the token before a row and the one behind it are the largest values there are.  Tokens at
    both ends of a row are drawn too."""
    print("case: top-p row starts", V, first, flush=True)
    rows = 9
    lp = I.build_logprob_inputs(rows, V, 2.5, V + first, temperature=0.9)
    x = lp.logits.clone()
    x[0, 0] = x[1, V - 1] = x[2, 1] = x[3, V - 2] = 30.0
    buf = torch.full((first + rows * V + 8,), 3.0e38, dtype=torch.bfloat16)
    buf[first:first + rows * V] = x.flatten()
    on_gpu = buf.cuda()[first:first + rows * V].view(rows, V)
    assert on_gpu.data_ptr() % 16 == 2 * first
    u = np.linspace(0.0, 0.999999, rows)
    check(x, u, 0.9, 0.9)                       # (the same rows in a buffer of their own)
    want_tok, want_lp = run_rows(x.cuda(), u, 0.9, 0.9)
    tok, got = run_rows(on_gpu, u, 0.9, 0.9)
    assert tok[:4].tolist() == [0, V - 1, 1, V - 2]
    for k in range(rows):                       # every row at a start of its own
        alone = x[k:k + 1].cuda()
        one_tok, one_lp = run_rows(alone, u[k:k + 1], 0.9, 0.9)
        assert one_tok[0] == tok[k] and one_lp[0] == got[k]
    np.testing.assert_array_equal(tok, want_tok)
    np.testing.assert_array_equal(got, want_lp)


def edge_uniforms(bits, T, top_p, n, rng):
    """Uniform numbers at the float32 next to n edges of the row's CDF inside its nucleus, where the last bits of the sums decide."""
    p, _ = ref.softmax_cdf(bits, T)
    keep = ref.nucleus(p, float(np.float32(top_p)))
    cdf = np.cumsum(np.where(keep, p, 0.0))
    return np.clip(cdf[rng.choice(np.nonzero(keep)[0], n)] / cdf[-1], 0.0, 1.0 - 2.0 ** -24)


def same_in_every_batch(V, sigma, T, top_p, rows, sizes):
    """One row `rows` times, with uniform numbers at its CDF's edges: token and log-probability of each are the same bits in
    batches of the given sizes, whatever the copy's alignment."""
    lp = I.build_logprob_inputs(1, V, sigma, V + 1, temperature=T)
    u = edge_uniforms(I.bf16_bits(lp.logits)[0], T, top_p, rows, np.random.default_rng(V))
    x = lp.logits.cuda().expand(rows, V).contiguous()
    want = run_rows(x, u, T, top_p)
    for n in sizes:
        for a in (0, rows - n):
            got = run_rows(x[a:a + n], u[a:a + n], T, top_p)
            np.testing.assert_array_equal(got[0], want[0][a:a + n])
            np.testing.assert_array_equal(got[1], want[1][a:a + n])
    by_token = {}
    for t, l in zip(*want):
        assert by_token.setdefault(int(t), l) == l


@pytest.mark.parametrize("V,sigma,T,top_p", [(32003, 2.0, 1.0, 0.95), (28673, 3.0, 1.0, 0.9), (4099, 2.0, 1.0, 0.95), (34816, 2.0, 1.0, 0.9)])
def test_a_row_is_the_same_at_every_alignment(V, sigma, T, top_p):
    """Copies of a row in a batch start at every distance from a 16-byte boundary, or all at an odd element."""
    print("case: top-p alignments", V, flush=True)
    if V % 2:
        same_in_every_batch(V, sigma, T, top_p, 40, [1, 7, 8, 33])
    lp = I.build_logprob_inputs(1, V, sigma, V, temperature=T)
    u = edge_uniforms(I.bf16_bits(lp.logits)[0], T, top_p, 100, np.random.default_rng(V))
    want = None
    for first in range(8):
        buf = torch.full((first + 100 * V + 8,), 3.0e38, dtype=torch.bfloat16, device="cuda")
        buf[first:first + 100 * V].view(100, V).copy_(lp.logits.cuda().expand(100, V))
        got = run_rows(buf[first:first + 100 * V].view(100, V), u, T, top_p)
        want = want or got
        np.testing.assert_array_equal(got[0], want[0])
        np.testing.assert_array_equal(got[1], want[1])


@pytest.mark.parametrize("rows,V,sigma,T,top_p", [
    (15, 20481, 3.0, 0.7, 0.8), (16, 20481, 3.0, 0.7, 0.8), (40, 65536, 3.0, 0.7, 0.8), (40, 2048, 4.0, 0.6, 0.8),
    (16, 152064, 6.0, 0.5, 0.5), (300, 4096, 3.0, 0.7, 0.8), (17, 152064, 2.0, 1.3, 0.9), (17, 152064, 2.0, 1.3, 0.92)])
def test_rows_whose_estimate_may_fail(rows, V, sigma, T, top_p):
    """Rows whose mass a handful of tokens hold, which a sample easily misses, and rows whose list may just overflow."""
    print("case: top-p estimate", rows, V, sigma, T, top_p, flush=True)
    lp = I.build_logprob_inputs(rows, V, sigma, V + rows, temperature=T)
    check(lp.logits, np.random.default_rng(rows).random(rows), T, top_p)


@pytest.mark.parametrize("V,sigma,T,top_p", [
    (20481, 3.0, 0.7, 0.8), (4096, 3.0, 0.7, 0.8), (32000, 2.0, 1.0, 0.95), (65536, 3.0, 0.7, 0.8), (20480, 4.0, 0.6, 0.8)])
def test_a_row_is_the_same_in_few_rows_and_in_many(V, sigma, T, top_p):
    """The cut, and with it what the list holds, follows from the row."""
    print("case: top-p batches", V, sigma, T, top_p, flush=True)
    same_in_every_batch(V, sigma, T, top_p, 60, [1, 7, 8, 15, 16, 17])


@pytest.mark.parametrize("V,sigma,T,top_p", [
    (49160, 2.0, 1.0, 0.95), (65536, 3.0, 1.3, 0.95), (152064, 3.0, 1.0, 0.95), (152064, 3.0, 1.3, 0.95), (152064, 2.0, 1.0, 0.9),
    (100003, 2.0, 1.0, 0.95), (156368, 2.0, 1.3, 0.9), (152064, 2.0, 1.3, 0.95), (65536, 1.0, 1.0, 0.99),
    (4095, 3.0, 1.0, 0.95), (4097, 3.0, 1.0, 0.95), (12287, 3.0, 1.0, 0.95), (12289, 3.0, 1.0, 0.95)])
def test_a_row_is_the_same_alone_on_a_cu_and_beside_others(V, sigma, T, top_p):
    """Lists that a third of a CU's LDS has room for, lists that only all of it has room for, and none of them; odd rows on both
    sides of the sizes from which they are shifted into place."""
    print("case: top-p alone or not", V, sigma, T, top_p, flush=True)
    same_in_every_batch(V, sigma, T, top_p, 300, [1, 64, 256, 257])
