"""Rows that one workgroup samples alone and rows that are divided, at the sizes where the one takes over from the
other and at the edges of their chunks of 4096 logits."""
import numpy as np
import pytest
import torch

from paper_2602_09578_amd import inputs as I
from tests.test_gpu_sampling import check, run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,vocab", [(3, 4095), (3, 4096), (3, 4097), (5, 30001), (4, 32768), (4, 32769), (700, 9001), (600, 28672),
                                        (512, 28673), (513, 28673), (238, 41000), (239, 41000), (253, 41001), (254, 41001), (256, 41001),
                                        (257, 41001), (477, 33000), (714, 32768), (715, 32768), (768, 33001), (1000, 33001),
                                        (1014, 33001), (1151, 33001), (1152, 33001),
                                        (238, 41001), (239, 41001), (478, 33001), (513, 30001)])
def test_whole_and_divided_rows(rows, vocab):
    """Some tokens and the whole tail masked; uniforms 0, just below 1 and in between.  A row's token and
    log-probability are the same bits in a batch that is divided and in one that is not."""
    print("case: sampling whole rows", rows, vocab, flush=True)
    rng = np.random.default_rng(rows * 31 + vocab)
    x = (rng.standard_normal((rows, vocab)) * 3).astype(np.float32)
    x[rng.random((rows, vocab)) < 0.3] = -np.inf
    x[::3, vocab - vocab // 7:] = -np.inf
    x[:, vocab // 2] = 0.5
    u = rng.random(rows)
    u[0], u[1] = 0.0, np.nextafter(np.float32(1.0), np.float32(0.0))
    lp = I.LogprobInputs(torch.from_numpy(x).to(torch.bfloat16), torch.zeros(rows, dtype=torch.int32), 0.8)
    pick = np.unique(np.r_[0:3, rng.integers(0, rows, 13)])          # (the reference is a loop over rows)
    tok, out = run(lp, u)
    sub = I.LogprobInputs(lp.logits[pick], lp.tokens[pick], lp.temperature)
    check(sub, u[pick])
    few, few_out = run(sub, u[pick])        # long rows: divided here
    assert np.array_equal(few, tok[pick]) and np.array_equal(few_out, out[pick])
    assert np.isfinite(x[np.arange(rows), tok]).all()


def test_rows_without_a_token():
    print("case: sampling whole rows, nothing to draw", flush=True)
    x = torch.full((4, 5000), float("-inf"), dtype=torch.bfloat16)
    x[1, 4999] = -3.0
    x[2, 0] = 7.0
    tok, out = run(I.LogprobInputs(x, torch.zeros(4, dtype=torch.int32), 1.0), np.array([0.5, 0.9999999, 0.0, 0.0]))
    assert tok.tolist() == [-1, 4999, 0, -1] and np.isnan(out[[0, 3]]).all() and np.abs(out[[1, 2]]).max() <= 1e-6
