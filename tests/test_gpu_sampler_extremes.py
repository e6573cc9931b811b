"""Parameters and rows at the end of what a caller may pass: an infinite temperature (all probabilities are equal, so that
every token ties with the threshold), and rows in which every token is ruled out (the last one is returned, with a cut or
without)."""
import math

import numpy as np
import pytest

from gpu_checks import compare_tokens

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def _run(x, t, top_p, top_k, min_p, u):
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_02534_amd import binding as B
    B.load()
    rows, vocab = x.shape
    to = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.full((max(256, B.sample_tokens_workspace_size(rows, vocab)),), 255, dtype=torch.uint8, device="cuda")
    tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    xd, td, pd, ud, kd, md = to(x), to(t), to(top_p), to(u), to(top_k), to(min_p)
    B.sample_tokens_filtered(xd, B.SPD_F32, rows, vocab, vocab, td, pd, kd, md, ud, tokens, ws)
    torch.cuda.synchronize()
    return tokens.cpu().numpy()


@pytest.mark.parametrize("filters", [False, True])
@pytest.mark.parametrize("vocab", [5248, 50257, 128256])
def test_an_infinite_temperature_keeps_every_token(oracle, vocab, filters):
    print(f"infinite temperature: vocab {vocab}, filters {filters}", flush=True)
    rng = np.random.default_rng(vocab)
    x = (rng.standard_normal((8, vocab)) * np.array([3.0, 1e30] * 4)[:, None]).astype(np.float32)
    t, top_p = np.full(8, math.inf, np.float32), np.array([0.7, 0.7, 0.1, 0.1, 0.95, 0.95, 1.0, 1.0], np.float32)
    u = rng.random(8, dtype=np.float32)
    top_k = np.array([0, 50] * 4, np.int32) if filters else None
    min_p = np.array([0.3, 0.0, 0.0, 0.0] * 2, np.float32) if filters else None
    o = oracle.sample_tokens_filtered(x, t, top_p, u, top_k, min_p) if filters else oracle.sample_tokens(x, t, top_p, u)
    compare_tokens(_run(x, t, top_p, top_k, min_p, u), o, u, vocab)


@pytest.mark.parametrize("vocab", [1000, 9001, 128256])
def test_rows_without_any_token_left(vocab):
    x = np.full((4, vocab), -np.inf, np.float32)
    one = np.ones(4, np.float32)
    top_k = np.array([1, 50, 2 * vocab, 1], np.int32)
    print(f"nothing left: vocab {vocab}", flush=True)
    for top_p in (1.0, 0.9):
        got = _run(x, one, one * np.float32(top_p), top_k, one * np.float32(0.0), one * np.float32(0.5))
        assert np.all(got == vocab - 1), (top_p, got)


@pytest.mark.parametrize("filters", [False, True])
@pytest.mark.parametrize("vocab", [5248, 9001, 50257, 128256])
def test_a_top_p_next_to_one(oracle, vocab, filters):
    print(f"top-p next to 1: vocab {vocab}, filters {filters}", flush=True)
    rng = np.random.default_rng(vocab + 5)
    shares = [1 - 1e-5, 1 - 4e-6, 1 - 2e-6, 1 - 1e-6, 1 - 2.0 ** -22, 1 - 2.0 ** -24]
    rows = 4 * len(shares)
    top_p = np.repeat(np.array(shares, np.float32), 4)
    x = (rng.standard_normal((rows, vocab)) * 3.0).astype(np.float32)
    x[1::4] += np.linspace(4.0, -4.0, vocab, dtype=np.float32)
    x[2::4] = np.round(x[2::4])                             # thousands of equal logits in the tail
    x[3::4, rng.permutation(vocab)[300:]] = -np.inf         # a few hundred tokens left
    t = rng.choice(np.array([0.7, 1.0, 2.0], np.float32), rows)
    u = rng.random(rows, dtype=np.float32)
    u[::3] = rng.random(rows, dtype=np.float32)[::3] * np.float32(1e-6)
    top_k = rng.choice(np.array([0, 40, 4000], np.int32), rows) if filters else None
    min_p = rng.choice(np.array([0.0, 1e-7], np.float32), rows) if filters else None
    o = oracle.sample_tokens_filtered(x, t, top_p, u, top_k, min_p) if filters else oracle.sample_tokens(x, t, top_p, u)
    compare_tokens(_run(x, t, top_p, top_k, min_p, u), o, u, vocab)
