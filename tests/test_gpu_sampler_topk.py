"""The k-th largest logit where it is hard to pin down: among hundreds or thousands of equal logits while the row's maximum
is small (its rounding says nothing about theirs), and far below the maximum (more than 64 octaves of probability), on
rows of 1, 2, 8 and 16 slices.  With top-p 1 whatever a lost filter keeps too much weighs enough to be drawn."""
import numpy as np
import pytest

from gpu_checks import compare_tokens

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

VOCABS = [8000, 9000, 128256, 262144]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_02534_amd import binding, device
    binding.load()
    return device


def _check(oracle, x, t, top_p, top_k, min_p, u, allow_exempt_mismatch=0):
    from paper_2502_02534_amd import binding as B
    rows, vocab = x.shape
    full = lambda v, dt: np.ascontiguousarray(np.broadcast_to(np.asarray(v, dt), (rows,)))
    t, top_p, top_k, min_p, u = full(t, np.float32), full(top_p, np.float32), full(top_k, np.int32), full(min_p, np.float32), full(u, np.float32)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.full((B.sample_tokens_workspace_size(rows, vocab),), 255, dtype=torch.uint8, device="cuda")
    tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    xd, td, pd, ud, kd, md = to(x), to(t), to(top_p), to(u), to(top_k), to(min_p)
    B.sample_tokens_filtered(xd, B.SPD_F32, rows, vocab, vocab, td, pd, kd, md, ud, tokens, ws)
    torch.cuda.synchronize()
    o = oracle.sample_tokens_filtered(x, t, top_p, u, top_k, min_p)
    compare_tokens(tokens.cpu().numpy(), o, u, vocab, allow_exempt_mismatch)


@pytest.mark.parametrize("vocab", VOCABS)
def test_fewer_than_k_within_64_octaves_of_the_maximum(dev, oracle, vocab):
    print(f"far below the maximum: vocab {vocab}", flush=True)
    rng = np.random.default_rng(vocab + 11)
    x = rng.uniform(-5.0, 5.0, (12, vocab)).astype(np.float32)
    x[np.arange(12), rng.integers(vocab // 2, vocab, 12)] = 60.0   # the others lie 79 to 94 octaves below
    x[4:6, : vocab // 3] = -np.inf
    top_k = np.array([5, 2, 40, 700, 5, 40, 5, 40, 3000, 5, 2, 700], np.int32)
    min_p = np.where(np.arange(12) >= 10, 1e-30, 0.0)
    u = np.where(np.arange(12) < 9, 0.0, rng.random(12))
    _check(oracle, x, 1.0, 1.0, top_k, min_p, u)


@pytest.mark.parametrize("maximum", [-0.5, 0.0, 0.2, 1.0])
@pytest.mark.parametrize("vocab", VOCABS)
def test_hundreds_of_equal_logits_at_the_kth_below_a_small_maximum(dev, oracle, vocab, maximum):
    print(f"ties at the k-th: vocab {vocab}, maximum {maximum}", flush=True)
    rng = np.random.default_rng(vocab + int(10 * maximum) + 100)
    rows = 18
    x = np.empty((rows, vocab), np.float32)
    top_k = np.empty(rows, np.int32)
    for r in range(rows):
        if r < 9:     # steps of 1, 1/2 and 1/4, the maximum subtracted
            step = (1.0, 0.5, 0.25)[r % 3]
            x[r] = np.round(rng.standard_normal(vocab) * 3.0 / step) * step
            top_k[r] = (vocab // 64, vocab // 26, vocab // 10)[r // 3]
            x[r] -= x[r].max()
        else:         # a thousand (513, 3000) ties and a heavy group just below them
            tied = (-3.3, -6.0, -10.0)[r % 3]
            where = rng.permutation(vocab)
            many = (513, 1000, 3000)[r // 3 - 3]
            x[r] = -30.0
            x[r, where[:many]] = tied
            x[r, where[many:many + 3000]] = tied - 0.25
            x[r, where[many + 3000]] = 0.0
            top_k[r] = 100
    x += np.float32(maximum)
    # Up to 32000 kept tokens a row: a uniform falls within 1e-7 (the rounding of an fp32 probability, 6e-8, and the sums') of a
    # boundary of the running mass in up to 2e-7 x 32000 = 0.6 % of the rows, 0.1 of the 18 at most; one has been seen, at 7e-10.
    _check(oracle, x, 1.0, 1.0, top_k, 0.0, rng.random(rows), allow_exempt_mismatch=1)
