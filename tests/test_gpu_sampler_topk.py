"""The k-th largest logit where it is hard to pin down: far below the maximum (more than 64 octaves of probability), on rows of
1, 2, 8 and 16 slices."""
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
