"""Logits of -inf (tokens that a caller has ruled out) have probability zero at every temperature and on every
path of the sampler: aligned and unaligned rows, short ones in one launch, whole slices of -inf, rows
without a cut, rows whose remaining logits are equal (more candidates than fit: the whole-row routine),
with and without filters."""
import numpy as np
import pytest

from gpu_checks import compare_tokens

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_02534_amd import binding, device
    binding.load()
    return device


# log2(e) / T is rounded up to a float at 0.4 and 0.7, down at 0.5 and 1.0
@pytest.mark.parametrize("temperature", [0.4, 0.5, 0.7, 1.0])
@pytest.mark.parametrize("filters", [False, True])
@pytest.mark.parametrize("vocab", [1000, 1001, 5001, 32003, 50256, 262144])
def test_masked_logits(dev, oracle, vocab, filters, temperature):
    from paper_2502_02534_amd import binding as B
    rows = 16 if vocab < 200000 else 6
    print(f"masked logits: vocab {vocab}, filters {filters}, T {temperature}", flush=True)
    rng = np.random.default_rng(vocab + int(10 * temperature))
    x = (rng.standard_normal((rows, vocab)) * 3.0).astype(np.float32)
    x[1::3, ::3] = -np.inf                   # every third
    x[2::3, vocab // 9:] = -np.inf           # all but the first ninth: whole slices
    x[4] = -np.inf                           # all but a few
    x[4, [7, vocab // 2, vocab - 1]] = [1.0, 2.0, 1.5]
    x[5] = 0.0                               # equal logits, half of them masked
    x[5, 1::2] = -np.inf
    t = np.full(rows, temperature, np.float32)
    top_p = np.full(rows, 0.95, np.float32)
    top_p[::4] = 1.0
    u = rng.random(rows, dtype=np.float32)
    top_k = rng.choice(np.array([0, 7, 300], np.int32), rows) if filters else None
    min_p = rng.choice(np.array([0.0, 0.05], np.float32), rows) if filters else None
    to = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.full((max(256, B.sample_tokens_workspace_size(rows, vocab)),), 255, dtype=torch.uint8, device="cuda")
    tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    xd, td, pd, ud, kd, md = to(x), to(t), to(top_p), to(u), to(top_k), to(min_p)
    B.sample_tokens_filtered(xd, B.SPD_F32, rows, vocab, vocab, td, pd, kd, md, ud, tokens, ws)
    torch.cuda.synchronize()
    got = tokens.cpu().numpy()
    assert np.all(np.isfinite(x[np.arange(rows), got]))       # never a masked token
    o = oracle.sample_tokens_filtered(x, t, top_p, u, top_k, min_p) if filters else oracle.sample_tokens(x, t, top_p, u)
    compare_tokens(got, o, u, vocab)
