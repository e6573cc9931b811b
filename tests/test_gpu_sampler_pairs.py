"""The row-level sampler step at the edges of how it shares its work out: every number of slices that a row is cut
into (one, two, four or eight wavefronts per slice, two slices per wavefront), sorted rows (all that is kept
in the first slices), and the cut among 3, 64, 65 or 700 equal logits (told apart directly, settled by their value and
count, or by those and a second look at the lists for what every slice keeps)."""
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


# 1, 2, 3, 4, 5, 7, 8, 13 and 16 slices
@pytest.mark.parametrize("filters", [False, True])
@pytest.mark.parametrize("vocab", [8000, 9000, 13001, 17000, 21003, 29000, 50256, 200000, 262144])
def test_slices_sorted_rows_and_ties_at_the_cut(dev, oracle, vocab, filters):
    from paper_2502_02534_amd import binding as B
    rows = 24
    print(f"vocab {vocab}, filters {filters}", flush=True)
    rng = np.random.default_rng(vocab)
    x = (rng.standard_normal((rows, vocab)) * 3.0).astype(np.float32)
    x[4:8] = np.sort(x[4:8], axis=1)[:, ::-1]            # descending, ascending
    x[8:12] = np.sort(x[8:12], axis=1)
    t = rng.choice(np.array([0.3, 0.7, 1.0, 1.2], np.float32), rows)
    top_p = rng.choice(np.array([0.5, 0.9, 0.98], np.float32), rows)
    for r, ties in zip(range(12, 20), (3, 64, 65, 700) * 2):
        # half the mass above the ties, which hold three tenths of the rest; others of the same bin around them
        x[r] = -30.0
        where = rng.permutation(vocab)
        x[r, where[:ties]] = 4.0
        x[r, where[ties]] = np.float32(4.0 + np.log(max(ties, 2)))
        x[r, where[ties + 1:ties + 41]] = 4.0 + rng.uniform(-0.03, 0.03, 40).astype(np.float32)
        x[r, where[ties + 41:ties + 61]] = rng.uniform(0.0, 3.0, 20).astype(np.float32)
        if r >= 16:
            x[r] = np.sort(x[r])
        t[r], top_p[r] = 1.0, 0.7
    u = rng.random(rows, dtype=np.float32)
    top_k = rng.choice(np.array([0, 5, 400], np.int32), rows) if filters else None
    min_p = rng.choice(np.array([0.0, 0.02], np.float32), rows) if filters else None
    to = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.full((B.sample_tokens_workspace_size(rows, vocab),), 255, dtype=torch.uint8, device="cuda")
    tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    xd, td, pd, ud, kd, md = to(x), to(t), to(top_p), to(u), to(top_k), to(min_p)
    B.sample_tokens_filtered(xd, B.SPD_F32, rows, vocab, vocab, td, pd, kd, md, ud, tokens, ws)
    torch.cuda.synchronize()
    o = oracle.sample_tokens_filtered(x, t, top_p, u, top_k, min_p) if filters else oracle.sample_tokens(x, t, top_p, u)
    compare_tokens(tokens.cpu().numpy(), o, u, vocab)


@pytest.mark.parametrize("filters", [False, True])
@pytest.mark.parametrize("vocab", [50257, 128256])
def test_the_same_call_returns_the_same_tokens(dev, oracle, vocab, filters):
    """Uniforms next to the boundaries of the running mass, on rows of long lists whose order differs from call to call: what is
    summed in 64 bits moves by 1e-16 with it, the nearest uniform is 3e-8 away."""
    from paper_2502_02534_amd import binding as B
    rows = 64
    print(f"the same call again: vocab {vocab}, filters {filters}", flush=True)
    rng = np.random.default_rng(vocab + 17)
    x = (rng.standard_normal((rows, vocab)) * 2.0).astype(np.float32)
    x[::4] += np.linspace(5.0, 0.0, vocab, dtype=np.float32)        # some slices are read again
    one = np.ones(rows, np.float32)
    top_p, top_k = one * np.float32(0.9), np.full(rows, 3000, np.int32) if filters else None
    u = rng.random(rows, dtype=np.float32)
    o = oracle.sample_tokens_filtered(x, one, top_p, u, top_k, None) if filters else oracle.sample_tokens(x, one, top_p, u)
    u = np.minimum(o["cdf_hi"].astype(np.float32), np.float32(1.0 - 2.0 ** -24))
    to = lambda a: None if a is None else torch.from_numpy(a).cuda()
    xd, td, pd, ud, kd = to(x), to(one), to(top_p), to(u), to(top_k)
    ws = torch.empty(B.sample_tokens_workspace_size(rows, vocab), dtype=torch.uint8, device="cuda")
    tokens = torch.full((12, rows), -7, dtype=torch.int32, device="cuda")
    for i in range(12):
        ws.fill_(255 if i % 2 else 127)
        B.sample_tokens_filtered(xd, B.SPD_F32, rows, vocab, vocab, td, pd, kd, None, ud, tokens[i], ws)
    torch.cuda.synchronize()
    assert bool((tokens == tokens[0]).all()) and bool((tokens >= 0).all())
