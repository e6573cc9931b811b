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
