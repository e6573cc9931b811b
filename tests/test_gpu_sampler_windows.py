"""The sampler's lists and windows where they can go wrong: rows whose slices differ so much that some window misses the
row's cut (they are read again), flat rows (the list does not begin at the top), cuts far down (more than one step of
binning), hundreds of equal logits at the cut (more than are told apart), slices that end inside a float4, and
vocabularies at the edge of what one slice holds or may list."""
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


@pytest.mark.parametrize("filters", [False, True])
@pytest.mark.parametrize("vocab", [5248, 5249, 16385, 40003, 131071, 131073])
def test_windows_that_miss_and_cuts_far_down(dev, oracle, vocab, filters):
    from paper_2502_02534_amd import binding as B
    rows = 24
    print(f"vocab {vocab}, filters {filters}", flush=True)
    rng = np.random.default_rng(vocab + 7)
    x = (rng.standard_normal((rows, vocab)) * 3.0).astype(np.float32)
    x[0:4] += np.linspace(4.0, -4.0, vocab, dtype=np.float32)      # falls over the vocabulary
    x[4:6, : vocab // 2] -= 12.0                                   # half of the slices far below
    x[6:9] *= np.array([0.05, 0.3, 0.5], np.float32)[:, None]      # flat
    x[9:11] = np.sort(x[9:11], axis=1)[:, ::-1]
    x[11, 3::7] = 2.0                                              # a seventh of the row equal
    x[12] = np.round(x[12])
    x[13, vocab // 3] += 30.0                                      # one logit holds the row
    x[14, -1] += 30.0                                              # ... the last one
    x[15] = np.float32(0.25)                                       # all equal
    t = rng.choice(np.array([0.2, 0.7, 1.0, 1.3], np.float32), rows)
    top_p = rng.choice(np.array([0.05, 0.9, 0.98], np.float32), rows)
    top_p[16:24] = [0.999, 0.9999, 0.99995, 0.999, 0.9999, 0.5, 0.01, 1.0]
    u = rng.random(rows, dtype=np.float32)
    top_k = rng.choice(np.array([0, 1, 600, 20000], np.int32), rows) if filters else None
    min_p = rng.choice(np.array([0.0, 1e-5, 0.3], np.float32), rows) if filters else None
    to = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.full((B.sample_tokens_workspace_size(rows, vocab),), 255, dtype=torch.uint8, device="cuda")
    tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    xd, td, pd, ud, kd, md = to(x), to(t), to(top_p), to(u), to(top_k), to(min_p)
    for _ in range(2):  # (the second time over the first's lists)
        B.sample_tokens_filtered(xd, B.SPD_F32, rows, vocab, vocab, td, pd, kd, md, ud, tokens, ws)
    torch.cuda.synchronize()
    o = oracle.sample_tokens_filtered(x, t, top_p, u, top_k, min_p) if filters else oracle.sample_tokens(x, t, top_p, u)
    compare_tokens(tokens.cpu().numpy(), o, u, vocab)


@pytest.mark.parametrize("filters", [False, True])
@pytest.mark.parametrize("rows, vocab", [(768, 5249), (769, 5249), (1025, 6144), (771, 40003)])
def test_more_rows_than_three_workgroups_a_cu(dev, oracle, rows, vocab, filters):
    from paper_2502_02534_amd import binding as B
    print(f"{rows} x {vocab}, filters {filters}", flush=True)
    rng = np.random.default_rng(rows + vocab)
    x = (rng.standard_normal((rows, vocab)) * rng.choice([0.3, 3.0], (rows, 1))).astype(np.float32)
    x[::97] += np.linspace(4.0, -4.0, vocab, dtype=np.float32)     # windows that miss
    t = rng.choice(np.array([0.0, 0.7, 1.0], np.float32), rows)
    top_p = rng.choice(np.array([0.5, 0.95, 1.0], np.float32), rows)
    u = rng.random(rows, dtype=np.float32)
    top_k = rng.choice(np.array([0, 1, 600], np.int32), rows) if filters else None
    min_p = rng.choice(np.array([0.0, 0.01], np.float32), rows) if filters else None
    to = lambda a: None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.full((B.sample_tokens_workspace_size(rows, vocab),), 255, dtype=torch.uint8, device="cuda")
    tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
    xd, td, pd, ud, kd, md = to(x), to(t), to(top_p), to(u), to(top_k), to(min_p)
    B.sample_tokens_filtered(xd, B.SPD_F32, rows, vocab, vocab, td, pd, kd, md, ud, tokens, ws)
    torch.cuda.synchronize()
    o = oracle.sample_tokens_filtered(x, t, top_p, u, top_k, min_p) if filters else oracle.sample_tokens(x, t, top_p, u)
    compare_tokens(tokens.cpu().numpy(), o, u, vocab)


@pytest.mark.parametrize("vocab", [9001, 32000, 128256, 262144])
def test_rows_read_again(dev, oracle, vocab):
    """Rows whose cut lies below some slices' lists or above their windows, by little or by much: the lists' own places are guesses
    from one slice each, and other slices hold more or less of the row."""
    from paper_2502_02534_amd import binding as B
    rows = 40
    print(f"rows read again: vocab {vocab}", flush=True)
    rng = np.random.default_rng(vocab + 3)
    x = rng.standard_normal((rows, vocab)).astype(np.float32)
    x *= np.repeat(np.array([3.0, 1.0, 2.5, 0.2], np.float32), 10)[:, None]
    fall = np.array([0, 2, 4, 6, 20, -2, -6, 0, 0, 0], np.float32)
    x += np.tile(fall, 4)[:, None] * np.linspace(1.0, 0.0, vocab, dtype=np.float32)
    for r in range(rows):
        if r % 10 == 7:       # fifty boosted tokens, in any slice
            x[r, rng.integers(0, vocab, 50)] += rng.uniform(2.0, 12.0, 50).astype(np.float32)
        elif r % 10 == 8:     # ... in the last one alone
            x[r, rng.integers(vocab - vocab // 9, vocab, 50)] += rng.uniform(2.0, 12.0, 50).astype(np.float32)
        elif r % 10 == 9:
            x[r] = np.sort(x[r])[::-1]
    one = np.ones(rows, np.float32)
    to = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
    ws = torch.full((B.sample_tokens_workspace_size(rows, vocab),), 255, dtype=torch.uint8, device="cuda")
    for share in (0.5, 0.9, 0.98, 0.9999):
        u = rng.random(rows, dtype=np.float32)
        tokens = torch.full((rows,), -7, dtype=torch.int32, device="cuda")
        xd, td, pd, ud = to(x), to(one), to(one * np.float32(share)), to(u)
        B.sample_tokens(xd, B.SPD_F32, rows, vocab, vocab, td, pd, ud, tokens, ws)
        torch.cuda.synchronize()
        # 160 rows in all, near a boundary by chance where tens of thousands of tokens are kept
        compare_tokens(tokens.cpu().numpy(), oracle.sample_tokens(x, one, one * np.float32(share), u), u, vocab)
