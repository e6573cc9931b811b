"""The size functions report enough for every smaller call too: a program that allocates once, for its
largest batch and longest lengths, is never refused a smaller one (general kernel: fp32, or head
dimensions other than 128); on the tiled path (bf16, 128 channels) they report the finest plan of the call itself.  Host
arithmetic, no GPU."""
import os
import random

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

TILED = [(1, 32, 8, 128), (1, 64, 8, 128), (1, 8, 8, 128), (1, 32, 1, 128)]
SHAPES = [(0, 32, 8, 128), (0, 4, 1, 64), (0, 8, 8, 256), (1, 8, 8, 256), (1, 32, 8, 64), (1, 24, 1, 96), (0, 1, 1, 8)]


@pytest.fixture(scope="module")
def B():
    from paper_2502_02534_amd import binding
    if not os.path.exists(binding.LIB_PATH):
        import __graft_entry__
        __graft_entry__.build()
    binding.load()
    return binding


def up(n):
    return (n + 255) // 256 * 256


def need(B, desc, max_prefix, max_suffix):
    """What the call itself asks for (the slots of its plan)."""
    _, splits, _, chunks = B.spd_attn_plan(desc, max_prefix, max_suffix)
    rows = (splits + chunks) * desc.num_samples * desc.num_q_heads
    return up(rows * desc.head_dim * 4) + up(rows * 8) + 256


def make(B, shape, n, prompts=1):
    dtype, hq, hkv, d = shape
    return B.make_desc(dtype=dtype, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_prompts=prompts, num_samples=n,
                       max_samples_per_prompt=(n + prompts - 1) // prompts)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("max_prefix,max_suffix", [(8192, 1024), (300, 40), (0, 2048), (100000, 30000)])
def test_the_largest_batch_serves_the_smaller_ones(B, shape, max_prefix, max_suffix):
    most, largest = 0, 0
    for n in range(1, 257):
        size = B.shared_prefix_decode_attn_workspace_size(make(B, shape, n), max_prefix, max_suffix)
        own = need(B, make(B, shape, n), max_prefix, max_suffix)
        assert size >= own
        assert size >= most, (n, size, most)      # never below a smaller batch's
        most = size
        largest = max(largest, own)
        assert size <= 1.5 * largest              # nor far above the most that a batch of up to n samples needs


@pytest.mark.parametrize("shape", SHAPES)
def test_fewer_samples_other_groupings_and_shorter_lengths_fit(B, shape):
    rng = random.Random(shape[3] + shape[1])
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    for _ in range(400):
        n, lp, ls = log(1, 3000), log(1, 200000), log(1, 50000)
        size = B.shared_prefix_decode_attn_workspace_size(make(B, shape, n, rng.randint(1, min(n, 9))), lp, ls)
        for _ in range(20):
            m = log(1, n)
            small = make(B, shape, m, rng.randint(1, min(m, 9)))
            p, s = log(1, lp) if rng.random() < 0.8 else lp, log(1, ls) if rng.random() < 0.8 else ls
            assert need(B, small, p, s) <= size, (n, lp, ls, m, small.num_prompts, p, s)


@pytest.mark.parametrize("shape", SHAPES)
def test_trees_of_prefixes_too(B, shape):
    rng = random.Random(5)
    dtype, hq, hkv, d = shape

    def size(n, levels, max_suffix):
        arr = (B.PrefixLevel * len(levels))()
        for i, (groups, length) in enumerate(levels):
            arr[i] = B.PrefixLevel(256, 256, 256, 256, 0, 256, groups, (n + groups - 1) // groups, length)
        desc = make(B, shape, n)
        return B.shared_prefix_decode_attn_levels_workspace_size(desc, arr, max_suffix)

    for _ in range(100):
        lens = [rng.randint(1, 9000) for _ in range(rng.randint(1, 4))]
        ls, n = rng.randint(1, 3000), rng.randint(1, 600)
        big = size(n, [(rng.randint(1, n), x) for x in lens], ls)
        for _ in range(10):
            m = rng.randint(1, n)
            small = size(m, [(rng.randint(1, m), rng.randint(1, x)) for x in lens], rng.randint(1, ls))
            assert 0 < small <= big, (n, lens, ls, m)


def finest(shape, n, prompts, max_prefix, max_suffix):
    """Slots of a tiled call in the finest plan: prefix splits for a workgroup per CU, chunks for a wavefront place each."""
    _, hq, hkv, _ = shape
    spp = (n + prompts - 1) // prompts
    base = prompts * hkv * -(-spp * (hq // hkv) // 128)
    split = max(128, up64(-(-max_prefix // min(64, -(-256 // base)))))
    pairs = n * hkv
    chunk = min(320, max(64, up64(-(-max_suffix // -(-2048 // pairs)))))
    chunk = {128: 96, 256: 192}.get(chunk, chunk)
    if max_suffix > 64 * chunk:
        chunk = up64(-(-max_suffix // 64))
    return -(-max_prefix // split) + -(-max_suffix // chunk)


def up64(n):
    return (n + 63) // 64 * 64


@pytest.mark.parametrize("shape", TILED)
def test_tiled_calls_report_their_finest_plan_and_need_no_more(B, shape):
    rng = random.Random(shape[1] * 7 + shape[2])
    log = lambda lo, hi: int(round(lo * (hi / lo) ** rng.random()))
    pairs = [1535, 1536, 1537, 2047, 2048, 2049, 1023, 1024, 767]
    lengths = [0, 63, 95, 96, 97, 128, 129, 192, 193, 255, 256, 257, 383, 385, 767, 768, 769, 1024, 4096, 4097, 6000, 20480, 20481, 46080, 47104]
    for i in range(4000):
        n = max(1, rng.choice(pairs) // shape[2]) if i % 3 == 0 else log(1, 3000)
        prompts = rng.randint(1, min(n, 9))
        lp, ls = log(1, 200000), rng.choice(lengths) if i % 2 == 0 else log(1, 50000)
        desc = make(B, shape, n, prompts)
        rows = finest(shape, n, prompts, lp, ls) * n * shape[1]
        size = B.shared_prefix_decode_attn_workspace_size(desc, lp, ls)
        assert size == up(rows * 512) + up(rows * 8) + 256, (n, prompts, lp, ls)
        assert need(B, desc, lp, ls) <= size, (n, prompts, lp, ls)
