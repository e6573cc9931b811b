"""The general attention kernel (fp32, head dimensions other than 128, more than 16 query heads per KV
head) at the sizes where its tiling can go wrong: padded head dimensions, row counts either side
of its 16- and 32-row blocks, ranges either side of its 16- and 32-token tiles, items shared by a
workgroup's wavefronts and items of one wavefront."""
import numpy as np
import pytest

from gpu_checks import check_attention
from paper_2502_02534_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

CASES = [
    # padded head dimensions (registers for 64, 128 or 256 channels), both types, contiguous and paged
    dict(dtype="f32", num_q_heads=2, num_kv_heads=1, head_dim=8, prefix_len=(17, 17), suffix_len=(0, 16)),
    dict(dtype="f32", num_q_heads=6, num_kv_heads=2, head_dim=72, prefix_len=(1, 130), suffix_len=(0, 65), page_size=16),
    dict(dtype="f32", num_q_heads=4, num_kv_heads=2, head_dim=200, prefix_len=(15, 90), suffix_len=(1, 33)),
    dict(dtype="f32", num_q_heads=4, num_kv_heads=2, head_dim=256, prefix_len=(63, 200), suffix_len=(0, 64), page_size=16),
    dict(dtype="bf16", num_q_heads=4, num_kv_heads=2, head_dim=40, prefix_len=(31, 140), suffix_len=(0, 33), page_size=16),
    dict(dtype="bf16", num_q_heads=6, num_kv_heads=2, head_dim=96, prefix_len=(1, 300), suffix_len=(0, 97)),
    dict(dtype="bf16", num_q_heads=4, num_kv_heads=2, head_dim=136, prefix_len=(65, 300), suffix_len=(1, 31)),
    dict(dtype="bf16", num_q_heads=8, num_kv_heads=2, head_dim=256, prefix_len=(1, 200), suffix_len=(0, 70), page_size=16),
    # one row, exactly one block, one more than a block, one more than two
    dict(dtype="f32", num_q_heads=1, num_kv_heads=1, head_dim=64, samples_per_prompt=1, prefix_len=(64, 64), suffix_len=(1, 1)),
    dict(dtype="f32", num_q_heads=4, num_kv_heads=1, head_dim=128, samples_per_prompt=4, prefix_len=(65, 65), suffix_len=(0, 3)),
    dict(dtype="bf16", num_q_heads=2, num_kv_heads=2, head_dim=64, samples_per_prompt=17, prefix_len=(129, 129), suffix_len=(0, 129)),
    dict(dtype="bf16", num_q_heads=3, num_kv_heads=1, head_dim=64, samples_per_prompt=11, prefix_len=(127, 127), suffix_len=(0, 33)),
    # more than 16 heads per KV head: suffix rows in several blocks (with head_dim 128 the prefix stays on its own kernel)
    dict(dtype="bf16", num_q_heads=24, num_kv_heads=1, head_dim=128, samples_per_prompt=5, prefix_len=(1, 300), suffix_len=(0, 200)),
    dict(dtype="bf16", num_q_heads=66, num_kv_heads=2, head_dim=64, samples_per_prompt=3, prefix_len=(1, 90), suffix_len=(0, 70), page_size=16),
    # one wavefront per suffix item (the first; its 504 prefix items are shared by four), per item of both kinds (the second)
    dict(dtype="f32", num_q_heads=8, num_kv_heads=4, head_dim=64, num_prompts=3, samples_per_prompt=333, prefix_len=(30, 70), suffix_len=(0, 20)),
    dict(dtype="bf16", num_q_heads=32, num_kv_heads=16, head_dim=64, num_prompts=9, samples_per_prompt=131, prefix_len=(0, 150), suffix_len=(0, 17),
         page_size=16),
]


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_02534_amd import binding, device
    binding.load()
    return device


@pytest.mark.parametrize("i", range(len(CASES)))
def test_general_kernel_shapes(dev, oracle, i):
    spec = dict(num_prompts=2, samples_per_prompt=3)
    spec.update(CASES[i])
    print(f"general kernel case {i}: {spec}", flush=True)
    check_attention(dev, oracle, W.make_attn_inputs(0, spec=W.small_spec(**spec), seed=900 + i, poison_padding=True))


@pytest.mark.parametrize("shared", [True, False], ids=["shared", "single"])
def test_tokens_with_minus_infinity_scores_add_nothing(dev, shared):
    """Keys whose score is -inf for every row, whole tiles of them at the start and in the middle of the prompt: the
    result is attention over the others (fp32: nothing but the order of the sums differs, 1e-5).  Prefix items
    are shared here, so a wavefront holds one tile; suffix items are shared or not, as the ids say (several
    tiles of one wavefront: test_tiles_of_minus_infinity_in_one_wavefront)."""
    spec = W.small_spec(dtype="f32", num_q_heads=4, num_kv_heads=4, head_dim=64, samples_per_prompt=400 if not shared else 5,
                        prefix_len=(200, 200), suffix_len=(40, 40))
    inp = W.make_attn_inputs(0, spec=spec, seed=950)
    inp.q[..., 0] = 1.0
    inp.k_prefix[:70, :, 0] = -np.inf
    inp.k_prefix[100:140, :, 0] = -np.inf
    inp.k_suffix[:, 3, :, 0] = -np.inf
    d = dev.upload_attn(inp)
    d.run()
    torch.cuda.synchronize()
    kept = np.r_[70:100, 140:200]
    k = np.concatenate([np.broadcast_to(inp.k_prefix[kept][None], (spec.num_samples,) + inp.k_prefix[kept].shape),
                        np.delete(inp.k_suffix, 3, axis=1)], axis=1).astype(np.float64)
    v = np.concatenate([np.broadcast_to(inp.v_prefix[kept][None], (spec.num_samples,) + inp.v_prefix[kept].shape),
                        np.delete(inp.v_suffix, 3, axis=1)], axis=1).astype(np.float64)
    s = np.einsum("nhd,nthd->nht", inp.q.astype(np.float64), k) / 8.0
    w = np.exp(s - s.max(-1, keepdims=True))
    ref = np.einsum("nht,nthd->nhd", w / w.sum(-1, keepdims=True), v)
    got = d.out.cpu().numpy()
    assert np.all(np.abs(got - ref) <= 1e-5 * np.abs(ref) + 1e-6)


@pytest.mark.parametrize("side", ["prefix", "suffix"])
@pytest.mark.parametrize("d", [64, 96, 256])
def test_bf16_inputs_keep_fp32_probabilities(dev, d, side):
    """Three values per channel that cancel to 2^-18 of their size: what is left shows the probabilities'
    own error.  Bound: fp32 probabilities are good to 2^-21 (the exponent, below 4 in magnitude, is
    rounded a few times at 2^-24, the exponential once at 2^-23) and the products are added in fp32, so
    2^-20 of sum p |v| / sum p covers them; beside it the result's roundings to fp16 and bf16, 2^-8 of the
    result and 2^-24 (fp16's smallest step)."""
    n, g = 5, 7
    rng = np.random.default_rng(d)
    spec = W.small_spec(dtype="bf16", num_q_heads=g, num_kv_heads=1, head_dim=d, num_prompts=1, samples_per_prompt=n,
                        prefix_len=(3, 3) if side == "prefix" else (0, 0), suffix_len=(0, 0) if side == "prefix" else (3, 3))
    inp = W.make_attn_inputs(0, spec=spec, seed=77)
    as_f64 = lambda bits: W.bf16_bits_to_f32(bits).astype(np.float64)
    inp.q[:] = W.f32_to_bf16_bits(rng.standard_normal(d).astype(np.float32))      # one query for all rows
    k = inp.k_prefix if side == "prefix" else inp.k_suffix.reshape(n * 3, 1, d)
    v = inp.v_prefix if side == "prefix" else inp.v_suffix.reshape(n * 3, 1, d)
    ref, mass = np.empty((n, d)), np.empty((n, d))
    for a in range(0, k.shape[0], 3):
        s = as_f64(k[a:a + 3, 0]) @ as_f64(inp.q[0, 0]) / np.sqrt(d)
        p = np.exp(s - s.max())
        left = np.zeros(d)
        for t in range(3):
            if t == 0:
                want = rng.uniform(100.0, 200.0, d).astype(np.float32)
            else:
                want = (-left / p[t]).astype(np.float32)
            v[a + t, 0] = W.f32_to_bf16_bits(want)
            left = left + p[t] * as_f64(v[a + t, 0])
        out, size = left / p.sum(), (p[:, None] * np.abs(as_f64(v[a:a + 3, 0]))).sum(0) / p.sum()
        sample = slice(None) if side == "prefix" else a // 3
        ref[sample], mass[sample] = out, size
    x = dev.upload_attn(inp)
    x.run()
    torch.cuda.synchronize()
    err = np.abs(x.out.float().cpu().numpy().astype(np.float64) - ref[:, None, :])
    assert np.abs(ref).max() < 2.0 ** -15 * mass.max()        # the values do cancel
    bound = 2.0 ** -20 * mass + 2.0 ** -8 * np.abs(ref) + 2.0 ** -24
    print(f"{side} {d}: error / bound at most {(err / bound[:, None, :]).max():.3f}", flush=True)
    assert np.all(err <= bound[:, None, :])


@pytest.mark.parametrize("d,page", [(64, 0), (64, 16), (128, 0), (200, 16)])
def test_an_infinite_value_stays_in_its_channel(dev, d, page):
    """fp32 values have no range limit: an infinite value in the last token of a range that ends inside a
    tile gives an infinite output in its own channel and leaves the other channels alone (1e-5: the
    order of the sums)."""
    spec = W.small_spec(dtype="f32", num_q_heads=4, num_kv_heads=2, head_dim=d, samples_per_prompt=5, prefix_len=(21, 21),
                        suffix_len=(7, 7), page_size=page)
    inp = W.make_attn_inputs(0, spec=spec, seed=960)
    plain = dev.upload_attn(inp)
    plain.run()

    def row(v, side, seq, t):   # [2 heads, d] view of token t
        if not page:
            return v[t] if side == "prefix" else v[seq, t]
        indptr = inp.prefix_indptr if side == "prefix" else inp.suffix_page_indptr
        pages = inp.prefix_page_indices if side == "prefix" else inp.suffix_page_indices
        return v[pages[indptr[seq] + t // page], :, t % page]

    row(inp.v_prefix, "prefix", 0, 20)[0, 3] = np.inf
    for n in range(5):
        row(inp.v_suffix, "suffix", n, 6)[1, d - 1] = -np.inf
    x = dev.upload_attn(inp)
    x.run()
    torch.cuda.synchronize()
    got, ref = x.out.cpu().numpy(), plain.out.cpu().numpy().copy()
    ref[:, :2, 3], ref[:, 2:, d - 1] = np.inf, -np.inf
    assert np.array_equal(np.isinf(got), np.isinf(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    fin = np.isfinite(ref)
    assert np.all(np.abs(got[fin] - ref[fin]) <= 1e-5 * np.abs(ref[fin]) + 1e-6)


# Shapes whose plan gives a wavefront several tiles: enough (split, prompt, KV head) items that a split is not cut
# and not shared, or shared by two.  (spec, prefix: wavefronts per item and tiles, suffix: the same)
MANY_TILES = [
    (dict(dtype="f32", num_q_heads=16, num_kv_heads=16, head_dim=24, num_prompts=65, samples_per_prompt=3, prefix_len=(200, 200),
          suffix_len=(190, 190)), (1, 13), (1, 12)),
    (dict(dtype="f32", num_q_heads=16, num_kv_heads=16, head_dim=64, num_prompts=40, samples_per_prompt=1, prefix_len=(200, 200),
          suffix_len=(60, 60)), (2, 13), (2, 4)),
    (dict(dtype="f32", num_q_heads=32, num_kv_heads=32, head_dim=64, num_prompts=33, samples_per_prompt=17, prefix_len=(200, 200),
          suffix_len=(20, 20)), (1, 13), (1, 2)),
    (dict(dtype="bf16", num_q_heads=16, num_kv_heads=16, head_dim=64, num_prompts=65, samples_per_prompt=3, prefix_len=(200, 200),
          suffix_len=(60, 60)), (1, 7), (1, 2)),
    (dict(dtype="bf16", num_q_heads=32, num_kv_heads=32, head_dim=64, num_prompts=33, samples_per_prompt=17, prefix_len=(200, 200),
          suffix_len=(20, 20)), (1, 7), (1, 1)),
    (dict(dtype="bf16", num_q_heads=16, num_kv_heads=16, head_dim=200, num_prompts=65, samples_per_prompt=1, prefix_len=(200, 200),
          suffix_len=(180, 180)), (1, 7), (1, 3)),
]


def tiles_of_a_wavefront(spec, lens):
    """(wavefronts per item, tiles of an item) of the prefix and the suffix items, as the launch shares them out."""
    from paper_2502_02534_amd import binding as B
    tile = 16 if spec.dtype == "f32" else 32
    g = spec.num_q_heads // spec.num_kv_heads
    desc = B.make_desc(dtype=B.SPD_F32 if spec.dtype == "f32" else B.SPD_BF16, num_q_heads=spec.num_q_heads,
                       num_kv_heads=spec.num_kv_heads, head_dim=spec.head_dim, num_prompts=spec.num_prompts,
                       num_samples=spec.num_samples, max_samples_per_prompt=spec.samples_per_prompt)
    split, splits, chunk, chunks = B.spd_attn_plan(desc, *lens)
    rows = spec.samples_per_prompt * g
    block = 32 if rows > 16 and spec.head_dim <= 64 else 16
    places = 1024 if spec.head_dim > 128 else 2048

    def share(items, tiles):
        n = 1
        while 2 * n <= 4 and 2 * n <= tiles and items * n * 2 <= places:
            n *= 2
        return n

    prefix_items = -(-rows // block) * splits * spec.num_prompts * spec.num_kv_heads
    suffix_items = -(-g // 16) * spec.num_kv_heads * chunks * spec.num_samples
    return ((share(prefix_items, split // tile), -(-min(split, lens[0]) // tile)),
            (share(suffix_items, chunk // tile), -(-min(chunk, lens[1]) // tile)))


@pytest.mark.parametrize("place", ["second", "last"])
@pytest.mark.parametrize("i", range(len(MANY_TILES)))
def test_the_reference_maximum_is_raised_in_a_wavefronts_later_tiles(dev, oracle, i, place):
    """A key twenty times as long as the others in the second or the last tile of a wavefront: scores that exceed the
    first tile's by more than the ten octaves up to which the reference stands make the kernel rescale what it
    has, in the prefix and in the suffix (asserted, as is the number of tiles)."""
    kw, prefix_tiles, suffix_tiles = MANY_TILES[i]
    spec = W.small_spec(**kw)
    lens = (spec.prefix_len[1], spec.suffix_len[1])
    assert tiles_of_a_wavefront(spec, lens) == (prefix_tiles, suffix_tiles)
    tile = 16 if spec.dtype == "f32" else 32
    inp = W.make_attn_inputs(0, spec=spec, seed=970 + i)
    d, hkv, n = spec.head_dim, spec.num_kv_heads, spec.num_samples
    g = spec.num_q_heads // hkv
    f32 = (lambda a: a) if spec.dtype == "f32" else W.bf16_bits_to_f32
    own = (lambda a: a) if spec.dtype == "f32" else W.f32_to_bf16_bits
    late = {}
    for side, k, length, (share, tiles) in (("prefix", inp.k_prefix.reshape(-1, lens[0], hkv, d), lens[0], prefix_tiles),
                                            ("suffix", inp.k_suffix, lens[1], suffix_tiles)):
        if tiles <= share:
            continue  # one tile per wavefront
        first_chunk = min(length, tiles * tile)
        at = share * tile + 3 if place == "second" else first_chunk - 2
        k[:, at] = own(f32(k[:, at]) * 20)
        part = at // tile % share                     # the wavefront that takes this tile, and its first one
        late[side] = (at, part * tile)
    rows = np.sort(np.random.default_rng(i).choice(n * spec.num_q_heads, 128, replace=False))
    largest = np.zeros(len(rows))                     # score of each row, as an exponent of e
    for side, (at, first) in late.items():            # the reference does have to be raised
        raised = 0
        for x, r in enumerate(rows):
            s, h = divmod(int(r), spec.num_q_heads)
            k = inp.k_prefix.reshape(-1, lens[0], hkv, d)[s // spec.samples_per_prompt] if side == "prefix" else inp.k_suffix[s]
            sc = f32(np.ascontiguousarray(k[:, h // g])) @ f32(inp.q[s, h]) / np.sqrt(d) * np.log2(np.e)
            raised += sc[at] - sc[first:first + tile].max() > 10.1
            largest[x] = max(largest[x], np.abs(sc).max() * np.log(2))
        assert raised >= 16, (side, raised)
    assert "prefix" in late
    print(f"late keys {late}, {spec.dtype} {d}", flush=True)
    if spec.dtype == "bf16":
        check_attention(dev, oracle, inp, rows=rows)
        return
    # fp32: a score of up to 100 is itself good to a few roundings (2^-24 of it each, eight are allowed), which is the
    # relative error of its probability, so of the result: that much of the largest value, beside the usual bound
    x = dev.upload_attn(inp)
    x.run()
    torch.cuda.synchronize()
    got, (ref, ref_lse) = x.out.cpu().numpy().astype(np.float64).reshape(-1, d)[rows], oracle.attention_inputs(inp, rows=rows)
    bound = 1e-5 * np.abs(ref) + 1e-6 + (2.0 ** -21 * largest * np.abs(inp.v_prefix).max())[:, None]
    assert np.all(np.abs(got - ref) <= bound), (np.abs(got - ref) / bound).max()
    assert np.all(np.abs(x.lse.cpu().numpy().reshape(-1)[rows] - ref_lse) <= 1e-4)


@pytest.mark.parametrize("i", [0, 1, 2])
def test_tiles_of_minus_infinity_in_one_wavefront(dev, i):
    """fp32: a wavefront's first two tiles and one in the middle hold nothing but scores of -inf, in the prefix and
    (where a wavefront has as many tiles) in the suffix; the result is attention over the other tokens (1e-5: the
    order of the sums)."""
    kw, prefix_tiles, suffix_tiles = MANY_TILES[i]
    spec = W.small_spec(**kw)
    lens = (spec.prefix_len[1], spec.suffix_len[1])
    assert tiles_of_a_wavefront(spec, lens) == (prefix_tiles, suffix_tiles)
    inp = W.make_attn_inputs(0, spec=spec, seed=990 + i)
    d, hkv, per = spec.head_dim, spec.num_kv_heads, spec.samples_per_prompt
    g = spec.num_q_heads // hkv
    inp.q[..., 0] = 1.0
    kept = {}
    for side, k, length, (share, tiles) in (("prefix", inp.k_prefix.reshape(-1, lens[0], hkv, d), lens[0], prefix_tiles),
                                            ("suffix", inp.k_suffix, lens[1], suffix_tiles)):
        out = np.zeros(length, bool)
        out[:16 * min(2 * share, tiles - 1)] = True
        if tiles > 4 * share:
            out[16 * 3 * share:16 * 4 * share] = True
        k[:, out, :, 0] = -np.inf
        kept[side] = ~out
    x = dev.upload_attn(inp)
    x.run()
    torch.cuda.synchronize()
    got = x.out.cpu().numpy()
    rng = np.random.default_rng(i)
    for r in rng.choice(spec.num_samples * spec.num_q_heads, 96, replace=False):
        s, h = divmod(int(r), spec.num_q_heads)
        pre = slice((s // per) * lens[0], (s // per + 1) * lens[0])
        k = np.concatenate([inp.k_prefix[pre, h // g][kept["prefix"]], inp.k_suffix[s, :, h // g][kept["suffix"]]]).astype(np.float64)
        v = np.concatenate([inp.v_prefix[pre, h // g][kept["prefix"]], inp.v_suffix[s, :, h // g][kept["suffix"]]]).astype(np.float64)
        sc = k @ inp.q[s, h].astype(np.float64) / np.sqrt(d)
        w = np.exp(sc - sc.max())
        ref = (w / w.sum()) @ v
        assert np.all(np.abs(got[s, h] - ref) <= 1e-5 * np.abs(ref) + 1e-6), (s, h)
