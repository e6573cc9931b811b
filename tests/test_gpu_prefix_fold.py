"""Two prefix splits by one workgroup: beside a suffix stream that lasts long enough (by the lengths on the device, not
by the call's bounds) the even splits take the odd ones' tokens too, which then hold nothing.  Both sides of that line,
odd numbers of splits, ragged prompts, more samples than lengths are summed."""
import numpy as np
import pytest

from gpu_checks import check_attention
from paper_2502_02534_amd import workloads as W

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    from paper_2502_02534_amd import binding, device
    binding.load()
    return device


# (query heads, KV heads, prompts, samples per prompt, prefix, suffix, bound, folded)
CASES = [(16, 8, 1, 9, (8500, 8500), (2500, 2600), 2600, True),     # 27 splits
         (16, 8, 1, 9, (8500, 8500), (0, 300), 2600, False),
         (16, 8, 2, 6, (3000, 8300), (3000, 3100), 3100, True),      # the shorter prompt ends inside a pair of splits
         (2, 1, 1, 600, (9000, 9000), (340, 380), 380, True),
         (2, 1, 1, 600, (9000, 9000), (100, 150), 380, False)]


@pytest.mark.parametrize("page", [0, 16])
@pytest.mark.parametrize("hq,hkv,prompts,spp,prefix,suffix,bound,folded", CASES)
def test_splits_folded_by_the_lengths(dev, oracle, hq, hkv, prompts, spp, prefix, suffix, bound, folded, page):
    from paper_2502_02534_amd import binding as B
    n = prompts * spp
    spec = W.small_spec(num_q_heads=hq, num_kv_heads=hkv, num_prompts=prompts, samples_per_prompt=spp, prefix_len=prefix,
                        suffix_len=(suffix[0], bound) if page == 0 else suffix, page_size=page)
    inp = W.make_attn_inputs(0, spec=spec, seed=2100 + n, poison_padding=page != 0)
    rng = np.random.default_rng(n)
    inp.suffix_lens[:] = np.minimum(inp.suffix_lens, rng.integers(suffix[0], suffix[1] + 1, n))
    inp.max_suffix_len = bound
    print(f"{prompts} x {spp} samples, prefix {prefix}, suffix {suffix} of {bound}, page {page}", flush=True)
    rows = np.sort(rng.choice(n * hq, min(n * hq, 96), replace=False))
    check_attention(dev, oracle, inp, rows=rows)

    d = dev.upload_attn(inp)
    d.run()
    torch.cuda.synchronize()
    _, splits, _, chunks = B.spd_attn_plan(d.desc, inp.max_prefix_len, bound)
    slots = splits + chunks
    at = (n * hq * slots * 128 * 4 + 255) // 256 * 256
    ml = d.workspace[at:at + n * hq * slots * 8].view(torch.float32).reshape(n * hq, slots, 2)
    assert splits >= 2 and bool((ml[:, 0, 1] > 0).all())
    assert bool((ml[:, 1, 1] > 0).all()) != folded and bool((ml[:, 1, 1] == 0).all()) == folded
    # the stages one call at a time: the same bits
    full, lse = d.out.clone(), d.lse.clone()
    d.out.zero_()
    d.workspace.fill_(255)
    for stage in (B.STAGE_PREFIX, B.STAGE_SUFFIX, B.STAGE_MERGE):
        d.run(stage)
    torch.cuda.synchronize()
    assert torch.equal(full.view(torch.int16), d.out.view(torch.int16)) and torch.equal(lse, d.lse)
