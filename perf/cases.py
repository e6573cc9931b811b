"""Performance cases: the work a user of this library has it do, through its public entry points.

Four kinds of case, each a dict of plain values:

  attn    one decode-attention call (`shared_prefix_decode_attn`): N samples over their prompt's shared
          KV and their own suffix; fp32 or bf16, head_dim 64 or 128, contiguous or paged KV
  tree    one call over a tree of shared prefixes (`shared_prefix_decode_attn_levels`)
  sample  one next-token sampling call (`sample_tokens`, or `sample_tokens_filtered` with top-k / min-p)
  loop    a run of decode steps with KV append (`DecodeLoop`, one captured step replayed): the
          generation loop itself, with its per-step launches

Sizes are those of the library's own configurations (`workloads.SPECS`) and tests, or generic.
"""
import math

import torch

from paper_2502_02534_amd import binding as B
from paper_2502_02534_amd import device as D

DEV = "cuda:0"


# ---- the cases ----------------------------------------------------------------------------------------

def _attn(name, dtype, hq, hkv, d, prompts, spp, prefix, suffix, page=0):
    return {"name": name, "kind": "attn", "dtype": dtype, "hq": hq, "hkv": hkv, "d": d, "prompts": prompts, "spp": spp,
            "prefix_lo": prefix[0], "prefix_hi": prefix[1], "suffix_lo": suffix[0], "suffix_hi": suffix[1], "page": page}


def _sample(name, rows, vocab, sigma, t, top_p, boosted=0, greedy_every=0, uncut_every=0, filters=0):
    return {"name": name, "kind": "sample", "rows": rows, "vocab": vocab, "sigma": sigma, "t_lo": t[0], "t_hi": t[1],
            "top_p": top_p, "boosted": boosted, "greedy_every": greedy_every, "uncut_every": uncut_every,
            "filters": filters}


def listed():
    return [
        # the smallest call: four samples of a short prompt, fp32 (configuration 1), all latency
        _attn("attn-f32-n4", "f32", 4, 1, 64, 1, 4, (256, 256), (32, 32)),
        # fp32 at a model's geometry: what a program that checks its numerics in fp32 runs
        _attn("attn-f32-n16", "f32", 32, 8, 128, 1, 16, (2048, 2048), (0, 256)),
        # an ordinary small batch: 16 samples of a 2k prompt (configuration 2)
        _attn("attn-n16-2k", "bf16", 32, 8, 128, 1, 16, (2048, 2048), (256, 256)),
        # the sampling job of 64 completions of one 8k prompt, up to 1024 generated tokens (configuration 3)
        _attn("attn-n64-8k", "bf16", 32, 8, 128, 1, 64, (8192, 8192), (128, 1024)),
        # one layer of a large model (64 query heads, G = 8) over a 16k prompt (configuration 4)
        _attn("attn-n32-16k-g8", "bf16", 64, 8, 128, 1, 32, (16384, 16384), (512, 512)),
        # a model with 64-channel heads, several prompts of odd lengths, paged KV
        _attn("attn-d64-paged", "bf16", 32, 8, 64, 3, 21, (500, 4001), (1, 501), page=16),
        # a serving batch: 8 prompts x 128 samples, ragged, paged KV (configuration 5), the largest call
        _attn("attn-paged-n1024", "bf16", 32, 8, 128, 8, 128, (1024, 16384), (0, 2048), page=16),
        # a tree of prompts: base prompt, demonstrations, 26 tasks of 16 samples each
        {"name": "tree-26x16", "kind": "tree", "hq": 32, "hkv": 8, "d": 128, "tasks": 26, "spp": 16, "root": 4096,
         "shared": 8192, "task_lo": 300, "task_hi": 512, "suffix_lo": 128, "suffix_hi": 1024},
        # next token of 64 completions, a 128k vocabulary with a few likely tokens (configuration 3)
        _sample("sample-n64", 64, 128256, 3.0, (1.0, 1.0), 0.95, boosted=50),
        # next token of a serving batch of 1024 rows, a temperature per prompt (configuration 5)
        _sample("sample-n1024", 1024, 128256, 3.0, (0.2, 1.2), 0.95),
        # a temperature sweep of 3 x 64 completions with top-k / min-p rows and greedy rows among them, over a
        # vocabulary whose rows are not 16-byte aligned
        _sample("sample-odd-filters", 192, 50257, 3.0, (0.4, 1.0), 0.95, boosted=50, greedy_every=16, uncut_every=11,
                filters=1),
        # sixteen steps in the middle of the generation of 64 completions: append, attention, sampling
        {"name": "loop-n64-8k", "kind": "loop", "hq": 32, "hkv": 8, "d": 128, "n": 64, "prefix": 8192, "start_lo": 128,
         "start_hi": 960, "capacity": 1024, "steps": 16, "vocab": 128256, "sigma": 3.0},
    ]


def _logint(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choices(["attn", "tree", "sample", "loop"], [5, 1, 3, 1])[0]
    if kind == "attn":
        dtype = "bf16" if rng.random() < 0.8 else "f32"
        c = _attn("", dtype, 0, rng.choice([1, 2, 4, 8]), 128 if rng.random() < 0.7 else 64, _logint(rng, 1, 8),
                  _logint(rng, 1, 128), (0, 0), (0, 0), 16 if rng.random() < 0.4 else 0)
        c["hq"] = c["hkv"] * rng.choice([1, 2, 4, 8])
        c["prefix_hi"] = _logint(rng, 64, 16384)
        c["prefix_lo"] = max(1, int(c["prefix_hi"] * rng.uniform(0.2, 1.0)))
        c["suffix_hi"] = _logint(rng, 16, 2048)
        c["suffix_lo"] = int(c["suffix_hi"] * rng.uniform(0.0, 1.0))
        # no dearer than the largest listed case: its KV, its products; fp32 and 64-channel heads a tenth of the latter
        limit = 1.5e11 if c["dtype"] == "bf16" and c["d"] == 128 else 1.5e10
        while c["spp"] > 1 and (work(c)["flops"] > limit or
                                c["prompts"] * c["spp"] * c["suffix_hi"] * c["hkv"] * c["d"] * 8 > 4e9):
            c["spp"] = (c["spp"] + 1) // 2
    elif kind == "tree":
        hkv = rng.choice([2, 4, 8])
        hi = _logint(rng, 64, 1024)
        t_hi = _logint(rng, 64, 1024)
        c = {"kind": "tree", "hq": hkv * rng.choice([2, 4]), "hkv": hkv, "d": 128, "tasks": rng.randint(2, 26),
             "spp": _logint(rng, 2, 24), "root": _logint(rng, 256, 4096), "shared": _logint(rng, 256, 8192),
             "task_lo": max(1, t_hi // 2), "task_hi": t_hi, "suffix_lo": hi // 8, "suffix_hi": hi}
    elif kind == "sample":
        vocab = _logint(rng, 1000, 262144)
        if rng.random() < 0.5:
            vocab = (vocab + 63) // 64 * 64 if vocab <= 262080 else 262144
        t_lo = rng.uniform(0.2, 1.0)
        c = _sample("", _logint(rng, 1, 1024), vocab, round(rng.uniform(1.5, 4.0), 2),
                    (round(t_lo, 2), round(rng.uniform(t_lo, 1.2), 2)), rng.choice([0.8, 0.9, 0.95, 0.98, 1.0]),
                    boosted=rng.choice([0, 50]), greedy_every=rng.choice([0, 0, 9]), uncut_every=rng.choice([0, 0, 7]),
                    filters=1 if rng.random() < 0.3 else 0)
        while c["rows"] * c["vocab"] > 1024 * 128256:
            c["rows"] = (c["rows"] + 1) // 2
    else:
        cap = rng.randint(128, 1024)
        c = {"kind": "loop", "hq": 32, "hkv": 8, "d": 128, "n": _logint(rng, 1, 96), "prefix": _logint(rng, 256, 8192),
             "start_lo": 0, "start_hi": cap - 16, "capacity": cap, "steps": 16,
             "vocab": rng.choice([32000, 50256, 128256]), "sigma": 3.0}
    c.pop("name", None)
    return c


# ---- inputs ---------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _lens(g, lo, hi, n):
    return torch.randint(int(lo), int(hi) + 1, (n,), generator=g, device=DEV, dtype=torch.int32)


def _normal(g, shape, dtype):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32 if dtype == "f32" else torch.bfloat16)


def _indptr(lens):
    z = torch.zeros(lens.numel() + 1, dtype=torch.int32, device=DEV)
    z[1:] = torch.cumsum(lens, 0)
    return z


def _outputs(n, hq, d, dtype):
    out = torch.empty((n, hq, d), dtype=torch.float32 if dtype == "f32" else torch.bfloat16, device=DEV)
    return out, torch.empty((n, hq), dtype=torch.float32, device=DEV)


def _device_attn(dtype, hq, hkv, d, prompts, spp, prefix_lens, suffix_lens, max_prefix, max_suffix, page, g):
    """One attention problem on the GPU: paged KV deals the pool's pages out at random, as a server's
    allocator does after a while; contiguous suffixes sit in slots of `max_suffix` tokens."""
    n = prompts * spp
    desc = B.make_desc(dtype=B.SPD_F32 if dtype == "f32" else B.SPD_BF16, num_q_heads=hq, num_kv_heads=hkv, head_dim=d,
                       num_prompts=prompts, num_samples=n, max_samples_per_prompt=spp, page_size=page)
    q = _normal(g, (n, hq, d), dtype)
    sample_indptr = torch.arange(prompts + 1, device=DEV, dtype=torch.int32) * spp
    out, lse = _outputs(n, hq, d, dtype)
    ws = torch.empty(B.shared_prefix_decode_attn_workspace_size(desc, max_prefix, max_suffix), dtype=torch.uint8,
                     device=DEV)
    if page:
        pp, sp = (prefix_lens + page - 1) // page, (suffix_lens + page - 1) // page
        n_pp, n_sp = int(pp.sum()), int(sp.sum())
        perm = torch.randperm(n_pp + n_sp, generator=g, device=DEV, dtype=torch.int32)
        pool = (n_pp + n_sp, hkv, page, d)
        k, v = _normal(g, pool, dtype), _normal(g, pool, dtype)
        return D.DeviceAttn(desc, q, k, v, prefix_lens, _indptr(pp), perm[:n_pp].clone(), sample_indptr, k, v,
                            suffix_lens, _indptr(sp), perm[n_pp:].clone(), max_prefix, max_suffix, out, lse, ws)
    total = int(prefix_lens.sum())
    kp, vp = _normal(g, (total, hkv, d), dtype), _normal(g, (total, hkv, d), dtype)
    ks, vs = _normal(g, (n, max_suffix, hkv, d), dtype), _normal(g, (n, max_suffix, hkv, d), dtype)
    return D.DeviceAttn(desc, q, kp, vp, prefix_lens, _indptr(prefix_lens), None, sample_indptr, ks, vs, suffix_lens,
                        None, None, max_prefix, max_suffix, out, lse, ws)


def _attn_state(c, seed):
    g = _gen(seed)
    prefix_lens = _lens(g, c["prefix_lo"], c["prefix_hi"], c["prompts"])
    suffix_lens = _lens(g, c["suffix_lo"], c["suffix_hi"], c["prompts"] * c["spp"])
    return _device_attn(c["dtype"], c["hq"], c["hkv"], c["d"], c["prompts"], c["spp"], prefix_lens, suffix_lens,
                        c["prefix_hi"], c["suffix_hi"], c["page"], g)


class _Tree:
    """The buffers and the level table that a program keeps for a tree of prompts."""

    def __init__(self, c, seed):
        g = _gen(seed)
        n, hq, hkv, d = c["tasks"] * c["spp"], c["hq"], c["hkv"], c["d"]
        self.desc = B.make_desc(dtype=B.SPD_BF16, num_q_heads=hq, num_kv_heads=hkv, head_dim=d, num_prompts=1,
                                num_samples=n)
        self.q = _normal(g, (n, hq, d), "bf16")
        one = torch.tensor([0, n], device=DEV, dtype=torch.int32)
        per_task = torch.arange(c["tasks"] + 1, device=DEV, dtype=torch.int32) * c["spp"]
        self.levels = []
        for lens, groups, most, top in ((_lens(g, c["root"], c["root"], 1), one, n, c["root"]),
                                        (_lens(g, c["shared"], c["shared"], 1), one, n, c["shared"]),
                                        (_lens(g, c["task_lo"], c["task_hi"], c["tasks"]), per_task, c["spp"], c["task_hi"])):
            total = int(lens.sum())
            self.levels.append(D.DeviceLevel(_normal(g, (total, hkv, d), "bf16"), _normal(g, (total, hkv, d), "bf16"), lens,
                                             _indptr(lens), groups, most, top))
        self.level_array = B.make_levels(self.levels)
        self.max_suffix_len = c["suffix_hi"]
        self.suffix_lens = _lens(g, c["suffix_lo"], c["suffix_hi"], n)
        self.k_suffix = _normal(g, (n, self.max_suffix_len, hkv, d), "bf16")
        self.v_suffix = _normal(g, (n, self.max_suffix_len, hkv, d), "bf16")
        self.out, self.lse = _outputs(n, hq, d, "bf16")
        self.workspace = torch.empty(
            B.shared_prefix_decode_attn_levels_workspace_size(self.desc, self.level_array, self.max_suffix_len),
            dtype=torch.uint8, device=DEV)

    def run(self):
        B.shared_prefix_decode_attn_levels(self.desc, self.q, self.level_array, self.k_suffix, self.v_suffix,
                                           self.suffix_lens, None, None, self.max_suffix_len, self.out, self.lse,
                                           self.workspace)
        return {"out": self.out, "lse": self.lse}


def _logits(g, rows, vocab, sigma, boosted):
    x = torch.randn((rows, vocab), generator=g, device=DEV) * sigma
    if boosted:
        where = torch.randint(0, vocab, (rows, boosted), generator=g, device=DEV)
        x.scatter_add_(1, where, torch.full((rows, boosted), 8.0, device=DEV))
    return x


def _device_sampler(logits, temperature, top_p, uniforms):
    rows, vocab = logits.shape
    ws = torch.empty(max(256, B.sample_tokens_workspace_size(rows, vocab)), dtype=torch.uint8, device=DEV)
    return D.DeviceSampler(logits, temperature, top_p, uniforms, torch.empty(rows, dtype=torch.int32, device=DEV), ws)


class _Sample:
    """The logits, the per-row parameters and the workspace of a sampling call."""

    def __init__(self, c, seed):
        g = _gen(seed)
        rows, vocab = c["rows"], c["vocab"]
        logits = _logits(g, rows, vocab, c["sigma"], c["boosted"])
        t = torch.rand(rows, generator=g, device=DEV) * (c["t_hi"] - c["t_lo"]) + c["t_lo"]
        top_p = torch.full((rows,), float(c["top_p"]), device=DEV)
        r = torch.arange(rows, device=DEV)
        if c["greedy_every"]:
            t[r % c["greedy_every"] == 0] = 0.0
        if c["uncut_every"]:
            top_p[r % c["uncut_every"] == 1] = 1.0
        self.top_k = self.min_p = None
        if c["filters"]:  # a third of the rows with top-k 50, a third with min-p 0.05, a third with neither
            self.top_k = torch.where(r % 3 == 0, 50, 0).to(torch.int32)
            self.min_p = torch.where(r % 3 == 1, 0.05, 0.0).to(torch.float32)
        self.s = _device_sampler(logits, t, top_p, torch.rand(rows, generator=g, device=DEV))

    def run(self):
        s = self.s
        if self.top_k is None:
            s.run()
        else:
            rows, vocab = s.logits.shape
            B.sample_tokens_filtered(s.logits, B.SPD_F32, rows, vocab, s.logits.stride(0), s.temperature, s.top_p,
                                     self.top_k, self.min_p, s.uniforms, s.tokens, s.workspace)
        return {"tokens": s.tokens}


class _Loop:
    """A generation loop: one decode step captured once, replayed for every step of a pass.  A pass starts
    from the same generated lengths each time, as a new batch of completions would."""

    END_TOKEN = 2

    def __init__(self, c, seed):
        g = _gen(seed)
        n, hq, hkv, d, steps = c["n"], c["hq"], c["hkv"], c["d"], c["steps"]
        self.steps = steps
        self.start = _lens(g, c["start_lo"], c["start_hi"], n)
        prefix_lens = torch.tensor([c["prefix"]], device=DEV, dtype=torch.int32)
        attn = _device_attn("bf16", hq, hkv, d, 1, n, prefix_lens, self.start.clone(), c["prefix"], c["capacity"], 0, g)
        sampler = _device_sampler(_logits(g, n, c["vocab"], c["sigma"], 50), torch.full((n,), 1.0, device=DEV),
                                  torch.full((n,), 0.95, device=DEV), torch.rand(n, generator=g, device=DEV))
        self.loop = D.DecodeLoop(attn, sampler, _normal(g, (steps, n, hq, d), "bf16"),
                                 _normal(g, (steps, n, hkv, d), "bf16"), _normal(g, (steps, n, hkv, d), "bf16"),
                                 torch.rand((steps, n), generator=g, device=DEV), end_token=self.END_TOKEN)
        self.reset()
        self.loop.one_step()  # loads the kernels; the pass starts over from the same lengths
        torch.cuda.synchronize()
        self.graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(self.graph):
            self.loop.one_step()

    def reset(self):
        lp = self.loop
        lp.attn.suffix_lens.copy_(self.start)
        lp.step.zero_()
        lp.finished.zero_()
        lp.sampler.tokens.fill_(-1)

    def run(self):
        self.reset()
        for _ in range(self.steps):
            self.graph.replay()
        lp = self.loop
        lp.flush()
        return {"out": lp.out_steps, "tokens": lp.tokens_steps, "lens": lp.lens_steps, "k": lp.attn.k_suffix,
                "v": lp.attn.v_suffix}


class _Attn:
    def __init__(self, c, seed):
        self.a = _attn_state(c, seed)

    def run(self):
        self.a.run()
        return {"out": self.a.out, "lse": self.a.lse}


_KINDS = {"attn": _Attn, "tree": _Tree, "sample": _Sample, "loop": _Loop}


def prepare(case, seed):
    return _KINDS[case["kind"]](case, seed)


def run(state):
    return state.run()


# ---- what a pass cannot do without -------------------------------------------------------------------------

def work(case):
    c = case
    if c["kind"] == "sample":
        n = c["rows"] * c["vocab"]
        return {"bytes": 4 * n + 20 * c["rows"], "flops": 4 * n}
    if c["kind"] == "attn":
        elt, n = (4 if c["dtype"] == "f32" else 2), c["prompts"] * c["spp"]
        lp, ls = (c["prefix_lo"] + c["prefix_hi"]) / 2, (c["suffix_lo"] + c["suffix_hi"]) / 2
        tokens, rows_tokens = c["prompts"] * lp + n * ls, n * c["hq"] * (lp + ls)
    elif c["kind"] == "tree":
        elt, n = 2, c["tasks"] * c["spp"]
        lt, ls = (c["task_lo"] + c["task_hi"]) / 2, (c["suffix_lo"] + c["suffix_hi"]) / 2
        tokens = c["root"] + c["shared"] + c["tasks"] * lt + n * ls
        rows_tokens = n * c["hq"] * (c["root"] + c["shared"] + lt + ls)
    else:
        elt, n = 2, c["n"]
        ls = (c["start_lo"] + c["start_hi"] + c["steps"]) / 2
        tokens, rows_tokens = c["prefix"] + n * ls, n * c["hq"] * (c["prefix"] + ls)
    kv = 2 * c["hkv"] * c["d"] * elt
    io = n * c["hq"] * (2 * c["d"] * elt + 4)
    w = {"bytes": tokens * kv + io, "flops": 4 * c["d"] * rows_tokens}
    if c["kind"] == "loop":
        logits = n * c["vocab"]
        w = {"bytes": c["steps"] * (w["bytes"] + 4 * logits + 4 * n * kv), "flops": c["steps"] * (w["flops"] + 4 * logits)}
    return w


def tolerance(case):
    """Measured against `exact`: bf16 outputs carry one rounding of the result, one of the probabilities
    and one of the partial states (relative error 2.2e-3 to 2.7e-3); fp32 outputs 2e-7 to 5e-7.  A token may differ where its
    uniform falls within rounding of a boundary of the running mass."""
    if case["kind"] == "sample":
        return {"rel": 0.0, "differ": 0.005}
    if case["kind"] == "attn" and case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 1e-4}
    return {"rel": 1e-2, "max": 0.2, "differ": 0.005}


# ---- the same in 64 bits --------------------------------------------------------------------------------------

def _rows(k, pages, start, length, page):
    """[Hkv, length, D] fp64 of one sequence."""
    if page:
        got = k[pages.long()].permute(1, 0, 2, 3).reshape(k.shape[1], -1, k.shape[3])[:, :length]
    else:
        got = k[start:start + length].permute(1, 0, 2)
    return got.double().contiguous()


class _Exact:
    """Running softmax state of all rows in fp64: scores of a range are added with `add`."""

    def __init__(self, q, hkv):
        n, hq, d = q.shape
        self.scale, self.g = 1.0 / math.sqrt(d), hq // hkv
        self.q = q.double().view(n, hkv, self.g, d) * self.scale
        self.m = torch.full((n, hkv, self.g), -math.inf, dtype=torch.float64, device=q.device)
        self.l = torch.zeros_like(self.m)
        self.o = torch.zeros((n, hkv, self.g, d), dtype=torch.float64, device=q.device)

    def add(self, s0, s1, k, v):
        """Samples s0 .. s1-1 attend over k, v [Hkv, L, D]."""
        if k.shape[1] == 0:
            return
        hkv, d = k.shape[0], k.shape[2]
        kt = k.transpose(1, 2).contiguous()
        for j in range(hkv):
            rows = self.q[s0:s1, j].reshape(-1, d)
            s = rows @ kt[j]
            m = s.max(dim=1).values
            p = torch.exp(s - m[:, None])
            l, o = p.sum(1), p @ v[j]
            m, l, o = m.view(-1, self.g), l.view(-1, self.g), o.view(-1, self.g, d)
            m0, l0, o0 = self.m[s0:s1, j], self.l[s0:s1, j], self.o[s0:s1, j]
            top = torch.maximum(m0, m)
            a, b = torch.exp(m0 - top), torch.exp(m - top)
            self.o[s0:s1, j] = o0 * a[..., None] + o * b[..., None]
            self.l[s0:s1, j] = l0 * a + l * b
            self.m[s0:s1, j] = top

    def result(self):
        n, hkv, g, d = self.o.shape
        return (self.o / self.l[..., None]).view(n, hkv * g, d), (self.m + torch.log(self.l)).view(n, hkv * g)


def _exact_attn(a, suffix_lens=None, q=None):
    page, hkv = a.desc.page_size, a.desc.num_kv_heads
    e = _Exact(a.q if q is None else q, hkv)
    prefix_lens, pi, si = a.prefix_lens.tolist(), a.prefix_indptr.tolist(), a.sample_indptr.tolist()
    lens = (a.suffix_lens if suffix_lens is None else suffix_lens).tolist()
    for b, length in enumerate(prefix_lens):
        pages = a.prefix_page_indices[pi[b]:pi[b + 1]] if page else None
        e.add(si[b], si[b + 1], _rows(a.k_prefix, pages, pi[b], length, page), _rows(a.v_prefix, pages, pi[b], length, page))
    ti = a.suffix_page_indptr.tolist() if page else None
    for n, length in enumerate(lens):
        if page:
            pages = a.suffix_page_indices[ti[n]:ti[n + 1]]
            k, v = _rows(a.k_suffix, pages, 0, length, page), _rows(a.v_suffix, pages, 0, length, page)
        else:
            k, v = _rows(a.k_suffix[n], None, 0, length, 0), _rows(a.v_suffix[n], None, 0, length, 0)
        e.add(n, n + 1, k, v)
    return e.result()


def _exact_tokens(logits, temperature, top_p, uniforms, top_k=None, min_p=None):
    tokens = []
    for r in range(logits.shape[0]):
        x = logits[r].double()
        t = float(temperature[r])
        if t == 0.0:
            tokens.append(int(torch.nonzero(x == x.max())[0]))
            continue
        p = torch.exp((x - x.max()) / t)
        kept = torch.ones_like(p, dtype=torch.bool)
        if min_p is not None and float(min_p[r]) > 0:
            kept &= p >= float(min_p[r])
        if top_k is not None and int(top_k[r]) > 0:
            q = torch.where(kept, p, torch.zeros_like(p))
            kept &= p >= torch.topk(q, min(int(top_k[r]), q.numel())).values[-1]
        if float(top_p[r]) < 1.0:
            order = torch.sort(torch.where(kept, p, torch.zeros_like(p)), descending=True).values
            mass = torch.cumsum(order, 0)
            at = int(torch.searchsorted(mass, float(top_p[r]) * mass[-1]))
            kept &= p >= order[min(at, order.numel() - 1)]
        run_mass = torch.cumsum(torch.where(kept, p, torch.zeros_like(p)), 0)
        target = float(uniforms[r]) * run_mass[-1]
        tokens.append(min(int(torch.searchsorted(run_mass, target, right=True)), p.numel() - 1))
    return torch.tensor(tokens, dtype=torch.int32, device=logits.device)


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "attn":
        out, lse = _exact_attn(s.a)
        return {"out": out, "lse": lse}
    if case["kind"] == "tree":
        e = _Exact(s.q, case["hkv"])
        for lv in s.levels:
            lens, at, groups = lv.lens.tolist(), lv.indptr.tolist(), lv.sample_indptr.tolist()
            for i, length in enumerate(lens):
                e.add(groups[i], groups[i + 1], _rows(lv.k, None, at[i], length, 0), _rows(lv.v, None, at[i], length, 0))
        for n, length in enumerate(s.suffix_lens.tolist()):
            e.add(n, n + 1, _rows(s.k_suffix[n], None, 0, length, 0), _rows(s.v_suffix[n], None, 0, length, 0))
        out, lse = e.result()
        return {"out": out, "lse": lse}
    if case["kind"] == "sample":
        return {"tokens": _exact_tokens(s.s.logits, s.s.temperature, s.s.top_p, s.s.uniforms, s.top_k, s.min_p)}
    # the loop: append, attention and sampling step by step; a sample that drew the end token stops growing
    lp, a = s.loop, s.loop.attn
    lens, done = s.start.clone(), torch.zeros(case["n"], dtype=torch.bool, device=DEV)
    outs, toks, all_lens = [], [], []
    for t in range(case["steps"]):
        if t:
            done |= toks[-1] == s.END_TOKEN
        for n in range(case["n"]):
            at = int(lens[n])
            if not bool(done[n]) and at < case["capacity"]:
                a.k_suffix[n, at] = lp.k_steps[t, n]
                a.v_suffix[n, at] = lp.v_steps[t, n]
                lens[n] += 1
        out, _ = _exact_attn(a, lens, lp.q_steps[t])
        outs.append(out)
        toks.append(_exact_tokens(lp.sampler.logits, lp.sampler.temperature, lp.sampler.top_p, lp.u_steps[t]))
        all_lens.append(lens.clone())
    return {"out": torch.stack(outs), "tokens": torch.stack(toks), "lens": torch.stack(all_lens), "k": a.k_suffix,
            "v": a.v_suffix}
