"""The work that a user of this framework has it do, as cases that can be timed.

A case is a dict of plain values.  `kind` names the calling sequence:

  step      DecodeLayer.step over `layers` resident layers: chunk_score, then selection and attention
            in one call (a decode step; every layer's caches are its own)
  separate  the same step through the three separate calls (DecodeLayer.step_separate)
  ahead     DecodeStack.step_select_ahead over `layers` layers: one evaluation and one selection for
            all layers of the step, then attention layer by layer
  grow      a decode step that first takes in the token generated before it: kv_chunk_abstract_append,
            chunk_score, chunk_score_pin (first and last chunk always kept), selection and attention
  build     kv_chunk_abstract_build of one layer after prefill
  compress  kv_chunk_compress of one layer, then kv_chunk_abstract_build of the compressed store
  tree      chunk_tree_refine from uniform chunks of 64 tokens, then selection and attention over the
            refined partition

`dtype` is the cache's element type, "q8q4" the 8-bit / 4-bit store.  Caches follow the structure the
benchmark's workloads have: Gaussian keys that carry a Zipf mass along a direction the query heads of a
kv head share, important tokens in runs of 64, chunk sizes between `lo` and `hi` that are small where
important tokens lie ("tree": short runs of important tokens in a desert).
"""
import math

import numpy as np
import torch

import paper_2506_20187_amd as L

D = 128
DTYPES = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16, "q8q4": torch.float16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}
TREE_CHUNK, TREE_ROUNDS, TREE_CAP = 64, 64, 8192


def listed():
    def case(name, kind, dtype, batch, hq, hkv, n_ctx, lo, hi, budget, layers=1, max_chunks=0):
        return {"name": name, "kind": kind, "dtype": dtype, "batch": batch, "hq": hq, "hkv": hkv, "n_ctx": n_ctx,
                "lo": lo, "hi": hi, "budget": budget, "layers": layers, "max_chunks": max_chunks}
    return [
        # the smallest step of the benchmark's configurations: fp32, one sequence, 128 chunks of 32, 16 kept;
        # a few microseconds of work per launch
        case("step f32 4K", "step", "f32", 1, 8, 8, 4096, 32, 32, 0, max_chunks=16),
        # single-user decoding, multi-head attention in fp16 (32 heads), 32K context: eight layers of a model
        case("step f16 mha 32K", "step", "f16", 1, 32, 32, 32768, 16, 128, 2048, layers=8),
        # single-user decoding, grouped queries in bf16, 128K context: eight layers of a model
        case("step bf16 gqa 128K", "step", "bf16", 1, 32, 8, 131072, 16, 256, 4096, layers=8),
        # the benchmark's default: sixteen sequences of 128K, one layer (half a gigabyte per step)
        case("step bf16 gqa 128K x16", "step", "bf16", 16, 32, 8, 131072, 16, 256, 4096),
        # groups of eight query heads, three sequences of an odd length
        case("step bf16 g8 40003 x3", "step", "bf16", 3, 64, 8, 40003, 16, 128, 3001, layers=2),
        # half a million tokens in the 8-bit / 4-bit store: four layers of a model
        case("step q8q4 512K", "step", "q8q4", 1, 32, 8, 524288, 32, 512, 8192, layers=4),
        # the evaluation of all layers ahead of the step (the second case's shape with grouped queries)
        case("ahead bf16 gqa 128K", "ahead", "bf16", 1, 32, 8, 131072, 16, 256, 4096, layers=8),
        # serving many users at short contexts, each with its own length, with the caches growing
        case("grow bf16 gqa 9K x24", "grow", "bf16", 24, 32, 8, 9000, 16, 64, 1024),
        # a quarter of the context kept (accuracy first), pairs of query heads, through the separate calls
        case("separate f16 g2 64K x2", "separate", "f16", 2, 32, 16, 65521, 16, 128, 16384),
        # after prefill: the abstracts of one layer of four sequences
        case("build bf16 128K x4", "build", "bf16", 4, 32, 8, 131072, 16, 256, 4096),
        # after prefill: one layer's cache to the compressed store, and the store's abstracts
        case("compress bf16 256K", "compress", "bf16", 1, 32, 8, 262139, 32, 512, 8192),
        # exact search for the most important tokens in a deep layer, sixteen sequences
        case("tree bf16 128K x16", "tree", "bf16", 16, 32, 8, 131072, 64, 64, 4096),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["ahead", "grow", "separate", "build", "compress", "tree"])
    dtype = {"step": rng.choice(["f32", "f16", "bf16", "bf16", "q8q4"]), "ahead": rng.choice(["f16", "bf16"]),
             "grow": rng.choice(["f16", "bf16"]), "separate": rng.choice(["f32", "f16", "bf16"]), "build": rng.choice(["f16", "bf16"]),
             "compress": rng.choice(["f16", "bf16"]), "tree": rng.choice(["f16", "bf16"])}[kind]
    hkv = rng.choice([2, 4, 8, 8, 16, 32])
    group = rng.choice([1, 2, 4, 4, 8]) if kind in ("step", "separate") else rng.choice([1, 2, 4, 4])
    lo, hi = rng.choice([(16, 128), (16, 256), (32, 512), (32, 32), (24, 100)])
    most = {"step": 131072, "ahead": 131072, "grow": 16384, "separate": 65536, "build": 131072, "compress": 262144, "tree": 131072}[kind]
    n_ctx = _log_uniform(rng, most // 16, most)
    if dtype == "q8q4":
        n_ctx = _log_uniform(rng, 32768, 524288)
        lo, hi = rng.choice([(32, 512), (48, 300)])
        group = min(group, 4)
    # sequences: as many as keep the layer's keys and values within 4 GiB (less where a pass reads all of
    # them, or several layers are resident)
    layers = rng.choice([1, 2, 4]) if kind in ("step", "ahead") else 1
    per_seq = 2 * hkv * n_ctx * D * BYTES.get(dtype, 2)
    room = {"compress": 1 << 30, "build": 1 << 31}.get(kind, 1 << 32 if layers == 1 else 1 << 30)
    batch = _log_uniform(rng, 1, max(1, min(32, room // per_seq)))
    budget = max(256, n_ctx // _log_uniform(rng, 8, 48))
    if kind == "tree":
        lo = hi = TREE_CHUNK
        batch = min(batch, max(1, 128 // hkv))
        budget = min(budget, 4096) // 32 * 32
    if kind == "separate":
        budget = n_ctx // rng.choice([3, 4, 6])
    if kind == "grow":
        lo, hi = rng.choice([(16, 64), (32, 32), (8, 64)])
    if dtype == "q8q4":
        budget = min(budget, 1024 * lo)
    return {"kind": kind, "dtype": dtype, "batch": batch, "hq": hkv * group, "hkv": hkv, "n_ctx": n_ctx, "lo": lo, "hi": hi,
            "budget": budget, "layers": layers, "max_chunks": 0}


# ---- inputs ------------------------------------------------------------------------------------------

def _boundaries(n, lo, hi, heavy, rng):
    """Chunk boundaries of [0, n): regions of `hi` tokens have a target size, small where the region holds
    important tokens, and chunks around it."""
    if lo == hi:
        return np.append(np.arange(0, n, lo), n).astype(np.int32)
    regions = -(-n // hi)
    is_heavy = np.add.reduceat(np.pad(heavy, (0, regions * hi - n)).astype(np.int64), np.arange(0, regions * hi, hi)) > 0
    frac = rng.random(regions) ** np.where(is_heavy, 2.5, 0.8)
    target = np.exp(math.log(lo) + frac * math.log(hi / lo))
    per = np.maximum(1, (hi / target)).astype(np.int64)
    sizes = np.repeat(target, per) * rng.uniform(0.6, 1.6, int(per.sum()))
    sizes = np.clip(sizes.astype(np.int64), lo, hi)
    ends = np.cumsum(sizes)
    ends = ends[ends < n]
    while ends.size and n - ends[-1] < lo:          # no fragment below the smallest size
        ends = ends[:-1]
    rest = n - (int(ends[-1]) if ends.size else 0)
    last = int(ends[-1]) if ends.size else 0
    more = np.arange(last + hi, n, hi) if rest > 2 * hi else np.zeros(0, np.int64)
    return np.concatenate([[0], ends, more, [n]]).astype(np.int32)


def _count_of_chunks(case):
    """Chunks of a typical sequence: the generator's law with a fifth of the tokens important."""
    n = case["n_ctx"] if case["kind"] != "grow" else 3 * case["n_ctx"] // 4
    rng = np.random.default_rng(1)
    heavy = np.repeat(rng.random(-(-n // 64)) < 0.2, 64)[:n]
    return len(_boundaries(n, case["lo"], case["hi"], heavy, rng)) - 1


def _capacity(case):
    """Chunks a sequence has room for, as a serving program reserves it: some more than a typical sequence
    has, a multiple of 32."""
    n = _count_of_chunks(case)
    if case["kind"] == "grow":
        n = 4 * n // 3 + 32
    elif case["lo"] != case["hi"]:
        n += int(2 * n * math.sqrt(case["hi"] / case["n_ctx"]))          # sequences differ by that much
    return (n + 31) // 32 * 32


def _pack(offs, n_ctx, c_max):
    """[B, c_max + 1] boundary rows padded with n_ctx, and the counts."""
    offs = [o if len(o) <= c_max + 1 else np.append(o[:c_max], o[-1]) for o in offs]      # a full table: one long last chunk
    counts = np.asarray([len(o) - 1 for o in offs], np.int32)
    packed = np.full((len(offs), c_max + 1), n_ctx, np.int32)
    for b, o in enumerate(offs):
        packed[b, : len(o)] = o
    return packed, counts


def _normal(gen, batch, hkv, n, dtype):
    x = torch.empty(batch, hkv, n, D, dtype=dtype, device="cuda")
    for row in x:
        row.normal_(generator=gen)
    return x


def _zipf_cache(case, gen, rng, lengths, depth):
    """K, V [B,Hkv,N,D], q [B,Hq,D] and the mask of important tokens per sequence."""
    B, hkv, n = case["batch"], case["hkv"], case["n_ctx"]
    g = case["hq"] // hkv
    dt = torch.bfloat16 if case["dtype"] == "q8q4" else DTYPES[case["dtype"]]
    shared = torch.randn(B, hkv, D, generator=gen, device="cuda")
    q = shared if g == 1 else (shared[:, :, None, :] + 0.5 * torch.randn(B, hkv, g, D, generator=gen, device="cuda"))
    q = q.reshape(B, hkv * g, D).to(DTYPES[case["dtype"]])
    K, V = _normal(gen, B, hkv, n, dt), _normal(gen, B, hkv, n, dt)
    if g == 1 and case["dtype"] == "f16":           # multi-head models: a few channels carry outliers
        K[..., :4] *= 8.0
    heavy = []
    exponent = 0.6 + 0.7 * depth if g > 1 else 1.1
    for b in range(B):
        segs = -(-n // 64)
        rank = (torch.randperm(segs, generator=gen, device="cuda")[:, None] * 64
                + torch.rand(segs, 64, generator=gen, device="cuda").argsort(dim=1)).reshape(-1)[:n] + 1
        a = -exponent * torch.log(rank.float())
        a = (a - a.mean()) * math.sqrt(D)
        heavy.append((rank <= 0.2 * lengths[b]).cpu().numpy()[: lengths[b]])
        for h in range(hkv):
            u = shared[b, h] / (shared[b, h] * shared[b, h]).sum()
            K[b, h] += (a[:, None] * u[None, :]).to(dt)
    return K, V, q, heavy


def _chunks(case, heavy, lengths, rng):
    offs = [_boundaries(lengths[b], case["lo"], case["hi"], heavy[b], rng) for b in range(case["batch"])]
    return _pack(offs, case["n_ctx"], _capacity(case))


def _k_max(case, c_max):
    if case["max_chunks"]:
        return min(c_max, case["max_chunks"])
    most = 1024 if case["dtype"] == "q8q4" else 8192
    return max(1, min(c_max, case["budget"] // case["lo"] + 1, most))


def _compress(K, V, off, counts, four, hq):
    B, hkv, n, _ = K.shape
    shape = L.make_shape(B, hq, hkv, D, n, off.shape[1] - 1, 1, K.dtype)
    room = L.leoam_compressed_bytes_bound(shape)
    st = {"shape": shape, "kblob": torch.zeros(room, dtype=torch.uint8, device="cuda"),
          "vblob": torch.zeros(room, dtype=torch.uint8, device="cuda"),
          "qmeta": torch.zeros(B, hkv, off.shape[1] - 1, 8, dtype=torch.int32, device="cuda"),
          "total": torch.zeros(1, dtype=torch.int64, device="cuda")}
    L.kv_chunk_compress(shape, K, V, off, counts, four, st["kblob"], st["vblob"], st["qmeta"], st["total"])
    return st


def _four_bit(offs, counts, heavy):
    """Half of a sequence's chunks, those without important tokens first, are 4-bit."""
    four = np.zeros((offs.shape[0], offs.shape[1] - 1), np.uint8)
    for b, n in enumerate(counts):
        has = np.add.reduceat(heavy[b].astype(np.int64), offs[b, :n]) > 0
        four[b, np.argsort(has, kind="stable")[: n // 2]] = 1
    return torch.from_numpy(four).cuda()


def _dense_or_compressed(case, seed, layer):
    """One layer's caches as a user holds them: (K, V, q, chunk_off, n_chunks, qmeta or None)."""
    key = [seed & 0x7FFFFFFF, layer]
    gen = torch.Generator(device="cuda").manual_seed(int(np.random.SeedSequence(key).generate_state(1)[0]))
    rng = np.random.default_rng(key)
    lengths = [case["n_ctx"]] * case["batch"]
    depth = (layer + 0.5) / max(1, case["layers"])
    K, V, q, heavy = _zipf_cache(case, gen, rng, lengths, depth)
    offs, counts = _chunks(case, heavy, lengths, rng)
    d_off, d_cnt = torch.from_numpy(offs).cuda(), torch.from_numpy(counts).cuda()
    if case["dtype"] != "q8q4":
        return K, V, q, d_off, d_cnt, None
    st = _compress(K, V, d_off, d_cnt, _four_bit(offs, counts, heavy), case["hq"])
    used = int(st["total"].item())
    return st["kblob"][:used].clone(), st["vblob"][:used].clone(), q, d_off, d_cnt, st["qmeta"]


def _layer(case, parts):
    K, V, q, off, cnt, qmeta = parts
    c_max = off.shape[1] - 1
    zeros = {"abstract": torch.zeros(case["batch"], case["hkv"], c_max, 2, D, dtype=q.dtype, device="cuda")}
    more = {} if qmeta is None else {"qmeta": qmeta, "n_kv_heads": case["hkv"], "n_ctx": case["n_ctx"]}
    lay = L.DecodeLayer(K, V, off, cnt, case["hq"], _k_max(case, c_max), case["max_chunks"], case["budget"], buffers=zeros, **more)
    lay.build_abstract()
    return lay


def _prepare_step(case, seed):
    parts = [_dense_or_compressed(case, seed, l) for l in range(case["layers"])]
    return {"layers": [_layer(case, p) for p in parts], "q": [p[2] for p in parts]}


def _prepare_ahead(case, seed):
    parts = [_dense_or_compressed(case, seed, l) for l in range(case["layers"])]
    k_max = max(_k_max(case, p[3].shape[1] - 1) for p in parts)
    stack = L.DecodeStack([p[0] for p in parts], [p[1] for p in parts], [p[3] for p in parts], [p[4] for p in parts],
                          case["hq"], k_max, case["max_chunks"], case["budget"])
    stack.build_abstract()
    return {"stack": stack, "q": torch.stack([p[2] for p in parts]).contiguous()}


def _prepare_grow(case, seed):
    """Sequences of their own lengths inside caches of n_ctx tokens, the next token's key and value stored."""
    gen = torch.Generator(device="cuda").manual_seed(int(np.random.SeedSequence([seed & 0x7FFFFFFF, 77]).generate_state(1)[0]))
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 78])
    lengths = [int(x) for x in rng.integers(case["n_ctx"] // 2, case["n_ctx"] - 1, case["batch"])]
    K, V, q, heavy = _zipf_cache(case, gen, rng, lengths, 0.5)
    offs, counts = _chunks(case, heavy, lengths, rng)
    c_max = offs.shape[1] - 1
    saved = torch.from_numpy(np.concatenate([offs.reshape(-1), counts])).cuda()
    book = saved.clone()                             # boundary rows, then counts: one buffer, as one table
    off = book[: offs.size].view(case["batch"], c_max + 1)
    cnt = book[offs.size:]
    lay = _layer(case, (K, V, q, off, cnt, None))
    status = torch.zeros(case["batch"], dtype=torch.int32, device="cuda")
    return {"lay": lay, "q": q, "book": book, "saved": saved, "status": status, "chunk_size": max(case["lo"], 8)}


def _prepare_build(case, seed):
    K, V, q, off, cnt, _ = _dense_or_compressed(case, seed, 0)
    del V
    shape = L.make_shape(case["batch"], case["hq"], case["hkv"], D, case["n_ctx"], off.shape[1] - 1, 1, K.dtype)
    return {"shape": shape, "K": K, "off": off, "cnt": cnt,
            "abstract": torch.zeros(case["batch"], case["hkv"], off.shape[1] - 1, 2, D, dtype=K.dtype, device="cuda")}


def _prepare_compress(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(int(np.random.SeedSequence([seed & 0x7FFFFFFF, 99]).generate_state(1)[0]))
    rng = np.random.default_rng([seed & 0x7FFFFFFF, 98])
    lengths = [case["n_ctx"]] * case["batch"]
    K, V, q, heavy = _zipf_cache(case, gen, rng, lengths, 0.5)
    offs, counts = _chunks(case, heavy, lengths, rng)
    d_off, d_cnt, four = torch.from_numpy(offs).cuda(), torch.from_numpy(counts).cuda(), _four_bit(offs, counts, heavy)
    st = _compress(K, V, d_off, d_cnt, four, case["hq"])
    c_max = offs.shape[1] - 1
    st.update(K=K, V=V, off=d_off, cnt=d_cnt, four=four,
              q_shape=L.make_shape(case["batch"], case["hq"], case["hkv"], D, case["n_ctx"], c_max, 1, L.binding.Q8Q4),
              abstract=torch.zeros(case["batch"], case["hkv"], c_max, 2, D, dtype=torch.float16, device="cuda"))
    return st


def _prepare_tree(case, seed):
    """Runs of 32 important tokens at distinct random places of a desert; the abstracts of the initial chunks."""
    B, hkv, n, hq = case["batch"], case["hkv"], case["n_ctx"], case["hq"]
    g, dt, k = hq // hkv, DTYPES[case["dtype"]], case["budget"]
    gen = torch.Generator(device="cuda").manual_seed(int(np.random.SeedSequence([seed & 0x7FFFFFFF, 55]).generate_state(1)[0]))
    K, V = _normal(gen, B, hkv, n, dt), _normal(gen, B, hkv, n, dt)
    K *= 0.1
    direction = torch.randn(B, hkv, D, generator=gen, device="cuda")
    direction = direction / direction.norm(dim=-1, keepdim=True)
    runs = max(1, k // 32)
    slot = n // runs
    start = torch.arange(runs, device="cuda") * slot + torch.randint(0, max(1, slot - 32), (B, hkv, runs), generator=gen, device="cuda")
    rows = (start[..., None] + torch.arange(32, device="cuda")).reshape(B, hkv, -1).clamp_(max=n - 1)
    hot = torch.zeros(B, hkv, n, dtype=torch.bool, device="cuda").scatter_(2, rows, True)
    for b in range(B):
        for h in range(hkv):
            K[b, h] += torch.where(hot[b, h][:, None], 6.0 * direction[b, h][None, :], torch.zeros((), device="cuda")).to(dt)
    q = (4.0 * direction[:, :, None, :] + 0.05 * torch.randn(B, hkv, g, D, generator=gen, device="cuda")).reshape(B, hq, D).to(dt)
    m0 = -(-n // TREE_CHUNK)
    shape = L.make_shape(B, hq, hkv, D, n, m0, 1, dt)
    off = torch.clamp(torch.arange(m0 + 1, dtype=torch.int32, device="cuda") * TREE_CHUNK, max=n).repeat(B, 1).contiguous()
    cnt = torch.full((B,), m0, dtype=torch.int32, device="cuda")
    ab = torch.empty(B, hkv, m0, 2, D, dtype=dt, device="cuda")
    L.kv_chunk_abstract_build(shape, K, off, cnt, ab)
    bh, k_max = B * hkv, min(TREE_CAP, 2048)
    a_shape = L.make_shape(bh, g, 1, D, n, TREE_CAP, k_max, dt)
    new = lambda *s, dtype=torch.int32: torch.zeros(*s, dtype=dtype, device="cuda")  # noqa: E731
    ws = torch.empty(max(16, (L.leoam_fused_workspace_bytes(a_shape, k) + 15) // 16 * 16), dtype=torch.uint8, device="cuda")
    L.leoam_workspace_init(ws)
    return {"shape": shape, "a_shape": a_shape, "K": K, "V": V, "q": q, "abstract": ab, "k": k, "ref_off": new(bh, TREE_CAP + 1),
            "ref_score": new(bh, 1, TREE_CAP, dtype=torch.float32), "ref_count": new(bh), "ref_evals": new(bh), "ref_status": new(bh),
            "tree_ws": torch.empty(L.leoam_tree_workspace_bytes(shape, TREE_CAP), dtype=torch.uint8, device="cuda"), "ws": ws,
            "sel_idx": new(bh, 1, k_max), "sel_count": new(bh, 1), "sel_tokens": new(bh, 1),
            "out": new(bh, g, D, dtype=torch.float32), "lse": new(bh, g, dtype=torch.float32)}


def prepare(case, seed):
    make = {"step": _prepare_step, "separate": _prepare_step, "ahead": _prepare_ahead, "grow": _prepare_grow,
            "build": _prepare_build, "compress": _prepare_compress, "tree": _prepare_tree}[case["kind"]]
    with torch.no_grad():
        state = make(case, seed)
    state["kind"] = case["kind"]
    return state


# ---- one pass ----------------------------------------------------------------------------------------

def _outputs(lay):
    return {"score": lay.score, "sel_idx": lay.sel_idx, "sel_count": lay.sel_count, "sel_tokens": lay.sel_tokens, "out": lay.out,
            "lse": lay.lse}


def run(state):
    kind = state["kind"]
    if kind == "step":
        for lay, q in zip(state["layers"], state["q"]):
            lay.step(q)
        return [_outputs(lay) for lay in state["layers"]]
    if kind == "separate":
        for lay, q in zip(state["layers"], state["q"]):
            lay.step_separate(q)
        return [_outputs(lay) for lay in state["layers"]]
    if kind == "ahead":
        state["stack"].step_select_ahead(state["q"])
        return _outputs(state["stack"])
    if kind == "grow":
        # (the token of the pass before is a draft that was not accepted: the boundaries are put back)
        lay, q = state["lay"], state["q"]
        state["book"].copy_(state["saved"])
        L.kv_chunk_abstract_append(lay.shape, lay.K, lay.chunk_off, lay.n_chunks, state["chunk_size"], lay.abstract, state["status"])
        L.chunk_score(lay.shape, q, lay.abstract, lay.n_chunks, lay.score)
        L.chunk_score_pin(lay.shape, lay.n_chunks, 1, 1, lay.score)
        L.chunk_select_attention_decode(lay.shape, lay.score, q, lay.K, lay.V, lay.chunk_off, lay.n_chunks, lay.max_chunks,
                                        lay.token_budget, lay.scale, lay.sel_idx, lay.sel_count, lay.sel_tokens, lay.out, lay.lse,
                                        lay.workspace)
        return dict(_outputs(lay), abstract=lay.abstract, chunk_off=lay.chunk_off, n_chunks=lay.n_chunks, status=state["status"])
    if kind == "build":
        L.kv_chunk_abstract_build(state["shape"], state["K"], state["off"], state["cnt"], state["abstract"])
        return state["abstract"]
    if kind == "compress":
        s = state
        L.kv_chunk_compress(s["shape"], s["K"], s["V"], s["off"], s["cnt"], s["four"], s["kblob"], s["vblob"], s["qmeta"], s["total"])
        L.kv_chunk_abstract_build(s["q_shape"], s["kblob"], s["off"], s["cnt"], s["abstract"], qmeta=s["qmeta"])
        return {n: s[n] for n in ("kblob", "vblob", "qmeta", "total", "abstract")}
    s = state
    L.chunk_tree_refine(s["shape"], s["q"], s["K"], s["abstract"], TREE_CHUNK, s["k"], TREE_ROUNDS, TREE_CAP, s["ref_off"],
                        s["ref_score"], s["ref_count"], s["ref_evals"], s["ref_status"], s["tree_ws"])
    L.chunk_select_attention_decode(s["a_shape"], s["ref_score"], s["q"], s["K"], s["V"], s["ref_off"], s["ref_count"], 0, s["k"],
                                    L.default_scale(D), s["sel_idx"], s["sel_count"], s["sel_tokens"], s["out"], s["lse"], s["ws"])
    return {n: s[n] for n in ("ref_off", "ref_score", "ref_count", "ref_evals", "ref_status", "sel_idx", "sel_count", "sel_tokens",
                              "out", "lse")}


# ---- what a pass cannot do without ---------------------------------------------------------------------

def work(case):
    B, hkv, hq, n, layers = case["batch"], case["hkv"], case["hq"], case["n_ctx"], case["layers"]
    kind, dtype = case["kind"], case["dtype"]
    e = BYTES.get(dtype, 2)
    rows = B * hkv
    if kind == "tree":
        # the initial chunks' abstracts; the keys of the runs' surroundings (every run of 32 touches two or three chunks,
        # each of which is read once); the kept tokens' keys and values
        m0, runs = -(-n // TREE_CHUNK), max(1, case["budget"] // 32)
        near = min(n, runs * 96)
        kept = rows * case["budget"]
        read = rows * (m0 * 2 * D * e + near * D * e) + kept * 2 * D * e
        return {"bytes": read + B * hq * D * (e + 4), "flops": rows * m0 * 4 * D * (hq // hkv) * 2 + rows * near * 2 * D * (hq // hkv)
                + kept * 4 * D * (hq // hkv)}
    chunks = rows * _count_of_chunks(case)
    if kind == "build":
        return {"bytes": rows * n * D * e + chunks * 2 * D * e + B * 4 * (chunks // rows), "flops": 2 * rows * n * D}
    if kind == "compress":
        codes = rows * n * (D + D // 2) // 2                                 # half of the chunks are 4-bit
        # K and V read once, both blobs written, records and abstracts written
        return {"bytes": rows * n * 2 * D * e + 2 * codes + chunks * (32 + 2 * D * 2), "flops": 10 * rows * n * 2 * D}
    if case["max_chunks"]:
        kept = rows * min(n, case["max_chunks"] * case["lo"])
    else:
        kept = rows * min(n if kind != "grow" else 3 * n // 4, case["budget"])
    kv = kept * 2 * D * e if dtype != "q8q4" else kept * 2 * D               # (kept chunks hold important tokens: mostly 8-bit)
    one = chunks * (2 * D * e + 8) + kv + B * hq * D * (e + 4)
    flops = chunks * 4 * D * (hq // hkv) + kept * 4 * D * (hq // hkv)
    if kind == "grow":
        one += rows * 5 * D * e
    return {"bytes": layers * one, "flops": layers * flops}


def tolerance(case):
    # abstracts, codes and records are exact; scores are double sums rounded once to float and selections follow from them;
    # attention is an fp32 softmax over fp32 logits (up to about 14 at its scale, sums of up to 16K terms)
    if case["kind"] in ("build", "compress"):
        return "exact"
    # measured against attention in 64 bits and between different splits: rel 2e-7 to 8e-7, max up to 6e-6
    return {"rel": 3e-6, "max": 3e-5, "differ": 0.0}
