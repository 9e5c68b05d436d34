"""The calls whose time is measured: what a rollout engine has this library do, over the sizes it is used at.

A case is a dict of plain values; its sequence lengths follow from the case alone (so that its bytes are known), all
other inputs from the seed.  Kinds:

  decode   one decode-attention call of a batch, through the plain binding or through PreparedDecode
  grouped  one decode call of a batch of response groups that share their prompts' pages
  append   one token of every sequence written into the pools of several layers (each pass takes the next token of a ring)
  migrate  pages of some sequences packed into one buffer and unpacked into another pool
"""
import ctypes
import math

import numpy as np
import torch

from paper_2604_26256_amd import dora

FP8_MAX = 448.0


def listed():
    return [
        # the smallest call: a handful of short sequences of a small model, in a host loop over prepared buffers
        {"name": "decode_tiny", "kind": "decode", "seqs": 8, "q_heads": 8, "kv_heads": 2, "d": 64, "page": 16, "fp8": False, "median": 256,
         "sigma": 1.0, "lo": 1, "hi": 2048, "prepared": True},
        # the first steps of a 7B-class rollout: the whole batch is running, its responses are still short
        {"name": "decode_early7b", "kind": "decode", "seqs": 64, "q_heads": 28, "kv_heads": 4, "d": 128, "page": 16, "fp8": False,
         "median": 320, "sigma": 0.5, "lo": 64, "hi": 1500, "prepared": True},
        # the last few responses of an fp8 rollout: an odd number of sequences, too little work to fill the chip
        {"name": "decode_survivors_fp8", "kind": "decode", "seqs": 3, "q_heads": 32, "kv_heads": 8, "d": 128, "page": 16, "fp8": True,
         "median": 6000, "sigma": 0.4, "lo": 1000, "hi": 20000, "prepared": True},
        # the 7B-class long-tailed batch
        {"name": "decode_rollout7b", "kind": "decode", "seqs": 64, "q_heads": 28, "kv_heads": 4, "d": 128, "page": 16, "fp8": False,
         "median": 2048, "sigma": 1.2, "lo": 64, "hi": 32768, "prepared": False},
        # only very long responses left
        {"name": "decode_tail_only", "kind": "decode", "seqs": 4, "q_heads": 32, "kv_heads": 8, "d": 128, "page": 16, "fp8": False,
         "median": 60000, "sigma": 0.3, "lo": 32768, "hi": 98304, "prepared": False},
        # a full batch whose sequences belong to several policy versions
        {"name": "decode_multi_version", "kind": "decode", "seqs": 512, "q_heads": 64, "kv_heads": 8, "d": 128, "page": 16, "fp8": False,
         "median": 1024, "sigma": 1.3, "lo": 16, "hi": 65536, "prepared": False},
        # the largest batch of one GPU: fp8 pages of 32 tokens
        {"name": "decode_moe_fp8", "kind": "decode", "seqs": 1024, "q_heads": 64, "kv_heads": 8, "d": 128, "page": 32, "fp8": True,
         "median": 4096, "sigma": 1.2, "lo": 128, "hi": 131072, "prepared": False},
        # 16 responses for each of 4 prompts, the prompt's pages shared
        {"name": "grouped_grpo7b", "kind": "grouped", "seqs": 64, "group": 16, "q_heads": 28, "kv_heads": 4, "d": 128, "page": 16,
         "fp8": False, "prompt_lo": 1024, "prompt_hi": 4096, "median": 2048, "sigma": 1.2, "lo": 64, "hi": 32768},
        # the same for the larger model, early in the responses: most of the context is prompt
        {"name": "grouped_moe_fp8", "kind": "grouped", "seqs": 256, "group": 16, "q_heads": 64, "kv_heads": 8, "d": 128, "page": 32,
         "fp8": True, "prompt_lo": 1024, "prompt_hi": 4096, "median": 512, "sigma": 1.0, "lo": 16, "hi": 8192},
        # the write before each decode: one token of every sequence, layer after layer, called as a native loop calls it
        {"name": "append_multi_version", "kind": "append", "seqs": 512, "kv_heads": 8, "d": 128, "page": 16, "fp8": False, "layers": 4},
        {"name": "append_moe_fp8", "kind": "append", "seqs": 1024, "kv_heads": 8, "d": 128, "page": 32, "fp8": True, "layers": 4},
        # 32 requests moved to another instance of their version
        {"name": "migrate_multi_version", "kind": "migrate", "seqs": 32, "kv_heads": 8, "d": 128, "page": 16, "fp8": False,
         "median": 1024, "sigma": 1.3, "lo": 16, "hi": 65536},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "decode", "decode", "grouped", "grouped", "append", "append", "migrate"])
    case = {"kind": kind, "d": rng.choice([64, 128, 128]), "page": rng.choice([16, 32]), "fp8": rng.random() < 0.5, "kv_heads": rng.choice([1, 2, 4, 8])}
    if kind == "append":
        case.update(seqs=_log(rng, 1, 1024), layers=rng.randint(1, 4))
        return case
    token_bytes = case["kv_heads"] * case["d"] * 2 * (1 if case["fp8"] else 2)
    if kind == "migrate":
        case.update(seqs=_log(rng, 1, 64), median=_log(rng, 64, 4096), sigma=rng.uniform(0.0, 1.3), lo=1)
        case["hi"] = min(65536, 16 * case["median"], max(64, (1 << 29) // token_bytes // case["seqs"]))
        return case
    heads = rng.choice([1, 2, 4, 6, 7, 8, 16])
    if kind == "grouped":
        case["group"] = rng.choice([g for g in (2, 4, 5, 8, 16) if g * heads <= 128])
        case.update(seqs=case["group"] * _log(rng, 1, 24), q_heads=heads * case["kv_heads"], prompt_lo=_log(rng, 64, 2048))
        case.update(prompt_hi=2 * case["prompt_lo"] + rng.randint(0, 900), median=_log(rng, 64, 2048), sigma=rng.uniform(0.0, 1.2), lo=1)
        case["hi"] = min(32768, 16 * case["median"])
        return case
    case.update(seqs=_log(rng, 1, 1024), q_heads=heads * case["kv_heads"], median=_log(rng, 64, 32768), sigma=rng.uniform(0.0, 1.3), lo=1,
                prepared=rng.random() < 0.5)
    # at most about 4 GB of keys and values
    case["hi"] = max(32, min(131072, 16 * case["median"], (1 << 32) // token_bytes // case["seqs"]))
    return case


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _lengths(case):
    """Tokens of each sequence: lognormal, clipped, the same for every seed of the case (a group's prompt included)."""
    rng = np.random.default_rng(case["seqs"] * 1000003 + case["median"])
    x = np.exp(rng.normal(math.log(case["median"]), case["sigma"], case["seqs"]))
    x = np.clip(np.rint(x), case["lo"], case["hi"]).astype(np.int64)
    if case["kind"] != "grouped":
        return x, None
    prompt = rng.integers(case["prompt_lo"], case["prompt_hi"] + 1, case["seqs"] // case["group"])
    prompt = np.repeat(prompt, case["group"])
    return x + prompt, prompt // case["page"]  # tokens, and the full pages shared in the group


def _page_shapes(case):
    x = 16 if case["fp8"] else 8
    return (case["kv_heads"], case["d"] // x, case["page"], x), (case["kv_heads"], case["d"], case["page"])


def _pages(case, n, gen):
    """n K or V pages' worth of N(0, 1) values: (bf16, None), or fp8 codes and one scale a page."""
    size = case["kv_heads"] * case["page"] * case["d"]
    if not case["fp8"]:
        t = torch.empty((n, size), dtype=torch.bfloat16, device="cuda")
        t.normal_(generator=gen)
        return t, None
    t = torch.empty((n, size), dtype=torch.uint8, device="cuda")
    scales = torch.empty(n, dtype=torch.float32, device="cuda")
    step = max(1, (1 << 28) // size)
    for i in range(0, n, step):
        x = torch.empty((min(step, n - i), size), dtype=torch.float32, device="cuda").normal_(generator=gen)
        s = x.abs().amax(dim=1) / FP8_MAX
        scales[i:i + step] = s
        t[i:i + step] = (x / s[:, None]).clamp_(-FP8_MAX, FP8_MAX).to(torch.float8_e4m3fn).view(torch.uint8)
    return t, scales


def _pool(case, n, gen):
    ks, vs = _page_shapes(case)
    k, k_scales = _pages(case, n, gen)
    v, v_scales = _pages(case, n, gen)
    return {"k": k.view((n,) + ks), "v": v.view((n,) + vs), "k_scales": k_scales, "v_scales": v_scales}


def _kw(case, pool):
    return {"num_kv_heads": case["kv_heads"], "page_size": case["page"], "kv_dtype": dora.DORA_KV_FP8_E4M3 if case["fp8"] else dora.DORA_KV_BF16,
            "k_scales": pool["k_scales"], "v_scales": pool["v_scales"]}


def _i32(x):
    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.int32)).cuda()


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    if case["kind"] == "append":
        return _prepare_append(case, gen, rng)
    lens, shared = _lengths(case)
    n = -(-lens // case["page"])
    num_pages = int(n.sum()) + int(n.sum()) // 8 + 1
    perm = rng.permutation(num_pages)  # pages lie scattered in the pool
    table = np.zeros((len(lens), int(n.max())), np.int32)
    at = 0
    for b, nb in enumerate(n):
        table[b, :nb] = perm[at:at + nb]
        at += int(nb)
    if shared is not None:
        for b in range(len(lens)):
            table[b, :shared[b]] = table[b - b % case["group"], :shared[b]]
    pool = _pool(case, num_pages, gen)
    if case["kind"] == "migrate":
        src = np.concatenate([table[b, :nb] for b, nb in enumerate(n)])
        desc = dora.make_pack_desc(kv_dtype=int(case["fp8"]), page_size=case["page"], num_kv_heads=case["kv_heads"], head_dim=case["d"],
                                   num_pages=num_pages, policy_version=1, n_seqs=case["seqs"])
        to = {name: None if t is None else torch.zeros_like(t) for name, t in pool.items()}
        return {"case": case, "pool": pool, "to": to, "src": _i32(src), "dst": _i32(rng.permutation(num_pages)[:len(src)]),
                "packed": torch.zeros(dora.dora_kv_packed_bytes(desc, len(src)), dtype=torch.uint8, device="cuda")}
    q = torch.empty((len(lens), case["q_heads"], case["d"]), dtype=torch.bfloat16, device="cuda").normal_(generator=gen)
    s = {"case": case, "pool": pool, "q": q, "out": torch.empty_like(q), "table": _i32(table), "lens": _i32(lens), "versions": _i32(0 * lens)}
    if case.get("prepared"):
        s["call"] = dora.PreparedDecode(q, pool["k"], pool["v"], s["table"], s["lens"], s["versions"], s["out"], **_kw(case, pool))
    return s


def _prepare_append(case, gen, rng):
    """Sequences in the middle of a page (some at its first slot), in a ring of as many tokens as a page holds: pass i
    writes token i of every sequence, so scales are set and grow as they do over the steps of a rollout."""
    b, page, layers = case["seqs"], case["page"], case["layers"]
    base = rng.integers(0, 64 * page, b)  # tokens in the cache before the ring
    first = base // page
    num_pages = 6 * b
    perm = rng.permutation(num_pages)
    table = rng.integers(0, num_pages, (b, 66)).astype(np.int32)
    for k in range(2):
        table[np.arange(b), first + k] = perm[k * b:(k + 1) * b]
    s = {"case": case, "pools": [_pool(case, num_pages, gen) for _ in range(layers)], "table": _i32(table), "at": 0, "base": base}
    shape = (page, layers, b, case["kv_heads"], case["d"])
    s["k_new"], s["v_new"] = (torch.empty(shape, dtype=torch.bfloat16, device="cuda").normal_(generator=gen) for _ in range(2))
    s["lens"] = _i32(base[None, :] + 1 + np.arange(page)[:, None])
    desc = dora.make_decode_desc(num_seqs=b, num_q_heads=case["kv_heads"], num_kv_heads=case["kv_heads"], head_dim=case["d"], page_size=page,
                                 block_table_stride=table.shape[1], num_pages=num_pages, kv_dtype=int(case["fp8"]))
    s["desc"], stream = desc, torch.cuda.current_stream().cuda_stream
    ptr = lambda t: None if t is None else t.data_ptr()  # noqa: E731
    s["calls"] = [[(ctypes.byref(desc), s["k_new"][i, n].data_ptr(), s["v_new"][i, n].data_ptr(), s["table"].data_ptr(), s["lens"][i].data_ptr(), None,
                    ptr(p["k"]), ptr(p["v"]), ptr(p["k_scales"]), ptr(p["v_scales"]), None, stream) for n, p in enumerate(s["pools"])]
                  for i in range(page)]
    s["append"] = dora.library().dora_kv_append
    return s


# ---------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------

def run(s):
    case = s["case"]
    if case["kind"] == "append":
        calls = s["calls"][s["at"]]
        s["at"] = (s["at"] + 1) % len(s["calls"])
        for args in calls:
            status = s["append"](*args)
            if status:
                raise RuntimeError(dora.status_string(status))
        return s["pools"]
    pool = s["pool"]
    if case["kind"] == "migrate":
        kw = dict(num_kv_heads=case["kv_heads"], page_size=case["page"], head_dim=case["d"], kv_dtype=int(case["fp8"]), policy_version=1)
        dora.dora_kv_page_pack(pool["k"], pool["v"], s["src"], s["packed"], n_seqs=case["seqs"], k_scales=pool["k_scales"],
                               v_scales=pool["v_scales"], **kw)
        to = s["to"]
        dora.dora_kv_page_unpack(s["packed"], s["dst"], to["k"], to["v"], src_version=1, k_scales=to["k_scales"], v_scales=to["v_scales"], **kw)
        return {"packed": s["packed"], "to": to}
    if "call" in s:
        return s["call"]()
    args = (s["q"], pool["k"], pool["v"], s["table"], s["lens"], s["versions"], s["out"])
    if case["kind"] == "grouped":
        return dora.dora_decode_attn_grouped(*args, group_size=case["group"], **_kw(case, pool))
    return dora.dora_decode_attn(*args, **_kw(case, pool))


# ---------------------------------------------------------------------------
# what a pass cannot do without, and how exact it is
# ---------------------------------------------------------------------------

def work(case):
    e = 1 if case["fp8"] else 2
    row = case["kv_heads"] * case["d"]  # values of one token's K (or V)
    if case["kind"] == "append":  # the token read and stored, its table entry and length, an fp8 page's scales read and written
        per = 2 * row * 2 + 2 * row * e + 8 + (16 if case["fp8"] else 0)
        return {"bytes": case["layers"] * case["seqs"] * per, "flops": 0}
    lens, shared = _lengths(case)
    n = -(-lens // case["page"])
    if case["kind"] == "migrate":  # pages read and written by the pack and by the unpack
        return {"bytes": int(n.sum()) * 4 * (2 * case["page"] * row * e + (8 if case["fp8"] else 0)), "flops": 0}
    tokens, pages = int(lens.sum()), int(n.sum())
    if shared is not None:
        again = int(shared[np.arange(len(lens)) % case["group"] != 0].sum())  # pages of a prompt that another member has read
        tokens, pages = tokens - again * case["page"], pages - again
    size = tokens * 2 * row * e + pages * (8 if case["fp8"] else 0) + int(n.sum()) * 4 + len(lens) * 4
    size += 2 * case["seqs"] * case["q_heads"] * case["d"] * 2
    return {"bytes": size, "flops": 4 * int(lens.sum()) * case["q_heads"] * case["d"]}


def tolerance(case):
    if case["kind"] in ("append", "migrate"):
        return "exact"
    # probabilities and outputs are rounded to bf16: 2.1e-3 to 2.4e-3 measured against 64 bits
    return {"rel": 8e-3, "max": 0.06}


def exact(case, seed):
    s = prepare(case, seed)
    if case["kind"] == "migrate":
        return None
    if case["kind"] == "append":
        return _exact_append(s) if case["fp8"] else None
    pool, lens, d = s["pool"], _lengths(case)[0], case["d"]
    b, hq, hkv = len(lens), case["q_heads"], case["kv_heads"]
    out = torch.zeros((b, hq, d), dtype=torch.float64, device="cuda")
    for i, length in enumerate(lens):
        rows = s["table"][i, :-(-int(length) // case["page"])].long()
        k, v = (_wide(pool[x][rows], pool[x + "_scales"], rows, case) for x in "kv")
        k = k.permute(1, 0, 3, 2, 4).reshape(hkv, -1, d)[:, :length]  # [Hkv][tokens][d]
        v = v.permute(1, 0, 3, 2).reshape(hkv, -1, d)[:, :length]
        q = s["q"][i].double().view(hkv, hq // hkv, d)
        p = torch.softmax(torch.matmul(k.contiguous(), q.transpose(1, 2).contiguous()) / math.sqrt(d), dim=1)  # [Hkv][tokens][G]
        out[i] = torch.matmul(p.transpose(1, 2).contiguous(), v.contiguous()).view(hq, d)
    return out


def _wide(t, scales, rows, case):
    if not case["fp8"]:
        return t.double()
    t = t.view(torch.float8_e4m3fn).float().double()
    return t * scales[rows].double().view((-1,) + (1,) * (t.dim() - 1))


def _exact_append(s):
    """Page scales after the first token; the codes have no 64-bit value of their own."""
    case, out = s["case"], []
    slot = torch.from_numpy(s["base"] % case["page"]).cuda()
    rows = s["table"].gather(1, torch.from_numpy(s["base"] // case["page"]).cuda()[:, None]).squeeze(1).long()
    for n, pool in enumerate(s["pools"]):
        got = {"k": None, "v": None}
        for name, new in (("k_scales", s["k_new"]), ("v_scales", s["v_new"])):
            scales = pool[name].double()
            fresh = (new[0, n].double().abs().amax(dim=(1, 2)) / FP8_MAX).clamp_min(2.0 ** -126)
            scales[rows] = torch.where(slot == 0, fresh, torch.maximum(fresh, scales[rows]))
            got[name] = scales
        out.append(got)
    return out
