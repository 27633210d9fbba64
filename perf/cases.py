"""The calls whose speed matters to a user of libgta, as measurable cases.

One case is one call of the C ABI (through the ctypes binding) on tensors that already live on the GPU: a
causal prefill that fills the caches, a decode step, or a chunk of new tokens behind cached ones.  The layers
are those of `paper_2506_17286_amd/workloads.py`, the tests and `bench.py`:

  tiny     the fp32 check workload: 8 heads of 32, two maps, a latent of 64, no RoPE
  paper    one attention layer of the paper's GTA-1B model: 20 heads of 64, 5 maps, one key, one latent of 128
  paper768 the same family at width 768: 12 heads of 64, 3 maps (the 160M-class models)
  1b       16 heads of 128, 4 maps and keys, one latent of 512
  wide     32 heads of 128, 8 maps and keys, one latent of 1024

The paper's layers run with the output projection W_O, as a model does; the others end at the gated heads, as
the repository's benchmark runs them.
"""
from __future__ import annotations

import math
import random
from typing import Dict, List

import torch

from paper_2506_17286_amd import binding as B

LAYERS: Dict[str, Dict] = {
    "tiny": dict(d_model=256, n_heads=8, n_qgroups=2, n_kgroups=2, n_cgroups=1, head_dim=32, latent_dim=64, rope=False),
    "paper": dict(d_model=1280, n_heads=20, n_qgroups=5, n_kgroups=1, n_cgroups=1, head_dim=64, latent_dim=128, rope=True),
    "paper768": dict(d_model=768, n_heads=12, n_qgroups=3, n_kgroups=1, n_cgroups=1, head_dim=64, latent_dim=128, rope=True),
    "1b": dict(d_model=2048, n_heads=16, n_qgroups=4, n_kgroups=4, n_cgroups=1, head_dim=128, latent_dim=512, rope=True),
    "wide": dict(d_model=4096, n_heads=32, n_qgroups=8, n_kgroups=8, n_cgroups=1, head_dim=128, latent_dim=1024, rope=True),
}
ROPE_BASE = 10000.0


def _case(kind: str, layer: str, dtype: str, batch: int, new: int, cached: int = 0, shortest: int = 0, page: int = 0,
          mix: int = 0) -> Dict:
    """new: tokens of the longest sequence in this call (1 for decode); cached: rows of the longest sequence before
    it; shortest > 0: lengths spread evenly over [shortest, longest] by the generator `mix`; page: rows of a page of
    a block-table cache, 0 for contiguous slots."""
    return dict(kind=kind, layer=layer, dtype=dtype, batch=batch, new=new, cached=cached, shortest=shortest, page=page,
                mix=mix)


def listed() -> List[Dict]:
    cases = [
        # the smallest call there is: one short fp32 prompt of a toy layer (the check workload); launches decide
        ("tiny_prefill_f32", _case("prefill", "tiny", "f32", 1, 128)),
        # the paper measures its layer in fp32 first (4 prompts is its small-GPU batch, 64 sequences its server batch)
        ("paper_prefill_f32", _case("prefill", "paper", "f32", 4, 1024)),
        ("paper_decode_f32", _case("decode", "paper", "f32", 64, 1, 2048)),
        # and then in 16 bits: the server batches, and one sequence being generated alone (latency)
        ("paper_prefill", _case("prefill", "paper", "bf16", 32, 2048)),
        ("paper_decode", _case("decode", "paper", "bf16", 64, 1, 2048)),
        ("paper_decode_single", _case("decode", "paper", "bf16", 1, 1, 1000)),
        # 1B-class layer: a full prompt batch, one prompt of an interactive user, a serving batch, long contexts
        # in pages, and the continuation of conversations (new tokens behind cached ones, in pages)
        ("1b_prefill", _case("prefill", "1b", "bf16", 4, 4096)),
        ("1b_prefill_short", _case("prefill", "1b", "bf16", 1, 500)),
        ("1b_decode_batch", _case("decode", "1b", "bf16", 64, 1, 8192)),
        ("1b_decode_long_paged", _case("decode", "1b", "bf16", 8, 1, 32768, page=64)),
        ("1b_chunk_paged", _case("chunk", "1b", "bf16", 4, 2048, 3000, shortest=1200, page=64, mix=3)),
        # the largest: a packed ragged batch of prompts through the wide layer
        ("wide_prefill_ragged", _case("prefill", "wide", "bf16", 16, 16384, shortest=512, mix=8)),
    ]
    return [dict(c, name=name) for name, c in cases]


def _log(rng: random.Random, lo: int, hi: int) -> int:
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng: random.Random) -> Dict:
    """Another case of the same ranges; every size is capped so that none costs more than the largest listed one."""
    family = rng.choice(["tiny", "paper_f32", "paper_f32_decode", "paper", "paper_decode", "prefill", "decode", "chunk",
                         "wide"])
    mix = rng.randrange(1 << 16)
    ragged = rng.random() < 0.5

    def low(n: int) -> int:
        return max(1, n // rng.choice([2, 4, 8])) if ragged else 0

    paper = rng.choice(["paper", "paper", "paper768"])
    if family == "tiny":
        n = _log(rng, 16, 512)
        return _case("prefill", "tiny", "f32", rng.randint(1, 8), n, shortest=low(n), mix=mix)
    if family == "paper_f32":
        n = _log(rng, 64, 1024)
        return _case("prefill", paper, "f32", rng.randint(1, max(1, min(8, 4096 // n))), n, shortest=low(n), mix=mix)
    if family == "paper_f32_decode":
        n = _log(rng, 128, 4096)
        return _case("decode", paper, "f32", _log(rng, 1, min(64, 131072 // n)), 1, n, shortest=low(n), mix=mix)
    if family == "paper":
        n = _log(rng, 64, 2048)
        return _case("prefill", paper, "bf16", _log(rng, 1, 32), n, shortest=low(n), mix=mix)
    page = rng.choice([0, 0, 16, 64])
    if family == "paper_decode":
        n = _log(rng, 128, 8192)
        return _case("decode", paper, "bf16", _log(rng, 1, min(128, 262144 // n)), 1, n, shortest=low(n), page=page, mix=mix)
    if family == "prefill":
        n = _log(rng, 64, 8192)
        return _case("prefill", "1b", "bf16", _log(rng, 1, max(1, min(16, 32768 // n))), n, shortest=low(n), mix=mix)
    if family == "decode":
        n = _log(rng, 256, 32768)
        return _case("decode", rng.choice(["1b", "1b", "wide"]), "bf16", _log(rng, 1, max(1, min(128, 524288 // n))), 1, n,
                     shortest=low(n), page=page, mix=mix)
    if family == "chunk":
        n = _log(rng, 32, 2048)
        return _case("chunk", "1b", "bf16", rng.randint(1, 8), n, rng.randint(1, 8192), shortest=low(n),
                     page=rng.choice([0, 64]), mix=mix)
    n = _log(rng, 512, 16384)
    return _case("prefill", "wide", "bf16", _log(rng, 1, max(1, 65536 // n)), n, shortest=low(n), mix=mix)


# ------------------------------------------------------------------------------------------ sizes
def _lengths(case: Dict):
    """(new tokens, rows cached before) of every sequence; the first sequence has the longest of both."""
    b, longest, cached, low = case["batch"], case["new"], case["cached"], case["shortest"]
    rng = random.Random(case["mix"])
    top = cached if case["kind"] == "decode" else longest
    spread = [top] + [rng.randint(min(low, top), top) if low else top for _ in range(b - 1)]
    if case["kind"] == "decode":
        return [1] * b, spread
    if case["kind"] == "chunk":
        return spread, [cached] + [rng.randint(1, cached) if low else cached for _ in range(b - 1)]
    return spread, [0] * b


def _capacity(case: Dict) -> int:
    """Rows of a cache slot: the longest sequence and some room, in whole pages of 64."""
    new, cached = _lengths(case)
    return (max(n + p for n, p in zip(new, cached)) + 64 + 63) // 64 * 64


def _with_wo(case: Dict) -> bool:
    return case["layer"].startswith("paper")


def work(case: Dict) -> Dict[str, float]:
    """Operands once: hidden states, weights, the rows of both caches that are read or written, outputs."""
    L = LAYERS[case["layer"]]
    es = 2 if case["dtype"] == "bf16" else 4
    new, cached = _lengths(case)
    H, dh, dl, nq, nh = L["d_model"], L["head_dim"], L["latent_dim"], L["n_qgroups"], L["n_heads"]
    row = L["n_kgroups"] * dh + L["n_cgroups"] * dl
    wtot = nq * dh + row + nh * dh
    tokens = sum(new)
    wo = _with_wo(case)
    weights = H * wtot + nh * dl * dh + (nh * dh * H if wo else 0)
    data = tokens * H + tokens * (H if wo else nh * dh) + row * (tokens + sum(cached))
    pairs = sum(n * p + n * (n + 1) // 2 for n, p in zip(new, cached))
    flops = 2.0 * tokens * H * wtot + 2.0 * nq * (dh + dl) * pairs + 2.0 * tokens * nh * dl * dh
    if wo:
        flops += 2.0 * tokens * nh * dh * H
    return {"bytes": float(es * (weights + data)), "flops": flops}


def tolerance(case: Dict) -> Dict[str, float]:
    # The two-norm error against 64 bits is 3e-3 for bf16 operands with fp32 sums (roundings of Q, K, C, P, L, the
    # gate and the output) and 3e-7 for fp32; another order of the sums or of the roundings stays within these.
    return {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 5e-6}


# ------------------------------------------------------------------------------------------ inputs
def _draw_inputs(case: Dict, seed: int) -> Dict:
    """Hidden states N(0,1), weights N(0, 0.02^2), rows cached before the call N(0,1), pages in random order."""
    L = LAYERS[case["layer"]]
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    g = torch.Generator(device="cuda")
    g.manual_seed(1000003 * (seed + 1) + case["mix"])

    def normal(*shape, std=1.0):
        t = torch.empty(shape, dtype=dt, device="cuda").normal_(0.0, 1.0, generator=g)
        return t if std == 1.0 else t.mul_(std)

    H, dh, dl, nh = L["d_model"], L["head_dim"], L["latent_dim"], L["n_heads"]
    kw, cw = L["n_kgroups"] * dh, L["n_cgroups"] * dl
    w = {"wq": normal(H, L["n_qgroups"] * dh, std=0.02), "wk": normal(H, kw, std=0.02), "wc": normal(H, cw, std=0.02),
         "wg": normal(H, nh * dh, std=0.02), "wp": normal(nh, dl, dh, std=0.02),
         "wo": normal(nh * dh, H, std=0.02) if _with_wo(case) else None}
    new, cached = _lengths(case)
    x = normal(sum(new), H)
    cap, page, b = _capacity(case), case["page"], case["batch"]
    fill = normal if max(cached) else lambda *shape: torch.zeros(shape, dtype=dt, device="cuda")
    if page:
        pages = b * (cap // page)
        perm = torch.randperm(pages, generator=torch.Generator().manual_seed(seed + 17)).to(torch.int32)
        k, c, table = fill(pages, page, kw), fill(pages, page, cw), perm.view(b, -1).cuda()
    else:
        k, c, table = fill(b, cap, kw), fill(b, cap, cw), None
    return dict(w=w, x=x, k=k, c=c, table=table, new=new, cached=cached)


def prepare(case: Dict, seed: int) -> Dict:
    L = LAYERS[case["layer"]]
    s = _draw_inputs(case, seed)
    s["kind"], s["batch"], s["total"], s["longest"] = case["kind"], case["batch"], sum(s["new"]), max(s["new"])
    s["cfg"] = B.make_config(dtype=case["dtype"], rope_base=ROPE_BASE, **L)
    s["weights"] = B.make_weights(s["w"])
    s["start"] = torch.tensor(s["cached"], dtype=torch.int32, device="cuda")
    s["seq_lens"], status = s["start"].clone(), torch.zeros_like(s["start"])
    s["status"] = status
    s["cache"] = (B.make_paged_cache(s["k"], s["c"], s["seq_lens"], status, s["table"]) if case["page"]
                  else B.make_cache(s["k"], s["c"], s["seq_lens"], status))
    ends = [0]
    for n in s["new"]:
        ends.append(ends[-1] + n)
    s["cu"] = torch.tensor(ends, dtype=torch.int32, device="cuda")
    width = L["d_model"] if _with_wo(case) else L["n_heads"] * L["head_dim"]
    s["out"] = torch.empty((s["total"], width), dtype=s["x"].dtype, device="cuda")
    mode = {"prefill": B.GTA_MODE_PREFILL, "decode": B.GTA_MODE_DECODE, "chunk": B.GTA_MODE_PREFILL_CHUNK}[case["kind"]]
    longest = s["cache"].max_seq if case["kind"] == "decode" else s["longest"]
    s["ws"] = B.alloc_workspace(B.gta_workspace_bytes(s["cfg"], mode, case["batch"], s["total"], longest))
    return s


def run(s: Dict) -> Dict:
    if s["kind"] == "prefill":
        B.gta_prefill(s["cfg"], s["weights"], s["x"], s["cu"], s["batch"], s["total"], s["longest"], s["cache"], None,
                      s["out"], s["ws"])
    else:
        # every pass starts from the same cached lengths: one small kernel where a serving loop sets its lengths
        torch.add(s["start"], 0, out=s["seq_lens"])
        if s["kind"] == "decode":
            B.gta_decode(s["cfg"], s["weights"], s["x"], s["batch"], s["cache"], None, s["out"], 0, s["ws"])
        else:
            B.gta_prefill_chunk(s["cfg"], s["weights"], s["x"], s["cu"], s["batch"], s["total"], s["longest"],
                                s["cache"], None, s["out"], s["ws"])
    return {"out": s["out"], "k": s["k"], "c": s["c"], "seq_lens": s["seq_lens"], "status": s["status"]}


# ------------------------------------------------------------------------------------------ 64-bit answer
def exact(case: Dict, seed: int) -> Dict:
    """The definition in float64: projections, RoPE, cache rows, one causal softmax map per group applied to the
    latent values, decoder, gate, W_O."""
    L = LAYERS[case["layer"]]
    s = _draw_inputs(case, seed)
    w = {n: t.double() for n, t in s["w"].items() if t is not None}
    dh, dl, nq, nk, nc, nh = (L[n] for n in ("head_dim", "latent_dim", "n_qgroups", "n_kgroups", "n_cgroups", "n_heads"))
    k_cache, c_cache = s["k"].double(), s["c"].double()
    k_rows, c_rows = k_cache.view(-1, nk * dh), c_cache.view(-1, nc * dl)
    cap, page = _capacity(case), case["page"]
    half = dh // 2
    theta = ROPE_BASE ** (-torch.arange(half, dtype=torch.float64, device="cuda") / half)
    out, at = [], 0
    for b, (n, p) in enumerate(zip(s["new"], s["cached"])):
        x = s["x"][at:at + n].double()
        at += n
        pos = torch.arange(p, p + n, device="cuda")
        cos, sin = (f(pos.double()[:, None] * theta)[:, None, :] for f in (torch.cos, torch.sin))

        def turned(t, groups):
            t = t.view(n, groups, dh)
            if not L["rope"]:
                return t
            lo, hi = t[..., :half], t[..., half:]
            return torch.cat([lo * cos - hi * sin, hi * cos + lo * sin], dim=-1)

        q = turned(x @ w["wq"], nq)
        rows = torch.arange(p + n, device="cuda")
        rows = s["table"][b].long()[rows // page] * page + rows % page if page else rows + b * cap
        k_rows[rows[p:]] = turned(x @ w["wk"], nk).reshape(n, nk * dh)
        c_rows[rows[p:]] = x @ w["wc"]
        k, c = k_rows[rows].view(p + n, nk, dh), c_rows[rows].view(p + n, nc, dl)
        gate = torch.sigmoid(x @ w["wg"])
        o = torch.empty((n, nh * dh), dtype=torch.float64, device="cuda")
        for g in range(nq):
            kg, cg = k[:, g // (nq // nk)].contiguous(), c[:, g // (nq // nc)].contiguous()
            for i in range(0, n, 2048):
                m = min(n, i + 2048)
                a = q[i:m, g] @ kg[:p + m].t() / math.sqrt(dh)
                a.masked_fill_(torch.arange(p + m, device="cuda")[None, :] > pos[i:m, None], -math.inf)
                l = torch.softmax(a, dim=-1) @ cg[:p + m]
                for h in range(g * (nh // nq), (g + 1) * (nh // nq)):
                    o[i:m, h * dh:(h + 1) * dh] = (l @ w["wp"][h]) * gate[i:m, h * dh:(h + 1) * dh]
        out.append(o @ w["wo"] if "wo" in w else o)
    lens = torch.tensor([n + p for n, p in zip(s["new"], s["cached"])], dtype=torch.int32, device="cuda")
    return {"out": torch.cat(out), "k": k_cache, "c": c_cache, "seq_lens": lens, "status": torch.zeros_like(lens)}
