"""What the framework is timed on: whole action-chunk calls, single attention
layers and vision-language prefill, through the entry points a serving
program calls (ActionExpert.generate / generate_steps, attention_noalloc,
PrefixProducer.run), over the range of sizes such a program meets.

A case is a dict of plain values.  Its "kind" says which path it takes:

  generate   a batch of robot requests through the action expert: the pi0
             shape (18 layers, width 1024, 8 query heads over one 256-wide KV
             head, MLP 4096, 32 actions).  "advance" > 0: step-level batching,
             requests at different Euler steps advanced by that many steps.
  attention  one layer of ragged prefix + action attention over device
             buffers, without a handle.
  prefill    prefix production by a PaliGemma-width backbone (width 2048, 8
             query heads over one 256-wide KV head, MLP 16384), a few layers
             of it; per-layer caches or the context form.

Horizons and step counts are comma-separated sets each request draws from;
prefix lengths are uniform in [prefix_lo, prefix_hi].  Everything runs in bf16,
the serving mode (fp32 is there for parity checks).
"""
import math

import numpy as np
import torch

from paper_2607_01088_amd import rosa

DEV = "cuda"
EPS = 1e-6


class Shape:
    """The sizes rosa.model_config and rosa.vlm_config read."""

    def __init__(self, **kw):
        self.action_dim, self.time_emb_dim, self.rms_eps, self.attention_layout, self.rope_base = 32, 1024, EPS, 0, 0.0
        self.__dict__.update(kw)
        self.qkv_dim = (self.n_q_heads + 2 * self.n_kv_heads) * self.head_dim


# ---------------------------------------------------------------- the cases

def _generate(name, robots, prefix, horizons, steps, layout="joint", advance=0):
    return {"name": name, "kind": "generate", "robots": robots, "prefix_lo": prefix[0], "prefix_hi": prefix[1],
            "horizons": horizons, "steps": steps, "layout": layout, "advance": advance}


def _attention(name, robots, prefix, horizons, heads=(8, 1, 256)):
    return {"name": name, "kind": "attention", "robots": robots, "prefix_lo": prefix[0], "prefix_hi": prefix[1],
            "horizons": horizons, "n_q": heads[0], "n_kv": heads[1], "head_dim": heads[2]}


def _prefill(name, jobs, prefix, layers, head_layers=0, causal=0, rope=0.0):
    return {"name": name, "kind": "prefill", "jobs": jobs, "prefix_lo": prefix[0], "prefix_hi": prefix[1],
            "layers": layers, "head_layers": head_layers, "causal": causal, "rope": rope}


def listed():
    return [
        # one robot's request served alone, three camera images and an instruction: the latency case
        _generate("one_robot", 1, (816, 816), "50", "10"),
        # the System-1 batch of 16 robots, short and long horizons and step counts mixed
        _generate("robots_16", 16, (512, 1280), "16,50", "5,10"),
        # a factory fleet in one call: the throughput case
        _generate("fleet_256", 256, (512, 1280), "16,50", "5,10"),
        # the largest: a big fleet with long contexts
        _generate("fleet_512_long", 512, (1024, 2048), "50", "10"),
        # step-level batching: 33 requests at different Euler steps advanced by one
        _generate("step_of_33", 33, (600, 1024), "16,50", "5,10", advance=1),
        # a GR00T-style head alternating cross- and self-attention, 64 robots
        _generate("alternating_64", 64, (512, 1280), "16,50", "5,10", layout="alternating"),
        # one attention layer for one robot: launches and host work
        _attention("attention_one", 1, (816, 816), "50"),
        # one attention layer of the fleet
        _attention("attention_fleet", 256, (512, 1280), "16,50"),
        # grouped-query heads of width 64 with ragged and odd lengths
        _attention("attention_gqa64", 37, (1, 700), "1,17,50", heads=(16, 4, 64)),
        # a new prefix for one robot: prefill of three images and an instruction
        _prefill("prefill_one", 1, (816, 816), 4),
        # prefixes of 32 robots in one call
        _prefill("prefill_32", 32, (600, 1024), 4),
        # the context form for a cross-attending head, instructions causal, rotary positions, odd sizes
        _prefill("prefill_context_5", 5, (333, 901), 2, head_layers=18, causal=48, rope=10000.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["generate", "generate", "attention", "prefill"])
    if kind == "generate":
        lo = _log_int(rng, 64, 1024)
        c = _generate("", _log_int(rng, 1, 300), (lo, lo + rng.randint(0, 768)), rng.choice(["16", "50", "16,50", "7,33,50"]),
                      rng.choice(["5", "10", "5,10", "4,9"]), rng.choice(["joint", "joint", "alternating"]),
                      rng.choice([0, 0, 0, 1]))
    elif kind == "attention":
        lo = _log_int(rng, 1, 1024)
        c = _attention("", _log_int(rng, 1, 300), (lo, lo + rng.randint(0, 768)), rng.choice(["16", "50", "1,17,50"]),
                       rng.choice([(8, 1, 256), (8, 1, 256), (8, 2, 128), (16, 4, 64)]))
    else:
        lo = _log_int(rng, 48, 900)
        form = rng.choice([0, 0, 18])
        c = _prefill("", _log_int(rng, 1, 32), (lo, lo + rng.randint(0, 400)), rng.randint(2, 4), form,
                     rng.choice([0, 0, 31]), rng.choice([0.0, 10000.0]))
    del c["name"]
    return c


def _rng(case, salt):
    """Lengths depend on the case alone, values on the seed."""
    return np.random.default_rng([salt, case.get("robots", case.get("jobs")), case["prefix_lo"], case["prefix_hi"]])


def _lengths(case):
    """(P, H, K, start) of every request: the case's own, the same for every seed."""
    r = _rng(case, 1)
    n = case["robots"]
    P = r.integers(case["prefix_lo"], case["prefix_hi"], size=n, endpoint=True)
    H = r.choice([int(x) for x in case["horizons"].split(",")], size=n)
    K = r.choice([int(x) for x in case.get("steps", "1").split(",")], size=n)
    s = np.floor(r.random(n) * K).astype(int) if case.get("advance") else np.zeros(n, int)
    return [(int(p), int(h), int(k), int(t)) for p, h, k, t in zip(P, H, K, s)]


def _jobs(case):
    r = _rng(case, 2)
    P = r.integers(case["prefix_lo"], case["prefix_hi"], size=case["jobs"], endpoint=True)
    return [int(p) for p in P]


def _expert_shape(case):
    return Shape(n_layers=18, d_model=1024, n_q_heads=8, n_kv_heads=1, head_dim=256, d_mlp=4096,
                 attention_layout=1 if case["layout"] == "alternating" else 0)


def _vlm_shape(case):
    return Shape(n_layers=case["layers"], d_model=2048, n_q_heads=8, n_kv_heads=1, head_dim=256, d_mlp=16384,
                 rope_base=case["rope"])


# ---------------------------------------------------------------- weights and handles
# A program holds one model for its lifetime: the weights are the same for
# every seed, and handles are kept (the last few, each sized for its case).

_kept = {}


def _keep(key, make, most):
    if key not in _kept:
        same = [k for k in _kept if k[0] == key[0]]
        if len(same) >= most:
            old = _kept.pop(same[0])
            if hasattr(old, "close"):
                torch.cuda.synchronize()
                old.close()
        _kept[key] = make()
    return _kept[key]


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    return g


def _bf16_randn(shape, std, g):
    return (torch.randn(shape, device=DEV, generator=g) * std).bfloat16()


def _expert_weights():
    """N(0, 0.02^2) projections; the gates of the residual branches are biased to
    about one half, as trained ones are open, so that every layer counts."""
    def make():
        L, d, f, A, Q = 18, 1024, 4096, 32, 2560
        g = _gen(1)
        sh = {"w_in": (A, d), "w_t1": (1024, d), "w_t2": (d, d), "w_mod": (L, d, 6 * d), "w_qkv": (L, d, Q),
              "w_o": (L, 2048, d), "w_up": (L, d, f), "w_down": (L, f, d), "w_fmod": (d, 2 * d), "w_out": (d, A)}
        w = {k: _bf16_randn(s, 0.02, g).float().cpu().numpy() for k, s in sh.items()}
        for k, n in {"b_in": (d,), "b_t1": (d,), "b_t2": (d,), "b_fmod": (2 * d,), "b_out": (A,)}.items():
            w[k] = (torch.randn(n, device=DEV, generator=g) * 0.02).cpu().numpy()
        b = (torch.randn((L, 6, d), device=DEV, generator=g) * 0.02).cpu().numpy()
        b[:, 2] += 0.5
        b[:, 5] += 0.5
        w["b_mod"] = np.ascontiguousarray(b.reshape(L, 6 * d))
        return w
    return _keep(("expert_weights",), make, 1)


def _vlm_weights(layers, head_layers):
    def make():
        d, f, Q = 2048, 16384, 2560
        g = _gen(2)
        sh = {"w_qkv": (layers, d, Q), "w_o": (layers, 2048, d), "w_up": (layers, d, f), "w_down": (layers, f, d)}
        w = {k: _bf16_randn(s, 0.02, g).float().cpu().numpy() for k, s in sh.items()}
        w["w_ctx"] = _bf16_randn((head_layers, d, 512), 0.02, g).float().cpu().numpy() if head_layers else None
        return w
    return _keep(("vlm_weights", layers, head_layers), make, 1)


def _expert(case):
    ls = _lengths(case)
    cap = (len(ls), max(l[1] for l in ls), sum(l[1] for l in ls), max(l[2] for l in ls), sum(l[0] for l in ls))
    shape = _expert_shape(case)
    return _keep(("expert", cap, shape.attention_layout),
                 lambda: rosa.ActionExpert(shape, "bf16", _expert_weights(), rosa.capacity(*cap)), 2)


def _producer(case):
    P = _jobs(case)
    shape = _vlm_shape(case)

    def make():
        w = _vlm_weights(case["layers"], case["head_layers"])
        return rosa.PrefixProducer(shape, "bf16", w, len(P), sum(P), context_weights=w["w_ctx"])
    return _keep(("producer", case["layers"], case["head_layers"], case["rope"], len(P), sum(P)), make, 2)


# ---------------------------------------------------------------- inputs

KEY_STD = 3.0   # prefix keys are larger than unit normal, so attention is peaked rather than uniform


def _prefixes(P, layers, n_kv, hd, seed):
    """One buffer for all requests' keys and one for their values; request i holds
    [layers][P_i][n_kv][hd] at its offset (in elements)."""
    g = _gen(seed)
    off = np.concatenate([[0], np.cumsum([layers * p * n_kv * hd for p in P])])
    k = torch.empty(int(off[-1]) + 8, device=DEV, dtype=torch.bfloat16).normal_(0.0, KEY_STD, generator=g)
    v = torch.empty(int(off[-1]) + 8, device=DEV, dtype=torch.bfloat16).normal_(0.0, 1.0, generator=g)
    return k, v, [int(x) for x in off[:-1]]


def prepare(case, seed):
    if case["kind"] == "prefill":
        return _prepare_prefill(case, seed)
    ls = _lengths(case)
    M = sum(l[1] for l in ls)
    rows = np.concatenate([[0], np.cumsum([l[1] for l in ls])])
    g = _gen(seed + 7)
    if case["kind"] == "generate":
        e = _expert(case)
        k, v, off = _prefixes([l[0] for l in ls], 18, 1, 256, seed)
        noise = torch.randn((M, 32), device=DEV, generator=g)
        actions = torch.empty_like(noise)
        reqs = []
        for (P, H, K, s), o, r in zip(ls, off, rows):
            reqs.append(rosa.request_struct(k.data_ptr() + 2 * o if P else None, v.data_ptr() + 2 * o if P else None,
                                            noise.data_ptr() + 128 * int(r), actions.data_ptr() + 128 * int(r), P, H, K, s))
        return {"kind": "generate", "expert": e, "k": k, "v": v, "off": off, "noise": noise, "actions": actions,
                "reqs": reqs, "advance": case["advance"]}
    nq, nkv, hd = case["n_q"], case["n_kv"], case["head_dim"]
    shape = _attention_shape(case)
    k, v, off = _prefixes([l[0] for l in ls], 2, nkv, hd, seed)
    qkv = torch.randn((M, (nq + 2 * nkv) * hd), device=DEV, generator=g)
    qkv[:, nq * hd:(nq + nkv) * hd] *= KEY_STD
    qkv = (qkv * 0.64).bfloat16()
    o = torch.empty((M, nq * hd), device=DEV, dtype=torch.bfloat16)
    reqs = [rosa.request_struct(k.data_ptr() + 2 * x if P else None, v.data_ptr() + 2 * x if P else None, o, o, P, H, K)
            for (P, H, K, _), x in zip(ls, off)]
    return {"kind": "attention", "shape": shape, "k": k, "v": v, "off": off, "qkv": qkv, "o": o, "reqs": reqs}


def _attention_shape(case):
    return Shape(n_layers=2, d_model=1024, n_q_heads=case["n_q"], n_kv_heads=case["n_kv"], head_dim=case["head_dim"],
                 d_mlp=4096)


def _prepare_prefill(case, seed):
    p = _producer(case)
    P = _jobs(case)
    g = _gen(seed + 7)
    emb = torch.randn((sum(P), 2048), device=DEV, generator=g).bfloat16()
    lc = case["head_layers"] or case["layers"]
    k = torch.empty(sum(P) * lc * 256, device=DEV, dtype=torch.bfloat16)
    v = torch.empty_like(k)
    jobs, row = [], 0
    for n in P:
        jobs.append(rosa.prefix_job(emb.data_ptr() + 4096 * row, k.data_ptr() + 512 * lc * row,
                                    v.data_ptr() + 512 * lc * row, n, min(case["causal"], n)))
        row += n
    return {"kind": "prefill", "producer": p, "emb": emb, "k": k, "v": v, "jobs": jobs}


def run(s):
    if s["kind"] == "generate":
        if s["advance"]:
            # requests under way bring the state the last call left; here that is the drawn one
            s["actions"].copy_(s["noise"])
            s["expert"].generate_steps(s["reqs"], s["advance"])
        else:
            s["expert"].generate(s["reqs"])
        return s["actions"]
    if s["kind"] == "attention":
        st = rosa.attention_noalloc(s["shape"], "bf16", s["reqs"], 1, s["qkv"], s["o"])
        if st != rosa.ROSA_OK:
            raise rosa.RosaError(st, rosa.last_error_global())
        return s["o"]
    s["producer"].run(s["jobs"])
    return {"k": s["k"], "v": s["v"]}


# ---------------------------------------------------------------- work and tolerance

def work(case):
    if case["kind"] == "prefill":
        P, L, e = _jobs(case), case["layers"], case["head_layers"]
        full = L if e else L - 1          # per-layer caches: the last layer ends with its keys and values
        M = sum(P)
        w = L * 2048 * 2560 + full * (2048 * 2048 + 2 * 2048 * 16384) + e * 2048 * 512
        flops = 2 * M * w
        for p in P:
            c = min(case["causal"], p)
            flops += full * 4 * 8 * 256 * (p * p - c * (c - 1) // 2)
        return {"bytes": 2 * w + 2 * M * 2048 + 2 * 2 * M * 256 * (e or L), "flops": flops}
    ls = _lengths(case)
    if case["kind"] == "attention":
        nq, nkv, hd = case["n_q"], case["n_kv"], case["head_dim"]
        return {"bytes": sum(4 * nkv * hd * P + 2 * H * (2 * nq + 2 * nkv) * hd for P, H, _, _ in ls),
                "flops": sum(4 * nq * hd * H * (P + H) for P, H, _, _ in ls)}
    per_token = 2 * (1024 * 2560 + 2048 * 1024 + 2 * 1024 * 4096)
    flops, taus = 0, set()
    for P, H, K, s in ls:
        n = min(K - s, case["advance"] or K)
        taus |= {(s + j) / K for j in range(n)}
        keys = P + H if case["layout"] == "joint" else (P + H) / 2     # alternating: half the layers each
        flops += n * H * (18 * (per_token + 4 * 8 * 256 * keys) + 4 * 1024 * 32)
    mod = 1024 * (18 * 6144 + 2048) + 2 * 1024 * 1024
    flops += 2 * len(taus) * mod
    kv = sum(P for P, _, _, _ in ls) * (18 if case["layout"] == "joint" else 9) * 1024
    return {"bytes": kv + per_token * 18 + 2 * mod + 2 * 128 * sum(l[1] for l in ls), "flops": int(flops)}


def tolerance(case):
    # bf16 operands between the projections (2^-9 each).  Measured against
    # exact(): whole calls 0.0007 - 0.0016, attention 0.0021 - 0.0026, prefill
    # 0.0027 - 0.0034; four times that, single values ten times further off.
    if case["kind"] == "generate":
        return {"rel": 0.0065, "max": 0.065}
    if case["kind"] == "attention":
        return {"rel": 0.01, "max": 0.1}
    return {"rel": 0.0135, "max": 0.135}


# ---------------------------------------------------------------- 64-bit values

def _f64(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV).double()


def _rms(h):
    return h / torch.sqrt((h * h).mean(-1, keepdim=True) + EPS)


def _attend(q, k, v, visible):
    """q [n, H, nq, hd], k and v [n, S, nkv, hd], visible [n, 1 or H, S] -> [n, H, nq, hd]."""
    n, H, nq, hd = q.shape
    nkv, S = k.shape[2], k.shape[1]
    G = nq // nkv
    qq = q.reshape(n, H, nkv, G, hd).permute(0, 2, 1, 3, 4).reshape(n * nkv, H * G, hd)
    kk = k.permute(0, 2, 3, 1).reshape(n * nkv, hd, S).contiguous()
    vv = v.permute(0, 2, 1, 3).reshape(n * nkv, S, hd).contiguous()
    s = torch.bmm(qq, kk).reshape(n, nkv, H, G, S) / math.sqrt(hd)
    s = s.masked_fill(~visible[:, None, :, None, :], -math.inf)
    o = torch.bmm(torch.softmax(s, -1).reshape(n * nkv, H * G, S), vv)
    return o.reshape(n, nkv, H, G, hd).permute(0, 2, 1, 3, 4).reshape(n, H, nq, hd)


def _chunks(ls, most):
    """Requests of equal horizon, steps and start, sorted by prefix length, at most `most` together."""
    order = sorted(range(len(ls)), key=lambda i: (ls[i][1:], ls[i][0]))
    out = []
    for i in order:
        if out and len(out[-1]) < most and ls[out[-1][0]][1:] == ls[i][1:]:
            out[-1].append(i)
        else:
            out.append([i])
    return out


def _gather(flat, off, P, layer, row):
    """Rows of `row` elements of layer `layer` of several requests, padded to the longest: [n, max P, row]."""
    Pm = max(max(P), 1)
    idx = torch.stack([(o // row + layer * p) + torch.clamp(torch.arange(Pm, device=DEV), max=max(p - 1, 0)) for o, p in zip(off, P)])
    return flat[: flat.numel() // row * row].view(-1, row)[idx]


def _mask(P, H, device=DEV):
    """Visibility over [prefix padded to the longest ; H action keys]: [n, 1, S]."""
    Pm = max(max(P), 1)
    pre = torch.arange(Pm, device=device)[None] < torch.tensor(P, device=device)[:, None]
    return pre, torch.ones((len(P), H), dtype=torch.bool, device=device)


def exact(case, seed):
    if work(case)["flops"] > 6e13:
        return None          # minutes in 64 bits
    s = prepare(case, seed)
    if case["kind"] == "attention":
        return _exact_attention(case, s)
    if case["kind"] == "prefill":
        return _exact_prefill(case, s)
    return _exact_generate(case, s)


def _exact_attention(case, s):
    ls = _lengths(case)
    nq, nkv, hd = case["n_q"], case["n_kv"], case["head_dim"]
    rows = np.concatenate([[0], np.cumsum([l[1] for l in ls])])
    out = torch.empty(s["o"].shape, device=DEV, dtype=torch.float64)
    for ch in _chunks(ls, 8):
        H, P = ls[ch[0]][1], [ls[i][0] for i in ch]
        x = torch.stack([s["qkv"][rows[i]:rows[i] + H] for i in ch]).double()
        q = x[..., : nq * hd].reshape(len(ch), H, nq, hd)
        k = torch.cat([_gather(s["k"], [s["off"][i] for i in ch], P, 1, nkv * hd).double(), x[..., nq * hd:(nq + nkv) * hd]], 1)
        v = torch.cat([_gather(s["v"], [s["off"][i] for i in ch], P, 1, nkv * hd).double(), x[..., (nq + nkv) * hd:]], 1)
        o = _attend(q, k.reshape(len(ch), -1, nkv, hd), v.reshape(len(ch), -1, nkv, hd), torch.cat(_mask(P, H), 1)[:, None])
        for j, i in enumerate(ch):
            out[rows[i]:rows[i] + H] = o[j].reshape(H, nq * hd)
    return out


def _exact_generate(case, s):
    ls = _lengths(case)
    rows = np.concatenate([[0], np.cumsum([l[1] for l in ls])])
    w = {k: _f64(a) for k, a in _expert_weights().items()}
    alt = case["layout"] == "alternating"
    silu, gelu = torch.nn.functional.silu, lambda t: torch.nn.functional.gelu(t, approximate="tanh")
    mods = {}

    def modulation(tau):
        if tau not in mods:
            i = torch.arange(512, device=DEV, dtype=torch.float64)
            a = 1000.0 * tau * torch.pow(torch.tensor(10000.0, device=DEV, dtype=torch.float64), -i / 512)
            c = silu(torch.cat([torch.sin(a), torch.cos(a)]) @ w["w_t1"] + w["b_t1"]) @ w["w_t2"] + w["b_t2"]
            c = silu(c)
            mods[tau] = [(c @ w["w_mod"][l] + w["b_mod"][l]).reshape(6, 1024) for l in range(18)] + [
                (c @ w["w_fmod"] + w["b_fmod"]).reshape(2, 1024)]
        return mods[tau]

    out = torch.empty(s["actions"].shape, device=DEV, dtype=torch.float64)
    for ch in _chunks(ls, 16):
        _, H, K, k0 = ls[ch[0]]
        P, off, n = [ls[i][0] for i in ch], [s["off"][i] for i in ch], len(ch)
        pre, own = _mask(P, H)
        x = torch.stack([s["noise"][rows[i]:rows[i] + H] for i in ch]).double()
        kv = [(_gather(s["k"], off, P, l, 256), _gather(s["v"], off, P, l, 256)) for l in range(18)]
        for k in range(k0, min(K, k0 + (case["advance"] or K))):
            m = modulation(float(np.float32(k) / np.float32(K)))
            h = x @ w["w_in"] + w["b_in"]
            for l in range(18):
                sa, ca, ga, sm, cm, gm = m[l]
                qkv = (_rms(h) * (1 + ca) + sa) @ w["w_qkv"][l]
                ka, va = qkv[..., 2048:2304], qkv[..., 2304:]
                if alt and l % 2:
                    kk, vv, vis = ka, va, own
                elif alt:
                    kk, vv, vis = kv[l][0].double(), kv[l][1].double(), pre
                else:
                    kk, vv = torch.cat([kv[l][0].double(), ka], 1), torch.cat([kv[l][1].double(), va], 1)
                    vis = torch.cat([pre, own], 1)
                o = _attend(qkv[..., :2048].reshape(n, H, 8, 256), kk[:, :, None], vv[:, :, None], vis[:, None])
                h = h + ga * (o.reshape(n, H, 2048) @ w["w_o"][l])
                h = h + gm * (gelu((_rms(h) * (1 + cm) + sm) @ w["w_up"][l]) @ w["w_down"][l])
            x = x + ((_rms(h) * (1 + m[18][1]) + m[18][0]) @ w["w_out"] + w["b_out"]) / K
        for j, i in enumerate(ch):
            out[rows[i]:rows[i] + H] = x[j]
    return out


def _exact_prefill(case, s):
    P, L, e = _jobs(case), case["layers"], case["head_layers"]
    w = {k: _f64(a) for k, a in _vlm_weights(L, e).items() if a is not None}
    lc = e or L
    out = {n: torch.empty(s[n].shape, device=DEV, dtype=torch.float64) for n in ("k", "v")}
    row = 0
    for p in P:
        h = s["emb"][row:row + p].double()
        c = min(case["causal"], p)
        t = torch.arange(p, device=DEV)
        vis = t[None] < torch.clamp(t + 1, min=p - c)[:, None]
        cache = []
        for l in range(L):
            qkv = _rms(h) @ w["w_qkv"][l]
            qk = qkv[:, :2304].reshape(p, 9, 256)
            if case["rope"]:
                a = t[:, None].double() * torch.pow(torch.tensor(case["rope"], device=DEV, dtype=torch.float64),
                                                    -torch.arange(128, device=DEV).double() / 128)
                co, si = torch.cos(a)[:, None], torch.sin(a)[:, None]
                qk = torch.cat([qk[..., :128] * co - qk[..., 128:] * si, qk[..., 128:] * co + qk[..., :128] * si], -1)
            kk, vv = qk[:, 8], qkv[:, 2304:]
            cache.append((kk, vv))
            if not e and l == L - 1:
                break
            o = _attend(qk[None, :, :8], kk[None, :, None], vv[None, :, None], vis[None])
            h = h + o.reshape(p, 2048) @ w["w_o"][l]
            h = h + torch.nn.functional.gelu(_rms(h) @ w["w_up"][l], approximate="tanh") @ w["w_down"][l]
        if e:
            cache = [torch.split(_rms(h) @ w["w_ctx"][i], 256, -1) for i in range(e)]
        for l, (kk, vv) in enumerate(cache):
            at = (row * lc + l * p) * 256
            out["k"][at:at + p * 256] = kk.reshape(-1)
            out["v"][at:at + p * 256] = vv.reshape(-1)
        row += p
    return out
