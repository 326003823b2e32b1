"""The work this library does for a model, as cases that can be timed and compared.

Twelve listed cases, each one layer's call (or the calls of one layer's step) through
`paper_2605_28640_amd.binding`; `draw` gives more of the same ranges.  Every kind of case:

  decode     one token: append to the gated cache with its page bounds, pick pages, attend
             (`rat_scan` + `sparse_attn_decode`, or `rat_decode_step`)
  dense      one token over a whole cache, as after a SnapKV compression (append + attend)
  scan       the recurrence over a prompt, or over the next chunk of one, with page bounds
  moba       block routing and the routed attention of a prompt
  prefill    causal attention of a prompt over all its tokens
  snapkv     cache compression after a prompt

Inputs follow the library's synthetic workloads (synth.py): standard normal keys and values,
gates sigmoid(N(4.2, 0.5^2)), a few tokens aligned with a retrieval direction that the queries
look for.  The stored states that the attention kinds start from are made here in plain torch,
by the same recurrence with one gate per channel.
"""
import math

import torch

from paper_2605_28640_amd import binding as rs

DEV = "cuda"
STEPS = 256  # decode steps that a cache has room for; the loop then starts over


def _decode(name, B, Hq, Hkv, D, T, P, K, dtype="bf16", device_length=False):
    return {"name": name, "kind": "decode", "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "T": T, "P": P, "K": K,
            "dtype": dtype, "device_length": device_length}


def _dense(name, B, Hq, Hkv, D, T, dtype="bf16"):
    return {"name": name, "kind": "dense", "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "T": T, "dtype": dtype}


def _scan(name, B, Hkv, D, t0, T, Tcap, P, dtype="bf16"):
    return {"name": name, "kind": "scan", "B": B, "Hkv": Hkv, "D": D, "t0": t0, "T": T, "Tcap": Tcap, "P": P,
            "dtype": dtype}


def _moba(name, B, Hq, Hkv, D, T, block, K):
    return {"name": name, "kind": "moba", "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "T": T, "block": block, "K": K}


def _prefill(name, B, Hq, Hkv, D, T):
    return {"name": name, "kind": "prefill", "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "T": T}


def _snapkv(name, B, Hq, Hkv, D, T, W, keep, pool):
    return {"name": name, "kind": "snapkv", "B": B, "Hq": Hq, "Hkv": Hkv, "D": D, "T": T, "W": W, "keep": keep,
            "pool": pool}


def listed():
    return [
        # the smallest call: float32 storage, two heads of 64 channels, a 2K prompt at 1/8 of its pages
        _decode("decode_f32_2k", 1, 2, 2, 64, 2048, 16, 16, dtype="f32"),
        # the paper's own setting, 4096 tokens and the 8 best pages of 64, for a batch of eight requests
        _decode("decode_4k_b8", 8, 32, 32, 128, 4096, 64, 8),
        # one long conversation with grouped queries, 1/8 of the pages, through the replayable step
        _decode("decode_gqa_32k", 1, 32, 8, 128, 32768, 16, 256, device_length=True),
        # the benchmark's workload: 7B-sized layer, batch 4, 64K tokens, 1/16 of the pages
        _decode("decode_64k_b4", 4, 32, 32, 128, 65536, 16, 256),
        # one token over the cache that a SnapKV compression of 128K tokens to 1/8 leaves
        _dense("decode_dense_16k", 1, 32, 8, 128, 16384 + 32),
        # the whole prompts of the benchmark's workload
        _scan("scan_64k_b4", 4, 32, 128, 0, 65536, 65536 + 512, 16),
        # the next piece of a long prompt that arrives in pieces of no round size
        _scan("scan_piece_3001", 1, 8, 128, 5003, 3001, 32768, 16),
        # routed prefill: 32K tokens, the 3 best blocks of 512
        _moba("moba_32k", 1, 32, 32, 128, 32768, 512, 3),
        # the paper's own routed prefill at about 4K tokens: the 8 best blocks of 64, two prompts of no round size
        _moba("moba_4001_b2", 2, 32, 32, 128, 4001, 64, 8),
        # an ordinary long prompt with grouped queries, all tokens attended
        _prefill("prefill_16001_gqa", 1, 32, 8, 128, 16001),
        # 128K tokens compressed to 1/8
        _snapkv("snapkv_128k", 1, 32, 8, 128, 131072, 32, 16384, 7),
        # the paper's own compression: 4096 tokens to 512, window 64, a batch of eight
        _snapkv("snapkv_4k_b8", 8, 32, 32, 128, 4096, 64, 512, 7),
    ]


def _spread(rng, lo, hi):
    """A whole number between lo and hi, evenly over its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["decode", "decode", "dense", "scan", "scan", "moba", "prefill", "snapkv"])
    Hkv = rng.choice([2, 4, 8, 8, 32])
    G = 1 if Hkv == 32 else rng.choice([1, 2, 4])
    D = rng.choice([64, 128, 128, 128])
    if kind == "decode":
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        P = rng.choice([16, 16, 32, 64])
        T = _spread(rng, 1000, 65536)
        B = _spread(rng, 1, max(1, min(16, (4 * 32 * 65536) // (Hkv * T))))
        K = max(3, int(-(-T // P) * rng.choice([1 / 4, 1 / 8, 1 / 16])))
        c = _decode("", B, Hkv * G, Hkv, D, T, P, K, dtype=dtype, device_length=rng.random() < 0.3)
    elif kind == "dense":
        T = _spread(rng, 200, 65536)
        B = _spread(rng, 1, max(1, min(16, (4 * 32 * 32768) // (Hkv * T))))
        c = _dense("", B, Hkv * G, Hkv, D, T, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]))
    elif kind == "scan":
        T = _spread(rng, 20, 65536)
        B = _spread(rng, 1, max(1, min(16, (4 * 32 * 32768) // (Hkv * T))))
        t0 = 0 if rng.random() < 0.5 else rng.randrange(1, 8192)
        Tcap = -(-(t0 + (4 if t0 else 1) * T) // 64) * 64
        c = _scan("", B, Hkv, D, t0, T, Tcap, rng.choice([16, 32, 64]), dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]))
    elif kind == "moba":
        block, K = rng.choice([(64, 16), (64, 8), (64, 4), (128, 8), (128, 4), (256, 4), (512, 3)])
        T = _spread(rng, 1500, min(32768, 200 * block))
        B = _spread(rng, 1, max(1, min(8, 32 * 32768 // (Hkv * G * T))))
        c = _moba("", B, Hkv * G, Hkv, D, T, block, K)
    elif kind == "prefill":
        T = _spread(rng, 100, 16000)
        B = _spread(rng, 1, max(1, min(8, 32 * 16000 ** 2 // (Hkv * G * T * T))))
        c = _prefill("", B, Hkv * G, Hkv, D, T)
    else:
        W = rng.choice([32, 64]) if G < 4 else 32
        T = _spread(rng, 2000, 131072)
        B = _spread(rng, 1, max(1, min(8, 8 * 131072 // (Hkv * T))))
        c = _snapkv("", B, Hkv * G, Hkv, D, T, W, (T - W) // rng.choice([4, 8, 16]), rng.choice([1, 5, 7]))
    del c["name"]
    return c


# ---- inputs -----------------------------------------------------------------------------


def _dt(case):
    return torch.float32 if case.get("dtype") == "f32" else torch.bfloat16


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(20260528 + 1000003 * int(seed))
    return g


def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEV)


def _gate(gen, *shape):
    return torch.sigmoid_(_normal(gen, *shape).mul_(0.5).add_(4.2))


def _directions(gen, B, Hkv, D):
    d = _normal(gen, B, Hkv, D)
    return d * (math.sqrt(D) / d.norm(dim=-1, keepdim=True))


def _needles(gen, x, dirs, n):
    """Plant n tokens aligned with the retrieval direction, at depths spread over the sequence."""
    B, H, T, D = x.shape
    pos = ((torch.arange(n, device=DEV) + 0.5) * T / n).long()
    x[:, :, pos] = 3.0 * dirs[:, :, None] + 0.3 * _normal(gen, B, H, n, D)


def _decayed(x, gate):
    """The recurrence s_t = a s_{t-1} + (1 - a) x_t with one gate per channel (its last 512 terms), in place."""
    x.mul_(1 - gate)
    a = gate
    for k in range(9):
        if (1 << k) >= x.shape[2]:
            break
        x[:, :, 1 << k:] += x[:, :, :-(1 << k)] * a
        a = a * a
    return x


def _cache(gen, B, Hkv, D, T, Tcap, dtype, dirs=None, n=16):
    """A cache [B, Hkv, Tcap, D] holding T states."""
    out = torch.zeros(B, Hkv, Tcap, D, device=DEV, dtype=dtype)
    gate = _gate(gen, 1, Hkv, 1, D)
    for b in range(B):
        x = _normal(gen, 1, Hkv, T, D)
        if dirs is not None:
            _needles(gen, x, dirs[b:b + 1], n)
        out[b:b + 1, :, :T] = _decayed(x, gate)
    return out


def _carry(cache, T):
    """The recurrence's carry after T stored tokens: a float32 copy of the last state, zeros before the first."""
    B, H, _, D = cache.shape
    carry = torch.zeros(B, H, D, device=DEV)
    if T:
        carry.copy_(cache[:, :, T - 1])
    return carry


def _page_bounds(kc, T, P):
    """[B, Hkv, Tcap / P, 2, D]: smallest and largest stored key of each page over its tokens below T."""
    B, H, Tcap, D = kc.shape
    meta = torch.zeros(B, H, Tcap // P, 2, D, device=DEV, dtype=kc.dtype)
    full = T // P
    x = kc[:, :, :full * P].view(B, H, full, P, D)
    meta[:, :, :full, 0], meta[:, :, :full, 1] = x.amin(3), x.amax(3)
    if T % P:
        x = kc[:, :, full * P:T]
        meta[:, :, full, 0], meta[:, :, full, 1] = x.amin(2), x.amax(2)
    return meta


def _queries(gen, dirs, Hq, rows=None, every=1):
    """Queries [B, Hq(, rows), D]: every `every`-th one looks for the retrieval direction, the others are noise."""
    B, Hkv, D = dirs.shape
    d = dirs.repeat_interleave(Hq // Hkv, 1)
    if rows is None:
        return d + 0.25 * _normal(gen, B, Hq, D)
    q = _normal(gen, B, Hq, rows, D)
    q[:, :, every - 1::every] = d[:, :, None] + 0.25 * q[:, :, every - 1::every]
    return q


def _new(*shape, dtype=torch.float32):
    return torch.empty(*shape, device=DEV, dtype=dtype)


def _inputs(case, seed):
    """The tensors of a case, without the library's handles."""
    gen, dt, kind = _gen(seed), _dt(case), case["kind"]
    B, Hkv, D, T = (case[n] for n in ("B", "Hkv", "D", "T"))
    if kind == "scan":
        x = {"k": _normal(gen, B, Hkv, T, D).to(dt), "v": _normal(gen, B, Hkv, T, D).to(dt), "g": _gate(gen, B, Hkv, T, D)}
        t0, Tcap = case["t0"], case["Tcap"]
        x["k_cache"], x["v_cache"] = (_cache(gen, B, Hkv, D, t0, Tcap, dt) if t0 else
                                      torch.zeros(B, Hkv, Tcap, D, device=DEV, dtype=dt) for _ in range(2))
        x["meta"] = _page_bounds(x["k_cache"], t0, case["P"])
        x["state_k"], x["state_v"] = (_carry(x[n], t0) for n in ("k_cache", "v_cache"))
        return x
    Hq, dirs = case["Hq"], _directions(gen, B, Hkv, D)
    if kind in ("decode", "dense"):
        P = case.get("P", 16)
        Tcap = -(-(T + STEPS) // P) * P
        x = {"k_cache": _cache(gen, B, Hkv, D, T, Tcap, dt, dirs), "v_cache": _cache(gen, B, Hkv, D, T, Tcap, dt)}
        if kind == "decode":
            x["meta"] = _page_bounds(x["k_cache"], T, P)
        x["state_k"], x["state_v"] = (_carry(x[n], T) for n in ("k_cache", "v_cache"))
        x["k"], x["v"] = (_normal(gen, B, Hkv, 1, D).to(dt) for _ in range(2))
        x["g"], x["q"] = _gate(gen, B, Hkv, 1, D), _queries(gen, dirs, Hq).to(dt)
        return x
    x = {"k_cache": _cache(gen, B, Hkv, D, T, T, dt, dirs), "v_cache": _cache(gen, B, Hkv, D, T, T, dt)}
    x["q"] = _queries(gen, dirs, Hq, case["W"], 1).to(dt) if kind == "snapkv" else _queries(gen, dirs, Hq, T, 64).to(dt)
    return x


def prepare(case, seed):
    s, kind, dt = _inputs(case, seed), case["kind"], _dt(case)
    B, Hkv, D, T = (case[n] for n in ("B", "Hkv", "D", "T"))
    s.update(case, scale=1.0 / math.sqrt(D))
    Hq = case.get("Hq", Hkv)
    if kind == "scan":
        s["shape"] = rs.make_shape(B, Hq, Hkv, D, case["Tcap"], case["P"], dt)
        s["ws"] = rs.Workspace(rs.rat_scan_workspace_bytes(s["shape"], T))
        s["at"] = case["t0"]
    elif kind in ("decode", "dense"):
        Tcap, P, K = s["k_cache"].shape[2], case.get("P", 16), case.get("K", 0)
        shape = s["shape"] = rs.make_shape(B, Hq, Hkv, D, Tcap, P, dt)
        s["end"], s["at"] = min(Tcap, T + STEPS), T
        s["out"], s["lse"] = _new(B, Hq, D, dtype=dt), _new(B, Hq)
        if kind == "decode":
            s["idx"] = _new(B, Hq, K, dtype=torch.int32)
        if case.get("device_length"):
            s["ws"] = rs.Workspace(rs.rat_decode_step_workspace_bytes(shape, s["end"], K))
            rs.rat_decode_state_set(s["ws"], T)
        else:
            s["ws"] = rs.Workspace(rs.sparse_attn_decode_workspace_bytes(shape, s["end"], K))
    elif kind in ("moba", "prefill"):
        shape = s["shape"] = rs.make_shape(B, Hq, Hkv, D, T, 16, dt)
        s["out"], s["lse"] = _new(B, Hq, T, D, dtype=dt), _new(B, Hq, T)
        block, K = case.get("block", 64), case.get("K", 0)
        need = rs.sparse_attn_prefill_workspace_bytes(shape, T, block, K)
        if kind == "moba":
            s["means"] = _new(B, Hkv, -(-T // block), D)
            s["idx"] = _new(B, Hq, T, K, dtype=torch.int32)
            need = max(need, rs.moba_select_prefill_workspace_bytes(shape, T, block))
        s["ws"] = rs.Workspace(need)
    else:
        shape = s["shape"] = rs.make_shape(B, Hq, Hkv, D, T, 16, dt)
        rows = s["rows"] = case["keep"] + case["W"]
        s["k_out"], s["v_out"] = _new(B, Hkv, rows, D, dtype=dt), _new(B, Hkv, rows, D, dtype=dt)
        s["idx"], s["votes"] = _new(B, Hkv, case["keep"], dtype=torch.int32), _new(B, Hkv, T - case["W"])
        s["ws"] = rs.Workspace(rs.snapkv_compress_workspace_bytes(shape, T, case["W"]))
    return s


# ---- one pass ---------------------------------------------------------------------------


def run(s):
    kind = s["kind"]
    if kind == "decode":
        if s["at"] >= s["end"]:  # the cache is full: the next request of this length
            s["at"] = s["T"]
            if s["device_length"]:
                rs.rat_decode_state_set(s["ws"], s["T"])
        t = s["at"]
        s["at"] = t + 1
        if s["device_length"]:
            rs.rat_decode_step(s["shape"], s["k"], s["v"], s["g"], s["state_k"], s["state_v"], s["k_cache"], s["v_cache"],
                               s["meta"], s["q"], s["scale"], s["K"], 1, 1, s["end"], s["out"], s["lse"], s["idx"], s["ws"])
        else:
            rs.rat_scan(s["shape"], s["k"], s["v"], s["g"], s["state_k"], s["state_v"], s["k_cache"], s["v_cache"], t, 1,
                        None, s["meta"])
            rs.sparse_attn_decode(s["shape"], s["q"], s["k_cache"], s["v_cache"], t + 1, s["scale"], None, s["K"], s["meta"],
                                  1, 1, s["out"], s["lse"], s["idx"], s["ws"])
        return [s["out"], s["lse"], s["idx"], s["state_k"], s["state_v"], s["k_cache"], s["v_cache"], s["meta"]]
    if kind == "dense":
        if s["at"] >= s["end"]:
            s["at"] = s["T"]
        t = s["at"]
        s["at"] = t + 1
        rs.rat_scan(s["shape"], s["k"], s["v"], s["g"], s["state_k"], s["state_v"], s["k_cache"], s["v_cache"], t, 1, None)
        rs.sparse_attn_decode(s["shape"], s["q"], s["k_cache"], s["v_cache"], t + 1, s["scale"], None, 0, None, 0, 0,
                              s["out"], s["lse"], None, s["ws"])
        return [s["out"], s["lse"], s["state_k"], s["state_v"], s["k_cache"], s["v_cache"]]
    if kind == "scan":
        t = s["at"]
        if t == 0:  # a fresh prompt
            s["state_k"].zero_()
            s["state_v"].zero_()
        else:  # the next piece; a full cache makes room for the next prompt's
            s["at"] = t + s["T"] if t + 2 * s["T"] <= s["Tcap"] else s["t0"]
        rs.rat_scan(s["shape"], s["k"], s["v"], s["g"], s["state_k"], s["state_v"], s["k_cache"], s["v_cache"], t, s["T"],
                    s["ws"], s["meta"])
        return [s["state_k"], s["state_v"], s["k_cache"], s["v_cache"], s["meta"]]
    if kind == "moba":
        rs.moba_select_prefill(s["shape"], s["q"], s["k_cache"], s["T"], s["block"], s["K"], 0, s["means"], s["idx"], s["ws"])
        rs.sparse_attn_prefill(s["shape"], s["q"], s["k_cache"], s["v_cache"], s["T"], s["block"], s["scale"], s["idx"],
                               s["K"], s["out"], s["lse"], s["ws"])
        return [s["out"], s["lse"], s["idx"], s["means"]]
    if kind == "prefill":
        rs.sparse_attn_prefill(s["shape"], s["q"], s["k_cache"], s["v_cache"], s["T"], 64, s["scale"], None, 0, s["out"],
                               s["lse"], s["ws"])
        return [s["out"], s["lse"]]
    rs.snapkv_compress(s["shape"], s["q"], s["k_cache"], s["v_cache"], s["T"], s["W"], s["keep"], s["pool"], s["scale"],
                       s["k_out"], s["v_out"], s["rows"], s["idx"], s["votes"], s["ws"])
    return [s["k_out"], s["v_out"], s["idx"], s["votes"]]


# ---- what a pass cannot do without ------------------------------------------------------


def work(case):
    kind, e = case["kind"], 4 if case.get("dtype") == "f32" else 2
    B, Hkv, D, T = (case[n] for n in ("B", "Hkv", "D", "T"))
    Hq = case.get("Hq", Hkv)
    if kind == "scan":  # k, v and gates in, states and page bounds out; four operations per state
        n = B * Hkv * T * D
        return {"bytes": n * (4 * e + 4) + 2 * e * n // case["P"], "flops": 8 * n}
    if kind == "decode":  # all page bounds, the picked pages of K and V, and small vectors
        pages = -(-(T + 1) // case["P"])
        rows = min(Hq * case["K"], Hkv * pages) * case["P"]
        return {"bytes": B * D * e * (2 * Hkv * pages + 2 * rows + 2 * Hq + 6 * Hkv),
                "flops": B * Hq * D * (4 * pages + 4 * case["K"] * case["P"])}
    if kind == "dense":
        return {"bytes": B * D * e * (2 * Hkv * T + 2 * Hq + 6 * Hkv), "flops": 4 * B * Hq * D * T}
    if kind == "prefill":
        return {"bytes": 2 * B * D * T * (2 * Hq + 2 * Hkv), "flops": 2 * B * Hq * D * T * (T + 1)}
    if kind == "moba":
        block, K = case["block"], case["K"]
        pairs = gate = 0
        for j in range(-(-T // block)):  # the rows of block j see their own block causally and up to K - 1 earlier ones
            n = min(block, T - j * block)
            pairs += n * (n + 1) // 2 + n * min(K - 1, j) * block
            gate += n * j
        return {"bytes": 2 * B * D * T * (2 * Hq + 2 * Hkv) + 4 * B * Hq * T * (K + 1),
                "flops": B * Hq * D * (4 * pairs + 2 * gate)}
    kept = case["keep"] + case["W"]
    return {"bytes": 2 * B * Hkv * D * (T + 3 * kept) + 4 * B * Hkv * (T + case["keep"]) + 2 * B * Hq * case["W"] * D,
            "flops": 2 * B * Hq * case["W"] * D * T}


def tolerance(case):
    kind, f32 = case["kind"], case.get("dtype") == "f32"
    if kind == "scan":  # states in 32 bits; a stored bf16 state may round to its other neighbour
        return {"rel": 1e-5, "max": 1e-4} if f32 else {"rel": 2e-3, "max": 1e-2}
    if kind in ("decode", "dense"):  # one page swapped at a tie moves the ascending list between the two
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-2} if f32 else {"rel": 5e-3, "max": 5e-2, "differ": 1e-2}
    if kind == "prefill":
        return {"rel": 1e-2, "max": 0.1}
    if kind == "moba":
        return {"rel": 1e-2, "max": 0.1, "differ": 1e-3}
    # votes are sums of 32-bit probabilities (7e-7 from the exact ones); the kept rows are copies
    return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}


# ---- the same in 64 bits ----------------------------------------------------------------


def _scan64(x, g, s0):
    """Eq. 1 over [N, T, D] in 64 bits, 256 pieces of the sequence side by side."""
    N, T, D = x.shape
    c = max(1, -(-T // 256))
    n = -(-T // c)
    xp = torch.zeros(N, n * c, D, device=DEV, dtype=torch.float64)
    gp = torch.ones(N, n * c, D, device=DEV, dtype=torch.float64)
    xp[:, :T], gp[:, :T] = x, g
    xp, gp = xp.view(N, n, c, D), gp.view(N, n, c, D)
    s = torch.zeros(N, n, D, device=DEV, dtype=torch.float64)
    a = torch.ones_like(s)
    loc, dec = torch.empty_like(xp), torch.empty_like(xp)
    for i in range(c):
        s = gp[:, :, i] * s + (1 - gp[:, :, i]) * xp[:, :, i]
        a = a * gp[:, :, i]
        loc[:, :, i], dec[:, :, i] = s, a
    carry = s0.double()
    for j in range(n):
        loc[:, j] += dec[:, j] * carry[:, None]
        carry = loc[:, j, -1]
    return loc.view(N, n * c, D)[:, :T], carry


def _exact_scan(case, x):
    B, Hkv, D, T, t0 = (case[n] for n in ("B", "Hkv", "D", "T", "t0"))
    got = []
    for n in ("k", "v"):
        cache = x[n + "_cache"].double()
        state = torch.empty(B, Hkv, D, device=DEV, dtype=torch.float64)
        for b in range(B):
            cache[b, :, t0:t0 + T], state[b] = _scan64(x[n][b], x["g"][b], x["state_" + n][b])
        got.append((state, cache))
    (sk, kc), (sv, vc) = got
    return [sk, sv, kc, vc, _page_bounds(kc, t0 + T, case["P"])]


def _append64(case, x):
    """States after the token, and the caches [B, Hkv, T + 1, D] with it stored, in 64 bits."""
    g, T, states, caches = x["g"][:, :, 0].double(), case["T"], [], []
    for n in ("k", "v"):
        s = g * x["state_" + n].double() + (1 - g) * x[n][:, :, 0].double()
        states.append(s)
        x[n + "_cache"][:, :, T] = s.to(x[n + "_cache"].dtype)
        caches.append(x[n + "_cache"][:, :, :T + 1])
    return states, caches


def _attend64(q, k, v, scale, keep=None):
    """q [n, D], k and v [T, D], keep [n, T] or None."""
    p = (q.double() @ k.double().T) * scale
    if keep is not None:
        p.masked_fill_(~keep, -math.inf)
    lse = torch.logsumexp(p, 1)
    return torch.exp(p - lse[:, None]) @ v.double(), lse


def _exact_decode(case, x):
    B, Hq, Hkv, D, T = (case[n] for n in ("B", "Hq", "Hkv", "D", "T"))
    (sk, sv), (kc, vc) = _append64(case, x)
    scale, G = 1.0 / math.sqrt(D), Hq // Hkv
    out = torch.empty(B, Hq, D, device=DEV, dtype=torch.float64)
    lse = torch.empty(B, Hq, device=DEV, dtype=torch.float64)
    idx = torch.empty(B, Hq, case.get("K", 0), device=DEV, dtype=torch.int64)
    meta = _page_bounds(x["k_cache"], T + 1, case["P"]) if case["kind"] == "decode" else None
    page = torch.arange(T + 1, device=DEV) // case.get("P", 1)
    for b in range(B):
        for h in range(Hkv):
            q, keep = x["q"][b, h * G:(h + 1) * G], None
            if meta is not None:
                n = -(-(T + 1) // case["P"])
                m, q64 = meta[b, h, :n].double(), q.double()
                score = q64.clamp(min=0) @ m[:, 1].T + q64.clamp(max=0) @ m[:, 0].T
                score[:, 0] = score[:, n - 1] = math.inf
                best = torch.sort(score, dim=1, descending=True, stable=True).indices[:, :case["K"]].sort(1).values
                idx[b, h * G:(h + 1) * G] = best
                picked = torch.zeros(G, n, device=DEV, dtype=torch.bool).scatter_(1, best, True)
                keep = picked[:, page]
            out[b, h * G:(h + 1) * G], lse[b, h * G:(h + 1) * G] = _attend64(q, kc[b, h], vc[b, h], scale, keep)
    if meta is None:
        return [out, lse, sk, sv, None, None]
    return [out, lse, idx, sk, sv, None, None, None]


def _exact_prefill(case, x):
    B, Hq, Hkv, D, T = (case[n] for n in ("B", "Hq", "Hkv", "D", "T"))
    G, scale, block, K = Hq // Hkv, 1.0 / math.sqrt(D), case.get("block", 0), case.get("K", 0)
    out = torch.empty(B, Hq, T, D, device=DEV, dtype=torch.float64)
    lse = torch.empty(B, Hq, T, device=DEV, dtype=torch.float64)
    t = torch.arange(T, device=DEV)
    if block:
        nb = -(-T // block)
        means = torch.stack([x["k_cache"][:, :, j * block:(j + 1) * block].double().mean(2) for j in range(nb)], 2)
        idx = torch.empty(B, Hq, T, K, device=DEV, dtype=torch.int64)
    for b in range(B):
        for h in range(Hq):
            k, v = x["k_cache"][b, h // G], x["v_cache"][b, h // G]
            for lo in range(0, T, 1024):
                rows, hi = t[lo:lo + 1024], min(T, lo + 1024)
                q = x["q"][b, h, lo:hi]
                keep = t[None, :hi] <= rows[:, None]
                if block:
                    own = rows // block
                    score = q.double() @ means[b, h // G].T
                    later = torch.arange(nb, device=DEV)[None] > own[:, None]
                    score.masked_fill_(later, -math.inf).scatter_(1, own[:, None], math.inf)
                    best = torch.sort(score, dim=1, descending=True, stable=True).indices[:, :K]
                    if best.shape[1] < K:
                        best = torch.nn.functional.pad(best, (0, K - best.shape[1]), value=nb)
                    best = torch.where(best > own[:, None], nb, best).sort(1).values
                    idx[b, h, lo:hi] = torch.where(best == nb, -1, best)
                    picked = torch.zeros(hi - lo, nb + 1, device=DEV, dtype=torch.bool).scatter_(1, best, True)
                    keep &= picked[:, t[:hi] // block]
                out[b, h, lo:hi], lse[b, h, lo:hi] = _attend64(q, k[:hi], v[:hi], scale, keep)
    return [out, lse, idx, means] if block else [out, lse]


def _exact_snapkv(case, x):
    B, Hq, Hkv, D, T, W = (case[n] for n in ("B", "Hq", "Hkv", "D", "T", "W"))
    G, scale, keep, pool = Hq // Hkv, 1.0 / math.sqrt(D), case["keep"], case["pool"]
    votes = torch.empty(B, Hkv, T - W, device=DEV, dtype=torch.float64)
    later = torch.arange(T, device=DEV)[None] > T - W + torch.arange(W, device=DEV)[:, None]
    for b in range(B):
        for h in range(Hkv):
            k = x["k_cache"][b, h].double()
            p = sum(torch.softmax((x["q"][b, h * G + i].double() @ k.T * scale).masked_fill_(later, -math.inf), 1).sum(0)
                    for i in range(G))
            votes[b, h] = torch.nn.functional.max_pool1d(p[None, None, :T - W], pool, 1, pool // 2)[0, 0]
    idx = torch.sort(votes, dim=2, descending=True, stable=True).indices[:, :, :keep].sort(2).values
    rows = torch.cat([idx, torch.arange(T - W, T, device=DEV).expand(B, Hkv, W)], 2)[..., None].expand(-1, -1, -1, D)
    return [x["k_cache"].gather(2, rows).double(), x["v_cache"].gather(2, rows).double(), idx, votes]


def exact(case, seed):
    x = _inputs(case, seed)
    return {"scan": _exact_scan, "decode": _exact_decode, "dense": _exact_decode, "moba": _exact_prefill,
            "prefill": _exact_prefill, "snapkv": _exact_snapkv}[case["kind"]](case, x)
