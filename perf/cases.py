"""Performance cases of the strict-prefix linear-attention library.

Each case is one call (or one save-and-restore pair) that a serving engine
makes through the public entry points: prefill (cold, resumed, paged),
decode, page copies and the joint restore.  `listed()` holds the fixed
cases, `draw(rng)` one more of the same ranges, `prepare` what an engine has
in hand before the call, `run` the call, `work` what the call cannot do
without, `tolerance` how far two correct implementations may differ, and
`exact` the same outputs in 64 bits from plain torch.

Prefill and decode inputs follow the distribution the library's workloads
use: q and k normalised per (token, head), v ~ N(0, 1), beta = sigmoid(N),
g = -softplus(N) * gate.  gate = 1 forgets within a chunk; small gates carry
the state across many chunks, as trained gates do.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2609_15030_amd import api
from paper_2609_15030_amd import linattn as la

DEV = "cuda"
KV_TOKEN_BYTES = 8268      # attention-cache bytes per token of one rank
KV_BLOCK_TOKENS = 16

# The 16-sequence batch: prompt lengths and the strict-prefix boundaries that
# its cached prefixes allow (0: nothing cached), C = 256.
VARLEN_N = [7760, 8016, 5376, 8064, 3136, 4000, 2656, 5136, 6080, 6320, 4096, 1216, 3696, 7152, 1968, 2784]
VARLEN_B = [0, 7936, 1536, 0, 0, 0, 1024, 0, 0, 6144, 0, 256, 3328, 6912, 1792, 1280]


def _text(values) -> str:
    return ",".join(str(int(v)) for v in values)


def _ints(text: str):
    return [int(v) for v in text.split(",")] if text else []


def _prefill(name, lens, heads, dk, dv, interval, dtype="bf16", starts="", variant=0, scale=1.0, gate=1.0,
             store="dense"):
    """lens: tokens each sequence computes in this call; starts: the absolute
    position each begins at (empty: a cold call); store: checkpoints and
    starting states in dense arrays or in pool pages."""
    return {"name": name, "kind": "prefill", "lens": _text(lens), "starts": _text(starts) if starts else "",
            "heads": heads, "dk": dk, "dv": dv, "interval": interval, "dtype": dtype, "variant": variant,
            "scale": scale, "gate": gate, "store": store}


def _decode(name, seqs, heads, dk, dv, dtype="bf16", variant=0, scale=1.0, gate=1.0):
    return {"name": name, "kind": "decode", "seqs": seqs, "heads": heads, "dk": dk, "dv": dv, "dtype": dtype,
            "variant": variant, "scale": scale, "gate": gate}


def _short_lens(seed, n, lo, hi):
    r = random.Random(seed)
    return [r.randint(lo, hi) for _ in range(n)]


def listed():
    return [
        # One generated token of one request: the smallest call there is.
        _decode("decode_1seq_h8_d128", 1, 8, 128, 128),
        # One generated token of a full serving batch.
        _decode("decode_64seq_h8_d128", 64, 8, 128, 128, gate=0.01),
        # A reloaded prompt's strict-prefix suffix: the 256 tokens past its
        # last usable checkpoint, from and into pool pages.
        _prefill("resume_256_h8_d128_paged", [256], 8, 128, 128, 256, starts=[3328], store="paged"),
        # One tensor-parallel rank's share of one 3,584-token prompt, cold.
        _prefill("cold_3584_h8_d128_paged", [3584], 8, 128, 128, 256, store="paged", gate=0.01),
        # A mixed batch: cold prompts, full and partial prefix hits in one call.
        _prefill("varlen16_h8_d128_paged", [n - b for n, b in zip(VARLEN_N, VARLEN_B)], 8, 128, 128, 256,
                 starts=VARLEN_B, store="paged"),
        # The longest prompt the model takes, checkpoints every 1,024 tokens.
        _prefill("cold_32768_h16_d128_C1024", [32768], 16, 128, 128, 1024, gate=0.01),
        # Many short prompts of ragged lengths at once.
        _prefill("short64_h8_d128", _short_lens(7, 64, 1, 300), 8, 128, 128, 128),
        # Ragged batch at smaller heads, an interval that is no multiple of the
        # chunk, the decayed-delta rule and an output scale.
        _prefill("ragged33_h8_dk64_dv128_C100", _short_lens(8, 33, 64, 700), 8, 64, 128, 100, variant=1, scale=0.125,
                 gate=0.1),
        # fp32, the accuracy path: the small prompt the library is brought up with.
        _prefill("fp32_cold_256_h1_d64_C16", [256], 1, 64, 64, 16, dtype="f32"),
        # fp32 at the full head size: three prompts of one rank, ragged.
        _prefill("fp32_ragged3_h8_d128_C256", [1791, 640, 257], 8, 128, 128, 256, dtype="f32", gate=0.01),
        # The whole page pool saved and restored through a permuted page table.
        {"name": "pool_save_restore_4096", "kind": "pool", "items": 4096, "pages": 4096, "page_elems": 16384},
        # The joint reload of one prompt: the KV blocks of [0, 3328) and 8 state pages.
        {"name": "hybrid_restore_3328_h8", "kind": "hybrid", "bounds": "3328", "heads": 8, "page_elems": 16384},
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["prefill", "prefill", "prefill", "prefill", "decode", "decode", "pool", "hybrid"])
    if kind == "decode":
        c = _decode("", _log_int(rng, 1, 256), rng.choice([1, 3, 8, 16]), rng.choice([64, 128, 128]),
                    rng.choice([64, 128, 128]), rng.choice(["bf16", "bf16", "f32"]), rng.randint(0, 1),
                    rng.choice([1.0, 0.125]), rng.choice([1.0, 0.01]))
    elif kind == "pool":
        items = _log_int(rng, 1, 4096)
        c = {"kind": "pool", "items": items, "pages": rng.randint(items, 4096), "page_elems": rng.choice([4096, 8192, 16384])}
    elif kind == "hybrid":
        n = rng.randint(1, 4)
        c = {"kind": "hybrid", "bounds": _text(256 * rng.randint(0, 16) for _ in range(n)),
             "heads": rng.choice([1, 8, 16]), "page_elems": rng.choice([4096, 8192, 16384])}
    else:
        dtype = rng.choice(["bf16", "bf16", "bf16", "bf16", "f32"])
        interval = rng.choice([16, 48, 64, 100, 128, 192, 256, 256, 256, 512, 1024])
        # a call costs by its tokens and by its longest sequence: both are kept
        # below the listed cases' (fp32 and small intervals cost more per token)
        small = dtype == "f32" or interval < 128
        total = _log_int(rng, 48, 4096 if small else 49152)
        longest = 2048 if small else (16384 if interval >= 512 else 8192)
        n = rng.randint(-(-total // longest), max(-(-total // longest), min(40, total // 32)))
        w = [rng.random() + 0.02 for _ in range(n)]
        lens = [min(longest, max(1, int(total * x / sum(w)))) for x in w]
        starts = [interval * rng.randint(0, 12) for _ in lens] if rng.random() < 0.4 else ""
        c = _prefill("", lens, rng.choice([1, 3, 8, 8]), rng.choice([64, 128, 128]), rng.choice([64, 128, 128]),
                     interval, dtype, starts, rng.randint(0, 1), rng.choice([1.0, 0.125]), rng.choice([1.0, 0.1, 0.01]),
                     rng.choice(["dense", "paged"]))
    c.pop("name", None)
    return c


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed) * 2654435761 % (2 ** 31) + 17)
    return g


def _dtype(case):
    return torch.bfloat16 if case["dtype"] == "bf16" else torch.float32


def _io(case):
    return la.LA_BF16 if case["dtype"] == "bf16" else la.LA_F32


def _rows(case):
    return sum(_ints(case["lens"])) if case["kind"] == "prefill" else case["seqs"]


def _tokens(case, gen):
    """q, k, v, g, beta for one call: [rows, heads, ...]."""
    T, H, dk, dv, td = _rows(case), case["heads"], case["dk"], case["dv"], _dtype(case)
    rnd = lambda *s: torch.randn(s, generator=gen, device=DEV, dtype=torch.float32)
    unit = lambda x: (x / x.norm(dim=-1, keepdim=True)).to(td)
    q, k = unit(rnd(T, H, dk)), unit(rnd(T, H, dk))
    v = rnd(T, H, dv).to(td)
    beta = torch.sigmoid(rnd(T, H))
    g = -torch.nn.functional.softplus(rnd(T, H)) * case["gate"]
    return q, k, v, g, beta


def _starts_of(case):
    return _ints(case["starts"]) or None


def _ckpt_rows(case):
    """Per sequence: (first row, rows) of the checkpoints at multiples of C in (B, B + len]."""
    C, lens = case["interval"], _ints(case["lens"])
    at, out = 0, []
    for n in lens:                      # starts are multiples of C
        out.append((at, n // C))
        at += n // C
    return out, at


def _prefill_inputs(case, seed):
    """Tokens, starting states of a resumed call (None: cold) and, for a paged
    call, the pool with those states in their pages and both page tables."""
    gen = _gen(seed)
    toks = _tokens(case, gen)
    lens, H, E = _ints(case["lens"]), case["heads"], case["dk"] * case["dv"]
    starts = _starts_of(case)
    state = None
    if starts:
        state = 0.1 * torch.randn((len(lens), H, case["dk"], case["dv"]), generator=gen, device=DEV)
        cold = torch.tensor([b == 0 for b in starts], device=DEV)
        state[cold] = 0.0
    if case["store"] != "paged":
        return toks, state, None, None, None
    _, rows = _ckpt_rows(case)
    n_state = len(lens) * H if starts else 0
    pages = rows * H + n_state + 8
    perm = torch.from_numpy(np.random.default_rng(seed).permutation(pages).astype(np.int32)).to(DEV)
    ck_ids = perm[:rows * H].contiguous() if rows else None
    pool = torch.zeros((pages, E), device=DEV)
    st_ids = None
    if starts:
        st_ids = perm[rows * H:rows * H + n_state].clone()
        st_ids[torch.tensor([b == 0 for b in starts], device=DEV).repeat_interleave(H)] = -1
        live = st_ids >= 0
        pool[st_ids[live].long()] = state.reshape(-1, E)[live]
    return toks, state, pool, ck_ids, st_ids


def _decode_inputs(case, seed):
    gen = _gen(seed)
    toks = _tokens(case, gen)
    state = 0.1 * torch.randn((case["seqs"], case["heads"], case["dk"], case["dv"]), generator=gen, device=DEV)
    return toks, state


def prepare(case, seed):
    kind = case["kind"]
    if kind == "prefill":
        (q, k, v, g, beta), state, pool, ck_ids, st_ids = _prefill_inputs(case, seed)
        cu = np.concatenate([[0], np.cumsum(_ints(case["lens"]))]).astype(np.int32)
        x = api.DeviceInputs(q, k, v, g, beta, torch.from_numpy(cu).to(DEV), cu, _io(case))
        plan = api.Prefill(x, case["interval"], case["variant"], case["scale"], _starts_of(case),
                           emit_ckpt=pool is None)
        return {"kind": kind, "plan": plan, "state": state, "pool": pool, "ck_ids": ck_ids, "st_ids": st_ids}
    if kind == "decode":
        (q, k, v, g, beta), state = _decode_inputs(case, seed)
        shape = la.make_shape(case["seqs"], case["heads"], case["dk"], case["dv"], 64, _io(case), case["variant"],
                              case["scale"])
        return {"kind": kind, "shape": shape, "q": q, "k": k, "v": v, "g": g, "beta": beta, "state": state,
                "o": torch.empty_like(v)}
    gen = _gen(seed)
    rng = np.random.default_rng(seed)
    ids = lambda a: torch.from_numpy(np.ascontiguousarray(a, dtype=np.int32)).to(DEV)
    if kind == "pool":
        n, pages, E = case["items"], case["pages"], case["page_elems"]
        return {"kind": kind, "states": torch.randn((n, E), generator=gen, device=DEV),
                "pool": torch.zeros((pages, E), device=DEV), "ids": ids(rng.permutation(pages)[:n]),
                "back": torch.zeros((n, E), device=DEV)}
    bounds = np.array(_ints(case["bounds"]), np.int64)
    H, E, block = case["heads"], case["page_elems"], KV_TOKEN_BYTES * KV_BLOCK_TOKENS
    nb = bounds // KV_BLOCK_TOKENS
    total, most = int(nb.sum()), max(1, int(nb.max()))
    src = np.full((len(bounds), most), -1, np.int32)
    dst = np.full((len(bounds), most), -1, np.int32)
    ps, pd = rng.permutation(total + 16), rng.permutation(total + 16)
    at = 0
    for i, b in enumerate(nb):
        src[i, :b], dst[i, :b] = ps[at:at + b], pd[at:at + b]
        at += int(b)
    kv_pool = torch.randint(0, 256, (total + 16, block), generator=gen, device=DEV, dtype=torch.uint8)
    cache = torch.zeros((total + 16, block), dtype=torch.uint8, device=DEV)
    return {"kind": kind, "kv": la.make_kv_blocks(kv_pool, cache, ids(src), ids(dst), KV_BLOCK_TOKENS),
            "cache": cache, "bounds": bounds, "bounds_dev": torch.from_numpy(bounds).to(DEV), "heads": H,
            "state_pool": torch.randn((len(bounds) * H + 16, E), generator=gen, device=DEV),
            "state_ids": ids(rng.permutation(len(bounds) * H + 16)[:len(bounds) * H]),
            "states": torch.zeros((len(bounds) * H, E), device=DEV)}


def run(state):
    s = state
    if s["kind"] == "prefill":
        p = s["plan"]
        if s["pool"] is not None:
            r = p.run_paged(s["pool"], s["ck_ids"], s["st_ids"])
            return [r.o, r.final_state, s["pool"]]
        r = p.run(s["state"])
        return [r.o, r.final_state] + ([r.ckpt] if r.ckpt is not None else [])
    if s["kind"] == "decode":
        la.la_decode_step(s["shape"], s["q"], s["k"], s["v"], s["g"], s["beta"], s["state"], s["o"])
        return [s["o"], s["state"]]
    if s["kind"] == "pool":
        la.la_state_save_paged(s["states"], s["pool"], s["ids"])
        la.la_state_restore_paged(s["pool"], s["ids"], s["back"])
        return [s["pool"], s["back"]]
    la.la_hybrid_restore(s["kv"], s["bounds_dev"], s["bounds"], s["state_pool"], s["state_ids"], s["states"],
                         s["heads"])
    return [s["cache"], s["states"]]


def work(case):
    kind = case["kind"]
    if kind == "pool":
        return {"bytes": 4.0 * case["items"] * case["page_elems"] * 4, "flops": 0}
    if kind == "hybrid":
        b = _ints(case["bounds"])
        return {"bytes": 2.0 * (sum(b) * KV_TOKEN_BYTES + len(b) * case["heads"] * case["page_elems"] * 4), "flops": 0}
    T, H, dk, dv = _rows(case), case["heads"], case["dk"], case["dv"]
    io, E = (2 if case["dtype"] == "bf16" else 4), 4 * dk * dv
    tok = T * H * (io * (2 * dk + 2 * dv) + 8)      # q, k, v, o and the gates
    if kind == "decode":
        return {"bytes": tok + 2.0 * T * H * E, "flops": 6.0 * T * H * dk * dv}
    n = len(_ints(case["lens"]))
    resumed = sum(b > 0 for b in _starts_of(case) or [])
    _, rows = _ckpt_rows(case)
    return {"bytes": tok + float(E) * H * (n + resumed + rows), "flops": 6.0 * T * H * dk * dv}


def tolerance(case):
    # About four times the error measured against exact(): bf16 outputs 4e-3
    # (prefill) and 1.7e-3 (decode, rounding of o), fp32 4e-7.
    if case["kind"] in ("pool", "hybrid"):
        return "exact"
    if case["kind"] == "decode":
        return {"rel": 7e-3} if case["dtype"] == "bf16" else {"rel": 2e-6}
    return {"rel": 1.5e-2} if case["dtype"] == "bf16" else {"rel": 4e-6}


# ---------------------------------------------------------------------------
# 64-bit reference
# ---------------------------------------------------------------------------

def _exact_tokens(q, k, v, g, beta, S, variant, scale):
    """Token by token over [chains, tokens, ...] in fp64: outputs and the state."""
    outs = []
    for t in range(q.shape[1]):
        a = torch.exp(g[:, t])[:, None]
        pred = torch.matmul(k[:, t, None, :], S)[:, 0]
        u = beta[:, t, None] * (v[:, t] - (a * pred if variant else pred))
        S = a[:, :, None] * S + k[:, t, :, None] * u[:, None, :]
        outs.append(scale * torch.matmul(q[:, t, None, :], S)[:, 0])
    return torch.stack(outs, 1), S


def _exact_chunk(q, k, v, g, beta, S, variant, scale):
    """The same over a chunk of up to 64 tokens in matrix form (fp64)."""
    n = q.shape[1]
    G = torch.cumsum(g, 1)
    Gp = G if variant else torch.cat([torch.zeros_like(G[:, :1]), G[:, :-1]], 1)
    kk = torch.matmul(k, k.transpose(1, 2).contiguous())
    low = torch.tril(torch.ones(n, n, dtype=torch.bool, device=q.device), -1)
    dec = torch.exp(torch.where(low, Gp[:, :, None] - G[:, None, :], torch.full((), -1e300, dtype=q.dtype, device=q.device)))
    A = beta[:, :, None] * dec * kk
    rhs = beta[:, :, None] * (v - torch.exp(Gp)[:, :, None] * torch.matmul(k, S))
    eye = torch.eye(n, dtype=q.dtype, device=q.device)
    u = torch.linalg.solve_triangular(eye + A, rhs, upper=False, unitriangular=True)
    low0 = torch.tril(torch.ones(n, n, dtype=torch.bool, device=q.device))
    P = torch.matmul(q, k.transpose(1, 2).contiguous()) * torch.exp(
        torch.where(low0, G[:, :, None] - G[:, None, :], torch.full((), -1e300, dtype=q.dtype, device=q.device)))
    o = scale * (torch.exp(G)[:, :, None] * torch.matmul(q, S) + torch.matmul(P, u))
    w = torch.exp(G[:, -1:] - G)[:, :, None] * k
    S = torch.exp(G[:, -1])[:, None, None] * S + torch.matmul(w.transpose(1, 2).contiguous(), u)
    return o, S


def exact(case, seed):
    if case["kind"] in ("pool", "hybrid"):
        return None
    f8 = lambda x: x.double()
    if case["kind"] == "decode":
        toks, S = _decode_inputs(case, seed)
        n = case["seqs"] * case["heads"]
        q, k, v, g, beta = (f8(x).reshape(n, 1, *x.shape[2:]) for x in toks)
        o, S2 = _exact_tokens(q, k, v, g, beta, f8(S).reshape(n, case["dk"], case["dv"]), case["variant"], case["scale"])
        return [o.reshape(case["seqs"], case["heads"], -1), S2.reshape(S.shape)]
    toks, state, pool, ck_ids, st_ids = _prefill_inputs(case, seed)
    lens, H, dk, dv, C = _ints(case["lens"]), case["heads"], case["dk"], case["dv"], case["interval"]
    n, L = len(lens), max(lens)
    # [sequence, head] chains padded to the longest; padding has zero key,
    # beta and gate, which leaves a state as it is
    def pad(x):
        p = torch.zeros((n, L, *x.shape[1:]), dtype=torch.float64, device=DEV)
        at = 0
        for i, m in enumerate(lens):
            p[i, :m] = x[at:at + m].double()
            at += m
        return p.transpose(1, 2).reshape(n * H, L, *x.shape[2:])
    q, k, v, g, beta = (pad(x) for x in toks)
    S = torch.zeros((n * H, dk, dv), dtype=torch.float64, device=DEV) if state is None else f8(state).reshape(n * H, dk, dv)
    offs, rows = _ckpt_rows(case)
    ck = torch.zeros((rows, H, dk, dv), dtype=torch.float64, device=DEV)
    out = torch.empty((n * H, L, dv), dtype=torch.float64, device=DEV)
    a = 0
    while a < L:                         # chunks end on the checkpoint positions
        b = min(a + 64, (a // C + 1) * C, L)
        out[:, a:b], S = _exact_chunk(q[:, a:b], k[:, a:b], v[:, a:b], g[:, a:b], beta[:, a:b], S, case["variant"],
                                      case["scale"])
        if b % C == 0:
            for i, (r0, nr) in enumerate(offs):
                if b // C <= nr:
                    ck[r0 + b // C - 1] = S.reshape(n, H, dk, dv)[i]
        a = b
    out = out.reshape(n, H, L, dv)
    o = torch.cat([out[i, :, :m].transpose(0, 1) for i, m in enumerate(lens)])
    final = S.reshape(n, H, dk, dv)
    if pool is not None:
        whole = f8(pool)
        if rows:
            whole[ck_ids.long()] = ck.reshape(rows * H, dk * dv)
        return [o, final, whole]
    return [o, final] + ([ck] if rows else [])
