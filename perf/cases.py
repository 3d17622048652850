"""Timed cases of the streamFFN routed-expert path on one MI355X.

Every case is one MoE layer as a serving process runs it through the C ABI
(``cep.py``): a layer of routed-token chunks under a launch policy
(``cep_begin_layer``, ``cep_submit_chunk``, ``cep_combine``, with the weight
fetch where the case has one), or one chunk through ``cep_ffn_noalloc``.  The
chunks are resident when the pass starts and per-phase timing is off, as in
production; a pass enqueues the layer and returns the layer's output buffer.

Keys of a case: call ("layer" or "noalloc"), w / x (weight and row format),
d, I, E of Eg experts local, k slots per token, R replicas of T token slots in
cpr chunks each, zipf (0: balanced routing), hot (popularity rank of the most
popular local expert, from zero), policy, theta, streams, fetched
(local experts whose weights a layer fetches from a donor region).
"""
from __future__ import annotations

import functools

import numpy as np
import torch

from paper_2609_33252_amd import cep

W_CODE = {"f32": cep.CEP_F32, "bf16": cep.CEP_BF16, "e4m3": cep.CEP_FP8_E4M3_B128,
          "mxfp4": cep.CEP_MXFP4}
POLICY = {"wait_all": cep.CEP_WAIT_ALL, "per_chunk": cep.CEP_PER_CHUNK,
          "theta": cep.CEP_THRESHOLD}
WEIGHT_BYTES = {"f32": 4.0, "bf16": 2.0, "e4m3": 1.0 + 4.0 / 128 ** 2, "mxfp4": 0.5 + 1.0 / 32}


def _case(name, w, x, d, I, E, Eg, k, R, T, cpr=1, zipf=0.0, hot=0, policy="wait_all",
          theta=1, streams=1, fetched=0, call="layer"):
    c = dict(call=call, w=w, x=x, d=d, I=I, E=E, Eg=Eg, k=k, R=R, T=T, cpr=cpr, zipf=zipf, hot=hot,
             policy=policy, theta=theta, streams=streams, fetched=fetched)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest layer of the repository's workloads, float32 end to end:
        # launches and their latency are all of it
        _case("tiny_f32", "f32", "f32", 256, 128, 8, 8, 2, 2, 256, cpr=2),
        # a handful of tokens in a loop that may not allocate: each touched
        # expert's weights are streamed for a few rows
        _case("noalloc_bf16", "bf16", "bf16", 4096, 2048, 8, 64, 8, 1, 24, call="noalloc"),
        _case("noalloc_mxfp4", "mxfp4", "bf16", 4096, 2048, 16, 128, 6, 1, 61, call="noalloc"),
        # one short prompt's tokens on e4m3 experts: ragged counts of some
        # twenty rows per expert
        _case("short_e4m3", "e4m3", "bf16", 6144, 2560, 16, 160, 8, 1, 397),
        # balanced synchronous layer, one batch of about 1000 rows per expert
        _case("sync_bf16_d4096", "bf16", "bf16", 4096, 2048, 8, 64, 8, 4, 2048),
        # asynchronous EP without threshold: every chunk of the skewed layer is
        # a batch of a few rows per expert beside one hot expert
        _case("per_chunk_bf16_d7168", "bf16", "bf16", 7168, 2048, 8, 256, 8, 8, 4096, cpr=8,
              zipf=1.2, hot=7, policy="per_chunk", streams=2),
        # the same layer under the launch threshold
        _case("theta_bf16_d7168", "bf16", "bf16", 7168, 2048, 8, 256, 8, 8, 4096, cpr=8,
              zipf=1.2, hot=7, policy="theta", theta=4096, streams=2),
        # float32 rows and weights at sizes that are no power of two
        _case("ragged_f32_d2304", "f32", "f32", 2304, 1408, 12, 60, 5, 3, 1777, cpr=2),
        # threshold batches on e4m3 experts: some 130 rows per expert each
        _case("theta_e4m3_d7168", "e4m3", "bf16", 7168, 2048, 16, 128, 8, 4, 2048, cpr=4,
              policy="theta", theta=2048, streams=2),
        # the largest layer, all replicas at once: e4m3 experts, four of them
        # fetched from a donor region
        _case("sync_e4m3_fetch_d6144", "e4m3", "bf16", 6144, 2560, 16, 160, 8, 8, 8192,
              zipf=1.5, hot=3, fetched=4),
        # MXFP4 experts: the synchronous layer and its per-chunk streaming
        _case("sync_mxfp4_d4096", "mxfp4", "bf16", 4096, 2048, 32, 256, 6, 8, 8192, cpr=8),
        _case("per_chunk_mxfp4_d4096", "mxfp4", "bf16", 4096, 2048, 32, 256, 6, 8, 8192, cpr=8,
              policy="per_chunk", streams=2),
    ]


def _log_int(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    """One more case of the same ranges: weight format, shape, token count,
    routing skew and launch policy drawn independently."""
    w = rng.choice(["f32", "bf16", "e4m3", "mxfp4", "bf16", "e4m3", "mxfp4"])
    x = "f32" if w == "f32" else "bf16"
    if w == "bf16" and rng.random() < 0.15:
        x = "f32"
    small_f32 = w == "f32"
    d = 256 * _log_int(rng, 1 if small_f32 else 4, 12 if small_f32 else 28)
    I = 128 * _log_int(rng, 1 if small_f32 else 6, 12 if small_f32 else 20)
    E = rng.choice([4, 5, 8, 12, 16, 24, 32])
    Eg = E * rng.choice([4, 8, 10])
    k = rng.choice([2, 4, 5, 6, 8])
    if rng.random() < 0.25:  # one small chunk of a serving loop
        return _case("", w, x, min(d, 4096), min(I, 2048), min(E, 16), 8 * min(E, 16), k, 1,
                     _log_int(rng, 3, 80), call="noalloc")
    R = rng.choice([1, 2, 3, 4, 8])
    T = _log_int(rng, 64, 4096)
    cpr = rng.choice([1, 1, 2, 3, 8])
    policy = rng.choice(["wait_all", "wait_all", "per_chunk", "theta"])
    # at most a third of the largest listed layer's work
    T = max(64, min(T, int(1.1e12 / (6.0 * d * I * R * k * E / Eg))))
    pairs = R * T * k * E // Eg
    theta = max(1, int(pairs * rng.uniform(0.1, 0.6)))
    streams = 1 if policy == "wait_all" else rng.choice([1, 2, 4])
    fetched = E // 4 if rng.random() < 0.2 else 0
    return _case("", w, x, d, I, E, Eg, k, R, T, cpr=cpr, zipf=rng.choice([0.0, 0.0, 1.2]),
                 hot=rng.randrange(Eg // E), policy=policy,
                 theta=theta, streams=streams, fetched=fetched)


# ------------------------------------------------------------------ inputs

def _log_popularity(c):
    """log popularity per global expert.  A popular expert's place is a property
    of the deployment, not of one seed's tokens: the local experts are spread
    over the popularity ranks (hot, hot + Eg/E, ...), so that one of them is
    hot and the others are not."""
    if not c["zipf"]:
        return np.zeros(c["Eg"])
    p = np.arange(1, c["Eg"] + 1, dtype=np.float64) ** -c["zipf"]
    local = np.arange(c["E"]) * (c["Eg"] // c["E"]) + c["hot"]
    remote = np.setdiff1d(np.arange(c["Eg"]), local)
    return np.log(p / p.sum())[np.concatenate([local, remote])]


@functools.lru_cache(maxsize=None)
def _inclusion(Eg, E, k, zipf, hot):
    """Probability that a token selects each local expert, and that it selects
    any (by simulation for skewed routing)."""
    if not zipf:
        return np.full(E, k / Eg), 1.0 - (1.0 - k / Eg) ** E
    logp = _log_popularity(dict(Eg=Eg, E=E, zipf=zipf, hot=hot))
    g = np.random.default_rng(1).gumbel(size=(8192, Eg)) + logp
    top = np.argpartition(-g, k - 1, axis=1)[:, :k]
    hit = np.zeros((8192, Eg), bool)
    np.put_along_axis(hit, top, True, axis=1)
    return hit[:, :E].mean(axis=0), hit[:, :E].any(axis=1).mean()


def _bounds(c):
    """Token ranges of a replica's chunks (contiguous, as even as T allows)."""
    return [(j * c["T"] // c["cpr"], (j + 1) * c["T"] // c["cpr"]) for j in range(c["cpr"])]


class _State:
    """Weights, context and resident chunks of one case."""

    ctx = None

    def __del__(self):
        if self.ctx:
            cep.cep_destroy(self.ctx)
            self.ctx = None


def _normal(gen, *shape, scale=1.0):
    return torch.randn(*shape, generator=gen, device="cuda") * scale


def _weights(c, gen):
    """Expert weights in the caller's layout: (gate, up, down, scales)."""
    d, I, E = c["d"], c["I"], c["E"]
    mats, scales = [], []
    for rows, cols in ((d, I), (d, I), (I, d)):
        if c["w"] == "mxfp4":  # output-major [cols][rows], two codes a byte
            mats.append(torch.randint(0, 256, (E, cols, rows // 2), generator=gen, device="cuda",
                                      dtype=torch.uint8))
            scales.append(torch.randint(119, 121, (E, cols, rows // 32), generator=gen,
                                        device="cuda", dtype=torch.uint8))
        elif c["w"] == "e4m3":
            q = torch.empty(E, rows, cols, dtype=torch.uint8, device="cuda")
            s = torch.empty(E, rows // 128, cols // 128, device="cuda")
            for e in range(E):
                t = _normal(gen, rows // 128, 128, cols // 128, 128, scale=0.02)
                s[e] = t.abs().amax(dim=(1, 3)) / 448.0
                q[e] = (t / s[e][:, None, :, None]).to(torch.float8_e4m3fn).view(
                    torch.uint8).view(rows, cols)
            mats.append(q)
            scales.append(s)
        else:
            dt = torch.bfloat16 if c["w"] == "bf16" else torch.float32
            m = torch.empty(E, rows, cols, dtype=dt, device="cuda")
            for e in range(E):
                m[e] = _normal(gen, rows, cols, scale=0.02)
            mats.append(m)
            scales.append(None)
    return mats, scales


def _tokens(c, gen):
    """Rows [R][T][d], local expert ids [R][T][k] (-1: remote), coefficients."""
    R, T, k, Eg = c["R"], c["T"], c["k"], c["Eg"]
    x = torch.empty(R, T, c["d"], device="cuda",
                    dtype=torch.bfloat16 if c["x"] == "bf16" else torch.float32)
    for r in range(R):
        x[r] = _normal(gen, T, c["d"])
    u = torch.rand(R, T, Eg, generator=gen, device="cuda").clamp_(1e-12, 1 - 1e-7)
    score = torch.from_numpy(_log_popularity(c)).float().cuda() - torch.log(-torch.log(u))
    ids = torch.topk(score, k, dim=-1).indices.int()
    ids = torch.where(ids < c["E"], ids, torch.full_like(ids, -1))
    wt = torch.softmax(_normal(gen, R, T, k), dim=-1)
    return x, ids, wt


def _generate(c, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 17)
    mats, scales = _weights(c, gen)
    return mats, scales, *_tokens(c, gen)


def prepare(case, seed):
    c = case
    mats, scales, x, ids, wt = _generate(c, seed)
    s = _State()
    s.case = c
    s.out = torch.zeros(c["R"], c["T"], c["d"], device="cuda")
    delivered = (ids >= 0).any(dim=-1)
    # token rows lie in one receive region, chunk after chunk
    s.chunks, rows = [], []
    for j, (t0, t1) in enumerate(_bounds(c)):
        for r in range(c["R"]):
            tok = torch.nonzero(delivered[r, t0:t1]).flatten() + t0
            rows.append(x[r, tok])
            s.chunks.append([r, tok.numel(), int((ids[r, tok] >= 0).sum()), tok.int(), None,
                             ids[r, tok].contiguous(), wt[r, tok].contiguous()])
    s.recv = torch.cat(rows)
    at = 0
    for ch in s.chunks:
        ch[4] = s.recv[at:at + ch[1]]
        at += ch[1]
    del x, ids, wt, rows
    cfg = cep.make_config(
        d_model=c["d"], d_ff=c["I"], n_local_experts=c["E"], top_k=c["k"], max_replicas=c["R"],
        max_tokens_per_replica=c["T"], w_dtype=W_CODE[c["w"]], x_dtype=W_CODE[c["x"]],
        n_streams=c["streams"], max_pairs_per_batch=max(1, sum(ch[2] for ch in s.chunks)))
    weights = cep.make_weights(*mats, *scales)
    blob = cep.cep_packed_expert_bytes(cfg)
    cfg.fetch_buffer_bytes = blob * c["fetched"]
    stream = torch.cuda.current_stream()
    s.fetch_ids = [i * c["E"] // c["fetched"] for i in range(c["fetched"])]
    resident = [0 if e in s.fetch_ids else 1 for e in range(c["E"])]
    if c["fetched"]:
        # the packed blobs a donor GPU would hold
        s.donor = torch.empty(len(s.fetch_ids), blob, dtype=torch.uint8, device="cuda")
        for i, e in enumerate(s.fetch_ids):
            cep.cep_pack_experts(cfg, weights, e, 1, s.donor[i], stream)
        s.donor_ptrs = [s.donor[i].data_ptr() for i in range(len(s.fetch_ids))]
    s.ctx = cep.cep_init_experts(cfg, weights, resident, stream)
    torch.cuda.synchronize()
    cep.cep_set_phase_timing(s.ctx, 0)
    cep.cep_set_policy(s.ctx, POLICY[c["policy"]], c["theta"], c["streams"])
    s.side = torch.cuda.Stream() if c["fetched"] else None
    s.chunks_per_replica = [c["cpr"]] * c["R"]
    s.generation = 0
    return s


def run(state):
    s, stream = state, torch.cuda.current_stream()
    if s.case["call"] == "noalloc":
        r, n, p, tok, x, ids, wt = s.chunks[0]
        cep.cep_ffn_noalloc(s.ctx, r, n, p, tok, x, ids, wt, s.out, stream)
        return s.out
    s.generation += 1
    cep.cep_begin_layer(s.ctx, s.generation, s.chunks_per_replica, s.out)
    if s.fetch_ids:
        cep.cep_weight_fetch(s.ctx, s.fetch_ids, s.donor_ptrs, s.side)
    for r, n, p, tok, x, ids, wt in s.chunks:
        cep.cep_submit_chunk(s.ctx, s.generation, r, n, p, tok, x, ids, wt)
    cep.cep_combine(s.ctx, stream)
    return s.out


# ------------------------------------------------------- work and tolerance

def work(case):
    """One pass: every invocation reads its touched experts' weights, rows and
    routing once (a launch policy asks for separate invocations, and an
    expert's weights do not stay on chip between them) and writes its tokens'
    output rows; a fetch reads and writes its experts' weights once more."""
    c = case
    share, any_local = _inclusion(c["Eg"], c["E"], c["k"], c["zipf"], c["hot"])
    tokens = c["R"] * c["T"]
    pairs = tokens * share.sum()
    batches = 1
    if c["policy"] == "per_chunk":
        batches = c["R"] * c["cpr"]
    elif c["policy"] == "theta":
        batches = max(1, min(c["R"] * c["cpr"], int(np.ceil(pairs / c["theta"]))))
    touched = (1.0 - (1.0 - share) ** (tokens / batches)).sum()
    expert = 3.0 * c["d"] * c["I"] * WEIGHT_BYTES[c["w"]]
    rows = tokens * any_local
    row = c["d"] * (2 if c["x"] == "bf16" else 4) + 8 * c["k"] + 4
    return {"bytes": float(batches * touched * expert + rows * (row + 4 * c["d"])
                           + 2 * c["fetched"] * expert),
            "flops": float(6.0 * c["d"] * c["I"] * pairs)}


def tolerance(case):
    # four times the distance from `exact` measured over the listed and some
    # drawn cases: float32 rows or weights run as bf16 (up to 4.1e-3), bf16
    # sums in float32 over a bf16 h whose last bit may differ (up to 6.6e-5),
    # e4m3 and MXFP4 round each output to bf16 and requantise h (up to 2.1e-3)
    if case["w"] == "f32" or case["x"] == "f32":
        return {"rel": 1.6e-2}
    return {"rel": 2.7e-4} if case["w"] == "bf16" else {"rel": 8e-3}


# ------------------------------------------------------------------- exact

def _mxfp8(v):
    """MXFP8 values of float32 rows: blocks of 32, scale 2^(floor(log2 amax)
    - 8), e4m3 elements, saturating."""
    b = v.view(*v.shape[:-1], -1, 32)
    amax = b.abs().amax(dim=-1, keepdim=True)
    e = (torch.frexp(amax).exponent - 1 - 8).clamp(min=-127)
    e = torch.where(amax > 0, e, torch.full_like(e, -127))
    q = torch.ldexp(b, -e).clamp(-448.0, 448.0).to(torch.float8_e4m3fn).double()
    return torch.ldexp(q, e).view(v.shape)


def _dense(c, m, s):
    """One expert matrix [K][N] in float64 from its stored form."""
    if c["w"] == "mxfp4":
        lut = torch.tensor([0, .5, 1, 1.5, 2, 3, 4, 6], dtype=torch.float64, device=m.device)
        lut = torch.cat([lut, -lut])
        v = torch.stack([lut[(m & 15).long()], lut[(m >> 4).long()]], dim=-1).view(m.shape[0], -1)
        f = torch.ldexp(torch.ones_like(s, dtype=torch.float64), s.int() - 127)
        return (v.view(m.shape[0], -1, 32) * f[..., None]).view(m.shape[0], -1).t()
    if c["w"] == "e4m3":
        f = s.double().repeat_interleave(128, 0).repeat_interleave(128, 1)
        return m.view(torch.float8_e4m3fn).double() * f
    return m.double()


def exact(case, seed):
    """The layer in float64 on the path's input formats: x and h as MXFP8 with
    e4m3 / MXFP4 weights, h in bf16 with bf16 weights, nothing rounded with
    float32 weights and rows."""
    c = case
    mats, scales, x, ids, wt = _generate(c, seed)
    quant = c["w"] in ("e4m3", "mxfp4")
    ids, wt = ids.view(-1, c["k"]), wt.view(-1, c["k"])
    x = x.view(-1, c["d"])
    out = torch.zeros(x.shape[0], c["d"], dtype=torch.float64, device="cuda")
    for e in range(c["E"]):
        tok, slot = torch.nonzero(ids == e, as_tuple=True)
        wg, wu, wd = (_dense(c, m[e], s[e] if s is not None else None)
                      for m, s in zip(mats, scales))
        for lo in range(0, tok.numel(), 8192):
            t, sl = tok[lo:lo + 8192], slot[lo:lo + 8192]
            xe = _mxfp8(x[t].float()) if quant else x[t].double()
            g = xe @ wg
            h = g / (1.0 + torch.exp(-g)) * (xe @ wu)
            if quant:
                h = _mxfp8(h.float())
            elif c["w"] == "bf16":
                h = h.bfloat16().double()
            out.index_add_(0, t, (h @ wd) * wt[t, sl].double()[:, None])
    return out.view(c["R"], c["T"], c["d"])
