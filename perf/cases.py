"""The measured work of this library: sessions of the FastGen path through its public entry points.

A case is one call sequence as a serving program issues it. `call` = "session": a context over
the program's workspace, attention profiling and policy choice of the prompt, compaction, and
`steps` generated tokens over the compressed caches (a session of one step is the time to the
first token). `call` = "static": profiling alone, by the entry point that needs no context.

  seqs, heads   B sequences x (layers * heads) K/V heads each; group: query heads per K/V head
  dim, dtype    head dimension and element type of Q, K, V and of the cache
  n, new, steps prompt tokens, tokens reserved for, tokens generated in the pass
  T, ratio      recovery threshold; ratio of the local window and of the frequent budget
  forced        -1: policy per head by recovery; 0..4: every head uses that policy
  lse           the program's prefill attention hands over the rows' log-sum-exp
  probe         every so many steps run with the stability probe (0: none)
  classify      token classes are derived from ids on the way (else known beforehand)
  export        the pass ends with a read-back of the whole cache state (a checkpoint)
  mix           weights of the planted attention patterns, "local special punct heavy broad"

Inputs are seeded noise with planted attention structure: a favoured special token, punctuation
columns, heavy-hitter columns, a local band, or nothing.
"""
import math

import torch

from paper_2310_01801_amd import binding

DEVICE = "cuda:0"
UNIFORM, LOCAL_OR_BROAD, HEAVY_TAILED = "20 20 20 20 20", "30 30 0 0 40", "15 25 25 15 20"
LOCAL, SPECIAL, PUNCT, HEAVY, BROAD = range(5)
SPECIAL_IDS, PUNCT_IDS = [0], list(range(1, 17))
VOCAB, PUNCT_SHARE = 32000, 0.1
CHECKPOINT = ("lengths", "offsets", "positions", "scores", "keys", "values", "status")   # in the C call's order
HELD = 0.5   # share of the tokens that adaptive caches hold (0.49 and 0.47 in the benchmark's workloads)

BASE = dict(call="session", seqs=1, heads=32, dim=128, dtype="bf16", n=2048, new=1, steps=1, T=0.95, ratio=0.3,
            forced=-1, group=1, lse=False, probe=0, classify=False, export=False, mix=UNIFORM)


def _case(**kw):
    return dict(BASE, **kw)


def listed():
    return [
        # the smallest configuration in use: float32, four heads; bound by launches and latency
        _case(name="tiny-f32", heads=4, dim=64, dtype="f32", n=128, new=32, steps=32, ratio=0.1, classify=True),
        # one layer of a short prompt, profiled without a context (graph capture, tight loops)
        _case(name="static-layer", call="static", heads=32, n=333, classify=True),
        # time to the first token of a 7B-shaped model: 32 layers x 32 heads
        _case(name="first-token-2k", heads=1024, new=256),
        # the same shape generating: the decode step is what repeats
        _case(name="generate-2k", heads=1024, new=128, steps=128),
        # a batch of ordinary prompts, lower threshold (shorter caches)
        _case(name="batch-1k", seqs=4, heads=1024, n=1024, new=256, T=0.9),
        # 13B-shaped, 40 layers x 40 heads: prompt and some tokens
        _case(name="session-4k", heads=1600, n=4096, new=16, steps=16, mix=LOCAL_OR_BROAD),
        # five layers of 64 heads, long prompts: the profiling sweeps at their largest
        _case(name="first-token-8k", seqs=2, heads=320, n=8192, new=128, mix=HEAVY_TAILED),
        # the same generating over long caches of very different lengths
        _case(name="generate-8k", seqs=2, heads=320, n=8192, new=128, steps=128, mix=HEAVY_TAILED),
        # grouped-query attention: 32 layers x 8 K/V heads, four query heads each, log-sum-exp handed over
        _case(name="grouped-2k", heads=256, group=4, new=64, steps=64, lse=True),
        # float32 model, prompt of a round but unaligned length
        _case(name="f32-1k", heads=64, dtype="f32", n=1000, new=16, steps=16),
        # head dimension 64, odd prompt length, three sequences, classes from ids, probed now and then
        _case(name="dim64-odd", seqs=3, heads=144, dim=64, n=1337, new=40, steps=40, probe=8, classify=True),
        # fixed special+punct.+frequent+local caches, checkpointed after a few tokens
        _case(name="checkpoint-3k", heads=256, n=3000, new=8, steps=8, forced=3, export=True),
    ]


def _log(rng, low, high):
    return int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))


def draw(rng):
    f32 = rng.random() < 0.15
    group = rng.choice([1, 1, 1, 2, 4, 8])
    n = _log(rng, 64, 1500 if f32 else 8192)
    steps = _log(rng, 1, 128)
    seqs = rng.choice([1, 1, 2, 3])
    # sessions stay below the largest listed ones: score elements of the prompt, tokens in memory,
    # tokens read while decoding
    most = min(6.0e7 / (group * n * n) if f32 else 4.0e10 / (group * n * n), 4.0e6 / (group * n),
               6.0e8 / (steps * group * n))
    heads = max(1, _log(rng, 4, max(4.0, min(4096.0, most))) // seqs)
    static = rng.random() < 0.1
    if static:
        group, seqs = 1, 1
        heads = max(1, min(heads, 1000000 // n))
    return _case(call="static" if static else "session", seqs=seqs, heads=heads, dim=rng.choice([64, 128, 128]),
                 dtype="f32" if f32 else "bf16", n=n, new=steps + rng.choice([0, 0, 64]), steps=1 if static else steps,
                 T=rng.choice([0.9, 0.95, 0.98]), ratio=rng.choice([0.1, 0.2, 0.3]), group=group,
                 forced=rng.choice([-1, -1, -1, -1, 2, 3, 4]), lse=rng.random() < 0.2 and n <= 2048,
                 probe=rng.choice([0, 0, 0, 8]), classify=rng.random() < 0.3, export=rng.random() < 0.15,
                 mix=rng.choice([UNIFORM, LOCAL_OR_BROAD, HEAVY_TAILED]))


# ---------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------

def _plant(case, plan, Q, K, pos, unit_cls, heavy):
    """Overwrites reserved dimensions of Q [U, G, m, d] and K [U, m, d] (tokens at positions
    `pos`) so that the scaled logits gain each unit's planted bias."""
    d, n = case["dim"], case["n"]
    pattern, strength, window, length = plan
    loc = torch.nonzero(pattern == LOCAL).flatten()
    if loc.numel():
        # a tapered cosine series in the distance: a band of about 0.6 windows
        m_sigma = length / (math.pi * (0.6 * window / 2.5))
        M = int(min(math.ceil(2.5 * m_sigma), d // 4))
        m = torch.arange(1, M + 1, dtype=torch.float64, device=DEVICE)
        g = torch.exp(-(m * m) / (2.0 * m_sigma * m_sigma))
        ang = pos.double()[:, None] * (math.pi * m / length)[None, :]
        wave = torch.stack([torch.cos(ang), torch.sin(ang)], dim=-1) * torch.sqrt(g / g.sum() * math.sqrt(d))[None, :, None]
        wave = wave.reshape(pos.numel(), 2 * M)
        for u in loc.tolist():
            row = (wave * math.sqrt(float(strength[u]))).to(Q.dtype)
            Q[u, :, :, :2 * M] = row
            K[u, :, :2 * M] = row
    for which, beta in ((SPECIAL, math.log(n)), (PUNCT, math.log((1.0 - PUNCT_SHARE) / PUNCT_SHARE)), (HEAVY, math.log(15.0))):
        ids = torch.nonzero(pattern == which).flatten()
        if not ids.numel():
            continue
        alpha = torch.sqrt((beta + strength[ids.cpu()].to(DEVICE)) * math.sqrt(d)).float()
        fav = heavy[ids] if which == HEAVY else (unit_cls[ids] & (1 if which == SPECIAL else 3)) != 0
        Q[ids, :, :, 0] = alpha[:, None, None].expand(-1, Q.shape[1], Q.shape[2]).to(Q.dtype)
        K[ids, :, 0] = torch.where(fav, alpha[:, None], 0.0).to(K.dtype)


def _inputs(case, seed):
    U, B, n, d, G, S = case["seqs"] * case["heads"], case["seqs"], case["n"], case["dim"], case["group"], case["steps"]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    host, gen = torch.Generator().manual_seed(seed), torch.Generator(device=DEVICE).manual_seed(seed)

    def ids(*shape):
        x = torch.randint(17, VOCAB, shape, generator=host)
        punct = torch.randint(1, 17, shape, generator=host)
        return torch.where(torch.rand(shape, generator=host) < PUNCT_SHARE, punct, x).to(torch.int32)

    prompt_ids, step_ids = ids(B, n), ids(S, B)
    prompt_ids[:, 0] = 0
    weights = torch.tensor([float(x) for x in case["mix"].split()])
    pattern = torch.multinomial(weights, U, replacement=True, generator=host)
    strength = torch.rand(U, generator=host, dtype=torch.float64)
    strength = torch.where(pattern == LOCAL, 6.0 + 4.0 * strength, 1.5 + 3.0 * strength)
    plan = (pattern.to(DEVICE), strength, max(1, math.floor(case["ratio"] * n)), n + case["new"])
    prompt_ids, step_ids = prompt_ids.to(DEVICE), step_ids.to(DEVICE)
    cls, step_cls = _classes(prompt_ids), _classes(step_ids)

    def noise(*shape):
        return torch.randn(shape, generator=gen, device=DEVICE, dtype=dtype)

    Q, K, V = noise(U, G, n, d), noise(U, n, d), noise(U, n, d)
    heavy = torch.rand((U, n), generator=gen, device=DEVICE) < 1.0 / 16.0
    _plant(case, plan, Q, K, torch.arange(n, device=DEVICE), cls.repeat_interleave(case["heads"], 0), heavy)
    q, k, v = noise(U, G, S, d), noise(U, S, d), noise(U, S, d)
    _plant(case, plan, q, k, torch.arange(n, n + S, device=DEVICE), step_cls.t().repeat_interleave(case["heads"], 0),
           torch.zeros((U, S), dtype=torch.bool, device=DEVICE))
    x = dict(Q=Q.view(U * G, n, d), K=K, V=V, ids=prompt_ids, cls=cls, step_ids=step_ids, step_cls=step_cls,
             q=q.permute(2, 0, 1, 3).reshape(S, U * G, d).contiguous(), k=k.transpose(0, 1).contiguous(),
             v=v.transpose(0, 1).contiguous(), lse=None)
    if case["lse"]:
        x["lse"] = torch.empty((U * G, n), device=DEVICE)
        hidden = torch.ones((n, n), dtype=torch.bool, device=DEVICE).triu(1)
        for u in range(U):
            s = torch.matmul(x["Q"][u * G:(u + 1) * G].reshape(G * n, d).float(), K[u].float().t().contiguous())
            s = (s * _scale(case)).view(G, n, n).masked_fill_(hidden, -math.inf)
            x["lse"][u * G:(u + 1) * G] = torch.logsumexp(s, dim=2)
    return x


def _classes(ids):
    return (ids == 0).to(torch.uint8) + 2 * ((ids >= 1) & (ids <= 16)).to(torch.uint8)


def _scale(case):
    return float(torch.tensor(1.0 / math.sqrt(case["dim"]), dtype=torch.float32))


def prepare(case, seed):
    x = _inputs(case, seed)
    U, G = case["seqs"] * case["heads"], case["group"]
    cfg = binding.make_config(U, case["seqs"], case["dim"], x["K"].dtype, case["n"], case["new"], case["T"],
                              case["ratio"], case["ratio"], forced_policy=case["forced"], group_size=G)
    state = dict(case=case, cfg=cfg, x=x)
    if case["call"] == "static":
        state["policy"] = torch.empty(U, dtype=torch.int32, device=DEVICE)
        state["recovery"] = torch.empty((U, 5), dtype=torch.float64, device=DEVICE)
        state["kept"] = torch.empty((U, 5), dtype=torch.int32, device=DEVICE)
        return state
    state["workspace"] = torch.empty(binding.fastgen_workspace_bytes(cfg), dtype=torch.uint8, device=DEVICE)
    state["out"] = torch.empty((case["steps"], U * G, case["dim"]), dtype=x["K"].dtype, device=DEVICE)
    if case["export"]:   # the program's checkpoint buffers, sized for the uncompressed cache
        room = U * (case["n"] + case["new"])
        sizes = dict(lengths=((U,), torch.int32), offsets=((U + 1,), torch.int64), positions=((room,), torch.int32),
                     scores=((room,), torch.float64), keys=((room, case["dim"]), x["K"].dtype),
                     values=((room, case["dim"]), x["K"].dtype), status=((1,), torch.int32))
        state["checkpoint"] = {name: torch.zeros(size, dtype=t, device=DEVICE) for name, (size, t) in sizes.items()}
    state["steps"] = list(zip(x["q"], x["k"], x["v"], x["step_ids"], x["step_cls"], state["out"]))
    return state


# ---------------------------------------------------------------------------------------
# one pass
# ---------------------------------------------------------------------------------------

def run(state):
    case, x = state["case"], state["x"]
    cls = binding.fastgen_classify(x["ids"], SPECIAL_IDS, PUNCT_IDS) if case["classify"] else x["cls"]
    if case["call"] == "static":
        binding.fastgen_profile_static(state["cfg"], x["Q"], x["K"], cls, state["policy"], state["recovery"],
                                       state["kept"], lse=x["lse"])
        return dict(policy=state["policy"], recovery=state["recovery"], kept=state["kept"])
    fg = binding.FastGen(state["cfg"], DEVICE, workspace=state["workspace"])
    policy, recovery, kept = fg.fastgen_profile(x["Q"], x["K"], cls, lse=x["lse"])
    fg.fastgen_compact(x["K"], x["V"])
    probes = []
    for t, (q, k, v, ids, step_cls, out) in enumerate(state["steps"]):
        if case["classify"]:
            step_cls = binding.fastgen_classify(ids, SPECIAL_IDS, PUNCT_IDS)
        if case["probe"] and t % case["probe"] == 0:
            probes.append(fg.fastgen_decode_step_probe(q, k, v, step_cls, out)[1])
        else:
            fg.fastgen_decode_step(q, k, v, step_cls, out)
    answer = dict(policy=policy, recovery=recovery, kept=kept, out=state["out"])
    if probes:
        answer["probes"] = probes
    if case["export"]:
        buffers = state["checkpoint"]
        fg._check(fg.lib.fastgen_export_state(fg._ctx, *[buffers[name].data_ptr() for name in CHECKPOINT],
                                              torch.cuda.current_stream().cuda_stream))
        answer["state"] = buffers
    fg.close()
    return answer


def work(case):
    U, G, n, d = case["seqs"] * case["heads"], case["group"], case["n"], case["dim"]
    e = 4 if case["dtype"] == "f32" else 2
    held = 1.0 if case["forced"] == 4 else HELD
    byts, flops = U * (G + 1) * n * d * e, U * G * d * n * (n + 1.0)
    if case["call"] == "session":
        tokens = case["steps"] * U * held * (n + case["steps"] / 2.0)      # held tokens over all steps
        byts += U * 3 * held * n * d * e + tokens * 2 * d * e + case["steps"] * U * (2 * G + 4) * d * e
        flops += tokens * G * 4 * d
        if case["export"]:
            byts += 4 * U * held * n * d * e
    return {"bytes": float(byts), "flops": float(flops)}


def tolerance(case):
    # the outputs are rounded to the cache's type: 1.0e-3 to 1.7e-3 off exact() in bf16, 1.6e-7 to
    # 2.8e-7 in float32; a head or token at the edge of its policy's threshold or budget may go
    # either way
    if case["dtype"] == "bf16":
        return {"rel": 5e-3, "max": 0.1, "differ": 2e-3}
    return {"rel": 1e-6, "max": 1e-3, "differ": 2e-3}


# ---------------------------------------------------------------------------------------
# the same in 64 bits, plain torch
# ---------------------------------------------------------------------------------------

def _column_sums(case, x):
    """Cumulative attention score of every prompt token and its part inside the local band."""
    U, G, n = case["seqs"] * case["heads"], case["group"], case["n"]
    w = max(1, math.floor(case["ratio"] * n))
    col = torch.zeros((U, n), dtype=torch.float64, device=DEVICE)
    band = torch.zeros_like(col)
    units = max(1, min(U, (1 << 26) // (n * min(n, 512))))
    j = torch.arange(n, device=DEVICE)
    for u0 in range(0, U, units):
        u1 = min(U, u0 + units)
        KT = x["K"][u0:u1].double().transpose(1, 2).contiguous()
        for h in range(G):
            Qh = x["Q"].view(U, G, n, -1)[u0:u1, h]
            for r0 in range(0, n, 512):
                r1 = min(n, r0 + 512)
                i = torch.arange(r0, r1, device=DEVICE)
                s = torch.matmul(Qh[:, r0:r1].double(), KT[:, :, :r1].contiguous()) * _scale(case)
                s = s.masked_fill_(j[None, :r1] > i[:, None], -math.inf)
                p = torch.softmax(s, dim=2)
                col[u0:u1, :r1] += p.sum(1)
                band[u0:u1, :r1] += p.masked_fill_(j[None, :r1] <= i[:, None] - w, 0.0).sum(1)
    return col, band


def _top(score, k):
    """Mask of the k largest entries of every row, equal ones by position."""
    mask = torch.zeros(score.shape, dtype=torch.bool, device=DEVICE)
    if k > 0:
        order = torch.sort(score, dim=1, descending=True, stable=True)[1][:, :k]
        mask.scatter_(1, order, True)
    return mask


def exact(case, seed):
    U, G, n, S = case["seqs"] * case["heads"], case["group"], case["n"], case["steps"]
    if U * G * n * n > 1.5e11:
        return None
    x = _inputs(case, seed)
    w = max(1, math.floor(case["ratio"] * n))
    col, band = _column_sums(case, x)
    cls = x["cls"].repeat_interleave(case["heads"], 0)
    special, punct = (cls & 1) != 0, (cls & 2) != 0
    top, tail = _top(col, math.floor(case["ratio"] * n)), torch.arange(n, device=DEVICE) >= n - w
    static = [special, special | punct, special | punct | top, special | punct | top]
    kept = [static[0], static[1], static[2], static[3] | tail, torch.ones_like(special)]
    recovery = torch.stack([torch.where(m, col, band if c == 3 else 0.0).sum(1) / (n * G) for c, m in enumerate(static)]
                           + [torch.ones(U, dtype=torch.float64, device=DEVICE)], dim=1)
    answer = dict(policy=None, recovery=recovery, kept=None)
    if case["call"] == "static":
        return answer
    policy = torch.full((U,), 4, device=DEVICE)
    for c in (3, 2, 1, 0):
        cheaper = kept[c].sum(1) <= torch.stack([m.sum(1) for m in kept], 1).gather(1, policy[:, None])[:, 0]
        policy = torch.where((recovery[:, c] >= case["T"]) & cheaper, c, policy)
    if case["forced"] >= 0:
        policy.fill_(case["forced"])
    held = torch.zeros((U, n + S), dtype=torch.bool, device=DEVICE)
    held[:, :n] = torch.stack(kept, 1).gather(1, policy[:, None, None].expand(U, 1, n))[:, 0]
    x.pop("Q")
    score = torch.cat([col, torch.zeros((U, S), dtype=torch.float64, device=DEVICE)], 1)
    cls = torch.cat([cls, x["step_cls"].t().repeat_interleave(case["heads"], 0)], 1)
    special, punct = (cls & 1) != 0, (cls & 2) != 0
    pos = torch.arange(n + S, device=DEVICE)
    p4 = policy[:, None]
    outs = torch.empty((S, U, G, case["dim"]), dtype=torch.float64, device=DEVICE)
    probes = []
    Kd = torch.cat([x["K"].double(), x["k"].transpose(0, 1).double()], 1)
    Vd = torch.cat([x["V"].double(), x["v"].transpose(0, 1).double()], 1)
    for t in range(S):
        p = n + t
        held[:, p] = True
        probing = case["probe"] > 0 and t % case["probe"] == 0
        s = torch.matmul(Kd, x["q"][t].view(U, G, -1).double().transpose(1, 2).contiguous()) * _scale(case)
        a = torch.softmax(s.masked_fill_(~held[:, :, None], -math.inf), dim=1).transpose(1, 2).contiguous()
        outs[t] = torch.matmul(a, Vd)
        score += torch.where((p4 == 2) | (p4 == 3) | probing, a.sum(1), 0.0)
        top = held & _top(torch.where(held, score, -1.0), math.floor(case["ratio"] * (p + 1)))
        recent = pos > p - w
        if probing:
            member = [special, special | punct, special | punct | top, special | punct | top | recent, held]
            probes.append(torch.stack([(a.sum(1) / G * m).sum(1) for m in member], 1))
        held &= (p4 >= 4) | special | (punct & (p4 >= 1)) | (top & (p4 >= 2)) | (recent & (p4 == 3))
    answer["out"] = outs.view(S, U * G, case["dim"])
    if probes:
        answer["probes"] = probes
    if case["export"]:
        def packed(rows):
            full = torch.zeros((U * (n + case["new"]),) + tuple(rows.shape[1:]), dtype=torch.float64, device=DEVICE)
            full[:rows.shape[0]] = rows
            return full
        answer["state"] = dict(lengths=None, offsets=None, positions=None, scores=packed(score[held]),
                               keys=packed(Kd[held]), values=packed(Vd[held]), status=None)
    return answer
