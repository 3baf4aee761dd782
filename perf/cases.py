"""The work that users of this framework have it do, as cases that can be timed.

Each case is one call pattern of a training or serving program, through the package's
public entry points: the policy query (Agent.act), a block of SAC updates
(Agent.sac_update), and the single stages that a program composes by itself (the squint
gather, the encoder, the twin critics and the actor forward and backward, the categorical
projection, the optimiser step).  Sizes come from the configurations, the tests and the
benchmark of this repository: batch 512 and 2048 on 64x64x9 frames, 128x128 frames squinted
to 16x16 and to 32x32, policy queries of 1 to 4096 observations, both precisions.

A case is a dict of plain values: what ("kind"), the network ("net"), the precision and the
rows ("n").  listed() gives the fixed cases, draw(rng) further ones of the same ranges,
prepare() what a program holds before the call, run() one pass, work() the bytes and
operations a pass cannot do without, exact() its results in 64 bits from plain torch.
"""
import math

import numpy as np
import torch
import torch.nn.functional as F

from paper_2602_21203_amd import _lib, api, configs

NETS = {"full": configs.FULL, "full128": configs.FULL128, "full32": configs.FULL32}
PRECS = {"bf16": _lib.SQ_BF16, "fp32": _lib.SQ_F32}
DEV = "cuda"
SEED_KEY = 2      # the agents' Philox key
REQUEST = 7       # the policy query's request id


def listed():
    return [
        # one robot asks for its next action: latency and launches
        dict(name="act_1", kind="act", net="full", prec="bf16", n=1, sample=False),
        # a pool of simulated environments acts at once (the agent's largest query)
        dict(name="act_4096", kind="act", net="full", prec="bf16", n=4096, sample=True),
        # the training loop of the benchmark: four updates per call, batch 512, raw frames
        dict(name="update_512", kind="update", net="full", prec="bf16", n=512, utd=4, store="raw"),
        # the benchmark's large-batch form
        dict(name="update_2048", kind="update", net="full", prec="bf16", n=2048, utd=4, store="raw"),
        # the encoder alone, forward and backward, at the training batch
        dict(name="encoder_512", kind="encoder", net="full", prec="bf16", n=512),
        # the higher-resolution input (32x32) in full precision, a ragged batch
        dict(name="encoder32_250_fp32", kind="encoder", net="full32", prec="fp32", n=250),
        # the twin critics alone, forward and every gradient, at the training batch
        dict(name="critic_512", kind="critic", net="full", prec="bf16", n=512),
        # the same in full precision on a large ragged batch
        dict(name="critic_2000_fp32", kind="critic", net="full", prec="fp32", n=2000),
        # the policy alone, sampled action and log-probability, forward and backward
        dict(name="actor_1000_fp32", kind="actor", net="full", prec="fp32", n=1000),
        # replay rows gathered and squinted from 128x128 frames
        dict(name="squint_2048", kind="squint", net="full128", prec="fp32", n=2048),
        # the distributional Bellman target of a large ragged batch
        dict(name="project_3000", kind="project", net="full", prec="fp32", n=3000),
        # the optimiser step over every parameter, with the target critic's average
        dict(name="adam_1493335", kind="adam", net="full", prec="fp32", n=1493335),
    ]


def _size(rng, lo, hi):
    """Log-uniform in [lo, hi]; any whole number, so mostly off the kernels' tiles."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["act", "act", "update", "update", "encoder", "encoder", "critic", "critic", "actor", "actor",
                       "squint", "project", "adam"])
    prec = rng.choice(["bf16", "fp32"])
    if kind == "act":
        return dict(kind=kind, net="full", prec=prec, n=_size(rng, 1, 4096), sample=rng.random() < 0.5)
    if kind == "update":
        return dict(kind=kind, net="full", prec=prec, n=_size(rng, 64, 2048), utd=rng.choice([1, 2]),
                    store=rng.choice(["raw", "ring"]))
    if kind == "encoder":
        net = rng.choice(["full", "full32"])
        return dict(kind=kind, net=net, prec=prec, n=_size(rng, 16, 1024 if net == "full" else 250))
    if kind == "squint":
        return dict(kind=kind, net=rng.choice(["full", "full128", "full32"]), prec=prec, n=_size(rng, 64, 2048))
    if kind == "project":
        return dict(kind=kind, net="full", prec="fp32", n=_size(rng, 64, 4096))
    if kind == "adam":
        return dict(kind=kind, net="full", prec="fp32", n=_size(rng, 20000, 1493335))
    return dict(kind=kind, net="full", prec=prec, n=_size(rng, 16, 2000))


# ---------------------------------------------------------------- geometry
def _sides(c):
    """Side of the squinted image, then of each convolution's output."""
    s = [c["H"] // c["k"]]
    for i in range(c["n_conv"]):
        s.append((s[-1] - 3) // 2 + 1 if i == 0 else s[-1] - 2)
    return s


def _table(c):
    """{name: (offset, shape)} of the flat parameter vector, and its blocks' ends."""
    flat, P, H, A = c["F"] * _sides(c)[-1] ** 2, c["proj"], c["hidden"], c["action"]
    shapes, ends = [], {}

    def dense(name, out, inp):
        shapes.extend([(name + ".W", (out, inp)), (name + ".b", (out,)), (name + ".g", (out,)), (name + ".h", (out,))])

    def mlp(name, inp, out):
        dense(name + ".l1", H, inp)
        dense(name + ".l2", H, H)
        shapes.extend([(name + ".out.W", (out, H)), (name + ".out.b", (out,))])

    def end(block):
        ends[block] = sum(math.prod(s) for _, s in shapes)

    for i in range(c["n_conv"]):
        shapes.extend([(f"conv{i}.W", (c["F"], c["C"] if i == 0 else c["F"], 3, 3)), (f"conv{i}.b", (c["F"],))])
    end("enc")
    dense("critic", P, flat)
    mlp("q1", P + c["proprio"] + A, c["atoms"])
    mlp("q2", P + c["proprio"] + A, c["atoms"])
    end("critic")
    dense("actor", P, flat)
    mlp("pi", P + c["proprio"], 2 * A)
    end("actor")
    shapes.append(("log_alpha", (1,)))
    end("total")
    table, o = {}, 0
    for name, s in shapes:
        table[name] = (o, s)
        o += math.prod(s)
    return table, ends


def _view(flat, table, base=0):
    return {k: flat[o - base:o - base + math.prod(s)].view(s) for k, (o, s) in table.items()
            if base <= o and o - base + math.prod(s) <= flat.numel()}


# ---------------------------------------------------------------- inputs
def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _params(c, g):
    """Weights and biases U(+-1/sqrt(fan in)), LayerNorm gains and shifts as after some
    training (near 1 and 0), log alpha as it starts."""
    table, ends = _table(c)
    p = torch.rand(ends["total"], generator=g, device=DEV) * 2 - 1
    z = torch.randn(ends["total"], generator=g, device=DEV)
    for name, (o, s) in table.items():
        n = math.prod(s)
        if name.endswith(".g"):
            p[o:o + n] = 1 + 0.05 * z[o:o + n]
        elif name.endswith(".h"):
            p[o:o + n] = 0.05 * z[o:o + n]
        elif name == "log_alpha":
            p[o] = 0.0
        else:
            fan = math.prod(table[name[:-1] + "W"][1][1:])
            p[o:o + n] *= fan ** -0.5
    return p


def _frames(n, c, g):
    """uint8 HWC camera frames: smooth structure plus sensor noise, every frame its own."""
    out = torch.empty((n, c["H"], c["W"], c["C"]), dtype=torch.uint8, device=DEV)
    for i in range(0, n, 512):
        m = min(512, n - i)
        f = F.interpolate(torch.rand((m, c["C"], 8, 8), generator=g, device=DEV), size=(c["H"], c["W"]),
                          mode="bilinear", align_corners=False)
        f = f * 224 + 32 * torch.rand((m, c["C"], c["H"], c["W"]), generator=g, device=DEV)
        out[i:i + m] = f.clamp(0, 255).to(torch.uint8).permute(0, 2, 3, 1)
    return out


def _transitions(n, c, g):
    r = lambda *s: torch.randn(s, generator=g, device=DEV)
    return dict(obs=_frames(n, c, g), next_obs=_frames(n, c, g), proprio=r(n, c["proprio"]),
                next_proprio=r(n, c["proprio"]),
                action=torch.rand((n, c["action"]), generator=g, device=DEV) * 2 - 1,
                reward=torch.rand(n, generator=g, device=DEV),
                done=(torch.rand(n, generator=g, device=DEV) < 0.01).to(torch.uint8))


def _rows(case):
    """Replay rows: many times the batch, and more frame bytes than the caches hold."""
    return 8192 if case["kind"] == "update" else 2 * case["n"] + 1024


def _inputs(case, seed):
    """Everything a pass reads, from the seed alone (shared by prepare and exact)."""
    c, g, n, kind = NETS[case["net"]], _gen(seed), case["n"], case["kind"]
    table, ends = _table(c)
    flat, A, N = c["F"] * _sides(c)[-1] ** 2, c["action"], c["atoms"]
    r = lambda *s: torch.randn(s, generator=g, device=DEV)
    u = lambda *s: torch.rand(s, generator=g, device=DEV)
    if kind == "act":
        return dict(params=_params(c, g), frames=_frames(n, c, g), proprio=r(n, c["proprio"]))
    if kind == "update":
        return dict(params=_params(c, g), replay=_transitions(_rows(case), c, g))
    if kind == "encoder":
        s = _sides(c)[0]
        p = _params(c, g)[:ends["enc"]].clone()
        x = F.interpolate(u(n, c["C"], 5, 5), size=(s, s), mode="bilinear", align_corners=False)
        return dict(params=p, x=(x * 0.875 + 0.125 * u(n, c["C"], s, s) - 0.5).contiguous(), dfeat=r(n, flat) / n)
    if kind == "critic":
        p = _params(c, g)[ends["enc"]:ends["critic"]].clone()
        feat = torch.relu(0.3 * r(n, flat))
        d = torch.softmax(r(2, n, N), -1) - torch.softmax(2 * r(2, n, N), -1)
        return dict(params=p, feat=feat, proprio=r(n, c["proprio"]), action=u(n, A) * 2 - 1, dlogits=d / n)
    if kind == "actor":
        p = _params(c, g)[ends["critic"]:ends["actor"]].clone()
        return dict(params=p, feat=torch.relu(0.3 * r(n, flat)), proprio=r(n, c["proprio"]), eps=r(n, A),
                    daction=r(n, A) / n, dlogp=(0.5 + u(n)) / n)
    if kind == "squint":
        rows = _rows(case)
        return dict(frames=_frames(rows, c, g),
                    idx=torch.randint(0, rows, (n,), generator=g, device=DEV, dtype=torch.int32))
    if kind == "project":
        return dict(p=torch.softmax(2 * r(n, N), -1), reward=u(n), done=(u(n) < 0.01).to(torch.uint8),
                    bonus=2 + r(n))
    lo = min(n, ends["enc"])
    return dict(p=0.05 * r(n), g=0.01 * r(n), m=0.01 * r(n), v=1e-4 * u(n), ema=0.05 * r(n - lo), lo=lo,
                step=torch.full((1,), 20, dtype=torch.int32, device=DEV))


def prepare(case, seed):
    c, prec, kind = NETS[case["net"]], PRECS[case["prec"]], case["kind"]
    s = dict(case=dict(case), cfg=c, prec=prec, **_inputs(case, seed))
    if kind in ("act", "update"):
        s["agent"] = api.Agent(c, s["params"], case["n"] if kind == "update" else 64, prec=prec, seed=SEED_KEY)
    if kind == "update":
        s["stats"] = torch.empty((case["utd"], 8), device=DEV)
        if case["store"] == "ring":
            # the program's replay holds squinted transitions, inserted as they were observed
            t, ring = s.pop("replay"), api.Ring(c, _rows(case))
            for i in range(0, _rows(case), 1024):
                ring.insert(*(t[k][i:i + 1024] for k in ring.FIELDS))
            s["replay"] = ring
        else:
            s["replay"]["size"] = _rows(case)
    if kind in ("actor", "adam"):
        s["hp"] = _lib.make_hparams(c["action"], prec=prec)
    return s


def run(s):
    case, c, prec, kind = s["case"], s["cfg"], s["prec"], s["case"]["kind"]
    if kind == "act":
        return s["agent"].act(s["frames"], s["proprio"], sample=case["sample"], request_id=REQUEST)
    if kind == "update":
        a = s["agent"]
        stats = a.sac_update(s["replay"], case["utd"], stats=s["stats"])
        return dict(stats=stats, params=a.params, target=a.target, m=a.m, v=a.v, grads=a.grads)
    if kind == "encoder":
        feat, ws = api.encoder_fwd(c, prec, s["params"], s["x"])
        return dict(feat=feat, grad=api.encoder_bwd(c, prec, s["params"], ws, s["dfeat"], s["params"].numel()))
    if kind == "critic":
        logits, ws = api.critic_fwd(c, prec, s["params"], s["feat"], s["proprio"], s["action"])
        dp, df, da = api.critic_bwd(c, prec, s["params"], ws, s["dlogits"])
        return dict(logits=logits, grad=dp, dfeat=df, daction=da)
    if kind == "actor":
        action, logp, ws = api.actor_fwd(c, prec, s["hp"], s["params"], s["feat"], s["proprio"], s["eps"])
        return dict(action=action, logp=logp,
                    grad=api.actor_bwd(c, prec, s["hp"], s["params"], ws, s["daction"], s["dlogp"]))
    if kind == "squint":
        return api.squint_downsample(c, s["frames"], idx=s["idx"], prec=prec)
    if kind == "project":
        return api.c51_project(c, s["p"], s["reward"], s["done"], s["bonus"], 0.99)
    api.adam_step(s["p"], s["g"], s["m"], s["v"], s["hp"], s["step"], ema_target=s["ema"], ema_begin=s["lo"])
    return dict(p=s["p"], m=s["m"], v=s["v"], ema=s["ema"], step=s["step"])


# ---------------------------------------------------------------- the work of a pass
def work(case):
    c, n, kind = NETS[case["net"]], case["n"], case["kind"]
    table, ends = _table(c)
    sides, P, H, A, S, N = _sides(c), c["proj"], c["hidden"], c["action"], c["proprio"], c["atoms"]
    flat, frame = c["F"] * sides[-1] ** 2, c["H"] * c["W"] * c["C"]
    n_enc, n_critic, n_actor = ends["enc"], ends["critic"] - ends["enc"], ends["actor"] - ends["critic"]
    # multiply-adds per row: each convolution, the critics, the actor
    conv = [c["F"] * (c["C"] if i == 0 else c["F"]) * 9 * sides[i + 1] ** 2 for i in range(c["n_conv"])]
    enc, enc_bwd = sum(conv), sum(conv) + sum(conv[1:])
    q_in, q_mid = flat * P, 2 * ((P + S + A) * H + H * H + H * N)
    pi_in, pi_mid = flat * P, (P + S) * H + H * H + 2 * A * H
    critic, actor = q_in + q_mid, pi_in + pi_mid
    actor_bwd = actor + P * H + H * H + 2 * A * H
    if kind == "act":
        return dict(bytes=n * (frame + 4 * (S + A)) + 4 * (n_enc + n_actor), flops=2 * n * (enc + actor))
    if kind == "update":
        stored = frame if case["store"] == "raw" else sides[0] ** 2 * c["C"]
        b = n * (2 * stored + 4 * (2 * S + A + 1) + 1) + 28 * ends["total"] + 8 * n_critic
        macs = n * (2 * enc + enc_bwd + 2 * actor + 2 * critic + 2 * critic
                    + critic + 2 * (A * H + H * H + H * N) + actor_bwd)
        return dict(bytes=case["utd"] * b, flops=2 * case["utd"] * macs)
    if kind == "encoder":
        return dict(bytes=4 * (n * (2 * c["C"] * sides[0] ** 2 + 2 * flat) + 3 * n_enc), flops=2 * n * (enc + enc_bwd))
    if kind == "critic":
        return dict(bytes=4 * (n * (3 * flat + 2 * (S + A) + A + 4 * N) + 3 * n_critic), flops=6 * n * critic)
    if kind == "actor":
        return dict(bytes=4 * (n * (2 * flat + 2 * S + 4 * A + 2) + 3 * n_actor), flops=2 * n * (actor + actor_bwd))
    if kind == "squint":
        return dict(bytes=n * (frame + 4 + (4 if case["prec"] == "fp32" else 2) * c["C"] * sides[0] ** 2),
                    flops=n * frame)
    if kind == "project":
        return dict(bytes=n * (8 * N + 9), flops=8 * n * N)
    return dict(bytes=28 * n + 8 * (n - min(n, ends["enc"])), flops=16 * n)


# ---------------------------------------------------------------- 64 bits
def _conv(x, W, b, stride):
    """3x3 valid convolution as one product over its patches."""
    n, _, h, _ = x.shape
    o = (h - 3) // stride + 1
    cols = F.unfold(x, 3, stride=stride)                                     # [n, C 9, o o]
    y = cols.transpose(1, 2).reshape(n * o * o, -1) @ W.reshape(W.shape[0], -1).t() + b
    return y.reshape(n, o * o, -1).transpose(1, 2).reshape(n, -1, o, o)


def _encode(P, x, n_conv):
    for i in range(n_conv):
        x = torch.relu(_conv(x, P[f"conv{i}.W"], P[f"conv{i}.b"], 1 if i else 2))
    return x.flatten(1)


def _dense(P, name, x, act):
    y = x @ P[name + ".W"].t() + P[name + ".b"]
    return act(F.layer_norm(y, (y.shape[1],), P[name + ".g"], P[name + ".h"], 1e-5))


def _mlp(P, name, x):
    x = _dense(P, name + ".l2", _dense(P, name + ".l1", x, torch.relu), torch.relu)
    return x @ P[name + ".out.W"].t() + P[name + ".out.b"]


def _critic(P, feat, s, a):
    x = torch.cat([_dense(P, "critic", feat, torch.tanh), s, a], 1)
    return torch.stack([_mlp(P, "q1", x), _mlp(P, "q2", x)])


def _policy(P, feat, s, eps):
    """(action, log pi) of the tanh-Gaussian sample at noise eps; the mean action for None."""
    out = _mlp(P, "pi", torch.cat([_dense(P, "actor", feat, torch.tanh), s], 1))
    mu, us = out.chunk(2, 1)
    if eps is None:
        return torch.tanh(mu), None
    log_std = -5 + 3.5 * (torch.tanh(us) + 1)
    v = mu + log_std.exp() * eps
    logp = -0.5 * eps * eps - log_std - 0.5 * math.log(2 * math.pi) - 2 * (math.log(2) - v - F.softplus(-2 * v))
    return torch.tanh(v), logp.sum(1)


def _squint(frames, k):
    n, h, w, c = frames.shape
    x = frames.double().reshape(n, h // k, k, w // k, k, c).sum((2, 4)) / (255.0 * k * k) - 0.5
    return x.permute(0, 3, 1, 2).contiguous()


def _stored(frames, k):
    """The block means that a ring keeps: whole numbers, ties to even."""
    n, h, w, c = frames.shape
    return torch.round(frames.double().reshape(n, h // k, k, w // k, k, c).sum((2, 4)) / (k * k)).to(torch.uint8)


def _project(p, reward, done, bonus, gamma, c):
    N = p.shape[1]
    dz = (c["v_max"] - c["v_min"]) / (N - 1)
    z = c["v_min"] + dz * torch.arange(N, dtype=torch.float64, device=p.device)
    b = ((reward[:, None] + gamma * (1 - done[:, None]) * (z + bonus[:, None]) - c["v_min"]) / dz).clamp(0, N - 1)
    lo = b.floor()
    w = b - lo
    m = torch.zeros_like(p).scatter_add_(1, lo.long(), p * (1 - w))
    return m.scatter_add_(1, (lo + 1).clamp(max=N - 1).long(), p * w), z


def _philox(c0, c1, c2, c3):
    """Philox4x32-10 (Salmon et al., SC'11) at the agents' key; the first two words."""
    x = [np.asarray(v, dtype=np.uint64) for v in np.broadcast_arrays(c0, c1, c2, c3)]
    k0, k1, low = SEED_KEY, 0, np.uint64(0xFFFFFFFF)
    for _ in range(10):
        p0, p1 = np.uint64(0xD2511F53) * x[0], np.uint64(0xCD9E8D57) * x[2]
        x = [(p1 >> np.uint64(32)) ^ x[1] ^ np.uint64(k0), p1 & low,
             (p0 >> np.uint64(32)) ^ x[3] ^ np.uint64(k1), p0 & low]
        k0, k1 = (k0 + 0x9E3779B9) & 0xFFFFFFFF, (k1 + 0xBB67AE85) & 0xFFFFFFFF
    return x[0], x[1]


def _normal(words):
    u = [((w >> np.uint64(9)).astype(np.float64) + 0.5) * 2.0 ** -23 for w in words]
    return torch.from_numpy(np.sqrt(-2 * np.log(u[0])) * np.cos(2 * np.pi * u[1])).to(DEV)


def _adam(p, g, m, v, t, lr=3e-4, b1=0.9, b2=0.999, eps=1e-8):
    m.mul_(b1).add_((1 - b1) * g)
    v.mul_(b2).add_((1 - b2) * g * g)
    p.sub_(lr * (m / (1 - b1 ** t)) / ((v / (1 - b2 ** t)).sqrt() + eps))


def _exact_update(case, i):
    c, B, A, gamma = NETS[case["net"]], case["n"], NETS[case["net"]]["action"], 0.99
    table, ends = _table(c)
    e, q, a_end = ends["enc"], ends["critic"], ends["actor"]
    p = i["params"].double()
    target, m, v, grads = p[e:q].clone(), torch.zeros_like(p), torch.zeros_like(p), torch.zeros_like(p)
    rep, rows, stats = i["replay"], _rows(case), []
    for u in range(case["utd"]):
        w, _ = _philox(u, 0, np.arange(B), 0)
        idx = torch.from_numpy(((w * np.uint64(rows)) >> np.uint64(32)).astype(np.int64)).to(DEV)
        eps = [_normal(_philox(u, k, np.arange(B * A), 0)).view(B, A) for k in (1, 2)]
        t = {k: rep[k][idx] for k in rep}
        f64 = lambda k: t[k].double()
        if case["store"] == "raw":
            x = torch.cat([_squint(t["obs"], c["k"]), _squint(t["next_obs"], c["k"])])
        else:
            x = torch.cat([_squint(_stored(t["obs"], c["k"]), 1), _squint(_stored(t["next_obs"], c["k"]), 1)])
        s, s2, r, done = f64("proprio"), f64("next_proprio"), f64("reward"), f64("done")
        leaf = p.clone().requires_grad_(True)
        P = _view(leaf, table)
        feat = _encode(P, x, c["n_conv"])
        alpha = P["log_alpha"].exp().item()
        with torch.no_grad():
            a2, logp2 = _policy(P, feat[B:], s2, eps[0])
            bar = torch.softmax(_critic(_view(target, table, e), feat[B:], s2, a2), -1).mean(0)
            want, z = _project(bar, r, done, -alpha * logp2, gamma, c)
        logits = _critic(P, feat[:B], s, f64("action"))
        loss = -(want * torch.log_softmax(logits, -1)).sum(-1).mean(1).sum()
        grads[:q] = torch.autograd.grad(loss, leaf)[0][:q]
        q_rep = (torch.softmax(logits.detach(), -1) @ z).mean()
        with torch.no_grad():
            _adam(p[:q], grads[:q], m[:q], v[:q], u + 1)
        a_t, logp = _policy(P, feat[:B].detach(), s, eps[1])
        ent = -logp.detach().mean()
        grads[a_end:] = alpha * (ent + A)
        with torch.no_grad():
            _adam(p[a_end:], grads[a_end:], m[a_end:], v[a_end:], u + 1)
        alpha2 = p[a_end:].exp().item()
        qa = (torch.softmax(_critic(_view(p, table), feat[:B].detach(), s, a_t), -1) @ z).mean(0)
        pi_loss = (alpha2 * logp - qa).mean()
        grads[q:a_end] = torch.autograd.grad(pi_loss, leaf)[0][q:a_end]
        with torch.no_grad():
            _adam(p[q:a_end], grads[q:a_end], m[q:a_end], v[q:a_end], u + 1)
            target.mul_(0.995).add_(0.005 * p[e:q])
        stats.append([loss.item(), pi_loss.item(), (alpha * (ent + A)).item(), alpha2, ent.item(), q_rep.item(),
                      (want @ z).mean().item(), 0.0])
    return dict(stats=torch.tensor(stats, dtype=torch.float64), params=p, target=target, m=m, v=v, grads=grads)


def exact(case, seed):
    c, kind, n = NETS[case["net"]], case["kind"], case["n"]
    table, ends = _table(c)
    i = _inputs(case, seed)
    d = {k: t.double() if torch.is_tensor(t) and t.is_floating_point() else t for k, t in i.items()}
    if kind == "act":
        P = _view(d["params"], table)
        e = np.arange(n * c["action"])
        eps = _normal(_philox(e, 3, REQUEST, 0)).view(n, -1) if case["sample"] else None
        out = [_policy(P, _encode(P, _squint(i["frames"][k:k + 1024], c["k"]), c["n_conv"]), d["proprio"][k:k + 1024],
                       None if eps is None else eps[k:k + 1024])[0] for k in range(0, n, 1024)]
        return torch.cat(out)
    if kind == "update":
        return _exact_update(case, i)
    if kind == "encoder":
        leaf = d["params"].requires_grad_(True)
        feat = _encode(_view(leaf, table), d["x"], c["n_conv"])
        return dict(feat=feat.detach(), grad=torch.autograd.grad(feat, leaf, d["dfeat"])[0])
    if kind == "critic":
        leaves = [d[k].requires_grad_(True) for k in ("params", "feat", "action")]
        logits = _critic(_view(leaves[0], table, ends["enc"]), leaves[1], d["proprio"], leaves[2])
        dp, df, da = torch.autograd.grad(logits, leaves, d["dlogits"])
        return dict(logits=logits.detach(), grad=dp, dfeat=df, daction=da)
    if kind == "actor":
        leaf = d["params"].requires_grad_(True)
        action, logp = _policy(_view(leaf, table, ends["critic"]), d["feat"], d["proprio"], d["eps"])
        grad = torch.autograd.grad([action, logp], leaf, [d["daction"], d["dlogp"]])[0]
        return dict(action=action.detach(), logp=logp.detach(), grad=grad)
    if kind == "squint":
        return torch.cat([_squint(i["frames"][i["idx"][k:k + 256].long()], c["k"]) for k in range(0, n, 256)])
    if kind == "project":
        return _project(d["p"], d["reward"], i["done"].double(), d["bonus"], 0.99, c)[0]
    p, m, v = d["p"].clone(), d["m"].clone(), d["v"].clone()
    _adam(p, d["g"], m, v, 21)
    return dict(p=p, m=m, v=v, ema=0.995 * d["ema"] + 0.005 * p[i["lo"]:], step=None)
