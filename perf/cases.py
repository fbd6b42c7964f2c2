"""The workloads this framework's speed is measured on.

Every case goes through the public Python binding over libdedloc, with the
buffers, call handles and workspace a training program keeps from one
averaging round to the next.  Six kinds of call cover what such a program
has the library do on the GPU:

  round       one averaging round over every peer's message with the LAMB or
              LARS step (dedloc_round / dedloc_round_lars), as a rule with
              this GPU's own fp32 gradient encoded on the way (local peer);
  step        the optimizer step alone on a gradient averaged elsewhere;
  reduce      one reducer's shard: the weighted average of the peers'
              messages, re-encoded;
  group       the group all-reduce (all its iterations);
  accumulate  a peer's side between two rounds: micro-batch gradients added
              up, then the mean encoded as its message;
  codec       a message encoded by the sender and decoded by the receiver.

The load balancer and the shard bounds are host planning, done when the
membership changes, and are not timed here.
"""

import math

import numpy as np
import torch

from paper_2106_10207_amd import dedloc as D
from paper_2106_10207_amd import workloads as W

BLOCK = D.DEDLOC_I8_BLOCK
CODEC = {"fp16": D.DEDLOC_CODEC_FP16, "i8": D.DEDLOC_CODEC_I8, "f32": D.DEDLOC_CODEC_F32}
# The benchmark's hyper-parameters.  LARS: a learning rate of the warm-up,
# so that thousands of timed steps on one state stay finite.
LAMB = dict(lr=1e-3, beta1=0.9, beta2=0.999, eps=1e-6, weight_decay=0.01, step=10)
LARS = dict(lr=0.1, momentum=0.9, trust_coef=1e-3, weight_decay=1e-6)


# ------------------------------------------------------------------ the cases

def listed():
    return [
        # the smallest round: 2^20 parameters over 4 peers; launches and latency count
        dict(name="round tiny", kind="round", table="tiny", peers=4, zero=0, wire="fp16", opt="lamb", local=True),
        # the headline: ALBERT-large trained by 16 peers, fp16 messages
        dict(name="round albert_large", kind="round", table="albert_large", peers=16, zero=0, wire="fp16", opt="lamb",
             local=True),
        # SwAV's shape: ResNet-50 (161 tensors, most of them tiny) with LARS, 32 peers
        dict(name="round resnet50 lars", kind="round", table="resnet50", peers=32, zero=0, wire="fp16", opt="lars",
             local=True),
        # sahajBERT-XL's shape: int8 messages of 64 peers, four of them without samples
        dict(name="round albert_xlarge i8", kind="round", table="albert_xlarge", peers=64, zero=4, wire="i8",
             opt="lamb", local=True),
        # the largest: 2^30 parameters in 1024 tensors, 8 peers
        dict(name="round stress", kind="round", table="stress", peers=8, zero=0, wire="fp16", opt="lamb", local=False),
        # a collaboration of volunteers: more peers than one launch takes, some without samples
        dict(name="round 150 peers", kind="round", table="albert_large", peers=150, zero=6, wire="fp16", opt="lamb",
             local=True),
        # the step alone, on an fp32 gradient averaged elsewhere
        dict(name="lamb step f32", kind="step", table="albert_large", wire="f32", opt="lamb"),
        # the LARS step on a decoded-on-the-way int8 message, a table of mixed odd sizes
        dict(name="lars step i8", kind="step", table="mixed:3:90:6000013", wire="i8", opt="lars"),
        # one reducer's equal share of ALBERT-large (a ragged length), 16 peers
        dict(name="reduce shard fp16", kind="reduce", n=1105243, peers=16, zero=0, wire="fp16"),
        # 64 peers in groups of 4 (three iterations), int8 messages of ALBERT-large
        dict(name="group 64 by 4 i8", kind="group", n=17683968, peers=64, zero=3, wire="i8", m=4),
        # a fast peer's round: four fp16 micro-batches added up, then its fp16 message
        dict(name="accumulate fp16", kind="accumulate", n=17683968, grads="fp16", batches=4, wire="fp16"),
        # one ResNet-50 message through the int8 wire: sender, then receiver
        dict(name="codec i8", kind="codec", n=25557032, wire="i8"),
    ]


def draw(rng):
    """One more case of the listed ones' ranges."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    def wire():
        return rng.choice(["fp16", "fp16", "i8"])

    kind = rng.choice(["round"] * 5 + ["step", "step", "reduce", "group", "accumulate", "codec"])
    if kind == "round":
        peers = log(2, 200)
        # messages of at most the largest listed round's (16 GB), and 2^30 parameters
        P = min(log(100_000, 1 << 30), int(8e9 / peers))
        table = "mixed:%d:%d:%d" % (rng.randrange(1 << 20), log(1, 600), P)
        zero = rng.choice([0, 0, rng.randrange(0, max(1, peers // 8))])
        return dict(kind=kind, table=table, peers=peers, zero=zero, wire=wire(), opt=rng.choice(["lamb", "lamb", "lars"]),
                    local=rng.random() < 0.7)
    if kind == "step":
        table = "mixed:%d:%d:%d" % (rng.randrange(1 << 20), log(1, 600), log(20_000, 200_000_000))
        return dict(kind=kind, table=table, wire=rng.choice(["f32", "fp16", "i8"]), opt=rng.choice(["lamb", "lars"]))
    n = log(10_000, 60_000_000)
    if kind == "reduce":
        peers = log(2, 200)
        return dict(kind=kind, n=min(n, int(4e9 / peers)), peers=peers, zero=rng.choice([0, peers // 10]), wire=wire())
    if kind == "group":
        peers = log(4, 128)
        return dict(kind=kind, n=min(n, int(3e9 / peers)), peers=peers, zero=rng.choice([0, peers // 10]), wire=wire(),
                    m=rng.choice([2, 3, 4, 8]))
    if kind == "accumulate":
        return dict(kind=kind, n=n, grads=rng.choice(["fp16", "f32"]), batches=rng.randrange(1, 9), wire=wire())
    return dict(kind=kind, n=n, wire=wire())


# ------------------------------------------------------------ inputs of a case

def table_of(case):
    """(offsets uint64[T+1], kinds) of the case's tensor table."""
    name = case["table"]
    if name in W.WORKLOADS:
        t = W.WORKLOADS[name].tensors
        sizes, kinds = [n for _, n, _ in t], [k for _, _, k in t]
    else:
        # "mixed:seed:T:P": T tensors of P elements in all, matrices of very
        # different sizes among small gains and biases; every size but the
        # last a multiple of 8
        _, seed, T, P = name.split(":")
        r, T, P = np.random.default_rng(int(seed)), int(T), int(P)
        small = r.random(T) < 0.5
        small[-1] = False
        share = np.where(small, 0.0, np.exp(r.normal(0.0, 1.3, T)))
        sizes = np.where(small, 8 * r.integers(8, 257, T), 0).astype(np.int64)
        rest = max(0, P - int(sizes.sum()))
        sizes = sizes + (rest * share / share.sum()).astype(np.int64) // 8 * 8
        end = np.minimum(np.cumsum(sizes), P // 8 * 8)
        end[-1] = P
        sizes = np.diff(np.concatenate([[0], end]))
        kinds = ["g" if s and i % 2 else "b" if s else "w" for i, s in enumerate(small)]
    off = np.zeros(len(sizes) + 1, np.uint64)
    off[1:] = np.cumsum(np.asarray(sizes, np.uint64))
    return off, kinds


def flags_of(kinds):
    return np.array([{"w": 3, "g": 2, "b": 2}[k] for k in kinds], np.uint8)


def elements(case):
    return int(table_of(case)[0][-1]) if "table" in case else int(case["n"])


def counts_of(case, seed):
    """Samples per peer: 8 to 256 each; `zero` of the peers have none."""
    r = np.random.default_rng(1000 + seed)
    c = r.integers(8, 257, case["peers"]).astype(np.uint32)
    c[r.choice(case["peers"], case["zero"], replace=False)] = 0
    return c


def generator(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    return g


def gradient(n, g):
    """A mean gradient: N(0, 1e-3^2)."""
    return torch.randn(n, generator=g, device="cuda").mul_(1e-3)


def message(x, wire):
    """(codes, scales) of a message as the wire format defines it."""
    if wire == "fp16":
        return x.half().view(torch.int16), None
    n = x.numel()
    pad = torch.nn.functional.pad(x, (0, -n % BLOCK)).view(-1, BLOCK)
    s = pad.abs().amax(1) / 127.0
    q = (pad / torch.where(s > 0, s, 1.0)[:, None]).round_().clamp_(-127, 127).to(torch.int8)
    return q.view(-1)[:n].clone(), s


def messages(case, n, seed):
    """Every peer's message; a peer without samples has none."""
    counts, g = counts_of(case, seed), generator(seed)
    out = [message(gradient(n, g), case["wire"]) if c else (None, None) for c in counts]
    return counts, [c for c, _ in out], [s for _, s in out]


def state_of(case, seed):
    """x, m, v as in the middle of training."""
    off, kinds = table_of(case)
    P, g = int(off[-1]), generator(seed + 500_000_000)
    x = torch.randn(P, generator=g, device="cuda").mul_(0.02)
    for i, k in enumerate(kinds):
        if k != "w":
            x[int(off[i]):int(off[i + 1])] = 1.0 if k == "g" else 1e-3
    m = torch.randn(P, generator=g, device="cuda").mul_(1e-4)
    v = torch.randn(P, generator=g, device="cuda").mul_(1e-3).square_()
    return off, kinds, x, m, v


def empty_message(n, wire):
    codes = torch.empty(n, dtype=torch.int16 if wire == "fp16" else torch.int8, device="cuda")
    return codes, torch.empty(-(-n // BLOCK), device="cuda") if wire == "i8" else None


def local_of(counts):
    return int(np.flatnonzero(counts)[0])


def micro_batches(case, seed):
    g = generator(seed)
    grads = [gradient(case["n"], g) for _ in range(case["batches"])]
    sizes = np.random.default_rng(seed).integers(1, 33, case["batches"])
    return [x.half() if case["grads"] == "fp16" else x for x in grads], [int(b) for b in sizes]


# ----------------------------------------------------------------- a pass

def prepare(case, seed):
    kind, wire, n = case["kind"], case["wire"], elements(case)
    codec = CODEC[wire]
    s = dict(kind=kind, n=n, codec=codec)
    if kind == "round":
        counts, codes, scales = messages(case, n, seed)
        off, kinds, x, m, v = state_of(case, seed)
        out, out_scales = empty_message(n, wire)
        trust = torch.empty(len(kinds), device="cuda")
        # more than 64 peers with samples need the fp32 average's buffer
        mean = torch.empty(n, device="cuda") if np.count_nonzero(counts) > 64 else None
        bounds = D.dedloc_partition(n, case["peers"], None, BLOCK if wire == "i8" else 64)
        local = None
        if case["local"]:
            p = local_of(counts)
            local = (p, gradient(n, generator(seed + 900_000_000)))
        lamb = case["opt"] == "lamb"
        cfg = D.lamb_cfg(**LAMB) if lamb else D.lars_cfg(**LARS)
        s["call"] = D.RoundCall(codes, counts, bounds, codec, out, x, m if lamb else None, v if lamb else m, off,
                                flags_of(kinds), cfg, D.make_workspace(n, off), scales if wire == "i8" else None,
                                out_scales, trust, mean, BLOCK, local)
        s["out"] = dict(codes=out, x=x, m=m, trust=trust)
        if lamb:
            s["out"]["v"] = v
        if wire == "i8":
            s["out"]["scales"] = out_scales
        if mean is not None:
            s["out"]["mean"] = mean
        if local is not None:
            s["out"]["sent"] = codes[p]
            if wire == "i8":
                s["out"]["sent_scales"] = scales[p]
    elif kind == "step":
        off, kinds, x, m, v = state_of(case, seed)
        grad = gradient(n, generator(seed))
        scales = None
        if wire != "f32":
            grad, scales = message(grad, wire)
        trust = torch.empty(len(kinds), device="cuda")
        lamb = case["opt"] == "lamb"
        s.update(lamb=lamb, x=x, m=m, v=v, grad=grad, scales=scales, off=off, flags=flags_of(kinds), trust=trust,
                 cfg=D.lamb_cfg(**LAMB) if lamb else D.lars_cfg(**LARS), ws=D.make_workspace(n, off))
    elif kind == "reduce":
        counts, codes, scales = messages(case, n, seed)
        out, out_scales = empty_message(n, wire)
        s.update(counts=counts, codes=codes, scales=scales if wire == "i8" else None, out=out, out_scales=out_scales,
                 mean=torch.empty(n, device="cuda") if np.count_nonzero(counts) > 64 else None)
    elif kind == "group":
        counts, codes, scales = messages(case, n, seed)
        s["call"] = D.GroupAllreduce(codes, counts, case["m"], n, codec, scales if wire == "i8" else None)
    elif kind == "accumulate":
        grads, sizes = micro_batches(case, seed)
        out, out_scales = empty_message(n, wire)
        s.update(grads=grads, sizes=sizes, acc=torch.zeros(n, device="cuda"), out=out, out_scales=out_scales)
    else:
        out, out_scales = empty_message(n, wire)
        s.update(x=gradient(n, generator(seed)), out=out, out_scales=out_scales, back=torch.empty(n, device="cuda"))
    return s


def run(s):
    kind = s["kind"]
    if kind == "round":
        s["call"]()
        return s["out"]
    if kind == "step":
        if s["lamb"]:
            D.dedloc_lamb_step(s["x"], s["m"], s["v"], s["grad"], s["off"], s["flags"], s["cfg"], s["codec"],
                               s["scales"], trust_out=s["trust"], ws=s["ws"])
            return dict(x=s["x"], m=s["m"], v=s["v"], trust=s["trust"])
        D.dedloc_lars_step(s["x"], s["m"], s["grad"], s["off"], s["flags"], s["cfg"], s["codec"], s["scales"],
                           trust_out=s["trust"], ws=s["ws"])
        return dict(x=s["x"], m=s["m"], trust=s["trust"])
    if kind == "reduce":
        D.dedloc_reduce_shard(s["codes"], s["counts"], s["n"], s["codec"], s["scales"], out_codes=s["out"],
                              out_scales=s["out_scales"], out_mean=s["mean"])
        return dict(codes=s["out"], scales=s["out_scales"], mean=s["mean"])
    if kind == "group":
        g = s["call"]()
        out = g.out[:g.n_out * g.stride].view(g.n_out, g.stride)  # every group's message, in its padded row
        return dict(out=out[:, :s["n"] * (2 if s["codec"] == CODEC["fp16"] else 1)], scales=g.out_scales,
                    peer_out=g.peer_out)
    if kind == "accumulate":
        for grad, b in zip(s["grads"], s["sizes"]):
            D.dedloc_accumulate(s["acc"], grad, b)
        D.dedloc_finalize(s["acc"], sum(s["sizes"]), s["codec"], codes=s["out"], scales=s["out_scales"])
        return dict(codes=s["out"], scales=s["out_scales"], acc=s["acc"])
    D.dedloc_encode(s["x"], s["codec"], codes=s["out"], scales=s["out_scales"])
    D.dedloc_decode(s["out"], s["out_scales"], s["n"], s["codec"], out=s["back"])
    return dict(codes=s["out"], scales=s["out_scales"], back=s["back"])


# ------------------------------------------------------- what a pass needs

def code_bytes(wire):
    return {"fp16": 2.0, "i8": 1.0 + 4.0 / BLOCK, "f32": 4.0}[wire]


def work(case):
    """Every input read once, every output written once."""
    n, kind, b = elements(case), case["kind"], code_bytes(case["wire"])
    if kind == "round":
        active = case["peers"] - case["zero"]
        state, ops = (24, 22) if case["opt"] == "lamb" else (16, 10)
        per = active * b + b + state + (4 if case["local"] else 0) + (4 if active > 64 else 0)
        return dict(bytes=per * n, flops=(2 * active + ops) * n)
    if kind == "step":
        return dict(bytes=(b + (24 if case["opt"] == "lamb" else 16)) * n, flops=(22 if case["opt"] == "lamb" else 10) * n)
    if kind == "reduce":
        active = case["peers"] - case["zero"]
        return dict(bytes=(active * b + b + (4 if active > 64 else 0)) * n, flops=2 * active * n)
    if kind == "group":
        # the peers' messages and the group messages every peer ends with
        active, d = case["peers"] - case["zero"], D.group_iterations(case["peers"], case["m"])
        return dict(bytes=(active + case["m"] ** (d - 1)) * b * n, flops=2 * active * n)
    if kind == "accumulate":
        # the micro-batches, the zeroed accumulator and the message
        return dict(bytes=(case["batches"] * code_bytes(case["grads"]) + 4 + b) * n, flops=2 * case["batches"] * n)
    return dict(bytes=(4 + b + 4) * n, flops=3 * n)


def tolerance(case):
    """Codes, scales and averages are fixed bit by bit by the wire format and
    by the order of the average.  The optimizer's norms may be added in any
    order, which moves the ratios, and by them the parameters, by fp32
    rounding: measured against 64 bits with the same codes, 2.6e-8 in x and
    up to 6.7e-8 in the ratios."""
    if case["kind"] in ("round", "step"):
        return dict(rel=3e-7, max=1e-6, differ=0.0)
    return "exact"


# --------------------------------------------------- the same in 64 bits

def decoded(codes, scales, wire):
    if wire == "f32":
        return codes.double()
    if wire == "fp16":
        return codes.view(torch.float16).double()
    return codes.double() * scales.double().repeat_interleave(BLOCK)[:codes.numel()]


def wired(x, wire):
    """(decode(encode(x)), scales) for x in 64 bits."""
    if wire == "fp16":
        return x.half().double(), None
    n = x.numel()
    pad = torch.nn.functional.pad(x, (0, -n % BLOCK)).view(-1, BLOCK)
    s = pad.abs().amax(1) / 127.0
    q = (pad / torch.where(s > 0, s, 1.0)[:, None]).round_().clamp_(-127, 127)
    return (q * s[:, None]).view(-1)[:n], s


def average(counts, values):
    """The sample-weighted mean of the decoded messages."""
    total, out = float(sum(int(c) for c in counts)), None
    for c, v in zip(counts, values):
        if c:
            out = v() * (int(c) / total) if out is None else out.add_(v(), alpha=int(c) / total)
    return out


def f32(v):
    return float(np.float32(v))


def optimized(case, off, kinds, x, m, v, g):
    """x', m', v', trust of one optimizer step in 64 bits (v: LAMB only)."""
    flags, trust = flags_of(kinds), torch.ones(len(kinds), dtype=torch.float64, device="cuda")
    x, m = x.double(), m.double()
    if case["opt"] == "lamb":
        b1, b2, c = f32(LAMB["beta1"]), f32(LAMB["beta2"]), LAMB
        v = v.double()
        m.mul_(b1).add_(g, alpha=1 - b1)
        v.mul_(b2).addcmul_(g, g, value=1 - b2)
        c1, c2 = 1 - b1 ** c["step"], 1 - b2 ** c["step"]
    for t in range(len(kinds)):
        a, b = int(off[t]), int(off[t + 1])
        if a == b:
            continue
        xt, wd = x[a:b], f32((LAMB if case["opt"] == "lamb" else LARS)["weight_decay"]) if flags[t] & 1 else 0.0
        if case["opt"] == "lamb":
            u = (m[a:b] / c1) / ((v[a:b] / c2).sqrt_() + f32(LAMB["eps"])) + wd * xt
            X, Y = xt.norm(), u.norm()
            r = torch.where((X > 0) & (Y > 0), X / Y, 1.0)
            xt.sub_(f32(LAMB["lr"]) * r * u)
        else:
            gt = g[a:b]
            X, Y = xt.norm(), gt.norm()
            r = torch.where((X > 0) & (Y > 0), f32(LARS["trust_coef"]) * X / (Y + wd * X), 1.0)
            m[a:b] = f32(LARS["momentum"]) * m[a:b] + f32(LARS["lr"]) * r * (gt + wd * xt)
            xt.sub_(m[a:b])
        trust[t] = r
    out = dict(x=x, m=m, trust=trust)
    if case["opt"] == "lamb":
        out["v"] = v
    return out


def exact(case, seed):
    kind, wire, n = case["kind"], case["wire"], elements(case)
    if kind == "round":
        counts, codes, scales = messages(case, n, seed)
        p = local_of(counts) if case["local"] else -1
        out = {}

        def value(i):
            if i != p:
                return decoded(codes[i], scales[i], wire)
            d, s = wired(gradient(n, generator(seed + 900_000_000)).double(), wire)
            out["sent_scales"] = s
            return d

        mean = average(counts, [lambda i=i: value(i) for i in range(case["peers"])])
        g, out["scales"] = wired(mean, wire)
        if np.count_nonzero(counts) > 64:
            out["mean"] = mean
        del codes, scales
        off, kinds, x, m, v = state_of(case, seed)
        out.update(optimized(case, off, kinds, x, m, v, g))
        return out
    if kind == "step":
        off, kinds, x, m, v = state_of(case, seed)
        grad, scales = gradient(n, generator(seed)), None
        if wire != "f32":
            grad, scales = message(grad, wire)
        return optimized(case, off, kinds, x, m, v, decoded(grad, scales, wire))
    if kind == "reduce":
        counts, codes, scales = messages(case, n, seed)
        if wire == "fp16" and np.count_nonzero(counts) <= 64:
            return None  # codes only
        mean = average(counts, [lambda i=i: decoded(codes[i], scales[i], wire) for i in range(case["peers"])])
        return dict(codes=None, scales=wired(mean, wire)[1], mean=mean if np.count_nonzero(counts) > 64 else None)
    if kind == "group":
        return None  # codes only, each rounded once an iteration: no value in 64 bits
    if kind == "accumulate":
        grads, sizes = micro_batches(case, seed)
        mean = average(sizes, [lambda g=g: g.double() for g in grads])
        return dict(codes=None, scales=wired(mean, wire)[1], acc=torch.zeros(n, dtype=torch.float64, device="cuda"))
    x = gradient(n, generator(seed)).double()
    back, s = wired(x, wire)
    return dict(codes=None, scales=s, back=back)
