"""The work that this library is measured on: whole passes of one MoE layer and of its scheduler, through
the public entry points, as a program that uses the library calls them.

A case is a dict of plain values.  Kinds:
  forward    gate, token scheduling, permute, expert FFN, combine
  train      the same with pre-activations kept (or not), then the backward pass
  schedule   the scheduler alone, for the next micro-batch of a stream under a restricted placement
  search     construction of an expert placement from known expert loads
Fields of the layer kinds: T, d, f, E, K, G, dtype as in the library; bias (std of the gate's per-expert
bias, which skews the routing) or hot (bias of expert 0 alone); ffn ("ranks": one call per logical rank, as
when a rank is a GPU of its own; "all": one call for all ranks); slots (0: every expert on every rank; else
replica slots per rank of a placement built from the layer's own loads); train: keep ("h": pre-activations
and H kept by the forward pass, "act": pre-activations, "none": recomputed), batches (micro-batches whose
gradients are accumulated).
"""
import math

import numpy as np
import torch

import paper_2511_16947_amd as fm


def _forward(name, T, d, f, E, K, G, dtype="bf16", bias=1.0, hot=0.0, ffn="ranks", slots=0):
    return dict(name=name, kind="forward", T=T, d=d, f=f, E=E, K=K, G=G, dtype=dtype, bias=bias, hot=hot, ffn=ffn,
                slots=slots)


def _train(name, T, d, f, E, K, G, bias=1.0, hot=0.0, ffn="ranks", slots=0, keep="h", batches=1):
    return dict(_forward(name, T, d, f, E, K, G, "bf16", bias, hot, ffn, slots), kind="train", keep=keep, batches=batches)


def listed():
    return [
        # a tiny fp32 layer (unit tests, validation of a training script): launches and latency
        _forward("f32_tiny", 256, 128, 256, 8, 2, 4, dtype="f32", bias=1.5),
        # an fp32 layer of ordinary size: the reference run that a bf16 run is compared with
        _forward("f32_layer", 2048, 1024, 2816, 16, 2, 4, dtype="f32", ffn="all"),
        # one decoding step of a batch of sequences on few large experts, and on many small ones: a few rows
        # per expert, so the experts' weights are what has to be read
        _forward("decode_large_experts", 64, 4096, 14336, 8, 2, 8, ffn="all"),
        _forward("decode_many_experts", 128, 2048, 768, 128, 8, 8, bias=2.0, ffn="all"),
        # prompt processing / the forward half of training on large experts: long segments, bound by the
        # matrix cores (the 8-expert layer of the benchmark)
        _forward("prefill_large_experts", 8192, 4096, 14336, 8, 2, 8),
        # many small experts under heavy skew, one launch per rank (the benchmark's 128-expert layer)
        _forward("prefill_many_experts", 4096, 2048, 768, 128, 8, 8, bias=2.0),
        # 256 experts on 32 ranks, ten replica slots per rank: the regime in which a rank holds a fixed number
        # of experts; 22.5 GB of weights
        _forward("prefill_256_experts", 4096, 7168, 2048, 256, 8, 32, ffn="all", slots=10),
        # sizes that are multiples of nothing much: 1305 tokens on 5 ranks, 17 and 13 64-columns, two to three
        # replicas per expert, three experts per token
        _forward("ragged", 1305, 1088, 832, 20, 3, 5, slots=10),
        # a whole training step, one expert drawing half of all pairs (the benchmark's default workload)
        _train("train_hot_expert", 32768, 2048, 8192, 64, 2, 16, bias=0.0, hot=4.0),
        # training with little memory on many small experts: pre-activations recomputed, gradients
        # accumulated over two micro-batches
        _train("train_recompute", 4096, 2048, 768, 128, 8, 8, ffn="all", keep="none", batches=2),
        # the scheduler alone: the next micro-batch of a stream, started from the last one's replica loads
        dict(name="schedule_stream", kind="schedule", T=4096, E=256, K=8, G=32, slots=10, bias=1.0, drift=0.05),
        # a placement for the loads that the scheduler reported: replica counts and 4096 random candidates
        dict(name="placement_search", kind="search", T=32768, E=64, K=2, G=16, slots=5, n=4096, skew=1.0),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    kind = rng.choice(["forward", "forward", "forward", "decode", "train", "f32", "schedule", "search"])
    if kind == "search":
        G = rng.choice([4, 8, 12, 16])
        E = rng.randint(max(8, G), 128)
        slots = max(-(-E // G), rng.randint(-(-E // G), 2 * -(-E // G)))
        return dict(kind="search", T=32768, E=E, K=2, G=G, slots=slots, n=int(_log(rng, 256, 4096)), skew=rng.uniform(0.3, 1.6))
    if kind == "schedule":
        G = rng.choice([4, 8, 16, 32])
        E = rng.randint(max(8, G), 256)
        return dict(kind="schedule", T=G * int(_log(rng, 512, 8192) / G), E=E, K=rng.randint(1, 8), G=G,
                    slots=-(-5 * E // (4 * G)), bias=rng.uniform(0.3, 1.5), drift=rng.uniform(0.02, 0.1))
    f32 = kind == "f32"
    lo, hi = {"decode": (16, 512), "forward": (512, 8192), "train": (1024, 16384), "f32": (128, 2048)}[kind]
    while True:
        G = rng.choice([1, 2, 4, 5, 8, 8, 16])
        K = rng.choice([1, 2, 2, 3, 4, 6, 8])
        E = max(K, int(_log(rng, 8, 32 if f32 else 192)))
        T = G * max(1, int(_log(rng, lo, hi) / G))
        # fp32 layers of any width, bf16 layers in multiples of 64
        d = int(_log(rng, 128, 1024)) if f32 else 64 * int(_log(rng, 8, 64))
        f = int(_log(rng, 128, 2816)) if f32 else 64 * int(_log(rng, 8, 160))
        flops, weights = 6.0 * T * K * d * f, 3.0 * E * d * f
        if f32 and flops > 7e10:
            continue
        if flops * (3 if kind == "train" else 1) <= 6e12 and weights <= (1e9 if kind == "train" else 6e9):
            break
    slots = 0 if rng.random() < 0.5 or G == 1 else min(E, -(-3 * E // (2 * G)))
    ffn = "all" if kind == "decode" or rng.random() < 0.5 else "ranks"
    if kind == "train":
        c = _train("", T, d, f, E, K, G, rng.uniform(0.3, 2.0), 0.0, ffn, slots, rng.choice(["h", "act", "none"]), rng.choice([1, 1, 2]))
    else:
        c = _forward("", T, d, f, E, K, G, "f32" if f32 else "bf16", rng.uniform(0.3, 2.0), 0.0, ffn, slots)
    del c["name"]
    return c


# ---------------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------------

def _normal(shape, std, gen, dtype):
    t = torch.empty(shape, dtype=dtype, device="cuda")
    t.normal_(0.0, std, generator=gen)
    return t


def _tokens(c, gen, w_router, bias, dtype):
    """x ~ N(0, 1), in which tokens whose choice of experts hangs on the last bits of their logits (two of the
    K + 1 largest closer than 2e-4) are drawn again, so that every correct gate picks the same experts."""
    x = _normal((c["T"], c["d"]), 1.0, gen, dtype)
    kk = min(c["K"] + 1, c["E"])
    for _ in range(20):
        logits = x.double() @ w_router.double() + bias.double()
        top = torch.topk(logits, kk, dim=1).values
        close = ((top[:, :-1] - top[:, 1:]) < 2e-4).any(1).nonzero().flatten() if kk > 1 else top.new_zeros(0)
        if close.numel() == 0:
            break
        x[close] = _normal((close.numel(), c["d"]), 1.0, gen, dtype)
    return x


def _placement(shape, load, slots):
    """The library's own construction: replica counts, then the best of 256 random candidates."""
    i32 = dict(dtype=torch.int32, device="cuda")
    counts, best = torch.empty(shape.E, **i32), torch.empty(1, **i32)
    num, den = torch.empty(256, dtype=torch.int64, device="cuda"), torch.empty(256, **i32)
    place = torch.empty(shape.E, shape.G, dtype=torch.uint8, device="cuda")
    fm.fine_replica_counts(shape, load, slots, counts)
    fm.fine_place_search(shape, load, counts, slots, 256, 1, num, den, best, place)
    return place


class _Layer:
    """What a program keeps for one layer: weights, and the buffers of one micro-batch after another."""

    def __init__(self, c, seed):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        self.c, train = c, c["kind"] == "train"
        flags = fm.FLAG_LOCALITY | (fm.FLAG_ACT_SAVE_H if train and c["keep"] == "h" else 0)
        s = self.shape = fm.Shape(c["T"], c["d"], c["f"], c["E"], c["K"], c["G"],
                                  fm.FINE_F32 if c["dtype"] == "f32" else fm.FINE_BF16, flags)
        dt, E, d, f = s.torch_dtype, s.E, s.d, s.f
        self.w_router = _normal((d, E), 0.02, gen, dt)
        self.bias = _normal((E,), c["bias"], gen, torch.float32) if c["bias"] else torch.zeros(E, device="cuda")
        self.bias[0] += c["hot"]
        n = c.get("batches", 1)
        self.x = [_tokens(c, gen, self.w_router, self.bias, dt) for _ in range(n)]
        self.w_gate, self.w_up = _normal((E, d, f), 0.02, gen, dt), _normal((E, d, f), 0.02, gen, dt)
        self.w_down = _normal((E, f, d), 0.02, gen, dt)

        def rows(n_rows, width=d, dtype=dt):
            return torch.empty(n_rows, width, dtype=dtype, device="cuda")

        self.topk_idx = [rows(s.T, s.K, torch.int32) for _ in range(n)]
        self.topk_w = [rows(s.T, s.K, torch.float32) for _ in range(n)]
        self.sched = fm.SchedBuffers(s)
        self.x_perm, self.y_perm = rows(s.P), rows(s.P)
        self.out = [rows(s.T) for _ in range(n)]
        self.ws_topk, self.ws_ffn = fm.alloc_workspace(s, fm.WS_TOPK), fm.alloc_workspace(s, fm.WS_FFN)
        self.act = None
        if train:
            if c["keep"] != "none":
                self.act = torch.empty(s.P * (3 if c["keep"] == "h" else 2) * f, dtype=dt, device="cuda")
            self.d_out = [_normal((s.T, d), 1.0, gen, dt) for _ in range(n)]
            self.d_x, self.d_topk_w = [rows(s.T) for _ in range(n)], [rows(s.T, s.K, torch.float32) for _ in range(n)]
            self.d_w = [torch.empty(E, *m, device="cuda") for m in ((d, f), (d, f), (f, d))]
            self.ws_bwd = fm.alloc_workspace(s, fm.WS_BACKWARD)
        self.place = None
        if c["slots"]:
            fm.fine_topk(s, self.x[0], self.w_router, self.bias, self.topk_idx[0], self.topk_w[0], self.ws_topk)
            self.sched.run(s, self.topk_idx[0])
            self.place = _placement(s, self.sched.load, c["slots"])

    def forward(self, i):
        s, b = self.shape, self.sched
        fm.fine_topk(s, self.x[i], self.w_router, self.bias, self.topk_idx[i], self.topk_w[i], self.ws_topk)
        b.run(s, self.topk_idx[i], self.place)
        fm.fine_permute(s, self.x[i], b.pair_of_row, self.x_perm)
        for rank in range(s.G) if self.c["ffn"] == "ranks" else (-1,):
            fm.fine_grouped_ffn(s, rank, self.x_perm, self.w_gate, self.w_up, self.w_down, b.seg_off, self.y_perm,
                                self.act, self.ws_ffn)
        fm.fine_combine(s, self.y_perm, b.row_of_pair, self.topk_w[i], self.out[i])

    def backward(self, i):
        b = self.sched
        fm.fine_backward(self.shape, -1, self.d_out[i], self.x_perm, self.y_perm, self.act, self.w_gate, self.w_up,
                         self.w_down, b.row_of_pair, b.pair_of_row, b.seg_off, self.topk_w[i], self.d_x[i],
                         self.d_topk_w[i], *self.d_w, i > 0, self.ws_bwd)

    def run(self):
        res = {"topk_idx": self.topk_idx, "topk_w": self.topk_w, "out": self.out}
        for i in range(len(self.x)):
            self.forward(i)
            if self.c["kind"] == "train":
                self.backward(i)
        if self.c["kind"] == "train":
            res.update(d_x=self.d_x, d_topk_w=self.d_topk_w, d_w=self.d_w)
        return res


class _Schedule:
    def __init__(self, c, seed):
        gen = torch.Generator(device="cuda")
        gen.manual_seed(seed)
        s = self.shape = fm.Shape(c["T"], 64, 64, c["E"], c["K"], c["G"])
        bias = torch.randn(s.E, generator=gen, device="cuda") * c["bias"]

        def routing(b):      # K experts per token in proportion to exp(b), without replacement
            u = torch.rand(s.T, s.E, generator=gen, device="cuda").clamp_(1e-20, 1 - 1e-7)
            return torch.topk(b - torch.log(-torch.log(u)), s.K, dim=1).indices.to(torch.int32).contiguous()

        before = routing(bias)
        self.topk_idx = routing(bias + c["drift"] * torch.randn(s.E, generator=gen, device="cuda"))
        self.out = fm.SchedBuffers(s)
        self.out.run(s, before)
        self.place = _placement(s, self.out.load, c["slots"])
        self.out.run(s, before, self.place)
        self.x_prev = self.out.x_eg.clone()

    def run(self):
        o = self.out
        fm.fine_sched_warm(self.shape, self.topk_idx, self.place, self.x_prev, o.load, o.input_eg, o.x_eg, o.max_load,
                           o.pair_dst, o.row_of_pair, o.pair_of_row, o.seg_off, o.rank_off, o.ws)
        return [o.load, o.input_eg, o.x_eg, o.max_load, o.pair_dst, o.row_of_pair, o.pair_of_row, o.seg_off, o.rank_off]


class _Search:
    def __init__(self, c, seed):
        rng = np.random.default_rng(seed)
        self.c, self.seed = c, int(rng.integers(1 << 31))
        self.shape = fm.Shape(c["T"], 64, 64, c["E"], c["K"], c["G"])
        w = np.arange(1, c["E"] + 1, dtype=np.float64) ** -c["skew"]      # Zipf loads that sum to T K
        load = np.floor(w / w.sum() * c["T"] * c["K"]).astype(np.int32)
        load[0] += c["T"] * c["K"] - int(load.sum())
        i32 = dict(dtype=torch.int32, device="cuda")
        self.load = torch.tensor(rng.permutation(load), **i32)
        self.counts, self.best = torch.empty(c["E"], **i32), torch.empty(1, **i32)
        self.num, self.den = torch.empty(c["n"], dtype=torch.int64, device="cuda"), torch.empty(c["n"], **i32)
        self.place = torch.empty(c["E"], c["G"], dtype=torch.uint8, device="cuda")

    def run(self):
        c = self.c
        fm.fine_replica_counts(self.shape, self.load, c["slots"], self.counts)
        fm.fine_place_search(self.shape, self.load, self.counts, c["slots"], c["n"], self.seed, self.num, self.den,
                             self.best, self.place)
        return [self.counts, self.num, self.den, self.best, self.place]


def prepare(case, seed):
    return {"schedule": _Schedule, "search": _Search}.get(case["kind"], _Layer)(case, seed)


def run(state):
    return state.run()


# ---------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------------------------------------

def _experts_used(c):
    """Experts that get at least one of T tokens, from the choice frequencies of a sample of tokens."""
    rng = np.random.default_rng(1)
    bias = c["bias"] * rng.standard_normal(c["E"])
    bias[0] += c["hot"]
    logits = bias + 0.02 * math.sqrt(c["d"]) * rng.standard_normal((1024, c["E"]))
    chosen = np.argpartition(-logits, c["K"] - 1, axis=1)[:, :c["K"]]
    freq = np.bincount(chosen.ravel(), minlength=c["E"]) / 1024.0
    return float(np.sum(1.0 - (1.0 - freq) ** c["T"]))


def work(case):
    c = case
    T, E, K, G = c["T"], c["E"], c["K"], c["G"]
    P = T * K
    if c["kind"] == "schedule":      # routing and previous loads in; tables, loads and three index arrays out
        return {"bytes": 4 * (P + E * G) + E * G + 4 * (E + 2 * E * G + 3 * P + G * (E + 1) + G + 2), "flops": 0}
    if c["kind"] == "search":        # Eq. 3 over all subsets: G 2^(G-1) additions per candidate
        return {"bytes": 4 * E + 12 * c["n"] + E * G + 4 * E + 4, "flops": c["n"] * G * 2.0 ** (G - 1)}
    d, f, es = c["d"], c["f"], 4 if c["dtype"] == "f32" else 2
    used, n = _experts_used(c), c.get("batches", 1)
    io = n * (2 * T * d * es + 8 * P) + d * E * es                       # x, out, routing; router weights
    weights = 3 * used * d * f * es
    flops = n * (2.0 * T * d * E + 6.0 * P * d * f)
    if c["kind"] == "train":
        io += n * (2 * T * d * es + 4 * P) + 4 * 3 * E * d * f           # d_out, d_x, d_topk_w; weight gradients
        flops += n * 12.0 * P * d * f
    return {"bytes": int(io + weights), "flops": flops}


def tolerance(case):
    if case["kind"] in ("schedule", "search"):
        return "exact"
    if case["dtype"] == "f32":      # seen against 64-bit sums: 1.3e-6, largest 1e-5
        return {"rel": 1e-5, "max": 4e-5, "differ": 0.0}
    # H, y_perm and (backward) the row gradients are rounded to bf16 between the steps.  Seen against the same
    # in 64 bits: out 2.9e-3 (largest 0.018), d_x 4.2e-3, weight gradients 3.5e-3 (largest 0.093)
    return {"rel": 1e-2, "max": 0.4 if case["kind"] == "train" else 0.08, "differ": 0.0}
