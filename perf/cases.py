"""The work that users of this library have it do, as cases that can be timed.

A case is one of these kinds of work, each through the public entry points in
``paper_2401_11469_amd.zr``:

  layer    one resized step of a layer shard: the kept sets of all projections (one selection
           launch), the forward products in order, the backward products (dX and dW) in reverse
           order.  The training step of a straggling task, and what bench.py times.
  refresh  the epoch boundary of priority pruning: weight-variation scores of a layer's shards
           from two snapshots with the incremental rule, and the count above the threshold.
  select   selection from score lists that are not one layer shard's: one long list over a whole
           model, or a batch of equal vectors.
  receive  a receiver's share of the lightweight migration: the migrated columns' partial
           products added to its own results.

The listed cases take their sizes from the workloads in ``workloads.py``; ``draw`` spreads sizes,
ratios, policies, storage layouts and alignments over the ranges those stand for.
"""
from __future__ import annotations

import math

import torch

from paper_2401_11469_amd import workloads as wl
from paper_2401_11469_amd import zr

POLICY = {"zero": zr.ZERO, "average": zr.AVERAGE, "same": zr.SAME}


# ---------------------------------------------------------------------------
# Which cases
# ---------------------------------------------------------------------------
def _shard(cid):
    """The projections of a workload as text: kind:KxN, comma separated."""
    return ",".join(f"{p.parallel}:{p.K}x{p.N}" for p in wl.CONFIGS[cid].projections)


def _layer(name, projections, M, col, row, dtype="bf16", policy="zero", scratch=True, layout="rows", scores="l2"):
    c = dict(kind="layer", projections=projections, M=M, ratio_col=col, ratio_row=row, dtype=dtype, policy=policy,
             scratch=scratch, layout=layout, scores=scores)
    return dict(name=name, **c) if name else c


def listed():
    c = wl.CONFIGS
    llama, gpt2, vit, wide = c[4], c[2], c[3], c[5]
    return [
        # the smallest call in the repository: one fp32 column-parallel linear with the binding's
        # default arguments; launches and host work are what it costs
        _layer("linear-tiny-fp32", _shard(1), c[1].M, 0.25, 0.25, dtype="f32", scratch=False, layout="kn"),
        # small shards, half of them pruned: products of 10 to 40 us each
        _layer("gpt2-medium-tp4-r0.50", _shard(2), gpt2.M, 0.5, 0.5),
        # the token count of an image batch (64 x 197: no multiple of a tile), skewed scores
        _layer("vit-large-tp2-r0.20", _shard(3), vit.M, 0.2, 0.2, scores="lognormal"),
        # a task that does not straggle this step: nothing is pruned
        _layer("llama2-7b-tp4-r0.00", _shard(4), llama.M, 0.0, 0.0),
        # the headline workload at the middle of its ratio list
        _layer("llama2-7b-tp4-r0.25", _shard(4), llama.M, 0.25, 0.25),
        # wide model on many tasks: narrow shards, a ratio of its own per kind of shard
        _layer("llama2-13b-tp8-mixed", _shard(5), wide.M, 0.3, 0.15, scores="uniform"),
        # training in fp32: the image model's shard with a batch of 8 images
        _layer("vit-large-tp2-fp32", _shard(3), 8 * 197, 0.2, 0.2, dtype="f32", scratch=False, scores="lognormal"),
        # the binding's default arguments in bf16: [K x N] storage, no scratch buffer, so every
        # gather happens in flight; the mean as the imputed value
        _layer("gpt2-medium-tp4-defaults", _shard(2), 2 * 1024 - 24, 0.25, 0.25, policy="average", scratch=False,
               layout="kn"),
        # shapes that no vector load fits (a patch embedding or a class head of odd size): rows of
        # 2-byte granularity, the previous step's values as the imputed ones
        _layer("ragged-bf16-same", "col:1001x771,row:771x1001", 5 * 197, 0.25, 0.25, policy="same", layout="kn"),
        # the epoch boundary of one layer: scores from two weight snapshots, half of the model's
        # shards score their columns and half their rows
        dict(name="refresh-llama2-7b", kind="refresh", projections=_shard(4), ratio=0.25, dtype="bf16", layout="kn"),
        # one kept set over all 32 layers of that model (12352 prunable indices a layer)
        dict(name="select-whole-model", kind="select", batch=1, n=32 * 12352, ratio=0.25, scores="lognormal"),
        # the second of three receivers takes its third of what a straggler gives away of a
        # column-parallel shard (backward) and of a row-parallel one (forward; an odd third)
        dict(name="receive-llama2-7b", kind="receive", M=llama.M, col="4096x768", row="688x4096", tasks=4, rank=2,
             dtype="bf16"),
    ]


def _log(rng, lo, hi, step=1):
    """An integer in [lo, hi], uniform in its logarithm, a multiple of `step`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return int(min(hi, max(lo, round(v / step) * step)))


_MOST = 6.0 * 8192 * sum(p.K * p.N for p in wl.CONFIGS[4].projections)      # the largest listed case


def _fit_tokens(M, projections, share):
    """M, lowered until the products of one step stay within `share` of the largest listed case."""
    per = 6.0 * sum(K * N for _, K, N in _parse(projections))
    return max(16, min(M, int(share * _MOST / per)))


def draw(rng):
    kind = rng.choice(["layer"] * 5 + ["fp32", "defaults", "ragged", "refresh", "select", "receive"])
    ratio = 0.0 if rng.random() < 0.1 else round(rng.uniform(0.02, 0.6), 3)
    other = rng.choice([ratio, round(rng.uniform(0.02, 0.6), 3)])
    policy = rng.choice(["zero"] * 6 + ["same", "average"])
    scores = rng.choice(["l2", "lognormal", "uniform"])
    if kind in ("layer", "defaults"):
        # a hidden size and shard widths that 16-byte loads fit, a token count of any kind
        H = _log(rng, 256, 5120, 8)
        ws = [_log(rng, 128, 4096, 8) for _ in range(rng.choice([1, 1, 2]))]
        text = ",".join(f"col:{H}x{w}" for w in ws) + f",row:{ws[-1]}x{H}"
        M = rng.choice([_log(rng, 64, 16384), _log(rng, 64, 16384, 64), 197 * _log(rng, 1, 64)])
        if kind == "layer":
            layout = rng.choice(["rows"] * 3 + ["kn"])
            return _layer(None, text, _fit_tokens(M, text, 0.5 if layout == "rows" else 0.25), ratio, other, policy=policy,
                          layout=layout, scores=scores)
        return _layer(None, text, _fit_tokens(M, text, 0.1), ratio, other, policy=policy, scratch=False,
                      layout=rng.choice(["kn", "rows"]), scores=scores)
    if kind == "fp32":
        K, N = (_log(rng, 64, 2048, rng.choice([4, 4, 1])) for _ in range(2))
        text = rng.choice([f"col:{K}x{N}", f"row:{K}x{N}", f"col:{K}x{N},row:{N}x{K}"])
        return _layer(None, text, _fit_tokens(_log(rng, 32, 4096), text, 0.03), ratio, other, dtype="f32", policy=policy,
                      scratch=rng.random() < 0.5, layout=rng.choice(["kn", "rows"]), scores=scores)
    if kind == "ragged":
        K, N = (_log(rng, 50, 2000) | 1 for _ in range(2))
        text = rng.choice([f"col:{K}x{N}", f"row:{K}x{N}", f"col:{K}x{N},row:{N}x{K}"])
        return _layer(None, text, _fit_tokens(_log(rng, 32, 4096), text, 0.01), ratio, other, policy=policy,
                      scratch=rng.random() < 0.5, layout=rng.choice(["kn", "rows"]), scores=scores)
    if kind == "refresh":
        shapes = [(_log(rng, 64, 8192, rng.choice([8, 8, 1])), _log(rng, 64, 8192, rng.choice([8, 8, 1])))
                  for _ in range(rng.choice([1, 2, 4]))]
        text = ",".join(f"{rng.choice(['col', 'row'])}:{K}x{N}" for K, N in shapes)
        return dict(kind="refresh", projections=text, ratio=max(ratio, 0.02), dtype=rng.choice(["bf16", "bf16", "f32"]),
                    layout=rng.choice(["kn", "rows"]))
    if kind == "select":
        if rng.random() < 0.5:
            return dict(kind="select", batch=1, n=_log(rng, 512, 1 << 23), ratio=ratio, scores=scores)
        n = _log(rng, 256, 12000)
        return dict(kind="select", batch=_log(rng, 2, 4096), n=n, ratio=ratio, scores=scores)
    H = _log(rng, 256, 5120, 8)
    return dict(kind="receive", M=_log(rng, 64, 12608), col=f"{H}x{_log(rng, 48, 1536)}", row=f"{_log(rng, 48, 1536)}x{H}",
                tasks=rng.choice([2, 3, 4, 8]), rank=1, dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]))


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _parse(projections):
    out = []
    for p in projections.split(","):
        kind, shape = p.split(":")
        K, N = shape.split("x")
        out.append((kind, int(K), int(N)))
    return out


def _dtype(case):
    return torch.float32 if case["dtype"] == "f32" else torch.bfloat16


class _Draws:
    """Seeded draws on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, *shape, sigma=1.0, dtype=torch.float32):
        t = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(0.0, sigma, generator=self.g)
        return t if dtype == torch.float32 else t.to(dtype)

    def scores(self, kind, *shape):
        """Importance scores: skewed, flat, or the norms of a weight's slices (around sqrt(length) sigma)."""
        if kind == "lognormal":
            return torch.exp(self.normal(*shape))
        if kind == "uniform":
            return torch.empty(shape, dtype=torch.float32, device="cuda").uniform_(generator=self.g)
        return 1.28 + 0.0141 * self.normal(*shape)

    def subset(self, n, n_keep):
        return torch.randperm(n, generator=self.g, device="cuda")[:n_keep].sort().values.to(torch.int32)


def _mode(kind):
    return zr.DROP_N if kind == "col" else zr.DROP_K


def _layout(case, kind):
    """"rows": the kept list selects rows of the stored shard ([N x K] for column-parallel shards,
    [K x N] for row-parallel ones); "kn": every shard is stored [K x N]."""
    return zr.W_NK if case["layout"] == "rows" and kind == "col" else zr.W_KN


def _prepare_layer(case, d):
    dt, M = _dtype(case), case["M"]
    same = case["policy"] == "same"
    ps = []
    for kind, K, N in _parse(case["projections"]):
        mode, layout = _mode(kind), _layout(case, kind)
        n = N if mode == zr.DROP_N else K
        ratio = case["ratio_col"] if kind == "col" else case["ratio_row"]
        n_keep = zr.keep_count(n, ratio)
        wshape = (N, K) if layout == zr.W_NK else (K, N)
        W = d.normal(*wshape, sigma=wl.W_SIGMA, dtype=dt)
        if case["scores"] == "l2":          # the norm of each prunable slice of the weight
            pruned_axis = 1 if mode == zr.DROP_N and layout == zr.W_KN else 0
            scores = torch.linalg.vector_norm(W.float(), dim=1 - pruned_axis)
        else:
            scores = d.scores(case["scores"], n)
        p = dict(mode=mode, layout=layout, ratio=ratio, W=W, scores=scores,
                 X=d.normal(M, K, dtype=dt), dY=d.normal(M, N, dtype=dt),
                 Y=torch.empty((M, N), dtype=dt, device="cuda"), dX=torch.empty((M, K), dtype=dt, device="cuda"),
                 dW=torch.empty(wshape, dtype=dt, device="cuda"),
                 keep=torch.empty(n, dtype=torch.int32, device="cuda"), drop=torch.empty(n, dtype=torch.int32, device="cuda"),
                 prev_Y=None, prev_dX=None, prev_dW=None, ws=None)
        if same:                            # the previous step's results
            p.update(prev_Y=d.normal(M, N, dtype=dt), prev_dX=d.normal(M, K, dtype=dt), prev_dW=d.normal(*wshape, dtype=dt))
        if case["scratch"]:                 # one buffer per projection: it carries the pruned input to the backward pass
            p["ws"] = torch.empty(zr.workspace_bytes(M, K, N, n_keep, mode, dt), dtype=torch.uint8, device="cuda")
        ps.append(p)
    return dict(kind="layer", ps=ps, policy=POLICY[case["policy"]])


def _prepare_refresh(case, d):
    dt = _dtype(case)
    ps = []
    for kind, K, N in _parse(case["projections"]):
        layout = _layout(case, kind)
        rows, cols = (N, K) if layout == zr.W_NK else (K, N)
        # the scored axis of the stored matrix: a shard stored [N x K] is scored as that matrix, with the other mode
        by_cols = kind == "col" and layout == zr.W_KN
        n = cols if by_cols else rows
        W_prev = d.normal(rows, cols, sigma=wl.W_SIGMA)
        change = 0.2 * wl.W_SIGMA * torch.exp(d.normal(n))          # some slices move much more than others
        W_t = W_prev + d.normal(rows, cols) * (change[None, :] if by_cols else change[:, None])
        mode = zr.DROP_N if by_cols else zr.DROP_K
        ps.append(dict(W_t=W_t.to(dt), W_prev=W_prev.to(dt), mode=mode, prev_scores=torch.exp(d.normal(n)) * 0.003,
                       prev_keep=d.subset(n, zr.keep_count(n, case["ratio"])),
                       scores=torch.empty(n, dtype=torch.float32, device="cuda"),
                       count=torch.empty(1, dtype=torch.int32, device="cuda"),
                       ws=torch.empty(max(16, zr.priority_workspace_bytes(rows, cols, mode)), dtype=torch.uint8, device="cuda")))
    return dict(kind="refresh", ps=ps, theta=0.003)


def _prepare_select(case, d):
    batch, n = case["batch"], case["n"]
    scores = d.scores(case["scores"], n) if batch == 1 else d.scores(case["scores"], batch, n)
    ws = torch.empty(max(16, zr.select_workspace_bytes(n)), dtype=torch.uint8, device="cuda") if batch == 1 else None
    shape = (n,) if batch == 1 else (batch, n)
    return dict(kind="select", scores=scores, ratio=case["ratio"], ws=ws,
                keep=torch.empty(shape, dtype=torch.int32, device="cuda"), drop=torch.empty(shape, dtype=torch.int32, device="cuda"))


def _sizes(text):
    a, b = text.split("x")
    return int(a), int(b)


def _share(case, L):
    return zr.migration_range(case["rank"], 0, case["tasks"], L)


def _prepare_receive(case, d):
    dt, M = _dtype(case), case["M"]
    K, Lc = _sizes(case["col"])         # a column-parallel shard W[K x N] gave away Lc of its columns
    Lr, N = _sizes(case["row"])         # a row-parallel one gave away Lr of its rows
    (cb, ce), (rb, re_) = _share(case, Lc), _share(case, Lr)
    # what the straggler broadcast, and this task's own results that its share is added to
    dY, Wc = d.normal(M, Lc, dtype=dt), d.normal(K, Lc, sigma=wl.W_SIGMA, dtype=dt)
    X, Wr = d.normal(M, Lr, dtype=dt), d.normal(Lr, N, sigma=wl.W_SIGMA, dtype=dt)
    return dict(kind="receive", dY=dY[:, cb:ce], Wc=Wc[:, cb:ce], X=X[:, rb:re_], Wr=Wr[rb:re_, :],
                dX=d.normal(M, K, dtype=dt), Y=d.normal(M, N, dtype=dt))


_PREPARE = {"layer": _prepare_layer, "refresh": _prepare_refresh, "select": _prepare_select, "receive": _prepare_receive}


def prepare(case, seed):
    return _PREPARE[case["kind"]](case, _Draws(seed))


# ---------------------------------------------------------------------------
# One pass
# ---------------------------------------------------------------------------
def _run_layer(s):
    ps, policy = s["ps"], s["policy"]
    keeps, drops = zr.resize_select_multi([p["scores"] for p in ps], [p["ratio"] for p in ps],
                                          keep_idx=[p["keep"] for p in ps], drop_idx=[p["drop"] for p in ps])
    for p, keep in zip(ps, keeps):
        zr.resized_linear_fwd(p["X"], p["W"], keep, p["mode"], policy=policy, prev_Y=p["prev_Y"], Y=p["Y"],
                              workspace=p["ws"], w_layout=p["layout"])
    for p, keep in zip(reversed(ps), reversed(keeps)):
        zr.resized_linear_bwd(p["X"], p["W"], p["dY"], keep, p["mode"], policy=policy, prev_dX=p["prev_dX"],
                              prev_dW=p["prev_dW"], dX=p["dX"], dW=p["dW"], workspace=p["ws"], w_layout=p["layout"],
                              workspace_holds_forward=p["ws"] is not None)
    return dict(keep=keeps, drop=[x for x in drops if x.numel()], Y=[p["Y"] for p in ps], dX=[p["dX"] for p in ps],
                dW=[p["dW"] for p in ps])


def _run_refresh(s):
    for p in s["ps"]:
        zr.priority_scores(p["W_t"], p["W_prev"], p["mode"], prev_scores=p["prev_scores"], prev_keep_idx=p["prev_keep"],
                           scores=p["scores"], workspace=p["ws"])
        zr.count_above(p["scores"], s["theta"], count=p["count"])
    return [(p["scores"], p["count"]) for p in s["ps"]]


def _run_select(s):
    if s["scores"].dim() == 1:
        keep, drop = zr.resize_select_ws(s["scores"], s["ratio"], s["ws"], keep_idx=s["keep"], drop_idx=s["drop"])
    else:
        keep, drop = zr.resize_select(s["scores"], s["ratio"], keep_idx=s["keep"], drop_idx=s["drop"])
    return [keep, drop] if drop.numel() else [keep]


def _run_receive(s):
    zr.migrated_accumulate(s["dX"], s["dY"], s["Wc"], True)
    zr.migrated_accumulate(s["Y"], s["X"], s["Wr"], False)
    return [s["dX"], s["Y"]]


_RUN = {"layer": _run_layer, "refresh": _run_refresh, "select": _run_select, "receive": _run_receive}


def run(state):
    return _RUN[state["kind"]](state)


# ---------------------------------------------------------------------------
# What a pass cannot do without, and how exact it is
# ---------------------------------------------------------------------------
def work(case):
    if case["kind"] == "layer":
        esz, M = (4 if case["dtype"] == "f32" else 2), case["M"]
        nbytes = flops = 0
        for kind, K, N in _parse(case["projections"]):
            n = N if kind == "col" else K
            kept = zr.keep_count(n, case["ratio_col"] if kind == "col" else case["ratio_row"])
            k, nn = (K, kept) if kind == "col" else (kept, N)       # the kept part of the shard
            nbytes += esz * (M * k + k * nn + M * nn)               # X, W, dY: what is kept of them
            nbytes += esz * (M * N + M * K + K * N)                 # Y, dX, dW in their full shape
            if case["policy"] == "same":                            # the dropped parts of the previous results
                nbytes += esz * (M * (N - nn) + M * (K - k) + K * N - k * nn)
            nbytes += 8 * n                                         # scores, and the two index lists
            flops += 6 * M * k * nn
        return dict(bytes=nbytes, flops=flops)
    if case["kind"] == "refresh":
        esz = 4 if case["dtype"] == "f32" else 2
        nbytes = flops = 0
        for kind, K, N in _parse(case["projections"]):
            n = N if kind == "col" else K
            kept = zr.keep_count(n, case["ratio"])                  # the others keep their previous score
            length = K * N // n
            nbytes += 2 * esz * kept * length + 4 * n + 4 * (n - kept) + 4 * kept
            flops += 3 * kept * length
        return dict(bytes=nbytes, flops=flops)
    if case["kind"] == "select":
        return dict(bytes=8 * case["batch"] * case["n"], flops=case["batch"] * case["n"])
    esz, M = (4 if case["dtype"] == "f32" else 2), case["M"]
    (K, Lc), (Lr, N) = _sizes(case["col"]), _sizes(case["row"])
    c, r = (e - b for b, e in (_share(case, Lc), _share(case, Lr)))
    return dict(bytes=esz * (M * c + K * c + 2 * M * K + M * r + r * N + 2 * M * N), flops=2 * M * (K * c + r * N))


def tolerance(case):
    # Each product was compared with the same sum in 64 bits, rounded once to the output type.
    if case["kind"] == "select":
        return "exact"                              # whole numbers only
    if case["kind"] == "refresh":
        # sums of up to 8192 terms in fp32: 6e-8 and at most 2e-7 of a value measured; other
        # orders of summation lose a little more
        return dict(rel=1e-6, max=5e-6)
    if case["dtype"] == "f32":
        # 7e-7 and at most 6e-6 of the rms at a contraction of 2048; it grows with its root
        return dict(rel=5e-6, max=5e-5)
    # bf16 results that fall on the other side of a rounding boundary: 5e-5 over a whole tensor
    # (more over the few hundred elements of the smallest drawn ones), one unit of the last
    # place (2**-7 of the value at most) at an element
    return dict(rel=1e-3, max=0.03)
