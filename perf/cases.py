"""The forward passes whose speed is measured: what a user of the library has it do, over the range they do it.

A case is a model shape, a set of request lengths and the way the library is called:

  batch    one flame_gr_forward over a jagged batch of requests, inputs on the device;
  request  one user's request per call, on an executor in latency mode with frozen weights;
  replay   one user's request of a fixed shape, as a replay of its captured graph;
  session  flame_gr_prefill of a batch of users, then candidate micro-batches with flame_gr_score;
  climber  the paper's own model: block stacks over slices of the history (softmax attention), fusion and task head;
  serve    requests from host memory through the orchestrator's jagged micro-batches, scores back in host memory.

Values have the distributions of the benchmark workloads: embeddings N(0, 0.1^2), Xavier-uniform projections, relative-position
bias N(0, 0.02^2), temperatures U[0.5, 2].  Lengths follow from the case alone, values from the seed.
"""
import math

import numpy as np
import torch

from paper_2509_22681_amd import binding as B
from paper_2509_22681_amd import workloads as W

DEVICE = "cuda:0"


def _model(d, heads, layers, buckets=128, dtype="bf16", attn="silu"):
    return dict(d=d, heads=heads, layers=layers, buckets=buckets, dtype=dtype, attn=attn)


def _lengths(requests, hist_lo, hist_hi, cand_lo, cand_hi, zipf=0.0, draw=0):
    """Histories uniform in [hist_lo, hist_hi]; candidates uniform in [cand_lo, cand_hi], or Zipf(zipf) clipped to it."""
    return dict(requests=requests, hist_lo=hist_lo, hist_hi=hist_hi, cand_lo=cand_lo, cand_hi=cand_hi, zipf=zipf, draw=draw)


def listed():
    production = _model(512, 8, 16)
    return [
        # the smallest call: one small fp32 request, bound by launches and latency
        dict(name="tiny_f32", kind="batch", static=0, **_model(64, 2, 2, dtype="f32"), **_lengths(1, 64, 64, 16, 16)),
        # the fp32 element type on ordinary traffic: models kept in fp32, or of a width the matrix kernels do not cover
        dict(name="base_f32", kind="batch", static=0, **_model(256, 4, 4, dtype="f32"), **_lengths(32, 512, 512, 128, 128)),
        # ordinary batches of equal requests on a small model
        dict(name="uniform", kind="batch", static=0, **_model(256, 4, 4), **_lengths(32, 512, 512, 128, 128)),
        # ordinary ragged batches
        dict(name="jagged", kind="batch", static=0, **_model(512, 8, 8), **_lengths(64, 256, 2048, 16, 1024, 1.2)),
        # long histories: attention decides
        dict(name="long", kind="batch", static=0, **_model(512, 8, 8, buckets=512), **_lengths(16, 8192, 8192, 512, 512)),
        # the largest call: a full production batch
        dict(name="production", kind="batch", static=0, **production, **_lengths(128, 1024, 4096, 32, 2000, 1.1)),
        # the same traffic on softmax attention with temperature
        dict(name="softmax", kind="batch", static=0, **dict(production, attn="softmax"), **_lengths(32, 1024, 4096, 32, 2000, 1.1)),
        # a request on its own, whose latency the user of an online service sees
        dict(name="request", kind="request", **production, **_lengths(1, 2573, 2573, 217, 217)),
        # the same with the explicit-shape executor: the forward of a fixed shape as one graph
        dict(name="replay", kind="replay", **production, **_lengths(1, 1024, 1024, 256, 256)),
        # users whose history is cached while several candidate micro-batches arrive for them
        dict(name="session", kind="session", rounds=2, **production, **_lengths(32, 1024, 4096, 32, 2000, 1.1)),
        # the paper's own model at its base scenario, two block stacks, many users per pass
        dict(name="climber", kind="climber", blocks=2, expert=256, tasks=2, **_model(192, 3, 12, attn="softmax"), **_lengths(64, 512, 512, 128, 128)),
        # requests arriving in host memory, gathered into micro-batches of up to eight
        dict(name="serve", kind="serve", batch=8, **production, **_lengths(16, 1024, 4096, 32, 2000, 1.1)),
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _traffic(rng, requests, hist_lo, hist_hi, cand_hi):
    """Requests of one kind: a longest history and a largest candidate count, most requests below them."""
    top, most = _log_int(rng, hist_lo, hist_hi), _log_int(rng, 16, cand_hi)
    return _lengths(requests, max(1, int(top * rng.choice([0.25, 0.5, 1.0]))), top, min(most, rng.choice([1, 16, 32])), most,
                    rng.choice([0.0, 1.1, 1.2]), rng.randrange(1 << 16))


def draw(rng):
    kind = rng.choice(["f32", "batch", "batch", "batch", "request", "request", "replay", "session", "climber", "serve"])
    while True:
        if kind == "f32":
            d, heads = rng.choice([(64, 2), (96, 2), (128, 2), (192, 3), (256, 4), (256, 8)])
            c = dict(kind="batch", static=rng.randrange(2), **_model(d, heads, rng.choice([1, 2, 4]), dtype="f32", attn=rng.choice(["silu", "silu", "softmax"])),
                     **_traffic(rng, _log_int(rng, 1, 32), 32, 1024, 256))
        elif kind == "batch":
            d, heads = rng.choice([(64, 2), (128, 2), (128, 4), (192, 3), (256, 4), (256, 8), (384, 6), (512, 8), (512, 8), (512, 16)])
            c = dict(kind="batch", static=rng.randrange(2), **_model(d, heads, rng.choice([2, 4, 8, 16]), rng.choice([128, 512]), attn=rng.choice(["silu", "silu", "softmax"])),
                     **_traffic(rng, _log_int(rng, 1, 128), 128, 8192, 2000))
        elif kind in ("request", "replay"):
            d, heads, layers = rng.choice([(256, 4, 4), (512, 8, 8), (512, 8, 16)])
            hist, cand = _log_int(rng, 64, 4096), _log_int(rng, 16, 2000)
            c = dict(kind=kind, **_model(d, heads, layers, attn=rng.choice(["silu", "silu", "softmax"])), **_lengths(1, hist, hist, cand, cand))
        elif kind == "session":
            c = dict(kind="session", rounds=rng.choice([1, 2, 4]), **_model(512, 8, rng.choice([8, 16])), **_traffic(rng, _log_int(rng, 1, 48), 256, 4096, 2000))
        elif kind == "climber":
            hist, cand = _log_int(rng, 256, 1024), _log_int(rng, 64, 512)
            c = dict(kind="climber", blocks=2, expert=256, tasks=2, **_model(192, 3, 12, attn="softmax"), **_lengths(_log_int(rng, 1, 64), hist, hist, cand, cand))
        else:
            c = dict(kind="serve", batch=rng.choice([4, 8]), **_model(512, 8, rng.choice([8, 16])), **_traffic(rng, _log_int(rng, 1, 24), 256, 4096, 2000))
        # nothing larger than the production batch; fp32 within what its vector and matrix rates turn round in comparable time
        if work(c)["flops"] <= (1e11 if c["dtype"] == "f32" else 4.6e13):
            return c


# ----------------------------------------------------------------------------------------------
# lengths and work
# ----------------------------------------------------------------------------------------------
def _counts(case):
    """History lengths and candidate counts of the requests."""
    rng = np.random.default_rng(case["draw"])
    n = case["requests"]
    L = rng.integers(case["hist_lo"], case["hist_hi"] + 1, n)
    if case["zipf"]:
        M = np.clip(rng.zipf(case["zipf"], n), case["cand_lo"], case["cand_hi"])
    else:
        M = rng.integers(case["cand_lo"], case["cand_hi"] + 1, n)
    return L.astype(np.int64), M.astype(np.int64)


def _config(case):
    return W.GRConfig(case["layers"], case["d"], case["heads"], case["buckets"], max(W._pow2_above(case["hist_hi"]), case["buckets"] // 2), case["dtype"],
                      attn_kind=case["attn"])


def _slices(L, blocks):
    """History slices of the block stacks, one row of lengths per stack."""
    return [np.array([np.subtract(*reversed(B.flame_climber_block_range(int(n), blocks, b))) for n in L], np.int64) for b in range(blocks)]


def work(case):
    cfg, (L, M) = _config(case), _counts(case)
    d, layers = cfg.d_model, cfg.n_layers
    size = 4 if cfg.dtype == "f32" else 2
    weights = layers * 5 * d * d * size
    if case["kind"] == "climber":
        nb, E, T = case["blocks"], case["expert"], case["tasks"]
        rows = int(M.sum())
        parts = _slices(L, nb)
        flops = sum(W.algorithmic_flops(cfg, s, M) - 2.0 * rows * d for s in parts) + 2.0 * rows * (nb * nb * d * d + T * E * d)
        return {"bytes": float(nb * weights + (int(L.sum()) + nb * rows) * d * size + (nb + 1) * rows * d * 4 + rows * T * 4), "flops": flops}
    flops = W.algorithmic_flops(cfg, L, M)
    rows, rounds = int(M.sum()), case.get("rounds", 1)
    if rounds > 1:
        # the history part once, the candidate part in every round
        nothing = np.zeros_like(M)
        flops += (rounds - 1) * (flops - W.algorithmic_flops(cfg, L, nothing))
    return {"bytes": float(weights + (int(L.sum()) + rounds * rows) * d * size + rounds * rows * 4), "flops": float(flops)}


# Measured against the oracle in 64 bits: the fp16 matrix path is off by up to 6e-3 (2-norm over a production request's scores), its
# largest single score by 3e-2 of their root mean square; the fp32 path by 8e-7.
def tolerance(case):
    if case["dtype"] == "f32":
        return {"rel": 5e-6, "max": 5e-5}
    return {"rel": 2e-2, "max": 1.5e-1}


# ----------------------------------------------------------------------------------------------
# what a user's program holds before the call
# ----------------------------------------------------------------------------------------------
class _Handles:
    """Library handles that live as long as the state they belong to."""

    def __init__(self):
        self.gr, self.dso = [], []

    def __del__(self):
        torch.cuda.synchronize()
        for h in self.dso:
            B.flame_dso_destroy(h)
        for h in self.gr:
            B.flame_gr_destroy(h)


def _offsets(n):
    return np.concatenate([[0], np.cumsum(n)]).astype(np.int32)


def _weights(cfg, gen):
    d, H, layers = cfg.d_model, cfg.n_heads, cfg.n_layers
    dt = torch.float32 if cfg.dtype == "f32" else torch.bfloat16

    def uniform(shape, a):
        return ((2 * torch.rand(shape, generator=gen, device=DEVICE) - 1) * a).to(dt)

    a = math.sqrt(3.0 / d)
    w = dict(w1=uniform((layers, 4 * d, d), a), w2=uniform((layers, d, d), a), w_s=uniform((d,), math.sqrt(6.0 / (d + 1))),
             b1=torch.zeros(layers, 4 * d, dtype=dt, device=DEVICE), b2=torch.zeros(layers, d, dtype=dt, device=DEVICE),
             ln_g=torch.ones(layers, d, dtype=dt, device=DEVICE), ln_b=torch.zeros(layers, d, dtype=dt, device=DEVICE),
             rab=0.02 * torch.randn(layers, H, cfg.n_buckets, generator=gen, device=DEVICE), b_s=0.0)
    if cfg.attn_kind == "softmax":
        w["temperature"] = 0.5 + 1.5 * torch.rand(layers, H, generator=gen, device=DEVICE)
    return w


def _embeddings(cfg, rows, gen):
    dt = torch.float32 if cfg.dtype == "f32" else torch.bfloat16
    return (0.1 * torch.randn(int(rows), cfg.d_model, generator=gen, device=DEVICE)).to(dt)


def _make_config(cfg, L, M, **options):
    return B.make_config(cfg.n_layers, cfg.d_model, cfg.n_heads, cfg.n_buckets, cfg.max_rel_dist, cfg.dtype, ln_eps=cfg.ln_eps, attn_scale=cfg.attn_scale,
                         max_requests=len(L), max_total_tokens=int(L.sum() + M.sum()), attn_kind=cfg.attn_kind, **options)


def prepare(case, seed):
    gen = torch.Generator(device=DEVICE)
    gen.manual_seed(int(seed) * 2654435761 % (1 << 62) + 1)
    cfg, (L, M) = _config(case), _counts(case)
    kind, handles = case["kind"], _Handles()
    state = dict(kind=kind, handles=handles, history_offsets=_offsets(L), cand_offsets=_offsets(M))
    if kind == "climber":
        return _prepare_climber(case, cfg, L, M, gen, state)
    state["held"] = _weights(cfg, gen)                 # keeps the device arrays alive
    state["weights"] = B.pack_weights(state["held"])
    if kind == "serve":
        requests = []
        for n, m in zip(L, M):
            history, cand = _embeddings(cfg, n, gen), _embeddings(cfg, m, gen)
            requests.append(tuple(np.ascontiguousarray(t.view(torch.int16).cpu().numpy()).view(np.uint16) for t in (history, cand)))
        state["requests"] = requests
        state["scores"] = [np.zeros(int(m), np.float32) for m in M]
        model = B.make_config(cfg.n_layers, cfg.d_model, cfg.n_heads, cfg.n_buckets, cfg.max_rel_dist, cfg.dtype, ln_eps=cfg.ln_eps, attn_scale=cfg.attn_scale)
        torch.cuda.synchronize()
        handles.dso.append(B.flame_dso_create(model, state["weights"], case["hist_hi"], [case["cand_hi"]], 2, explicit_shapes=2, max_batch=case["batch"]))
        return state
    state["history"], state["cand"] = _embeddings(cfg, L.sum(), gen), _embeddings(cfg, M.sum(), gen)
    state["scores"] = torch.zeros(int(M.sum()), device=DEVICE)
    options = {"batch": dict(weights_static=case.get("static", 0)), "request": dict(latency_mode=1, weights_static=1), "replay": dict(weights_static=1),
               "session": dict(kv_cache=1)}[kind]
    handles.gr.append(B.flame_gr_create(_make_config(cfg, L, M, **options)))
    if kind == "session":
        state["capacity"] = M.astype(np.int32)
        state["rounds"] = [(_embeddings(cfg, M.sum(), gen), torch.zeros(int(M.sum()), device=DEVICE)) for _ in range(case["rounds"])]
    if kind == "replay":
        state["stream"] = torch.cuda.Stream()
        torch.cuda.synchronize()
        B.flame_gr_capture(handles.gr[0], state["weights"], state["history"], state["history_offsets"], state["cand"], state["cand_offsets"], state["scores"],
                           record_stream=state["stream"])
    return state


def _prepare_climber(case, cfg, L, M, gen, state):
    nb, d, E, T = case["blocks"], cfg.d_model, case["expert"], case["tasks"]
    rows = int(M.sum())

    def normal(*shape, scale):
        return scale * torch.randn(*shape, generator=gen, device=DEVICE)

    cand = _embeddings(cfg, rows, gen)
    state["stacks"] = []
    for n in _slices(L, nb):
        held = _weights(cfg, gen)
        state["handles"].gr.append(B.flame_gr_create(_make_config(cfg, n, M)))
        state["stacks"].append(dict(held=held, weights=B.pack_weights(held), history=_embeddings(cfg, n.sum(), gen), offsets=_offsets(n), cand=cand))
    state["hidden"] = [torch.zeros(rows, d, device=DEVICE) for _ in range(nb)]
    state["head"] = dict(wg=normal(nb, d, nb * d, scale=1 / math.sqrt(nb * d)), cg=torch.zeros(nb, d, device=DEVICE), a_w=normal(T, E, d, scale=1 / math.sqrt(d)),
                         a_b=torch.zeros(T, E, device=DEVICE), v=normal(T, E, scale=1 / math.sqrt(E)), c=torch.zeros(T, device=DEVICE))
    state["fused"], state["probs"] = torch.zeros(rows, d, device=DEVICE), torch.zeros(rows, T, device=DEVICE)
    return state


# ----------------------------------------------------------------------------------------------
# one pass
# ----------------------------------------------------------------------------------------------
def run(state):
    kind = state["kind"]
    if kind == "serve":
        dso = state["handles"].dso[0]
        for (history, cand), scores in zip(state["requests"], state["scores"]):
            B.flame_dso_submit_jagged(dso, history, cand, scores)
        B.flame_dso_drain(dso)
        return np.concatenate(state["scores"])
    if kind == "climber":
        for handle, s, hidden in zip(state["handles"].gr, state["stacks"], state["hidden"]):
            B.flame_gr_forward_hidden(handle, s["weights"], s["history"], s["offsets"], s["cand"], state["cand_offsets"], hidden)
        B.flame_climber_head(state["head"], state["hidden"], state["fused"], state["probs"])
        return dict(hidden=state["hidden"], fused=state["fused"], probs=state["probs"])
    handle = state["handles"].gr[0]
    if kind == "session":
        B.flame_gr_prefill(handle, state["weights"], state["history"], state["history_offsets"], state["capacity"])
        for cand, scores in state["rounds"]:
            B.flame_gr_score(handle, state["weights"], cand, state["cand_offsets"], scores)
        return [scores for _, scores in state["rounds"]]
    if kind == "replay":
        state["stream"].wait_stream(torch.cuda.current_stream())
        B.flame_gr_replay(handle, stream=state["stream"])
        torch.cuda.current_stream().wait_stream(state["stream"])
        return state["scores"]
    B.flame_gr_forward(handle, state["weights"], state["history"], state["history_offsets"], state["cand"], state["cand_offsets"], state["scores"])
    return state["scores"]
