"""Attention weights on every route of the SiLU, at the edges of their ranges.  Embeddings are zero, so Q = K = 0, V is the same for all keys, and the logits of a row are the
bias of its distances: O_r = V * sum over its keys of silu(bias[r - c])."""
import numpy as np
import pytest

from paper_2509_22681_amd import workloads as W

pytestmark = pytest.mark.gpu

H16 = 2.0 ** -11      # half an ulp of fp16, relative
EDGES = [0.01, 0.12, 0.25, 0.25 + 2.0 ** -14, 0.2502, 0.5, 1.0, 1.002, 1.5, 2.0, 2.01, 3.0, 4.0, 4.01, 9.0]
LENGTHS = dict(L=[300, 70, 1], M=[40, 5, 3])


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2509_22681_amd import binding
    return binding


def silu(x):
    return x / (1.0 + np.exp(-x))


def weight_error(x, top):
    """Largest error of a weight at logit x in a block whose largest |logit| is top: that of the approximation (csrc/attn_mfma.hip), four roundings of its fp16 arithmetic on the
    term beside the logit, and the rounding of the weight."""
    t = (x / 2) ** 2
    if top <= 4.0 + 2.0 ** -8:
        # the short polynomial's bracket is off by 3.4e-3 of itself where that is most, at the smallest logits (a1 against 1/4); the long one's weight by 5.4e-4
        approx, term = np.where(top <= 2.002, 3.5e-3 * t, 5.4e-4), np.minimum(t, np.abs(x) / 2)
    else:
        approx, term = 0.0, 0.0
    return approx + 4 * H16 * term + H16 * np.abs(silu(x)) + 2.0 ** -25


def outputs(B, wl, latency):
    import torch
    h = B.flame_gr_create(B.config_for(wl, latency_mode=latency))
    try:
        dw, hist, cand = B.to_device(wl)
        B.flame_gr_debug_capture(h, 0)
        scores = torch.zeros(int(wl.cand_offsets[-1]), device="cuda:0")
        B.flame_gr_forward(h, dw, hist, wl.history_offsets, cand, wl.cand_offsets, scores)
        torch.cuda.synchronize()
        n = int(wl.history_offsets[-1] + wl.cand_offsets[-1])
        return B.flame_gr_debug_stage(h, 1, n, wl.cfg.d_model), B.flame_gr_debug_stage(h, 4, n, wl.cfg.d_model)
    finally:
        B.flame_gr_destroy(h)


def workload(d, H, bias):
    """One layer, bias[distance] for all heads, V = silu(1)."""
    wl = W.make_custom(LENGTHS["L"], LENGTHS["M"], d=d, H=H, n_layers=1, n_buckets=1024, max_rel_dist=512, dtype="bf16", seed=1, emb_std=0.0, name=f"routes{d}_{H}")
    wl.weights["rab"] = np.broadcast_to(np.asarray(bias, np.float32)[None, None], (1, H, 1024)).copy()
    b1 = np.zeros((1, 4 * d), np.float32)
    b1[:, d:2 * d] = 1.0
    wl.weights["b1"] = b1
    return wl


def check(B, d, H, bias, latency):
    wl = workload(d, H, bias)
    V, O = outputs(B, wl, latency)
    v, bias = float(V[0, 0]), np.asarray(bias, np.float64)
    assert abs(v - silu(1.0)) <= 2 * H16 and (V == V[0, 0]).all()
    # the blocks: 32 rows of a request's history (or candidates) x 64 keys, of which the positions past a row's horizon hold the bias of distance 0
    for L, M, h0, c0 in zip(LENGTHS["L"], LENGTHS["M"], wl.history_offsets, wl.cand_offsets):
        base = int(h0 + c0)           # rows of a request follow one another: history, then candidates
        for q0 in list(range(0, L, 32)) + [L]:
            rows = range(q0, min(q0 + 32, L)) if q0 < L else range(L, L + M)
            pos = np.array([min(r, L) for r in rows])
            want, bound = np.zeros(len(pos)), np.zeros(len(pos))
            last = L if q0 == L else min(q0 + 32, L)
            for k0 in range(0, last, 64):
                keys = np.arange(k0, k0 + 64)
                # (a tile's window also holds rows and keys past the ends: what counts as the block's largest logit is taken over all that it may hold)
                span = np.clip(np.arange(pos[0] - k0 - 64, pos[0] + 32 - k0 + 1), 0, 511)
                dist = np.clip(pos[:, None] - keys[None], 0, 511)
                x = bias[dist]
                seen = keys[None] < (L if q0 == L else pos[:, None] + 1)
                e = np.maximum(weight_error(x, np.abs(x).max()), weight_error(x, np.abs(bias[span]).max()))
                want += (silu(x) * seen).sum(1)
                bound += (e * seen).sum(1)
            if q0 == L:
                want += silu(bias[0])
                bound += weight_error(bias[0], 100.0)
            got = O[base + np.array(list(rows))]
            err = np.abs(got - v * want[:, None]).max(1)
            # the sums are in fp32, the output is rounded to fp16 once
            assert (err <= v * bound + (H16 + 1e-6) * np.abs(v * want) + 2.0 ** -24).all(), (L, q0, float((err / (v * bound)).max()))


@pytest.mark.parametrize("latency", [0, 1])
@pytest.mark.parametrize("d,H", [(64, 1), (64, 2)])
def test_weights_at_the_edges_of_the_routes(B, d, H, latency):
    for x in EDGES:
        for sign in (1.0, -1.0):
            check(B, d, H, np.full(1024, sign * x), latency)


@pytest.mark.parametrize("latency", [0, 1])
@pytest.mark.parametrize("d,H", [(64, 1), (64, 2)])
def test_blocks_of_different_routes_follow_one_another(B, d, H, latency):
    rng = np.random.default_rng(3)
    for amplitudes in ([0.2, 3.0, 0.2, 0.9, 0.1], [9.0, 0.2, 1.8, 0.05, 0.25], [0.05, 0.05, 0.9, 0.05, 3.9]):
        bias = np.zeros(1024)
        for i, a in enumerate(amplitudes):
            bias[64 * i:64 * (i + 1)] = a * rng.uniform(-1, 1, 64)
        check(B, d, H, bias, latency)
