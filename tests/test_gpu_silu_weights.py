"""Attention weights of small logits, bit for bit those of the polynomial that covers |x| <= 2 (csrc/attn_mfma.hip): no shorter form, which would be further off somewhere in its range,
takes its place below.  Embeddings are zero, so Q = K = 0 and the logits are the bias; the first history row has one key: O = V * weight."""
import re

import numpy as np
import pytest

from paper_2509_22681_amd import build as build_mod
from paper_2509_22681_amd import workloads as W

pytestmark = pytest.mark.gpu


def polynomial(x):
    """silu(x) = s + t (c1 + c3 t + c5 t^2), s = x / 2, t = s^2: t and the bracket in fp16, the last step in fp32, rounded to fp16."""
    with open(f"{build_mod.CSRC}/device_common.h") as f:
        a1, a3, a5 = (np.float32(v) for v in re.search(r"kPolyA1 = (\S+)f, kPolyA3 = (\S+)f, kPolyA5 = (\S+)f;", f.read()).groups())
    c1, c3, c5 = (np.float64(np.float16(k * a)) for k, a in ((np.float32(4), a1), (np.float32(16), a3), (np.float32(64), a5)))
    s = (np.asarray(x, np.float32) / np.float32(2)).astype(np.float64)
    y = s.astype(np.float16).astype(np.float64)
    t = (y * y).astype(np.float16).astype(np.float64)
    r = (c5 * t + c3).astype(np.float16).astype(np.float64)
    r = (r * t + c1).astype(np.float16).astype(np.float64)
    return (t * r + s).astype(np.float32).astype(np.float16)


@pytest.mark.parametrize("latency", [0, 1])
@pytest.mark.parametrize("H", [8, 16])
def test_small_logits_have_the_weights_of_the_polynomial(H, latency):
    import torch
    from paper_2509_22681_amd import binding as B
    d, rng = 512, np.random.default_rng(H)
    logits = rng.permutation(np.concatenate([s * np.linspace(0.01, 1.99, 16 * H) for s in (1, -1)])).astype(np.float32).reshape(-1, H)
    wl = W.make_custom([300, 70, 1], [40, 5, 3], d=d, H=H, n_layers=1, n_buckets=64, max_rel_dist=512, dtype="bf16", seed=1, emb_std=0.0, name="weights")
    wl.weights["b1"] = np.zeros((1, 4 * d), np.float32)
    wl.weights["b1"][:, d:2 * d] = 1.0
    h = B.flame_gr_create(B.config_for(wl, latency_mode=latency))
    try:
        B.flame_gr_debug_capture(h, 0)
        scores = torch.zeros(int(wl.cand_offsets[-1]), device="cuda:0")
        for x in logits:
            wl.weights["rab"] = np.ascontiguousarray(np.broadcast_to(x[None, :, None], (1, H, 64)))
            dw, hist, cand = B.to_device(wl)
            B.flame_gr_forward(h, dw, hist, wl.history_offsets, cand, wl.cand_offsets, scores)
            torch.cuda.synchronize()
            n = int(wl.history_offsets[-1] + wl.cand_offsets[-1])
            V, O = (B.flame_gr_debug_stage(h, stage, n, d) for stage in (1, 4))
            assert (V == V[0, 0]).all()
            want = (np.float32(V[0, 0]) * polynomial(x).astype(np.float32)).astype(np.float16).astype(np.float32)
            for first in (wl.history_offsets + wl.cand_offsets)[:-1]:
                got = O[first].reshape(H, -1)
                assert (got == want[:, None]).all(), (x[(got != want[:, None]).any(1)], got[:, 0], want)
    finally:
        B.flame_gr_destroy(h)
