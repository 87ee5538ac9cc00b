"""GPU parity of the latency configuration of the MFMA attention kernel (flame_gr_config.latency_mode = 1: several
wavefronts split the keys of a query tile) against the fp64 oracle, for both attention kinds, and its own
determinism and batch independence.  Its sums are grouped differently from the throughput configuration, so the
two are compared to rounding only."""
import re
from pathlib import Path

import numpy as np
import pytest

from paper_2509_22681_amd import workloads as W
from tests.oracle_cache import request_scores, sample_requests
from tests.test_gpu_parity import STRESS, TOL, TOL_HOT, oracle_all, score_err, stress
from tests.test_gpu_softmax import gpu_out, oracle_out, soft

pytestmark = pytest.mark.gpu

# kLatencyWideTiles* and kLatencyShortHistory of csrc/plan.h
LIMITS = dict(re.findall(r"constexpr int kLatency(?:WideTiles|Short)(\w*) = (\d+);", (Path(W.__file__).parent / "csrc" / "plan.h").read_text()))
LIMITS = {k: int(v) for k, v in LIMITS.items()}


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2509_22681_amd import binding
    return binding


@pytest.mark.parametrize("case", list(STRESS))
@pytest.mark.parametrize("kind", ["silu", "softmax"])
def test_latency_mode_against_the_oracle(B, case, kind):
    if kind == "silu":
        wl = stress(dtype="bf16", name=case, hot=True, **STRESS[case])
        want = oracle_all(wl)
    else:
        wl = soft(dtype="bf16", name=case, **STRESS[case])
        want = oracle_out(wl)
    g = gpu_out(B, wl, latency_mode=1)
    base = gpu_out(B, wl)
    assert np.isfinite(g).all()
    err = score_err(g, want)
    print(f"{case} {kind}: latency mode score error {err:.3e}; against the throughput configuration {score_err(g, base):.3e}")
    assert err <= TOL_HOT["bf16"], err
    assert score_err(g, base) <= TOL_HOT["bf16"]


def test_latency_mode_determinism_and_independence(B):
    wl = stress(dtype="bf16", name="S4", hot=True, **STRESS["S4"])
    a = gpu_out(B, wl, latency_mode=1)
    assert np.array_equal(a, gpu_out(B, wl, latency_mode=1))
    co = wl.cand_offsets
    for i in range(wl.n_requests):
        assert np.array_equal(gpu_out(B, wl.subset([i]), latency_mode=1), a[co[i]:co[i + 1]])


@pytest.mark.parametrize("kind", ["silu", "softmax"])
@pytest.mark.parametrize("lengths", ["short", "mixed"])
@pytest.mark.parametrize("d,H", [(128, 2), (64, 2), (320, 5)])
def test_latency_mode_same_bits_on_tiles_of_64_and_128_rows(B, d, H, lengths, kind):
    """A batch that fills the chip runs on query tiles of 128 rows and two wavefronts per row group, a request alone on 64 and four:
    the same partial sums, added in the same order.  Lengths on both sides of the 64-key blocks, of either tile's key tile and of its query tile."""
    edges = [0, 1, 31, 33, 63, 64, 65, 127, 128]
    if lengths == "mixed":
        edges += [129, 191, 193, 255, 256, 257, 300, 383, 385, 511, 513]
    L = edges * 11
    M = [(7 * i) % 131 if i % 5 else [0, 1, 32, 64, 128][i // 5 % 5] for i in range(len(L))]
    M = [max(m, 1) if n == 0 else m for n, m in zip(L, M)]
    wl = W.make_custom(L, M, d=d, H=H, n_layers=2, n_buckets=32, max_rel_dist=256, dtype="bf16", seed=9, emb_std=1.0, rab_std=1.0, bias_amp=0.1,
                       affine_random=True, attn_kind=kind, name=f"tiles{d}")

    def wide(idx):      # the rule of csrc/plan.cpp
        limit = LIMITS["Short"] if max(L[i] for i in idx) <= LIMITS["History"] else LIMITS["Softmax32" if kind == "softmax" and d // H == 32 else ""]
        return sum(-(-L[i] // 64) + -(-M[i] // 64) for i in idx) * H >= limit

    assert wide(range(len(L)))
    whole, co = gpu_out(B, wl, latency_mode=1), wl.cand_offsets
    assert np.isfinite(whole).all()
    for idx in [[i] for i in range(len(edges))] + [list(range(20, 28))]:
        assert not wide(idx)
        part = gpu_out(B, wl.subset(idx), latency_mode=1)
        assert np.array_equal(part, np.concatenate([whole[co[i]:co[i + 1]] for i in idx])), (idx, [L[i] for i in idx], [M[i] for i in idx])


def test_latency_mode_prefill_and_score_choose_tiles_by_their_own_rows(B):
    """Two-stage scoring on a latency handle: the history stage is past the limit of the 128-row tiles, the candidate stage below it, and the
    scores are those of the one-pass forward."""
    import torch
    L, M = [700, 513, 640, 1, 129] * 10, [3, 0, 1, 9, 2] * 10
    wl = W.make_custom(L, M, d=256, H=4, n_layers=2, n_buckets=32, max_rel_dist=1024, dtype="bf16", seed=9, emb_std=1.0, rab_std=1.0, bias_amp=0.1,
                       affine_random=True, name="two_stage_tiles")
    hist, cand = (sum(-(-n // 64) for n in x) * 4 for x in (L, M))
    assert hist >= LIMITS[""] > cand
    h = B.flame_gr_create(B.config_for(wl, latency_mode=1, kv_cache=1))
    try:
        dw, he, ce = B.to_device(wl)
        out = torch.full((int(wl.cand_offsets[-1]),), float("nan"), device="cuda:0")
        B.flame_gr_prefill(h, dw, he, wl.history_offsets, np.array(M, np.int32))
        B.flame_gr_score(h, dw, ce, wl.cand_offsets, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), gpu_out(B, wl, latency_mode=1))
    finally:
        B.flame_gr_destroy(h)


@pytest.mark.parametrize("name", ["uniform", "jagged", "long"])
def test_latency_mode_on_benchmark_workloads(B, name):
    wl = W.make_workload(name)
    g = gpu_out(B, wl, latency_mode=1)
    co = wl.cand_offsets
    worst = 0.0
    for i in sample_requests(wl, name):
        worst = max(worst, score_err(g[co[i]:co[i + 1]], request_scores(wl, i)))
    print(f"{name}, latency mode: max score error {worst:.3e}")
    assert worst <= TOL["bf16"]


def test_latency_mode_is_ignored_by_fp32_handles(B):
    wl = stress(dtype="f32", name="S2", hot=True, **STRESS["S2"])
    assert np.array_equal(gpu_out(B, wl, latency_mode=1), gpu_out(B, wl))
    cfg = B.config_for(wl)
    cfg.latency_mode = 2
    with pytest.raises(B.FlameGRError) as e:
        B.flame_gr_create(cfg)
    assert e.value.code == -1


def test_latency_mode_graph_replay(B):
    """A handle in latency mode can be captured right after its creation (its kernels' launch attributes are set
    at create, not inside the capture) and replays what its eager forward computes."""
    import torch
    wl = stress(dtype="bf16", name="S6", hot=True, **STRESS["S6"])
    want = gpu_out(B, wl, latency_mode=1)
    h = B.flame_gr_create(B.config_for(wl, latency_mode=1))
    try:
        dw, hist, cand = B.to_device(wl)
        out = torch.zeros(int(wl.cand_offsets[-1]), device="cuda:0")
        B.flame_gr_capture(h, dw, hist, wl.history_offsets, cand, wl.cand_offsets, out)
        for _ in range(2):
            out.zero_()
            B.flame_gr_replay(h)
            torch.cuda.synchronize()
            assert np.array_equal(out.cpu().numpy(), want)
    finally:
        B.flame_gr_destroy(h)
