"""Attention of small launches: four wavefronts make the weights of a row group's keys and one per feature block adds the values up in key order, as a
wavefront alone does in larger launches.  The same bits either way: few requests (small launches) against the batch of all of them (large)."""
import numpy as np
import pytest

from paper_2509_22681_amd import workloads as W
from tests.test_gpu_parity import TOL_HOT, oracle_all, score_err
from tests.test_gpu_softmax import gpu_out
from tests.test_routes import KEY_ORDERED, key_ordered

pytestmark = pytest.mark.gpu

LIMIT, HISTORY = KEY_ORDERED["Workgroups"], KEY_ORDERED["History"]

# lengths on both sides of the 32-row groups, the 64-key blocks, the 64-row tiles, the 128-row items and the 256-key tiles
L = [HISTORY + n for n in (0, 1, 31, 33, 63, 64, 65, 96, 127, 128, 129, 191, 255, 256, 257, 639, 641)] + [0, 1, 33, 64, 127, 129, 256, HISTORY - 1]
M = [1, 0, 3, 32, 33, 64, 65, 5, 128, 129, 96, 0, 31, 7, 64, 130, 1, 200, 63, 2, 127, 17, 70, 0, 9]
SMALL = [[i] for i in range(17)] + [[0, 17], [3, 18, 19], [12, 20], [21, 5], [9, 22]]     # short histories come along with a long one


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "these tests need the MI355X"
    from paper_2509_22681_amd import binding
    return binding


def routed(L, M, H):
    """Whether the launch of all tiles of these requests is key-ordered, by the library's own rule."""
    cand = sum(-(-m // 128) for m in M)
    items = sum(-(-l // 128) for l in L) + cand
    return key_ordered(items * H, items, cand, max(L))


@pytest.mark.parametrize("amp", [0.1, 1.0])      # weights from the short polynomial mostly, and from all three routes
@pytest.mark.parametrize("d,H", [(64, 1), (64, 2), (128, 2), (512, 8), (320, 10)])
def test_small_launches_give_the_same_bits(B, d, H, amp):
    import torch
    n = -(-(2 * LIMIT) // (H * sum(-(-l // 128) + -(-m // 128) for l, m in zip(L, M))))
    wl = W.make_custom(L * n, M * n, d=d, H=H, n_layers=2, n_buckets=32, max_rel_dist=256, dtype="bf16", seed=9, emb_std=amp, rab_std=1.0, bias_amp=0.1,
                       affine_random=True, name=f"small{d}")
    whole, co = gpu_out(B, wl), wl.cand_offsets
    assert np.isfinite(whole).all() and not routed(L * n, M * n, H)
    for idx in SMALL:
        assert routed([L[i] for i in idx], [M[i] for i in idx], H)
        part = gpu_out(B, wl.subset(idx))
        assert np.array_equal(part, np.concatenate([whole[co[i]:co[i + 1]] for i in idx])), [(L[i], M[i]) for i in idx]
    if d == 64 and amp < 1:      # (the batch runs the one-wavefront kernel alone, whose hot cases are held to the oracle where their bar is set; here the bits count)
        assert score_err(whole, oracle_all(wl)) <= TOL_HOT["bf16"]
    # two-stage: a small history pass, then candidates against it
    sub = wl.subset([15])
    h = B.flame_gr_create(B.config_for(sub, kv_cache=1))
    try:
        dw, he, ce = B.to_device(sub)
        out = torch.full((M[15],), float("nan"), device="cuda:0")
        B.flame_gr_prefill(h, dw, he, sub.history_offsets, np.array([M[15]], np.int32))
        B.flame_gr_score(h, dw, ce, sub.cand_offsets, out)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), whole[co[15]:co[16]])
    finally:
        B.flame_gr_destroy(h)


def sides():
    """Batches on both sides of each limit: (L, M, key-ordered).  One long request, and others that fill the launch."""
    k = KEY_ORDERED
    out = [([k["History"] - 1], [40], False), ([k["History"]], [40], True)]
    for longest, limit in ((k["LongHistory"] - 1, k["Workgroups"]), (k["LongHistory"], k["LongWorkgroups"]), (k["LongerHistory"] - 1, k["LongWorkgroups"]),
                           (k["LongerHistory"], k["LongerWorkgroups"])):
        for tiles in (limit, limit + 1):
            left = tiles - -(-longest // 128) - 1
            out.append(([longest] + [100] * left, [5] + [0] * left, tiles == limit))
    for tiles in (k["Workgroups"], k["Workgroups"] + 1):            # candidate tiles prevail: the lowest limit, whatever the history
        out.append(([k["LongerHistory"]], [128 * (tiles - k["LongerHistory"] // 128) - 60], tiles == k["Workgroups"]))
    return out


@pytest.mark.parametrize("case", range(len(sides())))
def test_both_sides_of_each_limit_give_the_same_bits(B, case):
    L, M, want = sides()[case]
    assert routed(L, M, 1) == want
    wl = W.make_custom(L, M, d=64, H=1, n_layers=2, n_buckets=32, max_rel_dist=2048, dtype="bf16", seed=9, emb_std=1.0, rab_std=1.0, bias_amp=0.1,
                       affine_random=True, name="sides")
    n = 1 + KEY_ORDERED["LongerWorkgroups"] // sum(-(-a // 128) + -(-b // 128) for a, b in zip(L, M))
    assert not routed(L * n, M * n, 1)
    out = gpu_out(B, wl)
    assert np.isfinite(out).all() and np.array_equal(out, gpu_out(B, wl.subset(list(range(len(L))) * n))[:len(out)])
