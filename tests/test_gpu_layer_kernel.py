"""The kernel that makes a layer's output projection and the next layer's projections in one launch, against the two kernels that run
where a handle's planes are to be looked at: the same instructions in the same order, so the same bits, in each pass that can take it,
from two row blocks to sizes that stream (which of them ran is read from the launches that a profiled handle counts); and against the fp64 oracle at the hot bar."""
import numpy as np
import pytest

import oracle
from paper_2509_22681_amd import workloads as W
from tests.test_gpu_parity import TOL_HOT, score_err

pytestmark = pytest.mark.gpu

# (width, heads, 64-row blocks of the batch, an even number): the smallest, sizes between, and both sides of the 16 MB of a plane past which the two kernels stream
SIZES = [(128, 2, 2), (192, 3, 2), (256, 4, 2), (128, 4, 66), (192, 6, 132), (256, 8, 310)]
for width, heads in ((128, 2), (192, 3), (256, 4)):
    last = (16 << 20) // (64 * 2 * width)
    SIZES += [(width, heads, n) for n in (last // 2 * 2, last // 2 * 2 + 2)]
SIZES += [(256, 4, 600), (192, 3, 800), (128, 2, 1300)]


def batch(blocks):
    """Ragged lengths, one block each side: whole blocks, one row, and all remainders between."""
    n = blocks // 2
    return [[64, 1, 63, 17, 33, 40][i % 6] for i in range(n)], [[1, 64, 32, 5, 49][i % 5] for i in range(n)]


@pytest.mark.parametrize("kind", ["silu", "softmax"])
@pytest.mark.parametrize("d,H,blocks", SIZES)
def test_one_launch_per_layer_gives_the_same_bits(d, H, blocks, kind):
    import torch
    from paper_2509_22681_amd import binding as B
    L, M = batch(blocks)
    wl = W.make_custom(L, M, d=d, H=H, n_layers=3, n_buckets=16, max_rel_dist=128, dtype="bf16", seed=11, emb_std=1.0, rab_std=1.0,
                       bias_amp=0.1, affine_random=True, attn_kind=kind, name="layer")
    dw, hist, cand = B.to_device(wl)
    n = int(wl.cand_offsets[-1])

    def scores(two_stage, captured, n_streams=0, launches=None):
        h = B.flame_gr_create(B.config_for(wl, n_streams=n_streams, kv_cache=int(two_stage)))
        try:
            if captured:
                B.flame_gr_debug_capture(h, 0)
            out = torch.full((n,), float("nan"), device="cuda:0")
            if two_stage:
                B.flame_gr_prefill(h, dw, hist, wl.history_offsets, np.asarray(M, np.int32))
                B.flame_gr_score(h, dw, cand, wl.cand_offsets, out)
            else:
                if launches is not None:
                    B.flame_gr_debug_profile(h, True)
                B.flame_gr_forward(h, dw, hist, wl.history_offsets, cand, wl.cand_offsets, out)
                if launches is not None:
                    launches.update({k: n for k, (_, n) in B.flame_gr_debug_profile_read(h).items()})
            torch.cuda.synchronize()
            return out.cpu().numpy()
        finally:
            B.flame_gr_destroy(h)

    two, one = {}, {}
    want = scores(False, True, launches=two)
    assert np.isfinite(want).all()
    assert np.array_equal(scores(False, False, launches=one), want)
    assert two["uvqk"] == 3 and one["uvqk"] == 1          # (the projections of the first layer)
    assert np.array_equal(scores(False, False, n_streams=2), want)
    assert np.array_equal(scores(True, False), want) and np.array_equal(scores(True, True), want)
    if blocks <= 160:
        full = oracle.forward(wl.cfg.to_dict(), wl.weights, wl.history_emb, wl.history_offsets, wl.cand_emb, wl.cand_offsets)
        err = score_err(want, full)
        print(f"d={d} blocks={blocks} {kind}: {err:.2e}")
        if kind == "silu":                 # (hot softmax logits amplify the operands' rounding; that bar is derived where the stages are at hand)
            assert err <= TOL_HOT["bf16"], err
