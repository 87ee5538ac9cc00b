"""The layer kernel where its launches change shape: all row blocks as halves, whole blocks and halves, whole blocks only, and launches that stream.  Bit for bit the two kernels that run
where a handle's planes are to be looked at."""
import numpy as np
import pytest

from paper_2509_22681_amd import workloads as W
from tests.test_gpu_layer_kernel import batch

pytestmark = pytest.mark.gpu

UNITS = 256           # compute units: blocks beyond a multiple of them go as halves up to half as many
# (an even number of blocks); the two kernels stream from 16 MB of a plane on: past 512 blocks of d = 256, 682 of d = 192 and 1024 of d = 128
SIZES = [(128, 2, n) for n in (UNITS // 2, UNITS // 2 + 2, UNITS, UNITS + 2, 2 * UNITS + 4, 5 * UNITS + 2)] + [(192, 3, n) for n in (UNITS + UNITS // 2, UNITS + UNITS // 2 + 2, 854)] + [(256, 4, n) for n in (UNITS // 2, 640, 900)]


@pytest.mark.parametrize("d,H,blocks", SIZES)
def test_halves_of_blocks_give_the_same_bits(d, H, blocks):
    import torch
    from paper_2509_22681_amd import binding as B
    L, M = batch(blocks)
    wl = W.make_custom(L, M, d=d, H=H, n_layers=3, n_buckets=16, max_rel_dist=128, dtype="bf16", seed=5, emb_std=1.0, rab_std=1.0, bias_amp=0.1, affine_random=True, attn_scale=0.7,
                       name="split")
    dw, hist, cand = B.to_device(wl)

    def scores(captured):
        h = B.flame_gr_create(B.config_for(wl))
        try:
            if captured:
                B.flame_gr_debug_capture(h, 0)
            B.flame_gr_debug_profile(h, True)
            out = torch.full((int(wl.cand_offsets[-1]),), float("nan"), device="cuda:0")
            B.flame_gr_forward(h, dw, hist, wl.history_offsets, cand, wl.cand_offsets, out)
            torch.cuda.synchronize()
            return out.cpu().numpy(), B.flame_gr_debug_profile_read(h)["uvqk"][1]
        finally:
            B.flame_gr_destroy(h)

    want, launches = scores(True)
    got, fused = scores(False)
    assert launches == 3 and fused == 1            # the projections of the first layer alone are a launch of their own
    assert np.isfinite(want).all() and np.array_equal(got, want)
