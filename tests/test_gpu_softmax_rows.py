"""Softmax attention: a row's bits do not depend on the rows that share its wavefront, whichever of them move the running maximum and when.  (Its place among the 32 may show in the last bit
of its sum of weights, which two lanes hold: the one that the place names adds the row's own key.  The rows compared here keep theirs.)"""
import numpy as np
import pytest

from paper_2509_22681_amd import workloads as W

pytestmark = pytest.mark.gpu


# one wavefront and several, throughput and latency kernels, both head widths; histories of 1 to 40 key tiles
@pytest.mark.parametrize("latency", [0, 1])
@pytest.mark.parametrize("d,H,L,M", [(128, 2, 2500, 70), (128, 4, 700, 33), (64, 1, 60, 64)])
def test_candidates_have_the_same_bits_beside_any_others(d, H, L, M, latency):
    import torch
    from paper_2509_22681_amd import binding as B
    rng = np.random.default_rng(L)
    wl = W.make_custom([L], [M], d=d, H=H, n_layers=2, n_buckets=64, max_rel_dist=4096, dtype="bf16", seed=3, emb_std=1.0, rab_std=1.0, bias_amp=0.1, affine_random=True,
                       attn_kind="softmax", name="rows")
    # maxima that grow along the history, by far less than 2^8 in some rows and by far more in others
    wl.history_emb = W._round_storage((wl.history_emb * np.linspace(0.3, 4.0, L)[:, None]).astype(np.float32), "bf16")
    wl.cand_emb = W._round_storage((wl.cand_emb * np.exp(rng.uniform(np.log(0.1), np.log(6.0), M))[:, None]).astype(np.float32), "bf16")
    dw, hist, cand = B.to_device(wl)
    h = B.flame_gr_create(B.config_for(wl, latency_mode=latency))
    try:
        def scores(idx):
            out = torch.full((len(idx),), float("nan"), device="cuda:0")
            B.flame_gr_forward(h, dw, hist, wl.history_offsets, cand[torch.as_tensor(idx, device="cuda:0")].contiguous(), np.array([0, len(idx)], np.int32), out)
            torch.cuda.synchronize()
            return out.cpu().numpy()

        want = scores(np.arange(M))
        assert np.isfinite(want).all()
        for keep in (np.arange(0, M, 2), np.arange(1, M, 2), np.arange(0, M, 5), np.array([M - 1])):
            for _ in range(3):
                idx = rng.integers(0, M, M)                # the others: any candidates, some of them twice
                idx[keep] = keep
                got = scores(idx)
                assert np.array_equal(got[keep], want[keep]), (int((got[keep] != want[keep]).sum()), len(keep))
        for first in (32, 64):                             # another group, the same places
            if first < M:
                assert np.array_equal(scores(np.arange(first, M)), want[first:])
    finally:
        B.flame_gr_destroy(h)
