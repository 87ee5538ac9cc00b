"""K1 and K3 choose their tiles by the size of a launch and change none of an output's arithmetic with it: a request scored alone,
in a middling batch and in a batch past every limit has the same bits.  (Accuracy against the oracle: the parity tests.)"""
import numpy as np
import pytest

from paper_2509_22681_amd import workloads as W

pytestmark = pytest.mark.gpu

# requests of 64 + 64 rows (two row blocks), then a few ragged ones; the counts pass the limits of the width
MODELS = {64: (2, 60), 128: (2, 260), 192: (3, 260), 256: (4, 540), 384: (6, 210), 512: (8, 210), 320: (5, 40)}


@pytest.mark.parametrize("d", list(MODELS))
def test_same_bits_at_every_launch_size(d):
    import torch
    from paper_2509_22681_amd import binding as B
    H, n = MODELS[d]
    L, M = [64] * n + [65, 1, 130, 0], [64] * n + [3, 70, 0, 5]
    wl = W.make_custom(L, M, d=d, H=H, n_layers=3, n_buckets=16, max_rel_dist=128, dtype="bf16", seed=3, emb_std=1.0, rab_std=1.0, bias_amp=0.1,
                       affine_random=True, name=f"sizes{d}")

    def scores(w):
        h = B.flame_gr_create(B.config_for(w))
        try:
            dw, hist, cand = B.to_device(w)
            out = torch.full((int(w.cand_offsets[-1]),), float("nan"), device="cuda:0")
            B.flame_gr_forward(h, dw, hist, w.history_offsets, cand, w.cand_offsets, out)
            torch.cuda.synchronize()
            return out.cpu().numpy()
        finally:
            B.flame_gr_destroy(h)

    whole, co = scores(wl), wl.cand_offsets
    assert np.isfinite(whole).all()
    for idx in ([0], [n - 1], [n], [n + 1], [n + 3], list(range(30, 44)), list(range(n - 100 if n > 120 else 0, n + 4))):
        part = scores(wl.subset(idx))
        assert np.array_equal(part, np.concatenate([whole[co[i]:co[i + 1]] for i in idx])), (d, idx[0], len(idx))


@pytest.mark.parametrize("d,H", [(64, 2), (192, 3), (320, 5)])
def test_hidden_rows_at_any_alignment(d, H):
    """The gather of the candidates' rows stores 16 bytes at a time where the caller's array allows it."""
    import torch
    from paper_2509_22681_amd import binding as B
    wl = W.make_custom([70, 0, 33], [65, 3, 16], d=d, H=H, n_layers=2, n_buckets=16, max_rel_dist=128, dtype="bf16", seed=5, name=f"hidden{d}")
    n = int(wl.cand_offsets[-1]) * d
    h = B.flame_gr_create(B.config_for(wl))
    try:
        dw, hist, cand = B.to_device(wl)
        rows = []
        for shift in (0, 1, 2, 4):
            buf = torch.full((n + 8,), float("nan"), device="cuda:0")
            B.flame_gr_forward_hidden(h, dw, hist, wl.history_offsets, cand, wl.cand_offsets, buf[shift:shift + n].view(-1, d))
            torch.cuda.synchronize()
            got = buf.cpu().numpy()
            assert np.isnan(got[:shift]).all() and np.isnan(got[shift + n:]).all()
            rows.append(got[shift:shift + n])
    finally:
        B.flame_gr_destroy(h)
    assert np.isfinite(rows[0]).all()
    for r in rows[1:]:
        assert np.array_equal(r, rows[0])
