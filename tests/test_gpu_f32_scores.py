"""fp32 models of up to 64 features: the last output projection makes the scores.  Against the hidden rows that the same forward gives, whose projection writes them, in 64 bits; and each
request alone against the batch, bit for bit."""
import numpy as np
import pytest

from paper_2509_22681_amd import workloads as W

pytestmark = pytest.mark.gpu


# widths of one and two 32-column blocks, whole and not
@pytest.mark.parametrize("d,H", [(64, 2), (32, 1), (36, 2), (60, 2), (4, 1)])
@pytest.mark.parametrize("static", [0, 1])
def test_scores_are_those_of_the_hidden_rows(d, H, static):
    import torch
    from paper_2509_22681_amd import binding as B
    wl = W.make_custom([70, 0, 33, 1], [65, 3, 64, 31], d=d, H=H, n_layers=2, n_buckets=16, max_rel_dist=128, dtype="f32", seed=5, emb_std=1.0, rab_std=1.0, bias_amp=0.1, affine_random=True,
                       name=f"scores{d}")
    wl.weights["b_s"] = 0.25

    def run(batch, hidden=False):
        h = B.flame_gr_create(B.config_for(batch, weights_static=static))
        try:
            dw, hist, cand = B.to_device(batch)
            n = int(batch.cand_offsets[-1])
            out = torch.full((n, d) if hidden else (n,), float("nan"), device="cuda:0")
            (B.flame_gr_forward_hidden if hidden else B.flame_gr_forward)(h, dw, hist, batch.history_offsets, cand, batch.cand_offsets, out)
            torch.cuda.synchronize()
            return out.cpu().numpy()
        finally:
            B.flame_gr_destroy(h)

    scores, rows = run(wl), run(wl, hidden=True).astype(np.float64)
    w = wl.weights["w_s"].astype(np.float64)
    want = rows @ w + 0.25
    # a product's rounding, and one per addition, of at most the sum of magnitudes
    assert (np.abs(scores - want) <= (d + 2) * 2.0 ** -24 * (np.abs(rows) @ np.abs(w) + 0.25)).all()
    co = wl.cand_offsets
    for i in range(wl.n_requests):
        assert np.array_equal(run(wl.subset([i])), scores[co[i]:co[i + 1]])
