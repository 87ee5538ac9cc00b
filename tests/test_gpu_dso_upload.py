"""Micro-batches of which a part was uploaded ahead when a wait, a drain or a full batch sends the rest: every request's scores are those of its own eager forward, bit for bit."""
import numpy as np
import pytest

from paper_2509_22681_amd import workloads as W
from tests.test_gpu_parity import run_gpu

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("order", [[0, 1], [1, 0, 2], [0, 1, 2, 3], [3, 0, 3, 1, 1, 0, 2]])
@pytest.mark.parametrize("how", ["wait", "drain"])
def test_partly_uploaded_batches(how, order):
    from paper_2509_22681_amd import binding as B
    # 3.3 MB, 50 KB, 4.2 MB and candidates alone
    wl = W.make_custom([3200, 40, 4096, 0], [70, 9, 33, 5], d=512, H=8, n_layers=1, n_buckets=64, max_rel_dist=4096, dtype="bf16", seed=9, emb_std=1.0, rab_std=1.0, bias_amp=0.1,
                       affine_random=True, name="upload")
    dw, _, _ = B.to_device(wl)
    ref, _ = run_gpu(B, wl)
    ho, co = wl.history_offsets, wl.cand_offsets
    dso = B.flame_dso_create(B.config_for(wl), dw, 4096, [128], n_executors=2, explicit_shapes=2, max_batch=4)
    try:
        for _ in range(2):
            outs = [np.full(int(co[i + 1] - co[i]), np.nan, np.float32) for i in order]
            tickets = [B.flame_dso_submit_jagged(dso, B.host_embedding(wl.history_emb[ho[i]:ho[i + 1]], "bf16"), B.host_embedding(wl.cand_emb[co[i]:co[i + 1]], "bf16"), o)
                       for i, o in zip(order, outs)]
            if how == "wait":
                for t in tickets[::-1]:
                    B.flame_dso_wait(dso, t)
            else:
                B.flame_dso_drain(dso)
            for i, o in zip(order, outs):
                assert np.array_equal(o, ref[co[i]:co[i + 1]]), (order, i)
    finally:
        B.flame_dso_destroy(dso)
