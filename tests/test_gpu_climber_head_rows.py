"""Fusion and task head in one launch, for passes of many rows: the bits of the two kernels that passes of fewer rows take, for every shape that it takes and one that it does not."""
import re

import numpy as np
import pytest

from paper_2509_22681_amd import build as build_mod
from tests.test_gpu_climber import head_weights

pytestmark = pytest.mark.gpu


# (blocks, width, units, tasks): 12, 4, 16, 2 and 14 wavefronts; heads with two strips a wavefront; the last does not fit
@pytest.mark.parametrize("nb,d,E,T", [(2, 192, 256, 2), (2, 64, 128, 1), (4, 128, 256, 2), (1, 128, 256, 1), (1, 448, 128, 2), (2, 320, 128, 1)])
def test_many_rows_give_the_bits_of_few(nb, d, E, T):
    import torch
    from paper_2509_22681_amd import binding as B
    with open(f"{build_mod.CSRC}/climber_head.hip") as f:
        first = int(re.search(r"kHeadRows = (\d+)", f.read()).group(1))
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(nb * d)
    w = {k: torch.from_numpy(v).to("cuda:0") for k, v in head_weights(nb, d, T, E, 7).items()}
    for rows in (first, first + 30, first + 32):
        hidden = [torch.randn(rows, d, generator=gen, device="cuda:0") for _ in range(nb)]

        def head(a, b):
            fused, probs = torch.full((b - a, d), float("nan"), device="cuda:0"), torch.full((b - a, T), float("nan"), device="cuda:0")
            B.flame_climber_head(w, [h[a:b].contiguous() for h in hidden], fused, probs)
            torch.cuda.synchronize()
            return fused.cpu().numpy(), probs.cpu().numpy()

        whole, parts = head(0, rows), [head(0, 2000), head(2000, rows)]
        assert np.isfinite(whole[0]).all() and np.isfinite(whole[1]).all()
        for i in range(2):
            assert np.array_equal(whole[i], np.concatenate([p[i] for p in parts])), (rows, i)
