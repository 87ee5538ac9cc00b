"""K1's small tile of 256 columns: a request has the bits it has alone on either side of where the tile becomes so wide, up to where the large tile takes over."""
import re

import pytest

from tests import test_gpu_launch_sizes as sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [384, 512])
def test_same_bits_where_the_tile_becomes_wide(d, monkeypatch):
    text = (sizes.CSRC / "gemm_mfma.hip").read_text()
    first = int(re.search(rf"kWideFrom{d} = (\d+)", text).group(1))
    # the last even number of blocks before, and (the last layer's launches over the candidates' blocks alone) twice that
    monkeypatch.setattr(sizes, "limits", lambda _: [(first - 1) // 2 * 2, (first - 1) // 2 * 4])
    sizes.test_same_bits_at_every_launch_size(d)
