"""K1's small tile of 256 columns: a request has the bits it has alone on either side of where the tile becomes so wide, up to where the large tile takes over."""
import re

import pytest

from tests import test_gpu_launch_sizes as sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [384, 512])
def test_same_bits_where_the_tile_becomes_wide(d, monkeypatch):
    text = (sizes.CSRC / "gemm_mfma.hip").read_text()
    names = ["kWideFrom384"] if d == 384 else ["kWideFrom512", "kWideOneEach512", "kWideAgainFrom512"]
    limits = [int(re.search(rf"{n} = (\d+)", text).group(1)) for n in names]
    # the last even number of blocks before each, and (the last layer's launches over the candidates' blocks alone) twice that
    monkeypatch.setattr(sizes, "limits", lambda _: [k * ((n - 1) // 2 * 2) for n in limits for k in (1, 2)])
    sizes.test_same_bits_at_every_launch_size(d)
