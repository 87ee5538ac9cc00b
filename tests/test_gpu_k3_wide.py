"""K3 with six and eight wavefronts: on either side of the limits of its launches, and of the one below which the features are cut in four, a request has the bits it has alone."""
import re

import pytest

from tests import test_gpu_launch_sizes as sizes

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [384, 512])
def test_same_bits_where_the_wavefronts_change(d, monkeypatch):
    text = (sizes.CSRC / "kernels.h").read_text()
    limits = [int(re.search(rf"kK3{n} = (\d+)", text).group(1)) for n in ("CutInFour", "CutInTwo", "OneEach")]
    assert limits == sorted(limits)
    # (the last layer's launches have the candidates' blocks alone, half of them)
    monkeypatch.setattr(sizes, "limits", lambda _: [2] + limits + [2 * n for n in limits])
    sizes.test_same_bits_at_every_launch_size(d)
