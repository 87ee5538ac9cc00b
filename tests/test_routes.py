"""Properties of the launch code that need no GPU to check."""
import re
from pathlib import Path

from paper_2509_22681_amd import build as build_mod

CSRC = Path(build_mod.CSRC)


def test_the_plane_that_the_layer_kernel_overwrites_is_not_restrict():
    """The layer kernel reads U of its layer and writes U of the next to the same plane: a promise that U does not change would be a false one."""
    params = re.search(r"void layer_kernel\((.*?)\)\s*\{", (CSRC / "layer_mfma.hip").read_text(), re.S).group(1)
    by_name = {p.split()[-1].lstrip("*"): p for p in params.split(",")}
    assert "__restrict__" not in by_name["U"] and "__restrict__" in by_name["O"]
