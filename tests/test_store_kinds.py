"""Where the kernels' stores leave the outputs (no GPU: the assembly is read): the
reader of a call's outputs comes next, so those that fit stay in a cache."""
import re

import pytest

from test_wait_states import listing_of


def stores(source, name, words):
    """{template arguments of kernel `name`: kinds of its stores of that width}"""
    out, where = {}, None
    for line in listing_of(source).splitlines():
        m = re.match(r"(\S+):\s*;\s*@", line)
        if m:
            k = re.search(name + r"I(\w+?)EEEv", m[1])
            where = out.setdefault(k[1], set()) if k else None
        m = re.match(r"\s+global_store_dwordx%d (.*)" % words, line)
        if m and where is not None:
            where.add(" ".join(w for w in m[1].split() if w in ("sc0", "sc1", "nt")))
    assert out
    return out


@pytest.mark.parametrize("kernel", ["k_band_single", "k_band_batched", "k_band_args"])
def test_uint8_outputs(kernel):
    """Through the L2, into the Infinity Cache (agent scope), past both."""
    for args, kinds in stores("sobel4x5_band.hip", kernel, 4).items():
        to = int(re.search(r"Li(\d)$", args)[1])
        assert kinds == {{0: "", 1: "sc1", 2: "nt"}[to]}, (args, kinds)


def test_fp32_magnitudes_and_gradients():
    """Magnitudes in either way, gradients past the caches."""
    for args, kinds in stores("sobel4x5_f32.hip", "k_f32_fwd", 2).items():
        assert kinds == {"nt" if args.endswith("Lb1") else ""}, (args, kinds)
    for args, kinds in stores("sobel4x5_f32.hip", "k_f32_bwd", 2).items():
        assert kinds == {"nt"}, (args, kinds)
