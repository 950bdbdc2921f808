"""bench.py's metric counts evaluated signal-unit pairs: every network it times is pinned to the
exhaustive scan of its batch size, unless a variant is asked for."""
from types import SimpleNamespace

import pytest

import bench
from paper_1503_08294_amd import gsn


@pytest.mark.parametrize("m_max", [1, 64, 256, 257, 16_384])
@pytest.mark.parametrize("asked,variant", [(0, 6), (3, 3)])
def test_networks_are_pinned_to_the_exhaustive_scan(m_max, asked, variant):
    calls = []
    net = SimpleNamespace(params=SimpleNamespace(m_max=m_max),
                          tune=lambda key, value: calls.append((key, value)))
    bench.tune(gsn, net, SimpleNamespace(variant=asked, split=0, grab=0, rebucket=0))
    # (variant 6 is the small-batch scan up to 256 signals and the split-binary16 scan above)
    assert calls == [(gsn.GSN_TUNE_VARIANT, variant)]
