"""The edge list of an export is the imported one, ascending: rows at the edges of the listing's
workgroups (256 units), a hub whose row is long, units with no edge, and a network past the
largest count of workgroups whose sums are folded."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,e", [(2, 0), (2, 1), (255, 300), (256, 400), (257, 700),
                                 (5_000, 14_000), (530_001, 40_000)])
@pytest.mark.parametrize("hub", [False, True])
def test_import_then_export(n, e, hub):
    import torch
    from paper_1503_08294_amd import gsn
    rng = np.random.default_rng(n + e)
    pairs = rng.integers(0, n, (4 * e + 8, 2))
    if hub and n > 2:
        pairs[: min(n, 600), 0] = n // 2
    pairs = np.sort(pairs[pairs[:, 0] != pairs[:, 1]], axis=1)
    pairs = np.unique(pairs, axis=0)
    pairs = pairs[rng.permutation(len(pairs))[:e]]
    e = len(pairs)
    edges = np.concatenate([pairs.T, rng.integers(0, 50, (1, e))]).astype(np.int32)
    xyz = rng.standard_normal((3, n)).astype(np.float32)
    err = rng.random(n).astype(np.float32)
    net = gsn.Network(gsn.make_params(n_max=n + 3, e_max=e + 1, m_max=16),
                      torch.from_numpy(xyz))
    net.import_state(torch.from_numpy(xyz), torch.from_numpy(err),
                     torch.from_numpy(np.ascontiguousarray(edges)))
    got = net.export()
    order = np.lexsort((edges[1], edges[0]))
    np.testing.assert_array_equal(got["edges"].numpy(), edges[:, order])
    np.testing.assert_array_equal(got["xyz"].numpy(), xyz)
    np.testing.assert_array_equal(got["err"].numpy(), err)
