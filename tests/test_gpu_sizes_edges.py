"""GPU parity at the sizes where a launch rule or a tile edge can go wrong: one small case per edge, against the oracle."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_18780_amd import binding as sb
from paper_2604_18780_amd import synth

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("T,C", [(1, 3), (511, 5), (512, 24), (513, 4), (1500, 24), (2048, 1)])
def test_entropies_over_many_workgroups(T, C):
    rng = np.random.default_rng(T)
    pm = rng.random((3, T, C), dtype=np.float32)
    pm[:, ::7] = 0.0
    bd = rng.random((3, T + 1), dtype=np.float32)
    lengths = np.array([T, (T + 1) // 2, 1], dtype=np.int32)
    h_pos, h_bdy = sb.semicrf_entropies(dev(pm), dev(bd), dev(lengths))
    rp, rb = oracle.entropies(pm, bd, lengths)
    np.testing.assert_allclose(h_pos.cpu().numpy(), rp, rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(h_bdy.cpu().numpy(), rb, rtol=1e-6, atol=1e-6)


@pytest.mark.parametrize("C", [1, 2, 7, 8])
@pytest.mark.parametrize("offset", [0, 1, 2, 3])
def test_entropies_of_few_labels(C, offset):
    """Every number of threads a workgroup can have, marginals at every place relative to the 16 bytes of a load."""
    rng = np.random.default_rng(C)
    pm, bd = rng.random((3, 1030, C), dtype=np.float32), rng.random((3, 1031), dtype=np.float32)
    lengths = np.array([1030, 513, 0], dtype=np.int32)
    flat = dev(np.concatenate([np.full(offset, np.nan, dtype=np.float32), pm.ravel()]))
    h_pos, h_bdy = sb.semicrf_entropies(flat[offset:].view(3, 1030, C), dev(bd), dev(lengths))
    rp, rb = oracle.entropies(pm, bd, lengths)
    np.testing.assert_allclose(h_pos.cpu().numpy(), rp, rtol=1e-6, atol=1e-7)
    np.testing.assert_allclose(h_bdy.cpu().numpy(), rb, rtol=1e-6, atol=1e-6)


def test_entropy_terms_of_single_values():
    """One value per sequence, so that its -x log x shows: the ends of the float's range, both sides of the powers of two and of
    the square root of one half, 1, values that are no probabilities, and none at all."""
    x = [1e-45, 1.2e-38, 3e-20, 0.25, 0.5, 0.70710677, 0.70710683, 0.99999994, 1.0, 1.0000001, 1.4142135, 1.4142137, 2.0, 1e36]
    x = np.concatenate([np.array(x, dtype=np.float32), np.random.default_rng(1).random(200, dtype=np.float32)])
    odd = np.array([0.0, -1.0, np.nan, np.inf], dtype=np.float32)
    pm = np.concatenate([x, odd]).reshape(-1, 1, 1)
    h = sb.semicrf_entropies(dev(pm), dev(np.ones((len(pm), 2), dtype=np.float32)), None)[0].cpu().numpy()
    want = (-x.astype(np.float64) * np.log(x.astype(np.float64))).astype(np.float32)
    np.testing.assert_allclose(h[: len(x)], want, rtol=1.2e-7, atol=0)  # 64-bit terms: the float's rounding, on either side
    assert (h[len(x):-1] == 0).all() and h[-1] == -np.inf


@pytest.mark.parametrize("T,C", [(1, 1), (7, 3), (8, 24), (255, 5), (256, 24), (257, 64), (1000, 33), (1024, 130)])
@pytest.mark.parametrize("scale", [1.0, 30.0])
def test_prefix_sums_at_chunk_and_segment_edges(T, C, scale):
    """Chunks of 256 and segments of 8 positions; scale 30 shortens the scaling blocks below a segment."""
    rng = np.random.default_rng(1000 * T + C)
    emis = (scale * rng.standard_normal((3, T, C))).astype(np.float32)
    lengths = np.array([T, (T + 1) // 2, 0], dtype=np.int32)
    cum = sb.semicrf_cum_scores(dev(emis), dev(lengths)).cpu().numpy()
    for b in range(3):
        L = int(lengths[b])
        f = emis[b, :L].astype(np.float64)
        ref = np.zeros((T + 1, C))
        if L:
            ref[1:L + 1] = np.cumsum(f - f.mean(axis=0), axis=0)
        np.testing.assert_allclose(cum[b], ref, rtol=0, atol=1e-10 * scale * max(1, T))


@pytest.mark.parametrize("T", [130815, 131072])
def test_prefix_sums_either_side_of_the_inline_limit(T):
    """512 chunks are the most the prefix kernel sums itself; beyond that a launch of its own does."""
    rng = np.random.default_rng(T)
    emis = rng.standard_normal((1, T, 2)).astype(np.float32)
    cum = sb.semicrf_cum_scores(dev(emis), None).cpu().numpy()
    f = emis[0].astype(np.float64)
    np.testing.assert_allclose(cum[0, 1:], np.cumsum(f - f.mean(axis=0), axis=0), rtol=0, atol=1e-8)


@pytest.mark.parametrize("T", [5, 700, 3000])
def test_entropies_of_an_empty_boundary_posterior(T):
    """No mass at all (a caller's own weights, or a sequence without a valid path): an entropy of 0, as for length 0."""
    pm = np.full((3, T, 4), 0.25, dtype=np.float32)
    bd = np.zeros((3, T + 1), dtype=np.float32)
    bd[1, :T] = 1.0
    h_pos, h_bdy = sb.semicrf_entropies(dev(pm), dev(bd), dev(np.array([T, T, 0], dtype=np.int32)))
    np.testing.assert_allclose(h_pos.cpu().numpy(), [np.log(4.0), np.log(4.0), 0.0], rtol=1e-6)
    np.testing.assert_allclose(h_bdy.cpu().numpy(), [0.0, np.log(T), 0.0], rtol=1e-6)
