"""Few lanes are decoded by teams of waves, many by a wave each: the same
containers alone, with one lane per CU, with two and with more, against the
images and the encoder's symbols (exact: every decoder computes the encoder's
CDFs bit for bit). Lane sizes with one row, one column, a step of more than 16
rows and steps without a pixel; every number of streams; also a lane too tall
for a team's window.
"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

SHAPES = [(9, 14), (1, 20), (20, 1), (5, 2), (3, 70), (23, 90)]


def batch(h, shapes, seed):
    import paper_2201_05213_amd as nx

    torch.cuda.set_device(0)
    rng = np.random.Generator(np.random.PCG64(seed))
    m = nx.Model(synth.write_blob(h, 16, 1, synth.init_params(h, 16, 1, 60 + h)))
    base = [torch.from_numpy(rng.integers(0, 256, size=(a, b, 3)).astype(np.uint8)).cuda() for a, b in SHAPES + shapes]
    return nx, m, base


def check(nx, m, imgs, order, K):
    shapes = [t.shape[:2] for t in imgs]
    data, offs = m.encode(imgs, order=nx.WAVEFRONT, interleave=K)
    out, _, dump = m.decode(data, offs, shapes, order=order, interleave=K, trace=True)
    for k, (a, b) in enumerate(zip(out, imgs)):
        assert torch.equal(a, b), (k, tuple(b.shape))
    assert torch.equal(dump, m.debug_symbols(imgs)[0])


@pytest.mark.parametrize("K", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("h", [1, 2, 3])
def test_lane_counts_around_the_rule(h, K):
    nx, m, base = batch(h, [], 7)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    for lanes in (1, len(base), cus, cus + 1, 2 * cus, 2 * cus + 1):
        check(nx, m, (base * (lanes // len(base) + 1))[:lanes], nx.WAVEFRONT, K)
    check(nx, m, base, nx.SHEARED, K)


@pytest.mark.parametrize("K", [1, 8, 16])
def test_lanes_taller_than_a_window(K):
    nx, m, base = batch(3, [(1100, 6)], 8)
    check(nx, m, base, nx.WAVEFRONT, K)
    check(nx, m, base, nx.SHEARED, K)


@pytest.mark.parametrize("h", [1, 2, 3])
def test_samples_do_not_depend_on_the_lane_count(h):
    nx, m, _ = batch(h, [], 9)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ref = m.sample(SHAPES, [100 + k for k in range(len(SHAPES))])
    for lanes in (cus + 1, 2 * cus + 1):
        k = [q % len(SHAPES) for q in range(lanes)]
        for order in (nx.WAVEFRONT, nx.SHEARED):
            out = m.sample([SHAPES[q] for q in k], [100 + q for q in k], order=order)
            assert all(torch.equal(a, ref[q]) for a, q in zip(out, k))
