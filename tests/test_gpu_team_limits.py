"""Teams of waves with the wide model, whose weights leave little LDS: lanes as
tall as a team's context window can be and one row taller (a wave per lane
then), with one and with two teams per CU, each kind of pops, against the
images, the encoder's symbols and, for samples, the same draw among more lanes
than teams take (exact).
"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

H, C, NB = 3, 64, 2
LDS_WORDS = 163840 // 4


def tallest_lane(teams, serial):
    """Rows of the tallest lane whose window fits: the LDS holds the weights,
    and per team four waves' head tables, the serial pops' tables, 32 shared
    words and the window, 96 planes of int16."""
    mt = C // 16
    weights = mt * 5 * 256 + 2 * NB * mt * mt * 256 + 7 * mt * 256 + C + 2 * NB * C + 112
    left = (LDS_WORDS - weights) // teams - 4 * 4 * 132 - (16 * 48 + 256 if serial else 0) - 32
    rows = left // 48 // 4 * 4
    return rows - H  # the window has h rows more, rounded up to 4


@pytest.fixture(scope="module")
def model():
    import paper_2201_05213_amd as nx

    torch.cuda.set_device(0)
    return nx, nx.Model(synth.write_blob(H, C, NB, synth.init_params(H, C, NB, 71)))


def lane_shapes(teams, serial, over):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    tall = tallest_lane(teams, serial) + over
    few = [(tall, 5), (33, 40), (18, 21), (tall, 23), (7, 3)]
    return few if teams == 1 else (few * cus)[:cus + 3]


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("K", [1, 4, 8, 16])
@pytest.mark.parametrize("teams", [1, 2])
def test_window_at_its_limit(model, teams, K, over):
    nx, m = model
    rng = np.random.Generator(np.random.PCG64(72))
    shapes = lane_shapes(teams, K < 8, over)
    base = {s: torch.from_numpy(rng.integers(0, 256, size=(*s, 3)).astype(np.uint8)).cuda() for s in set(shapes)}
    imgs = [base[s] for s in shapes]
    data, offs = m.encode(imgs, order=nx.WAVEFRONT, interleave=K)
    for order in (nx.WAVEFRONT, nx.SHEARED):
        out, _, dump = m.decode(data, offs, shapes, order=order, interleave=K, trace=True)
        assert all(torch.equal(a, b) for a, b in zip(out, imgs)), order
        assert torch.equal(dump, m.debug_symbols(imgs)[0]), order


@pytest.mark.parametrize("over", [0, 1])
@pytest.mark.parametrize("teams", [1, 2])
def test_samples_at_the_window_limit(model, teams, over):
    nx, m = model
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    shapes = lane_shapes(teams, False, over)
    seeds = [200 + k % 5 for k in range(len(shapes))]
    out = m.sample(shapes, seeds)
    ref = m.sample(shapes[:5] + [(2, 2)] * (2 * cus), seeds[:5] + [1] * (2 * cus))
    assert all(torch.equal(a, ref[k % 5]) for k, a in enumerate(out))
