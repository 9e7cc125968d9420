"""A wave that decodes a lane alone takes the network of a group of few pixels
eight and four pixels at a time, of a full one as a tile of 16: lanes whose
steps have 1 to 20 rows (each count from the ramps of a tall lane, and alone),
in every order, against the images and the encoder's symbols (exact). More
lanes than teams take, so that every lane has one wave.
"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("h,C,K", [(1, 32, 1), (3, 64, 2), (2, 64, 4), (3, 64, 8), (1, 16, 16), (3, 32, 4)])
def test_groups_of_every_size(h, C, K):
    import paper_2201_05213_amd as nx

    torch.cuda.set_device(0)
    rng = np.random.Generator(np.random.PCG64(31))
    m = nx.Model(synth.write_blob(h, C, 2, synth.init_params(h, C, 2, 90 + h)))
    shapes = [(20, 20 * (h + 1) + 3)] + [(n, (h + 1) * n + 2) for n in (1, 3, 4, 5, 8, 9, 12, 13, 16, 17)]
    base = [torch.from_numpy(rng.integers(0, 256, size=(a, b, 3)).astype(np.uint8)).cuda() for a, b in shapes]
    lanes = 2 * torch.cuda.get_device_properties(0).multi_processor_count + 1
    imgs = (base * (lanes // len(base) + 1))[:lanes]
    symbols = m.debug_symbols(imgs)[0]
    data, offs = m.encode(imgs, order=nx.WAVEFRONT, interleave=K)
    for order in (nx.WAVEFRONT, nx.SHEARED):
        out, _, dump = m.decode(data, offs, [t.shape[:2] for t in imgs], order=order, interleave=K, trace=True)
        assert all(torch.equal(a, b) for a, b in zip(out, imgs)), order
        assert torch.equal(dump, symbols), order
    if K == 1:
        data, offs = m.encode(imgs, order=nx.RASTER)
        out, _ = m.decode(data, offs, [t.shape[:2] for t in imgs], order=nx.RASTER)
        assert all(torch.equal(a, b) for a, b in zip(out, imgs))
    ref = m.sample(shapes, list(range(len(shapes))))
    for order in (nx.WAVEFRONT, nx.SHEARED):
        out = m.sample([t.shape[:2] for t in imgs], [k % len(shapes) for k in range(lanes)], order=order)
        assert all(torch.equal(a, ref[k % len(shapes)]) for k, a in enumerate(out)), order
