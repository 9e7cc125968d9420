"""Decoding and sampling with 16 channels at the depths where the decoders'
choices change (4 and 5 residual blocks) and far beyond: alone, with one, two
and more lanes per CU, against the images and the encoder's symbols (exact:
every decoder computes the encoder's CDFs bit for bit).
"""
import numpy as np
import pytest
import torch

import synth

pytestmark = pytest.mark.gpu

SHAPES = [(4, 17), (5, 9), (9, 40), (17, 70), (1, 6), (7, 2)]


@pytest.mark.parametrize("nb", [4, 5, 24])
@pytest.mark.parametrize("h", [1, 3])
def test_deep_narrow_models(h, nb):
    import paper_2201_05213_amd as nx

    torch.cuda.set_device(0)
    rng = np.random.Generator(np.random.PCG64(10 * h + nb))
    m = nx.Model(synth.write_blob(h, 16, nb, synth.init_params(h, 16, nb, 70 + nb)))
    base = [torch.from_numpy(rng.integers(0, 256, size=(a, b, 3)).astype(np.uint8)).cuda() for a, b in SHAPES]
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ref = m.sample(SHAPES, list(range(len(SHAPES))), order=nx.RASTER)
    for lanes in (len(base), cus + 1, 2 * cus + 1):
        imgs = (base * (lanes // len(base) + 1))[:lanes]
        shapes = [t.shape[:2] for t in imgs]
        symbols = m.debug_symbols(imgs)[0]
        for K in (1, 2, 4, 8, 16):
            data, offs = m.encode(imgs, interleave=K)
            for order in (nx.WAVEFRONT, nx.SHEARED):
                out, _, dump = m.decode(data, offs, shapes, order=order, interleave=K, trace=True)
                assert all(torch.equal(a, b) for a, b in zip(out, imgs)), (lanes, K, order)
                assert torch.equal(dump, symbols), (lanes, K, order)
        out = m.sample(shapes, [k % len(base) for k in range(lanes)])
        assert all(torch.equal(a, ref[k % len(base)]) for k, a in enumerate(out)), lanes
    data, offs = m.encode(base, order=nx.RASTER)
    out, _ = m.decode(data, offs, SHAPES, order=nx.RASTER)
    assert all(torch.equal(a, b) for a, b in zip(out, base))
