"""The causal context at the borders of images and patches: code lengths per
pixel against the FP64 oracle, for sizes at which the gather changes form
(images narrower than the horizon, one row, corner pixels) or masks taps
(every side of a lane), every horizon. Bar: the per-pixel bar of the parity
tests, 1e-5 relative with a floor of 1e-4 bits (a wrong or unmasked tap moves
a pixel's bits by far more).
"""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

SHAPES = [(1, 1), (1, 2), (2, 2), (5, 1), (1, 40), (2, 33), (9, 3), (4, 4), (6, 17), (19, 50)]


@pytest.mark.parametrize("h", [1, 2, 3])
@pytest.mark.parametrize("patch", [None, (1, 1), (2, 3), (5, 16), (4, 7), (16, 2)])
def test_bits_per_pixel_at_borders(h, patch):
    import paper_2201_05213_amd as nx

    torch.cuda.set_device(0)
    blob = synth.write_blob(h, 16, 1, synth.init_params(h, 16, 1, 40 + h))
    m, om = nx.Model(blob), oracle.Model.from_blob(blob)
    rng = np.random.Generator(np.random.PCG64(100 + h))
    imgs = [rng.integers(0, 256, size=(a, b, 3)).astype(np.uint8) for a, b in SHAPES]
    _, px = m.nll([torch.from_numpy(a).cuda() for a in imgs], patch=patch, per_pixel=True)
    ph, pw = patch or (0, 0)
    ref = np.concatenate([om.stats(a, ph, pw, px_bits=True)["px_bits"].reshape(-1) for a in imgs])
    err = np.abs(px.cpu().numpy().astype(np.float64) - ref)
    assert np.all(err <= np.maximum(1e-5 * np.abs(ref), 1e-4)), float(err.max())
