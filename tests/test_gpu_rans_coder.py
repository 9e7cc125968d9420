"""The rANS encoder's bytes against the oracle's coder, stream by stream.

The symbols (start, freq) are the GPU's own (`debug_symbols`); the oracle codes
the same symbols in plain C, so every stream's bytes must be equal. Sizes sit
at the edges of the encoder's batches (64 symbols for a wave per stream, 16 for
a thread per stream) and on both sides of the stream counts at which it changes
from one to the other; the models give frequencies in the middle of the range
(random weights), and 1 and 65281 alone (all mass in one bin).
"""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def nx():
    import paper_2201_05213_amd as nx

    torch.cuda.set_device(0)
    return nx


def make_model(nx, kind):
    if kind == "random":
        return nx.Model(synth.model_blob("tiny")[0])
    return nx.Model(synth.write_blob(1, 8, 0, synth.delta_params(1, 8)))


def make_images(kind, shapes, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    out = []
    for h, w in shapes:
        a = rng.integers(0, 256, size=(h, w, 3))
        if kind == "delta":
            # mostly the likely bins (0, 255, 0), with runs of unlikely ones
            likely = np.broadcast_to(np.array([0, 255, 0]), a.shape)
            a = np.where(rng.random((h, w, 1)) < 0.8, likely, a)
        out.append(np.ascontiguousarray(a.astype(np.uint8)))
    return out


def streams_of(c, n):
    ends = np.frombuffer(c[32:32 + 4 * n], dtype="<u4").astype(np.int64)
    pay = c[32 + 4 * n:]
    return [pay[a:b] for a, b in zip(np.concatenate([[0], ends[:-1]]), ends)]


def check(nx, m, imgs, order, K):
    ts = [torch.from_numpy(a).cuda() for a in imgs]
    data, offs = m.encode(ts, order=order, interleave=K)
    sym = m.debug_symbols(ts)[0].cpu().numpy().view(np.uint32)
    data, offs = data.cpu().numpy().tobytes(), offs.cpu().tolist()
    at = 0
    for k, a in enumerate(imgs):
        h, w, _ = a.shape
        s = sym[3 * at:3 * (at + h * w)].reshape(h, 3 * w)
        at += h * w
        rows = s if K == nx.ROWS else s.reshape(1, -1)
        got = streams_of(data[offs[k]:offs[k + 1]], len(rows))
        for r, (row, bytes_) in enumerate(zip(rows, got)):
            assert oracle.rans_encode(row & 0xffff, row >> 16) == bytes_, f"image {k} {a.shape} stream {r}"


@pytest.mark.parametrize("kind", ["random", "delta"])
@pytest.mark.parametrize("n_images", [1, "many"])
def test_one_stream_images(nx, kind, n_images):
    m = make_model(nx, kind)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    # symbols 3 n: around 16, 48, 64 and 128
    shapes = [(1, 1), (1, 5), (1, 6), (2, 8), (1, 21), (2, 11), (6, 7), (1, 43), (11, 13)]
    if n_images == "many":
        shapes = (shapes * (16 * cus // len(shapes) + 1))[:16 * cus + 1]
    check(nx, m, make_images(kind, shapes, 5), nx.RASTER, 1)


@pytest.mark.parametrize("kind", ["random", "delta"])
@pytest.mark.parametrize("many", [False, True])
def test_row_streams(nx, kind, many):
    m = make_model(nx, kind)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    shapes = [(3, 1), (2, 5), (2, 6), (2, 21), (2, 22), (2, 43)]
    if many:
        shapes = shapes + [(32 * cus + 1, 6)]
    check(nx, m, make_images(kind, shapes, 6), nx.WAVEFRONT, nx.ROWS)
