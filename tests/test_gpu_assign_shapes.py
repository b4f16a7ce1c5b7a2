"""The association's index arithmetic (quotients by S through a fixed
multiplier) and its selection of the two nearest of nine candidates, against
the oracle, bit for bit: very wide and very tall images, steps from 1 to
beyond the image, powers of two and their neighbours."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slic():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1509_04232_amd as slic
    return slic


@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("w,h,S", [
    (70001, 3, 7), (70000, 4, 16), (3, 50001, 13), (4, 40000, 8), (1000, 9, 1), (517, 130, 31),
    (517, 130, 33), (640, 96, 64), (333, 211, 127), (640, 200, 128), (96, 80, 1000),
])
def test_quotients_and_selection(slic, squared, w, h, S):
    rng = np.random.default_rng(w + 7 * h + S)
    # few colours: exact ties between candidates beside ordinary pixels
    pal = rng.integers(0, 256, (5, 3), dtype=np.uint8)
    img = pal[rng.integers(0, 5, (h, w))]
    noisy = rng.random((h, w)) < 0.5
    img[noisy] = rng.integers(0, 256, (int(noisy.sum()), 3), dtype=np.uint8)
    dist = oracle.DIST_SQUARED if squared else oracle.DIST_EQ1
    want = oracle.segment(img, S, 10.0, 3, True, False, 0, oracle.COLOR_LAB, dist)
    p = slic.Params(w, h, S=S, m=10.0, squared_distance=squared)
    out = slic.segment(torch.from_numpy(np.ascontiguousarray(img).reshape(-1)).cuda(), p, 3,
                       want_centres=True)
    torch.cuda.synchronize()
    assert np.array_equal(out["labels"].cpu().numpy(), want["labels"])
    assert np.array_equal(out["centres"].cpu().numpy(), want["centres"])
