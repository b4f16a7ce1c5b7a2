"""Connectivity of small frames in one workgroup (csrc/ccl.hip) against the
oracle, bit for bit: one tile, ragged tiles, single rows and columns, the
largest frame of the path and the first beyond it, noisy label maps whose
chains of joins cross tiles, and the in-place relabelling of a context."""
import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def slic():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1509_04232_amd as slic
    return slic


@pytest.mark.parametrize("w,h,S,sigma", [(1, 1, 1, 8.0), (32, 32, 8, 8.0), (33, 31, 4, 30.0),
                                         (97, 75, 8, 12.0), (80, 100, 16, 8.0), (100, 80, 8, 40.0),
                                         (63, 126, 5, 40.0), (126, 63, 8, 40.0), (1, 700, 4, 30.0),
                                         (2000, 4, 8, 30.0), (8000, 1, 8, 8.0), (8001, 1, 8, 8.0),
                                         (128, 128, 8, 40.0), (96, 72, 8, 60.0)])
def test_small_frames_match_oracle(slic, w, h, S, sigma):
    img = synth.voronoi_image(w + 3 * h, w, h, max(2, w * h // 300), sigma)
    rgb = torch.from_numpy(np.ascontiguousarray(img).reshape(-1)).cuda()
    p = slic.Params(w, h, S=S, m=10.0)
    want = oracle.segment(img, S, 10.0, 3, True, True, 0)
    out = slic.segment(rgb, p, 3, enforce=True)
    ctx = slic.Context(p, rgb)
    ctx.iterate(3)
    n = ctx.enforce_connectivity()
    lb = ctx.labels()
    torch.cuda.synchronize()
    assert np.array_equal(out["labels"].cpu().numpy(), want["seg_labels"])
    assert int(out["n_segments"].cpu()[0]) == want["n_segments"]
    assert np.array_equal(lb.cpu().numpy(), want["seg_labels"])
    assert int(n.cpu()[0]) == want["n_segments"]
    ctx.close()
