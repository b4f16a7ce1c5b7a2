"""All rounds of a frame in one launch (csrc/rounds.hip) against the oracle,
bit for bit: tiles at the image's edges, cells that meet few and many tiles,
both distances, rounds continued by later calls, a captured segmentation
replayed beside other work, and frames that share the chip with other
streams' kernels (so that not every workgroup of the launch starts at
once)."""
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


def _img(w, h, seed):
    return synth.voronoi_image(seed, w, h, max(2, w * h // 900), 8.0)


def _gpu(img):
    return torch.from_numpy(np.ascontiguousarray(img).reshape(-1)).cuda()


@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("w,h,S", [
    (64, 48, 4), (65, 33, 5), (129, 97, 8), (320, 240, 16), (333, 251, 27), (640, 31, 16),
    (97, 640, 32), (512, 400, 85), (512, 400, 86), (1030, 1027, 8), (1500, 1400, 12),
])
def test_split_rounds_match_oracle(slic, squared, w, h, S):
    img = _img(w, h, w + h + S)
    dist = oracle.DIST_SQUARED if squared else oracle.DIST_EQ1
    p = slic.Params(w, h, S=S, m=10.0, squared_distance=squared)
    ctx = slic.Context(p, _gpu(img))
    done = 0
    for n in (3, 1, 4):
        ctx.iterate(n)
        done += n
        want = oracle.segment(img, S, 10.0, done, True, False, 0, oracle.COLOR_LAB, dist)
        lb, (cen, cnt) = ctx.labels(), ctx.centres()
        torch.cuda.synchronize()
        assert np.array_equal(lb.cpu().numpy(), want["labels"]), done
        assert np.array_equal(cen.cpu().numpy(), want["centres"]), done
        assert np.array_equal(cnt.cpu().numpy(), want["counts"]), done
    ctx.close()


def test_empty_clusters_keep_their_centres(slic):
    # two flat halves at m = 0: most centres lose all their pixels
    w, h, S = 192, 128, 8
    img = np.zeros((h, w, 3), np.uint8)
    img[:, w // 2:] = (200, 30, 90)
    want = oracle.segment(img, S, 0.0, 6, False, False)
    p = slic.Params(w, h, S=S, m=0.0, perturb=False)
    out = slic.segment(_gpu(img), p, 6, want_centres=True)
    torch.cuda.synchronize()
    assert np.array_equal(out["labels"].cpu().numpy(), want["labels"])
    assert np.array_equal(out["centres"].cpu().numpy(), want["centres"])


def test_captured_segmentation_replayed(slic):
    from paper_1509_04232_amd import _abi
    w, h, S = 320, 200, 16
    imgs = [_img(w, h, s) for s in (1, 2, 3)]
    want = [oracle.segment(i, S, 10.0, 5, True, True) for i in imgs]
    p = slic.Params(w, h, S=S, m=10.0)
    cp = p.c()
    rgb = _gpu(imgs[0]).clone()
    ws = slic.workspace_for(p)
    labels = torch.empty((h, w), dtype=torch.int32, device="cuda")

    def segment(stream):
        _abi.slic_segment(cp, rgb.data_ptr(), 5, 1, labels.data_ptr(), None, None, None,
                          stream.cuda_stream, ws.data_ptr(), ws.numel())

    segment(torch.cuda.current_stream())
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        segment(torch.cuda.current_stream())
    for k in (1, 2, 0, 1):
        rgb.copy_(_gpu(imgs[k]))
        other = torch.randn(512, 512, device="cuda")
        (other @ other).sum()
        labels.fill_(-1)
        g.replay()
        torch.cuda.synchronize()
        assert np.array_equal(labels.cpu().numpy(), want[k]["seg_labels"])


def test_frames_beside_other_kernels(slic):
    w, h, S = 640, 480, 16
    imgs = [_img(w, h, s) for s in (11, 12)]
    want = [oracle.segment(i, S, 10.0, 6, True, False) for i in imgs]
    p = slic.Params(w, h, S=S, m=10.0)
    rgb = [_gpu(i) for i in imgs]
    ws = [slic.workspace_for(p) for _ in imgs]
    big = torch.randn(4096, 4096, device="cuda")
    streams = [torch.cuda.Stream() for _ in imgs]
    load = torch.cuda.Stream()
    torch.cuda.synchronize()
    outs = []
    for _ in range(4):
        with torch.cuda.stream(load):
            for _ in range(3):
                big @ big
        for i, s in enumerate(streams):
            with torch.cuda.stream(s):
                outs.append((i, slic.segment(rgb[i], p, 6, workspace=ws[i])["labels"]))
    torch.cuda.synchronize()
    for i, lb in outs:
        assert np.array_equal(lb.cpu().numpy(), want[i]["labels"])


@pytest.mark.parametrize("w,h", [(1, 1), (1, 40), (63, 17), (65, 15), (130, 33), (5, 70000)])
def test_stray_filter_and_energy_at_tile_edges(slic, w, h):
    rng = np.random.default_rng(w * 131 + h)
    img = rng.integers(0, 256, (h, w, 3), dtype=np.uint8)
    S = 5
    want = oracle.segment(img, S, 5.0, 2, True, False)
    ctx = slic.Context(slic.Params(w, h, S=S, m=5.0), _gpu(img))
    ctx.iterate(2)
    e = ctx.energy()
    ctx.filter_stray(3)
    lb = ctx.labels()
    torch.cuda.synchronize()
    assert float(e.cpu()[0]) == pytest.approx(want["energy"], rel=1e-9)
    assert np.array_equal(lb.cpu().numpy(), oracle.stray_filter(want["labels"], 3))
    ctx.close()


@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("w,h,S,threshold", [(320, 240, 16, 2.0), (333, 251, 27, 1.0),
                                             (700, 500, 8, 3.0), (96, 72, 8, 0.0), (640, 480, 16, 1e4)])
def test_convergence_stop_in_one_launch(slic, squared, w, h, S, threshold):
    img = _img(w, h, 7 * w + S)
    ctx = slic.Context(slic.Params(w, h, S=S, m=10.0, squared_distance=squared), _gpu(img))
    n = ctx.iterate_converge(12, threshold)
    lb, (cen, cnt) = ctx.labels(), ctx.centres()
    torch.cuda.synchronize()
    rounds = int(n.cpu()[0])
    if squared:  # (the oracle's rule is stated for Eq. 1: the rounds run are taken as given)
        want = oracle.segment(img, S, 10.0, rounds, True, False, 0, oracle.COLOR_LAB,
                              oracle.DIST_SQUARED)
        want = (want["labels"], want["centres"], want["counts"], rounds)
    else:
        want = oracle.kmeans_converge(oracle.rgb_to_lab(img), S, 10.0, True, 12, threshold)
    assert np.array_equal(lb.cpu().numpy(), want[0])
    assert np.array_equal(cen.cpu().numpy(), want[1])
    assert np.array_equal(cnt.cpu().numpy(), want[2])
    assert rounds == want[3]
    ctx.close()


@pytest.mark.parametrize("w,h,S,rounds", [(96, 72, 16, 0), (97, 75, 8, 1), (131, 77, 8, 3), (700, 500, 16, 3)])
def test_given_centres_with_overflowing_distances(slic, w, h, S, rounds):
    """m = 0 and given centres so far out that their spatial distances
    overflow: 0 * inf is no distance, and each pixel keeps its own cell (the
    cells outside the grid are never taken) until the first means."""
    img = _img(w, h, 3 * w)
    lab = oracle.rgb_to_lab(img)
    cen = oracle.kmeans(lab, S, 0.0, True, 0)[1].copy()
    cen[:, 3] = 1e30
    p = slic.Params(w, h, S=S, m=0.0)
    ctx = slic.Context(p, _gpu(img), centres=torch.from_numpy(cen).cuda())
    labels = (np.arange(h)[:, None] // S) * -(-w // S) + np.arange(w)[None] // S
    labels = np.ascontiguousarray(labels, dtype=np.int32)
    for _ in range(rounds):
        cen, _ = oracle.update(lab, labels, cen)
        labels = oracle.assign(lab, S, 0.0, cen)
    ctx.iterate(rounds)
    lb, (got, _) = ctx.labels(), ctx.centres()
    torch.cuda.synchronize()
    assert np.array_equal(lb.cpu().numpy(), labels)
    assert np.array_equal(got.cpu().numpy(), cen)
    ctx.close()
