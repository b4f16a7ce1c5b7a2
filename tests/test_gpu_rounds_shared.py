"""The rounds launch (csrc/rounds.hip) when some of its workgroups start too
late to take part, as on a chip that other streams share, bit for bit against
the oracle.  slic_test_rounds (csrc/slic_internal.h) names those workgroups, so
that every run takes this path; bit b of `absent` stands for the workgroups
b, b + 31, b + 62, ..."""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import synth

pytestmark = pytest.mark.gpu

ABSENT = [0x1, 0x55555555, 0x7FFFFFFD, 0x7FFFFBFE, 0x0]


@pytest.fixture(scope="module")
def slic():
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    import paper_1509_04232_amd as slic
    return slic


def _rounds(slic, ctx, n, absent, threshold=-1.0, polls=0):
    fn = slic._abi.lib.slic_test_rounds
    fn.argtypes = [ctypes.c_void_p, ctypes.c_int32, ctypes.c_uint32, ctypes.c_int32, ctypes.c_float,
                   ctypes.c_void_p]
    done = torch.full((1,), -1, dtype=torch.int32, device="cuda")
    assert fn(ctx.ctx, n, absent, polls, threshold, done.data_ptr()) == slic.SLIC_OK
    return done


def _gpu(img):
    return torch.from_numpy(np.ascontiguousarray(img).reshape(-1)).cuda()


@pytest.fixture
def variant(slic):
    held = []

    def choose(w, h, S, v):
        slic.slic_set_assign_variant(w, h, S, v)
        held.append((w, h, S))
    yield choose
    for key in held:
        slic.slic_set_assign_variant(*key, 0)


SHAPES = [(64, 48, 8, 0), (97, 75, 8, 0), (300, 200, 16, 0), (333, 51, 27, 3), (640, 480, 16, 5),
          (480, 320, 10, 7), (1024, 1024, 8, 5)]


@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("absent", ABSENT)
@pytest.mark.parametrize("w,h,S,v", SHAPES)
def test_rounds_without_all_workgroups(slic, variant, w, h, S, v, absent, squared):
    img = synth.voronoi_image(w + h + S, w, h, max(2, w * h // 900), 8.0)
    dist = oracle.DIST_SQUARED if squared else oracle.DIST_EQ1
    variant(w, h, S, v)
    ctx = slic.Context(slic.Params(w, h, S=S, m=10.0, squared_distance=squared), _gpu(img))
    done = 0
    for n, shared in ((2, True), (3, True), (1, False), (2, False), (4, True)):
        if shared:
            _rounds(slic, ctx, n, absent)
        else:
            ctx.iterate(n)
        done += n
        want = oracle.segment(img, S, 10.0, done, True, False, 0, oracle.COLOR_LAB, dist)
        lb, (cen, cnt) = ctx.labels(), ctx.centres()
        torch.cuda.synchronize()
        assert np.array_equal(lb.cpu().numpy(), want["labels"]), done
        assert np.array_equal(cen.cpu().numpy(), want["centres"]), done
        assert np.array_equal(cnt.cpu().numpy(), want["counts"]), done
    ctx.close()


@pytest.mark.parametrize("threshold", [0.0, 0.3, 1.0, 1e4])
@pytest.mark.parametrize("absent", ABSENT)
@pytest.mark.parametrize("w,h,S,v", SHAPES[:3] + SHAPES[4:5])
def test_convergence_stop_without_all_workgroups(slic, variant, w, h, S, v, absent, threshold):
    img = synth.voronoi_image(3 * w + S, w, h, max(2, w * h // 900), 8.0)
    want = oracle.kmeans_converge(oracle.rgb_to_lab(img), S, 10.0, True, 12, threshold)
    variant(w, h, S, v)
    ctx = slic.Context(slic.Params(w, h, S=S, m=10.0), _gpu(img))
    n = _rounds(slic, ctx, 12, absent, threshold)
    lb, (cen, cnt) = ctx.labels(), ctx.centres()
    torch.cuda.synchronize()
    assert int(n.cpu()[0]) == want[3]
    assert np.array_equal(lb.cpu().numpy(), want[0])
    assert np.array_equal(cen.cpu().numpy(), want[1])
    assert np.array_equal(cnt.cpu().numpy(), want[2])
    ctx.close()


@pytest.mark.parametrize("w,h,S,v,m", [(97, 75, 8, 0, 0.0), (300, 200, 16, 0, 0.0),
                                       (640, 480, 16, 5, 0.0), (480, 320, 10, 7, 0.1)])
def test_clusters_that_empty_after_they_moved(slic, variant, w, h, S, v, m):
    """Noise of three colours: clusters lose their last pixel in the round
    after their centre moved, and keep the centre of that round.  With one
    workgroup in 31 absent, some have two tiles and are half a round behind
    their neighbours."""
    rng = np.random.default_rng(w)
    pal = rng.integers(0, 256, (3, 3), dtype=np.uint8)
    img = pal[rng.integers(0, 3, (h, w))]
    lab = oracle.rgb_to_lab(img)
    cen = oracle.kmeans(lab, S, m, True, 0)[1]
    labels = oracle.assign(lab, S, m, cen)
    moved = np.zeros(len(cen), bool)
    emptied = 0
    for _ in range(6):
        prev = cen
        cen, cnt = oracle.update(lab, labels, prev)
        emptied += int((moved & (cnt == 0)).sum())
        moved = (cen != prev).any(1)
        labels = oracle.assign(lab, S, m, cen)
    assert emptied > 0
    variant(w, h, S, v)
    for absent in [1 << b for b in range(31)] + ABSENT:
        ctx = slic.Context(slic.Params(w, h, S=S, m=m), _gpu(img))
        _rounds(slic, ctx, 6, absent)
        lb, (got, n) = ctx.labels(), ctx.centres()
        torch.cuda.synchronize()
        assert np.array_equal(lb.cpu().numpy(), labels)
        assert np.array_equal(got.cpu().numpy(), cen)
        assert np.array_equal(n.cpu().numpy(), cnt)
        ctx.close()


@pytest.mark.parametrize("squared", [False, True])
@pytest.mark.parametrize("threshold", [-1.0, 0.0])
@pytest.mark.parametrize("absent", [0x0, 0x55555555])
@pytest.mark.parametrize("w,h,S,v", SHAPES[:3] + SHAPES[4:5])
def test_waits_end_without_the_words(slic, variant, w, h, S, v, absent, threshold, squared):
    """A thread that has polled its share goes on with what it has read (words
    are only missing where another call uses the workspace at the same time):
    the launch ends, every label is a cluster, and the frame after it is right."""
    img = synth.voronoi_image(w + S, w, h, max(2, w * h // 900), 8.0)
    p = slic.Params(w, h, S=S, m=10.0, squared_distance=squared)
    variant(w, h, S, v)
    ws = slic.workspace_for(p)
    ctx = slic.Context(p, _gpu(img), workspace=ws)
    _rounds(slic, ctx, 9, absent, threshold, polls=1)
    lb = ctx.labels()
    torch.cuda.synchronize()
    assert 0 <= int(lb.min()) and int(lb.max()) < p.n_clusters
    ctx.close()
    dist = oracle.DIST_SQUARED if squared else oracle.DIST_EQ1
    want = oracle.segment(img, S, 10.0, 3, True, False, 0, oracle.COLOR_LAB, dist)
    ctx = slic.Context(p, _gpu(img), workspace=ws)
    ctx.iterate(3)
    lb = ctx.labels()
    torch.cuda.synchronize()
    assert np.array_equal(lb.cpu().numpy(), want["labels"])
    ctx.close()


@pytest.mark.parametrize("far,threshold,want_rounds", [(1e10, 9e9, 2), (1e10, 2e10, 1), (2.0 ** 33, 1.0, None)])
@pytest.mark.parametrize("absent", ABSENT)
@pytest.mark.parametrize("w,h,S,v", [(97, 75, 8, 0), (300, 200, 16, 0), (333, 51, 27, 3)])
def test_far_given_centres_without_all_workgroups(slic, variant, w, h, S, v, absent, far, threshold,
                                                  want_rounds):
    """Shifts too wide for their words, of tiles that change hands."""
    img = synth.voronoi_image(w + S, w, h, max(2, w * h // 900), 8.0)
    lab = oracle.rgb_to_lab(img)
    cen = oracle.kmeans(lab, S, 10.0, True, 2)[1].copy()
    cen[:, 3] += np.float32(far)
    variant(w, h, S, v)
    ctx = slic.Context(slic.Params(w, h, S=S, m=0.0), _gpu(img), centres=torch.from_numpy(cen).cuda())
    n = _rounds(slic, ctx, 6, absent, threshold)
    limit = int(np.rint(threshold * 2.0 ** 18)) * len(cen)
    labels = oracle.assign(lab, S, 0.0, cen)
    for rounds in range(1, 7):
        prev = cen
        cen, cnt = oracle.update(lab, labels, prev)
        labels = oracle.assign(lab, S, 0.0, cen)
        if oracle.residual(prev, cen) < limit:
            break
    assert want_rounds is None or rounds == want_rounds
    lb, (got, counts) = ctx.labels(), ctx.centres()
    torch.cuda.synchronize()
    assert int(n.cpu()[0]) == rounds
    assert np.array_equal(lb.cpu().numpy(), labels)
    assert np.array_equal(got.cpu().numpy(), cen)
    assert np.array_equal(counts.cpu().numpy(), cnt)
    ctx.close()
