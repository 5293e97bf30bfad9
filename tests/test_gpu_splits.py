"""GPU: work that one workgroup or lane would hold up, split over the chip, and
the forms behind a rule on sizes, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle
from test_point_forms import BOX, POINTS

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _point_backward(pts, sizes, H, W, radius, K, gz=True, gd=True, seed=0):
    """Gradient of the fragments' own ids against the oracle's; with the
    forward's workspace and with a new one."""
    from test_gpu_points import run_pbwd, run_pfwd
    from _util import threads
    from paper_2007_08501_amd import _lib
    rng = np.random.default_rng(seed)
    sizes = np.asarray(sizes, np.int64)
    first = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    N = len(sizes)
    p, f, n = _t(pts), _t(first), _t(sizes)
    idx, _, _, ws = run_pfwd(p, f, n, H, W, radius, K)
    up = [rng.standard_normal((N, H, W, K)).astype(np.float32) if on else None for on in (gz, gd)]
    dev = [None if u is None else _t(u) for u in up]
    got = run_pbwd(p, f, n, H, W, radius, K, idx, *dev, ws, _lib.RAST_BWD_REUSE_FORWARD)
    ws2 = _lib.alloc_workspace(_lib.rast_points_workspace_size(N, H, W, len(pts)), "cuda")
    assert torch.equal(got, run_pbwd(p, f, n, H, W, radius, K, idx, *dev, ws2, 0))
    full = [np.zeros((N, H, W, K), np.float32) if u is None else u for u in up]
    ref = oracle.points_backward(pts, (H, W), idx.cpu().numpy(), *full, nthreads=threads())
    assert (idx >= 0).sum() > 0 and np.abs(ref).max() > 0
    # (FP64 sums, rounded once)
    assert np.abs(got.cpu().numpy() - ref).max() <= 1e-6 * np.abs(ref).max()


def _in_tile(rng, m, H, W, tx, ty):
    """m points whose one-pixel discs start in tile (tx, ty): pixel columns and rows 1 to 6 of it."""
    c = rng.uniform(8 * tx + 1.5, 8 * tx + 6.5, m)
    r = rng.uniform(8 * ty + 1.5, 8 * ty + 6.5, m)
    return np.c_[1 - 2 * c / W, 1 - 2 * r / H, rng.uniform(0.5, 3, m)].astype(np.float32)


# Tiles of more points than a chunk holds (512 for the 9 cells here): exactly
# a chunk, one point more, several chunks, beside tiles of one chunk and none.
@pytest.mark.parametrize("counts", [[512], [513], [1024, 1, 511], [3000, 700, 513, 40], [512, 512, 5000]])
def test_point_backward_tiles_of_several_chunks(counts):
    rng = np.random.default_rng(sum(counts))
    H, W, K = 64, 64, 40
    pts = np.concatenate([_in_tile(rng, m, H, W, 1 + 2 * i, 1 + i) for i, m in enumerate(counts)])
    _point_backward(pts, [len(pts)], H, W, float(np.float32(2.0 / W)), K)


# More than 256 tiles of several chunks (256 points for discs of 14 pixels a
# side, 128 for 20), so that their chunks are summed in several turns, and more
# chunks than workgroups; several images, one without points.
@pytest.mark.parametrize("rpx,K", [(13.0, 2), (19.0, 1)])
def test_point_backward_many_tiles_of_several_chunks(rpx, K):
    rng = np.random.default_rng(int(rpx))
    H = W = 104
    sizes = [60000, 0, 70000, 50000]
    n = sum(sizes)
    pts = np.c_[rng.uniform(-0.99, 0.99, (n, 2)), rng.uniform(0.5, 3, n)].astype(np.float32)
    _point_backward(pts, sizes, H, W, float(np.float32(rpx / W)), K)


# The per-face backward takes four lanes a face from 16,384 faces with fewer than
# two pixels each, with two faces a group of lanes in turn from 131,072, else
# sixteen: a face fewer, exactly as many, part workgroups, boxes of a few pixels
# and (the coarse mesh beside the fine one) of more than 256.  The suite's
# gradient bound.
@pytest.mark.parametrize("faces,n,image,K", [(16383, 1, 24, 4), (16384, 1, 24, 3), (16384, 1, 160, 3),
                                             (70001, 1, 40, 5), (131072, 2, 20, 2), (150003, 2, 33, 4)])
def test_per_face_backward_lanes(faces, n, image, K):
    from _util import compare_grad, run_bwd, threads, tie_masked_grads
    from paper_2007_08501_amd import meshgen
    b = meshgen.make_config(2, n_override=n + 1, level_override=6, image_override=image)
    coarse = meshgen.make_config(2, n_override=1, level_override=0)
    per = b.num_faces[0]
    count = np.array([min(per, faces - 20 - i * per) for i in range(n)] + [20], np.int64)
    first = np.concatenate([[0], np.cumsum(count)[:-1]])
    b.faces = np.concatenate([b.faces[i * per:i * per + count[i]] for i in range(n)]
                             + [coarse.faces + len(b.verts)]).astype(b.faces.dtype)
    b.verts = np.concatenate([b.verts, coarse.verts]).astype(np.float32)
    b.first_idx, b.num_faces, b.faces_per_pixel = first, count, K
    assert len(b.faces) == faces
    o = oracle.rasterize(b.verts, b.faces, b.first_idx, b.num_faces, b.image_size, b.blur_radius, K,
                         nthreads=threads())
    g = tie_masked_grads(b, o["p2f"], *meshgen.upstream_grads(b))
    ref = oracle.backward(b.verts, b.faces, b.image_size, o["p2f"], *g)
    assert (o["p2f"] >= faces - 20).any()
    got = run_bwd(b, _t(o["p2f"].astype(np.int32)), *g, bs=0)
    compare_grad(got.cpu().numpy(), ref, f"{faces} faces")


# The vertex table of the backward's face sums (1,024 entries, the faces of a
# workgroup): 768 vertices of their own per 256 faces, their ids scattered over
# a large range, in runs of sixteen, in part runs that start the same bucket, and
# all alike in their low bits.  The suite's gradient bound.
@pytest.mark.parametrize("bs", [0, 8])
@pytest.mark.parametrize("ids", ["scattered", "runs", "part", "strided"])
def test_backward_vertex_table(ids, bs):
    from _util import compare_grad, run_bwd, threads, tie_masked_grads
    from paper_2007_08501_amd import meshgen
    rng = np.random.default_rng(len(ids))
    F, V, H, W, K = 800, 60000, 30, 44, 6
    n = 3 * F
    if ids == "scattered":
        at = rng.permutation(V)[:n]
    elif ids == "strided":
        at = 16 * rng.permutation(n)
    else:
        m = 16 if ids == "runs" else 5
        at = (16 * rng.permutation(V // 16)[:-(-n // m), None] + np.arange(m)).ravel()[:n]
    xy = rng.uniform(-1, 1, (F, 1, 2)) + 10.0 ** rng.uniform(-1.5, -0.3, (F, 1, 1)) * rng.uniform(-1, 1, (F, 3, 2))
    v = np.zeros((V, 3), np.float32)
    v[at] = np.concatenate([xy.reshape(-1, 2), rng.uniform(1, 5, (n, 1))], 1)
    b = meshgen.Batch(name="table", verts=v, faces=at.reshape(F, 3).astype(np.int32), first_idx=np.array([0]),
                      num_faces=np.array([F]), verts_first_idx=np.array([0]), num_verts=np.array([V]),
                      image_size=(H, W), faces_per_pixel=K, blur_radius=float(np.float32(1e-4)), bin_size=8,
                      max_faces_per_bin=None)
    o = oracle.rasterize(b.verts, b.faces, b.first_idx, b.num_faces, b.image_size, b.blur_radius, K,
                         nthreads=threads())
    g = tie_masked_grads(b, o["p2f"], *meshgen.upstream_grads(b, seed=3))
    ref = oracle.backward(b.verts, b.faces, b.image_size, o["p2f"], *g)
    got = run_bwd(b, _t(o["p2f"].astype(np.int32)), *g, bs=bs)
    compare_grad(got.cpu().numpy(), ref, ids)


# The silhouette blend's backward with one to four slots a pixel, where a lane
# skips the slots that no pixel has: holes, empty pixels, deep inside and far
# outside, part waves.  The bounds of the same blend's other sizes.
@pytest.mark.parametrize("K", [1, 2, 3, 4])
@pytest.mark.parametrize("P", [1, 64, 127, 128, 129, 1000])
def test_silhouette_few_slots(K, P):
    import test_gpu_paths
    test_gpu_paths.test_silhouette_lane_groups(K, P)


# The softmax blend's instance of two channels, with the bounds of the others.
@pytest.mark.parametrize("K,P", [(1, 1), (1, 67), (2, 64), (3, 65), (4, 130), (9, 17), (17, 9), (64, 5)])
def test_softmax_two_channels(K, P):
    import test_gpu_paths
    test_gpu_paths.test_softmax_lane_groups(K, P, 2)


# The point pass's prefixes of a long queue: every pixel holds exactly `hits`
# points, over several batches of candidates in arbitrary order, around eight,
# sixteen and thirty-two keys in queues of 16, 32 and 64.  Fragments are exact.
@pytest.mark.parametrize("K", [16, 17, 32, 33, 64])
@pytest.mark.parametrize("hits", [1, 7, 8, 9, 15, 17, 32, 33, 70])
def test_point_queue_prefixes(hits, K):
    from test_gpu_points import check_case
    rng = np.random.default_rng(100 * hits + K)
    H, W = 16, 24
    c, r = (x.ravel() for x in np.meshgrid(np.arange(W), np.arange(H)))
    at = np.c_[1 - (2 * c + 1) / W, 1 - (2 * r + 1) / H]
    pts = np.repeat(at, hits, 0) + rng.uniform(-0.01, 0.01, (hits * H * W, 2))
    pts = np.c_[pts, rng.uniform(0.5, 3, len(pts))][rng.permutation(len(pts))].astype(np.float32)
    check_case(pts, np.array([0]), np.array([len(pts)]), H, W, 0.03, K, f"{hits} hits")


# The point backward's forms for large discs, each reached by the rule
# (test_point_forms.py evaluates it for these sizes), one gradient or both.
@pytest.mark.parametrize("H,W,K,sizes,radius,gz,gd", BOX + POINTS)
def test_point_backward_large_discs(H, W, K, sizes, radius, gz, gd):
    rng = np.random.default_rng(H + W + K)
    n = sum(sizes)
    pts = np.c_[rng.uniform(-0.95, 0.95, (n, 2)), rng.uniform(0.5, 3, n)].astype(np.float32)
    _point_backward(pts, sizes, H, W, float(np.float32(radius)), K, gz, gd)


# Scan and tile order of the points in one workgroup up to 15,360 tiles in all,
# else in six launches; counts in LDS up to 16,384 tiles, else by one global
# atomic a point.  At each limit and past it, with one cloud and with several,
# an empty one among them.  Fragments are exact.
@pytest.mark.parametrize("H,W,sizes", [(960, 1024, [150]), (640, 768, [100, 80]), (568, 568, [70, 0, 90]),
                                       (576, 576, [90, 0, 60]), (512, 512, [60, 0, 80, 30]), (1024, 1024, [150]),
                                       (1024, 1032, [120]), (960, 1024, [150, 0, 90])])
def test_point_sort_limits(H, W, sizes):
    from test_gpu_points import check_case
    rng = np.random.default_rng(H + len(sizes))
    n = sum(sizes)
    pts = np.c_[rng.uniform(-0.95, 0.95, (n, 2)), rng.uniform(0.5, 3, n)].astype(np.float32)
    first = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    o = check_case(pts, first, np.array(sizes, dtype=np.int64), H, W, 0.02, 2, f"{H}x{W}")
    assert (o["idx"] >= 0).any()


# Crowded cells with K above 16, whose slots do not fit a workgroup's registers:
# a cell that names more than 160 faces (a chunk), or more than its table
# holds, is read again through its bin's list, also where the bin is larger
# than the cell.  The suite's gradient bound.
@pytest.mark.parametrize("F,K,bs", [(1500, 24, 8), (4000, 24, 16), (4000, 64, 8), (1500, 64, 16), (6000, 64, 24)])
def test_crowded_cells_of_long_queues(F, K, bs):
    from test_gpu_parity import crowded_batch
    from _util import compare_grad, run_bwd, threads, tie_masked_grads
    from paper_2007_08501_amd import meshgen
    b = crowded_batch(F, seed=F + K, size=24, K=K)
    p2f = oracle.rasterize(b.verts, b.faces, b.first_idx, b.num_faces, b.image_size, b.blur_radius, K,
                           nthreads=threads())["p2f"]
    cells = p2f.reshape(3, 8, 3, 8, K).transpose(0, 2, 1, 3, 4).reshape(9, -1)
    assert max(len(np.unique(c[c >= 0])) for c in cells) > 160
    g = tie_masked_grads(b, p2f, *meshgen.upstream_grads(b))
    ref = oracle.backward(b.verts, b.faces, b.image_size, p2f, *g, nthreads=threads())
    got = run_bwd(b, _t(p2f.astype(np.int32)), *g, bs=bs)
    compare_grad(got.cpu().numpy(), ref, f"F {F} K {K} bins {bs}")


# Bins that the backward's cells do not divide (odd multiples of 8: cells of 16
# or 32 pixels touch up to four bins), on images that cut bins and cells; empty
# bins beside filled ones.  The suite's gradient bound, and the same gradient
# as with bins of 8 up to the order of the sums.
@pytest.mark.parametrize("bs,K,level,image", [(24, 1, 3, (77, 50)), (24, 3, 2, (100, 130)), (24, 8, 3, (61, 90)),
                                              (24, 16, 3, (45, 61)), (40, 1, 1, (130, 90)), (40, 2, 3, (83, 125)),
                                              (40, 8, 2, (90, 41)), (56, 1, 3, (120, 70))])
def test_cells_that_cross_bins(bs, K, level, image):
    from _util import compare_grad, run_bwd, threads, tie_masked_grads
    from paper_2007_08501_amd import meshgen
    b = meshgen.make_config(2, n_override=3, level_override=level)
    b.verts = b.verts.copy()
    b.verts[:, :2] *= 0.6  # (leaves the outer bins empty)
    b.image_size, b.faces_per_pixel = image, K
    o = oracle.rasterize(b.verts, b.faces, b.first_idx, b.num_faces, b.image_size, b.blur_radius, K,
                         nthreads=threads())
    g = tie_masked_grads(b, o["p2f"], *meshgen.upstream_grads(b))
    ref = oracle.backward(b.verts, b.faces, b.image_size, o["p2f"], *g)
    p2f = _t(o["p2f"].astype(np.int32))
    got = run_bwd(b, p2f, *g, bs=bs).cpu().numpy()
    compare_grad(got, ref, f"bins {bs} K {K}")
    other = run_bwd(b, p2f, *g, bs=8).cpu().numpy()
    assert np.abs(got - other).max() <= 1e-5 * np.abs(ref).max()


# The same with cells that name more than 160 faces, read again through the
# lists of all their bins: a face in several of them counts once.
@pytest.mark.parametrize("F,K,bs", [(2500, 8, 24), (6000, 8, 24), (1200, 2, 40), (9000, 3, 24)])
def test_crowded_cells_that_cross_bins(F, K, bs):
    from test_gpu_parity import crowded_batch
    from _util import compare_grad, run_bwd, threads, tie_masked_grads
    from paper_2007_08501_amd import meshgen
    b = crowded_batch(F, seed=F + K, size=48, K=K)
    p2f = oracle.rasterize(b.verts, b.faces, b.first_idx, b.num_faces, b.image_size, b.blur_radius, K,
                           nthreads=threads())["p2f"]
    h, w = {8: (8, 16), 3: (16, 16), 2: (16, 32)}[K]
    cells = [p2f[0, r:r + h, c:c + w] for r in range(0, 48, h) for c in range(0, 48, w)]
    assert max(len(np.unique(c[c >= 0])) for c in cells) > 160
    g = tie_masked_grads(b, p2f, *meshgen.upstream_grads(b))
    ref = oracle.backward(b.verts, b.faces, b.image_size, p2f, *g, nthreads=threads())
    got = run_bwd(b, _t(p2f.astype(np.int32)), *g, bs=bs)
    compare_grad(got.cpu().numpy(), ref, f"F {F} K {K} bins {bs}")


# The backward's rows of sums per face: eight up to K = 3, four to 7, two to 15,
# then one, and fewer where a cell names many faces.  Few large faces (every
# lane of a wave names the same) and many small ones; the suite's gradient bound.
@pytest.mark.parametrize("K", [3, 4, 7, 8, 15, 16, 17])
@pytest.mark.parametrize("level", [0, 3])
@pytest.mark.parametrize("options", [0, 0x300])
def test_rows_of_sums(K, level, options):
    from _util import compare_grad, run_bwd, run_fwd, to_dev
    from paper_2007_08501_amd import meshgen
    b = meshgen.make_config(2, n_override=2, level_override=level)
    b.image_size, b.faces_per_pixel = (50, 70), K
    d = to_dev(b)
    out, _ = run_fwd(b, 16, dev_inputs=d, options=options)
    g = [_t(x) for x in meshgen.upstream_grads(b)]
    per_face = run_bwd(b, out.pix_to_face, *g, dev_inputs=d, bs=0, flags=options)
    for bs in (8, 16, 32):
        got = run_bwd(b, out.pix_to_face, *g, dev_inputs=d, bs=bs, flags=options)
        compare_grad(got.cpu().numpy(), per_face.cpu().numpy(), f"bins {bs}")


# Compositing where nearly all slots are empty: waves and spans of pixels without
# any, spans with one point, more spans than workgroups (a workgroup's table is
# clear again for its next one), and a last part span.  The bound of the feature
# gradients elsewhere; opacity gradients are zero at empty slots.
@pytest.mark.parametrize("K,D,npix,filled", [(4, 3, 9_000_001, 4000), (16, 2, 300_001, 700), (50, 8, 50_003, 90),
                                             (64, 1, 4099, 1)])
@pytest.mark.parametrize("norm", [False, True])
def test_compositing_of_nearly_empty_slots(K, D, npix, filled, norm):
    from paper_2007_08501_amd.points import alpha_composite, norm_composite
    rng = np.random.default_rng(K + D)
    P = 500
    rows = np.unique(np.concatenate([rng.integers(0, npix, filled), [0, npix - 1]]))
    sub = np.full((len(rows), K), -1, np.int32)
    n = rng.integers(1, min(K, 4) + 1, len(rows))
    for i, m in enumerate(n):
        sub[i, :m] = rng.integers(0, P, m)
    al = rng.uniform(0.1, 0.9, sub.shape).astype(np.float32)
    f = rng.uniform(-1, 1, (P, D)).astype(np.float32)
    g = rng.standard_normal((len(rows), D)).astype(np.float32)
    idx = torch.full((npix, K), -1, dtype=torch.int32, device="cuda")
    w = torch.zeros((npix, K), device="cuda")
    up = torch.randn((npix, D), device="cuda")
    at = _t(rows)
    idx[at], w[at], up[at] = _t(sub), _t(al), _t(g)
    ft, wt = _t(f).requires_grad_(True), w.requires_grad_(True)
    img = (norm_composite if norm else alpha_composite)(idx, wt, ft)
    gw, gf = torch.autograd.grad(img, (wt, ft), up)
    args = sub, al.astype(np.float64), f.astype(np.float64)
    ref = (oracle.norm_composite if norm else oracle.alpha_composite)(*args)
    back = oracle.norm_composite_backward if norm else oracle.alpha_composite_backward
    rw, rf = back(*args, g)
    _, size = back(*args, np.abs(g))
    assert np.abs(img.detach()[at].cpu().numpy() - ref).max() <= 1e-5
    assert (np.abs(gf.cpu().numpy() - rf) <= 8e-6 * np.abs(size) + 1e-30).all()
    assert np.abs(gw[at].cpu().numpy() - rw).max() <= 1e-5 * np.abs(rw).max()
    assert (gw[idx < 0] == 0).all() and int((img.detach() != 0).any(-1).sum()) <= len(rows)
