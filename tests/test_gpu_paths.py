"""GPU: the edges of the kernels' own splits -- lane groups, tiles, batches,
tables and their remainders -- against the FP64 oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


# One lane holds four slots, 1..16 lanes a pixel, 64 / lanes pixels a wave:
# K around every multiple of the group size, pixel counts that leave a part
# wave, every channel count with an instance of its own and the general ones.
# Bounds: sums of at most 64 FP32 terms of size <= 1 are within 64 ulps
# (4e-6) of the largest, the image within 1e-5.  The depth and distance
# gradients are G w / W times a scale, where G = sum_c g_c (c - image) is a
# difference of terms of size max |g|, which may cancel entirely (one slot:
# exactly zero): their error is absolute in those terms, C max |g| times 32
# ulps (2e-6), times the scale 1 / sigma or 1 / ((zfar - znear) gamma).
@pytest.mark.parametrize("K,P,C", [(1, 1, 1), (1, 67, 3), (3, 65, 4), (4, 64, 3), (5, 33, 3), (8, 31, 2), (8, 129, 8),
                                   (9, 17, 4), (16, 70, 1), (17, 9, 3), (33, 5, 5), (50, 7, 3), (64, 6, 3),
                                   (64, 5, 7)])
def test_softmax_lane_groups(K, P, C):
    from paper_2007_08501_amd.raster import softmax_blend
    rng = np.random.default_rng(1000 * K + 10 * P + C)
    cnt = rng.integers(0, K + 1, size=(P, 1))
    on = np.arange(K)[None] < cnt
    on[:, 1:] &= rng.uniform(size=(P, K - 1)) < 0.9  # holes are honoured too
    p2f = np.where(on, rng.integers(0, 50, (P, K)), -1).astype(np.int32)
    z = np.where(on, rng.uniform(1, 3, (P, K)), -1).astype(np.float32)
    d = np.where(on, rng.standard_normal((P, K)) * 1e-4, -1).astype(np.float32)
    col = rng.uniform(size=(P, K, C)).astype(np.float32)
    g = rng.standard_normal((P, C)).astype(np.float32)
    prm = dict(sigma=1e-4, gamma=1e-2, znear=1.0, zfar=100.0)
    f64 = [a.astype(np.float64) for a in (z, d, col)]
    ref = oracle.softmax_blend(p2f, *f64, **prm)
    refs = oracle.softmax_blend_backward(p2f, *f64, **prm, grad_image=g)
    zt, dt, ct = (_t(a).requires_grad_(True) for a in (z, d, col))
    img = softmax_blend(_t(p2f), zt, dt, ct, **prm)
    assert np.abs(img.detach().cpu().numpy() - ref).max() <= 1e-5
    got = torch.autograd.grad(img, (zt, dt, ct), _t(g))
    gmax = float(np.abs(g).max())
    tol = (2e-6 * C * gmax / (99.0 * 1e-2), 2e-6 * C * gmax / 1e-4, 1e-5 * gmax)
    for x, r, e in zip(got, refs, tol):
        assert np.abs(x.cpu().numpy() - r).max() <= e


# The per-face backward: sixteen lanes a face, sixteen faces a workgroup at a
# time, more of them in turn above 16,384 faces, boxes above 256 pixels in
# the cooperative kernel.  Levels 0 and 1 mix both at this size; two spheres of
# level 5 (40,960 faces) take two faces in turn.  The suite's gradient bound.
@pytest.mark.parametrize("level,n,image,K", [(0, 1, 33, 3), (0, 3, 40, 4), (1, 2, 45, 7), (3, 3, 37, 5), (5, 2, 24, 8)])
def test_per_face_backward_splits(level, n, image, K):
    from _util import compare_grad, run_bwd, threads, tie_masked_grads
    from paper_2007_08501_amd import meshgen
    b = meshgen.make_config(2, n_override=n, level_override=level, image_override=image)
    b.faces_per_pixel = K
    o = oracle.rasterize(b.verts, b.faces, b.first_idx, b.num_faces, b.image_size, b.blur_radius, K,
                         nthreads=threads())
    g = tie_masked_grads(b, o["p2f"], *meshgen.upstream_grads(b))
    ref = oracle.backward(b.verts, b.faces, b.image_size, o["p2f"], *g)
    got = run_bwd(b, _t(o["p2f"].astype(np.int32)), *g, bs=0)
    compare_grad(got.cpu().numpy(), ref, f"level {level}")


# The binned backward's cells: 8, 16 or 32 pixels a side by the slots they
# hold and the bins they divide (24-pixel bins only by 8), cut by the image's
# edges; K above 16 reads its ids again; faces over more than four cells go to
# the vertices.  Coarse meshes for the latter, finer ones for partial rows.
@pytest.mark.parametrize("bs,K,level,image", [(8, 1, 2, (45, 61)), (8, 16, 3, (45, 61)), (8, 20, 3, (29, 43)),
                                              (16, 3, 1, (77, 50)), (16, 8, 3, (50, 77)), (24, 5, 2, (61, 45)),
                                              (32, 1, 2, (70, 100)), (32, 2, 3, (100, 70)), (32, 4, 1, (66, 65)),
                                              (64, 4, 3, (66, 65)), (16, 33, 2, (33, 50)), (32, 64, 3, (40, 33))])
def test_binned_backward_cells(bs, K, level, image):
    from _util import compare_grad, run_bwd, threads, tie_masked_grads
    from paper_2007_08501_amd import meshgen
    b = meshgen.make_config(2, n_override=3, level_override=level)
    b.image_size, b.faces_per_pixel = image, K
    o = oracle.rasterize(b.verts, b.faces, b.first_idx, b.num_faces, b.image_size, b.blur_radius, K,
                         nthreads=threads())
    g = tie_masked_grads(b, o["p2f"], *meshgen.upstream_grads(b))
    ref = oracle.backward(b.verts, b.faces, b.image_size, o["p2f"], *g)
    got = run_bwd(b, _t(o["p2f"].astype(np.int32)), *g, bs=bs)
    compare_grad(got.cpu().numpy(), ref, f"bins {bs} K {K}")


# Upstream gradients over 40 orders of magnitude (sums in FP64 have no grid and
# no range): the gradient is linear in them.
@pytest.mark.parametrize("scale", [1e-30, 1e-12, 1e12, 1e20])
def test_binned_backward_any_scale(scale):
    from _util import run_bwd, run_fwd, to_dev
    from paper_2007_08501_amd import meshgen
    b = meshgen.make_config(2, n_override=2, level_override=3, image_override=48)
    d = to_dev(b)
    out, _ = run_fwd(b, 8, dev_inputs=d)
    g = [_t(x) for x in meshgen.upstream_grads(b)]
    one = run_bwd(b, out.pix_to_face, *g, dev_inputs=d, bs=8)
    s = float(np.float32(scale))
    got = run_bwd(b, out.pix_to_face, *(x * s for x in g), dev_inputs=d, bs=8)
    # each side within a few ulps per added term: a few hundred terms a vertex
    assert ((got.double() / s - one.double()).abs().max() <= 1e-4 * one.abs().max()).item()


# Feature gradients: a span of pixels per workgroup, its points in an LDS table
# (1,024 entries for up to four channels, 512 above), points without a place
# added directly.  Few points (every span names the same ones), about as many as
# a span names, and many more than the table holds; K and pixel counts that
# leave part spans.  A term is a product of at most 64 factors and one add:
# 130 roundings of 2^-24 of the sum of the terms' sizes.
@pytest.mark.parametrize("norm", [False, True])
@pytest.mark.parametrize("K,D,P,npix", [(1, 1, 3, 5), (1, 3, 5000, 4099), (5, 8, 40, 700), (8, 5, 3000, 1025),
                                        (16, 3, 100000, 2050), (17, 4, 9, 130), (50, 2, 2000, 97),
                                        (64, 8, 100000, 200)])
def test_feature_gradient_table(K, D, P, npix, norm):
    from paper_2007_08501_amd.points import alpha_composite, norm_composite
    rng = np.random.default_rng(K * 100 + D)
    idx = rng.integers(0, P, (npix, K)).astype(np.int32)
    idx[rng.uniform(size=idx.shape) < 0.2] = -1
    al = rng.uniform(0, 1, (npix, K)).astype(np.float32)
    f = rng.uniform(-1, 1, (P, D)).astype(np.float32)
    g = rng.standard_normal((npix, D)).astype(np.float32)
    back = oracle.norm_composite_backward if norm else oracle.alpha_composite_backward
    _, ref = back(idx, al.astype(np.float64), f.astype(np.float64), g)
    _, size = back(idx, al.astype(np.float64), f.astype(np.float64), np.abs(g))
    ft = _t(f).requires_grad_(True)
    img = (norm_composite if norm else alpha_composite)(_t(idx), _t(al), ft)
    got, = torch.autograd.grad(img, (ft,), _t(g))
    assert (np.abs(got.cpu().numpy() - ref) <= 8e-6 * np.abs(size) + 1e-30).all()


# The slot-major point backward for pixel ranges of one pixel to 21 a side and
# the forms behind it, on an image whose sides differ, with chunks (all points
# homed in few tiles) and without.  The sums are FP64, rounded once.
@pytest.mark.parametrize("radius,n_pts,spread", [(0.005, 300, 0.9), (0.04, 2000, 0.9), (0.09, 3000, 0.05),
                                                 (0.16, 500, 0.9), (0.3, 300, 0.9), (0.44, 200, 0.5),
                                                 (0.6, 100, 0.9)])
def test_point_backward_ranges(radius, n_pts, spread):
    from test_gpu_points import oracle_pfwd, run_pbwd, run_pfwd
    from _util import threads
    from paper_2007_08501_amd import _lib
    rng = np.random.default_rng(int(1000 * radius))
    H, W, K = 43, 70, 6
    pts = np.c_[rng.uniform(-spread, spread, (n_pts, 2)), rng.uniform(0.5, 3, n_pts)].astype(np.float32)
    radius = float(np.float32(radius))
    p, f = _t(pts), torch.zeros(1, dtype=torch.int64, device="cuda")
    n = torch.full((1,), n_pts, dtype=torch.int64, device="cuda")
    idx, _, _, ws = run_pfwd(p, f, n, H, W, radius, K)
    gz, gd = (rng.standard_normal((1, H, W, K)).astype(np.float32) for _ in range(2))
    got = run_pbwd(p, f, n, H, W, radius, K, idx, _t(gz), _t(gd), ws, _lib.RAST_BWD_REUSE_FORWARD)
    o = oracle_pfwd(pts, [0], [n_pts], H, W, radius, K)
    np.testing.assert_array_equal(idx.cpu().numpy(), o["idx"])
    ref = oracle.points_backward(pts, (H, W), o["idx"], gz, gd, nthreads=threads())
    assert np.abs(got.cpu().numpy() - ref).max() <= 1e-6 * np.abs(ref).max()


# Scan and tile order in one workgroup up to 15,360 tiles, in six launches
# above; several clouds, so that a counting block spans images (or, with an
# empty one between, skips them).  Fragments are exact.
@pytest.mark.parametrize("H,W,sizes", [(8, 8, [3]), (960, 1024, [150, 0, 90]), (968, 1024, [150]),
                                       (70, 41, [20000, 0, 1, 9000, 500])])
def test_point_sort_sizes(H, W, sizes):
    from test_gpu_points import check_case
    if H > 900:
        H, W, sizes = H, W, [sum(sizes)] if len(sizes) == 1 else [sizes[0]]
    rng = np.random.default_rng(H)
    n = sum(sizes)
    pts = np.c_[rng.uniform(-0.95, 0.95, (n, 2)), rng.uniform(0.5, 3, n)].astype(np.float32)
    first = np.concatenate([[0], np.cumsum(sizes)[:-1]]).astype(np.int64)
    check_case(pts, first, np.array(sizes, dtype=np.int64), H, W, 0.02, 2, f"{H}x{W}")


# An output without a gradient reaches the backward as None: the same gradient
# as with zeros (up to the order of the float atomics, a few ulps of the sums).
@pytest.mark.parametrize("bs", [0, 8])
@pytest.mark.parametrize("which", [0, 1, 2])
def test_missing_upstream_gradients_are_zeros(which, bs):
    from _util import run_bwd, to_dev
    from paper_2007_08501_amd import meshgen
    from paper_2007_08501_amd.raster import RasterSettings, rasterize_meshes
    b = meshgen.make_config(2, n_override=2, level_override=3, image_override=40)
    v, f, fi, nf = to_dev(b)
    v.requires_grad_(True)
    fr = rasterize_meshes(v, f, fi, nf, RasterSettings(image_size=40, blur_radius=b.blur_radius, faces_per_pixel=4,
                                                       bin_size=bs))
    g = [_t(x) for x in meshgen.upstream_grads(b)]
    got, = torch.autograd.grad((fr.zbuf, fr.bary, fr.dists)[which], (v,), g[which])
    full = [x if i == which else torch.zeros_like(x) for i, x in enumerate(g)]
    ref = run_bwd(b, fr.pix_to_face, *full, dev_inputs=(v.detach(), f, fi, nf), bs=bs)
    assert (got - ref).abs().max() <= 1e-5 * ref.abs().max()


def test_missing_point_gradients_are_zeros():
    from test_gpu_points import dev_cloud, run_pbwd, run_pfwd
    from paper_2007_08501_amd import meshgen
    from paper_2007_08501_amd.points import PointsRasterSettings, rasterize_points
    b = meshgen.make_points_config(1)
    H, W = b.image_size
    p, f, n = dev_cloud(b)
    idx, _, _, ws = run_pfwd(p, f, n, H, W, b.radius, 4)
    g = torch.randn((1, H, W, 4), device="cuda")
    p.requires_grad_(True)
    fr = rasterize_points(p, f, n, PointsRasterSettings(image_size=(H, W), radius=b.radius, points_per_pixel=4))
    for which in (1, 2):
        got, = torch.autograd.grad(fr[which], (p,), g, retain_graph=True)
        gz, gd = (g, torch.zeros_like(g)) if which == 1 else (torch.zeros_like(g), g)
        ref = run_pbwd(p.detach(), f, n, H, W, b.radius, 4, idx, gz, gd, ws)
        assert torch.equal(got, ref)


# The silhouette blend: four slots a lane, 1..16 lanes a pixel, two groups of
# pixels a wave, the last ones with bounds checks.  sigmoid(x) carries
# |x| 1.2e-7 (two roundings of x) and 6e-7 (its own operations) relative, so a
# product over slots S carries e(S) = sum_S (1.2e-7 |x| + 7e-7) and alpha that
# times the product and one rounding; a gradient carries the pixel's e(S)
# twice (its own factor and prob_k) relative, and an underflow of a factor.
@pytest.mark.parametrize("K,P", [(1, 1), (1, 127), (1, 129), (2, 300), (3, 64), (4, 63), (5, 65), (8, 131), (13, 33),
                                 (16, 32), (17, 15), (33, 9), (50, 8), (50, 77), (64, 1), (64, 24)])
def test_silhouette_lane_groups(K, P):
    from paper_2007_08501_amd.raster import silhouette_blend
    rng = np.random.default_rng(100 * K + P)
    on = (rng.uniform(size=(P, K)) < 0.7) & (rng.uniform(size=(P, 1)) < 0.7)  # holes and empty pixels
    sigma = 1e-4
    p2f = np.where(on, rng.integers(0, 50, (P, K)), -1).astype(np.int32)
    d = np.where(on, rng.uniform(-8, 8, (P, K)) * sigma, -1).astype(np.float32)
    ga = rng.standard_normal(P).astype(np.float32)
    d64 = d.astype(np.float64)
    ref, refg = oracle.silhouette_blend(p2f, d64, sigma), oracle.silhouette_blend_backward(p2f, d64, sigma, ga)
    e = np.where(on, 1.2e-7 * np.abs(d64 / sigma) + 7e-7, 0.0).sum(-1)
    dt = _t(d).requires_grad_(True)
    alpha = silhouette_blend(_t(p2f), dt, sigma)
    assert (np.abs(alpha.detach().cpu().numpy() - ref) <= (1 - ref) * e + 1.2e-7).all()
    gd = torch.autograd.grad(alpha, dt, _t(ga))[0].cpu().numpy()
    assert (np.abs(gd - refg) <= np.abs(refg) * (2 * e + 1e-6)[:, None] + 1e-30).all()
    assert (gd[~on] == 0).all()


# The fine pass's pixel ranges and edge masks: loose triangles of every size,
# thin ones, edges along the axes, vertices far off the screen, images smaller
# than a tile or cut by one, no blur and a wide one, more than 64 faces a tile
# (a block of records).  Against the oracle, and all bin sizes bit for bit.
@pytest.mark.parametrize("H,W,blur,K,F", [(1, 1, 0.0, 3, 40), (5, 3, 1e-3, 2, 60), (9, 70, 0.0, 24, 300),
                                          (64, 8, 1e-4, 5, 200), (37, 53, 2e-2, 6, 150), (40, 24, 0.0, 64, 900)])
def test_fine_pass_edges(H, W, blur, K, F):
    from _util import compare_fwd, frag_numpy, run_fwd, threads
    from paper_2007_08501_amd import meshgen
    rng = np.random.default_rng(H * 100 + W)
    size = 10.0 ** rng.uniform(-1.5, 0.5, (F, 1, 1))
    xy = rng.uniform(-1.1, 1.1, (F, 1, 2)) + size * rng.uniform(-1, 1, (F, 3, 2))
    xy[0::7, 1, 0] = xy[0::7, 0, 0]            # an edge along y
    xy[1::7, 2, 1] = xy[1::7, 0, 1]            # an edge along x
    t = rng.uniform(0, 1, (len(xy[2::7]), 1))  # thin: the third vertex near the first edge
    xy[2::7, 2] = xy[2::7, 0] * t + xy[2::7, 1] * (1 - t) + 0.01
    xy[3::7, 1] *= 6.0                         # a vertex off the screen
    v = np.concatenate([xy.reshape(-1, 2), rng.uniform(1, 5, (3 * F, 1))], 1).astype(np.float32)
    nf = np.array([F // 3, F - F // 3])
    b = meshgen.Batch(name="edges", verts=v, faces=np.arange(3 * F, dtype=np.int32).reshape(F, 3),
                      first_idx=np.array([0, F // 3]), num_faces=nf, verts_first_idx=np.array([0, F]),
                      num_verts=3 * nf, image_size=(H, W), faces_per_pixel=K, blur_radius=float(np.float32(blur)),
                      bin_size=8, max_faces_per_bin=None)
    naive, _ = run_fwd(b, 0)
    o = oracle.rasterize(b.verts, b.faces, b.first_idx, b.num_faces, b.image_size, b.blur_radius, K,
                         nthreads=threads())
    compare_fwd(frag_numpy(naive), o, b, f"{H}x{W}")
    for bs in (8, 16, 24):
        for x, y in zip(naive, run_fwd(b, bs)[0]):
            assert torch.equal(x, y)
