"""Filter 3 with every number of kept candidates: images of few distinct
values, where each pixel leaves out between none and all of its neighbours,
against the FP64 oracle.  FD gradients, whose one line per axis vanishes only
for equal raw values, so that no pixel is ill-conditioned.  The bar is the
library's own: FP32 output within 0.01 deg mean and 0.1 deg maximum."""
import numpy as np
import pytest
import torch

import oracle
from paper_2005_08165_amd import sne

from test_gpu_parity import ORACLE_KIND, check_parity, k32

pytestmark = pytest.mark.gpu

DTYPE = {"depth_f32": np.float32, "depth_u16": np.uint16, "depth_f16": np.float16,
         "disparity_f32": np.float32}


def _image(kind, values, H, W):
    """Runs of equal values of many lengths, so that windows with 0 to 8
    neighbours equal to their centre all occur."""
    rng = np.random.default_rng(9100 + values)
    img = rng.integers(2, 2 + values, size=(H, W))
    for _ in range(H * W // 24):
        v, u = rng.integers(0, H), rng.integers(0, W)
        img[v:v + rng.integers(1, 5), u:u + rng.integers(1, 5)] = rng.integers(2, 2 + values)
    return img.astype(DTYPE[kind])


def _kept(img):
    z = img.astype(np.float64)
    c = z[1:-1, 1:-1]
    return sum((z[1 + dv:z.shape[0] - 1 + dv, 1 + du:z.shape[1] - 1 + du] != c).astype(int)
               for dv in (-1, 0, 1) for du in (-1, 0, 1) if dv or du)


@pytest.mark.parametrize("agg", ["mean", "median"])
@pytest.mark.parametrize("kind", list(DTYPE))
def test_every_number_of_kept_candidates(kind, agg):
    K = (60.0, 60.0, 40.5, 30.25)
    for values in (2, 4, 9, 400):
        for H, W in ((61, 260), (12, 131)):
            img = _image(kind, values, H, W)
            if values == 4 and H == 61:
                assert set(np.unique(_kept(img))) == set(range(9))
            n, m = sne.estimate(torch.from_numpy(img).cuda(), K, kind, "fd", agg)
            on, om = oracle.estimate(img, ORACLE_KIND[kind], k32(K), "fd", agg)
            check_parity(n.double().cpu().numpy(), m.cpu().numpy(), on, om,
                         label="%s %s %d values %dx%d" % (kind, agg, values, H, W))


def _noisy(kind, H, W):
    """A slanted surface with noise and 25 % invalid samples of every sort."""
    rng = np.random.default_rng(9200)
    z = 1.5 + np.arange(W) / W + 0.4 * np.arange(H)[:, None] / H + 0.01 * rng.standard_normal((H, W))
    z = z * (1000.0 if kind == "depth_u16" else 20.0 if kind == "disparity_f32" else 1.0)
    z = z.astype(DTYPE[kind])
    bad = rng.random((H, W))
    z[bad < 0.25] = 0
    if kind != "depth_u16":
        for i, v in enumerate((np.nan, np.inf, -np.inf, -1.0, -0.0)):
            z[(bad >= 0.01 * i) & (bad < 0.01 * i + 0.01)] = v
    return z


@pytest.mark.parametrize("rule", ["strict", "lenient"])
@pytest.mark.parametrize("kind", list(DTYPE))
def test_validity_across_lane_and_tile_edges(kind, rule):
    """Holes on both sides of every boundary between lanes, half waves and
    tiles: each tile shape against the oracle."""
    H, W, K = 23, 516, (400.0, 400.0, 255.5, 12.0)
    img = _noisy(kind, H, W)
    dev = torch.from_numpy(img).cuda()
    ctx = sne.Context(0, tuning=False)
    suffix = "+lenient" if rule == "lenient" else ""
    # quantised depth: FD only (see above)
    second = "fd" if kind in ("depth_u16", "depth_f16") else "sobel"
    for grad, agg in (("fd", "mean"), (second, "median")):
        on, om = oracle.estimate(img, ORACLE_KIND[kind], k32(K), grad, agg, rule=rule)
        assert 0.01 < om.mean() < (0.95 if suffix else 0.2)
        for px, rows, lanes in ((1, 1, 64), (1, 5, 32), (2, 3, 64), (2, 4, 32), (4, 5, 64),
                                (4, 4, 32)):
            ctx.set_tile(px, rows, lanes)
            n, m = sne.estimate(dev, K, kind + suffix, grad, agg, ctx=ctx)
            check_parity(n.double().cpu().numpy(), m.cpu().numpy(), on, om,
                         label="%s %s-%s tile %dx%d/%d" % (kind + suffix, grad, agg, px, rows, lanes))


@pytest.mark.parametrize("out", ["f32", "f16"])
@pytest.mark.parametrize("kind", ["depth_f32+lenient"] + list(DTYPE))
def test_any_width_and_alignment_bitwise(kind, out):
    """Widths that cut the last lane's vector, rows and buffers that start at
    any element: 2 and 4 columns per lane equal 1 column per lane bit for bit,
    and nothing outside the frame's own elements is written."""
    base = kind.partition("+")[0]
    H, K = 9, (400.0, 400.0, 255.5, 4.0)
    dt = sne.OUT_DTYPE[sne.OUT[out]]
    ctx = sne.Context(0, tuning=False)
    for W, pad, skew in ((1, 0, 0), (2, 0, 1), (3, 2, 1), (5, 0, 3), (127, 0, 1), (257, 3, 0),
                         (258, 0, 1), (259, 1, 2), (516, 1, 1)):
        img = torch.from_numpy(_noisy(base, H, W)).cuda()
        pitch = W + pad
        store = torch.zeros(H * pitch + 8, dtype=img.dtype, device="cuda")
        raw = store[skew:skew + H * pitch].view(H, pitch)[:, :W]
        raw.copy_(img)
        ref = None
        for px, rows, lanes in ((1, 3, 64), (2, 2, 64), (2, 3, 32), (4, 4, 64), (4, 2, 32)):
            ctx.set_tile(px, rows, lanes)
            nbuf = torch.full((3 * H * pitch + 16,), 7.0, dtype=dt, device="cuda")
            mbuf = torch.full((H * pitch + 16,), 9, dtype=torch.uint8, device="cuda")
            n = nbuf[skew:skew + 3 * H * pitch].view(3, H, pitch)
            m = mbuf[skew:skew + H * pitch].view(H, pitch)
            for t in (n, m):  # what the call has to write
                t[..., :W] = 1
            sne.estimate(raw, K, kind, "fd", "median", out, normals=n[..., :W], mask=m[:, :W],
                         ctx=ctx)
            got = (nbuf.cpu().view(torch.int32 if out == "f32" else torch.int16), mbuf.cpu())
            if ref is None:
                ref = got
                on, om = oracle.estimate(img.cpu().numpy(), ORACLE_KIND[base], k32(K), "fd",
                                         "median", rule="lenient" if "+" in kind else "strict")
                check_parity(n[..., :W].double().cpu().numpy(), m[:, :W].cpu().numpy(), on, om,
                             out, "%s W=%d" % (kind, W))
                assert (n[..., W:] == 7).all() and (m[:, W:] == 9).all()
            for a, b in zip(ref, got):
                assert torch.equal(a, b), (kind, out, W, pad, skew, px, rows, lanes)


@pytest.mark.parametrize("agg", ["mean", "median"])
@pytest.mark.parametrize("kind,scale,offset", [("depth_u16", 1, 0), ("depth_u16", 1, 65500),
                                               ("depth_u16", 6000, 0), ("depth_f16", 2.0 ** -24, 0),
                                               ("depth_f16", 2.0 ** -12, 0), ("depth_f16", 4096, 0)])
def test_kept_candidates_at_the_ends_of_the_range(kind, scale, offset, agg):
    """Neighbours that differ by the type's smallest step, near its smallest
    and its largest values, and by most of its range: equal ones, and no
    others, are left out."""
    K = (60.0, 60.0, 40.5, 30.25)
    small = _image("depth_u16", 9, 37, 131).astype(np.float64)
    img = (small * scale + offset).astype(DTYPE[kind])
    assert (img.astype(np.float64) == small * scale + offset).all()  # exact
    for out in ("f32", "f16"):
        n, m = sne.estimate(torch.from_numpy(img).cuda(), K, kind, "fd", agg, out)
        on, om = oracle.estimate(img, ORACLE_KIND[kind], k32(K), "fd", agg)
        check_parity(n.double().cpu().numpy(), m.cpu().numpy(), on, om, out,
                     label="%s x %g + %g %s %s" % (kind, scale, offset, agg, out))


@pytest.mark.parametrize("kind", ["depth_f32", "disparity_f32"])
def test_single_ties_at_every_column_fp32(kind):
    """Single equal neighbours, in each of the 8 directions and at every column
    of a tile, in an image without other ties."""
    H, W, K = 57, 262, (60.0, 60.0, 130.5, 28.25)
    rng = np.random.default_rng(9300)
    scale = 2.0 if kind == "depth_f32" else 40.0
    base = rng.permutation(H * W).reshape(H, W)  # all distinct
    img = (scale * (1.0 + base / (H * W))).astype(np.float32)
    dirs = [(dv, du) for dv in (-1, 0, 1) for du in (-1, 0, 1) if dv or du]
    for v in range(2, H - 2, 4):
        for u in range(1 + v % 5, W - 1, 5):
            dv, du = dirs[(v // 4 + u) % 8]
            img[v + dv, u + du] = img[v, u]
    for out in ("f32", "f16"):
        n, m = sne.estimate(torch.from_numpy(img).cuda(), K, kind, "fd", "mean", out)
        on, om = oracle.estimate(img, ORACLE_KIND[kind], k32(K), "fd", "mean")
        check_parity(n.double().cpu().numpy(), m.cpu().numpy(), on, om, out,
                     label="%s %s" % (kind, out))


@pytest.mark.parametrize("out", ["f32", "f16"])
@pytest.mark.parametrize("kind", ["depth_f32+lenient", "depth_u16+lenient"] + list(DTYPE))
def test_any_width_and_alignment_bitwise_mean(kind, out):
    """As test_any_width_and_alignment_bitwise, for the means, which count
    their candidates in other ways than the medians."""
    base = kind.partition("+")[0]
    H, K = 9, (400.0, 400.0, 255.5, 4.0)
    dt = sne.OUT_DTYPE[sne.OUT[out]]
    ctx = sne.Context(0, tuning=False)
    for W, pad, skew in ((1, 0, 0), (3, 2, 1), (5, 0, 3), (127, 0, 1), (257, 3, 0), (258, 0, 1),
                         (259, 1, 2)):
        img = torch.from_numpy(_noisy(base, H, W)).cuda()
        pitch = W + pad
        store = torch.zeros(H * pitch + 8, dtype=img.dtype, device="cuda")
        raw = store[skew:skew + H * pitch].view(H, pitch)[:, :W]
        raw.copy_(img)
        ref = None
        for px, rows, lanes in ((1, 3, 64), (2, 2, 64), (2, 3, 32), (4, 4, 64), (4, 2, 32)):
            ctx.set_tile(px, rows, lanes)
            nbuf = torch.full((3 * H * pitch + 16,), 7.0, dtype=dt, device="cuda")
            mbuf = torch.full((H * pitch + 16,), 9, dtype=torch.uint8, device="cuda")
            n = nbuf[skew:skew + 3 * H * pitch].view(3, H, pitch)
            m = mbuf[skew:skew + H * pitch].view(H, pitch)
            sne.estimate(raw, K, kind, "fd", "mean", out, normals=n[..., :W], mask=m[:, :W],
                         ctx=ctx)
            got = (nbuf.cpu().view(torch.int32 if out == "f32" else torch.int16), mbuf.cpu())
            if ref is None:
                ref = got
                on, om = oracle.estimate(img.cpu().numpy(), ORACLE_KIND[base], k32(K), "fd",
                                         "mean", rule="lenient" if "+" in kind else "strict")
                check_parity(n[..., :W].double().cpu().numpy(), m[:, :W].cpu().numpy(), on, om,
                             out, "%s mean W=%d" % (kind, W))
                assert (n[..., W:] == 7).all() and (m[:, W:] == 9).all()
            for a, b in zip(ref, got):
                assert torch.equal(a, b), (kind, out, W, pad, skew, px, rows, lanes)
